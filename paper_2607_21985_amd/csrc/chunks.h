// Chunks: the 64 columns that the kernels in which every column takes part
// stage between two barriers, and which 16-byte pieces (8 columns) of an X
// row their loads may touch. Plain constant expressions, the same in the
// kernels and on the host.
#pragma once

#include <cstdint>

namespace spdp_dev {

constexpr int kGroupCols = 16;                         // columns of a record: the MFMA's k
constexpr int kChunkGroups = 4;
constexpr int kChunkCols = kGroupCols * kChunkGroups;  // columns staged between two barriers

// The chunks of a stripe: those that hold a column of the matrix. Tiles wider
// than a chunk pad the width past them; padding columns have no values, and a
// chunk of nothing else would start past the end of X's rows.
constexpr int64_t chunk_count(int64_t cols) { return (cols + kChunkCols - 1) / kChunkCols; }

// How many pieces the load of piece `piece` of chunk `chunk` goes back where
// it starts past the width: to the chunk's first one, which lies inside
// (chunk_count; widths here are multiples of 8). What it brings is masked.
constexpr int pieces_back(int chunk, int piece, int cols) {
  return (chunk + 1) * kChunkCols > cols && chunk * kChunkCols + 8 * piece >= cols ? piece : 0;
}

// The sample of the activations by which a gated call picks its form: four
// chunks spread over the width (the middles of its quarters), every token.
constexpr int kSampleChunks = 4;
constexpr int sample_chunk(int j, int chunks) { return (int)((2 * (int64_t)j + 1) * chunks / (2 * kSampleChunks)); }
constexpr int sample_columns(int chunks, int cols) {
  int n = 0;
  for (int j = 0; j < kSampleChunks; ++j) {
    const int left = cols - sample_chunk(j, chunks) * kChunkCols;
    n += left < kChunkCols ? left : kChunkCols;
  }
  return n;
}

}  // namespace spdp_dev
