"""The library's host code with a stand-in HIP runtime: what it allocates and
launches (no GPU)."""

import os
import re
import shutil
import subprocess

import pytest

from fakehip import ROOT, fake_hip, run  # noqa: F401


CSRC = os.path.join(ROOT, "paper_2607_21985_amd", "csrc")


def test_word_records_end_with_the_width(fake_hip):
    # tiles wider than a chunk (64 columns) pad the width by whole chunks,
    # whose activations would be loaded from past the end of X: the records
    # (2560 bytes a chunk, three spare) cover the chunks that hold a column
    out = run(fake_hip, """
    for tk in (16, 64, 128, 256):
        for cols in (8, 64, 72, 1032, 1152, 2056, 4160):
            hip.fake_clear()
            m = ones(300, cols, (256, tk))
            sizes = [int(l[1]) for l in log() if l[0] == "malloc"]
            out[f"{tk} {cols}"] = (2 * -(-cols // 64) + 3) * 2560 in sizes
            m.close()
    """)
    assert out and all(out.values()), out


def test_activation_loads_stay_inside_the_row(tmp_path):
    # every 16-byte piece that the all-columns decode form loads, over every
    # width (multiples of 8) up to 1088 and every chunk of it
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "t.cpp"
    src.write_text("""
#include "chunks.h"
#include <cstdio>
using namespace spdp_dev;
int main() {
  long n = 0;
  for (int cols = 8; cols <= 1088; cols += 8) {
    int seen = 0;
    for (int c = 0; c < chunk_count(cols); ++c)
      for (int p = 0; p < 8; ++p, ++n) {
        const int k = c * kChunkCols + 8 * p, from = k - 8 * pieces_back(c, p, cols);
        if (from < 0 || from + 8 > cols || (k < cols && from != k)) return std::printf("%d %d %d\\n", cols, c, p), 1;
        seen += k < cols;
      }
    for (int j = 0; j < kSampleChunks; ++j) {
      const int c = sample_chunk(j, (int)chunk_count(cols));
      if (c < 0 || c >= chunk_count(cols)) return std::printf("%d: sample %d\\n", cols, j), 1;
    }
    if (sample_columns((int)chunk_count(cols), cols) < 1) return 1;
    if (seen != cols / 8) return std::printf("%d: %d pieces\\n", cols, seen), 1;
  }
  return std::printf("%ld\\n", n) < 0;
}
""")
    exe = str(tmp_path / "t")
    subprocess.run([gxx, "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


SPMM_SIZES = [(2048, 8192, 16), (4096, 4096, 16), (512, 4093, 16), (300, 2048, 32), (5003, 3080, 16), (1024, 32768, 16)]


@pytest.mark.parametrize("rows,cols,tile_k", SPMM_SIZES)
def test_a_splitting_prefill_call_covers_every_capture_of_fewer_tokens(fake_hip, rows, cols, tile_k):
    # sequences of calls, each growing the workspace or not, then a capture of
    # any smaller count; the splits are not monotone in the token count
    out = run(fake_hip, f"""
    rng = np.random.default_rng(1)
    refused = []
    split = 0
    sequences = [[128, 511], [32, 64], [16, 33, 200], [64, 333, 400]] + [
        sorted(int(v) for v in np.exp(rng.uniform(0, np.log(1500), 3))) for _ in range(4)]
    for seq in sequences:
        m = ones({rows}, {cols}, (256, {tile_k}), 0.05)
        for n in seq:
            log()
            assert spmm(m, n) == 0, (seq, n)
        if any(k.startswith("18spmm_reduce") or "spmm_reduce" in k for k, _ in launches()):
            split += 1
            hip.fake_capturing(1)
            for n in list(range(1, min(seq[-1], 300))) + list(range(300, seq[-1], 7)):
                if spmm(m, n) != 0:
                    refused.append([seq, n])
            hip.fake_capturing(0)
        m.close()
    out["refused"], out["split"] = refused[:5], split
    """)
    assert out["split"] > 0 and not out["refused"], out


def test_prefill_workspace_without_memory_for_more_than_the_call(fake_hip):
    # room for this call's partials only: the call runs, and asks again for
    # no more than it lacks
    out = run(fake_hip, """
    m = ones(2048, 8192, (256, 16), 0.05)
    log()
    assert spmm(m, 511) == 0
    grid = [g for k, g in launches() if "spmm_rows" in k or "spmm_ws" in k][0]
    m.close()
    m = ones(2048, 8192, (256, 16), 0.05)
    hip.fake_budget(hip.fake_used() + grid[2] * 511 * 2048 * 4)
    log()
    out["status"] = [spmm(m, 511) for _ in range(3)]
    entries = log()
    out["failed"] = sum(l[0] == "malloc-failed" for l in entries)
    out["mallocs"] = sum(l[0] == "malloc" for l in entries)
    out["error"] = L.spdp_last_error().decode()
    m.close()
    out["live"] = hip.fake_live()
    """)
    assert out == {"status": [0, 0, 0], "failed": 1, "mallocs": 1, "error": "", "live": 0}, out


def test_prefill_without_workspace_keeps_its_ranges(fake_hip):
    # inside a capture, and without memory, the row form walks the same ranges
    # in one workgroup per stripe and token tile; what needed a workspace
    # before that form existed is refused as it was
    out = run(fake_hip, """
    for rows, cols, tk, n in ((512, 4093, 16, 33), (300, 2048, 32, 7)):
        m = ones(rows, cols, (256, tk), 0.05)
        log()
        hip.fake_capturing(1)
        assert spmm(m, n) == 0
        a = launches()
        hip.fake_capturing(0)
        hip.fake_budget(hip.fake_used())
        assert spmm(m, n) == 0
        b = launches()
        hip.fake_budget((1 << 62))
        assert spmm(m, n) == 0
        c = launches()
        out[f"same {rows}"] = a == b and len(a) == 1 and len(c) == 2 and a[0][1][:2] == c[0][1][:2]
        out[f"split {rows}"] = a[0][1][2] == 1 and c[0][1][2] > 1
        m.close()
    # a call that succeeds leaves no message: folded, and unsplit where the
    # older rule would have split
    m = ones(512, 4093, (256, 16), 0.05)
    hip.fake_capturing(1)
    out["folded"] = spmm(m, 33) == 0 and L.spdp_last_error() == b""
    m = ones(4096, 4096, (256, 16), 0.05)
    out["unsplit"] = all(spmm(m, n) != 0 or L.spdp_last_error() == b"" for n in range(1, 2200, 13))
    out["refused"] = spmm(m, 64) == -1
    """)
    assert all(out.values()), out


@pytest.mark.slow
def test_prefill_forms_address_their_tile_of_x_with_32_bits(fake_hip):
    # 2^25 + 64 columns: the last token of a tile starts 2 (tokens - 1) cols
    # bytes behind the first; the forms of 64, 128 and 256 tokens would wrap
    out = run(fake_hip, """
    cols = (1 << 25) + 64
    w = np.zeros((1, cols), np.float16)
    w[0, :100] = 1
    m = spdp.encode(w, (256, 16))
    del w
    log()
    for n in (20, 32, 33, 64, 129, 300):
        assert spmm(m, n) == 0
        k = launches()[0][0]
        tile = 256 if "ws256" in k else 128 if "spmm_ws" in k else 64 if "ILi2E" in k else 32
        out[f"{n}"] = min(n, tile) * cols * 2 <= 1 << 32
    """)
    assert len(out) == 6 and all(out.values()), out


def test_encode_fits_where_the_handle_without_records_fits(fake_hip):
    # the records take memory last and only what is left: every budget from
    # the bare handle's on is enough, and its products run
    out = run(fake_hip, """
    log()
    before = hip.fake_used()
    m = ones(600, 2048, (256, 16), 0.3)
    total = hip.fake_used() - before
    records = 3 * (2048 // 64) * 2560 + 3 * 2560
    assert records in [int(l[1]) for l in log() if l[0] == "malloc"]
    m.close()
    bare = total - records - (3 * 32 + 1) * 4 - 256
    ok = []
    for extra in [0, 100, 3000] + list(range(4096, records + 4096, 8192)):
        hip.fake_budget(before + bare + extra)
        m = ones(600, 2048, (256, 16), 0.3)
        hip.fake_budget(1 << 62)
        log()
        ok.append(many([m], 8) == 0 and len(launches()) == 1)
        m.close()
    out["ok"], out["live"] = all(ok), hip.fake_live()
    """)
    assert out == {"ok": True, "live": 0}, out


def test_encode_without_host_memory_for_the_records(fake_hip):
    # the records' chunk offsets are the only host array of their size: the
    # handle comes without records, and no exception leaves the call
    out = run(fake_hip, """
    records = (3 * 32 + 3) * 2560
    for fail in (0, (3 * 32 + 1) * 4):
        log()
        hip.fake_fail_new(fail)
        m = ones(600, 2048, (256, 16), 0.3)
        hip.fake_fail_new(0)
        out[f"{fail}"] = records in [int(l[1]) for l in log() if l[0] == "malloc"]
        assert many([m], 8) == 0 and spmm(m, 64) == 0
        m.close()
    out["live"] = hip.fake_live()
    """)
    assert out == {"0": True, "388": False, "live": 0}, out


# what one product takes: "columns" (the per-column kernels), "wide" (the
# all-columns form) or both (gated)
ROUTES = [
    # rows, cols, tokens, route
    (2048, 2048, 4, ["columns"]), (2048, 2048, 5, ["wide"]), (2048, 2048, 8, ["wide"]), (2048, 2048, 32, ["wide"]),
    (20000, 1000, 8, ["columns"]), (20000, 1000, 9, ["wide"]),              # many short stripes
    (5120, 5120, 7, ["wide", "columns"]), (5120, 5120, 8, ["wide"]),
    (1024, 8192, 5, ["wide", "columns"]), (1024, 8192, 8, ["wide"]),         # k, beside a q of 8192 rows
    (600, 8700, 8, ["wide", "columns"]), (600, 8700, 17, ["wide"]),          # beside one of 8700
    (4096, 11008, 7, ["wide", "columns"]), (4096, 11008, 8, ["wide"]), (4096, 11008, 16, ["wide"]),
    (11008, 4096, 5, ["columns"]), (11008, 4096, 8, ["columns"]), (11008, 4096, 9, ["wide", "columns"]),
    (11008, 4096, 17, ["wide"]),
    (13824, 5120, 5, ["wide", "columns"]), (13824, 5120, 8, ["wide", "columns"]), (13824, 5120, 17, ["wide"]),
    (5120, 13824, 7, ["wide", "columns"]), (5120, 13824, 8, ["wide"]),
    (28672, 4000, 7, ["columns"]), (28672, 4000, 8, ["columns"]), (28672, 4000, 9, ["wide", "columns"]),
    (28672, 4000, 32, ["wide", "columns"]),
    (4000, 28672, 7, ["columns"]), (4000, 28672, 8, ["wide", "columns"]),
]


def test_routes(fake_hip):
    # the rule's lines, from both sides; with a negative threshold every
    # column takes part, and nothing is gated
    out = run(fake_hip, f"""
    mats = {{}}
    for rows, cols, tokens, _ in {ROUTES!r}:
        if (rows, cols) not in mats:
            mats = {{(rows, cols): ones(rows, cols, (256, 16), 0.002)}}
        m = mats[rows, cols]
        for t in (0.5, -1.0):
            log()
            assert many([m], tokens, 0, [t]) == 0
            out[f"{{rows}} {{cols}} {{tokens}} {{t}}"] = ["wide" if "wide" in n else "columns" for n, g in launches()]
    """)
    for rows, cols, tokens, want in ROUTES:
        assert out[f"{rows} {cols} {tokens} 0.5"] == want, (rows, cols, tokens, out[f"{rows} {cols} {tokens} 0.5"])
        assert len(out[f"{rows} {cols} {tokens} -1.0"]) == 1
        if len(want) == 2:
            assert out[f"{rows} {cols} {tokens} -1.0"] == ["wide"]


def test_launches_of_a_grouped_call(fake_hip):
    # q, k and v of the 70B layer: one launch where no product is gated (up
    # to 4 tokens, from 8 on, one mask for the batch), and never more than
    # two, the second only with products that the first is a gate for; every
    # column kept (a negative threshold): one
    out = run(fake_hip, """
    q = ones(8192, 8192, (256, 16), 0.02)
    k = ones(1024, 8192, (256, 16), 0.02, 1)
    v = ones(1024, 8192, (256, 16), 0.02, 2)
    for tokens in (1, 2, 4, 5, 8, 16, 32):
        for mask in (0, 1):
            for t in (0.5, -1.0):
                log()
                assert many([q, k, v], tokens, mask, [t] * 3) == 0
                out[f"{tokens} {mask} {t}"] = [("wide" if "wide" in n else "columns", g[1]) for n, g in launches()]
    """)
    for key, got in out.items():
        tokens, mask, t = key.split()
        if int(tokens) < 5 or mask == "1":
            want = [["columns", 3]]
        elif t == "-1.0" or int(tokens) >= 8:
            want = [["wide", 3]]
        else:
            want = [["wide", 3], ["columns", 3]]
        assert got == want, (key, got)


def test_a_call_that_cannot_be_launched_launches_nothing(fake_hip):
    # a gated product is two launches: what can fail is asked before the first
    out = run(fake_hip, """
    m = ones(300, 8800, (256, 16), 1.0)  # dense: more than 64 KB of LDS
    hip.fake_fail_attribute(1)
    log()
    out["status"] = many([m], 8)
    out["launches"] = len(launches())
    hip.fake_fail_attribute(0)
    out["after"] = many([m], 8)
    """)
    assert out == {"status": -4, "launches": 0, "after": 0}, out
