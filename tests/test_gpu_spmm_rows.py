"""The row form of the prefill product (few tokens): the edges of its token
tiles (32, 64), chunks (64 columns), groups (16) and GTiles against the oracle,
bit for bit on inputs whose fp32 sums are exact in any order (weights k 2^-9
with |k| < 16, tokens j / 4 with |j| <= 8: every partial sum is a multiple of
2^-11 below 2^11 at these widths, so it has at most 22 bits)."""

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2607_21985_amd as spdp  # noqa: E402


def _to_dev(a16):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU (torch.cuda.is_available() is False)")
    return torch.from_numpy(np.ascontiguousarray(a16).view(np.int16)).view(torch.float16).to("cuda:0")


def _inputs(rows, cols, n, sw, seed):
    rng = np.random.default_rng(seed)
    w = (rng.integers(1, 16, (rows, cols)) * rng.choice([-1, 1], (rows, cols)) * 2.0 ** -9).astype(np.float16)
    w[rng.random((rows, cols)) < sw] = 0
    x = (rng.integers(1, 9, (n, cols)) * rng.choice([-1, 1], (n, cols)) * 0.25).astype(np.float16)
    return w, x


CASES = [
    # rows, cols, tile_k, weight sparsity, tokens, splits (None: the rule's)
    (1, 1, 16, 0.0, 1, None),
    (256, 64, 16, 0.0, 32, None),        # one dense chunk: the largest value slot
    (300, 63, 16, 0.5, 33, None),        # rows of X that are not 16-byte aligned
    (257, 65, 32, 0.3, 64, None),
    (255, 72, 64, 0.5, 65, None),        # half a group past a chunk
    (513, 200, 256, 0.6, 31, None),      # tile_k wider than a chunk
    (600, 1000, 16, 0.5, 97, "3"),
    (333, 520, 16, 0.02, 128, "1000"),   # one chunk per split
    (1030, 3333, 128, 0.7, 40, None),
]


@pytest.mark.parametrize("form", ["0", "4", "5"], ids=["rule", "rows32", "rows64"])
@pytest.mark.parametrize("rows,cols,tk,sw,n,splits", CASES)
def test_exact(monkeypatch, rows, cols, tk, sw, n, splits, form):
    monkeypatch.setenv("SPDP_SPMM_FORM", form)
    if splits:
        monkeypatch.setenv("SPDP_SPMM_SPLITS", splits)
    w, x = _inputs(rows, cols, n, sw, rows + cols + n)
    m = spdp.encode(w, (256, tk))
    print(f"[gpu] spmm rows {rows}x{cols} tile_k={tk} sw={sw} N={n} form={form} splits={splits}", flush=True)
    X = _to_dev(x)
    Y = torch.full((n, rows), float("nan"), dtype=torch.float16, device=X.device)
    m.spmm_into(X, Y)
    torch.cuda.synchronize()
    y64, _, _ = oracle.spmm(w, x)
    assert np.array_equal(Y.cpu().numpy().view(np.uint16), (y64 + 0.0).astype(np.float16).view(np.uint16))
    m.close()


@pytest.mark.parametrize("form", ["2", "3", "4", "5"])
def test_a_neighbours_infinity_past_the_width_stays_out(monkeypatch, form):
    # 72 columns: the last chunk's pieces past the width would read the next
    # token's first columns
    monkeypatch.setenv("SPDP_SPMM_FORM", form)
    w, x = _inputs(256, 72, 70, 0.5, 5)
    bad = x.copy()
    bad[1::2, :] = np.float16(np.inf)
    m = spdp.encode(w, (256, 16))
    X = _to_dev(bad)
    Y = torch.empty((70, 256), dtype=torch.float16, device=X.device)
    m.spmm_into(X, Y)
    torch.cuda.synchronize()
    y64, _, _ = oracle.spmm(w, x)
    assert np.array_equal(Y.cpu().numpy()[::2].view(np.uint16), (y64 + 0.0)[::2].astype(np.float16).view(np.uint16))
    m.close()


def test_a_call_covers_the_captures_of_fewer_tokens():
    # the workspace that 128 tokens take holds what every smaller count takes,
    # whatever its splits, so none of them has to grow inside a capture
    w, x = _inputs(1024, 4096, 128, 0.5, 8)
    m = spdp.encode(w, (256, 16))
    X = _to_dev(x)
    Y = torch.empty((128, 1024), dtype=torch.float16, device=X.device)
    m.spmm_into(X, Y)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    for n in (1, 32, 33, 64, 65, 100):
        g = torch.cuda.CUDAGraph()
        y = torch.empty((n, 1024), dtype=torch.float16, device=X.device)
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=s):
            m.spmm_into(X[:n], y)
        for _ in range(3):
            y.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, Y[:n])
        del g
    m.close()


@pytest.mark.parametrize("rows,cols,tile_k,n", [(512, 4093, 16, 33), (300, 2048, 32, 7), (40960, 264, 16, 128)])
def test_a_first_call_inside_a_capture(rows, cols, tile_k, n):
    # products that no split warp-specialized form serves (odd widths, other
    # tile widths, more stripes than half the CUs) fold their ranges in the
    # kernel where the stream is capturing and there is no workspace
    w, x = _inputs(rows, cols, n, 0.5, 9)
    m = spdp.encode(w, (256, tile_k))
    X = _to_dev(x)
    y = torch.empty((n, rows), dtype=torch.float16, device=X.device)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        m.spmm_into(X, y)
    want = m.spmm(X)
    for _ in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)  # dyadic inputs: the sums are exact in any order
    del g
    m.close()


@pytest.mark.parametrize("rows,cols,tile_k,n", [
    (512, 4093, 16, 20),    # unaligned rows, 32 tokens a workgroup
    (512, 4093, 16, 64),    # unaligned, 64
    (300, 2048, 32, 7),     # aligned, 32, ragged rows
    (300, 4096, 32, 150),   # aligned, several token tiles
    (1000, 3000, 64, 64),
    (40960, 264, 16, 128),  # more stripes than half the CUs
])
def test_a_call_without_workspace_gives_the_bits_of_the_others(rows, cols, tile_k, n):
    # the first call inside a capture has no workspace to split into and folds
    # its ranges in the kernel: the same sums in the same order
    rng = np.random.default_rng(rows + n)
    w = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.5)).astype(np.float16)
    X = _to_dev(rng.standard_normal((n, cols)).astype(np.float16))
    m = spdp.encode(w, (256, tile_k))
    y = torch.empty((n, rows), dtype=torch.float16, device=X.device)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        m.spmm_into(X, y)
    m.spmm(X[: max(1, n // 2)])
    want = m.spmm(X)
    for _ in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))
    del g
    m.close()
