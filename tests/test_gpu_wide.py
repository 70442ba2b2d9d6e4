"""The all-columns decode form (batches of several tokens): every edge of its
chunks (64 columns), groups (16) and tiles against the oracle and the
per-column kernels, bit for bit on
inputs whose fp32 sums are exact in any order (weights k 2^-9 with |k| < 16,
activations j / 4 with |j| <= 8: every partial sum is a multiple of 2^-11 below
2^11 at these widths, so it has at most 22 bits)."""

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


def _weights(rows, cols, sw, seed):
    rng = np.random.default_rng(seed)
    k = rng.integers(1, 16, (rows, cols)) * rng.choice([-1, 1], (rows, cols))
    w = (k * 2.0 ** -9).astype(np.float16)
    w[rng.random((rows, cols)) < sw] = 0
    return w


def _tokens(batch, cols, seed):
    rng = np.random.default_rng(seed)
    return (rng.integers(1, 9, (batch, cols)) * rng.choice([-1, 1], (batch, cols)) * 0.25).astype(np.float16)


def _expected(w, x, t, mask):
    y64, _, _ = oracle.spmspv(w, x, t, mask)
    return (y64 + 0.0).astype(np.float16).view(np.uint16)


def _run(m, x, t, mask):
    X = _to_dev(x)
    Y = torch.full((x.shape[0], m.rows), float("nan"), dtype=torch.float16, device=X.device)
    for _ in range(2):  # the second call meets the first one's partials
        m.spmspv_into(X, t, Y, mask=mask)
    torch.cuda.synchronize()
    return Y.cpu().numpy().view(np.uint16)


CASES = [
    # rows, cols, tile_k, weight sparsity, batch, splits (None: the rule's)
    (1, 1, 16, 0.0, 2, None),
    (64, 16, 16, 0.5, 5, None),
    (256, 64, 16, 0.0, 8, None),          # one dense chunk: the largest value slot
    (300, 63, 16, 0.5, 9, None),          # elements: rows of X that are not 16-byte aligned
    (257, 65, 32, 0.3, 16, None),
    (255, 72, 64, 0.5, 17, None),         # half a group past a chunk
    (513, 200, 256, 0.6, 32, None),       # tile_k wider than a chunk
    (600, 1000, 16, 0.5, 4, "64"),
    (600, 1000, 16, 0.5, 24, "3"),
    (320, 2056, 128, 0.02, 31, "2"),      # almost dense, several chunks per segment
    (1030, 3333, 16, 0.7, 12, None),
]


@pytest.mark.parametrize("mask", ["token", "batch"])
@pytest.mark.parametrize("rows,cols,tk,sw,batch,splits", CASES)
def test_every_row_exact(monkeypatch, rows, cols, tk, sw, batch, splits, mask):
    monkeypatch.setenv("SPDP_WIDE", "2")
    if splits:
        monkeypatch.setenv("SPDP_SPLITK", splits)
    w, x = _weights(rows, cols, sw, rows + cols), _tokens(batch, cols, cols + batch)
    x[0, :: 7] = np.float16("nan")  # never active; with one mask it drops the column
    m = spdp.encode(w, (256, tk))
    for t in (-1.0, 0.9, 1e9):
        t = t * (0.8 if mask == "batch" else 1.0)
        print(f"[gpu-wide] {rows}x{cols} tile_k={tk} sw={sw} B={batch} {mask} t={t} splits={splits}", flush=True)
        xt = x if t >= 0 else np.nan_to_num(x)
        expect = _expected(w, xt, t, mask)
        for form in ("2", "0"):  # all columns, and the per-column kernels
            monkeypatch.setenv("SPDP_WIDE", form)
            assert np.array_equal(_run(m, xt, t, mask), expect), form
    m.close()


def test_all_zero_weights_and_empty_chunks(monkeypatch):
    monkeypatch.setenv("SPDP_WIDE", "2")
    w = np.zeros((300, 400), np.float16)
    x = _tokens(6, 400, 1)
    m = spdp.encode(w, (256, 16))
    assert not _run(m, x, -1.0, "token").any()
    m.close()
    w[299, 399] = 0.5  # every chunk but the last one of the last stripe is empty
    m = spdp.encode(w, (256, 16))
    assert np.array_equal(_run(m, x, -1.0, "token"), _expected(w, x, -1.0, "token"))
    m.close()


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_weights_that_are_not_finite_skip_inactive_columns(bad):
    # a column that no token has active is not multiplied, whatever it holds
    w, x = _weights(256, 128, 0.5, 3), _tokens(16, 128, 4)
    w[17, 40] = bad
    x[:, 40] = 0
    m = spdp.encode(w, (256, 16))
    got = _run(m, x, 0.1, "token")
    w0 = w.copy()
    w0[17, 40] = 0
    assert np.array_equal(got, _expected(w0, x, 0.1, "token"))
    m.close()


def test_grouped_with_products_of_the_per_column_form():
    # tile_k 8 has no records: one call launches both forms, and every product
    # keeps the bits of its own call
    shapes = [((256, 16), 700, 500), ((256, 8), 300, 500), ((256, 32), 256, 500)]
    x = _tokens(8, 500, 7)
    X = _to_dev(x)
    ws = [_weights(r, c, 0.5, 10 + i) for i, (_, r, c) in enumerate(shapes)]
    ms = [spdp.encode(w, tile) for w, (tile, _, _) in zip(ws, shapes)]
    ys = [torch.full((8, w.shape[0]), float("nan"), dtype=torch.float16, device="cuda") for w in ws]
    for mask in ("token", "batch"):
        for _ in range(2):
            spdp.spmspv_many(ms, [X] * 3, [0.6] * 3, ys, mask=mask)
        torch.cuda.synchronize()
        for w, m, y in zip(ws, ms, ys):
            got = y.cpu().numpy().view(np.uint16)
            assert np.array_equal(got, _expected(w, x, 0.6, mask))
            assert np.array_equal(got, _run(m, x, 0.6, mask))
    for m in ms:
        m.close()


def test_noalloc_gives_the_same_bits_and_follows_smaller_calls():
    ms, ws = [], []
    for i, (r, c) in enumerate([(1024, 1200), (300, 2000), (256, 100)]):
        ws.append(_weights(r, c, 0.5, 30 + i))
        ms.append(spdp.encode(ws[-1], (256, 16)))
    for batch in (32, 5, 1, 17):  # the forms share the static workspace and its epoch
        for w, m in zip(ws, ms):
            x = _tokens(batch, w.shape[1], batch)
            X = _to_dev(x)
            Y = torch.full((batch, m.rows), float("nan"), dtype=torch.float16, device="cuda")
            m.spmspv_noalloc_into(X, 0.6, Y)
            torch.cuda.synchronize()
            got = Y.cpu().numpy().view(np.uint16)
            assert np.array_equal(got, _expected(w, x, 0.6, "token"))
            assert np.array_equal(got, _run(m, x, 0.6, "token"))
    for m in ms:
        m.close()


def _cancelling(rows, cols, batch, active, seed):
    """Weights and tokens whose exact products are 0 (column j + cols / 2
    takes back column j), so that the outputs are nothing but the rounding of
    the summation order: they tell which form ran. Column j is active (for one
    of the tokens) where ``active`` holds for j mod (cols / 2)."""
    rng = np.random.default_rng(seed)
    half = cols // 2
    w = (rng.standard_normal((rows, half)) * (rng.random((rows, half)) < 0.6)).astype(np.float16)
    x = (100.0 * rng.standard_normal((batch, half))).astype(np.float16)
    x[np.abs(x) < 1.0] = 1.5
    one = rng.integers(0, batch, half)
    low = np.arange(batch)[:, None] != one[None, :]  # inactive but for one token a column
    low |= ~active[:half][None, :]
    x[low] = 0.5
    w = np.concatenate([w, -w, np.zeros((rows, cols - 2 * half), np.float16)], 1)
    x = np.concatenate([x, x, np.zeros((batch, cols - 2 * half), np.float16)], 1)
    return w, x


def _sample(cols):
    """The sampled columns: the middle chunks of the width's quarters."""
    chunks = -(-cols // 64)
    firsts = [64 * ((2 * j + 1) * chunks // 8) for j in range(4)]
    return np.concatenate([np.arange(f, min(f + 64, cols)) for f in firsts])


@pytest.mark.parametrize("rows,cols,tile_k,batch", [
    (300, 4096, 16, 5), (300, 4096, 16, 8), (700, 3000, 32, 9), (257, 2056, 128, 16),
    (300, 4095, 16, 8), (300, 1001, 16, 17), (520, 6400, 16, 32),
])
@pytest.mark.parametrize("call", ["spmspv", "noalloc", "many"])
def test_gated_calls_pick_their_form_from_the_activations(rows, cols, tile_k, batch, call, monkeypatch):
    # all columns active, none, and one column of the sample more and less
    # than the share that the rule asks for (0.6, 0.5, 0.3 by batch)
    share = 0.6 if batch <= 8 else 0.5 if batch <= 16 else 0.3
    sample = _sample(cols)
    need = int(np.ceil(np.float32(share) * np.float32(len(sample))))
    half = cols // 2
    in_sample = np.zeros(half, int)  # how many sampled columns column j mod half stands for
    for k in sample:
        if k < 2 * half:
            in_sample[k % half] += 1
    rng = np.random.default_rng(batch)
    order = rng.permutation(np.nonzero(in_sample)[0])
    taken = np.cumsum(in_sample[order])
    cases = {"all": (np.ones(half, bool), True), "none": (np.zeros(half, bool), False)}
    for name, n in (("above", int(np.searchsorted(taken, need)) + 1), ("below", int(np.searchsorted(taken, need)))):
        on = np.zeros(half, bool)
        on[order[:n]] = True
        others = in_sample == 0
        on[others] = rng.random(int(others.sum())) < 0.5  # not looked at
        cases[name] = (on, name == "above")
    if need > taken[-1]:
        cases.pop("above")
    for name, (on, expect_all) in cases.items():
        w, x = _cancelling(rows, cols, batch, on, 7 + batch)
        m = spdp.encode(w, (256, tile_k))
        other = spdp.encode(w[: min(rows, 64)], (256, tile_k)) if call == "many" else None
        X = _to_dev(x)
        Y = torch.empty((batch, rows), dtype=torch.float16, device=X.device)
        Z = torch.empty((batch, min(rows, 64)), dtype=torch.float16, device=X.device)

        def product(wide):
            monkeypatch.setenv("SPDP_WIDE", wide)
            out = []
            for _ in range(2):
                Y.fill_(float("nan"))
                if call == "noalloc":
                    m.spmspv_noalloc_into(X, 1.0, Y)
                elif call == "many":
                    spdp.spmspv_many([other, m], [X, X], [1.0, 1.0], [Z, Y])
                else:
                    m.spmspv_into(X, 1.0, Y)
                out.append(Y.cpu().numpy().view(np.uint16))
            assert np.array_equal(out[0], out[1])
            return out[0]

        gated, columns, every = product("-5"), product("0"), product("5")
        if name != "none":
            assert not np.array_equal(columns, every), name  # the inputs tell the forms apart
        assert np.array_equal(gated, every if expect_all else columns), name
        # per-column sums of 100-sized terms: rounding only
        assert np.abs(gated.view(np.float16).astype(np.float64)).max() < 1.0, name
        m.close()
        if other is not None:
            other.close()


def test_a_captured_gated_call_follows_its_inputs(monkeypatch):
    # the gate is set and read inside the call: replays choose anew
    monkeypatch.setenv("SPDP_WIDE", "-5")
    rows, cols, batch = 512, 4096, 12
    inputs = []
    for seed, u in ((1, 1.0), (2, 0.05), (3, 1.0), (4, 0.0), (5, 0.3)):
        on = np.random.default_rng(seed).random(cols // 2) < u
        inputs.append(_cancelling(rows, cols, batch, on, 5)[1])
    w, _ = _cancelling(rows, cols, batch, np.ones(cols // 2, bool), 5)
    m = spdp.encode(w, (256, 16))
    m.reserve(batch)
    X = torch.empty((batch, cols), dtype=torch.float16, device="cuda:0")
    Y = torch.empty((batch, rows), dtype=torch.float16, device="cuda:0")
    want = []
    for x in inputs:
        X.copy_(_to_dev(x))
        m.spmspv_into(X, 1.0, Y)
        want.append(Y.clone())
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        m.spmspv_into(X, 1.0, Y)
    for _ in range(3):
        for x, y in zip(inputs, want):
            X.copy_(_to_dev(x))
            Y.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y.view(torch.int16), y.view(torch.int16))
    del g
    m.close()
