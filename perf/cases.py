"""Timed cases of the Tiled-CBC products, through the package's public calls.

A decoder uses the package in two ways. Each decode step multiplies the
layer's encoded matrices by one to 32 tokens whose small activations are
dropped (``Matrix.spmspv_into``, ``spmspv_many``, ``Matrix.spmspv_noalloc_into``,
or a layer's launches recorded in a ``Chain``); a prompt goes through the same
handles with every column taking part (``Matrix.spmm_into``). The listed cases
are those calls on the shapes of ``synth.WORKLOADS`` (Llama-7B, -13B and -70B
projections, the 1024 x 1024 layer) and on a ragged size.

A case is a dict of plain values:

* ``path``: "call" (one call per group), "noalloc", "chain" or "prefill";
* ``shapes``: the products, "ROWSxCOLS" each; products separated by blanks
  read one input and go out in one launch, "|" starts the next launch;
* ``tokens``, ``weight_sparsity``, ``act_sparsity`` (the quantile of |x| that
  the threshold drops), ``mask`` ("token" or "batch"), ``bits`` (16: fp16
  values, else round-to-nearest codes), ``tile_m``, ``tile_k``.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2607_21985_amd as spdp


def _case(name, path, shapes, tokens, weight_sparsity, act_sparsity=0.0, mask="token", bits=16, tile=(256, 16)):
    c = {"path": path, "shapes": shapes, "tokens": tokens, "weight_sparsity": weight_sparsity,
         "act_sparsity": act_sparsity, "mask": mask, "bits": bits, "tile_m": tile[0], "tile_k": tile[1]}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small layer, one token: the fixed cost of a call
        _case("decode 1024, 1 token", "call", "1024x1024", 1, 0.5, 0.5, tile=(64, 64)),
        # a 7B attention block's projections as a serving loop replays them
        _case("decode 7B attention, 1 token", "chain", "4096x4096 4096x4096 4096x4096|4096x4096", 1, 0.5, 0.5),
        # a 7B MLP with 4-bit values, one token
        _case("decode 7B MLP codes, 1 token", "chain", "11008x4096 11008x4096|4096x11008", 1, 0.6, 0.5, bits=4),
        # two tokens (speculative decoding, a pair of requests) from a loop
        # that may not allocate
        _case("decode 13B o, 2 tokens", "noalloc", "5120x5120", 2, 0.7, 0.5),
        # a whole 13B decoder layer's projections for eight requests
        _case("decode 13B layer, 8 tokens", "chain",
              "5120x5120 5120x5120 5120x5120|5120x5120|13824x5120 13824x5120|5120x13824", 8, 0.7, 0.5),
        # sixteen requests with one column set for the batch
        _case("decode 7B MLP, 16, shared", "chain", "11008x4096 11008x4096|4096x11008", 16, 0.6, 0.5, mask="batch"),
        # the largest grouped launch of one token, nothing dropped: bandwidth
        _case("decode 70B gate up, 1 token", "call", "28672x8192 28672x8192", 1, 0.5, 0.0),
        # the largest decode batch on the 70B MLP shapes
        _case("decode 70B MLP, 32 tokens", "chain", "28672x8192|8192x28672", 32, 0.7, 0.5),
        # a short prompt or a prefill chunk
        _case("prefill 7B q, 64 tokens", "prefill", "4096x4096", 64, 0.5),
        # an ordinary prompt
        _case("prefill 7B gate, 512 tokens", "prefill", "11008x4096", 512, 0.6),
        # ragged rows, a width that is no multiple of a GTile's, odd tokens
        _case("prefill 5003x3080, 333", "prefill", "5003x3080", 333, 0.5),
        # a long prompt on the largest projection
        _case("prefill 70B gate, 2048", "prefill", "28672x8192", 2048, 0.7),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same ranges: widths mostly multiples of 8 (hidden sizes
    are), some odd; rows and token counts of any value."""
    def rows_cols(cap):
        while True:
            r, c = _log_int(rng, 512, 28672), _log_int(rng, 512, 28672)
            if r * c <= cap:
                break
        if rng.random() < 0.5:
            r = (r + 127) // 128 * 128
        return r, (c + 7) // 8 * 8 if rng.random() < 0.9 else c

    sw = rng.choice([0.5, 0.6, 0.7, 0.8])
    p = rng.choice([0.0, 0.25, 0.5, 0.7])
    if rng.random() < 0.4:
        r, c = rows_cols(120_000_000)
        tokens = _log_int(rng, 16, 2048)
        return _case("", "prefill", f"{r}x{c}", tokens, sw, tile=(256, rng.choice([16, 16, 16, 32])))
    tile = rng.choice([(256, 16), (256, 16), (256, 16), (128, 32), (64, 64)])
    path = rng.choice(["call", "call", "chain", "noalloc"])
    tokens = _log_int(rng, 1, 32)
    mask = "batch" if path != "noalloc" and tokens > 1 and rng.random() < 0.3 else "token"
    bits = 4 if rng.random() < 0.15 else 16
    if path == "noalloc":
        # sizes whose partials the static workspace holds
        r, c = rows_cols(60_000_000)
        return _case("", path, f"{min(r, 4096)}x{c}", min(tokens, 16), sw, p, bits=bits, tile=tile)
    if path == "call":
        n = rng.choice([1, 1, 2, 3])
        r, c = rows_cols(200_000_000 // n)
        return _case("", path, " ".join([f"{r}x{c}"] * n), tokens, sw, p, mask, bits, tile)
    r, c = rows_cols(70_000_000)
    return _case("", path, f"{r}x{c} {r}x{c}|{c}x{r}", tokens, sw, p, mask, bits, tile)


def _groups(case):
    return [[tuple(int(v) for v in s.split("x")) for s in g.split()] for g in case["shapes"].split("|")]


def _weight(rows, cols, sparsity, gen):
    """N(0, 0.02) entries with a log-normal scale per input channel, the
    smallest magnitudes of the matrix pruned."""
    dev = "cuda"
    scale = torch.exp(0.5 * torch.randn(cols, device=dev, generator=gen))
    w = torch.empty((rows, cols), dtype=torch.float16, device=dev)
    step = max(1, (1 << 26) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        w[r:r + n] = (0.02 * torch.randn((n, cols), device=dev, generator=gen) * scale).half()
    mag = w.view(torch.int16) & 0x7FFF
    # the magnitude bits below which lies the share to prune
    count = torch.zeros(1 << 15, dtype=torch.int64, device=dev)
    for r in range(0, rows, step):
        count += torch.bincount(mag[r:r + step].reshape(-1).int(), minlength=1 << 15)
    cut = int(torch.searchsorted(torch.cumsum(count, 0), int(sparsity * rows * cols)))
    return w.masked_fill_(mag < cut, 0.0)


def _activations(tokens, cols, kind, gen):
    """Attention inputs: Laplace with 1 % outlier channels; the down
    projection's inputs: SiLU(g) u."""
    dev = "cuda"
    if kind == "swiglu":
        g = torch.randn((tokens, cols), device=dev, generator=gen)
        return (torch.nn.functional.silu(g) * torch.randn((tokens, cols), device=dev, generator=gen)).half()
    u = torch.rand((tokens, cols), device=dev, generator=gen) - 0.5
    x = -torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.4999999))
    outliers = torch.randperm(cols, device=dev, generator=gen)[: max(1, cols // 100)]
    x[:, outliers] *= 20.0
    return x.half()


def _threshold(x, case):
    """The threshold that drops the share ``act_sparsity`` of these inputs."""
    p = case["act_sparsity"]
    if p <= 0.0:
        return -1.0
    v = x.abs().float()
    if case["mask"] == "batch":
        v = v.mean(0)
    v = v.reshape(-1).sort().values
    return float(v[max(0, math.ceil(p * v.numel()) - 1)])


def _inputs(case, seed):
    """[(x, threshold, [weights])] of each launch, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * int(seed) + 17)
    out = []
    for i, group in enumerate(_groups(case)):
        kind = "swiglu" if i > 0 and group[0][1] > group[0][0] else "laplace"
        x = _activations(case["tokens"], group[0][1], kind, gen)
        t = _threshold(x, case) if case["path"] != "prefill" else -1.0
        out.append((x, t, [_weight(r, c, case["weight_sparsity"], gen) for r, c in group]))
    return out


def prepare(case, seed):
    """Encoded matrices with their workspaces sized, inputs and outputs on the
    GPU, and the recorded chain where the case replays one."""
    launches = []
    tile = (case["tile_m"], case["tile_k"])
    for x, t, ws in _inputs(case, seed):
        mats = []
        while ws:
            w = ws.pop(0).cpu().numpy()
            m = spdp.encode(w, tile) if case["bits"] == 16 else spdp.encode_rtn(w, tile, case["bits"])
            if case["path"] == "call":
                m.reserve(case["tokens"])
            mats.append(m)
        ys = [torch.empty((case["tokens"], m.rows), dtype=torch.float16, device="cuda") for m in mats]
        launches.append((mats, [x] * len(mats), [t] * len(mats), ys))
    state = {"path": case["path"], "mask": case["mask"], "launches": launches}
    if case["path"] == "chain":
        chain = spdp.Chain()
        for mats, xs, ts, ys in launches:
            chain.add(mats, xs, ts, ys, mask=case["mask"])
        state["chain"] = chain.capture()
    return state


def run(state):
    path = state["path"]
    if path == "chain":
        state["chain"].replay()
    else:
        for mats, xs, ts, ys in state["launches"]:
            if path == "prefill":
                for m, x, y in zip(mats, xs, ys):
                    m.spmm_into(x, y)
            elif path == "noalloc":
                for m, x, t, y in zip(mats, xs, ts, ys):
                    m.spmspv_noalloc_into(x, t, y)
            elif len(mats) == 1:
                mats[0].spmspv_into(xs[0], ts[0], ys[0], mask=state["mask"])
            else:
                spdp.spmspv_many(mats, xs, ts, ys, mask=state["mask"])
    return [y for _, _, _, ys in state["launches"] for y in ys]


def work(case):
    """Bytes: of every active column the bitmap and the nonzeros (2 bytes, or
    one byte a code), the inputs and the outputs; flops: two per nonzero and
    token that meet. A column is active for a batch with per-token masks if
    it is for any token."""
    n, p = case["tokens"], case["act_sparsity"] if case["path"] != "prefill" else 0.0
    cols_read = 1.0 - (p if case["mask"] == "batch" else p ** n)
    total = flops = 0.0
    for group in _groups(case):
        total += 2.0 * n * group[0][1]
        for r, c in group:
            nnz = (1.0 - case["weight_sparsity"]) * r * c
            total += cols_read * (r * c / 8.0 + nnz * (2.0 if case["bits"] == 16 else 1.0)) + 2.0 * n * r
            flops += 2.0 * nnz * n * (1.0 - p)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """The result is rounded to fp16 once: half a unit in the last place
    (2^-11 of the value at most, about 2e-4 in the 2-norm against 64 bits);
    four times that, and two units for the largest."""
    return {"rel": 8e-4, "max": 4e-3}


def _codes(w, bits):
    """Round-to-nearest codes and one scale per row, from their definition."""
    a = w.cpu().numpy().astype(np.float32)
    qmax = np.float32(2 ** (bits - 1) - 1)
    s = np.abs(a).max(axis=1) / qmax
    q = np.rint(np.divide(a, s[:, None], out=np.zeros_like(a), where=s[:, None] > 0))
    return torch.from_numpy(np.clip(q, -qmax, qmax)).cuda(), torch.from_numpy(s).cuda()


def exact(case, seed):
    out = []
    for x, t, ws in _inputs(case, seed):
        if case["path"] == "prefill":
            xm = x
        elif case["mask"] == "batch" and case["tokens"] > 1:
            score = torch.zeros(x.shape[1], dtype=torch.float32, device="cuda")
            for b in range(x.shape[0]):
                score += x[b].abs().float()
            limit = float(np.float32(float(np.float32(t)) * x.shape[0]))
            xm = x * (score > limit)
        else:
            xm = torch.where(x.abs().float() > t, x, torch.zeros_like(x))
        xd = xm.double()
        for w in ws:
            s = None
            if case["bits"] < 16:
                w, s = _codes(w, case["bits"])
            y = torch.empty((x.shape[0], w.shape[0]), dtype=torch.float64, device="cuda")
            step = max(1, (1 << 26) // w.shape[1])
            for r in range(0, w.shape[0], step):
                y[:, r:r + step] = xd @ w[r:r + step].double().t()
            out.append(y if s is None else y * s.double())
    return out
