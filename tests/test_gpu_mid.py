"""The middle path (33 and more activation rows where 512-row tiles would be few): 128 x 64 and 256 x 128
sparse tiles over slices of the reduction, the adapter's first product in the same launch, and the finish
that sums the slices, at the edges of their tiles, slices and rank groups, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2608_24070_amd import slim, synth
from tests.gpu_common import assert_close, dev, dev_bits, host, kernels_of, layer_inputs
from tests.plans import plan

pytestmark = pytest.mark.gpu


def _ws(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda")


def _counters_zero(ws):
    return int(ws[: 4096 * 4].view(torch.int32).abs().sum()) == 0


def _check_plan(kind, n, k, r, m, tc, split, uneven):
    p = plan(kind, m, n, k, r)
    chunks = (n if kind == "dx" else k) // 128
    assert p.mid and p.sp_cols_tile == tc and p.sp_split == split, (p.mid, p.sp_cols_tile, p.sp_split)
    assert (p.sp_chunks_per_split * split != chunks) == uneven


# tc: 64 for 128 x 64 tiles, 128 for 256 x 128; reduction slices; whether the last slice is shorter
@pytest.mark.parametrize("n,k,r,m,xdtype,tc,split,uneven", [
    (16, 128, 0, 33, "fp16", 64, 1, False),        # one row block, one chunk, no partials
    (16, 128, 16, 64, "bf16", 64, 1, False),       # one chunk with partials, one rank step
    (144, 640, 144, 65, "bf16", 64, 1, False),     # a ragged row tile, five chunks, ranks past one unit
    (256, 1664, 48, 100, "fp16", 64, 1, False),    # thirteen chunks, past two rounds of the six-chunk loop
    (528, 2048, 272, 128, "bf16", 64, 1, False),   # whole column tiles; ranks over three units
    (1040, 4096, 384, 129, "bf16", 64, 2, False),  # one row past a column tile, two slices
    (4112, 1024, 528, 256, "bf16", 64, 1, False),  # row tiles past a whole round; ranks past four passes of the finish
    (2048, 8192, 64, 333, "bf16", 64, 2, False),   # two slices
    (8208, 1152, 0, 700, "fp16", 128, 1, False),   # no partials
    (8208, 1152, 160, 300, "bf16", 64, 1, False),  # nine chunks, many row tiles
    (512, 512, 32, 3000, "bf16", 64, 1, False),    # many column tiles
    (2048, 14336, 192, 2048, "bf16", 128, 2, False),   # past the library's own scratch: 105 MB
    # slices, the last one shorter, without and with an adapter
    (32, 1792, 0, 33, "bf16", 64, 3, True),
    (16, 6272, 0, 43, "fp16", 64, 7, False),
    (32, 4864, 0, 43, "bf16", 64, 8, True),
    (96, 2432, 208, 33, "bf16", 64, 2, True),
    (32, 4480, 528, 35, "fp16", 64, 3, True),
    (16, 10368, 384, 37, "bf16", 64, 5, True),
    (48, 14080, 208, 34, "bf16", 64, 7, True),
    # 256 x 128 tiles over slices, and with an adapter (its units 128 rows wide in the same launch)
    (3264, 4224, 0, 606, "bf16", 128, 3, False),
    (3632, 9344, 0, 323, "fp16", 128, 5, True),
    (4656, 640, 544, 855, "bf16", 128, 1, False),
    (5408, 2816, 464, 331, "bf16", 128, 2, False),
    (2512, 2944, 176, 789, "fp16", 128, 3, True),
    (2496, 8064, 576, 513, "bf16", 128, 5, True),
    (1616, 12160, 96, 585, "bf16", 128, 7, True),
])
def test_forward_edges(n, k, r, m, xdtype, tc, split, uneven):
    print(f"mid fwd n={n} k={k} r={r} m={m} {xdtype} tc={tc} split={split}", flush=True)
    _check_plan("fwd", n, k, r, m, tc, split, uneven)
    W, X, L, R, dx, ad = layer_inputs(n, k, r, m, xdtype=xdtype, name="mid")
    p = slim.pack(dev(W))
    ws = _ws(slim.slim_linear_workspace(m, n, k, r))
    out = []
    names = kernels_of(lambda: out.append(slim.linear(dx, p, ad, ws=ws)))
    assert "mid_fwd" in names, names
    Y = out[0].clone()
    Y2 = slim.linear(dx, p, ad, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2), "runs differ"
    assert _counters_zero(ws)
    ms = np.unique(np.concatenate([np.arange(min(m, 3)), np.arange(m - 3, m),
                                   synth.stream(1, "m").choice(m, size=min(m, 40), replace=False)]))
    rows = np.arange(n) if n * k < 1 << 22 else np.unique(np.concatenate(
        [synth.stream(1, "n").choice(n, size=512, replace=False), np.arange(n - 80, n)]))
    ref = O.linear(X[ms], O.pack(W[rows]), L, None if R is None else R[:, rows], len(rows), k)
    assert_close(host(Y)[np.ix_(ms, rows)], ref, f"mid fwd n={n} k={k} r={r} m={m}")


@pytest.mark.parametrize("n,k,r,m,xdtype,tc,split,uneven", [
    (128, 128, 0, 33, "bf16", 64, 1, False),
    (640, 128, 16, 65, "bf16", 64, 1, False),
    (1664, 384, 144, 100, "fp16", 64, 1, False),
    (4096, 1024, 272, 200, "bf16", 64, 2, False),
    (1152, 8192, 0, 700, "bf16", 128, 1, False),   # whole scale groups per tile half, no partials
    (1152, 8192, 96, 300, "bf16", 64, 1, False),
    (8192, 512, 32, 8192, "bf16", 128, 2, False),  # past the library's own scratch
    # slices, the last one shorter
    (1792, 256, 0, 40, "bf16", 64, 3, True),
    (2432, 128, 208, 33, "fp16", 64, 2, True),
    (4864, 128, 96, 70, "bf16", 64, 3, True),
    (6272, 128, 0, 43, "bf16", 64, 7, False),
    (10368, 128, 384, 37, "bf16", 64, 5, True),
    # 256 x 128 tiles over slices, and with an adapter
    (4480, 2432, 0, 845, "bf16", 128, 3, True),
    (12288, 1664, 0, 591, "fp16", 128, 7, True),
    (768, 4480, 560, 899, "bf16", 128, 1, False),
    (3456, 7296, 272, 258, "bf16", 128, 2, True),
    (3200, 3456, 80, 581, "fp16", 128, 3, True),
    (12160, 1664, 48, 582, "bf16", 128, 7, True),
])
def test_backward_edges(n, k, r, m, xdtype, tc, split, uneven):
    print(f"mid bwd n={n} k={k} r={r} m={m} {xdtype} tc={tc} split={split}", flush=True)
    _check_plan("dx", n, k, r, m, tc, split, uneven)
    W = synth.weights(n, k, seed=2, name="midb/W")
    yb, dY = synth.activations(m, n, seed=2, name="midb/dY", dtype=xdtype, scale=1e-3)
    Lb, Rb, L, R = synth.adapter(k, n, max(r, 16), seed=2, name="midb/")
    pb = slim.pack_bwd(slim.pack(dev(W)))
    dy = dev_bits(yb, torch.bfloat16 if xdtype == "bf16" else torch.float16)
    dL = dev_bits(Lb[:, :r].copy(), torch.float16) if r else None
    dR = dev_bits(Rb[:r].copy(), torch.float16) if r else None
    ws = _ws(slim.slim_bwd_dx_workspace(m, n, k, r))
    out = []
    names = kernels_of(lambda: out.append(slim.bwd_dx(dy, pb, dL, dR, ws=ws)))
    assert "mid_bwd" in names, names
    dX = out[0].clone()
    dX2 = slim.bwd_dx(dy, pb, dL, dR, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(dX, dX2), "runs differ"
    assert _counters_zero(ws)
    ms = np.unique(np.concatenate([np.arange(3), np.arange(m - 3, m),
                                   synth.stream(2, "m").choice(m, size=min(m, 40), replace=False)]))
    # the backward pack is separable by 128-column group
    for g in range(k // 128) if n * k < 1 << 22 else (0, k // 256, k // 128 - 1):
        c = slice(128 * g, 128 * g + 128)
        ref = O.bwd_dx(dY[ms], O.pack_bwd(O.pack(W[:, c]), n, 128), L[c, :r] if r else None, R[:r] if r else None, n, 128)
        assert_close(host(dX)[np.ix_(ms, np.arange(128 * g, 128 * g + 128))], ref, f"mid bwd n={n} k={k} r={r} m={m}")


def _least(call):
    """The smallest workspace (in steps of 256 bytes) that `call(nbytes)` is not refused with."""
    lo, hi = 0, 1 << 18
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (mid + 1, hi) if call(256 * mid) == slim.SLIM_EWORKSPACE else (lo, mid)
    return 256 * lo


A = 1 << 20      # an address that is only looked at, never used: the workspace beside it is misaligned


@pytest.mark.parametrize("n,k,r,m", [(528, 2048, 272, 128), (80, 640, 32, 100), (2048, 4096, 64, 333)])
@pytest.mark.parametrize("kind", ["fwd", "qa", "dx"])
def test_short_workspace_runs_the_512_row_tiles(kind, n, k, r, m):
    # a workspace too small for the middle path: the least one that is accepted, and guard bytes behind it
    if kind == "dx":
        n = (n + 127) // 128 * 128
    if kind == "qa":
        r = (r + 31) // 32 * 32
    print(f"short ws {kind} n={n} k={k} r={r} m={m}", flush=True)
    W, X, L, R, dx, ad = layer_inputs(n, k, r, m, name="short")
    p = slim.pack(dev(W))
    if kind == "fwd":
        full = slim.slim_linear_workspace(m, n, k, r)
        least = _least(lambda b: slim.slim_linear(A, 1, m, n, k, A, A, A, A, A, r, A, A + 4, b, None))
        run = lambda ws: slim.linear(dx, p, ad, ws=ws)
        ref = O.linear(X, O.pack(W), L, R, n, k)
    elif kind == "qa":
        full = slim.slim_linear_qa_workspace(m, n, k, r)
        least = _least(lambda b: slim.slim_linear_qa(A, 1, m, n, k, A, A, A, A, A, A, A, r, A, A + 4, b, None))
        q = slim.pack_adapter_q(ad["L"], ad["R"])
        run = lambda ws: slim.linear_qa(dx, p, q, ws=ws)
        ref = O.linear_qa(X, O.pack(W), O.pack_adapter_q(L, R), n, k, r)
    else:
        full = slim.slim_bwd_dx_workspace(m, n, k, r)
        least = _least(lambda b: slim.slim_linear_bwd_dx(A, 1, m, n, k, A, A, A, A, A, r, A, A + 4, b, None))
        yb, dY = synth.activations(m, n, seed=2, name="short/dY")
        dy, pb = dev_bits(yb, torch.bfloat16), slim.pack_bwd(p)
        run = lambda ws: slim.bwd_dx(dy, pb, ad["L"], ad["R"], ws=ws)
        ref = O.bwd_dx(dY, O.pack_bwd(O.pack(W), n, k), L, R, n, k)
    assert least < full
    buf = _ws(least + 4096)
    buf[least:] = 0x5A
    ws = buf[:least]
    names = kernels_of(lambda: run(ws))
    assert any(x.startswith("tile_") for x in names) and not any(x.startswith("mid_") for x in names), names
    assert any(x.startswith("mid_") for x in kernels_of(lambda: run(_ws(full))))
    Y = run(ws)
    assert_close(host(Y), ref, f"short ws {kind}")
    assert torch.equal(Y, run(ws).clone())
    assert _counters_zero(buf) and bool((buf[least:] == 0x5A).all())


@pytest.mark.parametrize("n,k,r,m", [(11008, 1024, 80, 1000), (4096, 1024, 400, 2048)])
def test_first_product_alone(n, k, r, m):
    # 512-row tiles behind the middle path's first-product units: a rank that ends inside a unit and inside
    # a 16-rank group of eight steps, a row count that ends inside a unit
    print(f"tn n={n} k={k} r={r} m={m}", flush=True)
    assert plan("fwd", m, n, k, r).ad_tn
    W, X, L, R, dx, ad = layer_inputs(n, k, r, m, name="tn")
    ws = _ws(slim.slim_linear_workspace(m, n, k, r))
    Y = host(slim.linear(dx, slim.pack(dev(W)), ad, ws=ws))
    assert _counters_zero(ws)
    rows = np.sort(synth.stream(3, "r").choice(n, size=300, replace=False))
    ms = np.unique(np.concatenate([np.arange(3), np.arange(m - 3, m), synth.stream(3, "m").choice(m, size=40, replace=False)]))
    ref = O.linear(X[ms], O.pack(W[rows]), L, R[:, rows], len(rows), k)
    assert_close(Y[np.ix_(ms, rows)], ref, f"tn n={n} k={k} r={r} m={m}")
