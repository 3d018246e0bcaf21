"""The middle path (33 and more activation rows where 512-row tiles would be few): 128 x 64 and 256 x 128
sparse tiles over slices of the reduction, the adapter's first product in the same launch, and the finish
that sums the slices, at the edges of their tiles, slices and rank groups, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2608_24070_amd import slim, synth
from tests.gpu_common import assert_close, dev, dev_bits, host, kernels_of, layer_inputs

pytestmark = pytest.mark.gpu


def _ws(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda")


def _counters_zero(ws):
    return int(ws[: 4096 * 4].view(torch.int32).abs().sum()) == 0


@pytest.mark.parametrize("n,k,r,m,xdtype", [
    (16, 128, 0, 33, "fp16"),        # one row block, one chunk, no partials
    (16, 128, 16, 64, "bf16"),       # one chunk with partials, one rank step
    (144, 640, 144, 65, "bf16"),     # a ragged row tile, five chunks in one slice, ranks past one unit
    (256, 1664, 48, 100, "fp16"),    # thirteen chunks over uneven slices
    (528, 2048, 272, 128, "bf16"),   # whole column tiles; ranks over three units
    (1040, 4096, 384, 129, "bf16"),  # one row past a column tile
    (4112, 1024, 528, 256, "bf16"),  # row tiles past a whole round; ranks past four passes of the finish
    (2048, 8192, 64, 333, "bf16"),   # many slices
    (8208, 1152, 0, 700, "fp16"),    # 256 x 128 tiles, no partials
    (8208, 1152, 160, 300, "bf16"),  # 256 x 128 tiles with the adapter
    (512, 512, 32, 3000, "bf16"),    # many column tiles
    (2048, 14336, 192, 2048, "bf16"),   # past the library's own scratch: 256 x 128 tiles, two slices, 105 MB
])
def test_forward_edges(n, k, r, m, xdtype):
    print(f"mid fwd n={n} k={k} r={r} m={m} {xdtype}", flush=True)
    W, X, L, R, dx, ad = layer_inputs(n, k, r, m, xdtype=xdtype, name="mid")
    p = slim.pack(dev(W))
    ws = _ws(slim.slim_linear_workspace(m, n, k, r))
    Y = slim.linear(dx, p, ad, ws=ws).clone()
    Y2 = slim.linear(dx, p, ad, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2), "runs differ"
    assert _counters_zero(ws)
    ms = np.unique(np.concatenate([np.arange(min(m, 3)), np.arange(m - 3, m),
                                   synth.stream(1, "m").choice(m, size=min(m, 40), replace=False)]))
    ref = O.linear(X[ms], O.pack(W), L, R, n, k)
    assert_close(host(Y)[ms], ref, f"mid fwd n={n} k={k} r={r} m={m}")


@pytest.mark.parametrize("n,k,r,m,xdtype", [
    (128, 128, 0, 33, "bf16"),
    (640, 128, 16, 65, "bf16"),
    (1664, 384, 144, 100, "fp16"),
    (4096, 1024, 272, 200, "bf16"),
    (1152, 8192, 0, 700, "bf16"),    # 256 x 128 tiles (whole scale groups per tile half), no partials
    (1152, 8192, 96, 300, "bf16"),
    (8192, 512, 32, 8192, "bf16"),   # past the library's own scratch: 256 x 128 tiles, two slices
])
def test_backward_edges(n, k, r, m, xdtype):
    print(f"mid bwd n={n} k={k} r={r} m={m} {xdtype}", flush=True)
    W = synth.weights(n, k, seed=2, name="midb/W")
    yb, dY = synth.activations(m, n, seed=2, name="midb/dY", dtype=xdtype, scale=1e-3)
    Lb, Rb, L, R = synth.adapter(k, n, max(r, 16), seed=2, name="midb/")
    pb = slim.pack_bwd(slim.pack(dev(W)))
    dy = dev_bits(yb, torch.bfloat16 if xdtype == "bf16" else torch.float16)
    dL = dev_bits(Lb[:, :r].copy(), torch.float16) if r else None
    dR = dev_bits(Rb[:r].copy(), torch.float16) if r else None
    ws = _ws(slim.slim_bwd_dx_workspace(m, n, k, r))
    dX = slim.bwd_dx(dy, pb, dL, dR, ws=ws).clone()
    dX2 = slim.bwd_dx(dy, pb, dL, dR, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(dX, dX2), "runs differ"
    assert _counters_zero(ws)
    ms = np.unique(np.concatenate([np.arange(3), np.arange(m - 3, m),
                                   synth.stream(2, "m").choice(m, size=min(m, 40), replace=False)]))
    ref = O.bwd_dx(dY[ms], O.pack_bwd(O.pack(W), n, k), L[:, :r] if r else None, R[:r] if r else None, n, k)
    assert_close(host(dX)[ms], ref, f"mid bwd n={n} k={k} r={r} m={m}")


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
    W, X, L, R, dx, ad = layer_inputs(n, k, r, m, name="tn")
    ws = _ws(slim.slim_linear_workspace(m, n, k, r))
    Y = host(slim.linear(dx, slim.pack(dev(W)), ad, ws=ws))
    assert _counters_zero(ws)
    rows = np.sort(synth.stream(3, "r").choice(n, size=300, replace=False))
    ms = np.unique(np.concatenate([np.arange(3), np.arange(m - 3, m), synth.stream(3, "m").choice(m, size=40, replace=False)]))
    ref = O.linear(X[ms], O.pack(W[rows]), L, R[:, rows], len(rows), k)
    assert_close(Y[np.ix_(ms, rows)], ref, f"tn n={n} k={k} r={r} m={m}")
