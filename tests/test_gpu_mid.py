"""The middle path (33 and more activation rows where 512-row tiles would be few): 128 x 64 and 256 x 128
sparse tiles over slices of the reduction, the adapter's first product in the same launch, and the finish
that sums the slices, at the edges of their tiles, slices and rank groups, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2608_24070_amd import slim, synth
from tests.gpu_common import assert_close, dev, dev_bits, host, layer_inputs

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
