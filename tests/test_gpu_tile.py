"""The 512-row tile kernel at the edges of its tiles, of its six-chunk loop and of its epilogue's rank groups,
forward and backward, 96 and 128 columns wide, against the oracle. Every case asks the plan and the launched
kernels that it is this kernel that runs."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2608_24070_amd import slim, synth
from tests.gpu_common import assert_close, dev, dev_bits, host, kernels_of, layer_inputs
from tests.plans import plan

pytestmark = pytest.mark.gpu

# Activation rows that the plan gives 512 x 96 and 512 x 128 tiles on 1552 and 1664 weight rows (four row tiles, the
# last one of 16 and of 128 rows); both leave a ragged column tile
COLS = {96: 4101, 128: 7003}


def _sample(seed, total, count, last):
    return np.unique(np.concatenate([synth.stream(seed, "s").choice(total, size=min(count, total), replace=False),
                                     np.arange(max(0, total - last), total)]))


def _fwd(n, k, r, m, tc, xdtype="bf16", wide=None):
    print(f"tile fwd n={n} k={k} r={r} m={m} tc={tc} {xdtype}", flush=True)
    p = plan("fwd", m, n, k, r)
    assert not p.mid and not p.decode and p.sp_cols_tile == tc
    if wide is not None:
        assert p.ad_wide == wide
    W, X, L, R, dx, ad = layer_inputs(n, k, r, m, xdtype=xdtype, name="tile")
    pk = slim.pack(dev(W))
    out = []
    names = kernels_of(lambda: out.append(slim.linear(dx, pk, ad)))
    assert "tile_fwd" in names and not any(x.startswith(("mid_", "decode_")) for x in names), names
    rows, ms = _sample(1, n, 160, 40), _sample(2, m, 32, 12)
    ref = O.linear(X[ms], O.pack(W[rows]), L, None if R is None else R[:, rows], len(rows), k)
    assert_close(host(out[0])[np.ix_(ms, rows)], ref, f"tile fwd n={n} k={k} r={r} m={m}")
    assert torch.equal(out[0], slim.linear(dx, pk, ad))


def _bwd(n, k, r, m, tc, dydtype="bf16", groups=(0, 7, 12), wide=None):
    print(f"tile bwd n={n} k={k} r={r} m={m} tc={tc} {dydtype}", flush=True)
    p = plan("dx", m, n, k, r)
    assert not p.mid and not p.decode and p.sp_cols_tile == tc
    if wide is not None:
        assert p.ad_wide == wide
    W = synth.weights(n, k, seed=3, name="tile/W")
    yb, dY = synth.activations(m, n, seed=3, name="tile/dY", dtype=dydtype, scale=1e-3)
    Lb, Rb, L, R = synth.adapter(k, n, max(r, 16), seed=3, name="tile/")
    dy = dev_bits(yb, torch.bfloat16 if dydtype == "bf16" else torch.float16)
    dL = dev_bits(Lb[:, :r].copy(), torch.float16) if r else None
    dR = dev_bits(Rb[:r].copy(), torch.float16) if r else None
    pb = slim.pack_bwd(slim.pack(dev(W)))
    out = []
    names = kernels_of(lambda: out.append(slim.bwd_dx(dy, pb, dL, dR)))
    assert "tile_bwd" in names and not any(x.startswith(("mid_", "decode_")) for x in names), names
    ms = _sample(4, m, 24, 12)
    for g in groups:      # the backward pack is separable by 128-column group
        c = slice(128 * g, 128 * g + 128)
        ref = O.bwd_dx(dY[ms], O.pack_bwd(O.pack(W[:, c]), n, 128), L[c, :r] if r else None, R[:r] if r else None, n, 128)
        assert_close(host(out[0])[np.ix_(ms, np.arange(128 * g, 128 * g + 128))], ref, f"tile bwd group {g}")
    assert torch.equal(out[0], slim.bwd_dx(dy, pb, dL, dR))


# Chunk counts below, at and past one round of the six-chunk loop, every remainder among them; no adapter (fp16
# activations as given, and row-scaled bf16 ones) and a rank that ends inside a group of eight 16-rank steps
@pytest.mark.parametrize("tc", [96, 128])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11])
@pytest.mark.parametrize("r,dtype", [(0, "fp16"), (0, "bf16"), (48, "bf16")])
def test_forward_chunks(chunks, tc, r, dtype):
    _fwd(1552, 128 * chunks, r, COLS[tc], tc, dtype)


@pytest.mark.parametrize("tc", [96, 128])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11])
@pytest.mark.parametrize("r,dtype", [(0, "bf16"), (48, "fp16")])
def test_backward_chunks(chunks, tc, r, dtype):
    _bwd(128 * chunks, 1664, r, COLS[tc], tc, dtype)


# Three and four rank groups over two (128 wide) and three (96 wide) stages, the last whole, of one step, of seven
@pytest.mark.parametrize("tc", [96, 128])
@pytest.mark.parametrize("r", [272, 384, 496])
def test_rank_groups(tc, r):
    _fwd(1552, 640, r, COLS[tc], tc)
    _bwd(640, 1664, r, COLS[tc], tc, groups=(0, 12))


def test_whole_tiles():
    # rows and columns that fill whole 512 x 96 tiles: no ragged edge anywhere
    _fwd(2048, 1024, 64, 4608, 96)
    _bwd(1024, 2048, 64, 4608, 96)


@pytest.mark.parametrize("m,k", [(3900, 16512), (4096, 16384)])
def test_wide_adapter_gemm_splits(m, k):
    # T on the 256 x 256 adapter GEMM over eight reduction splits before the tiles: a ragged last m tile with a
    # shorter last split, and whole ones
    tc = plan("fwd", m, 1552, k, 512).sp_cols_tile
    _fwd(1552, k, 512, m, tc, wide=True)


def test_wide_adapter_gemm_splits_backward():
    tc = plan("dx", 3900, 16512, 1664, 512).sp_cols_tile
    _bwd(16512, 1664, 512, 3900, tc, groups=(0, 12), wide=True)
