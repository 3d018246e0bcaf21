"""PATCH hybrid dense / 2:4 tiles on the GPU (slim_pack_hybrid, slim_linear_hybrid) against the
oracle in oracle/patch_hybrid.py: bit-exact packs; products element by element within the fp32
summation bound. fp16 x fp16 products are exact in fp32, so the only error is the fp32 sum of K
terms: |Y - Y_exact| <= 2 K 2^-24 sum_k |x_k w_k| for any summation order."""
import numpy as np
import pytest
import torch

from oracle import patch_hybrid as P
from paper_2608_24070_amd import slim, synth
from tests.gpu_common import dev, host

pytestmark = pytest.mark.gpu


def _w(n, k, seed, tied=False):
    if tied:
        rng = synth.stream(seed, "ghyb/tied")
        lv = rng.integers(0, 4, size=(n, k)).astype(np.float32) * np.float32(0.5)
        w = lv * np.where(rng.random((n, k)) < 0.5, -1.0, 1.0).astype(np.float32)
        w[rng.random((n, k)) < 0.05] = -0.0
        return w
    return synth.weights(n, k, seed=seed, name="ghyb/W")


def _kinds(n, k, seed, frac):
    return (synth.stream(seed, "ghyb/kinds").random((n // 128, k // 128)) < frac).astype(np.uint8)


def _x(m, k, seed):
    return (synth.stream(seed, "ghyb/X").standard_normal((m, k)) * 1.0).astype(np.float16)


def _check_product(Y, X, Wp, rows=None):
    Xd = X.astype(np.float64)
    ref = Xd @ Wp.T
    bound = 2.0 * X.shape[1] * 2.0 ** -24 * (np.abs(Xd) @ np.abs(Wp).T) + 1e-30
    if rows is not None:
        Y = Y[rows]
    assert Y.shape == ref.shape
    assert np.all(np.abs(Y - ref) <= bound)


@pytest.mark.parametrize("n,k,frac,tied", [(128, 128, 1.0, False), (256, 512, 0.0, False), (384, 640, 0.6, True),
                                           (1024, 768, 0.7, False)])
def test_pack_bit_exact(n, k, frac, tied):
    print(f"hybrid pack n={n} k={k} frac={frac} tied={tied}", flush=True)
    W = _w(n, k, 1, tied)
    kinds = _kinds(n, k, 1, frac)
    p = slim.pack_hybrid(dev(W), kinds)
    ref = P.pack(W, kinds)
    assert np.array_equal(host(p["tile_info"]).view(np.uint64), ref["tile_info"])
    assert np.array_equal(host(p["payload"])[:ref["payload"].size], ref["payload"])


@pytest.mark.parametrize("m", [1, 16, 33, 128, 300])
@pytest.mark.parametrize("frac", [0.0, 0.7, 1.0])
def test_linear_parity(m, frac):
    n, k = 512, 1024
    print(f"hybrid linear m={m} frac={frac}", flush=True)
    W = _w(n, k, 2)
    kinds = _kinds(n, k, 2, frac)
    X = _x(m, k, 2)
    p = slim.pack_hybrid(dev(W), kinds)
    Y = host(slim.linear_hybrid(dev(X), p))
    _check_product(Y, X, P.hybrid_weight(W, kinds))


@pytest.mark.parametrize("n,k,m", [(384, 640, 40), (128, 256, 3), (640, 384, 200)])
def test_linear_odd_tile_rows(n, k, m):
    # N % 256 == 128: the last 256-row block holds one tile row (its second half lies past N)
    print(f"hybrid linear odd tile rows n={n} k={k} m={m}", flush=True)
    W = _w(n, k, 5)
    kinds = _kinds(n, k, 5, 0.5)
    X = _x(m, k, 5)
    p = slim.pack_hybrid(dev(W), kinds)
    Y = host(slim.linear_hybrid(dev(X), p))
    _check_product(Y, X, P.hybrid_weight(W, kinds))


# The kernel for few rows: each of its row counts' edges, its row-block shapes (up to 16 rows: N up to 4096, up to
# 12160, beyond; more: N times the halves of 32 rows up to 4096, beyond), an odd last row of tiles. 12288 x 640
# gives its eight waves at most one chunk; the next test goes past that.
@pytest.mark.parametrize("m", [1, 15, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("n,k,frac", [(128, 128, 0.5), (1152, 1152, 0.0), (4096, 2176, 0.7), (4224, 4224, 0.6),
                                      (12288, 640, 0.5)])
def test_linear_few_rows(n, k, m, frac):
    print(f"hybrid few n={n} k={k} m={m} frac={frac}", flush=True)
    W = _w(n, k, 6)
    kinds = _kinds(n, k, 6, frac)
    X = _x(m, k, 6)
    p = slim.pack_hybrid(dev(W), kinds)
    Y = host(slim.linear_hybrid(dev(X), p))
    _check_product(Y, X, P.hybrid_weight(W, kinds))


# The 32-row blocks with more chunks than waves: a second chunk for one wave, two for each, and the third and fourth
# of the pairs that are summed together.
@pytest.mark.parametrize("m", [1, 16, 17, 32])
@pytest.mark.parametrize("k", [1152, 2048, 3200])
def test_linear_few_rows_long_chains(k, m):
    n = 12288
    print(f"hybrid few n={n} k={k} m={m}", flush=True)
    W = _w(n, k, 8)
    kinds = _kinds(n, k, 8, 0.5)
    X = _x(m, k, 8)
    p = slim.pack_hybrid(dev(W), kinds)
    Y = host(slim.linear_hybrid(dev(X), p))
    cols = np.unique(np.concatenate([synth.stream(8, "cols").choice(n, size=512, replace=False), np.arange(n - 64, n)]))
    Wp = P.hybrid_weight(W.reshape(n // 128, 128, k)[np.unique(cols // 128)].reshape(-1, k), kinds[np.unique(cols // 128)])
    at = np.searchsorted(np.unique(cols // 128), cols // 128) * 128 + cols % 128
    _check_product(Y[:, cols], X, Wp[at])


def _split_chain_error(X, W, tiles):
    """Relative 2-norm error of X W^T where K is cut for about 512 blocks and every piece is one fp32 sum of exact
    8-term products, one after another (two to a matrix instruction: about its roundings), as are the pieces: the
    most accurate of the splits the GEMM considers, added up in the simplest order."""
    m, k = X.shape
    nch = k // 128
    s = min(nch, -(-512 // tiles)) if tiles < 256 else 1
    cps = -(-nch // s)
    steps = (X.astype(np.float64).reshape(m, 1, k // 8, 8) * W.astype(np.float64).reshape(1, -1, k // 8, 8)).sum(-1)
    total = np.zeros((m, W.shape[0]), dtype=np.float32)
    for c in range(0, k // 8, 16 * cps):
        acc = np.zeros_like(total)
        for t in range(c, min(c + 16 * cps, k // 8)):
            acc = (acc.astype(np.float64) + steps[:, :, t]).astype(np.float32)
        total = total + acc
    ref = X.astype(np.float64) @ W.astype(np.float64).T
    return float(np.linalg.norm(total - ref) / np.linalg.norm(ref))


# Long sums stay as accurate as K cut for 512 blocks: the kernel for few rows (both of its shapes for more than 16
# rows) and the GEMM. 1.15: the matrix instructions' own order of their terms, and the sample.
@pytest.mark.parametrize("m,n,k", [(32, 4224, 14336), (32, 2176, 14336), (64, 4096, 4096), (64, 2048, 4096), (16, 4224, 14336),
                                   (333, 5120, 5120), (100, 4096, 4096), (130, 1024, 8192), (500, 2048, 14336),
                                   (1332, 1024, 3584)])
def test_long_sums_stay_accurate(m, n, k):
    print(f"hybrid accuracy m={m} n={n} k={k}", flush=True)
    W = _w(n, k, 9)
    X = _x(m, k, 9)
    p = slim.pack_hybrid(dev(W), np.zeros((n // 128, k // 128), dtype=np.uint8))
    Y = host(slim.linear_hybrid(dev(X), p))
    rows = np.sort(synth.stream(9, "rows").choice(m, size=16, replace=False))
    cols = np.sort(synth.stream(9, "cols").choice(n, size=96, replace=False))
    Xs, Ws = X[rows], P.fp16_rne(W[cols])
    ref = Xs.astype(np.float64) @ Ws.astype(np.float64).T
    err = float(np.linalg.norm(Y[np.ix_(rows, cols)] - ref) / np.linalg.norm(ref))
    split = _split_chain_error(Xs, Ws, -(-n // 256) * -(-m // 128))
    print(f"error {err:.3e}, of the splits for 512 blocks {split:.3e}", flush=True)
    assert err <= 1.15 * split


# Split counts of the tile GEMM and its reduction: one, a few, and one per chunk; a shorter last split
@pytest.mark.parametrize("m,n,k", [(32, 512, 14336), (65, 256, 4224), (130, 4096, 4096), (1000, 2048, 1408), (2048, 4096, 256)])
def test_linear_splits(m, n, k):
    print(f"hybrid splits m={m} n={n} k={k}", flush=True)
    W = _w(n, k, 7)
    kinds = _kinds(n, k, 7, 0.6)
    X = _x(m, k, 7)
    p = slim.pack_hybrid(dev(W), kinds)
    Y = host(slim.linear_hybrid(dev(X), p))
    rows = np.arange(m) if m <= 130 else np.sort(synth.stream(7, "ghyb/rows").choice(m, size=64, replace=False))
    _check_product(Y, X[rows], P.hybrid_weight(W, kinds), rows=rows)


@pytest.mark.parametrize("m", [16, 2048])
def test_llama7b_gate_proj_full_size(m):
    # 11008 x 4096 at 35% sparsity (70% of the tiles 2:4), sampled rows of Y
    n, k = 11008, 4096
    print(f"hybrid full size m={m}", flush=True)
    W = _w(n, k, 3)
    kinds = _kinds(n, k, 3, 0.7)
    X = _x(m, k, 3)
    p = slim.pack_hybrid(dev(W), kinds)
    Y = host(slim.linear_hybrid(dev(X), p))
    rows = np.arange(m) if m <= 16 else np.sort(synth.stream(3, "ghyb/rows").choice(m, size=48, replace=False))
    _check_product(Y, X[rows], P.hybrid_weight(W, kinds), rows=rows)


def test_deterministic_and_errors():
    n, k, m = 256, 2048, 8                                    # small M: split reduction
    W = _w(n, k, 4)
    kinds = _kinds(n, k, 4, 0.5)
    p = slim.pack_hybrid(dev(W), kinds)
    X = dev(_x(m, k, 4))
    a, b = slim.linear_hybrid(X, p), slim.linear_hybrid(X, p)
    assert torch.equal(a, b)
    Wn = W.copy()
    Wn[7, 9] = np.nan
    with pytest.raises(slim.SlimError) as e:
        slim.pack_hybrid(dev(Wn), kinds)
    assert e.value.status == slim.SLIM_ENONFINITE
    with pytest.raises(slim.SlimError) as e:
        slim.slim_linear_hybrid_workspace(4, 256, 200)
    assert e.value.status == slim.SLIM_ESHAPE
