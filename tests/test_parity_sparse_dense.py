"""GPU parity of structadmm_conv_sparse_fwd where its scratch also holds the
dense matrix: the matrix-core product and its guard against the gathers, which a
scratch without room for the dense matrix runs.

Bar: max|dY| / RMS(Y) <= 2e-2 between the two, as against the oracle (bf16
outputs: one rounding step of a value of 4 RMS is 1.6e-2); a value that is not
finite is the same on both sides; tiles and layers that the guard runs are
bitwise the gathers' results.
"""
import numpy as np
import pytest

import oracle
import paper_1807_11091_amd as sa
from gpu_helpers import DEV, bf16_bits_to_f64, maxabs_over_rms, to_dev, torch

pytestmark = pytest.mark.gpu

TOL = 2e-2


def gather_bytes(A, nnz):
    """Scratch of the gathers alone: row starts, offsets and values padded to 8 entries a row."""
    up = lambda x, m: (x + m - 1) // m * m
    cap = up(nnz + 7 * A, 8)
    return up((A + 1) * 4, 256) + up(cap * 4, 256) + up(cap * 2, 256)


def random_csr(rng, A, K, frac):
    keep = rng.random((A, K)) < frac
    keep[A // 2] = False  # a row without entries
    rows, col = np.nonzero(keep)
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=A))]).astype(np.int32)
    val = ((0.05 * rng.standard_normal(len(col))).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    return rp, col.astype(np.int32), val


class Case:
    def __init__(self, N, Cin, H, W, A, C, D, stride, pad, groups, frac, seed):
        t, rng = torch(), np.random.default_rng(seed)
        self.shape, self.geo = (A, Cin // groups, C, D), (groups, stride, pad)
        self.csr = random_csr(rng, A, Cin // groups * C * D, frac)
        self.nnz = len(self.csr[1])
        self.X = rng.standard_normal((N, Cin, H, W)).astype(np.float32)
        self.load()
        need = sa.conv_sparse_workspace(self.Xp, self.shape, *self.geo, self.nnz)
        self.small = gather_bytes(A, self.nnz)
        assert need > self.small, "the layer must be one that takes the dense product"
        self.ws = t.full((need,), 255, dtype=t.uint8, device=DEV)

    def load(self):
        self.Xp, self.dev = sa.pack_nhwc(to_dev(self.X)), [to_dev(x) for x in self.csr]

    def run(self, ws, reuse=False):
        Y = sa.conv_sparse_fwd(self.Xp, *self.dev, self.shape, *self.geo, self.nnz, ws=ws, reuse_ws=reuse)
        torch().cuda.synchronize()
        return Y.cpu().numpy()

    def gathers(self):
        return self.run(torch().full((self.small,), 255, dtype=torch().uint8, device=DEV))


LAYERS = [
    (64, 64, 28, 28, 64, 3, 3, 1, 1, 1, 0.3, 1),     # slices in one tap
    (300, 48, 14, 14, 140, 3, 3, 1, 1, 2, 0.5, 2),   # two groups of 24 channels and 70 filters
    (257, 40, 27, 27, 75, 3, 2, 2, 1, 1, 0.9, 3),    # odd channels out, stride 2, ragged tiles
    (128, 256, 28, 28, 264, 1, 1, 1, 0, 1, 0.5, 4),  # 1x1, filters past a tile's edge
]


@pytest.mark.parametrize("layer", LAYERS)
def test_dense_product_equals_gathers(layer):
    c = Case(*layer)
    got, ref = bf16_bits_to_f64(c.run(c.ws)), bf16_bits_to_f64(c.gathers())
    assert maxabs_over_rms(got, ref) <= TOL
    assert not np.any(got[..., layer[4] // 2])
    rc = dict(zip(("row_ptr", "col", "val"), c.csr))
    img = layer[0] - 1
    Yref = oracle.conv_csr(oracle.pack(c.X[img:]), rc, c.shape, *c.geo)
    assert maxabs_over_rms(got[img:], Yref) <= TOL


@pytest.mark.parametrize("layer", LAYERS[:3])
def test_infinities_and_nans_stay_with_the_kept_weights(layer):
    """A pruned weight has no term: an infinity or a NaN that only meets pruned
    weights must not reach the output."""
    c = Case(*layer)
    rng = np.random.default_rng(7)
    flat = c.X.reshape(-1)
    at = rng.integers(0, flat.size, 60)
    flat[at[:20]], flat[at[20:40]], flat[at[40:]] = np.inf, -np.inf, np.nan
    c.X[0] = np.nan
    c.load()
    got, ref = bf16_bits_to_f64(c.run(c.ws)), bf16_bits_to_f64(c.gathers())
    fin = np.isfinite(ref)
    assert np.array_equal(got[~fin], ref[~fin], equal_nan=True) and np.all(np.isfinite(got[fin]))
    assert np.count_nonzero(~fin) and maxabs_over_rms(got[fin], ref[fin]) <= TOL
    assert np.array_equal(got[0], ref[0], equal_nan=True)


def test_scratch_of_either_size_and_reuse():
    c = Case(*LAYERS[0])
    g, full = c.gathers(), c.run(c.ws)
    assert np.array_equal(c.run(c.ws, reuse=True), full)
    assert np.array_equal(c.run(c.ws[: c.small], reuse=True), g)  # entries of a full scratch
    ws = torch().full_like(c.ws, 255)
    c.run(ws[: c.small])
    assert np.array_equal(c.run(ws, reuse=True), g)  # no dense matrix in it: the gathers


@pytest.mark.parametrize("fault", ["twice", "descending", "past the row"])
def test_columns_out_of_order_run_the_gathers(fault):
    """Entries that structadmm_csr does not write keep their meaning: a column
    that comes twice counts twice, one past the row not at all."""
    c = Case(*LAYERS[1])
    rp, col, _ = c.csr
    a, b = rp[5], rp[6]
    assert b - a > 4
    if fault == "twice":
        col[a + 1] = col[a]
    elif fault == "descending":
        col[a:b] = col[a:b][::-1].copy()
    else:
        col[b - 1] = 1 << 24
    c.load()
    got, ref = c.run(c.ws), c.gathers()
    if fault == "past the row":
        assert maxabs_over_rms(bf16_bits_to_f64(got), bf16_bits_to_f64(ref)) <= TOL
    else:
        assert np.array_equal(got, ref)
