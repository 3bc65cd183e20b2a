"""The initialisation's search over the photon list: pools around a chunk of 64
entries, around what its LDS holds in either launch and past it; scores of 32
and 64 bits; bins past the dense search's last, IRFs of 1 to 4000 bins; launches
whose average pool is below and above the line to the dense search, with pools
on both sides of it.  Counts and depths equal to the oracle's, the rest to the
rounding of the stored values."""
import numpy as np
import pytest

from gpu_util import device_to_oracle, to_dev_u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

GAUSS, TAIL = synth.gaussian_irf(1.5, 9), synth.exgauss_irf(3.0, 10.0, -18, 118)
WIDE, ONE = synth.gaussian_irf(300, 1000), synth.gaussian_irf(0.3, 0)


def pools(seed, T, irf, sizes, peak=12):
    """A pixel per size: that many entries, `peak` photons or more of them around a surface."""
    rng = np.random.default_rng(seed)
    Z = np.zeros((1, len(sizes), T), np.uint16)
    for j, n in enumerate(sizes):
        at = np.unique(np.clip(np.rint(0.1 * T + 0.8 * T * j / len(sizes) + irf.draw(rng, peak)), 0, T - 1).astype(int))[:n]
        free = rng.permutation(np.setdiff1d(np.arange(T), at))[:n - len(at)]
        Z[0, j, at] = rng.integers(1, 4, len(at))
        Z[0, j, free] = 1
    return Z


def photons(seed, rows, cols, T, irf, signal, bkg):
    rng = np.random.default_rng(seed)
    i, j = np.mgrid[0:rows, 0:cols].astype(np.float64)
    d = np.stack([0.02 * T + 0.9 * T * (j + 0.3 * i) / (cols + 0.3 * rows), np.full((rows, cols), 0.6 * T)])
    return synth.render(rng, irf, T, d, rng.uniform(0.7, 1.3, (2, rows, cols)) * signal, bkg / T)


SIZES = [0, 1, 2, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 4095, 4096, 4097, 5000]
CASES = {
    "sizes": lambda: (pools(1, 40000, GAUSS, SIZES), GAUSS, {}),
    "sizes_tail": lambda: (pools(2, 33000, TAIL, SIZES), TAIL, dict(k_init=4)),
    "sizes_nmin0": lambda: (pools(3, 33000, ONE, SIZES[:9]), ONE, dict(n_min=0, kappa=0.0)),
    "last_bins": lambda: (photons(4, 3, 7, 65535, GAUSS, 20.0, 30.0), GAUSS, dict(r_init=1, k_init=4)),
    "long_irf": lambda: (photons(5, 4, 6, 8100, synth.gaussian_irf(600, 2000), 30.0, 30.0), synth.gaussian_irf(600, 2000), {}),
    "bright": lambda: (photons(6, 5, 7, 33000, GAUSS, 60000.0, 20.0), GAUSS, dict(r_init=1)),
    "past16383": lambda: (photons(7, 6, 8, 300, GAUSS, 30000.0, 10.0), GAUSS, dict(r_init=2, k_init=4)),
    "weights_past_24_bits": lambda: (photons(8, 4, 6, 500, GAUSS, 9.0, 9.0), GAUSS, dict(sbr_guess=1e150, r_init=1)),
    "sparse_T8193": lambda: (photons(10, 9, 9, 8193, GAUSS, 1.5, 0.5), GAUSS, dict(r_init=1)),
    "dense_T8193": lambda: (photons(11, 9, 9, 8193, GAUSS, 8.0, 90.0), GAUSS, dict(r_init=1)),
    "both_sides": lambda: (pools(12, 20000, TAIL, [5, 40, 250, 300, 500, 533, 534, 1000, 1024, 1025, 9, 9]), TAIL, {}),
    "past_1024": lambda: (pools(15, 20000, TAIL, [5, 40, 150, 219, 220, 221, 9, 9, 1023, 1024, 1025] + [9] * 12), TAIL, {}),
    "sparse_L2001": lambda: (photons(13, 7, 8, 4613, WIDE, 20.0, 20.0), WIDE, dict(k_init=3)),
    "dense_L2001": lambda: (photons(14, 7, 8, 4613, WIDE, 20.0, 400.0), WIDE, dict(k_init=3)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_list_search_matches_oracle(name):
    Z, irf, kw = CASES[name]()
    rows, cols, T = Z.shape
    p = dict(dict(dz=0.1, p_xy=1.0, r_min=1.0, r_init=0), **kw)
    p["k_max"] = 4
    p.setdefault("k_init", 3)
    off, ent = oracle.compact(Z[None])
    so = oracle.Oracle(oracle.Model(irf.probs, T), oracle.Params(**p)).init(off, ent, oracle.State(1, rows, cols, 4))
    ctx = rt3d.Context(irf.probs, T, **p)
    print(f"[gpu-init-lists] {name}: {rows}x{cols}x{T}, {len(ent)} entries, largest count {Z.max()}", flush=True)
    sg = device_to_oracle(ctx.step(rt3d.STEP_INIT, None, to_dev_u32(off), to_dev_u32(np.append(ent, 0)), shape=(1, rows, cols)), 4)
    assert so.cnt.sum() > 0
    np.testing.assert_array_equal(sg.cnt, so.cnt)
    np.testing.assert_array_equal(sg.t, so.t)
    np.testing.assert_allclose(sg.r, so.r, rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(sg.b, so.b, rtol=1e-6, atol=1e-12)
