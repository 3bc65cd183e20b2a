"""The initialisation's dense search at the edges of its ranges: pooled counts
of 127 and 128 in one bin (bytes against scaled bytes), counts whose scores
pass 32 bits and windows of more than 127 pixels (the search from the lists),
bin counts around a block of 16 tau, a tile of 256 and the last count each
search takes, empty pixels with no minimum count.  Counts and depths must
equal the oracle's exactly, intensities and background to FP32 rounding (the
stored values are FP64 results rounded once: 2^-24 relative)."""
import numpy as np
import pytest

from gpu_util import device_to_oracle, to_dev_u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

GAUSS, TAIL = synth.gaussian_irf(1.5, 9), synth.exgauss_irf(3.0, 10.0, -18, 118)


def photons(seed, rows, cols, T, irf, signal, bkg):
    rng = np.random.default_rng(seed)
    i, j = np.mgrid[0:rows, 0:cols].astype(np.float64)
    d = 0.15 * T + 0.6 * T * (j + 0.3 * i) / (cols + 0.3 * rows)
    return synth.render(rng, irf, T, d[None], rng.uniform(0.7, 1.3, (1, rows, cols)) * signal, bkg / T)


def spike(T, z):
    """A pixel row whose pooled bin 40 holds exactly 127 or 128 photons beside ordinary ones."""
    Z = photons(7, 6, 12, T, GAUSS, 8.0, 4.0)
    Z[:, :, 40] = 0
    Z[3, 2, 40], Z[3, 3, 40] = z - 60, 60
    Z[1, 8, 40] = z
    return Z


CASES = {
    "bin127": lambda: (spike(300, 127), GAUSS, dict(r_init=1)),
    "bin128": lambda: (spike(300, 128), GAUSS, dict(r_init=1)),
    "bright": lambda: (photons(8, 12, 14, 400, GAUSS, 900.0, 20.0), GAUSS, dict(r_init=1)),
    "bright_tail": lambda: (photons(9, 10, 12, 700, TAIL, 4000.0, 300.0), TAIL, dict(r_init=1, k_init=4)),
    "past32bits": lambda: (photons(10, 6, 8, 300, GAUSS, 60000.0, 10.0), GAUSS, dict(r_init=1)),
    "window169": lambda: (np.maximum(photons(11, 14, 15, 200, GAUSS, 5.0, 3.0), (np.arange(200) % 50 == 7)).astype(np.uint16),
                          GAUSS, dict(r_init=6)),
    "empty_nmin0": lambda: (np.zeros((5, 7, 333), np.uint16), TAIL, dict(r_init=1, n_min=0)),
    "T32769": lambda: (photons(12, 4, 6, 32769, TAIL, 12.0, 30.0), TAIL, dict(r_init=1)),
    "T32768": lambda: (photons(13, 4, 6, 32768, TAIL, 12.0, 30.0), TAIL, dict(r_init=1)),
}
for _t in (137, 255, 256, 257, 767, 769, 4608, 4609, 4865):
    CASES[f"T{_t}"] = lambda t=_t: (photons(100 + t, 8, 9, t, TAIL, 6.0, 25.0), TAIL, dict(r_init=1, k_init=4))


@pytest.mark.parametrize("name", sorted(CASES))
def test_dense_search_matches_oracle(name):
    Z, irf, kw = CASES[name]()
    rows, cols, T = Z.shape
    p = dict(dict(dz=0.1, p_xy=1.0, r_min=1.0, k_init=3), **kw)
    off, ent = oracle.compact(Z[None])
    so = oracle.Oracle(oracle.Model(irf.probs, T), oracle.Params(**p)).init(off, ent, oracle.State(1, rows, cols, 4))
    ctx = rt3d.Context(irf.probs, T, **p)
    print(f"[gpu-init-dense] {name}: {rows}x{cols}x{T}, {len(ent)} entries, largest count {Z.max()}", flush=True)
    sg = device_to_oracle(ctx.step(rt3d.STEP_INIT, None, to_dev_u32(off), to_dev_u32(np.append(ent, 0)), shape=(1, rows, cols)), 4)
    np.testing.assert_array_equal(sg.cnt, so.cnt)
    np.testing.assert_array_equal(sg.t, so.t)
    np.testing.assert_allclose(sg.r, so.r, rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(sg.b, so.b, rtol=1e-6, atol=1e-12)
