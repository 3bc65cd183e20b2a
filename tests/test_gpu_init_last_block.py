"""The initialisation's search where its block marks end: 32768 bins are 2048
blocks of 16 tau, 32 marks per lane, and a tile of 16 blocks around one of the
last reaches past them.  A cluster in the last block has the largest bound and
is not the peak sought, a cluster in the first blocks is: because the first
accepted peak suppresses the last block's tau, or because the last block's
cluster has the larger bound of the two and the smaller score.  32657 bins: the
first count whose last tile reaches past the marks.  Depths, counts equal to
the oracle's, the rest to the rounding of the stored values."""
import numpy as np
import pytest

from gpu_util import device_to_oracle, to_dev_u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

IRF = synth.gaussian_irf(1.5, 9)
# (bins, parameters, {bin: photons})
CASES = {
    "suppressed": (32768, dict(k_init=2, w_nms=100), {32699: 12, 32700: 18, 32701: 10, 32759: 8, 32760: 10, 32761: 7,
                                                      59: 3, 60: 4, 61: 3}),
    "suppressed_32657": (32657, dict(k_init=2, w_nms=100), {32599: 12, 32600: 18, 32601: 10, 32656: 25,
                                                            7: 3, 8: 4, 9: 3}),
    "larger_bound": (32768, dict(k_init=1), {50: 7, 51: 4, 53: 2, 32757: 8, 32763: 8}),
}


@pytest.mark.parametrize("spread", [0, 700])     # single photons between the clusters: large pools too
@pytest.mark.parametrize("name", sorted(CASES))
def test_first_blocks_stay_in_the_search(name, spread):
    T, kw, photons = CASES[name]
    Z = np.zeros((1, 3, T), np.uint16)
    Z[:, :, 1000:1000 + 40 * spread:40] = 1
    for b, n in photons.items():
        Z[0, :2, b] = n
    p = dict(dict(dz=0.1, p_xy=1.0, r_min=1.0, r_init=0), **kw)
    off, ent = oracle.compact(Z[None])
    so = oracle.Oracle(oracle.Model(IRF.probs, T), oracle.Params(**p)).init(off, ent, oracle.State(1, 1, 3, 4))
    ctx = rt3d.Context(IRF.probs, T, **p)
    print(f"[gpu-init-last-block] {name}: {T} bins, {len(ent)} entries", flush=True)
    sg = device_to_oracle(ctx.step(rt3d.STEP_INIT, None, to_dev_u32(off), to_dev_u32(np.append(ent, 0)), shape=(1, 1, 3)), 4)
    assert so.t[0].min() >= 0 and (so.t[0, :so.cnt[0]] < 112).any()      # the first blocks hold a peak
    np.testing.assert_array_equal(sg.cnt, so.cnt)
    np.testing.assert_array_equal(sg.t, so.t)
    np.testing.assert_allclose(sg.r, so.r, rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(sg.b, so.b, rtol=1e-6, atol=1e-12)
