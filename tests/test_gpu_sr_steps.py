"""Super-resolved steps at their forks: IRFs with fewer and more segments than
the workgroup stages, blocks of 1 to 64 points, supports cut by both ends of the
histogram, against the oracle's gradients (the bar of the other gradient tests,
1e-4 of the sums' absolute terms); and the in-pixel merge fused with the
intensity step against the merge launched alone (a context that times it), bit
for bit."""
import numpy as np
import pytest

from gpu_util import sr_to_device, to_dev_hist, to_dev_u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402


def irf_of(name):
    return {"short": lambda: synth.gaussian_irf(1.5, 9), "long": lambda: synth.exgauss_irf(3.0, 30.0, -20, 300)}[name]()


@pytest.mark.parametrize("irf,s,T,points", [("short", 2, 60, 4), ("short", 3, 200, 1), ("short", 4, 90, 4),
                                            ("long", 2, 700, 3), ("long", 4, 350, 4)])
def test_sr_gradients_at_the_forks(irf, s, T, points):
    rng = np.random.default_rng(10 * s + points)
    rows, cols = 5, 7
    pr = irf_of(irf).probs
    st = oracle.SRState(1, rows, cols, s, 4)
    Pf, P = rows * cols * s * s, rows * cols
    st.cnt[:] = rng.integers(0, points + 1, Pf)
    for q in range(Pf):
        c = st.cnt[q]
        t = rng.uniform(0, T - 1, c)
        t[rng.random(c) < 0.2] = rng.choice([0.0, 1.5, T - 2.25, T - 1.0])
        st.t[q, :c] = np.sort(t)
        st.r[q, :c] = rng.uniform(0.05, 2.0, c)
    st.b[:] = rng.uniform(0.005, 0.1, P)
    z = rng.poisson(0.15, (1, P, T)).astype(np.uint16)
    z[0, 3] = 0                                       # a lidar pixel without entries
    off, ent = oracle.compact(z.reshape(1, rows, cols, T))
    O = oracle.Oracle(oracle.Model(pr, T), oracle.Params())
    ctx = rt3d.Context(pr, T, sr=s)
    (gt, gr, gb), (at, ar, ab) = O.sr_grad(off, ent, st)
    print(f"[gpu-sr-steps] gradients {irf} s={s} T={T}: {int(st.cnt.sum())} points", flush=True)
    dgt, dgr, dgb = ctx.gradients(sr_to_device(st), to_dev_u32(off), to_dev_u32(ent))
    live = np.arange(4)[None, :] < st.cnt[:, None]
    for g_gpu, g_or, a in ((dgt, gt, at), (dgr, gr, ar)):
        err = np.abs(g_gpu.cpu().numpy()[:4].T.astype(np.float64) - g_or)[live]
        assert np.all(err <= 1e-4 * a[live] + 1e-30), (err.max(), (err / a[live]).max())
    assert np.all(np.abs(dgb.cpu().numpy() - gb) <= 1e-4 * ab + 1e-30)


@pytest.mark.parametrize("s", [2, 3, 4])
def test_sr_merge_fused_equals_alone(s):
    sc = synth.sr_scene(5, rows=13, cols=9, s=s)
    m = sc.meta
    prm = dict(dz=m["dz"], p_xy=m["p_xy"], r_min=m["r_min"], r_init=m["r_init"], k_init=4, sr=s, d_merge=6.0)
    res = []
    for timed in (None, "merge"):
        ctx = rt3d.Context(sc.irf.probs, sc.T, **prm)
        ctx.profile(timed)
        print(f"[gpu-sr-steps] reconstruct s={s}, merge {'alone' if timed else 'fused'}", flush=True)
        o = ctx.reconstruct(to_dev_hist(sc.Z)[None])
        assert ctx.query().device_error == 0
        n = int(o.pt_off.cpu().numpy().astype(np.int64)[-1])
        res.append([o.pt_off.cpu().numpy(), o.background.cpu().numpy()] +
                   [x[:n].cpu().numpy() for x in (o.depth, o.intensity, o.normal)])
    assert res[0][2].size > 0
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)
