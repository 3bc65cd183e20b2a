"""APSS tiles of many points (a thread per two slots of a pixel) against the
same points spread over four tiles of few (a thread per point): both sum in the
window's order, so depths and normals are the same bits (the parity tests hold
the latter to the oracle).  Tiles at and next to the line between the two, full
tiles, windows of 1 to 5 rings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T, SIDE, FRAME = 200, 16, 40
IRF = synth.gaussian_irf(1.5, 9)


def state(points, at, seed):
    """A 40 x 40 frame, empty but for `points` points in the 16 x 16 pixels from (at, at) on."""
    rng = np.random.default_rng(seed)
    cnt = np.full(SIDE * SIDE, points // (SIDE * SIDE))
    cnt[rng.permutation(SIDE * SIDE)[:points % (SIDE * SIDE)]] += 1
    i, j = np.mgrid[0:SIDE, 0:SIDE]
    surf = np.stack([40 + 0.3 * i, 60 + 0.2 * j, 63 + 0.1 * i + 0.2 * j, 90 + 0 * i]).reshape(4, -1)
    t = np.sort(surf + rng.normal(0, 2.0, surf.shape), axis=0)
    n = rng.normal(0, 0.2, (3, 4, SIDE * SIDE)).astype(np.float32)
    n[2] = -1.0
    n /= np.linalg.norm(n, axis=0)
    r = rng.uniform(0.5, 5.0, surf.shape).astype(np.float32)
    st = rt3d.DeviceState.empty(1, FRAME, FRAME)
    px = ((i + at) * FRAME + j + at).reshape(-1)
    live = np.arange(4)[:, None] < cnt
    for name, v in (("t", np.where(live, t, 0.0)), ("r", np.where(live, r, 0).astype(np.float32)), ("n", n)):
        a = getattr(st, name).cpu().numpy()
        a[..., px] = v
        getattr(st, name).copy_(torch.from_numpy(a))
    c = np.zeros(FRAME * FRAME, np.uint8)
    c[px] = cnt
    st.cnt.copy_(torch.from_numpy(c))
    st.b.fill_(0.25)
    return st, px, live


@pytest.mark.parametrize("points", [447, 448, 449, 512, 513, 700, 1024])
@pytest.mark.parametrize("p_xy", [1.0, 0.8, 0.6, 0.45, 0.38])
def test_dense_tile_equals_sparse_tiles(points, p_xy):
    ctx = rt3d.Context(IRF.probs, T, dz=0.1, p_xy=p_xy, m_min=3)
    res = []
    for at in (16, 8):                       # one tile; a quarter of each of four
        st, px, live = state(points, at, 31 * points)
        print(f"[gpu-apss-dense] {points} points at {at}, p_xy {p_xy}", flush=True)
        out = ctx.step(rt3d.STEP_APSS, st)
        for a, b in ((out.cnt, st.cnt), (out.b, st.b), (out.r, st.r)):
            assert torch.equal(a, b)
        moved = (out.t.cpu().numpy() != st.t.cpu().numpy())[:, px][live].mean()
        assert moved > 0.5
        res.append((out.t.cpu().numpy()[:, px][live], out.n.cpu().numpy()[:, :, px][:, live]))
    np.testing.assert_array_equal(res[0][0], res[1][0])
    np.testing.assert_array_equal(res[0][1], res[1][1])
