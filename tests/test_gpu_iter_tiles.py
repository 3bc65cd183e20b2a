"""The iteration in three launches on tiles against the steps' own kernels,
bit for bit: a context whose background filter is timed runs the steps one by
one, and both paths promise the same arithmetic.  Frames of one pixel, around
the tile's sides, smaller than the filters' reach, of different sizes; windows
of 1 to 5 rings; no, narrow and wide background filters; four and eight lanes;
dead pixels and uneven gains; merges in the pixel."""
import numpy as np
import pytest

from gpu_util import to_dev_hist

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T = 120


def photons(rng, shapes):
    """Two surfaces a few bins apart under a sparse background."""
    z = []
    for rows, cols in shapes:
        i, j = np.meshgrid(np.arange(rows), np.arange(cols), indexing="ij")
        h = rng.poisson(0.02, (rows * cols, T))
        for base, share in ((40, 0.9), (47, 0.5), (85, 0.3)):
            at = base + 4 * np.sin(0.3 * i + 0.2 * j) + rng.normal(0, 0.5, i.shape)
            for _ in range(4):
                hit = rng.random(i.shape) < share
                b = np.clip(np.rint(at + rng.normal(0, 1.5, i.shape)), 0, T - 1).astype(int)
                np.add.at(h, (np.nonzero(hit.reshape(-1))[0], b.reshape(-1)[hit.reshape(-1)]), 1)
        z.append(h.astype(np.uint16))
    return np.concatenate(z)


CASES = {
    "one_pixel": dict(shapes=[(1, 1)]),
    "tile_4x16": dict(shapes=[(4, 16)] * 2),
    "tile_5x17": dict(shapes=[(5, 17)], lanes_per_pixel=4),
    "wide_1x70": dict(shapes=[(1, 70)]),
    "tall_37x2": dict(shapes=[(37, 2)], sigma_b=2.0),
    "batch": dict(shapes=[(23, 31)] * 3, gain=True),
    "sizes": dict(shapes=[(7, 9), (20, 33), (20, 33), (16, 4)], gain=True),
    "rings_2": dict(shapes=[(19, 21)], p_xy=0.8),
    "rings_5": dict(shapes=[(19, 21)], p_xy=0.37, lanes_per_pixel=4),
    "no_bfilter": dict(shapes=[(18, 18)], sigma_b=0.0),
    "wide_bfilter": dict(shapes=[(33, 18)], sigma_b=5.0),
    "box": dict(shapes=[(21, 22)], ilp_box=1, n_iter=3),
    "lanes_4": dict(shapes=[(64, 50)], lanes_per_pixel=4, gain=True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_three_launches_equal_the_steps(name):
    c = dict(CASES[name])
    shapes, with_gain = c.pop("shapes"), c.pop("gain", False)
    rng = np.random.default_rng(sorted(CASES).index(name))
    z = photons(rng, shapes)
    P = z.shape[0]
    gain = None
    if with_gain:
        g = rng.uniform(0.5, 2.0, P).astype(np.float32)
        g[rng.random(P) < 0.1] = 0.0
        gain = torch.from_numpy(g).cuda()
    irf = synth.gaussian_irf(1.5, 9).probs
    hist = to_dev_hist(z)
    res = []
    for timed in (None, "bfilter"):
        ctx = rt3d.Context(irf, T, dz=0.1, r_min=0.05, r_init=0, fused_loop=0, **c)
        ctx.profile(timed)
        rows, cols = shapes[0]
        kw = {} if len(set(shapes)) == 1 else dict(frame_shapes=shapes)
        if kw:
            ctx.workspace(1, 1, P, int(z.sum()) + 1)
        else:
            ctx.workspace(len(shapes), rows, cols, int(z.sum()) + 1)
        out = ctx.make_output(P)
        print(f"[gpu-iter-tiles] {name} {'steps' if timed else 'tiles'}: {shapes}", flush=True)
        ctx.reconstruct_into(out, len(shapes), rows, cols, hist=hist, gain=gain, **kw)
        assert ctx.query().device_error == 0
        n = int(out.pt_off.cpu().numpy().astype(np.int64)[-1])
        res.append([out.pt_off.cpu().numpy(), out.background.cpu().numpy()] +
                   [x[:n].cpu().numpy() for x in (out.depth, out.intensity, out.normal)])
    assert P == 1 or res[0][2].size > 0
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)
