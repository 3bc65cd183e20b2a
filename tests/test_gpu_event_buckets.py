"""The event ingest's buckets of pixels at their edges, bit-exact against the
oracle: pixel counts around a bucket and around the number of buckets, events
per pixel from none to past what a bucket's workgroup orders in LDS (the
direct way), a few pixels much brighter than the rest (both ways in one call),
segments around 64 and 128 events, invalid events among them, a capacity that cuts
the lists."""
import numpy as np
import pytest

from gpu_util import u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T = 700


def uniform(rng, P, n):
    return rng.integers(0, P, n), rng.integers(0, T, n)


def counts(rng, per_pixel, bins=T):
    return np.repeat(np.arange(len(per_pixel)), per_pixel), rng.integers(0, bins, int(np.sum(per_pixel)))


def skewed(rng, P, hot, each):
    c = rng.poisson(6, P)
    c[hot] = each
    return counts(rng, c)


CASES = {
    "one_pixel": lambda r: (1,) + counts(r, [500]),
    "five_pixels": lambda r: (5,) + counts(r, [0, 63, 64, 65, 1]),
    "4095_pixels": lambda r: (4095,) + uniform(r, 4095, 30000),
    "4097_pixels": lambda r: (4097,) + uniform(r, 4097, 30001),
    "65537_pixels": lambda r: (65537,) + uniform(r, 65537, 400000),
    "300000_pixels": lambda r: (300000,) + uniform(r, 300000, 50000),
    "cap_below": lambda r: (8,) + counts(r, [6144, 0, 0, 0, 6143, 1, 0, 0], 5),
    "cap_past": lambda r: (8,) + counts(r, [6144, 1, 0, 0, 20000, 3, 0, 70]),
    "skewed": lambda r: (20000,) + skewed(r, 20000, slice(9000, 9040), 3000),
    "hot_last": lambda r: (1030,) + skewed(r, 1030, slice(1029, 1030), 100000),
    "segments": lambda r: (2500,) + counts(r, r.integers(60, 68, 2500)),
    "segments_128": lambda r: (700,) + counts(r, r.integers(120, 136, 700)),
    "few_bins_100": lambda r: (400,) + counts(r, r.integers(66, 129, 400), 3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_event_buckets_bit_exact(name):
    rng = np.random.default_rng(sorted(CASES).index(name))
    P, pix, bins = CASES[name](rng)
    order = rng.permutation(pix.size)
    pix, bins = pix[order].astype(np.int32), bins[order].astype(np.int64)
    ctx = rt3d.Context(synth.gaussian_irf(1.5, 9).probs, T)
    dp = torch.from_numpy(pix).cuda()
    db = torch.from_numpy(bins.astype(np.uint16).view(np.int16)).cuda()
    print(f"[gpu-event-buckets] {name}: {pix.size} events, {P} pixels", flush=True)
    off, ent = ctx.compact_events(dp, db, P)
    assert ctx.query().device_error == 0
    oo, oe = oracle.compact_events(pix, bins, P, T)
    np.testing.assert_array_equal(u32(off), oo)
    np.testing.assert_array_equal(u32(ent)[:oo[-1]], oe)
    # a capacity inside the lists cuts them there
    cap = max(1, int(oo[-1]) * 2 // 3)
    off, ent = ctx.compact_events(dp, db, P, capacity=cap)
    np.testing.assert_array_equal(u32(off), np.minimum(oo, cap))
    np.testing.assert_array_equal(u32(ent)[:cap], oe[:cap])
    with pytest.raises(rt3d.Rt3dError) as e:
        ctx.query()
    assert e.value.status == rt3d.E_CAPACITY


def test_event_buckets_invalid_events_dropped():
    rng = np.random.default_rng(77)
    P = 5000
    pix, bins = skewed(rng, P, slice(100, 104), 4000)
    bad_p, bad_b = rng.integers(P, 2 * P, 300), rng.integers(T, 65536, 300)
    allp = np.concatenate([pix, bad_p, rng.integers(0, P, 300)]).astype(np.int32)
    allb = np.concatenate([bins, rng.integers(0, T, 300), bad_b])
    order = rng.permutation(allp.size)
    ctx = rt3d.Context(synth.gaussian_irf(1.5, 9).probs, T)
    off, ent = ctx.compact_events(torch.from_numpy(allp[order]).cuda(),
                                  torch.from_numpy(allb[order].astype(np.uint16).view(np.int16)).cuda(), P)
    with pytest.raises(rt3d.Rt3dError) as e:
        ctx.query()
    assert e.value.status == rt3d.E_INVALID
    oo, oe = oracle.compact_events(pix.astype(np.int32), bins.astype(np.int64), P, T)
    np.testing.assert_array_equal(u32(off), oo)
    np.testing.assert_array_equal(u32(ent)[:oo[-1]], oe)
