"""The learned denoiser's fused forward, backward and weight-gradient kernels at
the edges of their tiles: images below, at and past one 16 x 16 tile, one
64-column segment and one 8-row unit of the weight gradient, several frames,
more true surfaces than the forward kernel holds in registers.  Against the
FP64 oracle with the same FP16 storage: outputs within 2e-3 of the output
scale and every gradient element within 1e-2 of its layer's largest (the bars
of the network's other tests: a few FP16 steps, 2^-11, through four layers)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from oracle import cnn  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T = 400


def random_state(rng, F, H, W, S):
    P = F * H * W
    truth = np.where(rng.random((S, P)) < 0.8, rng.uniform(30, T - 30, (S, P)), np.nan)
    truth[0] = 120.0 + rng.normal(0, 2.0, P)
    cnt = rng.integers(0, 5, P)
    t = np.zeros((4, P))
    for k in range(4):
        src = truth[k % S]
        t[k] = np.where(np.isnan(src), rng.uniform(20, T - 20, P), src) + rng.normal(0, 3.0, P)
    t = np.sort(np.clip(t, 0, T - 1), axis=0)
    r = rng.uniform(0.2, 3.0, (4, P)).astype(np.float32)
    live = np.arange(4)[:, None] < cnt
    t, r = np.where(live, t, 0.0), np.where(live, r, 0.0).astype(np.float32)
    n = np.zeros((3, 4, P), np.float32)
    n[2] = -1.0
    st = rt3d.DeviceState(F, H, W, torch.from_numpy(t).cuda(), torch.from_numpy(r).cuda(), torch.from_numpy(n).cuda(),
                          torch.from_numpy(cnt.astype(np.uint8)).cuda(), torch.zeros(P, device="cuda"))
    return t, r, cnt, truth.astype(np.float32), st


@pytest.mark.parametrize("F,H,W,S", [(1, 3, 5, 1), (1, 16, 16, 2), (2, 17, 33, 3), (1, 9, 65, 3), (3, 8, 64, 6),
                                     (1, 33, 130, 4)])
def test_network_and_gradient_match_oracle(F, H, W, S):
    rng = np.random.default_rng(1000 * H + W)
    t, r, cnt, truth, st = random_state(rng, F, H, W, S)
    irf = synth.exgauss_irf(3.0, 10.0, -18, 118)
    ctx = rt3d.Context(irf.probs, T, denoiser=rt3d.DENOISE_CNN)
    ctx.workspace(F, H, W, 1)
    sig = float(np.sqrt(ctx.sigma2))
    w = cnn.he_init(H + W)
    ctx.cnn_set_weights(w)
    print(f"[gpu-cnn-tiles] {F} x {H} x {W}, {S} surfaces", flush=True)
    x = cnn.features(t.T, r.T, cnt, sig, F, H, W)
    yo, _ = cnn.forward(x, w.astype(np.float64), fp16=True)
    y = ctx.cnn_forward(st).cpu().numpy()
    scale = max(1.0, np.abs(yo).max())
    assert np.abs(y - yo.reshape(-1, 3).T).max() <= 2e-3 * scale
    loss = ctx.cnn_train_step(st, torch.from_numpy(truth).cuda(), lr=1e-3).cpu().numpy()
    g = ctx.cnn_last_gradient().astype(np.float64)
    tgt, msk = cnn.targets(t.T, cnt, truth.astype(np.float64), sig)
    lo, go = cnn.loss_and_grad(x, w.astype(np.float64), tgt.reshape(F, H, W, 3), msk.reshape(F, H, W, 3), fp16=True)
    assert int(loss[1]) == int(msk.sum()) and abs(loss[0] - lo) <= 1e-2 * max(lo, 1e-6)
    at = 0
    for ci, co in zip(cnn.CIN, cnn.COUT):
        n = 9 * ci * co + co
        assert np.abs(g[at:at + n] - go[at:at + n]).max() <= 1e-2 * max(np.abs(go[at:at + n]).max(), 1e-30)
        at += n
    w1, _, _ = cnn.adam(w.astype(np.float64), g, np.zeros_like(g), np.zeros_like(g), 1, 1e-3)
    np.testing.assert_allclose(ctx.cnn_get_weights(), w1, rtol=1e-5, atol=1e-6)
    # the FP16 layouts the next pass uses are the new weights'
    y1, _ = cnn.forward(x, ctx.cnn_get_weights().astype(np.float64), fp16=True)
    y = ctx.cnn_forward(st).cpu().numpy()
    assert np.abs(y - y1.reshape(-1, 3).T).max() <= 2e-3 * max(1.0, np.abs(y1).max())
