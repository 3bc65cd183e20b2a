"""Training steps of the learned denoiser on more work than its grids hold at
once: over 1024 tiles of 16 x 16 pixels (a workgroup of the forward kernel then
takes several, its LDS and its loss sums carried from one to the next) and over
256 units of the weight gradient (a workgroup's ring of rows used again), in
counts that no grid divides.  Against the FP64 oracle with the same FP16
storage, every gradient element within 1e-2 of its layer's largest as in the
network's other tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from oracle import cnn  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402
from test_gpu_cnn_tiles import T, random_state  # noqa: E402


@pytest.mark.parametrize("F,H,W,S", [(1100, 3, 5, 2), (1100, 17, 5, 3), (5, 70, 400, 2)])
def test_strided_training_matches_oracle(F, H, W, S):
    rng = np.random.default_rng(F + H + W)
    t, r, cnt, truth, st = random_state(rng, F, H, W, S)
    ctx = rt3d.Context(synth.exgauss_irf(3.0, 10.0, -18, 118).probs, T, denoiser=rt3d.DENOISE_CNN)
    ctx.workspace(F, H, W, 1)
    sig = float(np.sqrt(ctx.sigma2))
    w = cnn.he_init(F + W)
    ctx.cnn_set_weights(w)
    print(f"[gpu-cnn-strides] {F} x {H} x {W}, {S} surfaces", flush=True)
    x = cnn.features(t.T, r.T, cnt, sig, F, H, W)
    tgt, msk = cnn.targets(t.T, cnt, truth.astype(np.float64), sig)
    lo, go = cnn.loss_and_grad(x, w.astype(np.float64), tgt.reshape(F, H, W, 3), msk.reshape(F, H, W, 3), fp16=True)
    d_truth = torch.from_numpy(truth).cuda()
    for step in range(2):                        # a second pass on what the first one left behind
        ctx.cnn_set_weights(w)
        loss = ctx.cnn_train_step(st, d_truth, lr=1e-3).cpu().numpy()
        g = ctx.cnn_last_gradient().astype(np.float64)
        assert int(loss[1]) == int(msk.sum()) and abs(loss[0] - lo) <= 1e-2 * max(lo, 1e-6)
        at = 0
        for ci, co in zip(cnn.CIN, cnn.COUT):
            n = 9 * ci * co + co
            assert np.abs(g[at:at + n] - go[at:at + n]).max() <= 1e-2 * max(np.abs(go[at:at + n]).max(), 1e-30), (step, at)
            at += n
