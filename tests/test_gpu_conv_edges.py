"""The matrix-core convolutions at the edges of its tiles: kernels, channels, contraction indices and
positions that leave remainders, tiles that run from one image into the next, narrow maps, columns of
several 64-row bands, arrays that 32-bit offsets do not reach.  Encoded map, dense map in
fp32 and in bf16, against the direct convolution."""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_08314_amd import workloads

pytestmark = pytest.mark.gpu
FP32_TOL = 1e-5
BF16_TOL = 2e-2   # operands of 8 significant bits

# images, (C, H, W, K, kh, kw, stride, pad_h[, pad_w])
CASES = [
    (1, (1, 1, 1, 1, 1, 1, 1, 0)),        # one of everything
    (1, (1, 4, 4, 17, 3, 3, 1, 1)),       # fewer contraction indices than a step
    (3, (17, 7, 7, 65, 3, 3, 1, 1)),      # one channel and one kernel over; tiles across images
    (5, (33, 5, 3, 33, 3, 3, 1, 0)),      # one output column
    (2, (49, 13, 21, 31, 5, 5, 1, 2)),    # strips that end inside a tile
    (9, (3, 30, 30, 64, 7, 7, 2, 3)),     # few channels, stride 2
    (4, (20, 9, 9, 20, 3, 3, 4, 1)),      # stride beyond the kernel: columns no output needs
    (2, (24, 130, 6, 16, 3, 3, 1, 1)),    # three bands of 64 padded rows
    (1, (70, 12, 14, 130, 1, 7, 1, 0, 3)),
    (1, (5, 20, 20, 16, 11, 11, 1, 5)),   # the largest kernel
    (18, (3, 256, 256, 2, 11, 11, 250, 0)),   # a stride that leaves one output: windows of many images
    (3, (2, 254, 254, 3, 3, 3, 85, 1)),
    (6, (40, 9, 57, 40, 1, 3, 1, 0, 1)),   # strips wider than a wavefront's positions, taps of no kernel known
    (40, (160, 14, 14, 192, 3, 3, 1, 1)),  # more workgroups than the chip holds
]


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_08314_amd import api as _api
    _api.lib()
    return _api


@pytest.mark.parametrize("n_images,shape", CASES, ids=[f"{n}x{s}" for n, s in CASES])
def test_edges(api, n_images, shape):
    rng = np.random.default_rng(7)
    few = min(n_images, 9)
    acts = np.stack([workloads.random_case(100 + n % few, *shape[:8], zero_frac=0.5, zero_channels=0)[0] for n in range(n_images)])
    w_np = (rng.standard_normal((shape[3], shape[0], shape[4], shape[5])) * 0.2).astype(np.float32)
    ref = np.stack([oracle.conv_direct(acts[n], w_np, shape) for n in range(few)])
    ref = np.concatenate([ref] * (n_images // few) + [ref[:n_images % few]])
    buf = api.LayerBuffers(shape, n_images=n_images)
    act, w = torch.from_numpy(acts).cuda(), torch.from_numpy(w_np).cuda()
    api.cpoconv_prepare_weights(w, shape, buf.wt)
    api.cps_encode_batch(act, shape, buf.cps, buf.scratch)
    for run, tol in ((lambda: api.cps_conv_batch(buf.cps, shape, buf.wt, buf.out, buf.scratch), FP32_TOL),
                     (lambda: api.cpo_encode_conv(act, shape, buf.cpo, buf.wt, buf.out, buf.scratch), FP32_TOL),
                     (lambda: api.im2col_conv_batch(act, shape, n_images, w, buf.lowered, buf.out, 0), FP32_TOL),
                     (lambda: api.im2col_conv_batch(act, shape, n_images, w, buf.lowered, buf.out, 1), BF16_TOL)):
        buf.out.fill_(float("nan"))
        run()
        got = buf.out.cpu().numpy().reshape(ref.shape)
        assert np.abs(got - ref).max() <= tol * max(np.abs(ref).max(), 1e-30)


def test_weights_past_4_gib(api):
    shape = (256, 11, 11, 34700, 11, 11, 1, 0)
    torch.manual_seed(3)
    act = torch.relu(torch.randn(256, 11, 11, device="cuda"))
    w = torch.randn(34700, 256, 11, 11, device="cuda")
    ref = w.view(34700, -1) @ act.view(-1)
    buf = api.LayerBuffers(shape)
    assert 4 * buf.wt.numel() > 1 << 32 and 4 * w.numel() > 1 << 32
    api.cpoconv_prepare_weights(w, shape, buf.wt)
    for run, tol in ((lambda: api.cpo_encode_conv(act, shape, buf.cpo, buf.wt, buf.out, buf.scratch), FP32_TOL),
                     (lambda: api.im2col_conv(act, shape, w, buf.lowered, buf.out, 0), FP32_TOL),
                     (lambda: api.im2col_conv(act, shape, w, buf.lowered, buf.out, 1), BF16_TOL)):
        buf.out.fill_(float("nan"))
        run()
        assert (buf.out.view(-1) - ref).abs().max() <= tol * ref.abs().max()
