"""The training kernels where their row pieces end: 16 columns to a product
of the weight gradients, 32 to one of the convolution, runs of rows that
start and stop inside a column or cross into the next image, fewer pieces
than waves. Against the FP64 reference with the same bfloat16 roundings.

Tolerance: the weight gradients are FP32 sums of products of bfloat16
values; the gradient itself is rounded to bfloat16 (2^-9 relative per value)
at every layer it passes, and where a rounding falls the other way than in
the reference a value moves by 2^-8, so a layer's gradient may differ by
about 2^-8 times the number of layers behind it: 2^-6 in the worst case."""
import numpy as np
import pytest

from oracle import upsampler as U

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 2, 3), (2, 5, 16), (1, 16, 17), (3, 7, 33), (2, 31, 32), (1, 3, 130),
          (1, 130, 3), (5, 33, 49),
          (3, 6500, 1), (2, 10100, 2)]  # ten rows and more to a wave


@pytest.mark.parametrize("n,h,w", SHAPES)
def test_gradients_and_update_at_ragged_sizes(n, h, w):
    import torch

    from paper_1804_08197_amd import upsampler as up
    r = np.random.default_rng(100 * h + w)
    params = [(0.2 * r.normal(size=(9, ci, co)), 0.05 * r.normal(size=co))
              for ci, co in up.LAYERS]
    params[0][0][:, 5:, :] = 0.0
    params = [(U.to_bf16(k), np.float32(b).astype(np.float64)) for k, b in params]
    rgba = r.uniform(0, 1, (n, h, w, 4)).astype(np.float32)
    depth = r.uniform(10, 400, (n, h, w)).astype(np.float32)
    depth[r.uniform(size=depth.shape) < 0.2] = np.inf
    target = r.uniform(0, 1, (n, 2 * h, 2 * w, 4)).astype(np.float32)
    m = up.Upsampler(n * h * w)
    try:
        vec = up.pack(params)
        m.set_weights(vec)
        t = [torch.from_numpy(a).cuda() for a in (rgba, depth, target)]
        loss, grads = m.gradients(t[0], t[1], 200.0, t[2], 0.5)
        code = np.where(np.isfinite(depth), 1.0 / (1.0 + depth / 200.0), 0.0)
        x0 = np.zeros((n, h, w, 8))
        x0[..., :4], x0[..., 4] = rgba, code
        ref_loss, ref = U.loss_and_grads(params, U.to_bf16(x0), target, 0.5, act_round=U.to_bf16)
        assert abs(loss - ref_loss) <= 1e-4 * ref_loss
        for layer, (got, want) in enumerate(zip(up.unpack(grads), ref)):
            for a, b in zip(got, want):
                off = np.linalg.norm(a - b) / np.linalg.norm(b)
                assert off < 2.0 ** -6, (layer, off)
        # one Adam step from zero moments moves each weight by lr against its
        # gradient's sign; the GEMM copies follow: the next gradients are
        # those of the moved weights
        assert m.train_step(t[0], t[1], 200.0, t[2], 1e-3, 0.5, want_loss=True) == loss
        g64 = grads.astype(np.float64)
        want = vec - 1e-3 * g64 / (np.abs(g64) + 1e-8)
        now = m.get_weights()
        assert np.abs(now - want).max() <= 1e-5
        again = up.Upsampler(n * h * w)
        again.set_weights(now)
        a = m.gradients(t[0], t[1], 200.0, t[2], 0.5)
        b = again.gradients(t[0], t[1], 200.0, t[2], 0.5)
        again.close()
        assert a[0] == b[0] and np.array_equal(a[1], b[1])
    finally:
        m.close()
