"""A context serves any number of backward passes: keys of every length take each of two steps once (the partial
sums of keys reduced in pieces are left as the forward pass made them).  Against two Adagrad steps in double."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

COUNTS = [1, 9, 300, 2047, 2048, 2049, 5000]


@pytest.mark.parametrize("debug", [0, 2])            # the one-launch forward pass, and the large-batch kernels
@pytest.mark.parametrize("dim", [3, 6, 64, 130])
def test_two_backward_passes_on_one_context(dim, debug):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(5000 + dim)
    ids = rng.permutation(np.repeat(np.arange(len(COUNTS)) * 3, COUNTS)).astype(np.int64)
    B, lr, eps = len(ids), 0.05, 1e-8
    w = (rng.standard_normal((40, dim)) * 0.1).astype(np.float32)
    grads = [rng.standard_normal((B, dim)).astype(np.float32) for _ in range(2)]
    layer = PackedEmbedding([(40, dim, 0)], [(0, 0)], debug=debug)
    try:
        layer.load_table(0, w)
        layer.forward(torch.from_numpy(ids).cuda(), torch.arange(B + 1, dtype=torch.int32, device="cuda"), B)
        for g in grads:
            layer.backward_update(torch.from_numpy(g).cuda(), lr, eps)
        assert layer.error_word() == 0
        got_w, got_a = layer.W[0].cpu().numpy(), layer.A[0].cpu().numpy()
    finally:
        layer.close()
    ref_w, ref_a = w.astype(np.float64), np.zeros((40, dim))
    for g in grads:
        s = np.zeros((40, dim))
        np.add.at(s, ids, g.astype(np.float64))
        ref_a += s * s
        ref_w -= lr * s / (np.sqrt(ref_a) + eps)
    # per step: the sum is rounded to fp32, its square and the accumulator again (2 + 1 + 1 roundings of 2^-24 on a);
    # a weight takes a few roundings of steps that are at most lr in size, and of itself
    assert (np.abs(got_a - ref_a) <= 8 * 2.0 ** -24 * ref_a).all()
    assert (np.abs(got_w - ref_w) <= 16 * 2.0 ** -24 * (lr + np.abs(ref_w)) + 1e-9).all()
