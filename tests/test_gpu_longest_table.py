"""The longest table a plan takes (2^30 rows): its 8192 slices of 128 K keys go through the large-batch kernels
whatever the batch's size.  Against the rows picked by torch and one Adagrad step of them in double."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROWS = 1 << 30


@pytest.mark.timeout(300)
def test_longest_table_is_taken_at_every_batch_size():
    from paper_2204_04903_amd import binding as pk
    from paper_2204_04903_amd.layer import PackedEmbedding
    if torch.cuda.mem_get_info()[0] < 16 * 2 ** 30:
        pytest.skip("needs 16 GiB of free device memory")
    lr, eps = 0.05, 1e-8
    layer = PackedEmbedding([(ROWS, 1, pk.PK_BF16)], [(0, pk.PK_SUM)])
    try:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(5)
        layer.W[0].normal_(0.0, 0.01, generator=gen)
        rng = np.random.default_rng(5)
        for B in (1, 300, 70_001, 600_001):            # (tiles of 32 bags up to 512)
            print(f"[longest table] B={B}", flush=True)
            keys = np.unique(np.concatenate([rng.integers(0, ROWS, size=B // 2), [0, ROWS - 1]]))
            ids = np.concatenate([keys, rng.choice(keys, size=max(B - len(keys), 0))])[:B]
            ids = torch.from_numpy(rng.permutation(ids)).cuda()
            offsets = torch.arange(B + 1, dtype=torch.int32, device="cuda")
            grad = torch.randn((B, 1), device="cuda", generator=gen)
            uq, inv = torch.unique(ids, return_inverse=True)
            w0, a0 = layer.W[0][uq, 0].double(), layer.A[0][uq, 0].double()
            g = torch.zeros(len(uq), dtype=torch.float64, device="cuda").index_add_(0, inv, grad[:, 0].double())
            out = layer.forward(ids, offsets, B)
            assert torch.equal(out[:, 0], layer.W[0][ids, 0].float())
            layer.backward_update(grad, lr, eps)
            assert layer.error_word() == 0
            assert np.array_equal(layer.ctx(0)["unique"], uq.cpu().numpy().astype(np.uint32))
            a1 = a0 + g * g
            w1 = w0 - lr * g / (a1.sqrt() + eps)
            assert ((layer.A[0][uq, 0] - a1).abs() <= 1e-6 + 1e-5 * a1).all()
            # the step is exact to a few fp32 roundings, the weight is rounded to bf16
            assert ((layer.W[0][uq, 0].double() - w1).abs() <= 1e-6 + 2.0 ** -8 * w1.abs()).all()
    finally:
        layer.close()
