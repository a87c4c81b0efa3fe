"""The one-launch forward pass where blocks cannot wait for the blocks before them: distinct keys counted from the IDs
instead of waited for give the same context bit for bit, the same pooled rows and the same step, and bad offsets in another
block's share are still reported."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = {
    # tables: rows, dim; fields: table, pooling, longest bag; samples
    "one-hot": ([(100_000, 8)] * 26, [(t, 0, 1) for t in range(26)], 700),
    "one-hot, several slices": ([(1_000_000, 4), (70_000, 4), (3, 8)], [(0, 0, 1), (1, 0, 1), (2, 1, 1)], 4096),
    "slices of 128 K keys": ([(131_072, 4), (400_000, 4)], [(0, 1, 3), (1, 0, 2)], 150),
    "bags, sampled offsets": ([(900_000, 4), (5_000, 8), (300_000, 4)], [(0, 1, 5), (1, 0, 9), (2, 0, 3)], 5000),
    "shared tables": ([(200_000, 4), (900, 8), (150_000, 4)], [(0, 1, 4), (1, 0, 6), (0, 0, 1), (2, 1, 3), (1, 1, 2), (0, 0, 2)], 2500),
    "two blocks to a unit": ([(1_000_000, 4)] * 26, [(t, t % 2, 1) for t in range(26)], 8192),
    "two blocks to a unit, shared tables": ([(500_000, 4)] * 13, [(t % 13, t % 2, 1 + t % 3) for t in range(26)], 7000),
    "more than is kept": ([(50_000, 4), (2_000, 4)], [(0, 0, 9), (1, 1, 40)], 3000),
}


def _batch(name):
    tables, fields, B = CASES[name]
    rng = np.random.default_rng(sum(map(ord, name)))
    lens = [np.ones(B, np.int64) if hi == 1 else rng.integers(0, hi + 1, size=B) for _, _, hi in fields]
    ids = [(rng.random(n.sum()) ** 3 * tables[t][0]).astype(np.int64) for (t, _, _), n in zip(fields, lens)]
    offsets = np.zeros(len(fields) * B + 1, np.int32)
    offsets[1:] = np.cumsum(np.concatenate(lens))
    return tables, fields, B, np.concatenate(ids), offsets, rng


@pytest.mark.parametrize("name", CASES)
def test_numbers_counted_from_the_ids(name):
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables, fields, B, ids, offsets, rng = _batch(name)
    assert len(ids) < 1 << 19
    d_ids, d_off = torch.from_numpy(ids).cuda(), torch.from_numpy(offsets).cuda()
    W0, grad, got = None, None, []
    for debug in (0, 4):
        layer = PackedEmbedding([(r, d, 0) for r, d in tables], [(t, p) for t, p, _ in fields], debug=debug)
        try:
            if W0 is None:
                W0 = [torch.randn(W.shape, device="cuda") for W in layer.W]
                grad = torch.from_numpy(rng.integers(-3, 4, size=(B, layer.out_dim)).astype(np.float32)).cuda()
            for W, w in zip(layer.W, W0):
                W.copy_(w)
            for step in range(3):                         # (the library's words are clean for the next call)
                out = layer.forward(d_ids, d_off, B)
                assert layer.error_word() == 0
            ctx = [layer.ctx(p) for p in range(layer.n_packs)]
            layer.backward_update(grad, 0.5, 1e-8)
            got.append((out.cpu().numpy(), ctx, [A.cpu().numpy() for A in layer.A]))
        finally:
            layer.close()
    (out0, ctx0, A0), (out1, ctx1, A1) = got
    assert np.array_equal(out0.view(np.uint32), out1.view(np.uint32))
    for c0, c1 in zip(ctx0, ctx1):
        assert c0.keys() == c1.keys()
        uq, inv, cnt = np.unique(c0["keys"], return_inverse=True, return_counts=True)
        for c in (c0, c1):
            assert np.array_equal(c["unique"], uq) and np.array_equal(c["inverse"], inv)
            assert np.array_equal(c["seg_offsets"], np.concatenate([[0], np.cumsum(cnt)]))
        assert np.array_equal(c0["keys"], c1["keys"]) and np.array_equal(c0["packed_offsets"], c1["packed_offsets"])
    for a0, a1 in zip(A0, A1):                            # sum pooling: exact; mean: fp64 sums in another order, rounded once
        assert np.all(np.abs(a0 - a1) <= 2.0 ** -22 * np.abs(a0) + 1e-18)


@pytest.mark.parametrize("name", ["bags, sampled offsets", "shared tables"])
def test_bad_offsets_in_another_share_are_reported(name):
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables, fields, B, ids, offsets, _ = _batch(name)
    offsets[B // 9] = offsets[2 * B // 9 + 5] + 1         # inside the first field, in its first slice's share
    layer = PackedEmbedding([(r, d, 0) for r, d in tables], [(t, p) for t, p, _ in fields], debug=4)
    try:
        for W in layer.W:
            W.zero_()
        layer.forward(torch.from_numpy(ids).cuda(), torch.from_numpy(offsets).cuda(), B)
        assert layer.error_word() == 1
        layer.backward_update(torch.ones((B, layer.out_dim), device="cuda"), 0.5, 1e-8)
        p = layer.table_slot[0][0]
        assert not bool(layer.A[p].any())
    finally:
        layer.close()
