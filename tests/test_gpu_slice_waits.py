"""The large-batch dedup where blocks cannot wait for the blocks before them: their numbers counted from the records give
the same results bit for bit, and a block that gives up ends the pack's others at once and leaves the tables alone.  And the
published sums side by side, as where the scratch of calls that cannot allocate ends."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = {
    # tables: rows, IDs, dim, dtype, pooling, law; 64 slices of 65536 keys to a group
    "three groups": [(150 << 16, 700_000, 4, 0, 0, "even")],
    "slices of many records first": [(1000, 40_000, 4, 0, 1, "even"), (70 << 16, 300_000, 4, 0, 0, "even"), (900, 9_000, 4, 0, 1, "low")],
    "two packs, groups of both": [(40 << 16, 90_000, 4, 0, 1, "low"), (90 << 16, 90_000, 4, 0, 0, "even"),
                                  (65 << 16, 50_000, 8, 0, 0, "low"), (3, 20_000, 8, 0, 1, "even")],
    "many keys": [(5_000_000, 120_000, 4, 0, 1, "low"), (80 << 16, 10_000, 4, 0, 0, "even")],
    "128 K keys to a slice": [((4096 << 16) + 5, 60_000, 1, 1, 1, "low"), (200_000, 30_000, 1, 1, 0, "low")],
}


def _inputs(case, B, rng):
    ids, lens = [], []
    for rows, n, _, _, _, law in case:
        u = rng.random(n)
        ids.append(np.minimum((u if law == "even" else u ** 9) * rows, rows - 1).astype(np.int64))
        lens.append(np.array([n // 3, 0, 7, n - n // 3 - 7]))
    offsets = np.zeros(len(case) * B + 1, np.int32)
    offsets[1:] = np.cumsum(np.concatenate(lens))
    return ids, torch.from_numpy(np.concatenate(ids)).cuda(), torch.from_numpy(offsets).cuda()


@pytest.mark.parametrize("name", CASES)
def test_numbers_counted_from_the_records(name):
    from paper_2204_04903_amd.layer import PackedEmbedding
    case, B = CASES[name], 4
    ids, d_ids, d_off = _inputs(case, B, np.random.default_rng(sum(map(ord, name))))
    tables, fields = [(c[0], c[2], c[3]) for c in case], [(t, c[4]) for t, c in enumerate(case)]
    got = []
    for debug in (2, 2 | 4, 2 | 16):
        layer = PackedEmbedding(tables, fields, debug=debug)
        try:
            for W in layer.W:
                W.fill_(1.0)
            for step in range(2):                         # the second call finds the first one's workspace
                layer.forward(d_ids, d_off, B)
                torch.cuda.synchronize()
                assert layer.error_word() == 0
                ctx = [layer.ctx(p) for p in range(layer.n_packs)]
            for p, c in enumerate(ctx):
                keys = np.concatenate([layer.table_slot[t][1] + ids[t] for t in range(len(case)) if layer.table_slot[t][0] == p])
                uq, inv, cnt = np.unique(keys.astype(np.uint32), return_inverse=True, return_counts=True)
                assert np.array_equal(c["unique"], uq)
                assert np.array_equal(c["inverse"], inv)
                assert np.array_equal(c["seg_offsets"], np.concatenate([[0], np.cumsum(cnt)]))
            layer.backward_update(torch.ones((B, layer.out_dim), device="cuda"), 0.5, 1e-8)
            got.append(([d["unique"] for d in ctx], [A.cpu() for A in layer.A]))
        finally:
            layer.close()
    for other in got[1:]:
        for u0, u1 in zip(got[0][0], other[0]):
            assert np.array_equal(u0, u1)
        for a0, a1 in zip(got[0][1], other[1]):           # (sums in fp64, in another order)
            assert torch.allclose(a0, a1, rtol=1e-6, atol=0.0)


@pytest.mark.parametrize("rows", [400 << 16, (4096 << 16) + 5])
def test_giving_up_ends_the_pack_at_once(rows):
    from paper_2204_04903_amd.layer import PackedEmbedding
    case, B = [(rows, 50_000, 1, 1, 0, "even"), (1000, 9_000, 2, 1, 0, "even")], 4
    _, d_ids, d_off = _inputs(case, B, np.random.default_rng(3))
    layer = PackedEmbedding([(c[0], c[2], c[3]) for c in case], [(0, 0), (1, 0)], debug=2 | 8)
    try:
        for W in layer.W:
            W.fill_(1.0)
        layer._ensure_ws(B, d_ids.shape[0])
        torch.cuda.synchronize()
        t0 = time.monotonic()
        layer.forward(d_ids, d_off, B)
        layer.backward_update(torch.ones((B, layer.out_dim), device="cuda"), 0.5, 1e-8)
        torch.cuda.synchronize()
        assert time.monotonic() - t0 < 1.0                # one block's patience is 12 s
        assert layer.error_word() == 2
        p, q = layer.table_slot[0][0], layer.table_slot[1][0]
        assert p != q and bool((layer.W[p] == 1.0).all()) and not bool(layer.A[p].any())
        assert bool(layer.A[q].any())                     # the other pack has one group and is updated
    finally:
        layer.close()
