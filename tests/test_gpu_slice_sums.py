"""The large-batch dedup's slices: a pack of more slices than a group of sums holds, packs that begin inside one, slices
without records, slices of one frequent key with more records than are kept, slices of more distinct keys than a round
counts, bags too long for a record's bits.  Against numpy's unique and counts, whole numbers exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = {
    # rows and IDs per table, (dim, pooling); 64 slices to a group, 4096 records kept, 4096 keys to a round
    "one group exactly": [(64 << 10, 196_608, 4, 0)],
    "a slice more": [(65 << 10, 199_680, 4, 0)],
    "groups of two packs": [(70 << 10, 230_000, 4, 0), (200 << 10, 660_000, 8, 1), (90, 1, 4, 0), (3, 7, 8, 1)],
    "empty slices": [(9_000_000, 11, 4, 1), (1, 0, 4, 0), (5_000_001, 3, 4, 0)],
    "frequent key": [(4097, 60_000, 4, 1)],
    "many keys to a slice": [(40_000_000, 150_000, 4, 0)],
    "unequal": [(1000, 8193, 8, 1), (70_001, 4096, 8, 0), (70_001, 4097, 4, 0)],
}


@pytest.mark.parametrize("name", CASES)
def test_slices(name):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(sum(map(ord, name)))
    B = 5
    tables = [(rows, dim, 0) for rows, _, dim, _ in CASES[name]]
    layer = PackedEmbedding(tables, [(t, c[3]) for t, c in enumerate(CASES[name])], debug=2)
    try:
        ids, lens = [], []
        for rows, n, _, _ in CASES[name]:
            if name == "frequent key":                    # nine of ten occurrences are one key's
                k = np.where(rng.random(n) < 0.9, 1234, rng.integers(0, rows, size=n))
            elif name == "many keys to a slice":          # all in the first slices of a long table
                k = rng.integers(0, 30_000, size=n)
            else:
                k = rng.integers(0, rows, size=n)
            ids.append(k.astype(np.int64))
            # (one bag of nearly all: above 65535 IDs its length does not fit a record)
            lens.append(np.array([0, n - n // 4, 0, n // 4, 0]))
        offsets = np.zeros(len(tables) * B + 1, np.int32)
        offsets[1:] = np.cumsum(np.concatenate(lens))
        d_ids, d_off = torch.from_numpy(np.concatenate(ids)).cuda(), torch.from_numpy(offsets).cuda()
        for W in layer.W:
            W.fill_(1.0)
        grad = torch.ones((B, layer.out_dim), device="cuda")
        for step in range(2):                             # the second call finds the first one's workspace
            layer.forward(d_ids, d_off, B)
            torch.cuda.synchronize()
            assert layer.error_word() == 0
            for p in range(layer.n_packs):
                ctx = layer.ctx(p)
                uq, inv, cnt = np.unique(ctx["keys"], return_inverse=True, return_counts=True)
                want = np.concatenate([layer.table_slot[t][1] + ids[t] for t in range(len(tables)) if layer.table_slot[t][0] == p])
                assert np.array_equal(ctx["keys"], want.astype(np.uint32))
                assert np.array_equal(ctx["unique"], uq)
                assert np.array_equal(ctx["inverse"], inv)
                assert np.array_equal(ctx["seg_offsets"], np.concatenate([[0], np.cumsum(cnt)]))
        # a key's gradient: occurrences (sum) or occurrences over their bags' lengths (mean); the accumulator starts at 0
        layer.backward_update(grad, 0.5, 1e-8)
        for t, (rows, n, dim, pool) in enumerate(CASES[name]):
            bag = np.repeat(np.arange(B), lens[t])
            g = np.bincount(ids[t], weights=1.0 / np.maximum(lens[t], 1)[bag] if pool else None, minlength=rows)
            a = layer.acc_view(t).cpu().numpy().astype(np.float64)
            assert np.all(np.abs(a - (g * g)[:, None]) <= 1e-6 + 1e-5 * (g * g)[:, None]), t
    finally:
        layer.close()
