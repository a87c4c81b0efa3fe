"""pk_forward_static, the forward pass for callers that cannot allocate, against pk_forward: the same
kernels with the workspace in the library's static device array.  Two calls in a row, the second with a
smaller input (the array keeps the first call's contents), on the one-launch path and on the partitioned
one; then a call the array cannot hold, which must be refused."""
import numpy as np
import pytest
import torch

from helpers import small_problem

pytestmark = pytest.mark.gpu


def _run_pair(layer, pr, B):
    from paper_2204_04903_amd import binding as pk
    ids = torch.from_numpy(pr["ids"]).cuda()
    offsets = torch.from_numpy(pr["offsets"]).cuda()
    nnz = int(ids.shape[0])
    ref = layer.forward(ids, offsets, B).clone()
    got = torch.full((B, layer.out_dim), 3.0, dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    pk.pk_forward_static(layer.plan, layer.W, ids, offsets, B, nnz, got, got.stride(0), stream)
    torch.cuda.synchronize()
    assert layer.error_word() == 0
    return ref.cpu().numpy(), got.cpu().numpy()


@pytest.mark.parametrize("debug", [0, 2])          # 0: one launch; 2: occurrences partitioned by slice
def test_static_forward_equals_forward_twice_the_second_call_smaller(debug):
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables = [(5, 8, 0), (300, 64, 0), (40000, 8, 0), (3, 64, 1), (50000, 32, 0), (40, 32, 0)]
    fields = [(0, 0), (1, 1), (2, 0), (3, 1), (4, 0), (5, 1), (2, 1), (4, 1), (0, 1)]
    big = small_problem(900, B=1500, tables=tables, fields=fields, max_len=12)
    small = small_problem(901, B=200, tables=tables, fields=fields, max_len=5)
    layer = PackedEmbedding(tables, fields, debug=debug)
    try:
        for t, w in enumerate(big["Wt"]):
            layer.load_table(t, w)
        for name, pr in (("first", big), ("second, smaller", small)):
            print(f"[static] {name}: B={pr['B']} nnz={len(pr['ids'])} debug={debug}", flush=True)
            ref, got = _run_pair(layer, pr, pr["B"])
            assert np.array_equal(ref.view(np.uint32), got.view(np.uint32)), name      # the same kernels: the same bits
    finally:
        layer.close()


def test_static_forward_refuses_what_the_static_array_cannot_hold():
    from paper_2204_04903_amd import binding as pk
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables, fields = [(1000, 8, 0)], [(0, 0)]
    layer = PackedEmbedding(tables, fields)
    try:
        B = 1 << 21                                   # 2 M one-hot bags: the workspace alone exceeds 32 MiB
        assert pk.pk_workspace_bytes(layer.plan, B, B) > (32 << 20)
        ids = torch.zeros(B, dtype=torch.int64, device="cuda")
        offsets = torch.arange(B + 1, dtype=torch.int32, device="cuda")
        out = torch.zeros((B, 8), dtype=torch.float32, device="cuda")
        with pytest.raises(pk.PkError) as e:
            pk.pk_forward_static(layer.plan, layer.W, ids, offsets, B, B, out, 8, torch.cuda.current_stream().cuda_stream)
        assert e.value.status == pk.PK_EWORKSPACE
    finally:
        layer.close()


def test_static_forward_near_the_limit_leaves_the_stored_counts_out():
    from paper_2204_04903_amd import binding as pk
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables, fields = [(1_000_000, 8, 0)], [(0, 0)]
    layer = PackedEmbedding(tables, fields)
    try:
        lo, hi = 1 << 19, 1 << 21                     # the smallest one-hot batch whose workspace exceeds the array
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if pk.pk_workspace_bytes(layer.plan, mid, mid) <= (32 << 20) else (lo, mid)
        B = hi
        rng = np.random.default_rng(902)
        layer.load_table(0, rng.standard_normal((1_000_000, 8)).astype(np.float32))
        pr = dict(ids=rng.integers(0, 1_000_000, size=B).astype(np.int64), offsets=np.arange(B + 1, dtype=np.int32))
        print(f"[static] near the limit: B={B}", flush=True)
        ref, got = _run_pair(layer, pr, B)
        assert np.array_equal(ref.view(np.uint32), got.view(np.uint32))
    finally:
        layer.close()


def test_static_forward_at_the_largest_call_it_takes():
    # there the stored counts are left out and the slices' sums stand side by side (tests/test_layout.py)
    from paper_2204_04903_amd import binding as pk
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables, fields = [(6_000_000, 4, 0), (900, 8, 0)], [(0, 0), (1, 1)]
    layer = PackedEmbedding(tables, fields)
    try:
        lo, hi = 1 << 18, 1 << 20
        rng = np.random.default_rng(903)
        layer.load_table(0, rng.standard_normal((6_000_000, 4)).astype(np.float32))
        layer.load_table(1, rng.standard_normal((900, 8)).astype(np.float32))
        ids = torch.from_numpy(np.concatenate([rng.integers(0, 6_000_000, size=hi), rng.integers(0, 900, size=hi)])).cuda()
        out = torch.empty((hi, layer.out_dim), device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        while hi - lo > 1:
            B = (lo + hi) // 2
            offsets = torch.arange(2 * B + 1, dtype=torch.int32, device="cuda")
            try:
                pk.pk_forward_static(layer.plan, layer.W, ids, offsets, B, 2 * B, out, out.stride(0), stream)
                lo = B
            except pk.PkError as e:
                assert e.status == pk.PK_EWORKSPACE
                hi = B
        torch.cuda.synchronize()
        assert (1 << 18) < lo < (1 << 20) - 1
        pr = dict(ids=np.concatenate([rng.integers(0, 6_000_000, size=lo), rng.integers(0, 900, size=lo)]).astype(np.int64),
                  offsets=np.arange(2 * lo + 1, dtype=np.int32))
        print(f"[static] the largest: B={lo}", flush=True)
        ref, got = _run_pair(layer, pr, lo)
        assert np.array_equal(ref.view(np.uint32), got.view(np.uint32))
    finally:
        layer.close()


def test_static_forward_of_many_packs_at_the_limit():
    # 250 packs: the sums of the slices' distinct keys, 16 bytes and more a pack, do not count against the scratch's limit,
    # which is a call of 807 935 occurrences from what such a plan needs otherwise
    from paper_2204_04903_amd.layer import PackedEmbedding
    T, B, nnz = 250, 3231, 807_935
    layer = PackedEmbedding([(50, 1 + t, 0) for t in range(T)], [(t, 0) for t in range(T)])
    try:
        rng = np.random.default_rng(904)
        for W in layer.W:
            W.uniform_(-1.0, 1.0)
        offsets = np.arange(T * B + 1, dtype=np.int32)
        offsets[-1] = nnz                             # (one-hot but for the last bag)
        print(f"[static] many packs: B={B} nnz={nnz}", flush=True)
        ref, got = _run_pair(layer, dict(ids=rng.integers(0, 50, size=nnz).astype(np.int64), offsets=offsets), B)
        assert np.array_equal(ref.view(np.uint32), got.view(np.uint32))
    finally:
        layer.close()
