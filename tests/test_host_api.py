"""Host-side checks that need no GPU: the library loads, exports every symbol
the header declares, builds plans like the oracle does and rejects bad
arguments with status codes."""
import ctypes
import os
import re

import numpy as np
import pytest

import synth
from oracle import pk_oracle as orc
from paper_2204_04903_amd import binding as pk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "pk.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(pk_[a-z_]+)\s*\(", header))
    assert declared == set(pk.EXPORTS)
    L = ctypes.CDLL(pk.LIB_PATH)
    for name in declared:
        assert hasattr(L, name), name


@pytest.mark.parametrize("idx", [1, 2, 3, 4, 5])
def test_plan_matches_oracle_plan(idx):
    wl = synth.config(idx)
    tables = [(t.rows, t.dim, t.dtype) for t in wl.tables]
    fields = [(f.table, f.pool) for f in wl.fields]
    ref = orc.plan(tables, fields)
    plan = pk.pk_plan_create(tables, fields)
    try:
        assert pk.pk_plan_num_packs(plan) == ref.n_packs
        assert pk.pk_plan_out_dim(plan) == ref.out_dim
        for p in range(ref.n_packs):
            info = pk.pk_plan_pack_info(plan, p)
            assert (info["dim"], info["dtype"], info["total_rows"]) == (ref.pack_dim[p], ref.pack_dtype[p], ref.pack_rows[p])
            assert pk.pk_plan_pack_fields(plan, p) == list(ref.pack_fields[p])
            assert info["key_bytes"] == 4
        for t in range(len(tables)):
            assert pk.pk_plan_table_slot(plan, t) == (ref.table_pack[t], ref.table_base[t])
        for f in range(len(fields)):
            assert pk.pk_plan_field_col(plan, f) == ref.field_col[f]
        B = wl.batch
        nnz = int(wl.expected_nnz())
        assert pk.pk_workspace_bytes(plan, B, nnz) > 24 * nnz
    finally:
        pk.pk_plan_destroy(plan)


def test_sharded_plan_matches_oracle_plan():
    # Eq. 1 shard split: same packs, table slots and field columns as the oracle's plan
    rng = np.random.default_rng(9)
    dims = [8] * 8 + [32] * 8 + [16] * 3
    tables = [(int(rng.integers(10, 99)), d, 0) for d in dims]
    fields = [(t, t % 2) for t in range(len(tables))] + [(3, 0), (12, 1)]
    for kw in (dict(max_shards=8), dict(max_shards=3, field_volume=[float(v) for v in rng.integers(1, 50, len(fields))])):
        ref = orc.plan(tables, fields, **kw)
        plan = pk.pk_plan_create(tables, fields, **kw)
        try:
            assert pk.pk_plan_num_packs(plan) == ref.n_packs
            for p in range(ref.n_packs):
                info = pk.pk_plan_pack_info(plan, p)
                assert (info["dim"], info["dtype"], info["total_rows"]) == (ref.pack_dim[p], ref.pack_dtype[p], ref.pack_rows[p])
                assert list(pk.pk_plan_pack_fields(plan, p)) == list(ref.pack_fields[p])
            for t in range(len(tables)):
                assert pk.pk_plan_table_slot(plan, t) == (ref.table_pack[t], ref.table_base[t])
            for f in range(len(fields)):
                assert pk.pk_plan_field_col(plan, f) == ref.field_col[f]
        finally:
            pk.pk_plan_destroy(plan)


def test_plan_rejects_bad_arguments():
    def status(fn):
        with pytest.raises(pk.PkError) as e:
            fn()
        return e.value.status
    assert status(lambda: pk.pk_plan_create([(0, 8, 0)], [(0, 0)])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 0, 0)], [(0, 0)])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 8, 7)], [(0, 0)])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)], [(1, 0)])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)], [(0, 5)])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)], [])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 512, 0)], [(0, 0)])) == pk.PK_EOVERFLOW
    assert status(lambda: pk.pk_plan_create([(2 ** 31, 8, 0), (2 ** 31, 8, 0)], [(0, 0)])) == pk.PK_EOVERFLOW
    assert "rows" in pk.pk_last_error()
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)], [(0, 0)], interleave_groups=9)) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)], [(0, 0)], field_volume=[-1.0])) == pk.PK_EINVAL
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)], [(0, 0)] * 4097)) == pk.PK_EOVERFLOW
    assert status(lambda: pk.pk_plan_create([(10, 8, 0)] * 4097, [(0, 0)])) == pk.PK_EOVERFLOW


def test_forward_rejects_bad_arguments_before_touching_the_gpu():
    plan = pk.pk_plan_create([(100, 8, 0)], [(0, 0), (0, 1)], max_batch=64, max_nnz=1000)
    try:
        need = pk.pk_workspace_bytes(plan, 16, 100)
        fake = 0x10000   # never dereferenced: every call below fails validation first

        def fwd(**kw):
            a = dict(W=[fake], ids=fake, offsets=fake, B=16, nnz=100, out=fake, stride=16, ws=fake, ws_bytes=need)
            a.update(kw)
            with pytest.raises(pk.PkError) as e:
                pk.pk_forward(plan, a["W"], a["ids"], a["offsets"], a["B"], a["nnz"], a["out"], a["stride"],
                              a["ws"], a["ws_bytes"])
            return e.value.status
        assert fwd(B=0) == pk.PK_ESHAPE
        assert fwd(B=65) == pk.PK_ESHAPE
        assert fwd(nnz=1001) == pk.PK_ESHAPE
        assert fwd(nnz=-1) == pk.PK_ESHAPE
        assert fwd(ws=None) == pk.PK_EINVAL
        assert fwd(ws=fake + 4) == pk.PK_EWORKSPACE
        assert fwd(ws_bytes=need - 1) == pk.PK_EWORKSPACE
        assert fwd(ids=None) == pk.PK_EINVAL
        assert fwd(W=[None]) == pk.PK_EINVAL
        assert fwd(stride=15) == pk.PK_ESHAPE
        with pytest.raises(pk.PkError) as e:
            pk.pk_backward_update(plan, [fake], [fake], fake, 15, 16, 100, 0.01, 1e-8, fake, need)
        assert e.value.status == pk.PK_ESHAPE
        with pytest.raises(pk.PkError) as e:
            pk.pk_backward_update(plan, [fake], [None], fake, 16, 16, 100, 0.01, 1e-8, fake, need)
        assert e.value.status == pk.PK_EINVAL
        with pytest.raises(pk.PkError):
            pk.pk_workspace_bytes(plan, 16, 2 ** 31)
    finally:
        pk.pk_plan_destroy(plan)


def test_generator_is_reproducible_and_shaped_like_the_configs():
    wl = synth.config(3, batch=32, row_scale=0.001, n_fields=10)
    a, b = synth.make_batch(wl, 2), synth.make_batches(wl, 3)[2]
    assert np.array_equal(a.ids, b.ids) and np.array_equal(a.offsets, b.offsets) and np.array_equal(a.grad_out, b.grad_out)
    assert a.offsets[0] == 0 and a.offsets[-1] == a.nnz and (np.diff(a.offsets) >= 1).all()
    r1 = synth.table_rows(wl, 0, rows=[3, 1, 3])
    r2 = synth.table_rows(wl, 0, row0=0, n=5)
    assert np.array_equal(r1[0], r2[3]) and np.array_equal(r1[1], r2[1]) and np.array_equal(r1[0], r1[2])
    big = synth.table_rows(synth.config(2), 0, row0=0, n=20000)
    assert abs(float(big.std()) - 0.01) < 2e-4 and abs(float(big.mean())) < 2e-4


def test_hybrid_hash_calls_reject_bad_arguments_before_touching_the_gpu():
    plan = pk.pk_plan_create([(100, 8, 0)], [(0, 0)])
    try:
        fake = 0x10000   # never dereferenced: every call below fails validation first
        good = dict(W_cold=fake, A_cold=fake, W_hot=fake, A_hot=fake, slot_of=fake, hot_row=fake, fcounter=fake, hot_rows=10)
        assert pk.pk_hh_scratch_bytes(plan, [good]) > 0
        assert pk.pk_hh_scratch_bytes(plan, [dict(good, hot_rows=1000)]) > pk.pk_hh_scratch_bytes(plan, [good])

        def status(fn):
            with pytest.raises(pk.PkError) as e:
                fn()
            return e.value.status
        for missing in ("W_cold", "A_cold", "slot_of", "fcounter", "W_hot"):
            bad = dict(good, **{missing: None})
            assert status(lambda: pk.pk_hh_forward(plan, [bad], fake, fake, 4, 4, fake, 8, fake, 1 << 20)) == pk.PK_EINVAL
        assert status(lambda: pk.pk_hh_forward(plan, [dict(good, hot_rows=-1)], fake, fake, 4, 4, fake, 8, fake, 1 << 20)) == pk.PK_EINVAL
        need = pk.pk_workspace_bytes(plan, 4, 4)
        assert status(lambda: pk.pk_hh_end_iteration(plan, [good], 0, 1, 0, 4, 4, fake, need, fake, 1 << 30)) == pk.PK_EINVAL
        assert status(lambda: pk.pk_hh_end_iteration(plan, [good], 0, 1, 1, 4, 4, fake, need, fake, 16)) == pk.PK_EWORKSPACE
        assert pk.pk_hh_hot_count(plan, 0) == 0
    finally:
        pk.pk_plan_destroy(plan)


def test_micro_batch_size_follows_eq2():
    # Sec. III-C, Eq. 2 with the two resources the layer has: the activations (8 * out_dim bytes per sample,
    # an exact ratio, compared with the oracle's Eq. 2) and the workspace (whose cost per sample comes from
    # the layout: checked through what it must guarantee).
    wl = synth.config(2)
    plan = pk.pk_plan_create([(t.rows, t.dim, t.dtype) for t in wl.tables], [(f.table, f.pool) for f in wl.fields])
    try:
        B, nnz = wl.batch, wl.batch * wl.n_fields
        out_dim = pk.pk_plan_out_dim(plan)
        assert pk.pk_micro_batch_size(plan, B, nnz, 0, 0) == B
        for bound in (8 * out_dim * 1000, 8 * out_dim * 1000 + 17, 8 * out_dim - 1, 10 ** 12):
            assert pk.pk_micro_batch_size(plan, B, nnz, 0, bound) == orc.micro_batch_size(B, [bound], [8 * out_dim])
        full = pk.pk_workspace_bytes(plan, B, nnz)
        fixed = pk.pk_workspace_bytes(plan, 1, 0)
        assert pk.pk_micro_batch_size(plan, B, nnz, full, 0) == B
        assert pk.pk_micro_batch_size(plan, B, nnz, fixed, 0) == 0
        for frac in (0.9, 0.6, 0.45, 0.38):
            bound = int(full * frac)
            bs = pk.pk_micro_batch_size(plan, B, nnz, bound, 0)
            assert 0 < bs < B
            assert pk.pk_workspace_bytes(plan, bs, -(-nnz * bs // B)) <= bound          # it fits
            M = -(-B // bs)
            assert bs == -(-B // M)                                                     # an even cut
            if M > 1:                                                                   # and fewer micro-batches would not fit
                bigger = -(-B // (M - 1))
                assert pk.pk_workspace_bytes(plan, bigger, -(-nnz * bigger // B)) > bound
            # both bounds: the smaller of the two sizes decides
            both = pk.pk_micro_batch_size(plan, B, nnz, bound, 8 * out_dim * 100)
            assert both == min(bs, orc.micro_batch_size(B, [8 * out_dim * 100], [8 * out_dim]))
        with pytest.raises(pk.PkError):
            pk.pk_micro_batch_size(plan, 0, nnz, 0, 0)
        with pytest.raises(pk.PkError):
            pk.pk_micro_batch_size(0, B, nnz, 0, 0)
    finally:
        pk.pk_plan_destroy(plan)


@pytest.mark.parametrize("tables,n_fields,per_bag", [
    ([(1_000_000, 16, 0)] * 26, 26, 13),
    ([(1_000_000, 8, 0)], 1, 1),
    ([(400_000, 8, 0), (30_000, 16, 0)] * 500, 1000, 5),
    ([(500_000, 64, 1)] * 6, 6, 300),
    ([(140_000_000, 4, 0)] * 2, 4, 2),
])
def test_a_smaller_call_fits_a_larger_calls_workspace(tables, n_fields, per_bag):
    # callers size a workspace once, for their largest batch (MicroBatchPipeline does): wherever the tiles' size changes,
    # fewer bags or fewer IDs need no more room, and the size that Eq. 2 gives fits its bound after it is evened out
    plan = pk.pk_plan_create(tables, [(f % len(tables), f % 2) for f in range(n_fields)])
    try:
        B0 = -(-(1 << 19) // (n_fields * per_bag))                        # about where batches become large ones
        sizes = sorted({b for t in (32, 64, 128, 256, 512, 1024) for k in (1, 2, 3, 5, 40, 1023 // n_fields, 1024 // n_fields)
                        for b in (t * k - 1, t * k, t * k + 1) if b > 0} | {B0 - 1, B0, B0 + 1, 2 * B0, 3 * B0 + 1})
        nnzs = sorted({n_fields * b * per_bag // part for b in (B0, 3 * B0) for part in (1, 2, 7)} | {(1 << 19) - 1, 1 << 19})
        ws = np.array([[pk.pk_workspace_bytes(plan, b, n) for n in nnzs] for b in sizes], np.float64)
        assert (np.diff(ws, axis=0) >= 0).all() and (np.diff(ws, axis=1) >= 0).all()
        along = [pk.pk_workspace_bytes(plan, b, n_fields * b * per_bag) for b in sizes]
        assert along == sorted(along)
        for B in (B0 + 1, 2 * B0 + 1, 4 * B0 - 1):
            nnz = n_fields * B * per_bag
            for part in (1.5, 2, 2.3, 3, 4.1):
                bound = int(pk.pk_workspace_bytes(plan, B, nnz) / part)
                bs = pk.pk_micro_batch_size(plan, B, nnz, bound, 0)
                assert bs == 0 or pk.pk_workspace_bytes(plan, bs, -(-nnz * bs // B)) <= bound
    finally:
        pk.pk_plan_destroy(plan)


def test_calls_whose_positions_would_not_fit_32_bits_are_refused():
    # a kernel's last round counts up to 8192 positions past the last one
    plan = pk.pk_plan_create([(100, 8, 0)], [(0, 0)])
    try:
        for nnz in (2 ** 31 - 8191, 2 ** 31 - 1):
            need, fake = pk.pk_workspace_bytes(plan, 1, nnz), 0x10000
            for call in (lambda: pk.pk_forward(plan, [fake], fake, fake, 1, nnz, fake, 8, fake, need),
                         lambda: pk.pk_forward_dedup(plan, fake, fake, 1, nnz, fake, need, 0),
                         lambda: pk.pk_forward_pool(plan, [fake], 1, nnz, fake, 8, fake, need, 0),
                         lambda: pk.pk_backward_update(plan, [fake], [fake], fake, 8, 1, nnz, 0.01, 1e-8, fake, need)):
                with pytest.raises(pk.PkError) as e:
                    call()
                assert e.value.status == pk.PK_EOVERFLOW
    finally:
        pk.pk_plan_destroy(plan)


def test_forward_stages_reject_bad_arguments_before_touching_the_gpu():
    plan = pk.pk_plan_create([(100, 8, 0)], [(0, 0)])
    try:
        need = pk.pk_workspace_bytes(plan, 4, 4)
        with pytest.raises(pk.PkError) as e:
            pk.pk_forward_dedup(plan, 0x1000, 0, 4, 4, 0x1000, need, 0)          # offsets NULL
        assert e.value.status == pk.PK_EINVAL
        with pytest.raises(pk.PkError) as e:
            pk.pk_forward_dedup(plan, 0x1000, 0x1000, 4, 4, 0x1000, need - 1, 0)   # workspace too small
        assert e.value.status == pk.PK_EWORKSPACE
        with pytest.raises(pk.PkError) as e:
            pk.pk_forward_pool(plan, [0x1000], 4, 4, 0, 8, 0x1000, need, 0)      # out NULL
        assert e.value.status == pk.PK_EINVAL
        with pytest.raises(pk.PkError) as e:
            pk.pk_forward_pool(plan, [0x1000], 4, 4, 0x1000, 7, 0x1000, need, 0) # row stride below out_dim
        assert e.value.status == pk.PK_ESHAPE
        with pytest.raises(pk.PkError) as e:
            pk.pk_forward_pool(plan, [0], 4, 4, 0x1000, 8, 0x1000, need, 0)      # W[0] NULL
        assert e.value.status == pk.PK_EINVAL
    finally:
        pk.pk_plan_destroy(plan)


def test_split_batch_keeps_every_bag_and_gradient_row():
    # the micro-batches of D-Interleaving are a re-layout of the batch: every bag of every field, and every
    # sample's gradient row, turns up once, in sample order
    wl = synth.config(3, batch=37, row_scale=0.01, n_fields=5)
    b = synth.make_batch(wl, 0)
    for n_micro in (1, 4, 37, 100):
        parts = synth.split_batch(b, wl.n_fields, wl.batch, n_micro)
        sizes = [p.grad_out.shape[0] for p in parts]
        assert sum(sizes) == wl.batch and max(sizes) - min(sizes) <= 1 and min(sizes) >= 1
        assert sum(p.nnz for p in parts) == b.nnz
        assert np.array_equal(np.concatenate([p.grad_out for p in parts]), b.grad_out)
        first = 0
        for p in parts:
            Bm = p.grad_out.shape[0]
            assert p.offsets[0] == 0 and p.offsets[-1] == p.nnz and len(p.offsets) == wl.n_fields * Bm + 1
            for f in range(wl.n_fields):
                for s in range(Bm):
                    g, G = f * Bm + s, f * wl.batch + first + s
                    assert np.array_equal(p.ids[p.offsets[g]:p.offsets[g + 1]], b.ids[b.offsets[G]:b.offsets[G + 1]])
            first += Bm


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "ONE GPU" in r.stderr and r.stdout.strip() == ""
