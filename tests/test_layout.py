"""The workspace's layout on the host: the slices' sums of every pack fall into their array however the packs' slices are
dealt, arrays do not overlap, a smaller call's workspace fits a larger call's, and near the end of a scratch that cannot grow
the stored counts are left out and the sums moved together before a call is refused."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2204_04903_amd", "csrc")

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include "pk_internal.h"
using namespace pk;
namespace pk { void destroy_device_state(pk_plan*) {} }
#define CHECK(c) do { if (!(c)) { std::printf("%s: line %d, plan %d, B %d nnz %lld\n", #c, __LINE__, it, B, (long long)nnz); return 1; } } while (0)
int main()
{
    std::mt19937 r(11);
    auto law = [&](double a, double b) { return std::exp(std::log(a) + (std::log(b) - std::log(a)) * (r() / 4294967296.0)); };
    int together = 0, left_out = 0;
    for (int it = 0; it < 400; ++it) {
        const int T = (int)law(1, 1500), dims = (int)law(1, 200);
        const double lo = law(1, 1e6), hi = law(lo, 4e6);
        std::vector<pk_table_desc> t(T);
        std::vector<pk_field_desc> f(T);
        for (int i = 0; i < T; ++i) {
            t[i] = {(int64_t)law(lo, hi * 1.0001), 1 + i % dims, PK_F32};
            f[i] = {i, r() % 3 ? PK_SUM : PK_MEAN};
        }
        pk_plan_opts o{};
        o.debug = 2;
        pk_plan* p = nullptr;
        int B = (int)law(1, 20000);
        int64_t nnz = (int64_t)law(1, 3e6);
        CHECK(pk_plan_create(t.data(), T, f.data(), T, &o, &p) == PK_OK);
        const Layout L = make_layout(p, B, nnz), least = make_layout(p, B, nnz, 0);
        const int P = (int)p->packs.size();
        // the packs' slices as many as there can be, and as few: the sums' last word stands inside their array
        for (int few = 0; few < 2; ++few) {
            int64_t first = 0;
            for (int q = 0; q < P; ++q) {
                int64_t n = 0;
                for (const TableMeta& tm : p->sort_tables)
                    if (tm.pack == q) n += few ? ((int64_t)tm.rows + (1 << L.log_max) - 1) >> L.log_max : slice_count_max(tm.rows, nnz, kSliceOccLarge, L.log_max);
                if (first + n > L.n_slices) n = L.n_slices - first;
                if (n > 0) CHECK(first / kSumFan + q + (n - 1) / kSumFan < L.n_groups);
                first += n;
            }
        }
        for (const Layout* l : {&L, &least}) {
            CHECK(l->nu_group >= l->slice_nu + (size_t)l->n_slices * 4);
            CHECK(l->long_list >= l->nu_group + (size_t)l->n_groups * l->sum_stride * 16);
            CHECK(l->clear_begin + l->clear_bytes >= l->long_list + 4);
            CHECK(l->slice_cursor >= l->clear_begin + l->clear_bytes && l->slice_cursor >= l->long_list + (size_t)(1 + l->n_long_max) * 4);
            CHECK(l->slice_info >= l->slice_cursor + (size_t)l->n_slices * 4);
        }
        CHECK(L.sum_stride == kSumStride && least.sum_stride == 1);
        CHECK(make_layout(p, std::max(B / 2, 1), nnz / 2).total <= L.total && make_layout(p, B, nnz - nnz / 3).total <= L.total);
        // a scratch of every size from the least to the full
        for (int k = 0; k < 40; ++k) {
            const size_t room = least.total + (size_t)((L.total - least.total) * (k / 40.0));
            const Layout m = make_layout(p, B, nnz, room);
            CHECK(m.total <= room);
            CHECK(m.tile_hist + (size_t)m.tile_hist_stride * ((int64_t)T * ((B + m.bags_per_tile - 1) / m.bags_per_tile)) * 4 <= room);
            together += m.sum_stride == 1;
            left_out += L.tile_hist_stride && !m.tile_hist_stride;
        }
        CHECK(make_layout(p, B, nnz, least.total - 1).total > least.total - 1);
        pk_plan_destroy(p);
    }
    if (!together || !left_out) { std::printf("nothing near the end: %d %d\n", together, left_out); return 1; }
    return 0;
}
"""


def test_layout(tmp_path):
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src),
                           os.path.join(CSRC, "pk_plan.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
