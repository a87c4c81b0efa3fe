"""How a backward launch takes its keys (pk_internal.h): sizes that are close get batches that are close, narrow rows and
layers whose wide rows are few keep to handfuls.  On the host, as the launch uses the same code."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "pk_internal.h"
using namespace pk;
static KeyShare layer(int wide_dim, int n_wide, int dim, int n, uint32_t rows, int64_t ids)
{
    KeyShare s;
    for (int i = 0; i < n_wide; ++i) s.add(wide_dim, rows, 1, ids / (n + n_wide));
    for (int i = 0; i < n; ++i) s.add(dim, rows, 1, ids / (n + n_wide));
    return s;
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main()
{
    for (int handful = 1; handful <= 64; handful *= 2) {
        int before = keys_per_batch(0, handful);
        for (int64_t d = 0; d < ((int64_t)1 << 31); d += d / 100 + 1) {
            const int k = keys_per_batch(d, handful);
            CHECK(k >= before && k - before <= handful && k % handful == 0);       // a handful at a time
            CHECK(k >= handful && k <= 64 && k <= 8 * handful && k >= (8 * handful < 16 ? 8 * handful : 16));
            before = k;
        }
        CHECK(before == (8 * handful < 64 ? 8 * handful : 64));
    }
    for (int k = 8; k <= 64; ++k) {
        const uint32_t word = key_batch_word(k);
        CHECK(key_batch_size(word) == k && key_batches(0, word) == 0);
        for (int64_t u = 1; u <= kNnzMax; u = u == kNnzMax ? u + 1 : std::min<int64_t>(kNnzMax, u + u / 1000 + 1)) {
            const int64_t n = key_batches((int)u, word), exact = (u + k - 1) / k;
            CHECK(n >= exact && n <= exact + u / (1 << 24) + 1);
            CHECK(n == exact || u >= 1 << 16);
            CHECK((n + 7) / 8 * 7 * k < ((int64_t)1 << 31));         // where the last XCD's eighth starts
        }
    }
    CHECK(!keys_in_batches(layer(64, 1, 8, 7, 1000000, 1600000)));                 // wide rows in an eighth of the fields
    CHECK(keys_in_batches(layer(64, 1, 8, 2, 1000000, 1600000)));                  // ... in a third
    CHECK(!keys_in_batches(layer(64, 26, 0, 0, 1000000, 200000)) && keys_in_batches(layer(64, 26, 0, 0, 1000000, 1700000)));
    CHECK(!keys_in_batches(layer(32, 26, 0, 0, 1000000, 1700000)) && keys_in_batches(layer(32, 26, 0, 0, 1000000, 3400000)));
    CHECK(!keys_in_batches(layer(16, 100, 0, 0, 1000000, 3400000)) && keys_in_batches(layer(16, 100, 0, 0, 1000000, 8600000)));
    CHECK(keys_in_batches(layer(16, 500, 8, 500, 500000, 11000000)));
    CHECK(!keys_in_batches(layer(8, 200, 0, 0, 1000000, 21000000)) && !keys_in_batches(layer(4, 200, 0, 0, 1000000, 21000000)));
    CHECK(!keys_in_batches(layer(64, 20, 0, 0, 10000, 3000000)));                  // keys of many occurrences
    CHECK(!keys_in_batches(KeyShare{}));
    return 0;
}
"""


def test_key_batches_rule(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2204_04903_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
