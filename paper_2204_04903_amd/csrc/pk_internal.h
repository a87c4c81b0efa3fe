// Internal declarations shared by the host plan (pk_plan.cpp) and the device
// code (pk_device.hip).  Not part of the C ABI.
#pragma once

#include <cstdint>
#include <cstddef>
#include <algorithm>
#include <string>
#include <vector>

#include "pk.h"

namespace pk {

// The backward pass handles a key by its number of occurrences (dev_adagrad.h).
constexpr int kColdMax   = 8;      // keys with at most this many occurrences: one lane group per key
constexpr int kLongMin   = 256;    // up to this many: one wavefront per key; above: a block per piece of the key
constexpr int kMarkStep  = 256;    // every kMarkStep-th position of the grouped occurrences names its key: how long keys are found
constexpr int kPiece     = 1024;   // occurrences per piece of a long key (the last piece takes what is left, up to twice that)
static_assert(kMarkStep <= kLongMin && kPiece > kLongMin, "every piece of a long key holds a marked position");
// Occurrences of a call.  Kernels walk positions in 32 bits and in rounds: a round of up to kRoundMax positions can still
// be counted past the last position.  Longer ones count what is left (Rounds).
constexpr int kRoundMax = 8192;
constexpr int64_t kNnzMax = ((int64_t)1 << 31) - kRoundMax;
constexpr size_t kAlign = 256;

// The dedup cuts every table's key range into slices of 2^k keys; one block owns a slice and keeps
// the slice's bitmap, its popcount prefix and the occurrence counters of its distinct keys in LDS.
// Two shapes of slice block: 1024 threads for slices of up to 128 K keys (small batches, where a
// block scans its table's IDs itself, and large batches with tables too long for the other shape),
// and 512 threads for slices of up to 64 K keys (large batches: several blocks per compute unit hide the latency
// of the few dependent memory accesses a slice makes).
constexpr int kSliceLogMin = 10;           // 1 K keys
constexpr int kSliceLogMax = 17;           // 128 K keys: 4096 bitmap words
constexpr int kSliceLogFine = 16;          // 64 K keys: 2048 bitmap words
constexpr int kSliceWordsMax = 1 << (kSliceLogMax - 5);
// Occurrences per slice aimed at when the occurrences are partitioned (2048: bf16 sequences 597 us a step, 571).  Key ranges
// are powers of two, so even IDs give up to twice that, more than the 4096 that a block keeps in registers: 61 to 90 % of the
// slices are kept in skewed layers of 1 to 21 M IDs, with 41 to 70 % of the records, and all of them where a thousand tables
// share 3 M IDs.
constexpr int kSliceOccLarge = 3072;
constexpr int kLongSlice = 16384;          // records from which a slice is listed, up to kLongSlicesMax of them (8192: the same, but a block more per 8192 records)
constexpr int kLongSlicesMax = 256;
constexpr int32_t kListedFlag = 1 << 30;   // in SliceInfo::table
constexpr int kSumFan = 64;                // slices whose distinct keys add up in one word (SliceSums)
constexpr int32_t kSumStride = 16;         // 64-bit words of a cache line: the sums of the slices' distinct keys stand this far apart
constexpr int64_t kTilesMin = 1024;         // tiles that a launch of the keys and scatter kernels should have at least
// Counts per (tile, slice) kept from the keys to the scatter kernel: room for one per occurrence and kCountRoomMin
// more (a launch cut to kTilesMin tiles has up to twice as many, each with nnz / kSliceOccLarge + 1 slices), no more
// than kCountRoomMax.
constexpr int64_t kCountRoomMin = 2 * kTilesMin, kCountRoomMax = (int64_t)8 << 20;
constexpr int64_t kSmallNnz = 1 << 19;     // below this many occurrences the forward pass is one launch
constexpr int kSmallSlicesMax = 4096;      // ... if it has no more slices than this (descriptors the library owns)
constexpr int kTableSlicesMax = 8192;      // slices per table (their counters are staged in LDS): rows <= 2^30
constexpr int64_t kFineRowsMax = (int64_t)4096 << kSliceLogFine;   // longest table the 64 K-key shape is used with

#if defined(__HIPCC__)
#define PK_HD __host__ __device__
#else
#define PK_HD
#endif

// n positions in rounds of N, by what is left of them, which no round length takes out of 32 bits.
template <int N>
struct Rounds {
    int base = 0, left;                  // the round's first position; positions from there on
    PK_HD explicit Rounds(int n) : left(n) {}
    PK_HD bool any() const { return left > 0; }
    PK_HD void next() { base = (int)((unsigned)base + (unsigned)N); left -= N; }
};

// Slices of one table for a partitioned call: 2^log_keys keys each, n of them.  The aim is `target`
// occurrences per slice, given how many occurrences the table's fields have in THIS batch (the
// offsets say so: a layer's fields differ widely in length, Sec. II-B).  The kernels derive the cut
// from the offsets; the host only needs the most slices a batch can give (slice_count_max).
struct SliceGeom { int32_t log_keys; int32_t n; };
constexpr int kSliceWantMax = 1024;        // slices asked for a table on account of its occurrences
PK_HD inline SliceGeom slice_geom(uint32_t rows, int64_t occ, int32_t target, int32_t log_max)
{
    int64_t want = (occ + target - 1) / target;
    if (want < 1) want = 1;
    if (want > kSliceWantMax) want = kSliceWantMax;
    const int64_t per = ((int64_t)rows + want - 1) / want;
    int lg = kSliceLogMin;
    while (lg < log_max && ((int64_t)1 << lg) < per) ++lg;
    SliceGeom g;
    g.log_keys = lg;
    g.n = (int32_t)(((int64_t)rows + ((int64_t)1 << lg) - 1) >> lg);
    return g;
}
// The most slices slice_geom gives a table of a batch with nnz occurrences: either the slices are as
// large as they may be (2^log_max keys), or there are at most as many as were asked for.
inline int32_t slice_count_max(uint32_t rows, int64_t nnz, int32_t target, int32_t log_max)
{
    const int64_t coarse = ((int64_t)rows + ((int64_t)1 << log_max) - 1) >> log_max;
    const int64_t fine = ((int64_t)rows + ((int64_t)1 << kSliceLogMin) - 1) >> kSliceLogMin;
    const int64_t want = std::min<int64_t>(kSliceWantMax, nnz / target + 1);
    return (int32_t)std::min(fine, std::max(coarse, want));
}

// Small batches: a table's keys in about `want` slices, none longer than a block's LDS bitmap.  Lists for 1, 2, 4
// ... 64 are made once, on the host, and a call takes the one that its occurrences per table ask for: a slice
// block scans all IDs of its table, so slices with few occurrences only add blocks to wait for, and one with
// more occurrences than it keeps in LDS reads the IDs three times.
constexpr int kSmallCuts = 7;
inline SliceGeom slice_geom_small(int64_t rows, int32_t want)
{
    const int64_t per = (rows + want - 1) / want;
    int lg = kSliceLogMin;
    while (lg < kSliceLogMax && ((int64_t)1 << lg) < per) ++lg;
    SliceGeom g;
    g.log_keys = lg;
    g.n = (int32_t)((rows + ((int64_t)1 << lg) - 1) >> lg);
    return g;
}
// Occurrences per slice aimed at, and blocks that the chip holds at once (two per CU): with more slices than those,
// the later ones only start when the first are through.
constexpr int64_t kSmallSliceOcc = 1024;
constexpr int64_t kSmallBlocks = 512;
inline int small_cut(int64_t nnz, int64_t n_tables)
{
    int cut = 0;
    while (cut + 1 < kSmallCuts && nnz > ((int64_t)kSmallSliceOcc * n_tables << cut) && (n_tables << (cut + 1)) <= kSmallBlocks) ++cut;
    return cut;
}

// How a backward launch takes its keys, by what its packs hold when every field has the batch's average of IDs: keys one
// handful a wavefront, or (large batches) batches of more that are sorted by their number of occurrences first.
// kernel times in us, handfuls then batches, 1.05-Zipf IDs of one-hot fields or 1.1-Zipf of bags of 10:
//   rows of 48 columns and more in a quarter of the fields: 60 48-column fields of 0.7 M IDs 62, 56; 64 columns, 1.3 M 126, 117; 26
//     one-hot fields of 64 columns 246, 242; of 0.2 M the same, of 0.1 M 23, 28 (hence kBatchNnz); a third of the fields
//     84, 80 (1.5 M); an eighth 62, 65 (the narrow rows' loss)
//   of 32 and more in half: 1.6 M 68, 70; 2.4 M 109, 105; 3.4 M 144, 135; one-hot 3.4 M 230, 226
//   of 16 and more in half: 3.4 M 108, 107 and one-hot 176, 183; 5.5 M 155, 151 and 271, 274; 8.6 M 238, 230; 21 M 505, 485; 1000
//     fields of 8 and 16 columns, 5.5 M 229, 226, 11 M 423, 408
//   of 8: 3.4 M 98, 106; 8.6 M 198, 203; 21 M 421, 427; of 4: 83, 90 and 373, 386: a handful is 32 or 64 keys there anyway
// Where tables have few rows for their IDs, keys have many occurrences each and there is little to sort (37 ragged fields of
// 3.0 M IDs, 46 % of them distinct at most: 202, 183; before dense stretches had their own wavefronts 193, and of 3.5 M, 43 %, 221 and 237).
struct KeyShare {
    int64_t fields = 0, wide16 = 0, wide32 = 0, wide48 = 0;    // fields; those with rows of 16, 32, 48 columns and more
    int64_t ids = 0, distinct = 0;                             // IDs; rows that they can be, at most
    void add(int dim, uint32_t rows, int64_t n_fields, int64_t n)      // a table, its fields, their IDs
    {
        fields += n_fields; ids += n; distinct += std::min<int64_t>(rows, n);
        wide16 += dim >= 16 ? n_fields : 0; wide32 += dim >= 32 ? n_fields : 0; wide48 += dim >= 48 ? n_fields : 0;
    }
};
constexpr int64_t kBatchNnz = 5 << 16, kBatchNnz32 = 3 << 20, kBatchNnz16 = 5 << 20;
inline bool keys_in_batches(const KeyShare& s)
{
    if (16 * s.distinct < 7 * s.ids) return false;
    return (4 * s.wide48 >= s.fields && s.ids >= kBatchNnz) || (2 * s.wide32 >= s.fields && s.ids >= kBatchNnz32) ||
           (2 * s.wide16 >= s.fields && s.ids >= kBatchNnz16);
}
// Keys in a batch: whole handfuls, as many as leave the launch kKeyBatches batches (6144 wavefronts run at a time, and there
// are fewer distinct rows than can be: 37 ragged fields of 1.05 M IDs, 0.67 M rows at most, in batches of 16, 24, 32, 64: 76.6, 75.1,
// 78.2, 80.7 us; of 2.3 M, 1.2 M 156, 153, 150, 162; of 3.0 M, 1.4 M 195, 193, 195, 216), 16 at least (of 0.5 M 50.1, in
// batches of 8 55.7), eight handfuls or 64 at most.
constexpr int64_t kKeyBatches = 36864;
inline int keys_per_batch(int64_t distinct, int handful)
{
    const int most = std::min(64, 8 * handful), least = std::min(most, std::max(handful, 16));
    const int64_t n = (distinct / kKeyBatches + handful / 2) / handful * handful;
    return (int)std::min<int64_t>(most, std::max<int64_t>(least, n));
}
// A batch's size (8 and more), and what takes the place of the division by it: floor(2^24 / size) + 1.  Where U is large, the
// batches of U keys are up to U / 2^24 + 1 too many, which have no keys; none for U = 0.
inline uint32_t key_batch_word(int size) { return (uint32_t)size | (((uint32_t)1 << 24) / (uint32_t)size + 1) << 8; }
PK_HD inline int key_batch_size(uint32_t word) { return (int)(word & 255); }
PK_HD inline int key_batches(int U, uint32_t word) { return (int)(((uint64_t)((uint32_t)U + (word & 255) - 1) * (word >> 8)) >> 24); }

// One slice of the small-batch cut, with all that its block needs of the plan; static, device side, in
// (pack, table, slice) order.
struct SmallSlice {
    int32_t table;           // index in the table list
    int32_t idx;             // slice of the table
    int32_t log_keys;
    int32_t n_table_slices;
    int32_t pack_first;      // the pack's first slice
    int32_t is_last;         // the pack's last slice
    int32_t pack;
    int32_t field_begin, n_fields;    // the table's fields in the table field list
    uint32_t key_lo, rows;   // the table's first key inside its pack, its rows
    int32_t dim, wide;       // of the pack: dimension; entries carry bag lengths
    int32_t first_slot, pack_fields;  // the pack's first slot, its fields
    int32_t slot0, field0, col0, pool0;   // the table's first field: slot (over all packs), index, column, pooling
    int32_t pad;
    uint64_t magic;          // FieldMeta::magic
};

// Per field, device side (indexed by field index).
struct FieldMeta {
    uint32_t base_row;   // first row of the field's table inside its pack
    uint32_t rows;       // rows of the field's table
    int32_t  col;        // first output column of the field
    int32_t  pack;
    int32_t  slot;       // rank of the field among its pack's fields
    int32_t  pool;       // PK_SUM / PK_MEAN
    int32_t  stable;     // the field's table in the (pack, first key) ordered table list
    int32_t  pad;
    uint64_t magic;      // floor((2^64 - 1) / rows): folds an ID without a division
};

// Per pack, device side, static.
struct PackMeta {
    int32_t dim;
    int32_t dtype;
    int32_t n_fields;
    int32_t first_slot;      // index of the pack's slot 0 in the slot-ordered arrays
    int32_t has_mean;
    int32_t first_stable;    // index of the pack's first table in the (pack, key) ordered table list
    int32_t n_stables;       // tables of the pack that some field reads
    int32_t pad;
};

// A table that at least one field reads, and those fields; static, device side,
// listed in (pack, first key) order.
struct TableMeta {
    int32_t pack;
    uint32_t key_lo;         // first key of the table inside its pack
    uint32_t rows;
    int32_t field_begin;     // range in the table field list
    int32_t field_end;
    uint32_t word_base;      // first word of the table's bitmap and rank samples (a multiple of 4)
    int32_t pad[2];
};

// What the inverse kernel needs of a (pack, slot): static, device side, in slot order.
struct SlotMeta {
    uint32_t key_lo;         // first key of the slot's table inside its pack
    uint32_t word_base;      // where the table's bitmap starts
    uint32_t rows;           // rows of the table
    int32_t  pack;
};

// The cut of one table for the batch at hand (written by the keys kernel, read by the kernels after it).
struct TableCut {
    int32_t log_keys;        // 2^log_keys keys per slice
    int32_t n;               // slices of the table
    int32_t first;           // the table's first slice (slices are numbered over all packs)
    int32_t occ;             // occurrences of the table's fields in this batch
};

// One slice as the partitioned path hands it to the slice kernel (written by the scan kernel).
struct SliceInfo {
    int32_t table;           // index in the table list
    int32_t idx;             // slice of the table
    int32_t start;           // position of the slice's first record in the records (all packs)
    int32_t count;           // records
};

// Per pack, device side, rewritten by every forward call.
struct PackState {
    int32_t nnz;        // occurrences in the pack
    int32_t start;      // position of the pack's first occurrence in the packed order
    int32_t n_unique;
    int32_t error;      // bit 0: offsets rejected; bit 1: a scan waited too long
    int32_t first_slice;    // partitioned path: the pack's first slice
    int32_t pad[3];
};

struct Pack {
    int32_t dim = 0, dtype = 0;
    int64_t rows = 0;
    bool has_mean = false;
    std::vector<int32_t> tables;
    std::vector<int32_t> fields;
    int32_t first_slot = 0;
    int32_t first_stable = 0, n_stables = 0;
};

// Byte offsets of the workspace's arrays for one (plan, B, nnz).
struct Layout {
    size_t state, packed_offsets, keys, inverse, seg_ent, marks, unique, seg, ghot, ticket,
           clear_begin, slice_total, slice_nu, nu_group, long_list, slice_cursor, slice_info, tgeom, fscan, tile_hist, rec, bitmap, total;
    size_t clear_bytes;          // what the partitioned path clears before its first kernel: per-pack state,
                                 // slice totals and distinct-key counts, contiguous from `clear_begin`
    int32_t n_long_max;          // slices of many records that can be listed
    int32_t n_groups;            // groups of kSumFan slices, with room for a started one per pack
    int32_t sum_stride;          // 64-bit words from one group's sum to the next
    size_t sums_least;           // bytes of the sums side by side
    int32_t n_slices;            // slices of all tables for this call
    int32_t max_table_slices;    // most slices any table has
    int32_t log_max;             // partitioned path: largest slice (log2 of its keys) of this call
    int32_t dmax;
    int32_t bags_per_tile;       // bags per tile of the keys and scatter kernels
    int32_t tile_hist_stride;    // entries per tile of the stored per-slice counts (0: not stored, the scatter kernel counts again)
    int32_t small_cut;           // the cut of a small batch
    bool small;                  // the forward pass's dedup is one launch (every slice block scans its table's IDs)
};

}  // namespace pk

struct pk_plan {
    std::vector<pk_table_desc> tables;
    std::vector<pk_field_desc> fields;
    pk_plan_opts opts{};
    std::vector<pk::Pack> packs;
    std::vector<int32_t> table_pack;
    std::vector<int64_t> table_base;
    std::vector<int32_t> field_pack, field_slot;
    std::vector<int64_t> field_col;
    std::vector<int32_t> slot_field;      // fields in (pack, slot) order
    std::vector<pk::TableMeta> sort_tables;   // tables with fields, in (pack, first key) order
    std::vector<int32_t> table_fields;        // per entry of sort_tables: the fields that read it
    std::vector<pk::SmallSlice> small_slices[pk::kSmallCuts];   // the cuts the one-launch forward pass chooses from
    int64_t small_count[pk::kSmallCuts] = {};                   // their slices (above kSmallSlicesMax the list is not made)
    int64_t out_dim = 0;
    bool any_mean = false;
    int64_t bitmap_words = 0;             // all tables' bitmaps with their rank samples
    int32_t max_table_fields = 0;         // most fields reading one table
    int32_t dmax = 0;
    void* device_state = nullptr;         // owned by pk_device.hip (metadata upload, events)
    uint64_t serial = 0;                  // distinguishes plans, also when one is created where another was freed
};

namespace pk {
void set_error(const std::string& msg);
pk_status fail(pk_status s, const std::string& msg);
// `room`: bytes that the workspace must fit, where the caller cannot give more (what is only kept to save time is left out)
Layout make_layout(const pk_plan* plan, int32_t B, int64_t nnz, size_t room = ~(size_t)0);
void destroy_device_state(pk_plan* plan);   // defined in pk_device.hip
}  // namespace pk
