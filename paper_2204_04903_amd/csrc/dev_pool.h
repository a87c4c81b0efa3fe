// H3-H5: gather + pool + concatenate, and the kernel in which small batches share the dedup's launch.
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.

// ---------------------------------------------------------------------------
// H3+H4+H5: Gather and SegmentReduction (Sec. II-D) fused (K-Packing, Sec. III-B: both are memory-bound), all
// packs in one launch.  A lane group holds a row, four columns a lane (dev_rows.h); the concatenation of the
// fields of a sample is the write address.
//
// A wavefront takes a tile of consecutive bags of one field, a lane group a run of consecutive bags of it.
// The group walks the run's POSITIONS, R at a time, whatever bags they belong to: the keys of a round are two
// 16-byte reads, its R rows are in flight together, and a bag's sum is written when its last position has been
// added.  So one-hot bags keep as many rows in flight as long ones, and what a group waits for in vain is
// only the unevenness of whole runs.  The next round's keys are asked for before this round's rows are used.
// A field of sequences (kSeqAvg IDs per bag or more on average) is left to the cooperating wavefronts at the
// end of the grid: there all groups of a wavefront share a bag.
// Sums are kept in double and rounded once, when the bag is written: one fp32 accumulator loses a bit of every
// addition (bags of 25 normal weights: 1.4 times the error of adding four rows pairwise first, of 500: twice).
// ---------------------------------------------------------------------------
constexpr int kSeqAvg = 64;      // IDs per bag from which a field's bags take a whole wavefront each
constexpr int kRunMax = 8;       // most bags in a lane group's run
constexpr int kPoolPacks = 16;   // packs of one launch

struct PoolPack {
    const void* W; HotView hv; const int32_t* slot_field;
    uint32_t rows, po_begin;         // rows of the pack's table; where its packed offsets start
    int32_t D, sh, kind;             // dimension; log2 of the lanes per row; 1: bf16, 2: dimension below four
    int32_t n_fields, run, tiles;    // fields; bags per group; tiles per field
    int32_t item_begin, p;           // first tile of the pack among the launch's; pack
};
struct PoolJob {
    PoolPack pack[kPoolPacks];
    int32_t n_packs, B, n_items, coop_waves, n_fields;     // (fields of the plan)
    float* out; int64_t out_stride;
    const FieldMeta* fmeta;
    const uint32_t* keys; const int32_t* po; const PackState* st;          // from the workspace, or (small batches,
    const int64_t* ids; const int32_t* offsets; int64_t nnz;               // where the pooling runs beside the dedup)
};                                                                         // the caller's IDs, hashed here the same way

// keys of R consecutive positions from q on, without those past the pack's (or the IDs') end
template <bool IDS, int R>
struct KeySrc {
    const uint32_t* keys; const int64_t* ids; int n;
    uint32_t base, rows, last_row; uint64_t magic;
    __device__ __forceinline__ KeySrc(const PoolJob& job, const PoolPack& k, const FieldMeta& m)
    {
        const PackState* st = IDS ? nullptr : as_global(job.st) + k.p;
        n = IDS ? (int)job.nnz : st->nnz;
        keys = IDS ? nullptr : as_global(job.keys) + st->start;
        ids = as_global(job.ids);
        base = m.base_row; rows = m.rows; magic = m.magic; last_row = k.rows - 1;
    }
    __device__ __forceinline__ void raw(int q, uint32_t (&v)[IDS ? 2 * R : R]) const
    {
        if constexpr (IDS) {
            if (q + R <= n) {
#pragma unroll
                for (int i = 0; i < 2 * R; i += 4) load_u32<4>(reinterpret_cast<const uint32_t*>(ids + q) + i, v + i);
            } else {                                       // the last positions of all: nothing is read past the IDs' end
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const uint64_t id = (uint64_t)ids[min(q + i, n - 1)];
                    v[2 * i] = (uint32_t)id; v[2 * i + 1] = (uint32_t)(id >> 32);
                }
            }
        } else if constexpr (R == 1) {
            v[0] = keys[q];
        } else {                                           // (the workspace has room past the last key)
#pragma unroll
            for (int i = 0; i < R; i += 4) load_u32<4>(keys + q + i, v + i);
        }
    }
    // a key that is no row of the pack (only possible after rejected offsets, which raise the error word) is
    // bent to the last row so that no read leaves the table
    __device__ __forceinline__ uint32_t key(const uint32_t (&v)[IDS ? 2 * R : R], int i) const
    {
        if constexpr (IDS) return base + fold_id((int64_t)((uint64_t)v[2 * i] | (uint64_t)v[2 * i + 1] << 32), rows, magic);
        else return min(v[i], last_row);
    }
};

template <bool BF16, bool HYB>
__device__ __forceinline__ const char* pool_row(const PoolPack& k, uint32_t row, int d0)
{
    const char* w = as_global(static_cast<const char*>(k.W));
    if (HYB) {
        const int s = as_global(k.hv.slot_of)[row];
        if (s >= 0) { w = as_global(static_cast<const char*>(k.hv.W_hot)); row = (uint32_t)s; }
    }
    return w + (((size_t)((uint64_t)row * (uint32_t)k.D) + (size_t)d0) << (BF16 ? 1 : 2));
}

__device__ __forceinline__ const int32_t* pool_offsets(const PoolJob& job, const PoolPack& k, bool ids, int j, int f)
{
    return ids ? as_global(job.offsets) + (int64_t)f * job.B : as_global(job.po) + k.po_begin + (int64_t)j * job.B;
}

// Whether field i of `n` with consecutive offsets is one of sequences.  Where there are many fields (see
// pool_seq_likely) its kSeqGroup neighbours are asked too: they hold as many positions together, unless the offsets
// are rejected ones, and then tiles and cooperating wavefronts still have to agree.
constexpr int kSeqGroup = 8, kSeqMany = 64;
__device__ __forceinline__ bool pool_is_seq(const int32_t* offs, int n, int i, int B)
{
    const int64_t least = (int64_t)kSeqAvg * B;
    bool seq = (int64_t)offs[(int64_t)(i + 1) * B] - offs[(int64_t)i * B] >= least;
    if (n > kSeqMany) {
        const int g = i & ~(kSeqGroup - 1);
        seq &= (int64_t)offs[(int64_t)min(g + kSeqGroup, n) * B] - offs[(int64_t)g * B] >= least;
    }
    return seq;
}
__device__ __forceinline__ bool pool_is_seq(const PoolJob& job, const PoolPack& k, bool ids, int j, int f)
{
    return ids ? pool_is_seq(as_global(job.offsets), job.n_fields, f, job.B) : pool_is_seq(pool_offsets(job, k, false, 0, 0), k.n_fields, j, job.B);
}

// s_off: the wavefront's own LDS, 64 * kRunMax + 1 words; offs: the bag offsets of the tile's field (slot j of the pack)
template <bool BF16, bool NARROW, bool HYB, bool IDS, int R>
__device__ __forceinline__ void pool_tile_by(const PoolJob& job, const PoolPack& k, int item, int j, const FieldMeta& m, const int32_t* offs,
                                             int32_t* s_off)
{
    const int lane = threadIdx.x & 63, B = job.B;
    const KeySrc<IDS, R> src(job, k, m);
    const int b0 = (item - j * k.tiles) * ((64 >> k.sh) * k.run);
    const int nb = min((64 >> k.sh) * k.run, B - b0);
    for (int i = lane; i <= nb; i += 64) s_off[i] = min(max(offs[b0 + i], 0), src.n);   // whatever the offsets hold, no read leaves the keys
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int li = lane & ((1 << k.sh) - 1);
    int cb = (lane >> k.sh) * k.run;                       // the bag being added up ...
    const int last = min(cb + k.run, nb);
    if (cb >= last || 4 * li >= k.D) return;
    const int d0 = NARROW ? 0 : lane_col(li, k.D);
    int q = s_off[cb], c0 = q, ce = s_off[cb + 1];         // ... its first position and its end
    const int qe = s_off[last];
    float* o = as_global(job.out) + (size_t)(b0 + cb) * (size_t)job.out_stride + m.col + d0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    auto flush = [&]() {
        const int len = ce - c0;
        const float scale = m.pool == PK_MEAN && len > 0 ? 1.0f / (float)len : 1.0f;
        float y[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) y[v] = (float)acc[v] * scale;
        store_f32x4<NARROW>(o, k.D, y);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = 0.0;
        o += job.out_stride;
        c0 = ce;
        ce = ++cb < last ? s_off[cb + 1] : -1;
    };
    while (ce == q) flush();                               // empty bags before the first position
    uint32_t kv[IDS ? 2 * R : R];
    if (q < qe) src.raw(q, kv);
#pragma nounroll
    for (; q < qe; q += R) {
        float x[R][4];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint32_t first = src.key(kv, 0);
            const uint32_t row = i == 0 || q + i < qe ? src.key(kv, i) : first;      // past the run: a row that is there anyway, not used
            load_w4<BF16, NARROW>(pool_row<BF16, HYB>(k, row, d0), k.D, x[i]);
        }
        src.raw(min(q + R, qe - 1), kv);
#pragma unroll
        for (int i = 0; i < R; ++i) {
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] += (double)x[i][v];
            while (ce == q + i + 1) flush();               // its bag is complete (and the empty ones after it)
        }
    }
    while (cb < last) flush();                             // (only after rejected offsets: every bag is written, whatever they hold)
}

// A tile of two bags to a group, for fields of several IDs a bag.  A group takes the g-th longest bag of the tile and the
// g-th shortest, so that all groups have about as many positions, and a bag begins with a round: bags end at the ends of
// rounds only.  (In a walk across bags the groups' bags end at different positions of a round, and the forty instructions
// that write a bag are gone through at nearly every one of them where 32 groups have bags of 25 IDs.)  What is left is the
// rate of row requests: 200 fields of 25 IDs, batch 4096, beside the dedup chain 427 us a launch, 401 this way, 1024 bags
// alone 63 and 59.  Fields of kPairAvg IDs a bag and more, where a bag fills a round: with fewer, more is lost to rounds that
// are not full than is gained.  us a launch, walk and pairs, of 6, 7, 8, 10, 12 IDs a bag: 100 fields of 16 columns, batch 8192,
// 82.5 81.6, 90.9 87.4, 101 95.0, 116 110, 127 117; 600 of 8 and 16, 2048, 127 129, 146 145, 152 152, 186 184, 217 214; 60 of 64,
// 4096, 57.2 57.9, 63.5 63.0, 69.9 68.2, 82.7 81.2, 94.6 89.8; 1000 of 8 and 16 with 5.5 IDs 242 254, the ragged layer's 9.5 34.2 32.8.
constexpr int kPairAvg = 8, kPairShift = 4;
template <bool BF16, int R>
__device__ __forceinline__ void pool_tile_pairs(const PoolJob& job, const PoolPack& k, int item, int j, const FieldMeta& m, const int32_t* offs,
                                                int32_t* s_off)
{
    const int lane = threadIdx.x & 63, B = job.B;
    const KeySrc<false, R> src(job, k, m);
    const int b0 = (item - j * k.tiles) * (128 >> k.sh), nb = min(128 >> k.sh, B - b0);     // (at most 64)
    for (int i = lane; i <= nb; i += 64) s_off[i] = min(max(offs[b0 + i], 0), src.n);   // whatever the offsets hold, no read leaves the keys
    auto wave_order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };
    wave_order();
    int32_t* s_order = s_off + 128;                        // the bags, longest first
    {
        const int len = lane < nb ? min(max(s_off[lane + 1] - s_off[lane], 0), 1 << 24) : 0, key = len << 6 | lane;
        int rank = 0;
        for (int i = 0; i < nb; ++i) rank += __builtin_amdgcn_readlane(key, i) > key;
        if (lane < nb) s_order[rank] = lane;
    }
    wave_order();
    const int li = lane & ((1 << k.sh) - 1), g = lane >> k.sh;
    if (g >= nb || 4 * li >= k.D) return;
    const int d0 = lane_col(li, k.D);
    const int i2 = (128 >> k.sh) - 1 - g;                  // (the tile's last half may be missing)
    const int other = i2 < nb ? s_order[i2] : -1;
    const int q2 = s_off[max(other, 0)], e2 = s_off[max(other, 0) + 1];
    int bag = s_order[g], q = s_off[bag], c0 = q, ce = s_off[bag + 1];
    bool more = other >= 0;
    float* out = as_global(job.out) + (size_t)b0 * (size_t)job.out_stride + m.col + d0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    uint32_t kv[R];
    src.raw(q, kv);                                        // (an empty bag: keys of its neighbour or the room past the last, not used)
#pragma nounroll
    for (;;) {
        float x[R][4];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint32_t row = i == 0 || q + i < ce ? src.key(kv, i) : src.key(kv, 0);     // past the bag: a row that is there anyway, not used
            load_w4<BF16, false>(pool_row<BF16, false>(k, row, d0), k.D, x[i]);
        }
        const bool end = q + R >= ce;
        src.raw(end ? (more ? q2 : q) : q + R, kv);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (q + i < ce) {
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] += (double)x[i][v];
            }
        }
        q += R;
        if (end) {
            const int len = ce - c0;
            const float scale = m.pool == PK_MEAN && len > 0 ? 1.0f / (float)len : 1.0f;
            float y[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) { y[v] = (float)acc[v] * scale; acc[v] = 0.0; }
            store_f32x4<false>(out + (size_t)bag * (size_t)job.out_stride, k.D, y);
            if (!more) break;
            more = false;
            bag = other; q = c0 = q2; ce = e2;
        }
    }
}

// Rounds of R positions; of one where the field's runs hold about one (a round's idle places ask for a row again: 26
// one-hot fields of 2048 bags, one bag a run, pooled in 7.4 us with rounds of eight, 6.0 with rounds of one; for runs of
// three IDs on average rounds of four are slower than of eight, the longest run then takes two).
template <bool BF16, bool NARROW, bool HYB, bool IDS, bool PAIRS, int R>
__device__ __forceinline__ void pool_tile(const PoolJob& job, const PoolPack& k, int item, int32_t* s_off)
{
    const int j = item / k.tiles;
    const int f = as_global(k.slot_field)[j];
    const FieldMeta m = as_global(job.fmeta)[f];
    const int32_t* offs = pool_offsets(job, k, IDS, j, f);
    if (job.coop_waves && pool_is_seq(job, k, IDS, j, f)) return;       // (without them only rejected offsets look like a sequence field's)
    if constexpr (R == 8) {
        const int64_t per_run = ((int64_t)offs[job.B] - offs[0]) * k.run;      // times B
        if (2 * per_run <= (int64_t)3 * job.B) return pool_tile_by<BF16, NARROW, HYB, IDS, 1>(job, k, item, j, m, offs, s_off);
        // (Rows of four columns and fewer have more bags to a tile than lanes.  Of rows of more than 64 a wavefront has one or two
        // groups, little to even out, and an empty bag still takes a round: walk and pairs, 20 fields of 200 columns, 10 IDs a bag with half of
        // the bags empty, 73 84 us; 30 of 128, 67 70, and with bags of 1 to 20, 67 70; 60 of 64, 78 76, 77 74.)
        if constexpr (PAIRS && !NARROW) {
            if (k.run == 2 && k.sh >= 1 && k.sh <= kPairShift && per_run >= (int64_t)2 * kPairAvg * job.B) return pool_tile_pairs<BF16, R>(job, k, item, j, m, offs, s_off);
        }
    }
    pool_tile_by<BF16, NARROW, HYB, IDS, R>(job, k, item, j, m, offs, s_off);
}

// Whether one of `n` fields with consecutive offsets can be a sequence field: not where no kSeqGroup neighbours hold
// that many positions together.  (Every cooperating wavefront asks: looking at both ends of every field, 2000
// one-hot fields of 128 bags pooled in 43 us, this way in 13.)
__device__ __forceinline__ bool pool_seq_likely(const int32_t* offs, int n, int B)
{
    const int lane = threadIdx.x & 63;
    if (n <= kSeqMany) return true;                            // (looking at them is as quick)
    bool any = false;
    for (int g0 = 0; g0 * kSeqGroup < n; g0 += 63) {       // lane l: where the chunk's l-th group starts
        const int at = offs[(int64_t)min((g0 + lane) * kSeqGroup, n) * B];
        const int next = __shfl_down(at, 1, 64);
        any |= lane < 63 && (int64_t)next - at >= (int64_t)kSeqAvg * B;
    }
    return __any(any);
}

// Sequence fields: a wavefront per bag, R positions per group and round.
template <bool BF16, bool NARROW, bool HYB, bool IDS, int R>
__device__ __forceinline__ int pool_coop(const PoolJob& job, const PoolPack& k, int idx)
{
    const int lane = threadIdx.x & 63, B = job.B;
    const int lpr = 1 << k.sh, gpw = 64 >> k.sh, li = lane & (lpr - 1), g = lane >> k.sh;
    const int d0 = NARROW ? 0 : lane_col(li, k.D);
    if (!IDS && !pool_seq_likely(pool_offsets(job, k, false, 0, 0), k.n_fields, B)) return idx;
    for (int j0 = 0; j0 < k.n_fields; j0 += 64) {
        bool seq = false;
        if (j0 + lane < k.n_fields)
            seq = pool_is_seq(job, k, IDS, j0 + lane, IDS ? as_global(k.slot_field)[j0 + lane] : 0);
        for (uint64_t todo = __ballot(seq); todo; todo &= todo - 1) {
            const int j = j0 + __ffsll((unsigned long long)todo) - 1;
            const int f = as_global(k.slot_field)[j];
            const FieldMeta m = as_global(job.fmeta)[f];
            const int32_t* offs = pool_offsets(job, k, IDS, j, f);
            const KeySrc<IDS, R> src(job, k, m);
            for (; idx < B; idx += job.coop_waves) {
                const int q0 = min(max(offs[idx], 0), src.n), q1 = min(max(offs[idx + 1], q0), src.n);
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                int q = q0 + g * R;
                uint32_t kv[IDS ? 2 * R : R];
                if (q < q1) src.raw(q, kv);
#pragma nounroll
                for (; q < q1; q += R * gpw) {
                    float x[R][4];
#pragma unroll
                    for (int i = 0; i < R; ++i) {
                        const uint32_t row = i == 0 || q + i < q1 ? src.key(kv, i) : src.key(kv, 0);
                        load_w4<BF16, NARROW>(pool_row<BF16, HYB>(k, row, d0), k.D, x[i]);
                    }
                    src.raw(min(q + R * gpw, q1 - 1), kv);
                    // (the round's rows are added up as a tree in fp32 first: eight conversions to double would cost
                    // the launch 2.5 % on bf16 sequences, and three roundings do not grow with the bag)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
#pragma unroll
                        for (int i = 1; i < R; ++i) x[i][v] = q + i < q1 ? x[i][v] : 0.f;
#pragma unroll
                        for (int d = 1; d < R; d *= 2)
#pragma unroll
                            for (int i = 0; i + d < R; i += 2 * d) x[i][v] += x[i + d][v];
                        acc[v] += (double)x[0][v];
                    }
                }
#pragma nounroll
                for (int s = lpr; s < 64; s <<= 1)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[v] += __shfl_xor(acc[v], s, 64);
                if (g == 0 && 4 * li < k.D) {
                    const float scale = m.pool == PK_MEAN && q1 > q0 ? 1.0f / (float)(q1 - q0) : 1.0f;
                    float y[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) y[v] = (float)acc[v] * scale;
                    store_f32x4<NARROW>(as_global(job.out) + (size_t)idx * (size_t)job.out_stride + m.col + d0, k.D, y);
                }
            }
            idx -= B;
        }
    }
    return idx;
}

// the code for a pack's kind
#define PK_POOL_KINDS(FN, RES, ...)                                                             \
    switch (k.kind) {                                                                           \
        case 0: RES FN(false, false)(__VA_ARGS__); break;                                       \
        case 1: RES FN(true, false)(__VA_ARGS__); break;                                        \
        case 2: RES FN(false, true)(__VA_ARGS__); break;                                        \
        case 3: RES FN(true, true)(__VA_ARGS__); break;                                         \
    }
#define PK_POOL_TILE(BF16, NARROW) pool_tile<BF16, NARROW, HYB, IDS, PAIRS, R>
#define PK_POOL_COOP(BF16, NARROW) pool_coop<BF16, NARROW, HYB, IDS, R>

// one wavefront's share of a launch's pooling: `wave` counts its wavefronts
template <bool HYB, bool IDS, bool PAIRS, int R>
__device__ __forceinline__ void pool_wave(const PoolJob& job, int wave, int32_t* s_off)
{
    if (wave < job.n_items) {
        int i = 0;
        while (i + 1 < job.n_packs && wave >= job.pack[i + 1].item_begin) ++i;
        const PoolPack& k = job.pack[i];
        const int item = wave - k.item_begin;
        PK_POOL_KINDS(PK_POOL_TILE, , job, k, item, s_off)
        return;
    }
    int idx = wave - job.n_items;
    if (idx >= job.coop_waves) return;
    if constexpr (IDS) {                                   // (the launch has all packs: the offsets of all fields, in field order)
        if (!pool_seq_likely(as_global(job.offsets), job.n_fields, job.B)) return;
    }
    for (int i = 0; i < job.n_packs; ++i) {
        const PoolPack& k = job.pack[i];
        PK_POOL_KINDS(PK_POOL_COOP, idx =, job, k, idx)
    }
}

// PAIRS: for launches where two bags of a group hold eight IDs or more on average over all fields: some of them can then have
// kPairAvg a bag (80 one-hot fields and 20 of 25 IDs, 5.8 on average: 43.6 us, 39.6 with pairs).  Without that code the walk of
// one-hot fields is 1 % faster (26 of 65536 74.2 us, 75.2 with it); of 5.5 IDs a bag 181.5, 182.3, of sequences 128.7, 126.9.
template <bool HYB, bool PAIRS>
__global__ void __launch_bounds__(NT, 6)
pk_pool_kernel(PoolJob job)
{
    __shared__ int32_t s_off[NT / 64][64 * kRunMax + 1];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    pool_wave<HYB, false, PAIRS, 8>(job, (int)blockIdx.x * (NT / 64) + wv, s_off[wv]);
}

// Small batches: the whole forward pass is ONE launch.  The first blocks are the slices of the
// dedup (they find their occurrences in the caller's IDs), the next ones write what is per bag and
// per pack, and the rest pool: the pooling needs the rows' keys only, which it forms from the IDs
// itself, so it depends on nothing the other blocks write.  (With few occurrences a launch is
// mostly latency, and a second launch would wait for the first.)
// WAVES: wavefronts per SIMD the kernel is compiled for.  8 lets two blocks share a compute unit, which a
// launch with more blocks than compute units needs; 4 gives a block twice the registers (nothing is then
// kept in scratch memory), which is faster when every block has a compute unit to itself.
// MANY: for plans with a table that several fields read (a slice block then looks for its occurrences in all of
// them; without that code the other plans' launch keeps more in registers: 26 one-hot fields 52 us a step, 56 with it).
template <int WAVES, bool MANY>
__global__ void __launch_bounds__(kSliceThreads, WAVES)
pk_fused_kernel(SliceArgs a, PoolJob pj, int slice_blocks, int meta_blocks)
{
    extern __shared__ int32_t s_dyn[];                     // kSliceTfWords words per field of a table
    __shared__ int32_t s_main[kSmallLdsWords];
    static_assert(kSmallLdsWords >= kSliceThreads / 64 * (64 * kRunMax + 1), "the pooling's offsets must fit the block's LDS");
    static_assert(kSmallLdsWords >= 3 * 4096 + 2, "the field scan must fit the block's LDS");
    if ((int)blockIdx.x < slice_blocks) {
        // (the kernel's arguments where they stand: `a` is the first of them)
        small_slice_body<(WAVES > 4), MANY>((SliceArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(), blockIdx.x, s_main, s_dyn);
        return;
    }
    PK_PT(a, blockIdx.x, 0);
    if ((int)blockIdx.x < slice_blocks + meta_blocks) {
        meta_body(a, (int)blockIdx.x - slice_blocks, meta_blocks, s_main);
        PK_PT(a, blockIdx.x, 8);
        return;
    }
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    pool_wave<false, true, false, 4>(pj, ((int)blockIdx.x - slice_blocks - meta_blocks) * (kSliceThreads / 64) + wv,
                              s_main + wv * (64 * kRunMax + 1));
    PK_PT(a, blockIdx.x, 8);
}
