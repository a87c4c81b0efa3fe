// Small batches, H1 and H2 in the launch that also pools (dev_pool.h): one block per slice of a table's keys.
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.
//
// A block reads the IDs of its table's fields (they are few and sit in L2), keeps those of its slice in LDS, and
// needs one number from other blocks: the distinct keys of the pack's slices before its own.  (How many
// occurrences come before its own it knows: those of earlier tables from the offsets, those of earlier slices of its
// table from the IDs.)  What bounds it is the chain of dependent steps, so:
//   - everything a block needs of the plan stands in its SmallSlice; field sizes are reduced, not scanned;
//   - IDs and offsets are asked for before the first barrier;
//   - the block publishes its count as soon as the bitmap is complete and asks for the others' right then;
//     they arrive while it counts occurrences per key;
//   - an occurrence's place inside its key comes from the counting pass, kept in a register.
// Before (every field scanned in every block, a two-level look-back after the counting): 8 one-hot fields 15.5 us,
// 26 fields of 8192 29.8 us, 26 fields of 64 17 us a launch.
// A table that several fields read is one run of occurrences, numbered over its fields (field after field, each step
// waited for: 26 fields of 64 on two tables 55 us a launch, 15.5 this way).  Slices of frequent keys, with more
// occurrences than are kept, have the counters of all of them in one round where there is room (26 one-hot fields of
// 16384, low IDs frequent: 90 us a launch with 4096 counters, 60 with 8192).

// LDS words: bitmap | popcount prefix | counters | kept occurrences: key, position | bag offsets (or every 2^k-th of them)
constexpr int kSmallWords = 1 << (kSliceLogMax - 5);
constexpr int kSmallRanks = 4096;
constexpr int kSmallCache = 2 * kSliceThreads;
constexpr int kSmallOffs = 2048;
constexpr int kSmallLdsWords = 2 * kSmallWords + kSmallRanks + 2 * kSmallCache + kSmallOffs;
constexpr uint32_t kSmallKeyMask = (1u << kSliceLogMax) - 1u;      // of a kept occurrence's first word: its key; above, its field of the table
static_assert(kSliceLogMax + 12 <= 32, "a table has up to 4096 fields");
constexpr int kDescGroup = 16;           // slices whose distinct keys also add up in one word

__device__ __forceinline__ uint64_t small_load(const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// LEAN (two blocks per CU): the kernel's arguments and the slice's description are read where they are used,
// through pointers that the compiler loses track of between the phases: held from the start they are forty scalar
// registers more than there are, and with the spills of those the 26-field launch is 5 us slower.  A block that has
// its CU to itself has the registers and would only wait for the reads.
typedef const __attribute__((address_space(4))) SmallSlice* SmallSlicePtr;
__device__ __forceinline__ SmallSlicePtr slice_at(SliceArgsPtr a, int slice) { return (SmallSlicePtr)a->small_slices + slice; }

// what the phases of a block hand on, in LDS
struct SmallCtx { int32_t pstart, nnz_p, rec_before, n_rec, n_u, q0; };

// writes of one occurrence: its key and inverse, its entry in its key's segment
__device__ __forceinline__ void small_place(SliceArgsPtr a, SmallSlicePtr ss, const int32_t* tf, int pstart, int nnz_p, int base_u,
                                            uint32_t kl, int q, int rk, int pos, int b, int L)
{
    const uint32_t ref = (uint32_t)((int64_t)b * a->out_dim + tf[3]);
    const int qp = q + tf[2];
    if ((unsigned)qp < (unsigned)a->nnz) {
        as_global(a->keys)[qp] = ss->key_lo + ((uint32_t)ss->idx << ss->log_keys) + kl;
        as_global(a->inverse)[qp] = base_u + rk;
    }
    if ((unsigned)pos < (unsigned)nnz_p) {
        uint32_t* ent = as_global(a->ent_all) + (size_t)pstart * a->ent_mult;
        if (ss->wide) reinterpret_cast<uint2*>(ent)[pos] = make_uint2(ref, (tf[4] & 1) == PK_MEAN && L > 0 ? (uint32_t)L : 1u);   // the pack's entries carry the bag length
        else ent[pos] = ref;
    }
}

// counters of keys [r0, r0 + width) become the keys' first places; segment offsets and marks go out
__device__ __forceinline__ void small_starts(SliceArgsPtr a, SmallSlicePtr ss, int32_t* s_cnt, int pstart, int base_u, int r0, int width, int s0, int per)
{
    const int p = ss->pack;
    int32_t* seg = as_global(a->seg_all) + pstart + p + base_u + r0;
    int32_t* marks = as_global(a->marks) + (pstart / kMarkStep + p);
    for (int j = 0; j < per; ++j) {
        const int i = (int)threadIdx.x * per + j;
        if (i < width) {
            const int len = s_cnt[i];
            seg[i] = s0;
            s_cnt[i] = s0;
            for (int m = (s0 + kMarkStep - 1) / kMarkStep; (int64_t)m * kMarkStep < (int64_t)s0 + len; ++m) marks[m] = base_u + r0 + i;
            if (len >= 2 * kPiece) {                       // the key is reduced in pieces: its partial sums start at zero
                const size_t slot = (size_t)(pstart / kPiece + p) + (size_t)(s0 / kPiece);
                double* gh = as_global(a->ghot) + slot * a->dmax;
                for (int d = 0; d < ss->dim; ++d) gh[d] = 0.0;
                as_global(a->ticket)[slot] = 0;
            }
            s0 += len;
        }
    }
}

__device__ __forceinline__ int small_sum(const int32_t* s_cnt, int width, int per)
{
    int s = 0;
    for (int j = 0; j < per; ++j) {
        const int i = (int)threadIdx.x * per + j;
        s += i < width ? s_cnt[i] : 0;
    }
    return s;
}

__device__ __forceinline__ int small_rank(const uint32_t* s_bits, const uint32_t* s_pre, uint32_t kl)
{
    return (int)(s_pre[kl >> 5] + __popc(s_bits[kl >> 5] & ((1u << (kl & 31)) - 1u)));
}

// bag offsets in LDS: every 2^step_log-th
__device__ __forceinline__ int small_step(int B)
{
    int k = 0;
    while (((B + (1 << k) - 1) >> k) + 1 > kSmallOffs) ++k;
    return k;
}

// the bag of position q and its length, for a table with one field: from the samples in LDS (where they are),
// then the few bags between two of them
__device__ __forceinline__ int small_bag(const int32_t* __restrict__ offs, int B, const int32_t* s_offs, bool sampled, int guess, int q, int* L)
{
    int b;
    if (sampled) {
        const int step_log = small_step(B), n_offs = ((B + (1 << step_log) - 1) >> step_log) + 1;
        int k = upper_bound_i32(s_offs, n_offs, q) - 1;
        if (step_log == 0) {
            k = min(max(k, 0), B - 1);
            *L = s_offs[k + 1] - s_offs[k];
            return k;
        }
        k = max(k, 0) << step_log;
        b = min(max(k + upper_bound_i32(offs + k, max(min(1 << step_log, B - k), 0), q) - 1, 0), B - 1);
    } else {
        b = find_bag(offs, B, q, guess);
    }
    *L = offs[b + 1] - offs[b];
    return b;
}

// where the occurrences of a table of several fields stand: field, position of the v-th one, from where the last
// lookup ended
struct SmallField {
    int j = 0, next = -1, shift = 0;                       // the field; first occurrence after it; position minus number
    __device__ __forceinline__ int position(const int32_t* s_tf, int nf, int n_table, int v)
    {
        if (v >= next) {
            int hi = nf;                                   // the last field with no more than v occurrences before it
            while (hi - j > 1) {
                const int mid = (j + hi) >> 1;
                if (s_tf[kSliceTfWords * mid + 1] <= v) j = mid; else hi = mid;
            }
            next = j + 1 < nf ? s_tf[kSliceTfWords * (j + 1) + 1] : n_table;
            shift = s_tf[kSliceTfWords * j] - s_tf[kSliceTfWords * j + 1];
        }
        return v + shift;
    }
};

template <bool V> struct BoolTag { static constexpr bool value = V; };

// Distinct keys of the pack's slices before `slice`, and whether one of them has found bad offsets, for a block that
// has waited long: a block before it may not have started, and may not be able to while this one holds its place (as
// count_before of the large batches).  What is published is taken, the rest counted from the IDs, 64 K keys at a time.  One
// wavefront; s_map: kSmallOffs words.  (Its registers cost the launch some of what waiting alone takes: 26 fields of 64
// 10.9 -> 11.2 us, 889 tables of 70 samples 60 -> 62 a step, 26 fields of 8192 none.  The block begun again in code of its
// own, with nothing kept meanwhile: 11.0, 63 to 66 and 3 % for launches of many blocks.)
constexpr int kSmallPatience = 2048;                       // looks of about 2.5 us
template <bool MANY>
__device__ __forceinline__ void small_count_before(SliceArgsPtr a, int slice, uint32_t* s_map, uint32_t* before, uint32_t* flags)
{
    const int lane = threadIdx.x & 63, B = a->B, n_all = (int)a->nnz;
    uint32_t sum = 0, bad = 0;
#pragma nounroll
    for (int j = slice_at(a, slice)->pack_first; j < slice; ++j) {
        const uint64_t d = small_load(as_global(a->desc) + j);
        if (a->patience >= 0 && __all((d >> 48) != 0)) {
            sum += (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)d);
            bad |= (uint32_t)(d >> 40) & 1u;
            continue;
        }
        const SmallSlicePtr sj = slice_at(a, j);
        const int lg = sj->log_keys, nf = MANY ? sj->n_fields : 1;
        const int b_lo = (int)((int64_t)B * sj->idx / sj->n_table_slices), b_hi = (int)((int64_t)B * (sj->idx + 1) / sj->n_table_slices);
        int c = 0;
#pragma nounroll
        for (uint32_t w0 = 0; w0 < 1u << lg; w0 += 32u * kSmallOffs) {
#pragma nounroll
            for (int i = lane; i < kSmallOffs; i += 64) s_map[i] = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma nounroll
            for (int f = 0; f < nf; ++f) {
                const int field = MANY ? as_global(a->tfields)[sj->field_begin + f].field : sj->field0;
                const int32_t* offs = as_global(a->offsets) + (int64_t)field * B;
                const int fb = offs[0], fe = offs[B], q0 = min(max(fb, 0), n_all), q1 = min(max(fe, q0), n_all);
#pragma nounroll
                for (int b = b_lo + lane; b < b_hi; b += 64) bad |= offs[b] > offs[b + 1] || offs[b] < fb || offs[b + 1] > fe;
#pragma nounroll
                for (int q = q0 + lane; q < q1; q += 64) {
                    const uint32_t k = fold_id(as_global(a->ids)[q], sj->rows, sj->magic), kl = (k & ((1u << lg) - 1u)) - w0;
                    if ((k >> lg) == (uint32_t)sj->idx && kl < 32u * kSmallOffs) atomicOr(&s_map[kl >> 5], 1u << (kl & 31));
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma nounroll
            for (int i = lane; i < kSmallOffs; i += 64) c += __popc(s_map[i]);
        }
        sum += (uint32_t)wave_sum(c);
    }
    *before = sum;
    *flags = __any(bad) ? 1u : 0u;
}

// MANY: some table of the plan has several fields
template <bool LEAN, bool MANY>
__device__ __forceinline__ void small_slice_body(SliceArgsPtr a, int slice, int32_t* s_main, int32_t* s_tf)
{
    constexpr int NTH = kSliceThreads, NW = NTH / 64;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                          // (what shuffles and scans derive from the index is formed where it is used: 5 to 8 registers spilled, not 13)
    const int lane = tid & 63, wv = tid >> 6;
    uint32_t* s_bits = reinterpret_cast<uint32_t*>(s_main);
    uint32_t* s_pre = s_bits + kSmallWords;
    int32_t* s_cnt = s_main + 2 * kSmallWords;
    uint32_t* s_ckey = reinterpret_cast<uint32_t*>(s_cnt + kSmallRanks);
    int32_t* s_cpos = s_cnt + kSmallRanks + kSmallCache;
    int32_t* s_offs = s_cpos + kSmallCache;
    __shared__ int4 s_red[NW];
    __shared__ int s_n, s_before, s_flag, s_base;
    __shared__ SmallCtx s_ctx;
    const int F = a->F, B = a->B;
    const int patience = a->patience;                      // (read here, with what is waited for anyway)
    const int64_t nnz = a->nnz;
    const int32_t* __restrict__ offsets = as_global(a->offsets);
    const int64_t* __restrict__ ids = as_global(a->ids);
    PK_PT(*a, slice, 0);
    SmallSlicePtr ss = slice_at(a, slice);
    const int lg = ss->log_keys, nf = MANY ? ss->n_fields : 1;       // (fields of the table)
    const uint32_t lo = (uint32_t)ss->idx << lg;           // first key of the slice inside its table
    const int words = 1 << (lg - 5);

    // ---- what can be asked for at once, in the order it is needed ----
    // field sizes; the offsets of this slice's share of the table's bags; the first IDs
    int2 sf = make_int2(0, 0);
    if (tid < F) sf = as_global(a->slot_info)[tid];         // the slot's field, its table in the (pack, first key) order
    const int n_all = (int)nnz;
    const int32_t* __restrict__ offs0 = offsets + (int64_t)ss->field0 * B;
    const int fb0 = offs0[0], fe0 = offs0[B];              // the table's (first) field: where its occurrences are
    const int b_lo = (int)((int64_t)B * ss->idx / ss->n_table_slices), b_hi = (int)((int64_t)B * (ss->idx + 1) / ss->n_table_slices);
    int share0 = 0, share1 = 0;
    if (b_lo + tid < b_hi) { share0 = offs0[b_lo + tid]; share1 = offs0[b_lo + tid + 1]; }
    int o0 = 0, o1 = 0;
    if (tid < F) { o0 = offsets[(int64_t)sf.x * B]; o1 = offsets[(int64_t)(sf.x + 1) * B]; }
    const int q0 = min(max(fb0, 0), n_all), q1 = min(max(fe0, q0), n_all);
    const bool onehot = nf == 1 && q1 - q0 == B;           // as many occurrences as bags: most likely one each
    int64_t idv[4];
    auto fetch = [&](int base, int end) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + tid + u * NTH;
            idv[u] = i < end ? ids[i] : 0;
        }
    };
    fetch(q0, q1);
    // ---- sizes: occurrences of the packs before, of the tables before, of the pack, of the slots before ----
    int4 sum = make_int4(0, 0, 0, 0);
    int bad = 0, viol = 0;
    const int len0 = o1 - o0;
    for (int i = tid; i < F; i += NTH) {
        if (i >= NTH) {
            sf = as_global(a->slot_info)[i];
            o0 = offsets[(int64_t)sf.x * B]; o1 = offsets[(int64_t)(sf.x + 1) * B];
        }
        const int len = o1 - o0;
        bad |= len < 0 || (sf.x == 0 && o0 != 0) || (sf.x == F - 1 && (int64_t)o1 != nnz);
        sum.x += i < ss->first_slot ? len : 0;
        sum.y += sf.y < ss->table ? len : 0;
        sum.z += i >= ss->first_slot && i < ss->first_slot + ss->pack_fields ? len : 0;
        sum.w += i < ss->slot0 ? len : 0;
    }
    // the bags of this slice's share: inside the field and not decreasing
    for (int b = b_lo + tid; b < b_hi; b += NTH) {
        if (b >= b_lo + NTH) { share0 = offs0[b]; share1 = offs0[b + 1]; }
        viol |= share0 > share1 || share0 < fb0 || share1 > fe0;
    }
    const int step_log = small_step(B), n_offs = ((B + (1 << step_log) - 1) >> step_log) + 1;
    if (nf == 1 && !onehot)
        for (int i = tid; i < n_offs; i += NTH) s_offs[i] = offs0[min(i << step_log, B)];
    for (int w = tid; w < words; w += NTH) s_bits[w] = 0;
    for (int i = tid; i < kSmallRanks; i += NTH) s_cnt[i] = 0;
    if (tid == 0) { s_n = 0; s_before = 0; s_flag = 0; }
    if (wv * 64 < F) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            sum.x += __shfl_xor(sum.x, o, 64); sum.y += __shfl_xor(sum.y, o, 64);
            sum.z += __shfl_xor(sum.z, o, 64); sum.w += __shfl_xor(sum.w, o, 64);
        }
        if (lane == 0) s_red[wv] = sum;
    }
    bad = __syncthreads_or(bad);
    sum = make_int4(0, 0, 0, 0);
    for (int w = 0; w < NW && w * 64 < F; ++w) { const int4 x = s_red[w]; sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w; }
    if (bad) {                                             // every block sees the same boundaries: nobody publishes, nobody waits
        if (ss->is_last && tid == 0) { as_global(a->st)[ss->pack].n_unique = 0; as_global(a->st)[ss->pack].error = 1; }
        return;
    }
    if (tid == 0) { s_ctx.pstart = sum.x; s_ctx.nnz_p = sum.z; s_ctx.rec_before = sum.y - sum.x; s_ctx.q0 = q0; }
    PK_PT(*a, slice, 1);
    // the table's fields: where they begin, the table's occurrences before them, packed position minus position, column,
    // pooling | field
    int n_table = q1 - q0;                                 // occurrences of the table
    if (nf == 1) {
        if (tid == 0) { s_tf[0] = q0; s_tf[1] = 0; s_tf[2] = sum.w - fb0; s_tf[3] = ss->col0; s_tf[4] = ss->pool0 | (ss->field0 << 1); }
    } else {
        // (several fields: the slots' packed positions from one scan of their sizes, where the kept occurrences go later)
        int32_t* s_slotpos = s_cnt + kSmallRanks;
        int carry = 0;
        for (int i = tid; i - tid < F; i += NTH) {
            int len = len0;
            if (i >= NTH && i < F) {
                const int f = as_global(a->slot_info)[i].x;
                len = offsets[(int64_t)(f + 1) * B] - offsets[(int64_t)f * B];
            }
            int tot;
            const int ex = block_excl_scan<NTH, true>(i < F ? len : 0, &tot);
            if (i < F) s_slotpos[i] = carry + ex;
            carry += tot;
        }
        __syncthreads();
        n_table = 0;
        for (int j = tid; j - tid < nf; j += NTH) {
            int len = 0;
            int32_t* tf = s_tf + kSliceTfWords * j;
            if (j < nf) {
                const TableField x = as_global(a->tfields)[ss->field_begin + j];
                tf[0] = offsets[(int64_t)x.field * B];
                len = offsets[(int64_t)(x.field + 1) * B] - tf[0];
                tf[2] = s_slotpos[ss->first_slot + x.slot] - tf[0]; tf[3] = x.col; tf[4] = x.pool | (x.field << 1);
            }
            int tot;
            const int ex = block_excl_scan<NTH, true>(len, &tot);
            if (j < nf) tf[1] = n_table + ex;
            n_table += tot;
        }
        __syncthreads();
        // the bags of this slice's share of the other fields
        const unsigned share = (unsigned)(b_hi - b_lo);
        for (unsigned x = tid; x < share * (unsigned)(nf - 1); x += NTH) {
            const int j = 1 + (int)(x / share), b = b_lo + (int)(x % share);
            const int32_t* tf = s_tf + kSliceTfWords * j;
            const int32_t* offs = offsets + (int64_t)(tf[4] >> 1) * B;
            viol |= offs[b] > offs[b + 1] || offs[b] < tf[0] || offs[b + 1] > offs[B];
        }
    }

    // ---- which keys occur; the slice's occurrences are kept while they are at hand ----
    const uint32_t rows = ss->rows;
    const uint64_t magic = ss->magic;
    int before = 0;                                        // per wavefront: occurrences of the table in earlier slices
    uint32_t kk[4];
    auto find = [&](auto&& field, auto&& pos) {            // of the four occurrences per lane (rows kk): those of this slice
        uint64_t m[4];
        int n = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            before += __popcll(__ballot(kk[u] < lo));
            m[u] = __ballot((kk[u] >> lg) == (uint32_t)ss->idx);
            n += __popcll(m[u]);
        }
        if (n == 0) return;
        int at = 0;                                        // room for the wavefront's finds in one add
        if (lane == 0) at = atomicAdd(&s_n, n);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (m[u] >> lane & 1) {
                const uint32_t kl = kk[u] - lo, bit = 1u << (kl & 31);
                if (!(s_bits[kl >> 5] & bit)) atomicOr(&s_bits[kl >> 5], bit);
                const int x = at + __popcll(m[u] & ((1ull << lane) - 1ull));
                if (x < kSmallCache) { s_ckey[x] = kl | ((uint32_t)field(u) << kSliceLogMax); s_cpos[x] = pos(u); }
            }
            at += __popcll(m[u]);
        }
    };
    if (nf == 1) {
        for (int base = q0; base < q1; base += 4 * NTH) {
            if (base > q0) fetch(base, q1);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                kk[u] = base + tid + u * NTH < q1 ? fold_id(idv[u], rows, magic) : 0xFFFFFFFFu;      // (no row: rows <= 2^30)
            find([](int) { return 0; }, [&](int u) { return base + tid + u * NTH; });
        }
    } else {
        SmallField at;
        for (int base = 0; base < n_table; base += 4 * NTH) {
            int fj[4], q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                q[u] = at.position(s_tf, nf, n_table, min(base + tid + u * NTH, n_table - 1));
                fj[u] = at.j;
                idv[u] = ids[q[u]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                kk[u] = base + tid + u * NTH < n_table ? fold_id(idv[u], rows, magic) : 0xFFFFFFFFu;
            find([&](int u) { return fj[u]; }, [&](int u) { return q[u]; });
        }
    }
    if (lane == 0 && before) atomicAdd(&s_before, before);
    if (viol) s_flag = 1;
    __syncthreads();
    PK_PT(*a, slice, 2);
    a = forget<LEAN>(a);
    ss = slice_at(a, slice);
    const int n_rec = s_n;
    const uint32_t own_flags = s_flag ? 1u : 0u;

    // ---- popcount prefix of the words: thread i owns words [i * wpt, (i + 1) * wpt) ----
    const int wpt = max(1, words / NTH);
    int c = 0;
    if (tid * wpt < words)
        for (int j = 0; j < wpt; ++j) c += __popc(s_bits[tid * wpt + j]);
    int n_u;
    int run = block_excl_scan<NTH, true>(c, &n_u);
    // the number of this slice's distinct keys is out: in its own word and in its group's; and the words of the
    // slices before it are asked for (one lane each: those of the own group, and the earlier groups' sums)
    const int l = slice - ss->pack_first, g = l / kDescGroup, r = l % kDescGroup;
    uint64_t ack0 = 0, ack1 = 0, d_own = 0, d_grp = 0;     // (acks: old values, which say that the words have arrived)
    int ack2 = 0, ack3 = 0;
    if (wv == 0) {
        uint64_t* desc = as_global(a->desc) + slice;
        uint64_t* gd = as_global(a->gdesc) + (ss->pack_first / kDescGroup + ss->pack);     // the pack's groups (packs never share one)
        if (lane == 0) {
            const uint64_t v = ((uint64_t)1 << 48) | ((uint64_t)own_flags << 40) | (uint32_t)n_u;     // count of slices | flags | distinct keys
            ack0 = atomicExch((unsigned long long*)desc, (unsigned long long)v);
            ack1 = atomicAdd((unsigned long long*)gd + g, (unsigned long long)v);
        }
        if (lane < r) d_own = small_load(desc - 1 - lane);
        if (lane < g) d_grp = small_load(gd + lane);
    }
    if (tid * wpt < words)
        for (int j = 0; j < wpt; ++j) {
            s_pre[tid * wpt + j] = (uint32_t)run;
            run += __popc(s_bits[tid * wpt + j]);
        }
    if (tid == 0) { s_ctx.rec_before += s_before; s_ctx.n_rec = n_rec; s_ctx.n_u = n_u; }
    __syncthreads();
    PK_PT(*a, slice, 3);
    a = forget<LEAN>(a);
    ss = slice_at(a, slice);

    // ---- what needs the slices before ----
    auto finish_wait = [&]() {                             // wavefront 0: distinct keys of the slices before
        uint64_t* desc = as_global(a->desc) + slice;
        uint64_t* gd = as_global(a->gdesc) + (ss->pack_first / kDescGroup + ss->pack);
        bool gave_up = patience < 0;
        int spins = 0;
        while (__any(lane < r && (d_own >> 48) == 0)) {
            if (++spins > patience) { gave_up = true; break; }
            __builtin_amdgcn_s_sleep(1);
            if (lane < r && (d_own >> 48) == 0) d_own = small_load(desc - 1 - lane);
        }
        uint32_t u = lane < r ? (uint32_t)d_own : 0u, fl = lane < r ? (uint32_t)(d_own >> 40) & 1u : 0u;
        for (int k0 = 0; k0 < g; k0 += 64) {               // a group is complete when all its slices have added themselves
            const bool mine = k0 + lane < g;
            if (k0 && mine) d_grp = small_load(gd + k0 + lane);
            while (__any(mine && (d_grp >> 48) != kDescGroup)) {
                if (++spins > patience) { gave_up = true; break; }
                __builtin_amdgcn_s_sleep(1);
                if (mine && (d_grp >> 48) != kDescGroup) d_grp = small_load(gd + k0 + lane);
            }
            if (mine) { u += (uint32_t)d_grp; fl |= ((uint32_t)(d_grp >> 40) & 0xFFu) ? 1u : 0u; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) { u += __shfl_xor(u, o, 64); fl |= __shfl_xor(fl, o, 64); }
        if (__builtin_expect(gave_up, 0)) {
            small_count_before<MANY>(a, slice, reinterpret_cast<uint32_t*>(s_offs), &u, &fl);
            if (nf == 1 && !onehot) {                      // (the offsets' place was used)
                const int k = small_step(B);
#pragma nounroll
                for (int i = lane; i < ((B + (1 << k) - 1) >> k) + 1; i += 64) s_offs[i] = as_global(a->offsets)[(int64_t)ss->field0 * B + min(i << k, B)];
            }
        }
        if (lane == 0) {
            s_base = (int)u;
            s_flag = (int)(fl | own_flags);
        }
    };
    // The slice's distinct keys (ascending) in their place, the pack's totals.  Returns false when the sums cannot be
    // right (then nothing is written): whatever the words held, no write below leaves the pack's arrays.
    auto after_wait = [&]() -> bool {
        const int base_u = s_base, pstart = s_ctx.pstart, nnz_p = s_ctx.nnz_p, rec_before = s_ctx.rec_before;
        if (base_u < 0 || rec_before < 0 || (int64_t)base_u + n_u > (int64_t)nnz_p || (int64_t)rec_before + n_rec > (int64_t)nnz_p) {
            if (tid == 0) ack2 = atomicOr(as_global(a->done) + 1, 2);
            return false;
        }
        uint32_t* uq = as_global(a->unique) + pstart + base_u;
        if (tid * wpt < words) {
            int at = (int)s_pre[tid * wpt];
            for (int j = 0; j < wpt; ++j) {
                const int w = tid * wpt + j;
                uint32_t x = s_bits[w];
                const uint32_t key0 = ss->key_lo + lo + (uint32_t)w * 32u;
                while (x) {
                    const int bit = __ffs(x) - 1;
                    x &= x - 1;
                    uq[at++] = key0 + bit;
                }
            }
        }
        if (ss->is_last && tid == 0) {
            PackState* st = as_global(a->st) + ss->pack;
            st->n_unique = base_u + n_u;
            as_global(a->seg_all)[pstart + ss->pack + base_u + n_u] = nnz_p;
            ack3 = atomicExch(&st->error, s_flag);
        }
        PK_PT(*a, slice, 5);
        return true;
    };

    // ---- occurrences per distinct key; every kept occurrence keeps its key's rank and its place among them ----
    const bool guessed = nf > 1 || onehot;                 // the bag is looked for first where it is if all hold one
    if (n_rec <= kSmallCache && n_u <= kSmallRanks) {
        constexpr int PER = kSmallCache / NTH;
        int q[PER], ra[PER], g0[PER], g1[PER];             // ra: rank | place << 16
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int i = tid + e * NTH;
            const bool on = i < n_rec;
            const uint32_t ck = on ? s_ckey[i] : 0u;
            q[e] = on ? s_cpos[i] : 0;
            const int32_t* tf = s_tf + (MANY ? kSliceTfWords * (int)(ck >> kSliceLogMax) : 0);
            const int guess = min(max(q[e] - (MANY ? tf[0] : s_ctx.q0), 0), B - 1);
            const int32_t* offs = as_global(a->offsets) + (int64_t)(MANY ? tf[4] >> 1 : ss->field0) * B;
            g0[e] = guessed ? offs[guess] : 0;             // the bag it is in if all hold one
            g1[e] = guessed ? offs[guess + 1] : 0;
            const int rk = small_rank(s_bits, s_pre, ck & kSmallKeyMask);
            ra[e] = rk;
            if (wv * 64 + e * NTH < n_rec) ra[e] |= lds_inc_grouped(s_cnt, (uint32_t)rk, on) << 16;
        }
        __syncthreads();
        PK_PT(*a, slice, 6);
        const int per = (n_u + NTH - 1) / NTH;
        const int s = small_sum(s_cnt, n_u, per);
        if (wv == 0) finish_wait();
        int tot;
        const int ex = block_excl_scan<NTH, true>(s, &tot);      // (its barriers also publish what wavefront 0 found)
        PK_PT(*a, slice, 4);
        const bool ok = after_wait();
        if (ok) small_starts(a, ss, s_cnt, s_ctx.pstart, s_base, 0, n_u, s_ctx.rec_before + ex, per);
        __syncthreads();
        PK_PT(*a, slice, 7);
        a = forget<LEAN>(a);
        ss = slice_at(a, slice);
        if (ok) {
            const int pstart = s_ctx.pstart, nnz_p = s_ctx.nnz_p, base_u = s_base;
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (tid + e * NTH < n_rec) {
                    const uint32_t ck = s_ckey[tid + e * NTH];
                    const int32_t* tf = s_tf + (MANY ? kSliceTfWords * (int)(ck >> kSliceLogMax) : 0);
                    const int first = MANY ? tf[0] : s_ctx.q0;
                    int L = g1[e] - g0[e], b = min(max(q[e] - first, 0), B - 1);
                    if (!guessed || q[e] < g0[e] || q[e] >= g1[e])
                        b = small_bag(as_global(a->offsets) + (int64_t)(MANY ? tf[4] >> 1 : ss->field0) * B, B, s_offs, !guessed, -1, q[e], &L);
                    const int rk = ra[e] & 0xFFFF;
                    small_place(a, ss, tf, pstart, nnz_p, base_u, ck & kSmallKeyMask, q[e], rk, s_cnt[rk] + (ra[e] >> 16), b, L);
                }
        }
    } else {
        // ---- more occurrences than are kept: from the IDs again, in rounds of as many keys as there is room for
        //      counters (that of the kept occurrences with it: slices of frequent keys have more than kSmallRanks, and a
        //      second round reads the IDs twice more) ----
        constexpr int RANKS = kSmallRanks + 2 * kSmallCache;
        for (int i = kSmallRanks + tid; i < min(RANKS, n_u); i += NTH) s_cnt[i] = 0;
        __syncthreads();
        // fn(field of the table, key in slice, position, on, bounds of the bag it is in if all hold one): all lanes make every trip
        auto for_ids = [&](auto bags, auto&& fn) {
            constexpr int UN = decltype(bags)::value ? 2 : 4;
            SmallField at;
            for (int base = 0; base < n_table; base += UN * NTH) {
                int64_t v[UN];
                int fj[UN], q[UN], g0[UN], g1[UN];
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int i = min(base + tid + u * NTH, n_table - 1);
                    q[u] = MANY ? at.position(s_tf, nf, n_table, i) : s_ctx.q0 + i;
                    fj[u] = MANY ? at.j : 0;
                    v[u] = as_global(a->ids)[q[u]];
                    g0[u] = g1[u] = 0;
                    if (decltype(bags)::value && guessed) {
                        const int32_t* tf = s_tf + kSliceTfWords * fj[u];
                        const int32_t* offs = as_global(a->offsets) + (int64_t)(tf[4] >> 1) * B + min(max(q[u] - tf[0], 0), B - 1);
                        g0[u] = offs[0]; g1[u] = offs[1];
                    }
                }
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const uint32_t kk = base + tid + u * NTH < n_table ? fold_id(v[u], ss->rows, ss->magic) : 0xFFFFFFFFu;
                    const bool on = (kk >> lg) == (uint32_t)ss->idx;
                    fn(fj[u], on ? kk - lo : 0u, q[u], on, g0[u], g1[u]);
                }
            }
        };
        int placed = 0;
        bool ok = true;
        for (int r0 = 0; ok && r0 < n_u; r0 += RANKS) {
            const int width = min(RANKS, n_u - r0);
            if (r0) {
                __syncthreads();
                for (int i = tid; i < width; i += NTH) s_cnt[i] = 0;
                __syncthreads();
            }
            for_ids(BoolTag<false>{}, [&](int, uint32_t kl, int, bool on, int, int) {
                const uint32_t rr = (uint32_t)(small_rank(s_bits, s_pre, kl) - r0);
                (void)lds_inc_grouped(s_cnt, rr, on && rr < (uint32_t)width);
            });
            __syncthreads();
            const int per = (width + NTH - 1) / NTH;
            const int s = small_sum(s_cnt, width, per);
            if (r0 == 0 && wv == 0) finish_wait();
            int tot;
            const int ex = block_excl_scan<NTH, true>(s, &tot);
            if (r0 == 0) {
                        ok = after_wait();
                a = forget<LEAN>(a);
                ss = slice_at(a, slice);
            }
            if (!ok) break;
            small_starts(a, ss, s_cnt, s_ctx.pstart, s_base, r0, width, s_ctx.rec_before + placed + ex, per);
            __syncthreads();
            for_ids(BoolTag<true>{}, [&](int j, uint32_t kl, int q, bool on, int g0, int g1) {
                const int rk = small_rank(s_bits, s_pre, kl);
                const uint32_t rr = (uint32_t)(rk - r0);
                on = on && rr < (uint32_t)width;
                const int pos = lds_inc_grouped(s_cnt, rr, on);
                if (on) {
                    const int32_t* tf = s_tf + kSliceTfWords * j;
                    int L = g1 - g0, b = min(max(q - tf[0], 0), B - 1);
                    if (!guessed || q < g0 || q >= g1) b = small_bag(as_global(a->offsets) + (int64_t)(tf[4] >> 1) * B, B, s_offs, !guessed, -1, q, &L);
                    small_place(a, ss, tf, s_ctx.pstart, s_ctx.nnz_p, s_base, kl, q, rk, pos, b, L);
                }
            });
            placed += tot;
        }
    }
    PK_PT(*a, slice, 8);
    // The words belong to the library and must be zero when the next call starts: the block that is through its
    // wait last (every block has then published, and read what it needed) clears them.
    if (wv == 0) {
        int last = 0;
        if (lane == 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::"v"(ack0), "v"(ack1), "v"(ack2), "v"(ack3) : "memory");      // this block's own words have arrived
            last = atomicAdd(as_global(a->done), 1) == a->n_slices - 1;
        }
        if (__builtin_amdgcn_readfirstlane(last)) {
            for (int i = lane; i < a->n_slices; i += 64) publish_desc(as_global(a->desc) + i, 0);
            for (int i = lane; i < a->n_slices / kDescGroup + a->P + 2; i += 64) publish_desc(as_global(a->gdesc) + i, 0);
            if (lane == 0) {
                *as_global(a->done) = 0;
                // a block found sums that cannot be: bit 1 of every pack's error word
                if (atomicExch(as_global(a->done) + 1, 0))
                    for (int k = 0; k < a->P; ++k) atomicOr(&as_global(a->st)[k].error, 2);
            }
        }
    }
}
