// H1 and H2: packed keys, distinct keys (ascending), the inverse index and the per-key occurrence
// lists, by slices of the key space.
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.
//
// Unique (Sec. II-D) is a set over the pack's rows, so it is built where a set of rows is cheap:
// a table's key range is cut into slices of 2^k keys, and ONE block owns a slice.  In LDS it keeps
// the slice's bitmap (which rows occur), the popcount prefix of the bitmap's words (the index of a
// key among the slice's distinct keys is a prefix plus a popcount) and one counter per distinct
// key.  From those it writes, for its slice, the ascending distinct keys, the segment offsets, the
// marks by which the backward pass finds long keys, and the occurrences grouped by key -- everything the backward
// pass reads.  What a slice needs from the others is two numbers, the distinct keys and the
// occurrences of the slices before it in the pack.
//
// Which occurrences belong to a slice:
//   small batches   every slice block scans the IDs of its table's fields and keeps those whose
//                   row falls into its slice, so the whole dedup, with the pooling beside it, is ONE
//                   launch (dev_small.h);
//   large batches   the occurrences are partitioned by slice first: the keys kernel counts them
//                   per slice (block-local counts in LDS, one global add per touched slice), a
//                   scan turns the counts into places, a scatter kernel writes a
//                   (key in slice, bag) record per occurrence to its slice's place, and the slice
//                   kernel reads its records; the inverse index is then looked up per occurrence
//                   from the bitmap and rank samples the slice kernel leaves in memory.

// ---------------------------------------------------------------------------
// Field boundaries, and where each field's occurrences go in the packed order (fields in
// (pack, slot) order, one after the other).  s_fb [F+1], s_delta [F] (packed position minus
// position in ids), s_slotpos [F+1] (packed position of each (pack, slot)).  Returns non-zero
// when the boundaries are unusable (offsets[0] != 0, offsets[F*B] != nnz, or decreasing).
// ---------------------------------------------------------------------------
constexpr size_t field_scan_words(int F) { return (size_t)(3 * F + 2); }

template <int NTH>
__device__ __forceinline__ int field_scan(const int32_t* __restrict__ offsets, int B, int F, int64_t nnz,
                                          const int32_t* __restrict__ slot_field, int32_t* s_fb, int32_t* s_delta,
                                          int32_t* s_slotpos)
{
    const int tid = threadIdx.x;
    for (int f = tid; f <= F; f += NTH) s_fb[f] = offsets[(int64_t)f * B];
    __syncthreads();
    int mine = 0;
    for (int f = tid; f < F; f += NTH) mine |= s_fb[f + 1] < s_fb[f];
    if (tid == 0) mine |= (s_fb[0] != 0 || (int64_t)s_fb[F] != nnz);
    const int bad = __syncthreads_or(mine);
    int carry = 0;
    for (int base = 0; base < F; base += NTH) {
        const int i = base + tid;
        int len = 0, f = 0;
        if (i < F) {
            f = slot_field[i];
            len = bad ? 0 : s_fb[f + 1] - s_fb[f];
        }
        int tot;
        const int ex = block_excl_scan<NTH>(len, &tot);
        if (i < F) {
            s_slotpos[i] = carry + ex;
            s_delta[f] = carry + ex - s_fb[f];
        }
        carry += tot;
    }
    if (tid == 0) s_slotpos[F] = carry;
    __syncthreads();
    return bad;
}

// the same from the copy the keys kernel left in memory: fscan = s_fb | s_delta | s_slotpos | verdict
template <int NTH>
__device__ __forceinline__ int field_scan_load(const int32_t* __restrict__ fscan, int F, int32_t* s_fb)
{
    for (int i = threadIdx.x; i < 3 * F + 2; i += NTH) s_fb[i] = fscan[i];
    const int bad = fscan[3 * F + 2];
    __syncthreads();
    return bad;
}

// The cut of every table for this batch, from the field sizes the offsets give (s_fb: where every
// field's occurrences begin).  s_first [T+1]: the first slice of every table, in table-list order
// (slices are numbered over all packs); s_lg [T]: log2 of the keys per slice.
template <int NTH>
__device__ __forceinline__ void table_cut(const TableMeta* __restrict__ tmeta, const FieldMeta* __restrict__ fmeta,
                                          int T, int F, const int32_t* s_fb, int target, int log_max,
                                          int32_t* s_first, int32_t* s_lg, TableCut* out)
{
    for (int t = threadIdx.x; t < T; t += NTH) s_lg[t] = 0;       // first the tables' occurrences
    __syncthreads();
    for (int f = threadIdx.x; f < F; f += NTH) atomicAdd(&s_lg[fmeta[f].stable], max(s_fb[f + 1] - s_fb[f], 0));
    __syncthreads();
    int carry = 0;
    for (int base = 0; base < T; base += NTH) {
        const int t = base + (int)threadIdx.x;
        SliceGeom g{0, 0};
        int occ = 0;
        if (t < T) {
            occ = s_lg[t];
            g = slice_geom(tmeta[t].rows, occ, target, log_max);
        }
        int tot;
        const int ex = block_excl_scan<NTH>(g.n, &tot);
        if (t < T) {
            s_first[t] = carry + ex;
            s_lg[t] = g.log_keys;
            if (out) out[t] = TableCut{g.log_keys, g.n, carry + ex, occ};
        }
        carry += tot;
    }
    if (threadIdx.x == 0) s_first[T] = carry;
    __syncthreads();
}

// the same from the array the keys kernel wrote
template <int NTH>
__device__ __forceinline__ void table_cut_load(const TableCut* __restrict__ cut, int T, int32_t* s_first, int32_t* s_lg)
{
    for (int t = threadIdx.x; t < T; t += NTH) {
        const TableCut c = cut[t];
        s_first[t] = c.first;
        if (s_lg) s_lg[t] = c.log_keys;
        if (t == T - 1) s_first[T] = c.first + c.n;
    }
    if (T == 0 && threadIdx.x == 0) s_first[0] = 0;
    __syncthreads();
}

// the bag of field-local offsets `offs` [B+1] that holds position q (offsets that are not monotone give
// some bag of the field: the answer stays in range)
__device__ __forceinline__ int find_bag(const int32_t* __restrict__ offs, int B, int q, int guess)
{
    if ((unsigned)guess < (unsigned)B && offs[guess] <= q && q < offs[guess + 1]) return guess;
    int lo = 0, hi = B + 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (offs[mid] <= q) lo = mid + 1; else hi = mid;
    }
    return min(max(lo - 1, 0), B - 1);
}

// Large batches, first launch: the per-slice counters are zeroed by all blocks; block 0 clears the
// pack states and makes what every later kernel reads instead of deriving it again: the field scan
// (with its verdict), the cut of every table for this batch, and the packs' sizes.
constexpr int kSetupThreads = 1024;         // block 0's scans run over up to 4096 fields and tables
__global__ void __launch_bounds__(kSetupThreads)
pk_setup_kernel(uint4* zero, int64_t n4, const int32_t* __restrict__ offsets, int B, int F, int P, int T, int64_t nnz,
                int target, int log_max, const FieldMeta* __restrict__ fmeta, const PackMeta* __restrict__ pm,
                const TableMeta* __restrict__ tmeta, const int32_t* __restrict__ slot_field, PackState* st,
                int32_t* __restrict__ packed_offsets, int32_t* __restrict__ seg_all, TableCut* __restrict__ cut,
                int n_slices_max, int32_t* __restrict__ fscan)
{
    extern __shared__ int32_t s_dyn[];                     // block 0: field scan | first slices, slice sizes
    const uint4 z = make_uint4(0, 0, 0, 0);
    for (int64_t i = (int64_t)blockIdx.x * kSetupThreads + threadIdx.x; i < n4; i += (int64_t)gridDim.x * kSetupThreads) zero[i] = z;
    if (blockIdx.x != 0) return;
    int32_t* s_fb = s_dyn;
    int32_t* s_delta = s_fb + (F + 1);
    int32_t* s_slotpos = s_delta + F;
    int32_t* s_first = s_slotpos + (F + 1);
    int32_t* s_lg = s_first + (T + 1);
    const int tid = threadIdx.x;
    int bad = field_scan<kSetupThreads>(offsets, B, F, nnz, slot_field, s_fb, s_delta, s_slotpos);
    table_cut<kSetupThreads>(tmeta, fmeta, T, F, s_fb, target, log_max, s_first, s_lg, cut);
    bad |= s_first[T] > n_slices_max;                      // cannot be for offsets that pass the scan: the slices' arrays are that long
    for (int i = tid; i < 3 * F + 2; i += kSetupThreads) fscan[i] = s_fb[i];
    if (tid == 0) fscan[3 * F + 2] = bad;
    for (int p = tid; p < P; p += kSetupThreads) {
        const PackMeta k = pm[p];
        const int start = s_slotpos[k.first_slot];
        const int n = s_slotpos[k.first_slot + k.n_fields] - start;
        PackState ps{};
        ps.nnz = n; ps.start = start; ps.first_slice = s_first[k.first_stable]; ps.error = bad ? 1 : 0;
        st[p] = ps;
        if (k.n_stables == 0) seg_all[start + p] = 0;      // no table that a field reads: no slice writes the end of its segments
        packed_offsets[(int64_t)k.first_slot * B + p + (int64_t)k.n_fields * B] = n;
    }
}

// ---------------------------------------------------------------------------
// Large batches, H1: packed keys (Sec. III-B: one packed ID tensor per pack), packed bag offsets,
// and how many occurrences fall into every slice.  A tile is BT consecutive bags of ONE field, so
// its IDs are contiguous and hit one table; the tile's counts per slice are tallied in LDS and
// added to the slices' totals with one global add per touched slice.  The offsets of a tile are
// checked here: inside their field's range and not decreasing, else bit 0 of the pack's error
// word is raised and the tile is skipped (the kernels after this one skip that pack).
// ---------------------------------------------------------------------------
struct TileOf {
    int f, b0, nb;
    __device__ __forceinline__ TileOf(int64_t tile, int tiles_per_field, int B, int BT)
    {
        f = (int)(tile / tiles_per_field);
        b0 = (int)(tile - (int64_t)f * tiles_per_field) * BT;
        nb = min(BT, B - b0);
    }
};

__global__ void __launch_bounds__(NT)
pk_keys_kernel(const int64_t* __restrict__ ids, const int32_t* __restrict__ offsets, int B, int F, int BT,
               const FieldMeta* __restrict__ fmeta, const PackMeta* __restrict__ pm, PackState* st,
               uint32_t* __restrict__ keys, int32_t* __restrict__ packed_offsets, int32_t* slice_total,
               const TableCut* __restrict__ cut, const int32_t* __restrict__ fscan, int32_t* __restrict__ tile_hist,
               int tile_hist_stride)
{
    extern __shared__ int32_t s_dyn[];                     // the tile's bag offsets | its counts per slice of its table
    int32_t* s_po = s_dyn;
    int32_t* s_hist = s_po + BT + 1;
    __shared__ int s_flag;
    const int tid = threadIdx.x;
    if (fscan[3 * F + 2]) return;                          // the field boundaries are unusable: the packs' error words say so
    const int32_t* fb = fscan;                             // where every field's occurrences begin
    const int32_t* delta = fscan + (F + 1);                // packed position minus position in ids, per field
    const int32_t* slotpos = delta + F;                    // packed position of each (pack, slot)
    const int tpf = (B + BT - 1) / BT;
    const int64_t n_tiles = (int64_t)F * tpf;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const TileOf tl(tile, tpf, B, BT);
        const int f = tl.f;
        const FieldMeta m = fmeta[f];
        const PackMeta k = pm[m.pack];
        const TableCut tc = cut[m.stable];
        const int f_lo = fb[f], f_hi = fb[f + 1];
        const int dl = delta[f];
        const int pbase = slotpos[k.first_slot];
        SliceGeom g;
        g.log_keys = tc.log_keys;
        g.n = tc.n;
        const int64_t g0 = (int64_t)f * B + tl.b0;
        __syncthreads();                                   // the previous tile's LDS is consumed
        for (int t = tid; t <= tl.nb; t += NT) s_po[t] = offsets[g0 + t];
        for (int s = tid; s < g.n; s += NT) s_hist[s] = 0;
        if (tid == 0) s_flag = 0;
        __syncthreads();
        for (int t = tid; t < tl.nb; t += NT)
            if (s_po[t] > s_po[t + 1] || s_po[t] < f_lo || s_po[t + 1] > f_hi) s_flag = 1;
        __syncthreads();
        if (s_flag) {
            if (tid == 0) atomicOr(&st[m.pack].error, 1);
            continue;
        }
        for (int t = tid; t < tl.nb; t += NT)
            packed_offsets[(int64_t)k.first_slot * B + m.pack + (int64_t)m.slot * B + tl.b0 + t] = s_po[t] + dl - pbase;
        const int q_lo = s_po[0], q_hi = s_po[tl.nb];
        for (int base = q_lo; base < q_hi; base += 4 * NT) {       // the same trips for every lane: lanes combine their counts
            int64_t idv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {                  // the loads of four rounds in flight together
                const int i = base + tid + j * NT;
                idv[j] = i < q_hi ? ids[i] : 0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = base + tid + j * NT;
                const bool on = i < q_hi;
                const uint32_t kk = on ? fold_id(idv[j], m.rows, m.magic) : 0u;
                if (on) keys[i + dl] = m.base_row + kk;
                if (g.n <= kFewCounters) (void)lds_inc_few<false>(s_hist, kk >> g.log_keys, on, g.n);
                else if (on) atomicAdd(&s_hist[kk >> g.log_keys], 1);
            }
        }
        __syncthreads();
        const int slice0 = tc.first;
        for (int s = tid; s < g.n; s += NT) {
            const int c = s_hist[s];
            if (c) atomicAdd(&slice_total[slice0 + s], c);
            if (tile_hist) tile_hist[tile * tile_hist_stride + s] = c;     // the scatter kernel takes its counts from here
        }
    }
}

constexpr int kBigSlicesMax = 256;         // listed slices with many records
constexpr int kBigSliceFlag = 1 << 30;     // in SliceInfo::table: the slice is listed
constexpr int kBigSliceCount = 6144;       // records from which a slice is listed

// Large batches: the slices' totals become places.  A block takes 1024 slices; what lies before them
// it adds up itself (there are some thousand slices: a block reads a few values per thread).  Every slice
// gets its table, its index in the table, the place of its first record and the number of records; the
// cursors of the scatter kernel start at those places.
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads)
pk_slice_scan_kernel(const TableCut* __restrict__ cut, int T,
                     const int32_t* __restrict__ slice_total, int32_t* __restrict__ slice_cursor,
                     SliceInfo* __restrict__ slice_info, int n_slices, int big_count, int32_t* n_big,
                     int32_t* __restrict__ big_list)
{
    extern __shared__ int32_t s_first[];                   // [T+1]
    table_cut_load<kScanThreads>(cut, T, s_first, nullptr);
    const int base = blockIdx.x * kScanThreads;
    int before = 0;
    for (int i = threadIdx.x; i < base; i += kScanThreads) before += slice_total[i];
    int carry;
    (void)block_excl_scan<kScanThreads>(before, &carry);
    const int s = base + (int)threadIdx.x;
    const int c = s < n_slices ? slice_total[s] : 0;
    int tot;
    const int ex = block_excl_scan<kScanThreads>(c, &tot);
    if (s < n_slices) {
        const int t = upper_bound_i32(s_first, T + 1, s) - 1;
        SliceInfo si;
        si.table = t; si.idx = s - s_first[t]; si.start = carry + ex; si.count = c;
        if (s >= s_first[T]) { si.table = -1; si.idx = 0; si.count = 0; }      // room for slices this batch does not have
        // A slice that holds a hot key has many times the records of the others: such slices are listed,
        // and blocks of four times the threads take them, in launches that run beside the others'.
        if (c > big_count && si.table >= 0) {
            const int at = atomicAdd(n_big, 1);
            if (at < kBigSlicesMax) {
                big_list[at] = s;
                si.table |= kBigSliceFlag;
            }
        }
        slice_info[s] = si;
        slice_cursor[s] = carry + ex;
    }
}

// Large batches: one record per occurrence, (key inside its slice, place of its bag's gradient chunk), written to
// the slice's place.  A tile counts its occurrences per slice in LDS, reserves room in every
// touched slice with one global add, and then places its records from block-local cursors: one LDS word per slice
// of the tile's table, first its count, then its cursor (a table has up to kTableSlicesMax).
__global__ void __launch_bounds__(NT)
pk_scatter_kernel(const int32_t* __restrict__ offsets, int B, int F, int BT, int64_t nnz, int log_max,
                  const FieldMeta* __restrict__ fmeta, const TableCut* __restrict__ cut,
                  const PackState* __restrict__ st, const uint32_t* __restrict__ keys, int32_t* slice_cursor,
                  uint2* __restrict__ rec, int64_t out_dim, const int32_t* __restrict__ fscan,
                  const int32_t* __restrict__ tile_hist, int tile_hist_stride)
{
    extern __shared__ int32_t s_dyn[];                     // the tile's bag offsets | per slice of its table: count, then place
    int32_t* s_po = s_dyn;
    int32_t* s_hist = s_po + BT + 1;
    const int tid = threadIdx.x;
    if (fscan[3 * F + 2]) return;
    const int32_t* delta = fscan + (F + 1);
    const int tpf = (B + BT - 1) / BT;
    const int64_t n_tiles = (int64_t)F * tpf;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const TileOf tl(tile, tpf, B, BT);
        const int f = tl.f;
        const FieldMeta m = fmeta[f];
        if (st[m.pack].error) continue;                    // the keys kernel rejected offsets of this pack
        const TableCut tc = cut[m.stable];
        const int dl = delta[f];
        SliceGeom g;
        g.log_keys = tc.log_keys;
        g.n = tc.n;
        const int64_t g0 = (int64_t)f * B + tl.b0;
        __syncthreads();
        for (int t = tid; t <= tl.nb; t += NT) s_po[t] = offsets[g0 + t];
        for (int s = tid; s < g.n; s += NT) s_hist[s] = tile_hist ? tile_hist[tile * tile_hist_stride + s] : 0;
        __syncthreads();
        const int q_lo = s_po[0], q_hi = s_po[tl.nb];
        if (tile_hist) {
            // one word of every 128 bytes of the tile's keys, so that the placing pass finds them in the cache
            uint32_t pf = 0;
            for (int i = q_lo + tid * 32; i < q_hi; i += NT * 32) pf ^= keys[i + dl];
            asm volatile("" ::"v"(pf));
        }
        if (!tile_hist)                                    // (the keys kernel's counts of this tile were not kept)
        for (int base = q_lo; base < q_hi; base += 4 * NT) {      // four loads in flight
            uint32_t kv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + tid + u * NT;
                kv[u] = i < q_hi ? keys[i + dl] - m.base_row : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t s = kv[u] >> g.log_keys;
                if (g.n <= kFewCounters) (void)lds_inc_few<false>(s_hist, s, s < (uint32_t)g.n, g.n);
                else if (s < (uint32_t)g.n) atomicAdd(&s_hist[s], 1);
            }
        }
        __syncthreads();
        const int slice0 = tc.first;
        for (int s = tid; s < g.n; s += NT) {
            const int c = s_hist[s];
            s_hist[s] = c ? atomicAdd(&slice_cursor[slice0 + s], c) : 0;
        }
        __syncthreads();
        // Every wavefront takes a contiguous quarter of the tile's positions, 64 at a time, so that a lane's
        // positions rise by 64 from one to the next: where bags are not short, the bag of a position is found
        // by stepping on from the bag of the lane's previous one (one search at the start).
        const int lane = tid & 63;
        const int per_wave = ((q_hi - q_lo + NT - 1) / NT) * 64;
        const int w_lo = q_lo + (tid >> 6) * per_wave, w_hi = min(w_lo + per_wave, q_hi);
        const bool stepped = (int64_t)tl.nb * 64 <= (int64_t)6 * (q_hi - q_lo);     // (short bags: a search per position is shorter)
        int t = stepped && w_lo + lane < w_hi ? upper_bound_i32(s_po, tl.nb + 1, w_lo + lane) - 1 : 0;
        constexpr int UP = 8;                              // key loads in flight (they come from memory: nothing has read them since they were written)
        for (int base = w_lo; base < w_hi; base += UP * 64) {
            uint32_t kv[UP];
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                const int i = base + u * 64 + lane;
                kv[u] = i < w_hi ? keys[i + dl] - m.base_row : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                const int i = base + u * 64 + lane;
                const uint32_t kk = kv[u];
                const uint32_t s = kk >> g.log_keys;
                const bool valid = i < w_hi && s < (uint32_t)g.n;
                if (i < w_hi) {
                    if (stepped) { while (t + 1 < tl.nb && s_po[t + 1] <= i) ++t; }
                    else if (valid) t = upper_bound_i32(s_po, tl.nb + 1, i) - 1;
                }
                int at = 0;
                if (g.n <= kFewCounters) at = lds_inc_few<true>(s_hist, s, valid, g.n);   // (all lanes of the wavefront are here)
                else if (valid) at = atomicAdd(&s_hist[s], 1);
                if (!valid) continue;
                // the record: key inside the slice, the gradient's scale (bag length for mean pooling, 1 for sum;
                // 0 = too long for its bits, to be looked up) above it, and the place of the bag's gradient chunk
                uint32_t len = 1u;
                if (m.pool == PK_MEAN) {
                    const uint32_t L = (uint32_t)max(s_po[t + 1] - s_po[t], 1);
                    len = (L >> (32 - log_max)) ? 0u : L;
                }
                if ((uint64_t)(int64_t)at < (uint64_t)nnz)
                    rec[at] = make_uint2((kk - (s << g.log_keys)) | (len << log_max),
                                         (uint32_t)((int64_t)(tl.b0 + t) * out_dim + m.col));
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The slice kernel's body.
// ---------------------------------------------------------------------------
// a field of a table as the slice blocks need it; static, device side, indexed like the table field list
struct TableField { int32_t field, slot, col, pool; };

struct SliceArgs {
    const TableMeta* tmeta; const TableField* tfields; int T;
    const PackMeta* pm; const int32_t* slot_field; PackState* st; int P;
    int F, B; int64_t nnz; int target, log_max;
    const int64_t* ids; const int32_t* offsets; const SmallSlice* small_slices; const int2* slot_info;   // small batches: the block finds its occurrences itself
    const SliceInfo* slice_info; const uint2* rec;              // large batches: the slice's records
    const TableCut* cut;                                        // ... and the tables' cuts for this batch
    const FieldMeta* fmeta;
    int32_t* packed_offsets;
    uint32_t* keys; int32_t* inverse;                           // written here for small batches only
    uint32_t* bitmap; int32_t* slice_nu;                        // large batches only: bitmaps with rank samples, distinct keys per slice
    const int32_t* big_list; const int32_t* n_big;              // ... and the listed slices with many records
    uint32_t* unique; int32_t* seg_all; uint32_t* ent_all; int ent_mult;
    int32_t* marks; double* ghot; int32_t* ticket; int dmax;
    uint64_t* desc; uint64_t* gdesc; int32_t* done; int n_slices;   // small batches: descriptors the library owns, cleaned by the last block
    int64_t out_dim;
#ifdef PK_PHASE_TIMES
    long long* ptimes;
#endif
};
#ifdef PK_PHASE_TIMES
#define PK_PT(a, blk, k) do { if (threadIdx.x == 0 && (a).ptimes) (a).ptimes[(size_t)(blk) * 16 + (k)] = wall_clock64(); } while (0)
#else
#define PK_PT(a, blk, k) do { } while (0)
#endif

// LDS words of a slice block: bitmap words | their popcount prefix | counters of a round of distinct keys
constexpr int slice_lds_words(int log_max, int ranks) { return 2 * (1 << (log_max - 5)) + ranks; }
constexpr int kSliceTfWords = 5;           // dynamic LDS words per field of a table

// one occurrence of a slice: key minus the slice's first key, the place of its gradient chunk, the chunk's scale
struct SliceRec { uint32_t kl, ref, L; };

// MODE: what the block does with its slice of a large batch
//   kSliceMark   first half: which keys occur -> the slice's bitmap and its number of distinct keys
//   kSlicePlace  second half (after a scan of those numbers): everything else
// (With thousands of slices in flight a look-back makes every block wait for the slowest slice before it;
// two launches with a scan between them let every block run without waiting.)
enum { kSliceMark = 1, kSlicePlace = 2 };

template <int MODE, int NTH, int LOGMAX, int RANKS, bool BIG = false>
__device__ __forceinline__ void slice_body(const SliceArgs& a, int slice, int32_t* s_main, int32_t* s_tf)
{
    constexpr bool GROUPED = BIG || NTH > 256;             // lanes that share a key combine their counter updates
    constexpr int WMAX = 1 << (LOGMAX - 5);
    constexpr int KEEP = NTH > 256 ? 0 : 12;               // records per thread whose rank and place stay in a register
    const int tid = threadIdx.x;
    uint32_t* s_bits = reinterpret_cast<uint32_t*>(s_main);
    uint32_t* s_pre = s_bits + WMAX;
    int32_t* s_cnt = s_main + 2 * WMAX;
    const int B = a.B;
    const int64_t out_dim = a.out_dim;

    // ---- which slice, of which table; where the pack's arrays start ----
    const SliceInfo si = a.slice_info[slice];
    if (si.table < 0) return;                              // room for a slice this batch does not have
    if (BIG != ((si.table & kBigSliceFlag) != 0)) return;  // listed slices belong to the launch that takes the list
    const int t = si.table & ~kBigSliceFlag, idx = si.idx, rec_start = si.start, n_rec = si.count;
    const TableMeta tm = a.tmeta[t];
    const int p = tm.pack, nf = tm.field_end - tm.field_begin;
    const uint32_t key_lo = tm.key_lo, rows = tm.rows;
    const TableCut tc = a.cut[t];
    const int lg = tc.log_keys;
    const PackMeta k = a.pm[p];
    const int pstart = a.st[p].start, nnz_p = a.st[p].nnz, pack_first = a.st[p].first_slice;
    const bool is_last = t == k.first_stable + k.n_stables - 1 && idx + 1 == tc.n;     // last slice of the pack's last table
    if (a.st[p].error) return;                             // offsets of this pack were rejected
    if (MODE == kSlicePlace)
        for (int j = tid; j < nf; j += NTH) {
            const TableField tf = a.tfields[tm.field_begin + j];
            s_tf[kSliceTfWords * j] = tf.slot;
            s_tf[kSliceTfWords * j + 3] = tf.col;
        }
    const uint32_t lo = (uint32_t)idx << lg;               // first key of the slice inside its table
    const uint32_t nkeys = min((uint32_t)1 << lg, rows - lo);
    const int words = 1 << (lg - 5);

    // all records of the slice: fn(SliceRec, on).  Every lane makes the same trips and calls fn every time, with
    // on = false where it has none, so that fn may combine lanes.
    const uint2* __restrict__ rec = a.rec + rec_start;
    auto unpack = [&](uint2 r, bool valid, bool* on) {
        const uint32_t kl = r.x & ((1u << LOGMAX) - 1u);
        *on = valid && kl < nkeys;
        return SliceRec{*on ? kl : 0u, r.y, r.x >> LOGMAX};
    };
    auto for_records = [&](auto&& fn) {
        constexpr int UN = BIG ? 8 : 4;                    // records per thread in flight: a listed slice is long
        for (int base = 0; base < n_rec; base += UN * NTH) {
            uint2 r[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int i = base + tid + u * NTH;
                r[u] = i < n_rec ? rec[i] : make_uint2(0, 0);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                bool on;
                const SliceRec x = unpack(r[u], base + tid + u * NTH < n_rec, &on);
                fn(x, on);
            }
        }
    };

    // ---- which keys occur ----
    // The slice's bitmap in memory: word w of the table's bitmap stands at w + w / 3 of the table's
    // region, so that every 16 bytes hold three words and, in the fourth, the rank of their first key.
    uint32_t* bmw = a.bitmap + tm.word_base;
    const uint32_t tw0 = (uint32_t)idx * (uint32_t)words;
    if (MODE == kSliceMark) {
        for (int w = tid; w < words; w += NTH) s_bits[w] = 0;
        __syncthreads();
        for_records([&](const SliceRec& r, bool on) {
            if (on) {
                const uint32_t bit = 1u << (r.kl & 31);
                if (!(s_bits[r.kl >> 5] & bit)) atomicOr(&s_bits[r.kl >> 5], bit);
            }
        });
        __syncthreads();
        int c = 0;
        for (int w = tid; w < words; w += NTH) {
            const uint32_t x = s_bits[w];
            bmw[tw0 + w + (tw0 + w) / 3u] = x;             // the bitmap and the count go to memory; the rest follows the scan
            c += __popc(x);
        }
        int n_u;
        (void)block_excl_scan<NTH>(c, &n_u);
        if (tid == 0) a.slice_nu[slice] = n_u;
        return;
    }
    for (int w = tid; w < words; w += NTH) s_bits[w] = bmw[tw0 + w + (tw0 + w) / 3u];
    for (int i = tid; i < RANKS; i += NTH) s_cnt[i] = 0;
    const int base_u = a.slice_nu[slice] - a.slice_nu[pack_first];     // scanned: distinct keys of the pack's slices before
    const int rec_before = rec_start - pstart;
    __syncthreads();
    // popcount prefix of the words: thread i owns words [i * wpt, (i + 1) * wpt)
    const int wpt = max(1, words / NTH);
    int c = 0;
    if (tid * wpt < words)
        for (int j = 0; j < wpt; ++j) c += __popc(s_bits[tid * wpt + j]);
    int n_u;
    const int ex = block_excl_scan<NTH>(c, &n_u);
    // whatever the sums hold, no write below leaves the pack's arrays
    if (base_u < 0 || rec_before < 0 || (int64_t)base_u + n_u > (int64_t)nnz_p || (int64_t)rec_before + n_rec > (int64_t)nnz_p) {
        if (tid == 0) atomicOr(&a.st[p].error, 2);
        return;
    }
    uint32_t* __restrict__ uq = a.unique + pstart;
    int32_t* __restrict__ seg = a.seg_all + pstart + p;
    if (tid * wpt < words) {                               // prefix, and the slice's distinct keys (ascending) in their place
        int run = ex;
        for (int j = 0; j < wpt; ++j) {
            const int w = tid * wpt + j;
            s_pre[w] = (uint32_t)run;
            uint32_t x = s_bits[w];
            const uint32_t key0 = key_lo + lo + (uint32_t)w * 32u;
            while (x) {
                const int bit = __ffs(x) - 1;
                x &= x - 1;
                uq[base_u + run++] = key0 + bit;
            }
        }
    }
    if (is_last && tid == 0) {
        a.st[p].n_unique = base_u + n_u;
        seg[base_u + n_u] = nnz_p;
    }
    __syncthreads();
    for (uint32_t u = (tw0 + 2u) / 3u + tid; 3u * u < tw0 + (uint32_t)words; u += NTH)     // rank samples beside the bitmap, for the inverse kernel
        bmw[4u * u + 3u] = (uint32_t)(base_u + (int)s_pre[3u * u - tw0]);
    if (n_u == 0) return;

    // ---- occurrences per distinct key, segment offsets, marks for the backward pass, and every
    //      occurrence's gradient place at its key's next free position; a round handles RANKS keys ----
    const int dim = k.dim;
    const bool wide = k.has_mean != 0;                     // the pack's entries carry the bag length
    uint32_t* __restrict__ ent = a.ent_all + (size_t)pstart * a.ent_mult;
    int32_t* __restrict__ marks = a.marks + (pstart / kMarkStep + p);
    const int32_t* __restrict__ po = a.packed_offsets + (int64_t)k.first_slot * B + p;
    auto rank_of = [&](uint32_t kl) {
        return (int)(s_pre[kl >> 5] + __popc(s_bits[kl >> 5] & ((1u << (kl & 31)) - 1u)));
    };
    auto put = [&](const SliceRec& r, int pos) {
        if ((unsigned)pos >= (unsigned)nnz_p) return;
        if (!wide) { ent[pos] = r.ref; return; }
        uint32_t len = r.L;
        if (len == 0) {                                    // a bag too long for the record's bits: its length from the bag
            const uint32_t b = r.ref / (uint32_t)out_dim, col = r.ref - b * (uint32_t)out_dim;
            int j = 0;
            while (j + 1 < nf && (uint32_t)s_tf[kSliceTfWords * j + 3] != col) ++j;
            const uint32_t g = (uint32_t)s_tf[kSliceTfWords * j] * (uint32_t)B + b;
            len = (uint32_t)max(po[g + 1] - po[g], 1);
        }
        reinterpret_cast<uint2*>(ent)[pos] = make_uint2(r.ref, len);
    };
    // counters of keys [r0, r0 + width) become the keys' first places; segment offsets and marks go out
    int placed = 0;                                        // occurrences of the keys of earlier rounds
    auto starts = [&](int r0, int width) {
        const int per = (width + NTH - 1) / NTH;           // consecutive counters per thread
        int sum = 0;
        for (int j = 0; j < per; ++j) {
            const int i = tid * per + j;
            sum += i < width ? s_cnt[i] : 0;
        }
        int tot;
        const int ex_occ = block_excl_scan<NTH>(sum, &tot);
        int s0 = rec_before + placed + ex_occ;
        for (int j = 0; j < per; ++j) {
            const int i = tid * per + j;
            if (i < width) {
                const int len = s_cnt[i];
                const int u = base_u + r0 + i;
                seg[u] = s0;
                s_cnt[i] = s0;
                // every kMarkStep-th position names its key: how the backward pass finds the long ones
                for (int m = (s0 + kMarkStep - 1) / kMarkStep; (int64_t)m * kMarkStep < (int64_t)s0 + len; ++m) marks[m] = u;
                if (len >= 2 * kPiece) {                   // the key is reduced in pieces: its partial sums start at zero
                    const size_t slot = (size_t)(pstart / kPiece + p) + (size_t)(s0 / kPiece);    // (no two such keys share one)
                    double* gh = a.ghot + slot * a.dmax;
                    for (int d = 0; d < dim; ++d) gh[d] = 0.0;
                    a.ticket[slot] = 0;
                }
                s0 += len;
            }
        }
        placed += tot;
    };
    if (KEEP && n_rec <= KEEP * NTH && n_u <= RANKS) {
        // The counting pass gives every record its key's rank and its place among the key's occurrences: both fit a
        // register, and the placing pass needs no counter.
        uint32_t rp[KEEP ? KEEP : 1];
#pragma unroll
        for (int u0 = 0; u0 < KEEP; u0 += 4) {
            if (u0 * NTH >= n_rec) break;
            uint2 r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = tid + (u0 + u) * NTH;
                r[u] = i < n_rec ? rec[i] : make_uint2(0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                bool on;
                const SliceRec x = unpack(r[u], tid + (u0 + u) * NTH < n_rec, &on);
                const uint32_t rk = (uint32_t)rank_of(x.kl);
                rp[u0 + u] = on ? rk | ((uint32_t)atomicAdd(&s_cnt[rk], 1) << 16) : 0xFFFFFFFFu;
            }
        }
        __syncthreads();
        starts(0, n_u);
        __syncthreads();
#pragma unroll
        for (int u0 = 0; u0 < KEEP; u0 += 4) {
            if (u0 * NTH >= n_rec) break;
            uint2 r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = tid + (u0 + u) * NTH;
                r[u] = i < n_rec ? rec[i] : make_uint2(0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                bool on;
                const SliceRec x = unpack(r[u], tid + (u0 + u) * NTH < n_rec, &on);
                if (on) put(x, s_cnt[rp[u0 + u] & 0xFFFFu] + (int)(rp[u0 + u] >> 16));
            }
        }
        return;
    }
    for (int r0 = 0; r0 < n_u; r0 += RANKS) {
        const int width = min(RANKS, n_u - r0);
        if (r0) {
            __syncthreads();
            for (int i = tid; i < width; i += NTH) s_cnt[i] = 0;
            __syncthreads();
        }
        for_records([&](const SliceRec& r, bool on) {
            const uint32_t rr = (uint32_t)(rank_of(r.kl) - r0);
            if (GROUPED) (void)lds_inc_grouped(s_cnt, rr, on && rr < (uint32_t)width);
            else if (on && rr < (uint32_t)width) atomicAdd(&s_cnt[rr], 1);
        });
        __syncthreads();
        starts(r0, width);
        __syncthreads();
        for_records([&](const SliceRec& r, bool on) {
            const uint32_t rr = (uint32_t)(rank_of(r.kl) - r0);
            on = on && rr < (uint32_t)width;
            int pos = 0;
            if (GROUPED) pos = lds_inc_grouped(s_cnt, rr, on);
            else if (on) pos = atomicAdd(&s_cnt[rr], 1);
            if (on) put(r, pos);
        });
    }
}

// Large batches: one block per slice, in two launches with a scan between them.
constexpr int kFineThreads = 256, kFineRanks = 2048;
constexpr int kSliceThreads = 1024, kSliceRanks = 8192;

template <int MODE>
__global__ void __launch_bounds__(kFineThreads, 8)
pk_slices_kernel(SliceArgs a)
{
    extern __shared__ int32_t s_dyn[];
    __shared__ int32_t s_main[slice_lds_words(kSliceLogFine, kFineRanks)];
    slice_body<MODE, kFineThreads, kSliceLogFine, kFineRanks>(a, blockIdx.x, s_main, s_dyn);
}

// ... the listed slices with many records: four times the threads, same cut
template <int MODE>
__global__ void __launch_bounds__(kSliceThreads)
pk_slices_big_kernel(SliceArgs a)
{
    extern __shared__ int32_t s_dyn[];
    __shared__ int32_t s_main[slice_lds_words(kSliceLogFine, kSliceRanks)];
    if ((int)blockIdx.x >= min(*a.n_big, kBigSlicesMax)) return;
    slice_body<MODE, kSliceThreads, kSliceLogFine, kSliceRanks, true>(a, a.big_list[blockIdx.x], s_main, s_dyn);
}

// ... and the shape for calls with a table too long for slices of 32 K keys
template <int MODE>
__global__ void __launch_bounds__(kSliceThreads)
pk_slices_wide_kernel(SliceArgs a)
{
    extern __shared__ int32_t s_dyn[];
    __shared__ int32_t s_main[slice_lds_words(kSliceLogMax, kSliceRanks)];
    slice_body<MODE, kSliceThreads, kSliceLogMax, kSliceRanks>(a, blockIdx.x, s_main, s_dyn);
}

// Large batches: the slices' numbers of distinct keys become running sums, in place (exclusive, over all
// packs; a slice takes the difference to its pack's first slice).  Blocks as in the scan of the records.
__global__ void __launch_bounds__(kScanThreads)
pk_unique_scan_kernel(int32_t* __restrict__ slice_nu, int n_slices, int32_t* __restrict__ sums)
{
    const int base = blockIdx.x * kScanThreads;
    int before = 0;
    for (int i = threadIdx.x; i < base; i += kScanThreads) before += slice_nu[i];
    int carry;
    (void)block_excl_scan<kScanThreads>(before, &carry);
    const int s = base + (int)threadIdx.x;
    const int c = s < n_slices ? slice_nu[s] : 0;
    int tot;
    const int ex = block_excl_scan<kScanThreads>(c, &tot);
    if (s < n_slices) sums[s] = carry + ex;
}

// Small batches: the blocks beside the slice blocks that write what is per bag and per pack:
// packed bag offsets and the packs' sizes.  (The slice blocks check the offsets.)
__device__ __forceinline__ void meta_body(const SliceArgs& a, int block, int nblocks, int32_t* s_main)
{
    const int F = a.F, B = a.B, P = a.P, tid = threadIdx.x;
    int32_t* s_fb = s_main;
    int32_t* s_delta = s_fb + (F + 1);
    int32_t* s_slotpos = s_delta + F;
    const int bad = field_scan<kSliceThreads>(a.offsets, B, F, a.nnz, a.slot_field, s_fb, s_delta, s_slotpos);
    if (block == 0) {
        for (int p = tid; p < P; p += kSliceThreads) {
            const PackMeta k = a.pm[p];
            const int start = s_slotpos[k.first_slot];
            const int n = s_slotpos[k.first_slot + k.n_fields] - start;
            a.st[p].nnz = n;
            a.st[p].start = start;
            a.st[p].first_slice = 0;
            if (k.n_stables == 0) {                        // no slice block writes these
                a.st[p].n_unique = 0;
                a.st[p].error = bad ? 1 : 0;
                a.seg_all[start + p] = 0;
            }
            a.packed_offsets[(int64_t)k.first_slot * B + p + (int64_t)k.n_fields * B] = n;
        }
    }
    if (bad) return;
    int32_t* po = a.packed_offsets;
    const int64_t n_bags = (int64_t)F * B;
    for (int64_t g = (int64_t)block * kSliceThreads + tid; g < n_bags; g += (int64_t)nblocks * kSliceThreads) {
        const int f = (int)(g / B);
        const int b = (int)(g - (int64_t)f * B);
        const FieldMeta m = a.fmeta[f];
        const PackMeta k = a.pm[m.pack];
        const int o = min(max(a.offsets[g], s_fb[f]), s_fb[f + 1]);
        po[(int64_t)k.first_slot * B + m.pack + (int64_t)m.slot * B + b] = o + s_delta[f] - s_slotpos[k.first_slot];
    }
}

// ---------------------------------------------------------------------------
// Large batches: inverse[q] = number of distinct keys of the pack below key[q]: the rank sample that
// stands beside the key's three bitmap words (written by the slice kernel) plus the set bits before
// the key among them: one 16-byte read per position.  Tiles of KT consecutive positions of the packed order (all packs in one launch); which
// table a position belongs to follows from where its field's occurrences start, staged in LDS with
// the table's first key and the place of its bitmap.
// ---------------------------------------------------------------------------
template <int KT>
__global__ void __launch_bounds__(NT)
pk_inverse_kernel(int F, const int32_t* __restrict__ fscan, const SlotMeta* __restrict__ slot_meta,
                  const PackState* __restrict__ st, const uint32_t* __restrict__ keys,
                  const uint4* __restrict__ bitmap4, int32_t* __restrict__ inverse)
{
    extern __shared__ int32_t s_dyn[];                     // field scan | per slot: first key, bitmap place, rows, the pack's error word
    int32_t* s_fb = s_dyn;
    int32_t* s_slotpos = s_fb + (F + 1) + F;
    uint32_t* s_klo = reinterpret_cast<uint32_t*>(s_slotpos + (F + 1));
    uint32_t* s_wb = s_klo + F;
    uint32_t* s_rows = s_wb + F;
    int32_t* s_pack = reinterpret_cast<int32_t*>(s_rows + F);
    for (int j = threadIdx.x; j < F; j += NT) {
        const SlotMeta m = slot_meta[j];
        s_klo[j] = m.key_lo; s_wb[j] = m.word_base; s_rows[j] = m.rows; s_pack[j] = st[m.pack].error;   // (the error word, final by now)
    }
    if (field_scan_load<NT>(fscan, F, s_fb)) return;
    const int n = s_slotpos[F];
    const int n_tiles = (n + KT - 1) / KT;
    for (XcdTiles it(n_tiles); it.valid(); it.next()) {
        uint32_t key[KT / NT];
#pragma unroll
        for (int k = 0; k < KT / NT; ++k) {
            const int q = it.tile * KT + k * NT + (int)threadIdx.x;
            key[k] = q < n ? keys[q] : 0;
        }
        // the lookups of the tile's positions are all asked for before any is used
        int j = -1;
        uint32_t kk[KT / NT];
        uint4 x[KT / NT];
        bool ok[KT / NT];
#pragma unroll
        for (int k = 0; k < KT / NT; ++k) {
            const int q = it.tile * KT + k * NT + (int)threadIdx.x;
            ok[k] = q < n;
            kk[k] = 0;
            x[k] = make_uint4(0, 0, 0, 0);
            if (ok[k]) {
                if (j < 0 || q >= s_slotpos[j + 1]) j = upper_bound_i32(s_slotpos, F + 1, q) - 1;   // the slot of this position
                kk[k] = key[k] - s_klo[j];
                // no lookup for a pack with rejected offsets, nor for a key that is none of its table (only possible then)
                ok[k] = s_pack[j] == 0 && kk[k] < s_rows[j];
                if (ok[k]) x[k] = bitmap4[(size_t)s_wb[j] / 4 + (kk[k] >> 5) / 3u];
            }
        }
#pragma unroll
        for (int k = 0; k < KT / NT; ++k) {
            const int q = it.tile * KT + k * NT + (int)threadIdx.x;
            const uint32_t tw = kk[k] >> 5;
            const int wi = (int)(tw - tw / 3u * 3u);
            const uint32_t w[3] = {x[k].x, x[k].y, x[k].z};
            int r = (int)x[k].w;                           // the rank of the 16 bytes' first key
            uint32_t cur = 0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (i < wi) r += __popc(w[i]);
                if (i == wi) cur = w[i];
            }
            r += __popc(cur & ((1u << (kk[k] & 31)) - 1u));
            if (ok[k]) inverse[q] = r;
        }
    }
}

// ---------------------------------------------------------------------------
// Partition (Sec. II-D operator list; Sec. III-B fuses it with Unique): one GPU's share of it.  With the
// rows of a packed table dealt to n workers by row mod n, the distinct keys of a pack are regrouped by
// owner -- owner 0 first, ascending inside an owner -- with the place of every key in `unique` beside it
// (what Stitch needs for the rows that come back) and the offsets of the owners' groups.  A counting
// sort in two launches: counts per chunk and owner, and the placing pass, whose blocks add up the counts of the
// chunks before their own (there are at most kPartChunks, so that is a few thousand numbers; a launch of one
// block that scanned them took 4.7 us of a pack's 16.6).  A block owns a chunk and each of its wavefronts a
// quarter, so that the order inside an owner is the key order; which lanes share an owner comes from one ballot
// per bit of the owner's number.  Bound by the launches and their chains of loads, so all the loads of a step are
// in flight at once.
// ---------------------------------------------------------------------------
constexpr int kPartStep = 4 * NT, kPartChunks = 1024;   // a chunk is a multiple of kPartStep keys
constexpr int kPartOwnersMax = 64;

// keys per chunk: kPartStep, more where that gave more than kPartChunks chunks
__device__ __forceinline__ int part_chunk(int U) { return ((U + kPartChunks - 1) / kPartChunks + kPartStep - 1) / kPartStep * kPartStep; }

// key mod n: magic = floor((2^32 - 1) / n) gives the quotient or one below it
__device__ __forceinline__ uint32_t part_owner(uint32_t key, uint32_t n, uint32_t magic)
{
    const uint32_t r = key - __umulhi(key, magic) * n;
    return r >= n ? r - n : r;
}

// the lanes (of those with `on`) that have this lane's owner
__device__ __forceinline__ uint64_t part_peers(uint32_t o, bool on, int bits)
{
    uint64_t m = __ballot(on);
    for (int b = 0; b < bits; ++b) {
        const uint64_t x = __ballot(o >> b & 1);
        m &= (o >> b & 1) ? x : ~x;
    }
    return m;
}

// four keys of a lane at i, i + 64, ...: loaded without a condition (those at or past `end` are not used)
__device__ __forceinline__ void part_load(uint32_t key[4], const uint32_t* __restrict__ uq, int i, int end)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) key[j] = uq[min(i + 64 * j, end - 1)];
}

__global__ void __launch_bounds__(NT)
pk_partition_count_kernel(const PackState* __restrict__ st, int p, const uint32_t* __restrict__ unique_all,
                          int n_owners, int bits, uint32_t magic, int32_t* __restrict__ chunk_counts)
{
    __shared__ int s_cnt[kPartOwnersMax];
    const int tid = threadIdx.x, lane = tid & 63;
    const int U = st[p].n_unique;
    const uint32_t* uq = unique_all + st[p].start;
    const int chunk = part_chunk(U), c0 = blockIdx.x * chunk, end = min(c0 + chunk, U);
    if (c0 >= end) return;
    if (tid < kPartOwnersMax) s_cnt[tid] = 0;
    __syncthreads();
    for (int i = c0 + (tid & ~63) * 4 + lane; i - lane < end; i += kPartStep) {
        uint32_t key[4];
        part_load(key, uq, i, end);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool on = i + 64 * j < end;
            const uint32_t o = part_owner(key[j], (uint32_t)n_owners, magic);
            const uint64_t m = part_peers(o, on, bits);
            if (on && (m & ((1ull << lane) - 1ull)) == 0) atomicAdd(&s_cnt[o], __popcll(m));
        }
    }
    __syncthreads();
    if (tid < n_owners) chunk_counts[(size_t)blockIdx.x * n_owners + tid] = s_cnt[tid];
}

__global__ void __launch_bounds__(NT)
pk_partition_place_kernel(const PackState* __restrict__ st, int p, const uint32_t* __restrict__ unique_all,
                          int n_owners, int bits, uint32_t magic, const int32_t* __restrict__ chunk_counts,
                          uint32_t* __restrict__ part_keys, int32_t* __restrict__ part_index, int32_t* __restrict__ offsets)
{
    constexpr int NW = NT / 64;
    __shared__ int s_all[kPartOwnersMax], s_before[kPartOwnersMax], s_cur[NW][kPartOwnersMax];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int U = st[p].n_unique;
    const uint32_t* uq = unique_all + st[p].start;
    const int chunk = part_chunk(U), n_chunks = chunk ? (U + chunk - 1) / chunk : 0;
    const int c0 = blockIdx.x * chunk, end = min(c0 + chunk, U);
    if (c0 >= end) {
        if (blockIdx.x == 0 && tid <= n_owners) offsets[tid] = 0;     // no keys
        return;
    }
    const int quarter = chunk / NW, w0 = c0 + wv * quarter, w1 = min(w0 + quarter, end);
    uint32_t key[4];
    if (w0 < w1) part_load(key, uq, w0 + lane, w1);
    if (tid < kPartOwnersMax) { s_all[tid] = 0; s_before[tid] = 0; }
    s_cur[wv][lane] = 0;
    __syncthreads();
    // every owner's keys, in all chunks and in those before this block's
    const int per = NT / n_owners;                         // threads per owner
    if (tid < per * n_owners) {
        const int o = tid % n_owners;
        int all = 0, before = 0;
        for (int c = tid / n_owners; c < n_chunks; c += 8 * per) {
            int x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = chunk_counts[(size_t)min(c + j * per, n_chunks - 1) * n_owners + o];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int y = c + j * per < n_chunks ? x[j] : 0;
                all += y;
                before += c + j * per < (int)blockIdx.x ? y : 0;
            }
        }
        if (all) { atomicAdd(&s_all[o], all); atomicAdd(&s_before[o], before); }
    }
    // the keys of every wavefront by owner (a lane's count is read by others in the next step: the compiler is kept
    // from moving LDS accesses across the steps, the hardware does a wavefront's in order)
    auto wave_order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };
    for (int i = w0 + lane; i - lane < w1; i += 256) {
        if (i - lane > w0) part_load(key, uq, i, w1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool on = i + 64 * j < w1;
            const uint32_t o = part_owner(key[j], (uint32_t)n_owners, magic);
            const uint64_t m = part_peers(o, on, bits);
            if (on && (m & ((1ull << lane) - 1ull)) == 0) s_cur[wv][o] += __popcll(m);
            wave_order();
        }
    }
    __syncthreads();
    const int mine = lane < n_owners ? s_all[lane] : 0;    // lane o: owner o
    int inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (blockIdx.x == 0 && wv == 0) {
        if (lane < n_owners) offsets[lane] = inc - mine;
        if (lane == 0) offsets[n_owners] = U;
    }
    int cur = lane < n_owners ? inc - mine + s_before[lane] : 0;
    for (int w = 0; w < wv; ++w) cur += s_cur[w][lane];
    __syncthreads();                                       // (the counts are replaced by places)
    s_cur[wv][lane] = cur;
    wave_order();
    for (int i = w0 + lane; i - lane < w1; i += 256) {
        if (quarter > 256) part_load(key, uq, i, w1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool on = i + 64 * j < w1;
            const uint32_t o = part_owner(key[j], (uint32_t)n_owners, magic);
            const uint64_t m = part_peers(o, on, bits), below = m & ((1ull << lane) - 1ull);
            const int at = s_cur[wv][o] + __popcll(below); // lanes are in key order
            wave_order();
            if (on) {
                part_keys[at] = key[j];
                part_index[at] = i + 64 * j;
                if (below == 0) s_cur[wv][o] += __popcll(m);
            }
            wave_order();
        }
    }
}
