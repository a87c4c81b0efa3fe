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
//                   kernel reads its records (one launch for all slices); the inverse index is then looked up per occurrence
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
        constexpr int UK = 8;                              // IDs per thread in flight
        static_assert(UK * NT <= kRoundMax, "positions are counted in 32 bits");
        for (int base = q_lo; base < q_hi; base += UK * NT) {      // the same trips for every lane: lanes combine their counts
            const int64_t* id_at = ids + base;
            uint32_t* key_at = keys + (base + dl);
            const int left = q_hi - base;
            int64_t idv[UK];
#pragma unroll
            for (int j = 0; j < UK; ++j) idv[j] = id_at[min(tid + j * NT, left - 1)];      // (no condition: nothing is waited for in between)
#pragma unroll
            for (int j = 0; j < UK; ++j) {
                const int i = tid + j * NT;
                const bool on = i < left;
                const uint32_t kk = fold_id(idv[j], m.rows, m.magic);
                if (on) key_at[i] = m.base_row + kk;
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

// Large batches: the slices' totals become places.  A block takes 1024 slices; what lies before them
// it adds up itself (there are some thousand slices: a block reads a few values per thread).  Every slice
// gets its table, its index in the table, the place of its first record and the number of records; the
// cursors of the scatter kernel start at those places.
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads)
pk_slice_scan_kernel(const TableCut* __restrict__ cut, int T,
                     const int32_t* __restrict__ slice_total, int32_t* __restrict__ slice_cursor,
                     SliceInfo* __restrict__ slice_info, int n_slices, int32_t* __restrict__ long_list, int n_long_max)
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
        // Slices of many records are listed, and the slice kernel's first blocks take them: each is one block's work, so
        // the launch ends with the one that started last, and by their place in the pack they could all fall to one XCD
        // (every table's first slice, where low IDs are the frequent ones: the dedup of 200 fields of 21 M IDs 860 us,
        // 540 with the list; of 26 one-hot fields of 65536 248 and 154).
        if (c >= kLongSlice) {
            const int at = atomicAdd(long_list, 1);
            if (at < n_long_max) {
                long_list[1 + at] = s;
                si.table |= kListedFlag;
            }
        }
        slice_info[s] = si;
        slice_cursor[s] = carry + ex;
    }
}

// Large batches: one record per occurrence, (key inside its slice, place of its bag's gradient chunk), written to
// the slice's place.  A tile counts its occurrences per slice in LDS, reserves room in every
// touched slice with one global add, and then places its records from block-local cursors: one LDS word per slice
// of the tile's table, first its count, then its cursor (a table has up to kTableSlicesMax).  Bound by the latency of
// the keys and by its 8-byte stores, so a wavefront's keys are asked for eight at a time without a condition: under
// one, each was waited for before the next (averages beside the pooling: 200 fields 269 -> 149 us, bf16 sequences 118 ->
// 64; 26 one-hot fields of 65536 23 -> 17; touching the tile's keys ahead then gives nothing more).
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
        if (!tile_hist)                                    // (the keys kernel's counts of this tile were not kept)
        for (int base = q_lo; base < q_hi; base += 4 * NT) {      // four loads in flight
            uint32_t kv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) kv[u] = keys[min(base + tid + u * NT, q_hi - 1) + dl];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t s = base + tid + u * NT < q_hi ? (kv[u] - m.base_row) >> g.log_keys : 0xFFFFFFFFu;
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
        const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int per_wave = ((q_hi - q_lo + NT - 1) / NT) * 64;
        const int w_lo = q_lo + wv * per_wave, w_hi = min(w_lo + per_wave, q_hi);
        const bool stepped = (int64_t)tl.nb * 64 <= (int64_t)6 * (q_hi - q_lo);     // (short bags: a search per position is shorter)
        int t = stepped && w_lo + lane < w_hi ? upper_bound_i32(s_po, tl.nb + 1, w_lo + lane) - 1 : 0;
        constexpr int UP = 8;                              // key loads in flight (they come from memory: nothing has read them since they were written)
        static_assert(4 * NT <= kRoundMax && UP * NT <= kRoundMax, "positions are counted in 32 bits");
        for (int base = w_lo; base < w_hi; base += UP * 64) {
            const uint32_t* key_at = keys + (base + dl);
            const int left = w_hi - base;
            uint32_t kv[UP];
#pragma unroll
            for (int u = 0; u < UP; ++u) kv[u] = key_at[min(u * 64 + lane, left - 1)];     // (no condition, and no arithmetic before the last is asked for)
            uint32_t sl[UP];
            int at[UP];
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                kv[u] -= m.base_row;
                sl[u] = u * 64 + lane < left ? kv[u] >> g.log_keys : 0xFFFFFFFFu;
                at[u] = 0;
                if (g.n <= kFewCounters) at[u] = lds_inc_few<true>(s_hist, sl[u], sl[u] < (uint32_t)g.n, g.n);   // (all lanes of the wavefront are here)
                else if (sl[u] < (uint32_t)g.n) at[u] = atomicAdd(&s_hist[sl[u]], 1);
            }
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                const int i = base + u * 64 + lane;
                const bool valid = sl[u] < (uint32_t)g.n;
                if (i < w_hi) {
                    if (stepped) { while (t + 1 < tl.nb && s_po[t + 1] <= i) ++t; }
                    else if (valid) t = upper_bound_i32(s_po, tl.nb + 1, i) - 1;
                }
                if (!valid) continue;
                // the record: key inside the slice, the gradient's scale (bag length for mean pooling, 1 for sum;
                // 0 = too long for its bits, to be looked up) above it, and the place of the bag's gradient chunk
                uint32_t len = 1u;
                if (m.pool == PK_MEAN) {
                    const uint32_t L = (uint32_t)max(s_po[t + 1] - s_po[t], 1);
                    len = (L >> (32 - log_max)) ? 0u : L;
                }
                if ((uint64_t)(int64_t)at[u] < (uint64_t)nnz)
                    rec[at[u]] = make_uint2((kv[u] - (sl[u] << g.log_keys)) | (len << log_max),
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
    int F, B; int64_t nnz; int log_max;
    int patience;                                               // small batches: looks at what other blocks publish (beside what is read first)
    const int64_t* ids; const int32_t* offsets; const SmallSlice* small_slices; const int2* slot_info;   // small batches: the block finds its occurrences itself
    const SliceInfo* slice_info; uint2* rec;                    // large batches: the slice's records
    const TableCut* cut;                                        // ... and the tables' cuts for this batch
    const FieldMeta* fmeta;
    int32_t* packed_offsets;
    uint32_t* keys; int32_t* inverse;                           // written here for small batches only
    uint32_t* bitmap;                                           // large batches only: bitmaps with rank samples
    const int32_t* long_list; int n_long_max;                   // ... slices of many records: how many, which
    uint32_t* slice_nu; uint64_t* nu_group; int n_groups, sum_stride, waits;   // ... distinct keys per slice, and their sums (SliceSums)
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

// The kernel's arguments, and what the host or an earlier launch has written, through pointers that the compiler loses
// track of between the phases of a block: held from the start, all that a slice block needs is forty scalar registers
// more than there are.
typedef const __attribute__((address_space(4))) SliceArgs* SliceArgsPtr;
template <bool LEAN, typename P>
__device__ __forceinline__ P forget(P p)
{
    if (LEAN) asm volatile("" : "+s"(p));
    return p;
}
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* as_constant(const T* p) { return (const __attribute__((address_space(4))) T*)p; }

// ---------------------------------------------------------------------------
// Large batches, one launch for all slices: a block owns a slice.  It reads the slice's records once, keeps them in
// registers (kSliceKeep per thread), and
//   marks the bitmap -> popcount prefix of its words, number of distinct keys, which is published;
//   counts the occurrences per key (a record's rank and place go into a register) -> the keys' first places;
//   places every record's entry: that needs the records before the slice only, and their number is known;
//   adds up the distinct keys of the pack's slices before its own (SliceSums), published long ago by then;
//   writes what needs that sum: distinct keys, segment offsets, marks, the bitmap with its rank samples.
// A slice of more records reads them again for each of these passes, the next ones on their way while some are worked on,
// and counts up to RANKS keys a round, after which the records of later rounds' keys alone are left.  (All records read
// in every round, none ahead, and such slices not listed first: 26 one-hot fields of 65536, low IDs frequent, dedup 357 us,
// 154 now; 200 fields of 21 M IDs 1068 and 540; 2 M IDs of tables of ten rows 1298 and 943.)
// What bounds it is the chain of these steps, 13 us a block, so four blocks of 512 threads share a CU.  (Five launches,
// mark, scan, place, and mark and place for the slices with many records in blocks of four times the threads, wrote the
// bitmaps, read them back and read the records three times.  Launches of the step's dedup together, us, before and
// after: 200 fields of 21 M IDs 290 -> 185 without pooling beside; 26 one-hot fields of 65536 65 -> 29; 1 M IDs of
// unequal tables 71 -> 37.)  256 threads: 20 % slower, more for slices of frequent keys; 1024: the same alone, but they
// find no room beside the pooling (200 fields, forward alone 235 -> 265).
// ---------------------------------------------------------------------------
constexpr int kSliceTfWords = 5;           // dynamic LDS words per field of a table
constexpr int kFineThreads = 512, kFineRanks = 4096;
constexpr int kSliceThreads = 1024, kSliceRanks = 8192;
constexpr int kSliceKeep = 8;              // records per thread kept in registers

// LDS words of a slice block: bitmap words with their popcount prefix | counters of a round of distinct keys
constexpr int slice_lds_words(int log_max, int ranks) { return 2 * (1 << (log_max - 5)) + ranks; }

// one occurrence of a slice: key minus the slice's first key, the place of its gradient chunk, the chunk's scale
struct SliceRec { uint32_t kl, ref, L; };

// Distinct keys before a slice.  Every slice publishes its number and adds it to its group of kSumFan slices; the first
// slice of a group adds up the groups before and publishes that; the others take what was published for the group
// before theirs (long there, usually), that group, and the slices of their own before them.  (Every block looking at all
// groups itself: a thousand blocks then poll the same few lines, and a round trip takes 20 us instead of 3.)  Groups are
// counted from the pack's first slice, so a pack's sums never mix with another's.  The words carry their own validity (a
// flag, or how many have been added): relaxed accesses do, and nothing is returned to the publishing block.
// A block that has waited for long while no slice of the launch published counts what it lacks itself (count_before in
// slice_body), so it waits for no block that may not have started.
// (a loop: unrolled, the six shuffles' addresses are kept from one use to the next, in registers that there are not)
__device__ __forceinline__ int wave_sum(int v)
{
#pragma nounroll
    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}
static_assert(kSumFan == 64, "a wavefront's lanes look at the slices of a group, the last two at the groups");
constexpr int kLooks = 64, kPatience = 16;               // 16 times 64 looks of about 3 us
constexpr int kNotSeen = -2;
constexpr uint32_t kNuReady = 0x80000000u, kNuBegun = 0x40000000u;     // begun: a slice of more records than are kept, by its block
constexpr uint32_t kNuMask = kNuBegun - 1u;
enum { kWaitNever = 1, kWaitGivesUp = 2 };               // SliceArgs::waits, for tests
struct SliceSums {
    uint32_t* nu; uint64_t* group; uint64_t* prefix;     // per slice; per group: count << 32 | sum; kSumFan << 32 | sum before it
    const int32_t* error;                                // the pack's error word
    int i, stride;                                       // the slice, counted from the pack's first; words between groups
    __device__ __forceinline__ SliceSums(SliceArgsPtr a, int slice, int pack_first, int p)
    {
        i = slice - pack_first;
        nu = as_global(a->slice_nu) + pack_first;
        stride = a->sum_stride;
        group = as_global(a->nu_group) + (size_t)(pack_first / kSumFan + p) * stride;
        prefix = group + (size_t)a->n_groups * stride;
        error = &as_global(a->st)[p].error;
    }
    __device__ __forceinline__ void begin() const                              // one thread, the one that publishes
    {
        __hip_atomic_store(nu + i, kNuBegun, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void publish(int n_u) const                     // one thread
    {
        __hip_atomic_store(nu + i, kNuReady | (uint32_t)n_u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        (void)__hip_atomic_fetch_add(group + i / kSumFan * stride, (uint64_t)1 << 32 | (uint32_t)n_u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void publish_before(int sum) const              // one thread, a group's first slice
    {
        __hip_atomic_store(prefix + i / kSumFan * stride, (uint64_t)kSumFan << 32 | (uint32_t)sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t word(int j) const { return __hip_atomic_load(nu + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    // a slice of the pack gave up, or found sums that cannot be: its number may never come
    __device__ __forceinline__ bool given_up() const { return __hip_atomic_load(error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0; }
    // One wavefront, all lanes.  `ask` sends the loads out, `before` waits for them, and for the numbers themselves: the
    // distinct keys of the pack's slices before this one; kNotSeen where they have not come, -1 where they will not.
    struct Seen { uint32_t n; uint64_t g; };
    __device__ __forceinline__ Seen ask() const
    {
        // lanes 0 .. : the slices of the group before this one; the last two: the group before, and what is before that
        const int lane = threadIdx.x & 63, g = i / kSumFan, in = i % kSumFan;
        Seen s{kNuReady, (uint64_t)kSumFan << 32};
        if (lane < in) s.n = word((i - in) + lane);
        if (in != 0 && lane >= kSumFan - 2 && g > kSumFan - 1 - lane)
            s.g = __hip_atomic_load((lane == kSumFan - 2 ? prefix : group) + (g - 1) * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return s;
    }
    __device__ __forceinline__ int before(Seen s, SliceArgsPtr a) const
    {
        const int lane = threadIdx.x & 63, g = i / kSumFan;
        if (a->waits && i) {
            if (a->waits & kWaitNever) return kNotSeen;
            if (i % kSumFan == 0) return -1;
        }
        uint32_t seen = 0;
        int quiet = 0;
        for (int spin = 0; spin < kSpinLimit; ++spin) {
            bool ok = (s.n & kNuReady) && (s.g >> 32) == kSumFan;
            int sum = (int)((s.n & kNuMask) + (uint32_t)s.g);
            if (i % kSumFan == 0)
                for (int k = lane; k < g; k += 64) {
                    const uint64_t z = __hip_atomic_load(group + k * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = ok && (z >> 32) == kSumFan;
                    sum += (int)(uint32_t)z;
                }
            if (__all(ok)) {
                sum = wave_sum(sum);
                if (i % kSumFan == 0 && lane == 0) publish_before(sum);
                return sum;
            }
            if (spin % kLooks == kLooks - 1) {             // has any slice of the launch published since?
                if (__any(given_up())) return -1;
                uint32_t n = 0;
                for (int k = lane; k < a->n_groups; k += 64)
                    n += (uint32_t)(__hip_atomic_load(as_global(a->nu_group) + (size_t)k * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32);
                n = (uint32_t)wave_sum((int)n);
                quiet = n == seen ? quiet + 1 : 0;
                seen = n;
                if (quiet == kPatience) return kNotSeen;
            }
            __builtin_amdgcn_s_sleep(8);
            s = ask();
        }
        return kNotSeen;
    }
    // One thread: the number of a slice whose block has begun, which publishes before it waits for anything.
    __device__ __forceinline__ uint32_t published(int j) const
    {
        for (int spin = 0; spin < kSpinLimit; ++spin) {
            const uint32_t w = word(j);
            if (w & kNuReady) return w & kNuMask;
            if (given_up()) break;
            __builtin_amdgcn_s_sleep(8);
        }
        return ~0u;
    }
};

template <int N> struct InFlight { static constexpr int value = N; };

// KEPT: the slice's records fit the threads' registers
template <int NTH, int LOGMAX, int RANKS, bool KEPT>
__device__ __forceinline__ void slice_body(SliceArgsPtr a, int slice, int32_t* s_main, int32_t* s_tf, int32_t* s_base)      // s_base: four words
{
    constexpr int WMAX = 1 << (LOGMAX - 5), WPT = WMAX / NTH;       // bitmap words, of them per thread
    constexpr int KEEP = kSliceKeep;
    static_assert(WPT == 4 && KEEP * NTH <= 0xFFFF && KEEP * NTH <= RANKS, "a thread's words are two 16-byte reads; ranks and places of kept records fit 16 bits");
    static_assert(WMAX <= RANKS, "the counters' room holds another slice's bitmap");
    const int tid = threadIdx.x;
    uint2* s_bp = reinterpret_cast<uint2*>(s_main);        // a word of the bitmap, set bits before it
    int32_t* s_cnt = s_main + 2 * WMAX;

    // ---- which slice, of which table; its records ----
    const auto* si = as_constant(a->slice_info) + slice;
    const int t = si->table & ~kListedFlag, rec_start = si->start, n_rec = si->count;
    uint2* rec = as_global(a->rec) + rec_start;
    // (loads without a condition: under one, the compiler waits for each before the next; places without a record ask
    // for the last one again)
    auto load_record = [&](int base, int left, int i) {    // record base + i of `left` from base on, the same for the block: a 32-bit offset from a scalar address
        const char* at = reinterpret_cast<const char*>(rec + base);
        return *reinterpret_cast<const uint2*>(at + (uint32_t)min(i, max(left - 1, 0)) * (uint32_t)sizeof(uint2));
    };
    uint2 kept[KEEP];
#pragma unroll
    for (int u = 0; u < KEEP; ++u) kept[u] = KEPT ? load_record(0, n_rec, tid + u * NTH) : make_uint2(0, 0);
    const auto* tm = as_constant(a->tmeta) + t;
    const int p = tm->pack;
    const PackState* st = as_global(a->st) + p;
    const int pstart = st->start, nnz_p = st->nnz;
    if (st->error) return;                                 // offsets of this pack were rejected (so all its slices return here), or one gave up
    if (!KEPT && tid == 0) SliceSums(a, slice, st->first_slice, p).begin();
    const int lg = as_constant(a->cut)[t].log_keys;
    const bool wide = as_constant(a->pm)[p].has_mean != 0; // the pack's entries carry the bag length
    const int nf = tm->field_end - tm->field_begin;
    if (wide)
        for (int j = tid; j < nf; j += NTH) {
            const TableField tf = as_global(a->tfields)[tm->field_begin + j];
            s_tf[kSliceTfWords * j] = tf.slot;
            s_tf[kSliceTfWords * j + 3] = tf.col;
        }
    const uint32_t nkeys = min((uint32_t)1 << lg, tm->rows - ((uint32_t)si->idx << lg));
    const int words = 1 << (lg - 5);
    const bool mine = tid * WPT < words;                   // thread i owns words [i * WPT, (i + 1) * WPT)
    if (mine) {
#pragma unroll
        for (int j = 0; j < WPT; ++j) s_bp[tid * WPT + j] = make_uint2(0, 0);
    }
    for (int i = tid; i < min(RANKS, n_rec); i += NTH) s_cnt[i] = 0;
    __syncthreads();

    auto unpack = [&](uint2 r, bool valid, bool* on) {
        const uint32_t kl = r.x & ((1u << LOGMAX) - 1u);
        *on = valid && kl < nkeys;
        return SliceRec{*on ? kl : 0u, r.y, r.x >> LOGMAX};
    };
    // Records where they are not kept, UN per lane in flight: a wavefront takes a contiguous share of the slice's, of which
    // the first `n` are gone through, and every lane makes the same trips, so that fn(records, number left from the
    // lane's first on) may combine lanes.
    const int lane = tid & 63;
    const int share = (n_rec + NTH - 1) / NTH * 64, share_lo = min(__builtin_amdgcn_readfirstlane(tid >> 6) * share, n_rec);
    const int n_share = min(share, n_rec - share_lo);
    auto for_records = [&](auto in_flight, int n, auto&& fn) {
        constexpr int UN = decltype(in_flight)::value;
        int first = lane;                                  // (what follows from it is not kept over the rounds of keys)
        asm volatile("" : "+v"(first));
        uint2 r[UN], next[UN];
        if (n > 0) {
#pragma unroll
            for (int u = 0; u < UN; ++u) next[u] = load_record(share_lo, n, first + u * 64);
        }
#pragma nounroll
        for (Rounds<UN * 64> at(n); at.any(); at.next()) {
            const bool last = at.left <= UN * 64;
#pragma unroll
            for (int u = 0; u < UN; ++u) r[u] = next[u];
#pragma unroll
            for (int u = 0; u < UN; ++u)                   // (on their way while these are worked on; after the last, the last again)
                next[u] = load_record(share_lo + at.base + (last ? 0 : UN * 64), last ? at.left : at.left - UN * 64, first + u * 64);
            fn(r, at.left - first);
        }
    };

    // ---- which keys occur ----
    auto mark = [&](uint32_t kl, uint32_t seen, bool on) {
        const uint32_t bit = 1u << (kl & 31);
        if (on && !(seen & bit)) atomicOr(&s_bp[kl >> 5].x, bit);
    };
    if constexpr (KEPT) {
#pragma unroll
        for (int u = 0; u < KEEP; ++u) {
            if (u * NTH >= n_rec) break;
            bool on;
            const SliceRec x = unpack(kept[u], tid + u * NTH < n_rec, &on);
            mark(x.kl, on ? s_bp[x.kl >> 5].x : 0u, on);
        }
    } else {
        for_records(InFlight<8>{}, n_share, [&](const uint2 (&r)[8], int left) {
            uint32_t seen[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) seen[u] = s_bp[(r[u].x & ((1u << LOGMAX) - 1u)) >> 5].x;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                bool on;
                const SliceRec x = unpack(r[u], u * 64 < left, &on);
                mark(x.kl, seen[u], on);
            }
        });
    }
    __syncthreads();
    // popcount prefix of the words, number of distinct keys
    int n_u;
    {
        uint32_t x[WPT];
        int c = 0;
#pragma unroll
        for (int j = 0; j < WPT; ++j) {
            x[j] = mine ? s_bp[tid * WPT + j].x : 0u;
            c += __popc(x[j]);
        }
        int run = block_excl_scan<NTH>(c, &n_u);
        if (tid == 0) SliceSums(a, slice, st->first_slice, p).publish(n_u);
        if (mine) {
#pragma unroll
            for (int j = 0; j < WPT; ++j) {
                s_bp[tid * WPT + j].y = (uint32_t)run;
                run += __popc(x[j]);
            }
        }
    }
    __syncthreads();

    // ---- occurrences per distinct key, and every occurrence's gradient place at its key's next free position ----
    const int rec_before = rec_start - pstart;
    a = forget<true>(a);
    uint32_t* __restrict__ ent = as_global(a->ent_all) + (size_t)pstart * a->ent_mult;
    auto rank_of = [&](uint32_t kl) {
        const uint2 w = s_bp[kl >> 5];
        return (int)(w.y + __popc(w.x & ((1u << (kl & 31)) - 1u)));
    };
    auto put = [&](const SliceRec& r, int pos) {
        if ((unsigned)pos >= (unsigned)nnz_p) return;
        if (!wide) { ent[pos] = r.ref; return; }
        uint32_t len = r.L;
        if (len == 0) {                                    // a bag too long for the record's bits: its length from the bag
            const uint32_t out_dim = (uint32_t)a->out_dim;
            const uint32_t b = r.ref / out_dim, col = r.ref - b * out_dim;
            int j = 0;
            while (j + 1 < nf && (uint32_t)s_tf[kSliceTfWords * j + 3] != col) ++j;
            const uint32_t g = (uint32_t)s_tf[kSliceTfWords * j] * (uint32_t)a->B + b;
            const int32_t* po = as_global(a->packed_offsets) + (int64_t)as_constant(a->pm)[p].first_slot * a->B + p;
            len = (uint32_t)max(po[g + 1] - po[g], 1);
        }
        reinterpret_cast<uint2*>(ent)[pos] = make_uint2(r.ref, len);
    };
    // the counters of `width` keys become the keys' first places, after `placed` occurrences of the slice
    auto starts = [&](int width, int placed) {
        const int per = (width + NTH - 1) / NTH;           // consecutive counters per thread
        int sum = 0;
        for (int j = 0; j < per; ++j) {
            const int i = tid * per + j;
            sum += i < width ? s_cnt[i] : 0;
        }
        int tot;
        int s0 = block_excl_scan<NTH, !KEPT>(sum, &tot) + rec_before + placed;
        for (int j = 0; j < per; ++j) {
            const int i = tid * per + j;
            if (i < width) {
                const int len = s_cnt[i];
                s_cnt[i] = s0;
                s0 += len;
            }
        }
        __syncthreads();
        return tot;
    };
    // what the backward pass needs of key u with the places [s0, s1): its segment, the marks by which a long one is
    // found, and, where it is reduced in pieces, partial sums that start at zero.  From the keys' first places, or, where
    // the placing pass has moved them on, from where they end.
    auto segments = [&](int first, int width, int begin, int end) {
        a = forget<true>(a);
        int32_t* __restrict__ seg = as_global(a->seg_all) + pstart + p;
        int32_t* __restrict__ marks = as_global(a->marks) + (pstart / kMarkStep + p);
        for (int i = tid; i < width; i += NTH) {
            const int u = first + i;
            const int s0 = KEPT ? s_cnt[i] : i ? s_cnt[i - 1] : begin, s1 = !KEPT ? s_cnt[i] : i + 1 < width ? s_cnt[i + 1] : end;
            seg[u] = s0;
            for (int m = (s0 + kMarkStep - 1) / kMarkStep; (int64_t)m * kMarkStep < (int64_t)s1; ++m) marks[m] = u;
            if (s1 - s0 >= 2 * kPiece) {
                const size_t slot = (size_t)(pstart / kPiece + p) + (size_t)(s0 / kPiece);    // (no two such keys share one)
                double* gh = as_global(a->ghot) + slot * a->dmax;
                const int dim = as_constant(a->pm)[p].dim;
                for (int d = 0; d < dim; ++d) gh[d] = 0.0;
                as_global(a->ticket)[slot] = 0;
            }
        }
    };
    // the sum before this slice; false (for the whole block) where it cannot be had, or where what it and the records'
    // place say would leave the pack's arrays
    auto ask = [&]() { return tid < 64 ? SliceSums(a, slice, st->first_slice, p).ask() : SliceSums::Seen{0, 0}; };
    // Distinct keys of the pack's slices before this one where they have not come: a block before this one may not have
    // started, and may not be able to while this one holds its place.  (Blocks start in index order on each XCD, but
    // the XCDs take their shares of a launch at their own pace, and another launch's blocks may be waiting beside.)  So
    // what is published is taken, what a running block will publish is waited for, and the keys of a slice whose block has not
    // begun are counted here, from its records, in the bitmap's size of counters.  Only blocks of more records than they keep say
    // that they have begun: the others' records are few and nobody changes them, so those are counted whether begun or not.
    auto count_before = [&]() -> int {
        __syncthreads();                                   // (*s_base has been read)
        const SliceSums sums(a, slice, st->first_slice, p);
        uint32_t* s_map = reinterpret_cast<uint32_t*>(s_cnt);
        int sum = 0;
        for (int j0 = 0; j0 < sums.i; j0 += 64) {
            if (tid < 64) {
                uint32_t w = j0 + lane < sums.i ? sums.word(j0 + lane) : kNuReady;
                if (j0 + lane < sums.i && (a->waits & kWaitNever)) w = 0;
                const uint64_t m = __ballot(!(w & kNuReady));
                const int n = wave_sum(w & kNuReady ? (int)(w & kNuMask) : 0);
                if (tid == 0) { s_base[0] = n; s_base[1] = (int)(uint32_t)m; s_base[2] = (int)(uint32_t)(m >> 32); }
            }
            __syncthreads();
            sum += s_base[0];
            uint64_t todo = (uint64_t)(uint32_t)s_base[1] | (uint64_t)(uint32_t)s_base[2] << 32;
            __syncthreads();
            while (todo) {
                const int j = j0 + __ffsll((unsigned long long)todo) - 1;
                todo &= todo - 1;
                const auto* sj = as_constant(a->slice_info) + (slice - sums.i + j);
                const int n_j = sj->count, t_j = sj->table & ~kListedFlag;
                const uint2* __restrict__ rec_j = as_global(a->rec) + sj->start;
                const bool few = n_j <= KEEP * NTH;
                // number of the slice: ~0u = it will not come; its block has not begun: kNuBegun
                auto look = [&]() {
                    if (tid == 0) {
                        const uint32_t w = few ? 0u : sums.word(j);
                        s_base[3] = (int)(w == 0 ? kNuBegun : sums.published(j));
                    }
                    __syncthreads();
                    const uint32_t w = (uint32_t)s_base[3];
                    __syncthreads();
                    return w;
                };
                uint32_t n = look();
                if (n == kNuBegun) {
                    const int lg_j = as_constant(a->cut)[t_j].log_keys;
                    const uint32_t nkeys_j = min((uint32_t)1 << lg_j, as_constant(a->tmeta)[t_j].rows - ((uint32_t)sj->idx << lg_j));
                    for (int w = tid; w < WMAX; w += NTH) s_map[w] = 0;
                    __syncthreads();
                    for (Rounds<4 * NTH> at(n_j); at.any(); at.next()) {
                        uint32_t x[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) x[u] = rec_j[at.base + min(tid + u * NTH, at.left - 1)].x & ((1u << LOGMAX) - 1u);
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (x[u] < nkeys_j) atomicOr(&s_map[x[u] >> 5], 1u << (x[u] & 31));
                    }
                    __syncthreads();
                    int c = 0;
                    for (int w = tid; w < WMAX; w += NTH) c += __popc(s_map[w]);
                    c = wave_sum(c);
                    if (tid == 0) s_base[3] = 0;
                    __syncthreads();
                    if (lane == 0) atomicAdd(&s_base[3], c);
                    __syncthreads();
                    n = (uint32_t)s_base[3];
                    __syncthreads();
                    if (!few) {                            // its block may have begun meanwhile: what was read may have been changed
                        const uint32_t again = look();
                        if (again != kNuBegun) n = again;
                    }
                }
                if (n == ~0u) return -1;
                sum += (int)n;
            }
        }
        if (tid == 0 && sums.i % kSumFan == 0) sums.publish_before(sum);
        return sum;
    };
    auto get_base = [&](SliceSums::Seen seen) -> bool {
        if (tid < 64) {
            const int b = SliceSums(a, slice, st->first_slice, p).before(seen, a);
            if (tid == 0) *s_base = b;
        }
        __syncthreads();
        int base = *s_base;
        bool ok = rec_before >= 0 && (int64_t)rec_before + n_rec <= (int64_t)nnz_p;
        if (ok && base == kNotSeen) {
            // (the counters meanwhile in the slice's share of the inverse index, which is written after this launch)
            int32_t* save = as_global(a->inverse) + rec_start;
            const int n = min(min(RANKS, n_u), n_rec);
            for (int i = tid; i < n; i += NTH) save[i] = s_cnt[i];
            base = count_before();
            __syncthreads();
            for (int i = tid; i < n; i += NTH) s_cnt[i] = save[i];
            if (tid == 0) *s_base = base;
            __syncthreads();
        }
        ok = ok && base >= 0 && (int64_t)base + n_u <= (int64_t)nnz_p;
        if (!ok && tid == 0) atomicOr(&as_global(a->st)[p].error, 2);
        return ok;
    };
    if constexpr (KEPT) {
        // The counting pass gives every record its key's rank and its place among the key's occurrences: both fit a
        // register, and the placing pass needs no counter.
        uint32_t rp[KEEP];
#pragma unroll
        for (int u = 0; u < KEEP; ++u) {
            if (u * NTH >= n_rec) break;
            bool on;
            const SliceRec r = unpack(kept[u], tid + u * NTH < n_rec, &on);
            const uint32_t rk = (uint32_t)rank_of(r.kl);
            rp[u] = on ? rk | ((uint32_t)atomicAdd(&s_cnt[rk], 1) << 16) : 0xFFFFFFFFu;
        }
        __syncthreads();
        const int tot = starts(n_u, 0);
        const SliceSums::Seen seen = ask();                // (on its way while the records are placed)
#pragma unroll
        for (int u = 0; u < KEEP; ++u) {
            if (u * NTH >= n_rec) break;
            bool on;
            const SliceRec r = unpack(kept[u], tid + u * NTH < n_rec, &on);
            if (on) put(r, s_cnt[rp[u] & 0xFFFFu] + (int)(rp[u] >> 16));
        }
        if (!get_base(seen)) return;
        segments(*s_base, n_u, 0, rec_before + tot);
    } else {
        // Where IDs are scattered over the rows, most of a slice with many records is one frequent key's: the one that most
        // of the first 64 records have is counted and placed by ballots, a whole wavefront's at once; the others have one LDS
        // atomic each.  (Lanes that share a key combined for any key, 64 records are a chain of 1100 cycles: 52 K records 100 us.)
        if (tid < 64) {
            const uint32_t kl = min(load_record(0, n_rec, tid).x & ((1u << LOGMAX) - 1u), nkeys - 1u);
            int best = 0;
            uint32_t hot = 0;
            for (int l = 0; l < 64; l += 8) {
                const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)kl, l);
                const int n = __popcll(__ballot(kl == v));
                if (n > best) { best = n; hot = v; }
            }
            if (tid == 0) *s_base = (int)hot;
        }
        __syncthreads();
        const uint32_t hot = (uint32_t)*s_base;
        const int hot_rank = rank_of(hot);
        __syncthreads();
        auto below = [](uint64_t m) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); };
        int placed = 0;                                    // occurrences of the keys of earlier rounds
        int n_mine = n_share;                              // records of the wavefront that are still to be placed
        for (int r0 = 0; r0 < n_u; r0 += RANKS) {          // a round handles RANKS keys
            const int width = min(RANKS, n_u - r0);
            const bool hot_now = (unsigned)(hot_rank - r0) < (unsigned)width;
            const uint32_t hot_at = hot_now ? (uint32_t)(hot_rank - r0) : 0x80000000u;
            if (r0) {
                __syncthreads();
                for (int i = tid; i < width; i += NTH) s_cnt[i] = 0;
                __syncthreads();
            }
            // ranks in the round (above it: a later round's, or no record's), all asked for before any is used
            auto ranks = [&](auto& rr, const auto& r, int left) {
#pragma unroll
                for (int u = 0; u < (int)(sizeof(r) / sizeof(uint2)); ++u) {
                    bool on;
                    const SliceRec x = unpack(r[u], u * 64 < left, &on);
                    const uint32_t k = (uint32_t)(rank_of(x.kl) - r0);
                    rr[u] = on ? k : ~0u;
                }
            };
            int n_hot = 0;
            for_records(InFlight<8>{}, n_mine, [&](const uint2 (&r)[8], int left) {
                uint32_t rr[8];
                ranks(rr, r, left);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    n_hot += __popcll(__ballot(rr[u] == hot_at));
                    if (rr[u] != hot_at && rr[u] < (uint32_t)width) atomicAdd(&s_cnt[rr[u]], 1);
                }
            });
            if (lane == 0 && n_hot) atomicAdd(&s_cnt[hot_at], n_hot);
            __syncthreads();
            const int tot = starts(width, placed);
            // every wavefront takes room for all its records of the frequent key at once
            int at_hot = 0;
            if (lane == 0 && n_hot) at_hot = atomicAdd(&s_cnt[hot_at], n_hot);
            at_hot = __builtin_amdgcn_readfirstlane(at_hot);
            const bool more = r0 + width < n_u;
            int n_later = 0;                               // ... and moves those of later rounds' keys to the front of its share
            for_records(InFlight<4>{}, n_mine, [&](const uint2 (&r)[4], int left) {
                uint32_t rr[4];
                int at[4];
                ranks(rr, r, left);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint64_t m = __ballot(rr[u] == hot_at);
                    at[u] = at_hot + below(m);
                    at_hot += __popcll(m);
                    if (rr[u] != hot_at && rr[u] < (uint32_t)width) at[u] = atomicAdd(&s_cnt[rr[u]], 1);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (rr[u] < (uint32_t)width) put(SliceRec{0u, r[u].y, r[u].x >> LOGMAX}, at[u]);
                }
                if (more) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool later = rr[u] >= (uint32_t)width && rr[u] != ~0u;
                        const uint64_t m = __ballot(later);
                        if (later) rec[share_lo + n_later + below(m)] = r[u];
                        n_later += __popcll(m);
                    }
                }
            });
            n_mine = n_later;
            __syncthreads();                               // (the places have been moved on)
            if (r0 == 0 && !get_base(ask())) return;
            segments(*s_base + r0, width, rec_before + placed, 0);
            placed += tot;
        }
    }

    // ---- the slice's distinct keys (ascending) ----
    a = forget<true>(a);
    si = as_constant(a->slice_info) + slice;
    tm = as_constant(a->tmeta) + t;
    const int base_u = *s_base, idx = si->idx;
    uint32_t* __restrict__ uq = as_global(a->unique) + pstart + base_u;
    if (mine) {
        const uint32_t key0 = tm->key_lo + ((uint32_t)idx << lg) + (uint32_t)(tid * WPT) * 32u;
#pragma nounroll
        for (int j = 0; j < WPT; ++j) {
            const uint2 w = s_bp[tid * WPT + j];
            uint32_t y = w.x;
            int run = (int)w.y;
            while (y) {
                const int bit = __ffs(y) - 1;
                y &= y - 1;
                uq[run++] = key0 + 32u * (uint32_t)j + bit;
            }
        }
    }
    if (tid == 0) {
        const auto* k = as_constant(a->pm) + p;
        if (t == k->first_stable + k->n_stables - 1 && idx + 1 == as_constant(a->cut)[t].n) {     // last slice of the pack's last table
            as_global(a->st)[p].n_unique = base_u + n_u;
            as_global(a->seg_all)[pstart + p + base_u + n_u] = nnz_p;
        }
    }
    // ---- the bitmap for the inverse kernel: every 16 bytes hold three words and the rank of their first key.  Sixteen
    //      bytes without a key are not asked for, unless the slice shares them with a neighbour ----
    uint32_t* bmw = as_global(a->bitmap) + tm->word_base;
    const uint32_t tw0 = (uint32_t)idx * (uint32_t)words, tw1 = tw0 + (uint32_t)words;
    const uint32_t q0 = (tw0 + 2u) / 3u, q1 = tw1 / 3u;    // the 16 bytes that are the slice's alone
    for (uint32_t q = q0 + tid; q < q1; q += NTH) {
        const uint2* w = s_bp + (3u * q - tw0);
        if (w[0].x | w[1].x | w[2].x) reinterpret_cast<uint4*>(bmw)[q] = make_uint4(w[0].x, w[1].x, w[2].x, (uint32_t)base_u + w[0].y);
    }
    if (tid < 4) {
        const uint32_t w = tid < 2 ? tw0 + tid : 3u * q1 + (tid - 2);          // words before q0's and from q1's on
        if (tid < 2 ? w < min(3u * q0, tw1) : w < tw1 && w >= 3u * q0) {
            bmw[w + w / 3u] = s_bp[w - tw0].x;
            if (w % 3u == 0) bmw[4u * (w / 3u) + 3u] = (uint32_t)base_u + s_bp[w - tw0].y;
        }
    }
}

template <int NTH, int LOGMAX, int RANKS>
__device__ __forceinline__ void slice_block(SliceArgsPtr a, int32_t* s_tf)
{
    __shared__ __align__(16) int32_t s_main[slice_lds_words(LOGMAX, RANKS)];
    __shared__ int32_t s_base[4];
    // the first blocks have the listed slices, the others all that are not listed
    const int n_long_max = a->n_long_max;
    const bool listed = (int)blockIdx.x < n_long_max;
    const auto* list = as_constant(a->long_list);
    if (listed && (int)blockIdx.x >= list[0]) return;
    const int slice = listed ? list[1 + blockIdx.x] : (int)blockIdx.x - n_long_max;
    const auto* si = as_constant(a->slice_info) + slice;
    if (si->table < 0) return;                             // room for a slice this batch does not have
    if (!listed && (si->table & kListedFlag)) return;
    if (si->count <= kSliceKeep * NTH) slice_body<NTH, LOGMAX, RANKS, true>(a, slice, s_main, s_tf, s_base);
    else slice_body<NTH, LOGMAX, RANKS, false>(a, slice, s_main, s_tf, s_base);
}

__global__ void __launch_bounds__(kFineThreads, 8)
pk_slices_kernel(SliceArgs a)
{
    extern __shared__ int32_t s_dyn[];
    slice_block<kFineThreads, kSliceLogFine, kFineRanks>((SliceArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(), s_dyn);
}

// ... the shape for calls with a table too long for slices of 64 K keys.  Two blocks to a compute unit, though 16 registers
// are then spilled, some of the kept records among them: a launch is 59 us for 600 K IDs of 300 M rows and 182 for 4 M of 10^9
// rows, compiled for one block (nothing spilled) 76 and 240; slices of frequent keys would be 2 % faster that way.
__global__ void __launch_bounds__(kSliceThreads, 8)
pk_slices_wide_kernel(SliceArgs a)
{
    extern __shared__ int32_t s_dyn[];
    slice_block<kSliceThreads, kSliceLogMax, kSliceRanks>((SliceArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(), s_dyn);
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
    static_assert(KT <= kRoundMax, "positions are counted in 32 bits");
    const int n = s_slotpos[F];
    const int n_tiles = (n + KT - 1) / KT;
    for (XcdTiles it(n_tiles); it.valid(); it.next()) {
        // (every load without a condition, so that nothing is waited for in between)
        const int q0 = it.tile * KT, left = n - q0;
        const uint32_t* key_at = keys + q0;
        uint32_t kk[KT / NT];
#pragma unroll
        for (int k = 0; k < KT / NT; ++k) kk[k] = key_at[min(k * NT + (int)threadIdx.x, left - 1)];
        int j = -1;
        uint32_t at[KT / NT];
        bool ok[KT / NT];
#pragma unroll
        for (int k = 0; k < KT / NT; ++k) {
            const int q = min(q0 + k * NT + (int)threadIdx.x, n - 1);
            if (j < 0 || q >= s_slotpos[j + 1]) j = upper_bound_i32(s_slotpos, F + 1, q) - 1;   // the slot of this position
            kk[k] -= s_klo[j];
            // no lookup for a pack with rejected offsets, nor for a key that is none of its table (only possible then)
            ok[k] = k * NT + (int)threadIdx.x < left && s_pack[j] == 0 && kk[k] < s_rows[j];
            at[k] = s_wb[j] / 4 + (ok[k] ? (kk[k] >> 5) / 3u : 0u);
        }
        // the lookups of the tile's positions are all asked for before any is used
        uint4 x[KT / NT];
#pragma unroll
        for (int k = 0; k < KT / NT; ++k) x[k] = bitmap4[at[k]];
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
