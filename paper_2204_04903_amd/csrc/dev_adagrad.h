// H6 + H7: gradient reduction per distinct key fused with the sparse Adagrad update.
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.

// ---------------------------------------------------------------------------
// H6+H7: per distinct key, the gradients of its occurrences are reduced in double (mirror of the forward
// pooling, Sec. II-D) and the row takes one Adagrad step in place.  Fused so the reduced gradient never
// goes to memory; ONE launch for all packs, so that a pack's tail is filled by the next one's keys.
//
// The ID distribution is heavily skewed (Sec. II-B), so keys are handled by how many occurrences they have:
//   up to kColdMax:   one lane group per key (a group is as many lanes as the row has 16-byte chunks);
//   up to kLongMin:   the wavefront that met the key among its own, its groups stride over the occurrences; of
//                     narrow rows, several such keys side by side; in large batches, where such keys are neighbours, the
//                     blocks of the longer ones (ada_dense);
//   longer:           a block of its own, which the launch starts first, in pieces of kPiece occurrences; the
//                     pieces of a key with several add into a row of partial sums, the last one to arrive
//                     takes the step.
// A wavefront takes as many consecutive keys as it has lane groups (in large batches more, ada_batch_keys) and waits for
// nobody; only the blocks of large batches whose plan pools by the mean fill a table first (ada_recips).
// Against tiles of occurrences decoded into LDS with a second launch for long keys (one launch per pack):
// small layer 22.5 -> 18.4 us a step, mixed dtypes with dimensions that are no multiple of four 514 -> 315
// (they ran one column per lane), bf16 sequences 725 -> 660.  What bounds it: with one-hot fields of 8192 bags (26 fields,
// 27 us) the chain of dependent loads, 2.9 TB/s of the bytes it needs;
// else the gathered gradient chunks, which the L2s hold only while an XCD's wavefronts stay on neighbouring
// tables: hence the eighths per XCD below, for long keys too, and no more than kLongBlocks blocks of those.
// 80 registers, six wavefronts per SIMD: with 64 the compiler spills and everything is a quarter slower.
// ---------------------------------------------------------------------------
struct AdaPack {
    void* W; float* A; HotView hv;
    uint32_t addr_max;           // largest element offset into grad_out at which a chunk of the pack can start
    int32_t D, sh, p;            // dimension, log2 of the lanes per row, pack
    int32_t kind;                // 1: bf16, 2: mean pooling (entries carry bag lengths), 4: dimension below four
    uint32_t batch;              // how many keys a wavefront takes at once (ada_batch_keys), as key_batch_word
};
constexpr int kAdaPacks = 16;    // packs of one launch
struct AdaJob {
    AdaPack pack[kAdaPacks];
    int32_t n_packs, hot_blocks, key_blocks, ent_mult;
    const PackState* st; const uint32_t* unique; const int32_t* seg; const int32_t* marks; const uint32_t* ent;
    double* ghot; int32_t* ticket; int32_t dmax;
    const float* grad; int64_t gstride, out_dim;
    float lr, eps;
};

// what a lane needs to add up the gradient chunks of a range of entries
struct GradView {
    const float* grad;           // + the lane's first column
    const uint32_t* ent;
    const double* recip;         // 1 / L of bag lengths below kRecips, in LDS (large batches' launches)
    uint32_t gstride, out_dim, addr_max;
    int D;
};

// 1 / L in double without a division: the hardware's fp32 reciprocal (1 ulp, and L's own rounding above 2^24: 2^-22.4
// together) and two Newton steps.  Correctly rounded, as the division: the second step's error is 2^-89 of the result, and
// 1 / L for L below 2^31 is 2^-84 or more away from the middle between two doubles (unless L is a power of two: exact).
__device__ __forceinline__ double recip_len(uint32_t L)
{
    const double d = (double)max(L, 1u);
    double r = (double)__builtin_amdgcn_rcpf((float)d);
    r = fma(r, fma(-d, r, 1.0), r);
    return fma(r, fma(-d, r, 1.0), r);
}

// where entries' chunks stand: inside grad_out, whatever the list holds
template <int N>
__device__ __forceinline__ void grad_places(const GradView& g, uint32_t (&at)[N])
{
    if (g.gstride != g.out_dim) {                          // padded gradient rows
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const uint32_t b = at[k] / g.out_dim;
            at[k] = b * g.gstride + (at[k] - b * g.out_dim);
        }
    }
#pragma unroll
    for (int k = 0; k < N; ++k) at[k] = min(at[k], g.addr_max);
}

// Bag lengths whose reciprocals a block of a large batch keeps in LDS (mean pooling; TABLE below): one read where the two
// Newton steps and their conversions are nine instructions, in every lane, for every entry.  The other launches form
// them: the table gains those nothing (eight one-hot fields of 512, mean: 6.4 us with and without), and with the entries that
// accum_piece asks for ahead the Hot-storage's kernels spilled one and four registers (none and two without).
constexpr uint32_t kRecips = 512;
__device__ __forceinline__ double recip_of(const GradView& g, uint32_t L) { return L < kRecips ? g.recip[L] : recip_len(L); }

// a round's entries: the chunks' offsets and their bags' lengths (read past the range's end up to 3 entries far)
template <bool MEAN> struct Entries { uint32_t v[MEAN ? 8 : 4]; };
template <bool MEAN>
__device__ __forceinline__ Entries<MEAN> load_entries(const GradView& g, uint32_t s)
{
    Entries<MEAN> e;
    load_u32<4>(g.ent + (MEAN ? 2 : 1) * (size_t)s, e.v);
    if constexpr (MEAN) load_u32<4>(g.ent + 2 * (size_t)s + 4, e.v + 4);
    return e;
}

// acc += sum of scale * gradient chunk over the entries e of positions s to s + 3, of which those below s_end count (ALL:
// every one).
// The 1/L of mean pooling is formed and applied in double: the first Adagrad step of a row moves a weight by
// lr*g/(|g|+eps), so where the gradients of a key cancel (|g| near eps) an error of 1e-8 in g is an error of
// lr in the weight, and a float 1/L alone is off by 6e-8 of every term.
// The chunks of a round are asked for without branches between them (the compiler would wait for each before
// the next one's branch): where the range ends inside a round, its first chunk again, counted as zero.
template <bool MEAN, bool NARROW, bool ALL, bool TABLE, typename Fn>
__device__ __forceinline__ void accum_round(double (&acc)[4], const GradView& g, const Entries<MEAN>& e, uint32_t s, uint32_t s_end, Fn&& meanwhile)
{
    uint32_t at[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) at[k] = e.v[MEAN ? 2 * k : k];
    grad_places(g, at);
    float x[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) load_f32x4<NARROW>(g.grad + (ALL || s + k < s_end ? at[k] : at[0]), g.D, x[k]);
    double c[4] = {1.0, 1.0, 1.0, 1.0};
    if constexpr (MEAN && TABLE) {
        if (max(max(e.v[1], e.v[3]), max(e.v[5], e.v[7])) < kRecips) {
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = g.recip[e.v[2 * k + 1]];
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = recip_len(e.v[2 * k + 1]);
        }
    }
    meanwhile();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool on = ALL || k == 0 || s + k < s_end;
        if constexpr (MEAN && !TABLE) c[k] = recip_len(e.v[2 * k + 1]);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double d = (double)(on ? x[k][v] : 0.f);
            acc[v] = MEAN ? fma(c[k], d, acc[v]) : acc[v] + d;
        }
    }
}

// acc += the entries [s, s+4), [s+step, s+step+4), ... below s_end
template <bool MEAN, bool NARROW, bool TABLE>
__device__ __forceinline__ void accum_range(double (&acc)[4], const GradView& g, uint32_t s, uint32_t s_end, uint32_t step)
{
#pragma nounroll
    for (; s < s_end; s += step) accum_round<MEAN, NARROW, false, TABLE>(acc, g, load_entries<MEAN>(g, s), s, s_end, [] {});
}

// The same for a long key's piece in a large batch: nearly all its rounds are whole ones, and the next one's entries are on
// their way while the chunks of this one are.
template <bool MEAN, bool NARROW>
__device__ __forceinline__ void accum_piece(double (&acc)[4], const GradView& g, uint32_t s, uint32_t s_end, uint32_t step)
{
    Entries<MEAN> e = load_entries<MEAN>(g, min(s, s_end - 1));
#pragma nounroll
    for (; s + 4 <= s_end; s += step) {
        Entries<MEAN> next;
        accum_round<MEAN, NARROW, true, true>(acc, g, e, s, s_end, [&] { next = load_entries<MEAN>(g, min(s + step, s_end - 1)); });
        e = next;
    }
    if (s < s_end) accum_round<MEAN, NARROW, false, true>(acc, g, e, s, s_end, [] {});
}

// one Adagrad step of the lane's columns of a row: a += g^2 ; w -= lr * g / (sqrt(a) + eps)
template <bool BF16, bool NARROW>
__device__ __forceinline__ void row_step(const RowPtr& r, int D, const double (&acc)[4], float (&w)[4], float (&a)[4],
                                         float lr, float eps)
{
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float g = (float)acc[v];
        a[v] = a[v] + g * g;
        // square root and reciprocal as the hardware gives them (1 ulp each): the step is within
        // 3 ulp of lr*g/(sqrt(a)+eps), and it is at most lr in size
        w[v] = w[v] - lr * g * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(a[v]) + eps);
    }
    store_f32x4<NARROW>(r.a, D, a);
    store_w4<BF16, NARROW>(r.w, D, w);
}

// sum over the lane groups of `lanes` neighbouring lanes (butterfly); every lane ends with the total
__device__ __forceinline__ void wave_group_sum(double (&acc)[4], int lpr, int lanes)
{
#pragma nounroll
    for (int o = lpr; o < lanes; o <<= 1)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] += __shfl_xor(acc[v], o, 64);
}

// Long keys.  Every kMarkStep-th position names the key that holds it; a piece belongs to the first such
// position inside it (every piece is longer than kMarkStep), and a block to kMarksPerBlock of them.
constexpr int kMarksPerBlock = 4;      // (16: the mixed layer 16 % slower, a block then has several pieces one after the other)
constexpr int kLongBlocks = 768;

constexpr int kTeam = 4;               // lane groups that share a key of more than kColdMax occurrences at least

// Keys of more than kColdMax and up to kLongMin occurrences, lanes first to first + n - 1 holding their segments and rows (batches):
// dealt to teams of `team` lane groups: all groups for a key alone, several keys side by side.
template <bool BF16, bool MEAN, bool NARROW, bool HYB>
__device__ __forceinline__ void ada_team_keys(const AdaJob& job, const AdaPack& k, const GradView& gv, int d0, bool act, int first, int n,
                                              int p_a, int p_b, uint32_t p_row)
{
    const int lane = threadIdx.x & 63, lpr = 1 << k.sh, gpw = 64 >> k.sh, g = lane >> k.sh;
    int team = gpw;
    while (team > kTeam && gpw < team * n) team >>= 1;
    const int in_team = g & (team - 1);
#pragma nounroll
    for (int k0 = 0; k0 < n; k0 += gpw / team) {
        const int kk = k0 + g / team, src = first + min(kk, n - 1);
        const int wa = __shfl(p_a, src, 64), sb = __shfl(p_b, src, 64), wb = kk < n ? sb : wa;
        const uint32_t row = (uint32_t)__shfl((int)p_row, src, 64);
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        if (act) accum_range<MEAN, NARROW, true>(acc, gv, (uint32_t)(wa + 4 * in_team), (uint32_t)wb, (uint32_t)(4 * team));
        wave_group_sum(acc, lpr, lpr * team);
        if (in_team == 0 && act && kk < n) {               // (asked for earlier, the row would not fit the registers)
            const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, row, k.D, d0);
            float w[4], ac[4];
            load_w4<BF16, NARROW>(r.w, k.D, w);
            load_f32x4<NARROW>(r.a, k.D, ac);
            row_step<BF16, NARROW>(r, k.D, acc, w, ac, job.lr, job.eps);
        }
    }
}

// Stretches of kMarksPerBlock marks' positions that have few keys: in batches, where frequent IDs are neighbours, a wavefront
// would have 16 to 64 keys of up to kLongMin occurrences one after the other.  Those that begin in such a stretch are
// left to the block that looks for long keys there.  us with low IDs frequent, batches without this, this way, and handfuls:
// 100 fields of 16 columns, 8.2 M IDs 249 162 172; 60 of 64, 2.5 M 260 134 132; 20 of 200, 0.8 M 345 178 175; 100 of 32, 4.5 M 299
// 147 157.  Where they are scattered, the look at two marks costs the mixed layer of 1 M IDs 70.6 72.6, 200 fields of 21 M 592 597.
constexpr int kDenseKeys = 64, kRange = kMarksPerBlock * kMarkStep;
__device__ __forceinline__ bool ada_dense(const int32_t* marks, int n_marks, int range)
{
    const int m = range * kMarksPerBlock;
    return m + kMarksPerBlock < n_marks && marks[m + kMarksPerBlock] - marks[m] <= kDenseKeys;
}

// stretches of the XCD's eighth
__device__ __forceinline__ int ada_ranges(int n_marks, int x, int* per)
{
    const int n = (n_marks + kMarksPerBlock - 1) / kMarksPerBlock;
    *per = (n + 7) >> 3;
    return max(0, min(*per, n - x * *per));
}

// the lane's place among those of `mask`, after `before` others, as a byte address for a permute
__device__ __forceinline__ int lane_rank(uint64_t mask, int before)
{
    return (before + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))) * 4;
}

// How a launch takes the keys of up to kLongMin occurrences: handfuls, a key of more than kColdMax at a time, or several in
// teams of lane groups (ada_keys); batches by the number of occurrences (ada_batch_keys).
constexpr int kHandfuls = 0, kTeams = 1, kBatches = 2;

template <bool BF16, bool MEAN, bool NARROW, bool HYB, int KEYS>
__device__ __forceinline__ int ada_long_keys(const AdaJob& job, const AdaPack& k, int idx, int x, int stride, const double* recip, double (*s_red)[64][4])
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const PackState* st = as_global(job.st) + k.p;
    // A forward pass that raised the error word (input rejected, or a scan that ran out of patience)
    // left no lists worth reading: the tables are then left alone.
    const int n = st->error ? 0 : st->nnz, start = st->start;
    const int32_t* seg = as_global(job.seg) + start + k.p;
    const int32_t* marks = as_global(job.marks) + start / kMarkStep + k.p;
    const int n_marks = (n + kMarkStep - 1) / kMarkStep;
    int per;
    const int n_mine = ada_ranges(n_marks, x, &per);
    const int lpr = 1 << k.sh, gpw = 64 >> k.sh, li = lane & (lpr - 1), g = lane >> k.sh;
    const int d0 = NARROW ? 0 : lane_col(li, k.D);
    const bool act = 4 * li < k.D;
    const GradView gv{as_global(job.grad) + d0, as_global(job.ent) + (size_t)start * job.ent_mult, recip, (uint32_t)job.gstride,
                      (uint32_t)job.out_dim, k.addr_max, k.D};
    for (; idx < n_mine; idx += stride) {
        const int m0 = (x * per + idx) * kMarksPerBlock + lane;
        int u = 0, s0 = 0, s1 = 0, piece = 0, n_pieces = 1;
        bool mine = lane < kMarksPerBlock && m0 < n_marks;
        if (mine) {
            u = marks[m0];
            s0 = seg[u]; s1 = seg[u + 1];
            const int len = s1 - s0;
            n_pieces = max(1, len / kPiece);
            piece = min((m0 * kMarkStep - s0) / kPiece, n_pieces - 1);
            mine = len > kLongMin && (m0 * kMarkStep - s0) - piece * kPiece < kMarkStep;
        }
        for (uint64_t todo = __ballot(mine); todo; todo &= todo - 1) {     // the same in all wavefronts of the block
            const int lead = __ffsll((unsigned long long)todo) - 1;
            const int ku = __builtin_amdgcn_readlane(u, lead), ks0 = __builtin_amdgcn_readlane(s0, lead);
            const int ks1 = __builtin_amdgcn_readlane(s1, lead), kp = __builtin_amdgcn_readlane(piece, lead);
            const int kn = __builtin_amdgcn_readlane(n_pieces, lead);
            const int a = ks0 + kp * kPiece, b = kp + 1 == kn ? ks1 : a + kPiece;
            const bool fin = wv == 0 && g == 0 && act;                      // the lanes that take the step
            const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, as_global(job.unique)[start + ku], k.D, d0);
            float w[4], ac[4];
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            if (act) {
                const uint32_t s = (uint32_t)(a + (wv * gpw + g) * 4), step = (uint32_t)(4 * gpw * (NT / 64));
                if constexpr (KEYS == kBatches) accum_piece<MEAN, NARROW>(acc, gv, s, (uint32_t)b, step);
                else accum_range<MEAN, NARROW, false>(acc, gv, s, (uint32_t)b, step);
            }
            if (fin && kn == 1) { load_w4<BF16, NARROW>(r.w, k.D, w); load_f32x4<NARROW>(r.a, k.D, ac); }
            wave_group_sum(acc, lpr, 64);
            __syncthreads();                           // the previous piece's sums are consumed
            if (g == 0) {
#pragma unroll
                for (int v = 0; v < 4; ++v) s_red[wv][li][v] = acc[v];
            }
            __syncthreads();
            if (!fin) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double t = 0.0;
#pragma unroll
                for (int w2 = 0; w2 < NT / 64; ++w2) t += s_red[w2][li][v];
                acc[v] = t;
            }
            if (kn > 1) {
                // The pieces meet at device-scope atomics.  Every add returns its old value and the ticket is
                // taken after all of them have: so whoever draws the last ticket finds every piece's sums (no
                // fence, which would write the whole L2 back).
                const size_t slot = (size_t)(start / kPiece + k.p) + (size_t)(ks0 / kPiece);
                double* prow = as_global(job.ghot) + slot * job.dmax + d0;
                double old = 0.0;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (d0 + v >= 4 * li && v < k.D) old += atomicAdd(prow + v, acc[v]);   // (a column two lanes hold is added once)
                asm volatile("s_waitcnt vmcnt(0)" ::"v"(old) : "memory");
                int t = 0;
                if (li == 0) t = atomicAdd(as_global(job.ticket) + slot, 1);
                t = __builtin_amdgcn_readfirstlane(t);
                if (t != kn - 1) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[v] = v < k.D ? __hip_atomic_load(prow + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
                // ... and leaves them as the forward pass did, so that a context serves any number of backward passes
                // (after all lanes' loads: the last two may hold the same columns)
                asm volatile("s_waitcnt vmcnt(0)" ::"v"(acc[0]), "v"(acc[1]), "v"(acc[2]), "v"(acc[3]) : "memory");
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (v < k.D) __hip_atomic_store(prow + v, 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (li == 0) __hip_atomic_store(as_global(job.ticket) + slot, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                load_w4<BF16, NARROW>(r.w, k.D, w);
                load_f32x4<NARROW>(r.a, k.D, ac);
            }
            row_step<BF16, NARROW>(r, k.D, acc, w, ac, job.lr, job.eps);
        }
    }
    return idx - n_mine;
}

// The keys of more than kColdMax and up to kLongMin occurrences that begin in a dense stretch (launches in batches), every fourth
// of a stretch to a wavefront, after the long keys of the same blocks.  (The kernel spills a register, four with this inside
// ada_long_keys' loop, none in blocks of their own, but those cost the mixed layer of 1 M IDs 2 us of 72.6.)
template <bool BF16, bool MEAN, bool NARROW, bool HYB, int KEYS>
__device__ __forceinline__ int ada_stretch_keys(const AdaJob& job, const AdaPack& k, int idx, int x, int stride, const double* recip)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const PackState* st = as_global(job.st) + k.p;
    const int n = st->error ? 0 : st->nnz, start = st->start;
    const int32_t* seg = as_global(job.seg) + start + k.p;
    const int32_t* marks = as_global(job.marks) + start / kMarkStep + k.p;
    const int n_marks = (n + kMarkStep - 1) / kMarkStep;
    int per;
    const int n_mine = ada_ranges(n_marks, x, &per);
    const int li = lane & ((1 << k.sh) - 1), d0 = NARROW ? 0 : lane_col(li, k.D);
    const GradView gv{as_global(job.grad) + d0, as_global(job.ent) + (size_t)start * job.ent_mult, recip, (uint32_t)job.gstride,
                      (uint32_t)job.out_dim, k.addr_max, k.D};
#pragma nounroll
    for (; idx < n_mine; idx += stride) {
        const int range = x * per + idx;
        if (!ada_dense(marks, n_marks, range)) continue;
        // (the first and the last may begin outside the stretch)
        const int u0 = marks[range * kMarksPerBlock], u1 = marks[(range + 1) * kMarksPerBlock];
        const int u = u0 + wv + lane * (NT / 64), v = min(u, u1), a = seg[v], b = seg[v + 1];
        const bool on = u <= u1 && a / kRange == range && b - a > kColdMax && b - a <= kLongMin;
        const uint64_t mine = __ballot(on);
        if (mine == 0) continue;
        const int to = lane_rank(on ? mine : ~mine, on ? 0 : __popcll(mine));
        ada_team_keys<BF16, MEAN, NARROW, HYB>(job, k, gv, d0, 4 * li < k.D, 0, __popcll(mine), __builtin_amdgcn_ds_permute(to, a),
                                               __builtin_amdgcn_ds_permute(to, b), (uint32_t)__builtin_amdgcn_ds_permute(to, (int)as_global(job.unique)[start + v]));
    }
    return idx - n_mine;
}

// The other keys of a pack.  XCD x takes the x-th eighth of the keys (neighbouring keys share gradient
// columns: one L2 then holds them), its wavefronts take consecutive handfuls.
template <bool BF16, bool MEAN, bool NARROW, bool HYB, int KEYS>
__device__ __forceinline__ int ada_keys(const AdaJob& job, const AdaPack& k, int idx, int x, int stride)
{
    const int lane = threadIdx.x & 63;
    const PackState* st = as_global(job.st) + k.p;
    const int U = st->error ? 0 : st->n_unique, start = st->start;
    const int lpr = 1 << k.sh, gpw = 64 >> k.sh, li = lane & (lpr - 1), g = lane >> k.sh;
    const int n_chunks = (U + gpw - 1) >> (6 - k.sh);
    const int per = (n_chunks + 7) >> 3;
    const int n_mine = max(0, min(per, n_chunks - x * per));
    const int32_t* seg = as_global(job.seg) + start + k.p + (x * per) * gpw;
    const uint32_t* uq = as_global(job.unique) + start + (x * per) * gpw;
    const int u_end = U - (x * per) * gpw;
    const int d0 = NARROW ? 0 : lane_col(li, k.D);
    const bool act = 4 * li < k.D;
    const GradView gv{as_global(job.grad) + d0, as_global(job.ent) + (size_t)start * job.ent_mult, nullptr, (uint32_t)job.gstride,
                      (uint32_t)job.out_dim, k.addr_max, k.D};
    int s0 = 0, s1 = 0;
    uint32_t row = 0;
    auto fetch = [&](int c) {                              // the segment and the row of this group's key of handful c
        const int u = min(c * gpw + g, u_end - 1);         // (past the end: some key, not used)
        s0 = seg[u]; s1 = seg[u + 1]; row = uq[u];
        if (c * gpw + g >= u_end) s1 = s0;
    };
    if (idx < n_mine) fetch(idx);
#pragma nounroll
    for (; idx < n_mine; idx += stride) {
        const int a = s0, b = s1, len = b - a;
        const uint32_t r0 = row;
        fetch(min(idx + stride, n_mine - 1));
        if (len > 0 && len <= kColdMax && act) {
            const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, r0, k.D, d0);
            float w[4], ac[4];
            load_w4<BF16, NARROW>(r.w, k.D, w);
            load_f32x4<NARROW>(r.a, k.D, ac);
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            accum_range<MEAN, NARROW, false>(acc, gv, (uint32_t)a, (uint32_t)b, 4);
            row_step<BF16, NARROW>(r, k.D, acc, w, ac, job.lr, job.eps);
        }
        uint64_t todo = __ballot(li == 0 && len > kColdMax && len <= kLongMin);
        if (todo == 0) continue;
        if constexpr (KEYS != kTeams) {                            // one key after the other
#pragma nounroll
            for (; todo; todo &= todo - 1) {
                const int lead = __ffsll((unsigned long long)todo) - 1;
                const int wa = __builtin_amdgcn_readlane(a, lead), wb = __builtin_amdgcn_readlane(b, lead);
                const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, (uint32_t)__builtin_amdgcn_readlane((int)r0, lead), k.D, d0);
                const bool fin = g == 0 && act;
                float w[4], ac[4];
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                if (act) accum_range<MEAN, NARROW, false>(acc, gv, (uint32_t)(wa + 4 * g), (uint32_t)wb, (uint32_t)(4 * gpw));
                if (fin) { load_w4<BF16, NARROW>(r.w, k.D, w); load_f32x4<NARROW>(r.a, k.D, ac); }    // (on their way while the groups are added up)
                wave_group_sum(acc, lpr, 64);
                if (fin) row_step<BF16, NARROW>(r, k.D, acc, w, ac, job.lr, job.eps);
            }
        } else {
            // The keys met are dealt to teams of `team` lane groups: all groups for a key alone, several keys side by side.
            const int n = __popcll(todo);
            int team = gpw;
            while (team > kTeam && gpw < team * n) team >>= 1;
            const int in_team = g & (team - 1);
            const uint64_t below = (1ull << lane) - 1ull;
            const int rank = todo >> lane & 1 ? __popcll(todo & below) : n + __popcll(~todo & below);
            const int nth = __builtin_amdgcn_ds_permute(rank * 4, lane);       // lane k: the first lane of the k-th key met
#pragma nounroll
            for (int k0 = 0; k0 < n; k0 += gpw / team) {
                const int kk = k0 + g / team;
                const int src = __shfl(nth, min(kk, n - 1), 64);
                const int wa = __shfl(a, src, 64), sb = __shfl(b, src, 64), wb = kk < n ? sb : wa;
                const uint32_t row_k = (uint32_t)__shfl((int)r0, src, 64);
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                if (act) accum_range<MEAN, NARROW, false>(acc, gv, (uint32_t)(wa + 4 * in_team), (uint32_t)wb, (uint32_t)(4 * team));
                wave_group_sum(acc, lpr, lpr * team);
                if (in_team == 0 && act && kk < n) {       // (asked for earlier, the row would not fit the registers)
                    const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, row_k, k.D, d0);
                    float w[4], ac[4];
                    load_w4<BF16, NARROW>(r.w, k.D, w);
                    load_f32x4<NARROW>(r.a, k.D, ac);
                    row_step<BF16, NARROW>(r, k.D, acc, w, ac, job.lr, job.eps);
                }
            }
        }
    }
    return idx - n_mine;
}

// the code for a pack's kind
#define PK_ADA_KINDS(FN, ...)                                                                   \
    switch (k.kind) {                                                                           \
        case 0: idx = FN<false, false, false, HYB, KEYS>(__VA_ARGS__); break;                   \
        case 1: idx = FN<true, false, false, HYB, KEYS>(__VA_ARGS__); break;                    \
        case 2: idx = FN<false, true, false, HYB, KEYS>(__VA_ARGS__); break;                    \
        case 3: idx = FN<true, true, false, HYB, KEYS>(__VA_ARGS__); break;                     \
        case 4: if constexpr (KEYS != kHandfuls) idx = FN<false, false, true, HYB, KEYS>(__VA_ARGS__); break;  \
        case 5: if constexpr (KEYS != kHandfuls) idx = FN<true, false, true, HYB, KEYS>(__VA_ARGS__); break;   \
        case 6: if constexpr (KEYS != kHandfuls) idx = FN<false, true, true, HYB, KEYS>(__VA_ARGS__); break;   \
        case 7: if constexpr (KEYS != kHandfuls) idx = FN<true, true, true, HYB, KEYS>(__VA_ARGS__); break;    \
    }

// ---------------------------------------------------------------------------
// Large batches.  A wavefront takes batches of up to 64 consecutive keys, a lane per key at first: its segment, its row,
// its first entry, the next batches' on their way.  Then the keys are taken by their number of occurrences, one, few, more, a
// lane group each (or a team of groups), so that a wavefront's groups do about the same.  Two thirds of the keys have one
// occurrence: their entries are there, so row and gradient chunk are asked for at once.  Against handfuls of
// consecutive keys, each taking rounds of four entries: 150 M vector instructions for 200 fields of 21 M IDs, 86 M now.  What is
// left is the rate of line requests (26 M reads, of them 7 M for rows, and 11 M writes): with more wavefronts or
// fewer, or more rows in flight in each, the times are the same.  200 fields 654 us a launch, 594; 1000 fields of 8 and 16
// columns 423, 408; bf16 sequences 254, 212; the mixed layer of 1 M IDs 87, 69; 26 one-hot fields of 65536 126, 128.  A small batch
// (26 one-hot fields of 8192) is a chain of loads, one longer here: 20 us, 23.  (keys_in_batches has the line between them.)
// ---------------------------------------------------------------------------
// batches of the XCD's eighth of U keys (a division here stands in every wavefront's way once per pack: the mixed layer of
// eight packs 72.0 us, 70.1 with the product)
__device__ __forceinline__ int ada_batches(int U, const AdaPack& k, int x, int* per)
{
    const int n = key_batches(U, k.batch);
    *per = (n + 7) >> 3;
    return max(0, min(*per, n - x * *per));
}

template <bool BF16, bool MEAN, bool NARROW, bool HYB, int KEYS>
__device__ __forceinline__ int ada_batch_keys(const AdaJob& job, const AdaPack& k, int idx, int x, int stride, const double* recip)
{
    const int lane = threadIdx.x & 63;
    const PackState* st = as_global(job.st) + k.p;
    const int U = st->error ? 0 : st->n_unique, start = st->start;
    int per;
    const int n_mine = ada_batches(U, k, x, &per), K = key_batch_size(k.batch), u0 = x * per * K;
    if (idx >= n_mine) return idx - n_mine;
    const int lpr = 1 << k.sh, gpw = 64 >> k.sh, li = lane & (lpr - 1), g = lane >> k.sh;
    const int32_t* seg = as_global(job.seg) + start + k.p + u0;
    const uint32_t* uq = as_global(job.unique) + start + u0;
    const int32_t* marks = as_global(job.marks) + start / kMarkStep + k.p;
    const int n_marks = (st->nnz + kMarkStep - 1) / kMarkStep;
    const int u_end = U - u0;
    const int d0 = NARROW ? 0 : lane_col(li, k.D);
    const bool act = 4 * li < k.D;
    const GradView gv{as_global(job.grad) + d0, as_global(job.ent) + (size_t)start * job.ent_mult, recip, (uint32_t)job.gstride,
                      (uint32_t)job.out_dim, k.addr_max, k.D};
    struct Key { int a, b; uint32_t row; };                // a lane's key: its segment, its row
    struct First { uint32_t at, L; };                      // its first entry
    auto fetch = [&](int c) {
        const int u = c * K + lane, v = min(u, u_end - 1);      // (past the end: some key, not used)
        Key q{seg[v], seg[v + 1], uq[v]};
        if (u >= min(u_end, (c + 1) * K)) q.b = q.a;
        return q;
    };
    auto fetch_first = [&](const Key& q) {
        First f{0, 1};
        if constexpr (MEAN) { uint32_t e[2]; load_u32<2>(gv.ent + 2 * (size_t)q.a, e); f.at = e[0]; f.L = e[1]; }
        else f.at = gv.ent[q.a];
        return f;
    };
    Key cur = fetch(idx), next = fetch(min(idx + stride, n_mine - 1));
    First first = fetch_first(cur);
#pragma nounroll
    for (; idx < n_mine; idx += stride) {
        const Key q = cur;
        const First f = first;
        cur = next;
        first = fetch_first(cur);
        next = fetch(min(idx + 2 * stride, n_mine - 1));
        // the batch in the order of the keys' occurrences: one | up to 4 | up to kColdMax | up to kLongMin | others
        const int len = q.b - q.a;
        bool team = len > kColdMax && len <= kLongMin;
        if (team) team = !ada_dense(marks, n_marks, q.a / kRange);
        const uint64_t m1 = __ballot(len == 1), m4 = __ballot(len >= 2 && len <= 4), m8 = __ballot(len > 4 && len <= kColdMax);
        const uint64_t mt = __ballot(team), mo = ~(m1 | m4 | m8 | mt);
        const int n1 = __popcll(m1), n4 = n1 + __popcll(m4), n8 = n4 + __popcll(m8), nt = n8 + __popcll(mt);
        const bool none = len < 1 || (len > kColdMax && !team);
        const uint64_t mm = none ? mo : len == 1 ? m1 : len <= 4 ? m4 : len <= kColdMax ? m8 : mt;
        const int base = none ? nt : len == 1 ? 0 : len <= 4 ? n1 : len <= kColdMax ? n4 : n8;
        const int to = lane_rank(mm, base);
        const uint32_t p_row = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)q.row);
        if (n1) {
            const uint32_t p_at = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)f.at);
            const uint32_t p_L = MEAN ? (uint32_t)__builtin_amdgcn_ds_permute(to, (int)f.L) : 1u;
#pragma nounroll
            for (int h = 0; h < n1; h += gpw) {
                const int i = h + g, src = min(i, n1 - 1);
                const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, (uint32_t)__shfl((int)p_row, src, 64), k.D, d0);
                const uint32_t L = MEAN ? (uint32_t)__shfl((int)p_L, src, 64) : 1u;
                uint32_t at[1] = {(uint32_t)__shfl((int)p_at, src, 64)};
                grad_places(gv, at);
                float xg[4], w[4], a[4];
                load_f32x4<NARROW>(gv.grad + at[0], k.D, xg);
                load_w4<BF16, NARROW>(r.w, k.D, w);
                load_f32x4<NARROW>(r.a, k.D, a);
                if (i < n1 && act) {
                    double acc[4];
                    const double c = MEAN ? recip_of(gv, L) : 1.0;
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[v] = MEAN ? fma(c, (double)xg[v], 0.0) : 0.0 + (double)xg[v];
                    row_step<BF16, NARROW>(r, k.D, acc, w, a, job.lr, job.eps);
                }
            }
        }
        if (n1 == nt) continue;
        const int p_a = __builtin_amdgcn_ds_permute(to, q.a), p_b = __builtin_amdgcn_ds_permute(to, q.b);
#pragma nounroll
        for (int h = n1; h < n8; h += gpw) {
            const int i = h + g, src = min(i, n8 - 1);
            const int a = __shfl(p_a, src, 64), b = __shfl(p_b, src, 64);
            const uint32_t row = (uint32_t)__shfl((int)p_row, src, 64);
            if (i < n8 && act) {
                const RowPtr r = row_ptr<BF16, HYB>(k.W, k.A, k.hv, row, k.D, d0);
                float w[4], ac[4];
                load_w4<BF16, NARROW>(r.w, k.D, w);
                load_f32x4<NARROW>(r.a, k.D, ac);
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                accum_range<MEAN, NARROW, true>(acc, gv, (uint32_t)a, (uint32_t)b, 4);
                row_step<BF16, NARROW>(r, k.D, acc, w, ac, job.lr, job.eps);
            }
        }
        ada_team_keys<BF16, MEAN, NARROW, HYB>(job, k, gv, d0, act, n8, nt - n8, p_a, p_b, p_row);
    }
    return idx - n_mine;
}

// kTeams: for launches with rows of kTeamDim columns and fewer, where a wavefront's handful has 16 to 64 keys: where
// frequent IDs are neighbours, all of them can have more than kColdMax occurrences, and one after the other they take
// longer than everything else (16 tables of 82 K occurrences, dimension 3: 238 us, in teams 79; dimension 8: 79,
// 57).  Wider rows have few keys to a handful and keep the registers (26 one-hot fields of 32 columns, a
// step: 52 us, 54 with the teams' code).
constexpr int kTeamDim = 16;

// reciprocals of bag lengths, where some pack of the launch pools by the mean
__device__ __forceinline__ void ada_recips(const AdaJob& job, double* s_recip)
{
    if (job.ent_mult == 2) {
        for (uint32_t i = threadIdx.x; i < kRecips; i += NT) s_recip[i] = recip_len(i);
        __syncthreads();
    }
}

template <bool HYB, int KEYS>
__global__ void __launch_bounds__(NT, 6)
pk_adagrad_kernel(AdaJob job)
{
    __shared__ double s_red[NT / 64][64][4];               // per-wavefront sums of a long key's piece
    __shared__ double s_recip[KEYS == kBatches ? kRecips : 1];
    if constexpr (KEYS == kBatches) ada_recips(job, s_recip);
    if ((int)blockIdx.x < job.hot_blocks) {
        int idx = blockIdx.x >> 3;
        for (int i = 0; i < job.n_packs; ++i) {
            const AdaPack& k = job.pack[i];
            PK_ADA_KINDS(ada_long_keys, job, k, idx, blockIdx.x & 7, job.hot_blocks >> 3, s_recip, s_red)
        }
        if constexpr (KEYS == kBatches) {
            idx = blockIdx.x >> 3;
            for (int i = 0; i < job.n_packs; ++i) {
                const AdaPack& k = job.pack[i];
                PK_ADA_KINDS(ada_stretch_keys, job, k, idx, blockIdx.x & 7, job.hot_blocks >> 3, s_recip)
            }
        }
        return;
    }
    const int kb = (int)blockIdx.x - job.hot_blocks, stride = (job.key_blocks >> 3) * (NT / 64);
    // (the same in all lanes, so that a pack's work and the choice of its code are found on the scalar unit)
    int idx = (kb >> 3) * (NT / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (int i = 0; i < job.n_packs; ++i) {
        const AdaPack& k = job.pack[i];
        if constexpr (KEYS == kBatches) { PK_ADA_KINDS(ada_batch_keys, job, k, idx, kb & 7, stride, s_recip) }
        else { PK_ADA_KINDS(ada_keys, job, k, idx, kb & 7, stride) }
    }
}
