// Device helpers shared by the kernels: block scans, the folding hash, combined LDS counters, the XCD-aware tile order.
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.

constexpr int NT = 256;   // threads per block of the streaming kernels

// a pointer that came out of a struct, known to be a global one (the compiler cannot see it: it would use flat accesses)
template <typename T>
__device__ __forceinline__ T* as_global(T* p) { return (T*)(__attribute__((address_space(1))) T*)p; }

// FRESH: the shuffles' addresses are formed again, where a scan stands in a loop that has no registers to keep them in.
template <int NTHREADS, bool FRESH = false>
__device__ __forceinline__ int block_excl_scan(int v, int* total)
{
    __shared__ int wsum[NTHREADS / 64];
    int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    if (FRESH) asm volatile("" : "+v"(lane));
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = FRESH ? __builtin_amdgcn_ds_bpermute((lane - o) << 2, inc) : __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    __syncthreads();   // readers of the previous call are done with wsum
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NTHREADS / 64; ++i) {
        int s = wsum[i];
        if (i < w) base += s;
        tot += s;
    }
    *total = tot;
    return base + inc - v;
}

// The row of an ID: the ID, taken as an unsigned 64-bit number, modulo the table's rows (exact).
// magic = floor((2^64 - 1) / rows): the upper half of ID * magic is the quotient or up to two below
// it, so the remainder formed from it is put right by two conditional subtractions (rows <= 2^30:
// nothing overflows).  A dozen integer operations instead of a 64-bit division.
__device__ __forceinline__ uint32_t fold_id(int64_t id, uint32_t rows, uint64_t magic)
{
    const uint64_t u = (uint64_t)id;
    if (u < rows) return (uint32_t)u;
    const uint64_t q = __umul64hi(u, magic);
    uint64_t r = u - q * (uint64_t)rows;
    if (r >= rows) r -= rows;
    if (r >= rows) r -= rows;
    return (uint32_t)r;
}

// first index in [0, n) whose value exceeds x, for a non-decreasing array
template <typename P>
__device__ __forceinline__ int upper_bound_i32(P a, int n, int x)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Blocks that need numbers from the blocks before them (the one-launch forward pass, the slices of large batches).  A block
// publishes its own number before it waits, and waits for lower ones only.  A lower block may not have started all the same:
// workgroups go to the eight XCDs in turn and each XCD starts its share in index order but at its own pace, and a second
// launch whose blocks wait may hold the places that the first one's need.  So patience is short, and a block that has run
// out of it counts what it lacks itself (count_before, small_count_before): it ends whatever else runs.  Only a block
// that says it has begun is waited for longer, bounded all the same: giving up raises bit 1 of the pack's error word, the
// pack's other waiting blocks see it and end too, and the kernels after it skip their work: the tables stay as they are.
// ---------------------------------------------------------------------------
constexpr int kSpinLimit = 1 << 22;

__device__ __forceinline__ void publish_desc(uint64_t* d, uint64_t v)
{
    __hip_atomic_store(d, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// cnt[idx] += 1 for every lane with `active`, and the value before the lane's own increment is
// returned.  IDs are heavily skewed (Sec. II-B), so many lanes of a wavefront often hit one counter,
// and LDS atomics on one address run one after the other: the lanes that share the first active
// lane's counter are combined into one add (up to two such groups are peeled off); a wavefront whose
// first group is a single lane is taken to have few repeats and goes on with plain atomics.
// Must be called by all 64 lanes of a wavefront together.
__device__ __forceinline__ int lds_inc_grouped(int32_t* cnt, uint32_t idx, bool active)
{
    const int lane = threadIdx.x & 63;
    int pos = 0;
    bool todo = active;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const uint64_t m = __ballot(todo);
        if (!m) return pos;
        const int leader = __ffsll((unsigned long long)m) - 1;
        const uint32_t v = (uint32_t)__shfl((int)idx, leader, 64);
        const bool mine = todo && idx == v;
        const uint64_t same = __ballot(mine);
        const int n = __popcll(same);
        int base = 0;
        if (lane == leader) base = atomicAdd(&cnt[v], n);
        base = __shfl(base, leader, 64);
        if (mine) {
            pos = base + __popcll(same & ((1ull << lane) - 1ull));
            todo = false;
        }
        if (n == 1) break;
    }
    if (todo) pos = atomicAdd(&cnt[idx], 1);
    return pos;
}

// The same for counters that are few (idx < n, n small and the same for the whole wavefront): with a
// handful of counters nearly every lane shares its counter with others, and LDS atomics on one address
// run one after the other, so the wavefront goes through the counters and makes one add for each that
// some lane wants.  POS: the value before the lane's own increment is returned.
constexpr int kFewCounters = 2;
template <bool POS>
__device__ __forceinline__ int lds_inc_few(int32_t* cnt, uint32_t idx, bool active, int n)
{
    const int lane = threadIdx.x & 63;
    int pos = 0;
    for (int s = 0; s < n; ++s) {
        const bool mine = active && idx == (uint32_t)s;
        const uint64_t m = __ballot(mine);
        if (!m) continue;
        const int leader = __ffsll((unsigned long long)m) - 1;
        int base = 0;
        if (lane == leader) base = atomicAdd(&cnt[s], __popcll(m));
        if (POS) {
            base = __shfl(base, leader, 64);
            if (mine) pos = base + __popcll(m & ((1ull << lane) - 1ull));
        }
    }
    return pos;
}

// Workgroups are handed to the 8 XCDs round-robin and each XCD has its own L2.
// Giving XCD x the x-th contiguous eighth of the tiles keeps the irregular
// accesses of neighbouring tiles (same table, same gradient columns) in one L2.
// Only locality depends on this; any placement gives the same results.
struct XcdTiles {
    int tile, hi, step;
    __device__ __forceinline__ XcdTiles(int n_tiles)
    {
        const int x = blockIdx.x & 7, i = blockIdx.x >> 3;
        const int chunk = (n_tiles + 7) >> 3;
        step = (gridDim.x + 7) >> 3;
        tile = x * chunk + i;
        hi = min((x + 1) * chunk, n_tiles);
    }
    __device__ __forceinline__ bool valid() const { return tile < hi; }
    __device__ __forceinline__ void next() { tile += step; }
};
