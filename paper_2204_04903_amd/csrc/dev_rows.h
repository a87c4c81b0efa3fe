// Row access (fp32 / bf16, 16 bytes per lane) and where a row lives (plain table or HybridHash).
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.

// ---------------------------------------------------------------------------
// bf16 as bits
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint32_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);      // round to nearest, ties to even (finite inputs)
    return u >> 16;
}

// ---------------------------------------------------------------------------
// Four columns of a row per lane, for any dimension.  A lane group has as many lanes as the row has 16-byte
// chunks (of fp32), rounded up to a power of two; lane li covers columns [4 li, 4 li + 4), and where the
// dimension is no multiple of four the last lane's window is moved back to end with the row (it then shares
// columns with the lane before it: both hold, compute and store the same values, in lock step).  Rows,
// gradients and outputs need no alignment beyond their element's: gfx950's global accesses take any.
// Dimensions below four: one lane, element by element.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_b2 __attribute__((ext_vector_type(2), aligned(2)));

typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(4)));
template <int N>
__device__ __forceinline__ void load_u32(const uint32_t* p, uint32_t* v)
{
    static_assert(N == 2 || N == 4, "one access");
    if constexpr (N == 4) { const u32x4 x = *reinterpret_cast<const u32x4*>(p); v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; }
    else { const u32x2 x = *reinterpret_cast<const u32x2*>(p); v[0] = x.x; v[1] = x.y; }
}

__device__ __forceinline__ int lane_col(int li, int D) { return D >= 4 ? min(4 * li, D - 4) : 0; }

template <bool NARROW>
__device__ __forceinline__ void load_f32x4(const float* p, int D, float (&v)[4])
{
    if constexpr (!NARROW) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(p);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else {
        v[0] = p[0]; v[1] = v[2] = v[3] = 0.f;
        if (D > 1) { v[1] = p[1]; v[2] = p[D - 1]; }       // (of two columns the last one twice: a branch for the third would be waited for)
    }
}

template <bool NARROW>
__device__ __forceinline__ void store_f32x4(float* p, int D, const float (&v)[4])
{
    if constexpr (!NARROW) {
        f32x4 x;
        x.x = v[0]; x.y = v[1]; x.z = v[2]; x.w = v[3];
        *reinterpret_cast<f32x4*>(p) = x;
    } else {
        p[0] = v[0];
        if (D > 1) p[1] = v[1];
        if (D > 2) p[2] = v[2];
    }
}

// the same of a row of weights, fp32 or bf16
template <bool BF16, bool NARROW>
__device__ __forceinline__ void load_w4(const char* p, int D, float (&v)[4])
{
    if constexpr (!BF16) return load_f32x4<NARROW>(reinterpret_cast<const float*>(p), D, v);
    if constexpr (!NARROW) {
        const u32x2_b2 x = *reinterpret_cast<const u32x2_b2*>(p);
        v[0] = bf16_to_f32(x.x & 0xFFFFu); v[1] = bf16_to_f32(x.x >> 16);
        v[2] = bf16_to_f32(x.y & 0xFFFFu); v[3] = bf16_to_f32(x.y >> 16);
    } else {
        const uint16_t* h = reinterpret_cast<const uint16_t*>(p);
        v[0] = bf16_to_f32(h[0]); v[1] = v[2] = v[3] = 0.f;
        if (D > 1) { v[1] = bf16_to_f32(h[1]); v[2] = bf16_to_f32(h[D - 1]); }
    }
}

template <bool BF16, bool NARROW>
__device__ __forceinline__ void store_w4(char* p, int D, const float (&v)[4])
{
    if constexpr (!BF16) return store_f32x4<NARROW>(reinterpret_cast<float*>(p), D, v);
    if constexpr (!NARROW) {
        u32x2_b2 x;
        x.x = f32_to_bf16(v[0]) | (f32_to_bf16(v[1]) << 16);
        x.y = f32_to_bf16(v[2]) | (f32_to_bf16(v[3]) << 16);
        *reinterpret_cast<u32x2_b2*>(p) = x;
    } else {
        uint16_t* h = reinterpret_cast<uint16_t*>(p);
        h[0] = (uint16_t)f32_to_bf16(v[0]);
        if (D > 1) h[1] = (uint16_t)f32_to_bf16(v[1]);
        if (D > 2) h[2] = (uint16_t)f32_to_bf16(v[2]);
    }
}

// ---------------------------------------------------------------------------
// Where a row lives.  Plain tables: row r of the pack's table.  With HybridHash
// (Sec. III-D) the table passed to the kernel is the Cold-storage (every row) and
// the frequently queried rows live, and are updated, in a small Hot-storage:
// slot_of[r] >= 0 names the row's slot there.  slot_of == nullptr: no Hot-storage.
// ---------------------------------------------------------------------------
struct HotView {
    const int32_t* slot_of;
    void* W_hot;
    float* A_hot;
};

// the row's weights and its accumulators, from column d0 on
struct RowPtr { char* w; float* a; };
template <bool BF16, bool HYB>
__device__ __forceinline__ RowPtr row_ptr(void* W, float* A, const HotView& hv, uint32_t row, int D, int d0)
{
    char* w = as_global(static_cast<char*>(W));
    float* a = as_global(A);
    if (HYB) {
        const int s = as_global(hv.slot_of)[row];
        if (s >= 0) { w = as_global(static_cast<char*>(hv.W_hot)); a = as_global(hv.A_hot); row = (uint32_t)s; }
    }
    const size_t e = (size_t)((uint64_t)row * (uint32_t)D) + (size_t)d0;
    return RowPtr{w + (e << (BF16 ? 1 : 2)), a + e};
}
