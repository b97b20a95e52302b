// HIP kernels of libsmx for CDNA4 (gfx950, wave64).
//
// The method (paper, Section 2.1): one outer iteration of Algorithm 1 is a
// perturbation phase (trial steps z = x + beta v along v = -grad f/||grad f||,
// beta = gamma alpha^ell, accepted when f does not increase) followed by the
// feasibility step T = box projection of the relaxed simultaneous projection
// onto the bands lower <= Ax <= upper.  T streams A twice: pass 1 reads A row by
// row (r = A z and the band residual t), pass 2 reads the column-major copy
// (A^T of the weighted residual) and applies the box.
//
// Reductions that decide anything (proximity, objective values, gradient norms)
// run in float64 with a fixed order: every workgroup writes its partial sum and
// a one-workgroup kernel launched next sums the partials in workgroup order and
// updates the per-slice state (acceptance of trial steps included).  No kernel
// waits on, or signals, another workgroup of its own grid.
#include <algorithm>
#include <type_traits>
#include "smx_internal.h"
#include "phase_rounds.h"

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <math.h>

namespace smx {

// ---------------------------------------------------------------------------
// reductions
//
// A kernel that needs a grid-wide sum writes one partial per workgroup; a
// single-workgroup kernel launched after it sums the partials in workgroup
// order.  Kernel boundaries order the two, so no workgroup ever waits for or
// signals another one, and every sum is reproducible bit for bit.
// ---------------------------------------------------------------------------

// A float64 value moved across lanes by one DPP control (lanes with no source,
// and lanes outside row_mask, receive 0).
template <int CTRL, int ROW_MASK = 0xF>
__device__ inline double dpp_f64(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROW_MASK, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROW_MASK, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

__device__ inline double lane_value(double v, int lane)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the 64 lanes of a wave, returned in every lane.  Register-to-
// register DPP steps: prefix sums inside each row of 16 lanes (shifts by 1, 2,
// 4, 8), then row 0's total into row 1 and row 2's into row 3 (broadcast of
// lane 15), then lane 31's into rows 2 and 3; lane 63 ends with the total.
// The NV sums are independent, so their steps interleave.  Every lane of the
// wave must be active.
template <int NV>
__device__ inline void wave_sum(double (&v)[NV])
{
    constexpr int G = NV < 8 ? NV : 8; // values interleaved at a time (bounds the temporaries)
#pragma unroll
    for (int k0 = 0; k0 < NV; k0 += G) {
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] += dpp_f64<0x111>(v[k]);
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] += dpp_f64<0x112>(v[k]);
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] += dpp_f64<0x114>(v[k]);
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] += dpp_f64<0x118>(v[k]);
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] += dpp_f64<0x142, 0xA>(v[k]);
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] += dpp_f64<0x143, 0xC>(v[k]);
#pragma unroll
        for (int k = k0; k < k0 + G && k < NV; ++k) v[k] = lane_value(v[k], 63);
    }
}

// Sum of v over a workgroup of BS threads, valid in thread 0.  lds holds
// >= (BS/64)*NV doubles.
template <int NV, int BS = kBlock>
__device__ inline void block_sum(double (&v)[NV], double *lds)
{
    wave_sum<NV>(v);
    const int wid = threadIdx.x >> 6, wl = threadIdx.x & 63;
    if (wl == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) lds[wid * NV + k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double s = 0.0;
            for (int w = 0; w < BS / 64; ++w) s += lds[w * NV + k];
            v[k] = s;
        }
    }
    __syncthreads();
}

// Totals over `count` consecutive slots starting at `first` (each slot NV
// values), summed in slot order by one workgroup of BS threads; valid in
// thread 0.
template <int NV, int BS = kBlock>
__device__ inline void sum_slots(const double *__restrict__ partials, long long first, int count, double (&tot)[NV],
                                 double *lds)
{
#pragma unroll
    for (int k = 0; k < NV; ++k) tot[k] = 0.0;
    for (int b = threadIdx.x; b < count; b += BS) {
#pragma unroll
        for (int k = 0; k < NV; ++k) tot[k] += partials[(first + b) * NV + k];
    }
    block_sum<NV, BS>(tot, lds);
}

// ---------------------------------------------------------------------------
// value loads
// ---------------------------------------------------------------------------

template <typename VT, int VEC>
struct ValLoad;

template <>
struct ValLoad<float, 4> {
    static __device__ inline void load(const void *base, int p, float (&v)[4])
    {
        const float4 q = *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + p);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
};

template <>
struct ValLoad<float, 8> {
    static __device__ inline void load(const void *base, int p, float (&v)[8])
    {
        const float4 *q = reinterpret_cast<const float4 *>(static_cast<const float *>(base) + p);
        const float4 a = q[0], b = q[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
};

struct Bf16Tag {};
struct F16Tag {};

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ inline float f16_lo(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w & 0xffffu))); }
__device__ inline float f16_hi(uint32_t w) { return __half2float(__ushort_as_half((unsigned short)(w >> 16))); }

template <int VEC>
struct ValLoad16Base {
    static_assert(VEC == 4 || VEC == 8, "VEC");
};

template <>
struct ValLoad<Bf16Tag, 8> {
    static __device__ inline void load(const void *base, int p, float (&v)[8])
    {
        const uint4 q = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + p);
        v[0] = bf16_lo(q.x); v[1] = bf16_hi(q.x); v[2] = bf16_lo(q.y); v[3] = bf16_hi(q.y);
        v[4] = bf16_lo(q.z); v[5] = bf16_hi(q.z); v[6] = bf16_lo(q.w); v[7] = bf16_hi(q.w);
    }
};

template <>
struct ValLoad<Bf16Tag, 4> {
    static __device__ inline void load(const void *base, int p, float (&v)[4])
    {
        const uint2 q = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(base) + p);
        v[0] = bf16_lo(q.x); v[1] = bf16_hi(q.x); v[2] = bf16_lo(q.y); v[3] = bf16_hi(q.y);
    }
};

template <>
struct ValLoad<F16Tag, 8> {
    static __device__ inline void load(const void *base, int p, float (&v)[8])
    {
        const uint4 q = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + p);
        v[0] = f16_lo(q.x); v[1] = f16_hi(q.x); v[2] = f16_lo(q.y); v[3] = f16_hi(q.y);
        v[4] = f16_lo(q.z); v[5] = f16_hi(q.z); v[6] = f16_lo(q.w); v[7] = f16_hi(q.w);
    }
};

template <>
struct ValLoad<F16Tag, 4> {
    static __device__ inline void load(const void *base, int p, float (&v)[4])
    {
        const uint2 q = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(base) + p);
        v[0] = f16_lo(q.x); v[1] = f16_hi(q.x); v[2] = f16_lo(q.y); v[3] = f16_hi(q.y);
    }
};

template <int VEC>
__device__ inline void idx_load(const int32_t *base, int p, int (&c)[VEC])
{
    const int4 *q = reinterpret_cast<const int4 *>(base + p);
#pragma unroll
    for (int h = 0; h < VEC / 4; ++h) {
        const int4 a = q[h];
        c[4 * h + 0] = a.x; c[4 * h + 1] = a.y; c[4 * h + 2] = a.z; c[4 * h + 3] = a.w;
    }
}

struct Bf16PTag {};
struct F16PTag {};
struct F32U16Tag {}; // float32 values beside a uint16 index array

// VEC entries (values as float, indices) starting at p.
template <typename VT, int VEC>
struct Entries {
    static __device__ inline void load(const SpView &A, int p, float (&v)[VEC], int (&c)[VEC])
    {
        ValLoad<VT, VEC>::load(A.val, p, v);
        idx_load<VEC>(A.idx, p, c);
    }
};

template <int VEC, bool BF>
__device__ inline void packed_load(const SpView &A, int p, float (&v)[VEC], int (&c)[VEC])
{
    const uint4 *q = reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(A.val) + p);
#pragma unroll
    for (int h = 0; h < VEC / 4; ++h) {
        const uint4 a = q[h];
        const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[4 * h + k] = BF ? bf16_lo(w[k]) : f16_lo(w[k]);
            c[4 * h + k] = (int)(w[k] >> 16);
        }
    }
}

template <int VEC>
struct Entries<F32U16Tag, VEC> {
    static __device__ inline void load(const SpView &A, int p, float (&v)[VEC], int (&c)[VEC])
    {
        ValLoad<float, VEC>::load(A.val, p, v);
        const uint16_t *ib = reinterpret_cast<const uint16_t *>(A.idx) + p;
        if constexpr (VEC == 4) {
            const uint2 a = *reinterpret_cast<const uint2 *>(ib);
            c[0] = (int)(a.x & 0xFFFFu); c[1] = (int)(a.x >> 16); c[2] = (int)(a.y & 0xFFFFu); c[3] = (int)(a.y >> 16);
        } else {
            const uint4 a = *reinterpret_cast<const uint4 *>(ib);
            const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                c[2 * k] = (int)(w[k] & 0xFFFFu);
                c[2 * k + 1] = (int)(w[k] >> 16);
            }
        }
    }
};

template <int VEC>
struct Entries<Bf16PTag, VEC> {
    static __device__ inline void load(const SpView &A, int p, float (&v)[VEC], int (&c)[VEC])
    {
        packed_load<VEC, true>(A, p, v, c);
    }
};

template <int VEC>
struct Entries<F16PTag, VEC> {
    static __device__ inline void load(const SpView &A, int p, float (&v)[VEC], int (&c)[VEC])
    {
        packed_load<VEC, false>(A, p, v, c);
    }
};

// VEC stored entries at p as loaded, before any arithmetic on them (the
// bit patterns of the values, the index words), and their decoding.  Loops
// that keep several chunks in flight issue every chunk's loads first, each
// under its own predicate, and decode afterwards: a decode inside the
// predicated block would wait for that chunk's load before the next chunk's
// loads are issued, one memory round trip per chunk.  A chunk left
// unloaded decodes to value 0 at index 0.
template <typename VT, int VEC>
struct EntryRaw {
    static_assert(VEC == 4 || VEC == 8, "VEC");
    static constexpr int NV = std::is_same<VT, float>::value || std::is_same<VT, F32U16Tag>::value ? VEC
                              : (std::is_same<VT, Bf16PTag>::value || std::is_same<VT, F16PTag>::value) ? VEC
                                                                                                          : VEC / 2;
    static constexpr bool kIdx32 = !(std::is_same<VT, F32U16Tag>::value || std::is_same<VT, Bf16PTag>::value ||
                                     std::is_same<VT, F16PTag>::value);
    static constexpr int NI = kIdx32 ? VEC : (std::is_same<VT, F32U16Tag>::value ? VEC / 2 : 0);
    uint32_t vw[NV];
    uint32_t iw[NI > 0 ? NI : 1];

    __device__ inline void zero()
    {
#pragma unroll
        for (int k = 0; k < NV; ++k) vw[k] = 0u;
#pragma unroll
        for (int k = 0; k < (NI > 0 ? NI : 1); ++k) iw[k] = 0u;
    }
    __device__ inline void load(const SpView &A, int p)
    {
        if constexpr (std::is_same<VT, Bf16PTag>::value || std::is_same<VT, F16PTag>::value) {
            const uint4 *q = reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(A.val) + p);
#pragma unroll
            for (int h = 0; h < VEC / 4; ++h) {
                const uint4 a = q[h];
                vw[4 * h] = a.x; vw[4 * h + 1] = a.y; vw[4 * h + 2] = a.z; vw[4 * h + 3] = a.w;
            }
        } else {
            if constexpr (NV == VEC) { // 32-bit values
                const uint4 *q = reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(A.val) + p);
#pragma unroll
                for (int h = 0; h < VEC / 4; ++h) {
                    const uint4 a = q[h];
                    vw[4 * h] = a.x; vw[4 * h + 1] = a.y; vw[4 * h + 2] = a.z; vw[4 * h + 3] = a.w;
                }
            } else { // 16-bit values, two a word
                const uint16_t *b = static_cast<const uint16_t *>(A.val) + p;
                if constexpr (VEC == 8) {
                    const uint4 a = *reinterpret_cast<const uint4 *>(b);
                    vw[0] = a.x; vw[1] = a.y; vw[2] = a.z; vw[3] = a.w;
                } else {
                    const uint2 a = *reinterpret_cast<const uint2 *>(b);
                    vw[0] = a.x; vw[1] = a.y;
                }
            }
            if constexpr (kIdx32) {
                const uint4 *q = reinterpret_cast<const uint4 *>(A.idx + p);
#pragma unroll
                for (int h = 0; h < VEC / 4; ++h) {
                    const uint4 a = q[h];
                    iw[4 * h] = a.x; iw[4 * h + 1] = a.y; iw[4 * h + 2] = a.z; iw[4 * h + 3] = a.w;
                }
            } else { // 16-bit indices, two a word
                const uint16_t *ib = reinterpret_cast<const uint16_t *>(A.idx) + p;
                if constexpr (VEC == 8) {
                    const uint4 a = *reinterpret_cast<const uint4 *>(ib);
                    iw[0] = a.x; iw[1] = a.y; iw[2] = a.z; iw[3] = a.w;
                } else {
                    const uint2 a = *reinterpret_cast<const uint2 *>(ib);
                    iw[0] = a.x; iw[1] = a.y;
                }
            }
        }
    }
    __device__ inline void decode(float (&v)[VEC], int (&c)[VEC]) const
    {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if constexpr (std::is_same<VT, Bf16PTag>::value) {
                v[e] = bf16_lo(vw[e]);
                c[e] = (int)(vw[e] >> 16);
            } else if constexpr (std::is_same<VT, F16PTag>::value) {
                v[e] = f16_lo(vw[e]);
                c[e] = (int)(vw[e] >> 16);
            } else {
                if constexpr (NV == VEC) v[e] = __uint_as_float(vw[e]);
                else if constexpr (std::is_same<VT, Bf16Tag>::value) v[e] = (e & 1) ? bf16_hi(vw[e >> 1]) : bf16_lo(vw[e >> 1]);
                else v[e] = (e & 1) ? f16_hi(vw[e >> 1]) : f16_lo(vw[e >> 1]);
                if constexpr (kIdx32) c[e] = (int)iw[e];
                else c[e] = (int)((e & 1) ? (iw[e >> 1] >> 16) : (iw[e >> 1] & 0xFFFFu));
            }
        }
    }
};

// U chunks of VEC entries (chunk u at p + u * step, loaded where ok[u]):
// every load issued, then every chunk decoded.
template <typename VT, int VEC, int U>
__device__ inline void load_chunks(const SpView &A, int p, int step, const bool (&ok)[U], float (&v)[U][VEC],
                                   int (&c)[U][VEC])
{
    EntryRaw<VT, VEC> raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        raw[u].zero();
        if (ok[u]) raw[u].load(A, p + u * step);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u].decode(v[u], c[u]);
}

// Exchanges a chunk's entries so that place e holds entry e ^ (l mod VEC).
// Lanes l = 0, 1, ... hold consecutive chunks of a row, whose columns often
// follow one another: at one place of the unrolled loops the lanes' columns
// are then VEC apart, and their LDS words share banks (16 lanes of 8 entries:
// 64 clocks for a wave's ds_add_f64 against 16).  Exchanged, one place covers
// all residues.
template <int VEC>
__device__ inline void spread_entries(float (&v)[VEC], int (&c)[VEC], int l)
{
#pragma unroll
    for (int bit = 1; bit < VEC; bit <<= 1) {
        const bool sw = (l & bit) != 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            if ((e & bit) == 0) {
                const float va = v[e], vb = v[e | bit];
                const int ca = c[e], cb = c[e | bit];
                v[e] = sw ? vb : va;
                v[e | bit] = sw ? va : vb;
                c[e] = sw ? cb : ca;
                c[e | bit] = sw ? ca : cb;
            }
    }
}

// One entry at p: its value as float and its index.
template <typename VT>
__device__ inline void entry1(const SpView &A, int p, float &v, int &c);
template <>
__device__ inline void entry1<float>(const SpView &A, int p, float &v, int &c)
{
    v = static_cast<const float *>(A.val)[p];
    c = A.idx[p];
}
template <>
__device__ inline void entry1<Bf16Tag>(const SpView &A, int p, float &v, int &c)
{
    v = bf16_lo(static_cast<const uint16_t *>(A.val)[p]);
    c = A.idx[p];
}
template <>
__device__ inline void entry1<F16Tag>(const SpView &A, int p, float &v, int &c)
{
    v = f16_lo(static_cast<const uint16_t *>(A.val)[p]);
    c = A.idx[p];
}
template <>
__device__ inline void entry1<Bf16PTag>(const SpView &A, int p, float &v, int &c)
{
    const uint32_t w = static_cast<const uint32_t *>(A.val)[p];
    v = bf16_lo(w);
    c = (int)(w >> 16);
}
template <>
__device__ inline void entry1<F16PTag>(const SpView &A, int p, float &v, int &c)
{
    const uint32_t w = static_cast<const uint32_t *>(A.val)[p];
    v = f16_lo(w);
    c = (int)(w >> 16);
}
template <>
__device__ inline void entry1<F32U16Tag>(const SpView &A, int p, float &v, int &c)
{
    v = static_cast<const float *>(A.val)[p];
    c = reinterpret_cast<const uint16_t *>(A.idx)[p];
}

// Partial dot product of one row with a vector, lanes interleaved: lane l of
// an LPR-lane group takes entries beg + l, beg + l + LPR, ...  Neighbouring
// lanes read neighbouring entries (one coalesced load per instruction), and
// their gathers land on neighbouring entries of the row, which for a ray are
// often neighbouring pixels in one cache line.  Eight entries per lane in
// flight; entries past the row's end are skipped (LPR may exceed the row
// alignment).
template <int LPR, typename VT>
__device__ inline double row_dot_interleaved(const SpView &A, int beg, int end, int lane, const float *__restrict__ x)
{
    constexpr int U = 8;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int p = beg + lane;
    for (; p + (U - 1) * LPR < end; p += U * LPR) {
        float v[U];
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) entry1<VT>(A, p + u * LPR, v[u], c[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u & 3] = fma((double)v[u], (double)x[c[u]], acc[u & 3]);
    }
    for (; p < end; p += LPR) {
        float v0;
        int c0;
        entry1<VT>(A, p, v0, c0);
        acc[0] = fma((double)v0, (double)x[c0], acc[0]);
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Partial dot product of one row with a vector, by lane `lane` of an LPR-lane
// group.  [beg, end) is row-aligned, so every vector load is aligned and no
// entry needs a mask (padding entries are zeros with valid indices).  Products
// of two float32 numbers are exact in float64, so accumulating in float64
// leaves only the rounding of the sums; the pass is bound by memory traffic,
// not by the float64 rate.
template <int LPR, int VEC, typename VT>
__device__ inline double row_dot_chunked(const SpView &A, int beg, int end, int lane, const float *__restrict__ x)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int p = beg + lane * VEC;
    constexpr int STEP = LPR * VEC;
    // four independent loads in flight per lane; the row's last chunks (fewer
    // than four) are issued together as well, each under its own predicate,
    // so a row costs one load-then-gather round trip per four chunks
    for (; p < end; p += 4 * STEP) {
        float v[4][VEC];
        int c[4][VEC];
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ok[u] = p + u * STEP < end;
        load_chunks<VT, VEC, 4>(A, p, STEP, ok, v, c);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (ok[u]) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[u] = fma((double)v[u][e], (double)x[c[u][e]], acc[u]);
            }
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// VEC 1: interleaved lanes; otherwise chunks of VEC entries per lane.
template <int LPR, int VEC, typename VT>
__device__ inline double row_dot(const SpView &A, int beg, int end, int lane, const float *__restrict__ x)
{
    if constexpr (VEC == 1) return row_dot_interleaved<LPR, VT>(A, beg, end, lane, x);
    else return row_dot_chunked<LPR, VEC, VT>(A, beg, end, lane, x);
}

template <int LPR>
__device__ inline double group_sum(double v)
{
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, LPR);
    return v;
}

// ---------------------------------------------------------------------------
// pass 1: r = A z, t = clip(r, lower, upper) - r, c = S t, and one partial of
// the proximity 1/2 sum D t^2 per workgroup (or, in quadratic-form mode, of
// sum S r^2)
// ---------------------------------------------------------------------------

// Pass-1 epilogue of row `row` (slice s of B) from r = <a_i, v>: returns the
// row's partial term and stores c_i (not in quadratic-form mode).  With S = D
// this is exactly c_i = D_i t_i and the term D_i t_i^2.  A dose-volume row
// only keeps r: its bands are set after the pass, and the dose-volume kernels
// write its c_i and its proximity term.
__device__ inline double epi1(const RowW &w, double r, float lo, float up, float d, float sw, float *c,
                              long long row, int s, int B)
{
    if (w.qform) return (double)sw * r * r;
    if (w.dose && row >= w.dose_lo && row < w.dose_hi) {
        w.dose[(row - w.dose_lo) * B + s] = r;
        return 0.0;
    }
    const double t = fmin(fmax(r, (double)lo), (double)up) - r;
    const double dt = (double)d * t;
    *c = (float)((double)sw * t);
    return dt * t;
}

template <int LPR, int VEC, typename VT>
__global__ __launch_bounds__(kBlock) void k_pass1(SpView A, const float *__restrict__ x,
                                                  const float *__restrict__ lower, const float *__restrict__ upper,
                                                  RowW w, float *__restrict__ c,
                                                  const SliceState *__restrict__ st, int query,
                                                  double *__restrict__ partials)
{
    __shared__ double lds[4];
    constexpr int RPB = kBlock / LPR;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const bool live = query ? true : st[0].live != 0;
    double pacc[1] = {0.0};
    if (live) {
        const long long stride = (long long)gridDim.x * RPB;
        long long row = (long long)blockIdx.x * RPB + grp;
        int beg = 0, end = 0;
        if (row < A.rows) {
            beg = A.ptr[row];
            end = A.ptr[row + 1];
        }
        for (; row < A.rows; row += stride) {
            int nbeg = 0, nend = 0; // the next row's offsets, in flight meanwhile
            if (row + stride < A.rows) {
                nbeg = A.ptr[row + stride];
                nend = A.ptr[row + stride + 1];
            }
            // epilogue operands, fetched while the row streams (every lane of the
            // group reads the same words: no predicated block whose conversions
            // would wait for them before the row's loads are issued)
            const float lo = lower[row], up = upper[row], d = w.D[row], sw = w.S[row];
            const double r = group_sum<LPR>(row_dot<LPR, VEC, VT>(A, beg, end, lane, x)) * (double)A.vscale_inv;
            if (lane == 0) pacc[0] += epi1(w, r, lo, up, d, sw, c + row, row, 0, 1);
            beg = nbeg;
            end = nend;
        }
    }
    block_sum<1>(pacc, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
}

// Copies v[0, P) into LDS (dst, 16-byte aligned) with BS threads: float4
// loads, four in flight per thread (every load in bounds: past the end the
// last float4 is read again, and not stored), then the last P mod 4 values.
template <int BS>
__device__ inline void stage_vector(float4 *dst, const float *__restrict__ v, int P)
{
    const int q4 = P >> 2;
    const float4 *v4 = reinterpret_cast<const float4 *>(v);
    for (int e0 = threadIdx.x; e0 < q4; e0 += 4 * BS) {
        float4 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = v4[min(e0 + u * BS, q4 - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (e0 + u * BS < q4) dst[e0 + u * BS] = t[u];
    }
    if (threadIdx.x < (P & 3)) reinterpret_cast<float *>(dst)[4 * q4 + threadIdx.x] = v[4 * q4 + threadIdx.x];
}

// One unknown of the linear objective's trial point z = x + s v, v = -c/||c||
// (inv_gn = 1/||c||): the one expression every kernel forming z uses, so the
// pass that stages z and the apply kernel that forms it again agree bit for bit.
__device__ inline float linear_step_point(float xj, float cj, double s_acc, double inv_gn)
{
    return (float)((double)xj + s_acc * (-(double)cj * inv_gn));
}

// stage_vector of z = x + s v for the linear objective (x and c both read as
// float4, four loads of each in flight per thread).
template <int BS>
__device__ inline void stage_linear_point(float4 *dst, const float *__restrict__ x, const float *__restrict__ c, int P,
                                          double s_acc, double inv_gn)
{
    const int q4 = P >> 2;
    const float4 *x4 = reinterpret_cast<const float4 *>(x);
    const float4 *c4 = reinterpret_cast<const float4 *>(c);
    for (int e0 = threadIdx.x; e0 < q4; e0 += 4 * BS) {
        float4 tx[4], tc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            tx[u] = x4[min(e0 + u * BS, q4 - 1)];
            tc[u] = c4[min(e0 + u * BS, q4 - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (e0 + u * BS < q4)
                dst[e0 + u * BS] = make_float4(linear_step_point(tx[u].x, tc[u].x, s_acc, inv_gn),
                                               linear_step_point(tx[u].y, tc[u].y, s_acc, inv_gn),
                                               linear_step_point(tx[u].z, tc[u].z, s_acc, inv_gn),
                                               linear_step_point(tx[u].w, tc[u].w, s_acc, inv_gn));
    }
    if (threadIdx.x < (P & 3)) {
        const int j = 4 * q4 + threadIdx.x;
        reinterpret_cast<float *>(dst)[j] = linear_step_point(x[j], c[j], s_acc, inv_gn);
    }
}

// Row dot product whose gathers read the vector's first P entries from an
// LDS copy (xl) and the rest from memory; otherwise row_dot_chunked.
template <int LPR, int VEC, typename VT>
__device__ inline double row_dot_split(const SpView &A, int beg, int end, int lane, const float *__restrict__ x,
                                       const float *xl, int P)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int p = beg + lane * VEC;
    constexpr int STEP = LPR * VEC;
    for (; p < end; p += 4 * STEP) {
        float v[4][VEC];
        int c[4][VEC];
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ok[u] = p + u * STEP < end;
        load_chunks<VT, VEC, 4>(A, p, STEP, ok, v, c);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (ok[u]) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int ci = c[u][e];
                    float xv;
                    if (ci < P) xv = xl[ci];
                    else xv = x[ci];
                    acc[u] = fma((double)v[u][e], (double)xv, acc[u]);
                }
            }
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Pass 1 with the gathered vector partly in LDS.  A gather through the
// vector memory path costs about one address per CU per clock, whatever its
// locality; an LDS read serves many lanes per clock.  So each workgroup (one
// per CU, 1024 threads) first copies x[0, P) into LDS, P = min(n, 40,448),
// then runs the rows as k_pass1 does, gathering x_j from LDS when j < P.
template <int LPR, int VEC, typename VT>
__global__ __launch_bounds__(kLdsPassBlock) void k_pass1_lds(SpView A, const float *__restrict__ x, int P,
                                                              const float *__restrict__ lower,
                                                              const float *__restrict__ upper, RowW w,
                                                              float *__restrict__ c,
                                                              const SliceState *__restrict__ st, int query,
                                                              double *__restrict__ partials)
{
    extern __shared__ float4 xl4[];
    float *xl = reinterpret_cast<float *>(xl4);
    __shared__ double lds[kLdsPassBlock / 64];
    constexpr int RPB = kLdsPassBlock / LPR;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const bool live = query ? true : st[0].live != 0; // the same in every thread
    double pacc[1] = {0.0};
    if (live) {
        stage_vector<kLdsPassBlock>(xl4, x, P);
        __syncthreads();
        const long long stride = (long long)gridDim.x * RPB;
        long long row = (long long)blockIdx.x * RPB + grp;
        int beg = 0, end = 0;
        if (row < A.rows) {
            beg = A.ptr[row];
            end = A.ptr[row + 1];
        }
        for (; row < A.rows; row += stride) {
            int nbeg = 0, nend = 0; // the next row's offsets, in flight meanwhile
            if (row + stride < A.rows) {
                nbeg = A.ptr[row + stride];
                nend = A.ptr[row + stride + 1];
            }
            const float lo = lower[row], up = upper[row], d = w.D[row], sw = w.S[row]; // read by every lane
            const double r =
                group_sum<LPR>(row_dot_split<LPR, VEC, VT>(A, beg, end, lane, x, xl, P)) * (double)A.vscale_inv;
            if (lane == 0) pacc[0] += epi1(w, r, lo, up, d, sw, c + row, row, 0, 1);
            beg = nbeg;
            end = nend;
        }
    }
    block_sum<1, kLdsPassBlock>(pacc, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
}

// ---------------------------------------------------------------------------
// Streaming pass kernels.  A workgroup takes one row block (at most
// kStreamEntries entries): every lane issues all of its value/index loads and
// gathers at once, the exact float64 products go to LDS, and each row is then
// summed from LDS by a group of G lanes (G the largest power of two with
// G * rows <= kBlock).  A row longer than a block is summed by the whole
// workgroup.  Rows of one block are consecutive, so the loads are one
// contiguous stream per workgroup.
// ---------------------------------------------------------------------------

struct RowSplit {
    int G, rl, lane;
};

__device__ inline RowSplit split_rows(int nr)
{
    int G = 64;
    while (G > 1 && G * nr > kBlock) G >>= 1;
    RowSplit r;
    r.G = G;
    r.rl = threadIdx.x / G;
    r.lane = threadIdx.x & (G - 1);
    return r;
}

// Sums of the VEC-entry chunks of [e0, e1) with v: chunk j (entries e0 + j*VEC
// ..) into prod[j].  Rows start at multiples of kRowAlign (a multiple of VEC),
// so no chunk straddles two rows; each product of two float32 numbers is exact
// in float64.
template <int VEC, typename VT>
__device__ inline void stream_chunks(const SpView &A, int e0, int e1, const float *__restrict__ v, double *prod)
{
    constexpr int PER = kStreamEntries / (kBlock * VEC);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int j = k * kBlock + threadIdx.x;
        const int q = j * VEC;
        if (e0 + q < e1) {
            float val[VEC];
            int id[VEC];
            Entries<VT, VEC>::load(A, e0 + q, val, id);
            double acc = 0.0;
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc = fma((double)val[e], (double)v[id[e]], acc);
            prod[j] = acc;
        }
    }
}

// Sum over lanes of the G-lane group (every thread of the workgroup calls it).
__device__ inline double group_sum_rt(double s, int G)
{
    for (int off = G >> 1; off > 0; off >>= 1) s += __shfl_xor(s, off, G);
    return s;
}

// Whole-workgroup sum of one long row; valid in thread 0.
template <int VEC, typename VT>
__device__ inline double long_row_sum(const SpView &A, int e0, int e1, const float *__restrict__ v, double *lds)
{
    double acc = 0.0;
    for (int p = e0 + threadIdx.x * VEC; p < e1; p += kBlock * VEC) {
        float val[VEC];
        int id[VEC];
        Entries<VT, VEC>::load(A, p, val, id);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc = fma((double)val[e], (double)v[id[e]], acc);
    }
    double t[1] = {acc};
    block_sum<1>(t, lds);
    return t[0];
}

template <int VEC, typename VT>
__global__ __launch_bounds__(kBlock) void k_pass1_stream(SpView A, RowBlocks RB, const float *__restrict__ x,
                                                         const float *__restrict__ lower,
                                                         const float *__restrict__ upper,
                                                         RowW w, float *__restrict__ c,
                                                         const SliceState *__restrict__ st, int query,
                                                         double *__restrict__ partials)
{
    __shared__ double prod[kStreamEntries / VEC];
    __shared__ int rp[kBlock + 1];
    __shared__ double lds[4];
    const bool live = query ? true : st[0].live != 0;
    double pacc[1] = {0.0};
    if (live) {
        for (int b = blockIdx.x; b < RB.nblk; b += gridDim.x) {
            const int r0 = RB.rb[b], r1 = RB.rb[b + 1];
            const int e0 = A.ptr[r0], e1 = A.ptr[r1];
            if (e1 - e0 > kStreamEntries) {
                const double sum = long_row_sum<VEC, VT>(A, e0, e1, x, lds);
                if (threadIdx.x == 0)
                    pacc[0] += epi1(w, sum * (double)A.vscale_inv, lower[r0], upper[r0], w.D[r0], w.S[r0], c + r0,
                                    r0, 0, 1);
                continue;
            }
            const int nr = r1 - r0;
            const RowSplit rs = split_rows(nr);
            const bool owner = rs.rl < nr && rs.lane == 0;
            float lo = 0.f, up = 0.f, d = 0.f, sw = 0.f;
            if (owner) { // epilogue operands, fetched while the products stream
                lo = lower[r0 + rs.rl];
                up = upper[r0 + rs.rl];
                d = w.D[r0 + rs.rl];
                sw = w.S[r0 + rs.rl];
            }
            for (int i = threadIdx.x; i <= nr; i += kBlock) rp[i] = (A.ptr[r0 + i] - e0) / VEC;
            stream_chunks<VEC, VT>(A, e0, e1, x, prod);
            __syncthreads();
            double s = 0.0;
            if (rs.rl < nr)
                for (int q = rp[rs.rl] + rs.lane; q < rp[rs.rl + 1]; q += rs.G) s += prod[q];
            s = group_sum_rt(s, rs.G);
            if (owner) pacc[0] += epi1(w, s * (double)A.vscale_inv, lo, up, d, sw, c + r0 + rs.rl, r0 + rs.rl, 0, 1);
            __syncthreads();
        }
    }
    block_sum<1>(pacc, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
}

__device__ inline double nan64() { return __longlong_as_double(0x7ff8000000000000LL); }

// ---------------------------------------------------------------------------
// State buffers.  Every kernel reads the per-slice states from st_in; kernels
// that advance the state have exactly one writer per slice (thread 0 of the
// slice's workgroup 0), which writes the whole new state to the other buffer
// st_out.  The host alternates the two buffers launch by launch, so a kernel
// never reads a state another workgroup of the same grid is writing.
// ---------------------------------------------------------------------------

// Whether a slice runs its next iteration.
__device__ inline int slice_runs(const SliceState &S)
{
    return (S.enabled && S.k < S.k_end && S.stop_reason == STOP_NONE) ? 1 : 0;
}

// Stopping rules after a feasibility step that recorded proximity `prox`
// (Section 2.2.1: P <= P*, or |P^{k+1} - P^k| / max{1, P^k} < Delta P* for N
// consecutive iterations, or N_max iterations).  A superiorized run (a phase
// ran, so f_start = f(x^k) is set) only notes whether a proximity rule held;
// its objective condition is checked when the next phase opens.  The variance
// rule follows in k_stop_var.
__device__ inline void stop_rules_after_step(SliceState &S, double prox)
{
    if (!isnan(S.p_last)) {
        const double dp = fabs(prox - S.p_last) / fmax(1.0, S.p_last);
        S.dp_run = dp < S.stop_dprox ? S.dp_run + 1 : 0;
    }
    S.p_last = prox;
    const bool by_prox = prox <= S.stop_prox, by_dprox = S.dp_run >= S.stop_n;
    if (!isnan(S.f_start)) {
        S.feas_ok = (by_prox || by_dprox) ? 1 : 0;
        S.f_last = S.f_start;
    } else if (by_prox) {
        S.stop_reason = STOP_PROX;
    } else if (by_dprox) {
        S.stop_reason = STOP_DPROX;
    }
    if (S.stop_reason == STOP_NONE && S.stop_max > 0 && S.k >= S.stop_max) S.stop_reason = STOP_MAXIT;
}

// End of an outer iteration for slice s, by one thread: proximity (prox2 is
// pass 1's sum, twice of it), the history record, k + 1, and whether the next
// iteration runs.
__device__ inline void finish_slice(const SliceState *__restrict__ st_in, SliceState *__restrict__ st_out, int s,
                                    int B, double prox2, const Hist &h)
{
    SliceState S = st_in[s];
    S.ran = S.live;
    if (S.live) {
        const double prox = 0.5 * prox2;
        S.prox = prox;
        if (!isfinite(prox)) S.nonfinite = 1;
        if (S.k < h.cap) {
            const long long r = S.k * B + s;
            h.prox[r] = prox;
            h.f_start[r] = S.f_start;
            h.f_end[r] = S.f_cur;
            h.trials[r] = S.trials_it;
            h.accepts[r] = S.accepts_it;
        }
        S.k += 1;
        if (S.stop_on) stop_rules_after_step(S, prox);
    }
    if (!isnan(S.f_cur)) S.f_ref = S.f_cur; // where this iteration's phase ended
    S.f_start = S.f_cur = nan64();
    S.trials_it = 0;
    S.accepts_it = 0;
    S.phase = 0;
    S.live = slice_runs(S);
    st_out[s] = S;
}

// End of an outer iteration from pass 1's partials, called by every thread of
// one workgroup (BS threads; lds holds BS/64 doubles): the whole workgroup for
// one slice, a wave a slice for several.  It is a chain of loads, sums and
// stores that needs nothing of the column step, so the launch has a workgroup
// for it alone, the last one, beside those that take columns.  At the end of
// workgroup 0, and slice after slice, as it was before, it was the tail of the
// launch: 128 x 128 CT, 8 slices, pass 2 25.4 us, now 13.4; 64 x 64, one slice,
// 25.3 us an iteration, now 24.2.
template <int BS = kBlock>
__device__ inline void finish_iteration(const SliceState *__restrict__ st_in, SliceState *__restrict__ st_out, int B,
                                        const double *__restrict__ part1, int nparts, const Hist &h, double *lds)
{
    if (B == 1) {
        double tot[1];
        sum_slots<1, BS>(part1, 0, nparts, tot, lds);
        if (threadIdx.x == 0) finish_slice(st_in, st_out, 0, 1, tot[0], h);
        return;
    }
    const int lane = threadIdx.x & 63;
    for (int s = threadIdx.x >> 6; s < B; s += BS / 64) {
        const double *p = part1 + (long long)s * nparts;
        double tot[1] = {0.0};
#pragma unroll 8
        for (int b = lane; b < nparts; b += 64) tot[0] += p[b];
        wave_sum<1>(tot);
        if (lane == 0) finish_slice(st_in, st_out, s, B, tot[0], h);
    }
}

// Workgroups of a launch that take columns: all but the last, which closes
// the outer iteration, or all of them where a later launch closes it.
__device__ inline int column_groups(const ColStep &cs) { return (int)gridDim.x - (cs.defer ? 0 : 1); }
static inline unsigned column_grid(int groups, const ColStep &cs) { return (unsigned)groups + (cs.defer ? 0u : 1u); }

// ---------------------------------------------------------------------------
// pass 2: y = A^T c, x = clip(z + lambda y, lo, hi) (DROP: lambda Z_j y);
// one more workgroup closes the outer iteration.  For the extrapolated steps
// (deferred mode) y itself is kept, with per-workgroup partials of ||y||^2,
// and k_step_apply updates x and closes the iteration.
// ---------------------------------------------------------------------------

// Pass-2 epilogue of one column (x and ybuf index e); returns y^2 in deferred
// mode, else 0.
__device__ inline double epi2(const ColStep &cs, long long col, long long e, double y, float xo, float l, float u,
                              float *__restrict__ x)
{
    if (cs.defer) {
        cs.ybuf[e] = y;
        if (cs.ybuf32) cs.ybuf32[e] = (float)y;
        return y * y;
    }
    const double yy = cs.zcol ? y * (double)cs.zcol[col] : y;
    const double z = fma((double)cs.lambda, yy, (double)xo);
    x[e] = (float)fmin(fmax(z, (double)l), (double)u);
    return 0.0;
}

// End of a workgroup's columns (BS threads): the ||y||^2 partials in deferred
// mode.
template <int BS = kBlock>
__device__ inline void end_columns(const ColStep &cs, double yacc, double *lds)
{
    if (!cs.defer) return;
    double v[1] = {yacc};
    block_sum<1, BS>(v, lds);
    if (threadIdx.x == 0) cs.ypart[blockIdx.x] = v[0];
}

template <int LPR, int VEC, typename VT>
__global__ __launch_bounds__(kBlock) void k_pass2(SpView At, const float *__restrict__ c, float *__restrict__ x,
                                                  ColStep cs, const SliceState *__restrict__ st_in,
                                                  SliceState *__restrict__ st_out, const double *__restrict__ part1,
                                                  int nparts1, Hist h)
{
    __shared__ double lds[4];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, 1, part1, nparts1, h, lds);
        return;
    }
    constexpr int RPB = kBlock / LPR;
    double yacc = 0.0;
    if (st_in[0].live) {
        const int lane = threadIdx.x & (LPR - 1);
        const int grp = threadIdx.x / LPR;
        const long long stride = (long long)groups * RPB;
        for (long long col = (long long)blockIdx.x * RPB + grp; col < At.rows; col += stride) {
            const int beg = At.ptr[col], end = At.ptr[col + 1];
            float xo = 0.f, l = 0.f, u = 0.f;
            if (lane == 0 && !cs.defer) { // epilogue operands, fetched while the column streams
                xo = x[col];
                l = cs.lo[col];
                u = cs.hi[col];
            }
            const double y = group_sum<LPR>(row_dot<LPR, VEC, VT>(At, beg, end, lane, c)) * (double)At.vscale_inv;
            if (lane == 0) yacc += epi2(cs, col, col, y, xo, l, u, x);
        }
    }
    end_columns(cs, yacc, lds);
}

// Pass 2 with the gathered residual partly in LDS, as k_pass1_lds: one
// workgroup per CU copies c[0, P) into LDS, P = min(m, 40,448), then sums
// each column as k_pass2 does, reading c_i from LDS when i < P.
template <int LPR, int VEC, typename VT>
__global__ __launch_bounds__(kLdsPassBlock) void k_pass2_lds(SpView At, const float *__restrict__ c, int P,
                                                             float *__restrict__ x, ColStep cs,
                                                             const SliceState *__restrict__ st_in,
                                                             SliceState *__restrict__ st_out,
                                                             const double *__restrict__ part1, int nparts1, Hist h)
{
    extern __shared__ float4 cl4[];
    float *cl = reinterpret_cast<float *>(cl4);
    __shared__ double lds[kLdsPassBlock / 64];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration<kLdsPassBlock>(st_in, st_out, 1, part1, nparts1, h, lds);
        return;
    }
    constexpr int RPB = kLdsPassBlock / LPR;
    double yacc = 0.0;
    if (st_in[0].live) { // the same in every thread
        stage_vector<kLdsPassBlock>(cl4, c, P);
        __syncthreads();
        const int lane = threadIdx.x & (LPR - 1);
        const int grp = threadIdx.x / LPR;
        const long long stride = (long long)groups * RPB;
        long long col = (long long)blockIdx.x * RPB + grp;
        int beg = 0, end = 0;
        if (col < At.rows) {
            beg = At.ptr[col];
            end = At.ptr[col + 1];
        }
        for (; col < At.rows; col += stride) {
            int nbeg = 0, nend = 0; // the next column's offsets, in flight meanwhile
            if (col + stride < At.rows) {
                nbeg = At.ptr[col + stride];
                nend = At.ptr[col + stride + 1];
            }
            float xo = 0.f, l = 0.f, u = 0.f;
            if (lane == 0 && !cs.defer) {
                xo = x[col];
                l = cs.lo[col];
                u = cs.hi[col];
            }
            const double y =
                group_sum<LPR>(row_dot_split<LPR, VEC, VT>(At, beg, end, lane, c, cl, P)) * (double)At.vscale_inv;
            if (lane == 0) yacc += epi2(cs, col, col, y, xo, l, u, x);
            beg = nbeg;
            end = nend;
        }
    }
    end_columns<kLdsPassBlock>(cs, yacc, lds);
}

// Sum of one column segment [beg, end) of the column copy whose rows all lie
// in the panel staged in LDS (cl[row - base]).  Segments start anywhere in a
// column, so the chunks start at the aligned position before beg and the
// entries outside [beg, end) are masked (they are in bounds: a column is
// padded to a multiple of kRowAlign entries).
template <int LPR, int VEC, typename VT>
__device__ inline double seg_dot_lds(const SpView &A, int beg, int end, int lane, const float *cl, int base)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    constexpr int STEP = LPR * VEC;
    for (int p = (beg / VEC) * VEC + lane * VEC; p < end; p += 4 * STEP) {
        float v[4][VEC];
        int c[4][VEC];
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ok[u] = p + u * STEP < end;
        load_chunks<VT, VEC, 4>(A, p, STEP, ok, v, c);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (ok[u]) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int q = p + u * STEP + e;
                    if (q >= beg && q < end) acc[u] = fma((double)v[u][e], (double)cl[c[u][e] - base], acc[u]);
                }
            }
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Pass 2 for operators with many rows, over the column copy in row panels of
// P rows: a work item is (panel p, a range of columns); the workgroup stages
// c's rows of panel p in LDS, then each column's segment in that panel
// (entries pp[p*n + j] .. pp[(p+1)*n + j]) is summed from LDS into
// ypanel[p*n + j].  k_pass2_panel_sum adds a column's panel sums in panel
// order and applies the column step.
template <int LPR, int VEC, typename VT>
__global__ __launch_bounds__(kLdsPassBlock) void k_pass2_panel(SpView At, const int32_t *__restrict__ pp, int np,
                                                               int P, long long m, int cpt, int chunks, int local,
                                                               const float *__restrict__ c,
                                                               double *__restrict__ ypanel,
                                                               const SliceState *__restrict__ st_in)
{
    extern __shared__ float4 cl4[];
    const float *cl = reinterpret_cast<const float *>(cl4);
    constexpr int GROUPS = kLdsPassBlock / LPR;
    if (!st_in[0].live) return; // the same in every workgroup: k_pass2_panel_sum skips the slice too
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int n = (int)At.rows;
    for (int t = blockIdx.x; t < np * chunks; t += gridDim.x) {
        const int p = t / chunks, q = t % chunks;
        const long long base = (long long)p * P;
        const int len = (int)min((long long)P, m - base);
        __syncthreads(); // the previous item's readers are done with the LDS copy
        stage_vector<kLdsPassBlock>(cl4, c + base, len);
        __syncthreads();
        const int j1 = min(n, (q + 1) * cpt);
        for (int j = q * cpt + grp; j < j1; j += GROUPS) {
            const int beg = pp[(long long)p * n + j], end = pp[(long long)(p + 1) * n + j];
            const double y =
                group_sum<LPR>(seg_dot_lds<LPR, VEC, VT>(At, beg, end, lane, cl, local ? 0 : (int)base));
            if (lane == 0) ypanel[(long long)p * n + j] = y;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_pass2_panel_sum(int np, int n, const double *__restrict__ ypanel,
                                                            float vscale_inv, float *__restrict__ x, ColStep cs,
                                                            const SliceState *__restrict__ st_in,
                                                            SliceState *__restrict__ st_out,
                                                            const double *__restrict__ part1, int nparts1, Hist h)
{
    __shared__ double lds[4];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, 1, part1, nparts1, h, lds);
        return;
    }
    double yacc = 0.0;
    if (st_in[0].live) {
        for (int j = blockIdx.x * kBlock + threadIdx.x; j < n; j += groups * kBlock) {
            double y = 0.0;
            for (int p = 0; p < np; ++p) y += ypanel[(long long)p * n + j];
            float xo = 0.f;
            if (!cs.defer) xo = x[j];
            yacc += epi2(cs, j, j, y * (double)vscale_inv, xo, cs.lo[j], cs.hi[j], x);
        }
    }
    end_columns(cs, yacc, lds);
}

template <int VEC, typename VT>
__global__ __launch_bounds__(kBlock) void k_pass2_stream(SpView At, RowBlocks RB, const float *__restrict__ c,
                                                         float *__restrict__ x, ColStep cs,
                                                         const SliceState *__restrict__ st_in,
                                                         SliceState *__restrict__ st_out,
                                                         const double *__restrict__ part1, int nparts1, Hist h)
{
    __shared__ double prod[kStreamEntries / VEC];
    __shared__ int rp[kBlock + 1];
    __shared__ double lds[4];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, 1, part1, nparts1, h, lds);
        return;
    }
    double yacc = 0.0;
    if (st_in[0].live) {
        for (int b = blockIdx.x; b < RB.nblk; b += groups) {
            const int r0 = RB.rb[b], r1 = RB.rb[b + 1];
            const int e0 = At.ptr[r0], e1 = At.ptr[r1];
            if (e1 - e0 > kStreamEntries) {
                const double sum = long_row_sum<VEC, VT>(At, e0, e1, c, lds);
                if (threadIdx.x == 0)
                    yacc += epi2(cs, r0, r0, sum * (double)At.vscale_inv, x[r0], cs.lo[r0], cs.hi[r0], x);
                continue;
            }
            const int nr = r1 - r0;
            const RowSplit rs = split_rows(nr);
            const bool owner = rs.rl < nr && rs.lane == 0;
            float xo = 0.f, l = 0.f, u = 0.f;
            if (owner) {
                xo = x[r0 + rs.rl];
                l = cs.lo[r0 + rs.rl];
                u = cs.hi[r0 + rs.rl];
            }
            for (int i = threadIdx.x; i <= nr; i += kBlock) rp[i] = (At.ptr[r0 + i] - e0) / VEC;
            stream_chunks<VEC, VT>(At, e0, e1, c, prod);
            __syncthreads();
            double s = 0.0;
            if (rs.rl < nr)
                for (int q = rp[rs.rl] + rs.lane; q < rp[rs.rl + 1]; q += rs.G) s += prod[q];
            s = group_sum_rt(s, rs.G);
            if (owner) yacc += epi2(cs, r0 + rs.rl, r0 + rs.rl, s * (double)At.vscale_inv, xo, l, u, x);
            __syncthreads();
        }
    }
    end_columns(cs, yacc, lds);
}

// Copies a tile's nr rows of c (B floats each, slice-interleaved as in
// memory) into LDS.  Rows are moved as float4 where B allows, and each thread
// issues U loads before its first LDS store, so that a tile's staging costs a
// few memory round trips rather than one per row a thread copies.
template <int B>
__device__ inline void stage_rows(float *__restrict__ cl, const float *__restrict__ c, const int *__restrict__ rlist,
                                  int nr)
{
    constexpr bool V4 = B % 4 == 0;
    constexpr int PER = V4 ? B / 4 : B; // loads per row
    constexpr int U = V4 ? 4 : 8;
    using V = typename std::conditional<V4, float4, float>::type;
    const int units = nr * PER;
    V *dst = reinterpret_cast<V *>(cl);
    for (int e0 = threadIdx.x; e0 < units; e0 += kBlock * U) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { // every load in bounds (the last unit again past the end), none predicated
            const int e = min(e0 + u * kBlock, units - 1);
            v[u] = reinterpret_cast<const V *>(c + (long long)rlist[e / PER] * B)[e % PER];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * kBlock;
            if (e < units) dst[e] = v[u];
        }
    }
}

// Pass 2 over the image-tile column layout: a workgroup takes one tile at a
// time, copies the tile's rows of c into LDS (one gather per row instead of
// one per entry: a ray crosses several pixels of a tile), then sums each
// column of the tile with LPR lanes from LDS and applies the column step.
template <int LPR, int VEC, typename VT>
__global__ __launch_bounds__(kBlock) void k_pass2_tile(TileView T, const float *__restrict__ c,
                                                       float *__restrict__ x, ColStep cs,
                                                       const SliceState *__restrict__ st_in,
                                                       SliceState *__restrict__ st_out,
                                                       const double *__restrict__ part1, int nparts1, Hist h)
{
    extern __shared__ float cl[];
    __shared__ double lds[4];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, 1, part1, nparts1, h, lds);
        return;
    }
    constexpr int RPB = kBlock / LPR;
    double yacc = 0.0;
    if (st_in[0].live) {
        const int lane = threadIdx.x & (LPR - 1);
        const int grp = threadIdx.x / LPR;
        for (int t = blockIdx.x; t < T.ntiles; t += groups) {
            const int r0 = T.rptr[t], nr = T.rptr[t + 1] - r0;
            __syncthreads(); // the previous tile's readers are done with cl
            stage_rows<1>(cl, c, T.rlist + r0, nr);
            __syncthreads();
            const int p0 = T.pptr[t], np = T.pptr[t + 1] - p0;
            for (int q = grp; q < np; q += RPB) {
                const int col = T.tcol[p0 + q];
                const int beg = T.A.ptr[p0 + q], end = T.A.ptr[p0 + q + 1];
                float xo = 0.f, l = 0.f, u = 0.f;
                if (lane == 0 && !cs.defer) {
                    xo = x[col];
                    l = cs.lo[col];
                    u = cs.hi[col];
                }
                const double y = group_sum<LPR>(row_dot<LPR, VEC, VT>(T.A, beg, end, lane, cl)) * (double)T.A.vscale_inv;
                if (lane == 0) yacc += epi2(cs, col, col, y, xo, l, u, x);
            }
        }
    }
    end_columns(cs, yacc, lds);
}

// ---------------------------------------------------------------------------
// Fused single pass (one slice; y = A^T c small enough to live in LDS).  The
// two passes of the feasibility step touch the same entries: row i gives r_i,
// then t_i and c_i = D_i t_i, and c_i a_i is exactly row i's contribution to
// y = A^T c.  So each workgroup streams a contiguous range of CSR rows once,
// forms c_i as pass 1 does and, while the row is still in the cache, adds
// c_i a_i into its own copy of y in LDS (float64 atomics, or float32 when a
// float64 copy does not fit).  Rows inside their band (t_i = 0) add nothing.
// The workgroup's y leaves as one partial vector; k_fused_apply sums the
// partials in workgroup order and applies x = clip(z + lambda y).  A is read
// from memory once per iteration instead of twice, and the column copy of A
// is not read at all.  Summation order inside a workgroup follows the LDS
// atomics, so results agree with the two-pass kernels up to float64 rounding.
// ---------------------------------------------------------------------------

// smallest r in [0, rows] with ptr[r] >= target (ptr[rows] >= target)
__device__ inline int first_row_at(const int *__restrict__ ptr, int rows, long long target)
{
    int lo = 0, hi = rows;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ptr[mid] >= target) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// y[c_e] += sc * v_e for a lane's VEC entries (y in LDS; entries of value 0,
// padding among them, add nothing).  ds_add_f64 takes 8 to 16 clocks a wave
// where the addresses spread over the banks.  ds_add_f32 takes 3 clocks a
// lane whatever its addresses (192 a wave), a read and a compare-and-swap 15
// a wave: so a float32 y is added to by one compare-and-swap round for all
// VEC entries, a second one from the values the first found, and only the
// entries another row changed both times by ds_add_f32 (2.06M rows of 19,881
// columns, 400M entries, an iteration: float32 547 -> 475 us, bfloat16 503 ->
// 347).
template <int VEC>
__device__ inline void lds_add_entries(double *y, const int (&c)[VEC], const float (&v)[VEC], double sc)
{
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        if (v[e] != 0.f) atomicAdd(&y[c[e]], sc * (double)v[e]);
}
template <int VEC>
__device__ inline void lds_add_entries(float *y, const int (&c)[VEC], const float (&v)[VEC], double sc)
{
    unsigned *const w = reinterpret_cast<unsigned *>(y);
    float a[VEC];
    unsigned was[VEC], now[VEC];
    bool nz[VEC], any = false;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        nz[e] = v[e] != 0.f;
        a[e] = nz[e] ? (float)(sc * (double)v[e]) : 0.f; // sc may be infinite
        was[e] = __hip_atomic_load(&w[c[e]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) now[e] = atomicCAS(&w[c[e]], was[e], __float_as_uint(__uint_as_float(was[e]) + a[e]));
#pragma unroll
    for (int e = 0; e < VEC; ++e) any = any || (now[e] != was[e] && nz[e]);
    if (!any) return;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        if (now[e] != was[e] && nz[e]) {
            was[e] = atomicCAS(&w[c[e]], now[e], __float_as_uint(__uint_as_float(now[e]) + a[e]));
            if (was[e] != now[e]) atomicAdd(&y[c[e]], a[e]);
        }
    }
}

// The same for entries held in registers since the dot product, by the
// plain adds: the rows of a workgroup that wait for one another's loads reach
// their scatter together, and on the columns they share the swaps mostly fail
// (radiotherapy, 400M entries, 16 x 8 with a float32 y: 556 us by swaps,
// 547 by adds; without held entries 473 us by swaps, 660 by adds).
template <int VEC, typename AccT>
__device__ inline void lds_add_held(AccT *y, const int (&c)[VEC], const float (&v)[VEC], double sc)
{
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        if (v[e] != 0.f) atomicAdd(&y[c[e]], (AccT)(sc * (double)v[e]));
}

// y[c_j] += sc * a_ij over row [beg, end) (y in LDS), by lane `lane` of an
// LPR-lane group, the row's entries read again (from the cache) one chunk at
// a time.  Group `grp` starts at chunk grp mod (chunks of the row):
// neighbouring rows list the same columns in the same order, so the groups of
// a wave add into different words at once.  (Four chunks' loads in flight
// before their adds measured slower: 674 against 650 us on the radiotherapy
// operator, the LDS atomics rather than the loads setting the pace.)
template <int LPR, int VEC, typename VT, typename AccT>
__device__ inline void scatter_row(const SpView &A, int beg, int end, int lane, int grp, double sc, AccT *y)
{
    constexpr int STEP = LPR * VEC;
    const int nch = (end - beg + STEP - 1) / STEP;
    int q = grp % nch;
    for (int u = 0; u < nch; ++u) {
        const int p = beg + q * STEP + lane * VEC;
        if (++q == nch) q = 0;
        if (p >= end) continue;
        float v[VEC];
        int c[VEC];
        Entries<VT, VEC>::load(A, p, v, c);
        lds_add_entries<VEC>(y, c, v, sc);
    }
}

template <int LPR, int VEC, typename VT, typename AccT>
__global__ __launch_bounds__(kFusedBlock) void k_fused(SpView A, int n, const float *__restrict__ x,
                                                       const float *__restrict__ lower,
                                                       const float *__restrict__ upper, RowW w,
                                                       const SliceState *__restrict__ st,
                                                       double *__restrict__ partials, AccT *__restrict__ ypart)
{
    extern __shared__ __align__(16) unsigned char fused_lds[];
    AccT *y = reinterpret_cast<AccT *>(fused_lds);
    __shared__ double lds[kFusedBlock / 64];
    __shared__ int range[2];
    constexpr int RPB = kFusedBlock / LPR;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const bool live = st[0].live != 0;
    for (int j = threadIdx.x; j < n; j += kFusedBlock) y[j] = AccT(0);
    if (threadIdx.x == 0) { // an equal share of the stored entries
        const long long total = A.ptr[A.rows];
        range[0] = first_row_at(A.ptr, (int)A.rows, total * blockIdx.x / gridDim.x);
        range[1] = first_row_at(A.ptr, (int)A.rows, total * (blockIdx.x + 1) / gridDim.x);
    }
    __syncthreads();
    const int r0 = range[0], r1 = range[1];
    double pacc[1] = {0.0};
    if (live) {
        for (int row = r0 + grp; row < r1; row += RPB) {
            const int beg = A.ptr[row], end = A.ptr[row + 1];
            const float lo = lower[row], up = upper[row], d = w.D[row], sw = w.S[row];
            const double r = group_sum<LPR>(row_dot<LPR, VEC, VT>(A, beg, end, lane, x)) * (double)A.vscale_inv;
            const double t = fmin(fmax(r, (double)lo), (double)up) - r;
            const double dt = (double)d * t, ct = (double)sw * t;
            if (lane == 0) pacc[0] += dt * t;
            if (ct != 0.0 && end > beg) // the same entries again, now from the cache
                scatter_row<LPR, VEC, VT, AccT>(A, beg, end, lane, grp, ct * (double)A.vscale_inv, y);
        }
    }
    block_sum<1, kFusedBlock>(pacc, lds); // its barriers also order the LDS adds before the copy-out
    if (!live) return;
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
    AccT *out = ypart + (long long)blockIdx.x * n;
    for (int j = threadIdx.x; j < n; j += kFusedBlock) out[j] = y[j];
}

// Register-cached, software-pipelined form of the fused pass.  A group of
// LPR lanes keeps up to CAP chunks (LPR*VEC entries each) of its row in
// registers, so the scatter of c_i a_i reuses the loaded entries instead of
// reading them again.  While row i is being reduced and scattered, the
// entries of the group's next row and the offsets and band of the row after
// it are already in flight.  Within a group, lane l holds the chunk slots of
// lane (l + group) mod LPR: the groups of a wave (neighbouring rows, which
// often list the same columns in the same order) then touch different
// columns in the same LDS atomic instruction, and each group still reads one
// contiguous stretch of its row.  Entries past CAP chunks (rows longer than
// CAP*LPR*VEC) are streamed and re-read from the cache as in k_fused.  Two
// rows in registers need more than the 128 registers a 1024-thread
// workgroup leaves a lane, so these workgroups have 512 threads.
template <int VEC, int CAP>
struct RowRegs {
    float v[CAP][VEC];
    int c[CAP][VEC];
};

template <int LPR, int VEC, int CAP, typename VT>
__device__ inline void fetch_entries(const SpView &A, int beg, int end, int slot, RowRegs<VEC, CAP> &R)
{
    bool ok[CAP];
#pragma unroll
    for (int q = 0; q < CAP; ++q) ok[q] = beg + (q * LPR + slot) * VEC < end;
    load_chunks<VT, VEC, CAP>(A, beg + slot * VEC, LPR * VEC, ok, R.v, R.c);
}

template <int LPR, int VEC, int CAP, typename VT, typename AccT>
__global__ __launch_bounds__(kFusedRcBlock) void k_fused_rc(SpView A, int n, const float *__restrict__ x,
                                                          const float *__restrict__ lower,
                                                          const float *__restrict__ upper, RowW w,
                                                          const SliceState *__restrict__ st,
                                                          double *__restrict__ partials, AccT *__restrict__ ypart)
{
    extern __shared__ __align__(16) unsigned char fused_lds[];
    AccT *y = reinterpret_cast<AccT *>(fused_lds);
    __shared__ double lds[kFusedRcBlock / 64];
    __shared__ int range[2];
    constexpr int RPB = kFusedRcBlock / LPR;
    constexpr int STEP = LPR * VEC;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int slot = (lane + grp) & (LPR - 1);
    const bool live = st[0].live != 0;
    for (int j = threadIdx.x; j < n; j += kFusedRcBlock) y[j] = AccT(0);
    if (threadIdx.x == 0) {
        const long long total = A.ptr[A.rows];
        range[0] = first_row_at(A.ptr, (int)A.rows, total * blockIdx.x / gridDim.x);
        range[1] = first_row_at(A.ptr, (int)A.rows, total * (blockIdx.x + 1) / gridDim.x);
    }
    __syncthreads();
    const int r0 = range[0], r1 = range[1];
    double pacc[1] = {0.0};
    int row = r0 + grp;
    if (live && row < r1) {
        // row `row`: entries in cur; row + RPB: offsets/band in nb..; entries follow
        RowRegs<VEC, CAP> cur, nxt;
        int beg = A.ptr[row], end = A.ptr[row + 1];
        float lo = lower[row], up = upper[row], d = w.D[row], sw = w.S[row];
        fetch_entries<LPR, VEC, CAP, VT>(A, beg, end, slot, cur);
        int nb = 0, ne = 0;
        float nlo = 0.f, nup = 0.f, nd = 0.f, nsw = 0.f;
        if (row + RPB < r1) {
            nb = A.ptr[row + RPB];
            ne = A.ptr[row + RPB + 1];
            nlo = lower[row + RPB];
            nup = upper[row + RPB];
            nd = w.D[row + RPB];
            nsw = w.S[row + RPB];
        }
        for (;;) {
            float xg[CAP][VEC];
#pragma unroll
            for (int q = 0; q < CAP; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) xg[q][e] = x[cur.c[q][e]];
            const int rn = row + RPB, rnn = row + 2 * RPB;
            if (rn < r1) fetch_entries<LPR, VEC, CAP, VT>(A, nb, ne, slot, nxt);
            int hb = 0, he = 0;
            float hlo = 0.f, hup = 0.f, hd = 0.f, hsw = 0.f;
            if (rnn < r1) {
                hb = A.ptr[rnn];
                he = A.ptr[rnn + 1];
                hlo = lower[rnn];
                hup = upper[rnn];
                hd = w.D[rnn];
                hsw = w.S[rnn];
            }
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < CAP; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc = fma((double)cur.v[q][e], (double)xg[q][e], acc);
            const bool tail = end - beg > CAP * STEP;
            if (tail) acc += row_dot<LPR, VEC, VT>(A, beg + CAP * STEP, end, lane, x);
            const double r = group_sum<LPR>(acc) * (double)A.vscale_inv;
            const double t = fmin(fmax(r, (double)lo), (double)up) - r;
            const double dt = (double)d * t, ct = (double)sw * t;
            if (lane == 0) pacc[0] += dt * t;
            if (ct != 0.0) {
                const double sc = ct * (double)A.vscale_inv;
#pragma unroll
                for (int q = 0; q < CAP; ++q) lds_add_held<VEC>(y, cur.c[q], cur.v[q], sc);
                if (tail) {
                    for (int p = beg + CAP * STEP + lane * VEC; p < end; p += STEP) {
                        float v[VEC];
                        int c[VEC];
                        Entries<VT, VEC>::load(A, p, v, c);
                        lds_add_entries<VEC>(y, c, v, sc);
                    }
                }
            }
            if (rn >= r1) break;
            row = rn;
            beg = nb;
            end = ne;
            lo = nlo;
            up = nup;
            d = nd;
            sw = nsw;
            cur = nxt;
            nb = hb;
            ne = he;
            nlo = hlo;
            nup = hup;
            nd = hd;
            nsw = hsw;
        }
    }
    block_sum<1, kFusedRcBlock>(pacc, lds); // its barriers also order the LDS adds before the copy-out
    if (!live) return;
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
    AccT *out = ypart + (long long)blockIdx.x * n;
    for (int j = threadIdx.x; j < n; j += kFusedRcBlock) out[j] = y[j];
}

// Direction partials of the linear objective f = c^T x for the next
// perturbation phase: this workgroup's sums of c_j^2 and c_j x_j over the
// unknowns j0 + l (l < CW, j0 = CW blockIdx.x, stepping CW groups), each of
// its first CW threads adding its own in that order, then over the workgroup
// (BS threads), stored as the direction launch's partials would be (slot
// blockIdx.x of 2 x groups).  k_fused_apply calls it after writing x and
// k_lin_partials alone, with the same sums in the same order (CW = BS = kBlock:
// those of k_step_apply), so a phase does not depend on where a run starts.
template <int CW, int BS>
__device__ inline void lin_partials_block(const float *__restrict__ x, const float *__restrict__ c, int n,
                                          int groups, double *__restrict__ part, double *lds)
{
    double v[2] = {0.0, 0.0}; // sum c^2, c^T x
    if (threadIdx.x < CW)
        for (int j = blockIdx.x * CW + (int)threadIdx.x; j < n; j += groups * CW) {
            const double cj = (double)c[j];
            v[0] += cj * cj;
            v[1] += cj * (double)x[j];
        }
    block_sum<2, BS>(v, lds);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = v[0];
        part[groups + blockIdx.x] = v[1];
    }
}

template <int CW, int BS>
__global__ __launch_bounds__(BS) void k_lin_partials(const float *__restrict__ x, const float *__restrict__ c, int n,
                                                     double *__restrict__ part)
{
    __shared__ double lds[BS / 64 * 2];
    lin_partials_block<CW, BS>(x, c, n, (int)gridDim.x, part, lds);
}

// x = clip(z + lambda * Z_j * sum_g ypart[g], lo, hi) (Z_j = 1 unless DROP);
// CW unknowns per workgroup, whose waves' 64 / CW parts each sum every
// (waves * 64 / CW)th partial (loads issued eight at a time, added in order);
// a wave's parts are added by shuffles and the waves' sums in a fixed order.
// One more workgroup closes the outer iteration.  CW = 16 up to 1,024 unknowns,
// where the launch is a chain of loads over few vectors and a workgroup's
// share of them the longest link (256 x 128 dense, 40 iterations 534 us
// against 547 with 64); CW = 64 beyond (6,293 unknowns, 256 vectors: 6.5 us
// against 7.8 with 16).
template <typename AccT, int CW>
__global__ __launch_bounds__(kApplyBlock) void k_fused_apply(const AccT *__restrict__ ypart, int G, int n,
                                                        float *__restrict__ x, ColStep cs,
                                                        const SliceState *__restrict__ st_in,
                                                        SliceState *__restrict__ st_out,
                                                        const double *__restrict__ part1, int nparts1, Hist h,
                                                        const float *__restrict__ lin_c, double *__restrict__ lin_part,
                                                        int lin_z)
{
    __shared__ double red[kApplyBlock / 64][CW];
    __shared__ double lds[kApplyBlock / 64 * 2];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration<kApplyBlock>(st_in, st_out, 1, part1, nparts1, h, lds);
        return;
    }
    const int wid = threadIdx.x >> 6, wl = threadIdx.x & (CW - 1), part0 = (int)threadIdx.x / CW;
    double ysq = 0.0; // deferred mode: this thread's share of ||y||^2
    // the linear phase taken in the pass: x still holds x^k, z_j is formed here
    bool zstep = false;
    double zs = 0.0, zinv = 0.0;
    if (lin_z && st_in[0].applied && st_in[0].s_acc != 0.0) {
        zstep = true;
        zs = st_in[0].s_acc;
        zinv = 1.0 / st_in[0].gn;
    }
    if (st_in[0].live) {
        for (int j0 = blockIdx.x * CW; j0 < n; j0 += groups * CW) {
            const int j = j0 + wl;
            constexpr int W = kApplyBlock / 64, P = kApplyBlock / CW;
            double sum = 0.0;
            const bool owner = threadIdx.x < CW && j < n;
            float xo = 0.f, l = 0.f, u0 = 0.f;
            if (owner && !cs.defer) { // the step's operands, fetched beside the partials
                xo = x[j];
                l = cs.lo[j];
                u0 = cs.hi[j];
            }
            if (j < n) { // part p adds partials p, p + P, ... (eight loads in flight, then four)
                int g = part0;
                for (; g + 7 * P < G; g += 8 * P) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = (double)ypart[(long long)(g + u * P) * n + j];
#pragma unroll
                    for (int u = 0; u < 8; ++u) sum += v[u];
                }
                if (g + 3 * P < G) {
                    double v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = (double)ypart[(long long)(g + u * P) * n + j];
#pragma unroll
                    for (int u = 0; u < 4; ++u) sum += v[u];
                    g += 4 * P;
                }
                for (; g < G; g += P) sum += (double)ypart[(long long)g * n + j];
            }
#pragma unroll
            for (int off = CW; off < 64; off <<= 1) sum += __shfl_xor(sum, off, 64);
            if ((threadIdx.x & 63) < CW) red[wid][wl] = sum;
            __syncthreads();
            if (owner) {
                double yv = 0.0;
#pragma unroll
                for (int w = 0; w < W; ++w) yv += red[w][wl];
                if (cs.defer) { // the extrapolated steps: keep y, x moves in k_step_apply
                    cs.ybuf[j] = yv;
                    if (cs.ybuf32) cs.ybuf32[j] = (float)yv;
                    ysq += yv * yv;
                } else {
                    if (cs.zcol) yv *= (double)cs.zcol[j];
                    const float zj = zstep ? linear_step_point(xo, lin_c[j], zs, zinv) : xo;
                    const double z = fma((double)cs.lambda, yv, (double)zj);
                    x[j] = (float)fmin(fmax(z, (double)l), (double)u0);
                }
            }
            __syncthreads();
        }
    }
    // the next phase's direction partials from the x just written (each
    // lane rereads its own entries)
    if (lin_part) lin_partials_block<CW, kApplyBlock>(x, lin_c, n, groups, lin_part, lds);
    end_columns<kApplyBlock>(cs, ysq, lds);
}

// Extrapolated steps (one launch after pass 2, or after the quadratic-form
// pass): per slice, sigma from the totals of the partials, each summed in
// workgroup order by every workgroup (EL: t^T D t / ||y||^2, with t^T D t
// twice pass 1's proximity sum; EMR: ||y||^2 / sum_i w_i (A y)_i^2), 0 when the
// denominator is 0 or the quotient is not finite; then
// x = clip(z + lambda sigma y, lo, hi).  One more workgroup, the last, closes
// the iteration.  lin_c (one slice, linear objective): the pass took the phase
// and x still holds x^k where lin_z is set, so z_j is formed here, and the
// workgroups' partials of the next phase's direction go to lin_part, as
// k_fused_apply's do for the steps it applies (5,625 columns, dose-volume
// rows: 113.1 us an iteration, 115.2 with the phase in a launch of its own).
__global__ __launch_bounds__(kBlock) void k_step_apply(int n, int B, const double *__restrict__ y,
                                                       float *__restrict__ x, const float *__restrict__ lo,
                                                       const float *__restrict__ hi, float lambda, int emr,
                                                       const double *__restrict__ part1, int nparts1,
                                                       const double *__restrict__ party, int npartsy,
                                                       const double *__restrict__ partq, int npartsq,
                                                       const SliceState *__restrict__ st_in,
                                                       SliceState *__restrict__ st_out, Hist h,
                                                       const float *__restrict__ lin_c, double *__restrict__ lin_part,
                                                       int lin_z)
{
    __shared__ double lds[4 * 2];
    __shared__ double sigma[32];
    __shared__ int live[32];
    const int groups = (int)gridDim.x - 1;
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, B, part1, nparts1, h, lds);
        return;
    }
    for (int s = 0; s < B; ++s) {
        double num[1], den[1];
        if (emr) {
            sum_slots<1>(party, (long long)s * npartsy, npartsy, num, lds);
            sum_slots<1>(partq, (long long)s * npartsq, npartsq, den, lds);
        } else {
            sum_slots<1>(part1, (long long)s * nparts1, nparts1, num, lds);
            sum_slots<1>(party, (long long)s * npartsy, npartsy, den, lds);
        }
        if (threadIdx.x == 0) {
            const double q = num[0] / den[0];
            sigma[s] = (den[0] > 0.0 && isfinite(q)) ? q : 0.0;
            live[s] = st_in[s].live;
        }
    }
    __syncthreads();
    if (lin_c) {
        const bool zstep = lin_z && st_in[0].applied && st_in[0].s_acc != 0.0;
        const double zs = zstep ? st_in[0].s_acc : 0.0, zinv = zstep ? 1.0 / st_in[0].gn : 0.0;
        double v[2] = {0.0, 0.0}; // sum c^2, c^T x
        for (int j = blockIdx.x * kBlock + (int)threadIdx.x; j < n; j += groups * kBlock) {
            const float cj = lin_c[j];
            float xj = x[j];
            if (live[0]) {
                const float zj = zstep ? linear_step_point(xj, cj, zs, zinv) : xj;
                xj = (float)fmin(fmax(fma((double)lambda * sigma[0], y[j], (double)zj), (double)lo[j]), (double)hi[j]);
                x[j] = xj;
            }
            v[0] += (double)cj * (double)cj;
            v[1] += (double)cj * (double)xj;
        }
        block_sum<2>(v, lds);
        if (threadIdx.x == 0) {
            lin_part[blockIdx.x] = v[0];
            lin_part[groups + blockIdx.x] = v[1];
        }
        return;
    }
    const long long total = (long long)n * B;
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < total; e += (long long)groups * kBlock) {
        const int s = (int)(e % B);
        if (!live[s]) continue;
        const long long j = e / B;
        const double z = fma((double)lambda * sigma[s], y[e], (double)x[e]);
        x[e] = (float)fmin(fmax(z, (double)lo[j]), (double)hi[j]);
    }
}

// ---------------------------------------------------------------------------
// Multi-slice passes (B right-hand sides sharing A, slice-interleaved
// vectors).  A is read once for all slices; the B values of the gathered
// vector at an entry's index are one contiguous stretch of 4B bytes.  The
// lanes of a row group are split into LS = B/4 lanes over the slices (four
// slices each, one 16-byte load) times EG = LPR/LS lanes over the row's
// entries, so one load instruction of a wave fetches whole stretches (B = 32:
// eight entries, 128 bytes each).  (With all B slices in every lane, as these
// kernels were first written, each instruction touched 64 different cache
// lines for 16 bytes of each, and the vector memory path's address rate
// bound the pass: 256 x 256 CT, 15.0M entries, B = 32, bf16 297 us pass 1 and
// 254 us pass 2 against 112 and 101 now, 1.9 GB of gathered lines at 17 and
// 19 TB/s out of L2; 128 x 128, B = 8, float32 26 and 29 us against 16 and
// 19.)  The summation order of a slice does not depend on
// the other slices, so a slice's result is the same whichever slices run
// beside it.  A slice that is not live is neither read back nor written.
// ---------------------------------------------------------------------------

template <int B>
struct SliceLanes {
    static constexpr int LS = B >= 4 ? B / 4 : 1; // lanes over the slices
    static constexpr int NS = B / LS;             // slices a lane holds
};

template <int N>
__device__ inline void load_floats(const float *__restrict__ v, float (&out)[N])
{
    static_assert(N == 2 || N == 4, "slices of a lane");
    if constexpr (N == 4) {
        const float4 a = *reinterpret_cast<const float4 *>(v);
        out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
    } else {
        const float2 a = *reinterpret_cast<const float2 *>(v);
        out[0] = a.x; out[1] = a.y;
    }
}

// v[k] into out[k] where on[k] (one vector store when every one is on).
template <int N>
__device__ inline void store_floats(float *__restrict__ out, const float (&v)[N], const bool (&on)[N])
{
    bool all = true;
#pragma unroll
    for (int k = 0; k < N; ++k) all = all && on[k];
    if (all) {
        if constexpr (N == 4) *reinterpret_cast<float4 *>(out) = make_float4(v[0], v[1], v[2], v[3]);
        else *reinterpret_cast<float2 *>(out) = make_float2(v[0], v[1]);
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (on[k]) out[k] = v[k];
    }
}

// Dot products of one row with a lane's NS slices of v, by lane `lane` of an
// LPR-lane group; every lane of the group returns the sums of its slices.  Two
// chunks of VEC entries are gathered at a time (2 * VEC loads of the vector
// in flight per lane), the next two chunks' entries already requested.
template <int LPR, int VEC, typename VT, int B>
__device__ inline void row_dot_mm(const SpView &A, int beg, int end, int lane, const float *__restrict__ v,
                                  double (&acc)[SliceLanes<B>::NS])
{
    constexpr int LS = SliceLanes<B>::LS, NS = SliceLanes<B>::NS, EG = LPR / LS, STEP = EG * VEC, U = 2;
    static_assert(EG >= 1 && EG * LS == LPR, "lanes per row");
    const float *vs = v + (lane & (LS - 1)) * NS;
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = 0.0;
    int p = beg + (lane / LS) * VEC;
    EntryRaw<VT, VEC> raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        raw[u].zero();
        if (p + u * STEP < end) raw[u].load(A, p + u * STEP);
    }
    while (p < end) {
        float val[U][VEC];
        int id[U][VEC];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = p + u * STEP < end;
            raw[u].decode(val[u], id[u]);
        }
        p += U * STEP;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            raw[u].zero();
            if (p + u * STEP < end) raw[u].load(A, p + u * STEP);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ok[u]) {
                float xs[VEC][NS];
#pragma unroll
                for (int e = 0; e < VEC; ++e) load_floats<NS>(vs + (long long)id[u][e] * B, xs[e]);
#pragma unroll
                for (int e = 0; e < VEC; ++e)
#pragma unroll
                    for (int s = 0; s < NS; ++s) acc[s] = fma((double)val[u][e], (double)xs[e][s], acc[s]);
            }
    }
#pragma unroll
    for (int off = LS; off < LPR; off <<= 1)
#pragma unroll
        for (int s = 0; s < NS; ++s) acc[s] += __shfl_xor(acc[s], off, LPR);
}

// Workgroup sums per slice of v (lane l of a wave holds slices (l mod LS) NS
// ..), written by thread s < B to out[s * gridDim.x + blockIdx.x].
template <int B>
__device__ inline void slice_partials(double (&v)[SliceLanes<B>::NS], double *__restrict__ out)
{
    constexpr int LS = SliceLanes<B>::LS, NS = SliceLanes<B>::NS;
    __shared__ double red[kBlock / 64][B];
#pragma unroll
    for (int off = LS; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < NS; ++k) v[k] += __shfl_xor(v[k], off, 64);
    const int wid = threadIdx.x >> 6, wl = threadIdx.x & 63;
    if (wl < LS) {
#pragma unroll
        for (int k = 0; k < NS; ++k) red[wid][wl * NS + k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < B) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) t += red[w][threadIdx.x];
        out[(long long)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

template <int LPR, int VEC, typename VT, int B>
__global__ __launch_bounds__(kBlock) void k_pass1_mm(SpView A, const float *__restrict__ x,
                                                     const float *__restrict__ lower, const float *__restrict__ upper,
                                                     RowW w, float *__restrict__ c,
                                                     const SliceState *__restrict__ st, int query,
                                                     double *__restrict__ partials)
{
    constexpr int RPB = kBlock / LPR, LS = SliceLanes<B>::LS, NS = SliceLanes<B>::NS;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int s0 = (lane & (LS - 1)) * NS; // this lane's first slice
    bool live[NS];
    double pacc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        live[k] = query ? true : st[s0 + k].live != 0;
        pacc[k] = 0.0;
    }
    const long long stride = (long long)gridDim.x * RPB;
    long long row = (long long)blockIdx.x * RPB + grp;
    int beg = 0, end = 0;
    if (row < A.rows) {
        beg = A.ptr[row];
        end = A.ptr[row + 1];
    }
    for (; row < A.rows; row += stride) {
        int nbeg = 0, nend = 0; // the next row's offsets, in flight meanwhile
        if (row + stride < A.rows) {
            nbeg = A.ptr[row + stride];
            nend = A.ptr[row + stride + 1];
        }
        float lo[NS], up[NS], cv[NS]; // epilogue operands, fetched while the row streams
        load_floats<NS>(lower + row * B + s0, lo);
        load_floats<NS>(upper + row * B + s0, up);
        const float d = w.D[row], sw = w.S[row];
        double acc[NS];
        row_dot_mm<LPR, VEC, VT, B>(A, beg, end, lane, x, acc);
        if (lane < LS) {
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                cv[k] = 0.f;
                if (live[k]) pacc[k] += epi1(w, acc[k] * (double)A.vscale_inv, lo[k], up[k], d, sw, &cv[k], row, s0 + k, B);
            }
            const bool dose_row = w.dose && row >= w.dose_lo && row < w.dose_hi;
            if (!w.qform && !dose_row) store_floats<NS>(c + row * B + s0, cv, live);
        }
        beg = nbeg;
        end = nend;
    }
    slice_partials<B>(pacc, partials);
}

// Column step of a lane's NS slices of one column (x and ybuf index e .. e +
// NS - 1, live slices only); adds y^2 to yacc in the deferred mode.
template <int NS>
__device__ inline void epi2_slices(const ColStep &cs, long long col, long long e, const double (&y)[NS],
                                   const float (&xo)[NS], float l, float u, const bool (&live)[NS],
                                   float *__restrict__ x, double (&yacc)[NS])
{
    if (cs.defer) {
#pragma unroll
        for (int k = 0; k < NS; ++k)
            if (live[k]) yacc[k] += epi2(cs, col, e + k, y[k], xo[k], l, u, x);
        return;
    }
    const double f = cs.zcol ? (double)cs.zcol[col] : 1.0;
    float xn[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
        xn[k] = (float)fmin(fmax(fma((double)cs.lambda, y[k] * f, (double)xo[k]), (double)l), (double)u);
    store_floats<NS>(x + e, xn, live);
}

template <int LPR, int VEC, typename VT, int B>
__global__ __launch_bounds__(kBlock) void k_pass2_mm(SpView At, const float *__restrict__ c, float *__restrict__ x,
                                                     ColStep cs, const SliceState *__restrict__ st_in,
                                                     SliceState *__restrict__ st_out,
                                                     const double *__restrict__ part1, int nparts1, Hist h)
{
    __shared__ double lds[4];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, B, part1, nparts1, h, lds);
        return;
    }
    constexpr int RPB = kBlock / LPR, LS = SliceLanes<B>::LS, NS = SliceLanes<B>::NS;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int s0 = (lane & (LS - 1)) * NS;
    bool live[NS];
    double yacc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        live[k] = st_in[s0 + k].live != 0;
        yacc[k] = 0.0;
    }
    const long long stride = (long long)groups * RPB;
    long long col = (long long)blockIdx.x * RPB + grp;
    int beg = 0, end = 0;
    if (col < At.rows) {
        beg = At.ptr[col];
        end = At.ptr[col + 1];
    }
    for (; col < At.rows; col += stride) {
        int nbeg = 0, nend = 0; // the next column's offsets, in flight meanwhile
        if (col + stride < At.rows) {
            nbeg = At.ptr[col + stride];
            nend = At.ptr[col + stride + 1];
        }
        float xo[NS];
        load_floats<NS>(x + col * B + s0, xo);
        const float l = cs.lo[col], u = cs.hi[col];
        double acc[NS];
        row_dot_mm<LPR, VEC, VT, B>(At, beg, end, lane, c, acc);
        if (lane < LS) {
#pragma unroll
            for (int k = 0; k < NS; ++k) acc[k] *= (double)At.vscale_inv;
            epi2_slices<NS>(cs, col, col * B + s0, acc, xo, l, u, live, x, yacc);
        }
        beg = nbeg;
        end = nend;
    }
    if (cs.defer) slice_partials<B>(yacc, cs.ypart);
}

// Pass 2 over the image-tile column layout for B slices: the tile's rows of
// c (B values each, slice-interleaved as in memory) are staged in LDS, and
// every entry of a column reads its B values from there, as k_pass2_tile does
// for one slice.
template <int LPR, int VEC, typename VT, int B>
__global__ __launch_bounds__(kBlock) void k_pass2_tile_mm(TileView T, const float *__restrict__ c,
                                                          float *__restrict__ x, ColStep cs,
                                                          const SliceState *__restrict__ st_in,
                                                          SliceState *__restrict__ st_out,
                                                          const double *__restrict__ part1, int nparts1, Hist h)
{
    extern __shared__ float4 cl4[]; // 16-byte aligned: rows of B floats
    float *cl = reinterpret_cast<float *>(cl4);
    __shared__ double lds[4];
    const int groups = column_groups(cs);
    if ((int)blockIdx.x == groups) { // the same in every thread
        finish_iteration(st_in, st_out, B, part1, nparts1, h, lds);
        return;
    }
    __shared__ int any_live;
    constexpr int RPB = kBlock / LPR, LS = SliceLanes<B>::LS, NS = SliceLanes<B>::NS;
    if (threadIdx.x == 0) any_live = 0;
    __syncthreads();
    if (threadIdx.x < B && st_in[threadIdx.x].live) any_live = 1; // every writer stores 1
    __syncthreads();
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int s0 = (lane & (LS - 1)) * NS;
    bool live[NS];
    double yacc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        live[k] = st_in[s0 + k].live != 0;
        yacc[k] = 0.0;
    }
    if (any_live) {
        for (int t = blockIdx.x; t < T.ntiles; t += groups) {
            const int r0 = T.rptr[t], nr = T.rptr[t + 1] - r0;
            __syncthreads(); // the previous tile's readers are done with cl
            stage_rows<B>(cl, c, T.rlist + r0, nr);
            __syncthreads();
            const int p0 = T.pptr[t], np = T.pptr[t + 1] - p0;
            for (int q = grp; q < np; q += RPB) {
                const int col = T.tcol[p0 + q];
                const int beg = T.A.ptr[p0 + q], end = T.A.ptr[p0 + q + 1];
                const long long e = (long long)col * B + s0;
                float xo[NS];
                load_floats<NS>(x + e, xo);
                const float l = cs.lo[col], u = cs.hi[col];
                double acc[NS];
                row_dot_mm<LPR, VEC, VT, B>(T.A, beg, end, lane, cl, acc);
                if (lane < LS) {
#pragma unroll
                    for (int k = 0; k < NS; ++k) acc[k] *= (double)T.A.vscale_inv;
                    epi2_slices<NS>(cs, col, e, acc, xo, l, u, live, x, yacc);
                }
            }
        }
    }
    if (cs.defer) slice_partials<B>(yacc, cs.ypart);
}

// ---------------------------------------------------------------------------
// perturbation phase
//
// Launch sequence of one phase: gradient (partials of ||g||^2 and f(x^k) per
// tile), then trial launches, then a closing launch.  Each trial launch first
// re-derives, in every workgroup, what the previous launch decided (the first
// launch: the opening of the phase) from that launch's partials, then either
// evaluates the next batch of trial steps or, once the phase is over, adds the
// accepted step s_acc v to its own tile of x.  Partials are stored value-major
// ([value][slice*tiles + tile]) so the re-derivation reads them coalesced.
// ---------------------------------------------------------------------------

// Step of trial e (the trial exponent): the power law gamma alpha^e, or the
// phase's adaptive step (Section 2.1.2), the same for its one trial.
__device__ inline double trial_beta(const PertParams &pp, const SliceState &S, long long e)
{
    return pp.adaptive ? S.beta_ad : pp.gamma * pow(pp.alpha, (double)e);
}

// The steps of 64 trials from exponent `base` on, formed by the last wave of a
// workgroup while the others sum the partials that decide which of them are
// asked for: pow in float64 is ~0.7 us, and stood twice in the chain of every
// trial launch (187 x 171 CT, four steps a phase: 7.7 us a trial launch, now
// 6.75; 256 x 256, one step: 5.6, now 5.2).
struct StepWindow {
    long long base;
    double beta[64];
};

// Every thread calls it; the next barrier publishes the window.  first: the
// phase opens in this launch, so the exponent is the one that
// open_phase_state will start from.
template <int BS>
__device__ inline void form_steps(StepWindow &win, const PertParams &pp, const SliceState &S, int first)
{
    if (threadIdx.x < BS - 64 || pp.adaptive) return;
    long long e = S.ell;
    if (first && pp.restart_every > 0 && S.k > 0 && (S.k % pp.restart_every) == 0) e = S.restarts + 1;
    const int l = threadIdx.x & 63;
    win.beta[l] = pp.gamma * pow(pp.alpha, (double)(e + l));
    if (l == 0) win.base = e;
}

__device__ inline double step_of(const StepWindow &win, const PertParams &pp, const SliceState &S, long long e)
{
    if (!pp.adaptive && e >= win.base && e < win.base + 64) return win.beta[e - win.base];
    return trial_beta(pp, S, e);
}

// Trials a launch evaluates for slice state S, with `after` evaluating
// launches behind it: the first batch of a reduction step is the default
// width, widened to 1.5x the trials the previous step needed (step sizes
// shrink along the phase, so that is usually enough); a second batch takes
// every trial left up to the cap.  A first batch that fails costs the step a
// second launch: where the launches left would then not reach for one per
// remaining step, the first batch takes every trial at once.  The width only
// decides how many trials are evaluated speculatively: the accepted trial is
// the first acceptable one in order whatever the width.
__device__ inline int trial_width(const SliceState &S, const PertParams &pp, int after)
{
    if (!S.phase) return 0;
    const int left = pp.max_trials - S.step_tried;
    if (S.step_tried != 0 || after < pp.n_red - S.n_done) return left;
    int w = pp.first_width;
    const int want = S.need_last + (S.need_last >> 1);
    if (want > w) w = ((want + kFirstWidth - 1) / kFirstWidth) * kFirstWidth;
    return min(w, left);
}

// Workgroups of 1,024 threads that the device holds at once (two a CU).
constexpr long long kTvResident = 512;

// Whether a workgroup of the TV phase takes a tile's pixels of every slice
// (k_phase_tv_mm, k_trial_tv_mm) or of one (k_phase_tv, k_trial_tv).  While all
// (16 x 16 tile, slice) pairs are resident at once their strided reads cost
// little and a wave values a trial of its own; in whole lines the trials of a
// pixel are a chain in one thread.  Four reduction steps with rejected trials,
// an iteration, a slice a workgroup against whole lines: 64 x 64, 32 slices (512
// pairs) 114 us against 293; 128 x 128, 4 slices 52 against 70, 8 (512) 83
// against 88, 16 146 against 140, 32 274 against 178; 256 x 256, 2 (512) 91 each,
// 4 145 against 113, 32 973 against 357.
static inline bool tv_whole_lines(const PertParams &pp)
{
    const long long tiles = (long long)((pp.tv_rows + kTile - 1) / kTile) * ((pp.tv_cols + kTile - 1) / kTile);
    return pp.obj == OBJ_TV2D && pp.B > 1 && tiles * pp.B > kTvResident;
}

// Rows of a TV tile: kTile for a workgroup of one slice; in whole lines halved
// (down to 2) while the image has under 256 tiles.
static inline int tv_tile_rows(const PertParams &pp)
{
    int th = kTile;
    if (tv_whole_lines(pp))
        while (th > 2 && ((pp.tv_rows + th - 1) / th) * ((pp.tv_cols + kTile - 1) / kTile) < 256) th /= 2;
    return th;
}

// Grid of the phase kernels: blockIdx.y is the slice, blockIdx.x a tile (TV)
// or a chunk of the vector.
int phase_grid(const PertParams &pp)
{
    if (pp.obj == OBJ_TV2D)
        return ((pp.tv_rows + tv_tile_rows(pp) - 1) / tv_tile_rows(pp)) * ((pp.tv_cols + kTile - 1) / kTile);
    long long g = (pp.n + kBlock * 4 - 1) / (kBlock * 4);
    return (int)(g < 1 ? 1 : (g > kFlatPhaseGrid ? kFlatPhaseGrid : g));
}

// Totals over the `nt` tiles of slice s of rows v0 .. v0+nv-1 (rows of
// `nslots` slots, nv <= kTrialChunk) into tot[0..nv-1] (LDS), for a workgroup
// of BS threads; every thread must call it, and tot is valid for every thread
// on return.  Row v0+r is summed by wave r mod (BS/64): lane l adds tiles
// l, l+64, ... in order, then the lanes are added by wave_sum.  The rows of a
// wave, and U tiles of each, are loaded together, so their loads overlap.
template <int BS>
__device__ inline void chunk_totals(const double *__restrict__ part, long long nslots, int s, int nt, int v0, int nv,
                                    double *tot)
{
    constexpr int W = BS / 64, RPW = (kTrialChunk + W - 1) / W;
    constexpr int U = RPW >= 16 ? 1 : 16 / RPW;
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double a[RPW];
#pragma unroll
    for (int q = 0; q < RPW; ++q) a[q] = 0.0;
    if (wid < nv) {
        for (int b0 = lane; b0 < nt; b0 += 64 * U) {
            double v[U][RPW];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = min(b0 + 64 * u, nt - 1); // past nt: loaded, not added
#pragma unroll
                for (int q = 0; q < RPW; ++q)
                    v[u][q] = part[(long long)(v0 + min(wid + W * q, nv - 1)) * nslots + (long long)s * nt + b];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (b0 + 64 * u < nt) {
#pragma unroll
                    for (int q = 0; q < RPW; ++q) a[q] += v[u][q];
                }
        }
        wave_sum<RPW>(a);
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < RPW; ++q)
                if (wid + W * q < nv) tot[wid + W * q] = a[q];
        }
    }
    __syncthreads();
}

// Opening of a phase from the totals (sum g^2, f(x^k)).
__device__ inline void open_phase_state(SliceState &S, const PertParams &pp, double gsq, double f)
{
    S.trials_it = 0;
    S.accepts_it = 0;
    S.s_acc = 0.0;
    S.n_done = 0;
    S.step_tried = 0;
    S.applied = 0;
    if (!S.live) {
        S.phase = 0;
        S.f_start = S.f_cur = nan64();
        return;
    }
    // superiorized stopping rule (Section 2.2.3): a proximity rule held at the
    // last iteration and |f(x^k) - f(x^{k-1})| / max{1, f(x^{k-1})} < Delta f*
    if (S.stop_on && S.feas_ok && !isnan(S.f_last) && fabs(f - S.f_last) / fmax(1.0, S.f_last) < S.stop_dobj) {
        S.stop_reason = STOP_SM;
        S.live = 0;
        S.phase = 0;
        S.f_start = S.f_cur = nan64();
        return;
    }
    if (pp.restart_every > 0 && S.k > 0 && (S.k % pp.restart_every) == 0) {
        S.restarts += 1;
        S.ell = S.restarts;
    }
    S.gn = sqrt(gsq);
    S.f_start = S.f_cur = f;
    if (!isfinite(f) || !isfinite(S.gn)) S.nonfinite = 1;
    S.phase = (S.gn > 0.0 && isfinite(S.gn)) ? 1 : 0;
    if (pp.adaptive) { // one step to the reference value, none before there is one or when f is at or below it
        if (S.phase && !isnan(S.f_ref) && f > S.f_ref) S.beta_ad = (f - S.f_ref) / S.gn;
        else S.phase = 0;
    }
}

// The state after a batch of ntr trials (steps ell .. ell+ntr-1 of the power
// law, or the one adaptive step) was evaluated: acc_t is the first trial in
// order whose objective does not exceed f_cur (-1 when none does), acc_f its
// objective and beta its step.  Accepting ends the reduction step (and the
// phase after n_red of them); a step that reaches the trial cap unaccepted
// ends the phase.
__device__ inline void record_decision(SliceState &S, const PertParams &pp, int ntr, int acc_t, double acc_f,
                                       double beta)
{
    if (acc_t >= 0) {
        S.s_acc = S.s_acc + beta;
        S.f_cur = acc_f;
        if (!isfinite(acc_f)) S.nonfinite = 1;
        S.ell += acc_t + 1;
        S.trials_it += acc_t + 1;
        S.trials += acc_t + 1;
        S.accepts_it += 1;
        S.accepts += 1;
        S.n_done += 1;
        S.need_last = S.step_tried + acc_t + 1;
        S.step_tried = 0;
        if (S.n_done >= pp.n_red) S.phase = 0;
    } else {
        S.ell += ntr;
        S.trials_it += ntr;
        S.trials += ntr;
        S.step_tried += ntr;
        if (S.step_tried >= pp.max_trials) {
            if (!pp.adaptive) S.cap_hits += 1; // a rejected adaptive step simply ends the phase
            S.need_last = pp.max_trials;
            S.phase = 0;
        }
    }
}

// Every workgroup: the state after the previous trial launch of slice s, in
// sS (LDS).  The first trial in order whose objective does not exceed f_cur is
// accepted; reading stops at the chunk holding it.
template <int BS>
__device__ inline void derive_decision(SliceState &sS, const PertParams &pp, const double *__restrict__ part_prev,
                                       long long nslots, int s, int nt, double *tot, StepWindow &win, int after)
{
    __shared__ int acc_t;
    __shared__ double acc_f;
    const int ntr = trial_width(sS, pp, after + 1); // as the launch before this one saw it
    if (ntr == 0) return;
    if (threadIdx.x == 0) acc_t = -1;
    form_steps<BS>(win, pp, sS, 0);
    for (int t0 = 0; t0 < ntr; t0 += kTrialChunk) {
        const int nv = min(kTrialChunk, ntr - t0);
        chunk_totals<BS>(part_prev, nslots, s, nt, t0, nv, tot);
        if (threadIdx.x < 64) {
            const int l = threadIdx.x;
            const unsigned long long ok = __ballot(l < nv && tot[min(l, nv - 1)] <= sS.f_cur);
            if (l == 0 && ok) {
                acc_t = t0 + __ffsll(ok) - 1;
                acc_f = tot[acc_t - t0];
            }
        }
        __syncthreads();
        if (acc_t >= 0) break;
    }
    if (threadIdx.x == 0)
        record_decision(sS, pp, ntr, acc_t, acc_f, acc_t >= 0 ? step_of(win, pp, sS, sS.ell + acc_t) : 0.0);
    __syncthreads();
}

// Every workgroup: state of slice s at the start of this launch, in sS, and
// the steps of the trials from there on, in win.
// first: the first trial launch (opens the phase from the gradient partials);
// otherwise the decision of the previous trial launch (`after`: evaluating
// launches behind this one, -1 in the closing launch).
template <int BS>
__device__ inline void derive_state(SliceState &sS, const SliceState *__restrict__ st_in, const PertParams &pp,
                                    int first, const double *__restrict__ part_prev, int s, int nt, double *tot,
                                    StepWindow &win, int after = 0)
{
    if (threadIdx.x == 0) sS = st_in[s];
    const long long nslots = (long long)pp.B * nt;
    if (first) { // the state's loads overlap the partials' (thread 0 alone reads sS before the barriers)
        form_steps<BS>(win, pp, st_in[s], 1);
        chunk_totals<BS>(part_prev, nslots, s, nt, 0, 2, tot);
        if (threadIdx.x == 0) open_phase_state(sS, pp, tot[0], tot[1]);
        __syncthreads();
    } else {
        __syncthreads();
        derive_decision<BS>(sS, pp, part_prev, nslots, s, nt, tot, win, after);
    }
}

__device__ inline void publish_state(const SliceState &S, SliceState *__restrict__ st_out, int s, bool applied_here)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        SliceState o = S;
        if (applied_here) o.applied = 1;
        st_out[s] = o;
    }
}

// Whether this launch adds the accepted step to x (the phase is over).
__device__ inline bool must_apply(const SliceState &S) { return S.live && !S.phase && !S.applied && S.s_acc != 0.0; }

// -- TV2D: smoothed total variation on an R x C image, pixel (i,j) = unknown i*C + j.
//    Terms at (i,j) for i <= R-2, j <= C-2: tau = sqrt(dx^2 + dy^2 + eps^2) with
//    dx = X[i+1,j] - X[i,j], dy = X[i,j+1] - X[i,j].

__device__ inline double tv_tau(double x00, double x10, double x01, double eps2)
{
    const double dx = x10 - x00, dy = x01 - x00;
    return sqrt(dx * dx + dy * dy + eps2);
}

// Gradient (unless eval_only) and per-tile partials of ||g||^2 and f(x); the
// tile carries a one-pixel halo on every side.
__global__ __launch_bounds__(kBlock) void k_phase_tv(const float *__restrict__ x, float *__restrict__ g,
                                                     const SliceState *__restrict__ st, PertParams pp, int eval_only,
                                                     double *__restrict__ partials)
{
    __shared__ float tile[kTile + 2][kTile + 3];
    __shared__ double lds[4 * 2];
    const int s = blockIdx.y, B = pp.B;
    const int R = pp.tv_rows, C = pp.tv_cols;
    const int tiles_x = (C + kTile - 1) / kTile;
    const int i0 = (blockIdx.x / tiles_x) * kTile, j0 = (blockIdx.x % tiles_x) * kTile;
    const bool live = eval_only ? true : st[s].live != 0;
    double v[2] = {0.0, 0.0}; // sum g^2, f
    if (live) {
        for (int e = threadIdx.x; e < (kTile + 2) * (kTile + 2); e += kBlock) {
            const int li = e / (kTile + 2), lj = e % (kTile + 2);
            const int gi = i0 - 1 + li, gj = j0 - 1 + lj;
            float val = 0.f;
            if (gi >= 0 && gi < R && gj >= 0 && gj < C) val = x[((long long)gi * C + gj) * B + s];
            tile[li][lj] = val;
        }
        __syncthreads();
        const int li = threadIdx.x / kTile, lj = threadIdx.x % kTile;
        const int i = i0 + li, j = j0 + lj;
        if (i < R && j < C) {
#define XT(a, b) ((double)tile[(a) - i0 + 1][(b) - j0 + 1])
            double gv = 0.0;
            if (i <= R - 2 && j <= C - 2) {
                const double x00 = XT(i, j), x10 = XT(i + 1, j), x01 = XT(i, j + 1);
                const double tau = tv_tau(x00, x10, x01, pp.tv_eps2);
                v[1] = tau;
                if (tau > 0.0) gv -= ((x10 - x00) + (x01 - x00)) / tau;
            }
            if (i >= 1 && j <= C - 2) { // term (i-1, j): this pixel is its +1 row neighbour
                const double x00 = XT(i - 1, j), x10 = XT(i, j), x01 = XT(i - 1, j + 1);
                const double tau = tv_tau(x00, x10, x01, pp.tv_eps2);
                if (tau > 0.0) gv += (x10 - x00) / tau;
            }
            if (j >= 1 && i <= R - 2) { // term (i, j-1): this pixel is its +1 column neighbour
                const double x00 = XT(i, j - 1), x10 = XT(i + 1, j - 1), x01 = XT(i, j);
                const double tau = tv_tau(x00, x10, x01, pp.tv_eps2);
                if (tau > 0.0) gv += (x01 - x00) / tau;
            }
#undef XT
            if (!eval_only) {
                const float gf = (float)gv;
                g[((long long)i * C + j) * B + s] = gf;
                v[0] = (double)gf * (double)gf;
            }
        }
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        const long long nslots = (long long)gridDim.x * gridDim.y, slot = (long long)s * gridDim.x + blockIdx.x;
        partials[slot] = v[0];
        partials[nslots + slot] = v[1];
    }
}

// Squared norm (g = 2x), L1 norm (g = sign x) and linear objective (g = c) versions.
// With part_min (squared norm and L1, for k_trial_line) g receives x itself
// instead of the gradient, and part_min the least nonzero |x_j| per workgroup.
__global__ __launch_bounds__(kBlock) void k_phase_flat(const float *__restrict__ x, float *__restrict__ g,
                                                       const float *__restrict__ lin_c,
                                                       const SliceState *__restrict__ st, PertParams pp,
                                                       int eval_only, double *__restrict__ partials,
                                                       double *__restrict__ part_min)
{
    __shared__ double lds[4 * 2];
    const int s = blockIdx.y, B = pp.B;
    const bool live = eval_only ? true : st[s].live != 0;
    double v[2] = {0.0, 0.0}, least = INFINITY;
    if (live) {
        for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < pp.n; j += (long long)gridDim.x * kBlock) {
            const double xj = (double)x[j * B + s];
            if (pp.obj == OBJ_SQNORM) {
                v[1] += xj * xj;
                if (!eval_only) {
                    const float gf = (float)(2.0 * xj);
                    g[j * B + s] = part_min ? (float)xj : gf;
                    v[0] += (double)gf * (double)gf;
                }
            } else if (pp.obj == OBJ_L1) { // subgradient sign(x), 0 at 0
                v[1] += fabs(xj);
                if (!eval_only) {
                    const float gf = xj > 0.0 ? 1.f : (xj < 0.0 ? -1.f : 0.f);
                    g[j * B + s] = part_min ? (float)xj : gf;
                    v[0] += (double)gf * (double)gf;
                    if (gf != 0.f) least = fmin(least, fabs(xj));
                }
            } else { // OBJ_LINEAR
                const double cj = (double)lin_c[j];
                v[1] += cj * xj;
                v[0] += cj * cj;
            }
        }
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        const long long nslots = (long long)gridDim.x * gridDim.y, slot = (long long)s * gridDim.x + blockIdx.x;
        partials[slot] = v[0];
        partials[nslots + slot] = v[1];
    }
    if (part_min) {
        for (int off = 32; off > 0; off >>= 1) least = fmin(least, __shfl_xor(least, off, 64));
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = least;
        __syncthreads();
        if (threadIdx.x == 0)
            part_min[(long long)s * gridDim.x + blockIdx.x] = fmin(fmin(lds[0], lds[1]), fmin(lds[2], lds[3]));
    }
}

// Query: the proximity from pass 1's partials (query mode) to out[s], the
// objective from k_phase_*'s in eval_only mode to out[B + s]: one workgroup
// per slice (blockIdx.x) and value (blockIdx.y; 1 only where there is an
// objective).  out is pinned host memory, so the host needs no copy after this
// launch.  Two launches of one workgroup, slice after slice, and a copy to
// pageable memory made a query of 128 x 128 CT 55.5 us against 44.8.
__global__ __launch_bounds__(kBlock) void k_query_out(SliceState *__restrict__ st, int B,
                                                      const double *__restrict__ part_prox, int nparts,
                                                      const double *__restrict__ part_obj, int nt,
                                                      double *__restrict__ out)
{
    __shared__ double lds[4];
    __shared__ double tot[kTrialChunk];
    const int s = blockIdx.x;
    double v;
    if (blockIdx.y == 0) {
        double sum[1];
        sum_slots<1>(part_prox, (long long)s * nparts, nparts, sum, lds);
        v = 0.5 * sum[0];
    } else {
        chunk_totals<kBlock>(part_obj, (long long)B * nt, s, nt, 0, 2, tot);
        v = tot[1];
    }
    if (threadIdx.x == 0) {
        out[blockIdx.y * B + s] = v;
        if (!isfinite(v)) st[s].nonfinite = 1; // both workgroups of a slice store 1
    }
}

// Trial launch for TV (kTrialBlock threads per 16 x 16 tile): derive the
// state, then evaluate tau at z = x + (s_acc + beta_t) v for every trial t of
// this launch and every pixel term of the tile (one partial per trial per
// tile); or, once the phase is over, add s_acc v to the tile.  Wave w takes
// trials w*4 .. w*4+3, then the next 4 * (waves) trials, and so on; lane l of a
// wave takes pixels l, l+64, l+128, l+192 of the tile, adds its terms in that
// order, and wave_sum adds the lanes: each trial's tile sum is made by one
// wave, with no workgroup barrier, and the 16 waves keep the float64 square
// roots of different trials in flight together.
__global__ __launch_bounds__(kTrialBlock) void k_trial_tv(float *__restrict__ x, const float *__restrict__ g,
                                                          const SliceState *__restrict__ st_in,
                                                          SliceState *__restrict__ st_out, PertParams pp, int first,
                                                          int after, const double *__restrict__ part_prev,
                                                          double *__restrict__ part_out)
{
    static_assert(kTile * kTile == 256, "tile of 256 pixels");
    __shared__ float tx[kTile + 1][kTile + 2];
    __shared__ float tg[kTile + 1][kTile + 2];
    __shared__ double coef[1024];
    __shared__ double tot[kTrialChunk];
    __shared__ SliceState sS;
    __shared__ StepWindow win;
    constexpr int W = kTrialBlock / 64;
    const int s = blockIdx.y, B = pp.B, nt = gridDim.x;
    const int R = pp.tv_rows, C = pp.tv_cols;
    const int tiles_x = (C + kTile - 1) / kTile;
    const int i0 = (blockIdx.x / tiles_x) * kTile, j0 = (blockIdx.x % tiles_x) * kTile;
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // the tile of x and g (with its +1 row and column) is loaded while the state
    // is derived
    constexpr int TE = (kTile + 1) * (kTile + 1);
    static_assert(TE <= kTrialBlock, "one tile element per thread");
    float pxv = 0.f, pgv = 0.f;
    {
        const int e = threadIdx.x;
        const int gi = i0 + e / (kTile + 1), gj = j0 + e % (kTile + 1);
        if (e < TE && gi < R && gj < C) {
            pxv = x[((long long)gi * C + gj) * B + s];
            pgv = g[((long long)gi * C + gj) * B + s];
        }
    }
    derive_state<kTrialBlock>(sS, st_in, pp, first, part_prev, s, nt, tot, win, after);
    const SliceState &S = sS; // read from LDS (a register copy of the struct spills)
    const bool apply = must_apply(S);
    const int ntr = apply ? 0 : trial_width(S, pp, after);
    if (!apply && ntr == 0) {
        publish_state(S, st_out, s, false);
        return;
    }
    if (threadIdx.x < TE) {
        tx[threadIdx.x / (kTile + 1)][threadIdx.x % (kTile + 1)] = pxv;
        tg[threadIdx.x / (kTile + 1)][threadIdx.x % (kTile + 1)] = pgv;
    }
    if (apply) { // x and g at a pixel are the tile's (no other workgroup writes them)
        __syncthreads();
        if (threadIdx.x < kTile * kTile) {
            const int li = threadIdx.x / kTile, lj = threadIdx.x % kTile;
            const int i = i0 + li, j = j0 + lj;
            if (i < R && j < C) {
                const long long e = ((long long)i * C + j) * B + s;
                x[e] = (float)((double)tx[li][lj] + S.s_acc * (-(double)tg[li][lj] * (1.0 / S.gn)));
            }
        }
        publish_state(S, st_out, s, true);
        return;
    }
    publish_state(S, st_out, s, false);
    const long long nslots = (long long)B * nt, slot = (long long)s * nt + blockIdx.x;
    const double inv_gn = 1.0 / S.gn;
    for (int t = threadIdx.x; t < ntr; t += kTrialBlock) coef[t] = S.s_acc + step_of(win, pp, S, S.ell + t);
    __syncthreads();
    double x00[4], x10[4], x01[4], v00[4], v10[4], v01[4];
    bool has[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int pix = lane + 64 * h;
        const int li = pix / kTile, lj = pix % kTile;
        const int i = i0 + li, j = j0 + lj;
        has[h] = (i <= R - 2) && (j <= C - 2);
        x00[h] = tx[li][lj];
        x10[h] = tx[li + 1][lj];
        x01[h] = tx[li][lj + 1];
        v00[h] = -(double)tg[li][lj] * inv_gn;
        v10[h] = -(double)tg[li + 1][lj] * inv_gn;
        v01[h] = -(double)tg[li][lj + 1] * inv_gn;
    }
    if (ntr <= W) { // short batches: one trial a wave, so that no wave holds four trials' chains
        if (wid < ntr) {
            const double cf = coef[wid];
            double acc[1] = {0.0};
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (has[h])
                    acc[0] += tv_tau(x00[h] + cf * v00[h], x10[h] + cf * v10[h], x01[h] + cf * v01[h], pp.tv_eps2);
            wave_sum<1>(acc);
            if (lane == 0) part_out[(long long)wid * nslots + slot] = acc[0];
        }
        return;
    }
    for (int t0 = wid * 4; t0 < ntr; t0 += W * 4) {
        double acc[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            acc[k] = 0.0;
            if (t0 + k < ntr) {
                const double cf = coef[t0 + k];
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    if (has[h])
                        acc[k] += tv_tau(x00[h] + cf * v00[h], x10[h] + cf * v10[h], x01[h] + cf * v01[h],
                                         pp.tv_eps2);
            }
        }
        wave_sum<4>(acc);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (t0 + k < ntr) part_out[(long long)(t0 + k) * nslots + slot] = acc[k];
        }
    }
}

// -- TV2D for several slices: one workgroup takes a tile's pixels of every
//    slice, thread t slice t mod B of pixel t / B, then of the pixel
//    blockDim / B further on, ...  The layout is slice-interleaved, so a
//    wave's loads are whole cache lines; with a workgroup per (tile, slice),
//    as for one slice, each read 4 bytes of a line that B workgroups fetch
//    (B = 32 at 256 x 256: 124 us a trial launch, 25 us the gradient).  From
//    512 such pairs on (tv_whole_lines).
//    The tiles are kTile wide and tv_tile_rows(pp) high: 16 rows on large
//    images, fewer while that leaves the device with under 256 workgroups.

// Threads of such a workgroup: 256 for small tiles, whose barriers and
// reductions over 16 waves would outweigh the pixels.
constexpr int kTrialSmallBlock = 256;
static inline bool tv_small_block(const PertParams &pp) { return tv_tile_rows(pp) * kTile * pp.B < 2048; }

// Sums per slice over a workgroup of BS threads (thread t holds slice t mod
// B): the total of value v and slice s is returned to thread v * B + s.
// red holds (BS/64) * NV * B doubles; barriers inside.
template <int NV, int B, int BS>
__device__ inline double block_sum_slices(double (&v)[NV], double *red)
{
    static_assert(NV * B <= BS, "one total a thread");
#pragma unroll
    for (int off = B; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], off, 64);
    const int wid = threadIdx.x >> 6, wl = threadIdx.x & 63;
    __syncthreads(); // the previous use of red is over
    if (wl < B) {
#pragma unroll
        for (int k = 0; k < NV; ++k) red[(wid * NV + k) * B + wl] = v[k];
    }
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < NV * B) {
        for (int w = 0; w < BS / 64; ++w) t += red[w * NV * B + threadIdx.x];
    }
    return t;
}

template <int B, int BS>
__global__ __launch_bounds__(BS) void k_phase_tv_mm(const float *__restrict__ x, float *__restrict__ g,
                                                    const SliceState *__restrict__ st, PertParams pp, int th,
                                                    int eval_only, double *__restrict__ partials)
{
    constexpr int PX = BS / B;
    __shared__ double red[BS / 64 * 2 * B];
    const int s = threadIdx.x & (B - 1);
    const int R = pp.tv_rows, C = pp.tv_cols;
    const int tiles_x = (C + kTile - 1) / kTile;
    const int i0 = (blockIdx.x / tiles_x) * th, j0 = (blockIdx.x % tiles_x) * kTile;
    double v[2] = {0.0, 0.0}; // sum g^2, f
    if (eval_only || st[s].live != 0) {
        for (int pl = threadIdx.x / B; pl < th * kTile; pl += PX) {
            const int i = i0 + pl / kTile, j = j0 + pl % kTile;
            if (i >= R || j >= C) continue;
            const long long e = ((long long)i * C + j) * B + s, up = (long long)C * B;
            const bool here = i <= R - 2 && j <= C - 2, above = i >= 1 && j <= C - 2, left = j >= 1 && i <= R - 2;
            const double x00 = (double)x[e];
            double x10 = 0.0, x01 = 0.0, xm0 = 0.0, xm1 = 0.0, x0m = 0.0, x1m = 0.0;
            if (i <= R - 2) x10 = (double)x[e + up];
            if (j <= C - 2) x01 = (double)x[e + B];
            if (above) {
                xm0 = (double)x[e - up];
                xm1 = (double)x[e - up + B];
            }
            if (left) {
                x0m = (double)x[e - B];
                x1m = (double)x[e + up - B];
            }
            double gv = 0.0;
            if (here) {
                const double tau = tv_tau(x00, x10, x01, pp.tv_eps2);
                v[1] += tau;
                if (tau > 0.0) gv -= ((x10 - x00) + (x01 - x00)) / tau;
            }
            if (above) { // term (i-1, j): this pixel is its +1 row neighbour
                const double tau = tv_tau(xm0, x00, xm1, pp.tv_eps2);
                if (tau > 0.0) gv += (x00 - xm0) / tau;
            }
            if (left) { // term (i, j-1): this pixel is its +1 column neighbour
                const double tau = tv_tau(x0m, x1m, x00, pp.tv_eps2);
                if (tau > 0.0) gv += (x00 - x0m) / tau;
            }
            if (!eval_only) {
                const float gf = (float)gv;
                g[e] = gf;
                v[0] += (double)gf * (double)gf;
            }
        }
    }
    const double t = block_sum_slices<2, B, BS>(v, red);
    if (threadIdx.x < 2 * B) // value-major partials, slot (slice, tile)
        partials[(long long)threadIdx.x * gridDim.x + blockIdx.x] = t;
}

// Totals over the nt tiles of rows (value v0 + r / B, slice r mod B), r < nv *
// B, into tot[r] (LDS): row by row within a wave, lane l adding tiles l, l +
// 64, ... in order and wave_sum the lanes.  Every thread must call it.
template <int B, int BS>
__device__ inline void slice_totals(const double *__restrict__ part, int nt, int v0, int nv, double *tot)
{
    constexpr int W = BS / 64, Q = 4; // rows a wave sums at a time
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63, rows = nv * B;
    const double *p = part + (long long)v0 * B * nt;
    for (int r0 = wid; r0 < rows; r0 += W * Q) { // the same in every lane
        double a[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) a[q] = 0.0;
        for (int b = lane; b < nt; b += 64) {
#pragma unroll
            for (int q = 0; q < Q; ++q) a[q] += p[(long long)min(r0 + q * W, rows - 1) * nt + b];
        }
        wave_sum<Q>(a);
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (r0 + q * W < rows) tot[r0 + q * W] = a[q];
        }
    }
    __syncthreads();
}

// Trial launch for TV with several slices: k_trial_tv's decisions for every
// slice (thread s < B holds slice s's), then each slice either evaluates its
// next batch of trials or gets its accepted step, whichever its state asks
// for.  The totals a decision needs are read one trial first (usually
// accepted), the rest of the batch only while a slice is undecided.  `after`:
// evaluating launches behind this one; -1 in the phase's closing launch.
template <int B, int BS>
__global__ __launch_bounds__(BS) void k_trial_tv_mm(float *__restrict__ x, const float *__restrict__ g,
                                                    const SliceState *__restrict__ st_in,
                                                    SliceState *__restrict__ st_out, PertParams pp, int th,
                                                    int first, int after, const double *__restrict__ part_prev,
                                                    double *__restrict__ part_out)
{
    constexpr int PX = BS / B, T = 8; // trials evaluated at a time
    static_assert(sizeof(SliceState) % 8 == 0, "copied by words");
    static_assert(T * B <= BS, "one trial and slice a thread");
    __shared__ SliceState sS[B];
    __shared__ double tot[T * B];
    __shared__ double coef[T * B];
    __shared__ double red[BS / 64 * T * B];
    __shared__ int most; // trials the widest slice evaluates
    const int s = threadIdx.x & (B - 1), nt = gridDim.x;
    const int R = pp.tv_rows, C = pp.tv_cols;
    const int tiles_x = (C + kTile - 1) / kTile;
    const int i0 = (blockIdx.x / tiles_x) * th, j0 = (blockIdx.x % tiles_x) * kTile;
    {
        const unsigned long long *src = reinterpret_cast<const unsigned long long *>(st_in);
        unsigned long long *dst = reinterpret_cast<unsigned long long *>(sS);
        for (int k = threadIdx.x; k < (int)(B * sizeof(SliceState) / 8); k += BS) dst[k] = src[k];
    }
    if (threadIdx.x == 0) most = 0;
    if (first) {
        slice_totals<B, BS>(part_prev, nt, 0, 2, tot); // its barrier also publishes sS
        if (threadIdx.x < B) open_phase_state(sS[threadIdx.x], pp, tot[threadIdx.x], tot[B + threadIdx.x]);
        __syncthreads();
    } else {
        __syncthreads();
        int ntr = 0, acc_t = -1;
        double acc_f = 0.0;
        bool need = false;
        if (threadIdx.x < B) {
            ntr = trial_width(sS[threadIdx.x], pp, after + 1); // as the launch before this one saw it
            need = ntr > 0;
        }
        for (int t0 = 0, nv = 1; __syncthreads_or(need); t0 += nv, nv = T) { // ends: t0 passes every ntr
            slice_totals<B, BS>(part_prev, nt, t0, min(nv, pp.max_trials - t0), tot);
            if (need) {
                for (int w = 0; w < nv && t0 + w < ntr; ++w)
                    if (tot[w * B + threadIdx.x] <= sS[threadIdx.x].f_cur) {
                        acc_t = t0 + w;
                        acc_f = tot[w * B + threadIdx.x];
                        break;
                    }
                need = acc_t < 0 && t0 + nv < ntr;
            }
        }
        if (threadIdx.x < B && ntr > 0) {
            SliceState &D = sS[threadIdx.x];
            record_decision(D, pp, ntr, acc_t, acc_f, acc_t >= 0 ? trial_beta(pp, D, D.ell + acc_t) : 0.0);
        }
        __syncthreads();
    }
    const SliceState &S = sS[s];
    const bool apply = must_apply(S);
    const int ntr = (after >= 0 && !apply) ? trial_width(S, pp, after) : 0;
    if (threadIdx.x < B && ntr > 0) atomicMax(&most, ntr);
    if (blockIdx.x == 0 && threadIdx.x < B) {
        SliceState o = S;
        if (apply) o.applied = 1;
        st_out[threadIdx.x] = o;
    }
    const double inv_gn = 1.0 / S.gn, s_acc = S.s_acc;
    if (apply) { // x and g of this tile and slice: no other workgroup reads or writes them in this launch
        for (int pl = threadIdx.x / B; pl < th * kTile; pl += PX) {
            const int i = i0 + pl / kTile, j = j0 + pl % kTile;
            if (i < R && j < C) {
                const long long e = ((long long)i * C + j) * B + s;
                x[e] = (float)((double)x[e] + s_acc * (-(double)g[e] * inv_gn));
            }
        }
    }
    __syncthreads();
    const long long nslots = (long long)B * nt;
    for (int t0 = 0; t0 < most; t0 += T) {
        if (threadIdx.x < T * B) { // trial t0 + k of slice s
            const int k = threadIdx.x / B;
            coef[threadIdx.x] = t0 + k < ntr ? s_acc + trial_beta(pp, S, S.ell + t0 + k) : 0.0;
        }
        __syncthreads();
        double cf[T], acc[T];
#pragma unroll
        for (int k = 0; k < T; ++k) {
            cf[k] = coef[k * B + s];
            acc[k] = 0.0;
        }
        const int nk = ntr - t0;
        if (nk > 0) {
            for (int pl = threadIdx.x / B; pl < th * kTile; pl += PX) {
                const int i = i0 + pl / kTile, j = j0 + pl % kTile;
                if (i > R - 2 || j > C - 2) continue;
                const long long e = ((long long)i * C + j) * B + s, up = (long long)C * B;
                const double x00 = (double)x[e], x10 = (double)x[e + up], x01 = (double)x[e + B];
                const double v00 = -(double)g[e] * inv_gn, v10 = -(double)g[e + up] * inv_gn,
                             v01 = -(double)g[e + B] * inv_gn;
#pragma unroll
                for (int k = 0; k < T; ++k)
                    if (k < nk)
                        acc[k] += tv_tau(x00 + cf[k] * v00, x10 + cf[k] * v10, x01 + cf[k] * v01, pp.tv_eps2);
            }
        }
        const double t = block_sum_slices<T, B, BS>(acc, red); // its barriers also end this chunk's use of coef
        const int k = threadIdx.x / B;
        if (threadIdx.x < T * B && t0 + k < ntr)
            part_out[(long long)(t0 + k) * nslots + (long long)s * nt + blockIdx.x] = t;
    }
}

// Closing launch of a phase: the decision of the last trial launch and, when
// the phase ends there, the accepted step added to x (the same arithmetic as
// the trial launches' own apply), each workgroup on its own part of x.  Where
// an earlier trial launch has applied the step already, the launch only
// carries the state over (workgroup 0 publishes it).  nt: workgroups per slice
// of the trial launches (their partials' layout).
__global__ __launch_bounds__(kTrialBlock) void k_trial_close(float *__restrict__ x, const float *__restrict__ g,
                                                             const SliceState *__restrict__ st_in,
                                                             SliceState *__restrict__ st_out, PertParams pp, int nt,
                                                             const double *__restrict__ part_prev)
{
    __shared__ double tot[kTrialChunk];
    __shared__ SliceState sS;
    const int s = blockIdx.y, B = pp.B;
    const bool lin = pp.obj == OBJ_LINEAR;
    __shared__ StepWindow win;
    derive_state<kTrialBlock>(sS, st_in, pp, 0, part_prev, s, nt, tot, win, -1);
    const SliceState &S = sS;
    const bool apply = must_apply(S);
    if (apply) {
        const double inv_gn = 1.0 / S.gn;
        for (long long j = (long long)blockIdx.x * kTrialBlock + threadIdx.x; j < pp.n;
             j += (long long)gridDim.x * kTrialBlock) {
            const double gj = lin ? (double)g[j] : (double)g[j * B + s];
            x[j * B + s] = (float)((double)x[j * B + s] + S.s_acc * (-gj * inv_gn));
        }
    }
    publish_state(S, st_out, s, apply);
}

// Trials of a flat objective valued along the line x + t v, v = -g/||g||,
// where f is known from the direction's sums (f0 = f(x), gsq = ||g||^2):
//   f = c^T x       f0 - t ||g||,
//   f = ||x||^2     (1 - 2t/||g||)^2 f0,
//   f = ||x||_1     f0 - t gsq/||g|| while t/||g|| <= least, the least nonzero
//                   |x_j| (no entry changes sign).
// Wave 0 (all 64 lanes) calls it: lane l values the l-th next trial, the first
// acceptable one in order is recorded, and so on until the phase is over (0
// is returned) or a trial's value is not known (the trials the caller has to
// sum before calling again).  The power law's steps are those of the window,
// and formed once per 64 trials beyond it.  Ends: a round accepts a trial, rejects at least one, or returns.
template <int OBJ>
__device__ inline int line_trials(SliceState &sS, const PertParams &pp, const StepWindow &win, double f0, double gsq,
                                  double least, int most)
{
    const int l = threadIdx.x & 63;
    long long base = win.base; // beta holds the steps of trials base .. base + 63
    double beta = win.beta[l];
    bool formed = !pp.adaptive && sS.ell >= base;
    while (sS.phase) {
        if (!formed || sS.ell - base >= 64) {
            base = sS.ell;
            beta = trial_beta(pp, sS, base + l);
            formed = true;
        }
        const int off = (int)(sS.ell - base), left = pp.max_trials - sS.step_tried, nb = min(left, 64 - off);
        const double t = sS.s_acc + __shfl(beta, (off + l) & 63, 64), gn = sS.gn;
        double ft;
        bool known = true;
        if constexpr (OBJ == OBJ_LINEAR) {
            ft = f0 - t * gn;
        } else if constexpr (OBJ == OBJ_SQNORM) {
            const double a = 1.0 - 2.0 * t / gn;
            ft = f0 * a * a;
        } else {
            known = t <= least * gn;
            ft = f0 - t * (gsq / gn);
        }
        const unsigned long long ok = __ballot(l < nb && known && ft <= sS.f_cur), un = __ballot(l < nb && !known);
        const int a = ok ? __ffsll(ok) - 1 : 64, u = un ? __ffsll(un) - 1 : 64;
        if (u < a) return min(most, left);
        const double fa = __shfl(ft, a & 63, 64), ba = __shfl(beta, (off + a) & 63, 64);
        __threadfence_block(); // every lane has read the state ...
        __builtin_amdgcn_wave_barrier();
        if (l == 0) record_decision(sS, pp, nb, a < 64 ? a : -1, fa, ba);
        __threadfence_block(); // ... and reads it anew
        __builtin_amdgcn_wave_barrier();
    }
    return 0;
}

// The decision on ntr trials from each thread's share acc of their objectives
// (every thread of the workgroup calls it; lds holds (BS/64) * T doubles).
template <int T, int BS>
__device__ inline void sum_and_record(SliceState &sS, const PertParams &pp, const StepWindow &win, double (&acc)[T],
                                      int ntr, double *lds)
{
    block_sum<T, BS>(acc, lds);
    if (threadIdx.x != 0) return;
    int t = -1;
    for (int w = 0; w < ntr; ++w)
        if (acc[w] <= sS.f_cur) {
            t = w;
            break;
        }
    record_decision(sS, pp, ntr, t, t >= 0 ? acc[t] : 0.0, t >= 0 ? step_of(win, pp, sS, sS.ell + t) : 0.0);
}

// The phase of the linear objective f(x) = c^T x from its direction partials
// (sum c_j^2 and sum c_j x_j per workgroup of the launch that left them).  On
// v = -c/||c|| the objective at a trial point is known in closed form,
// f(x + t v) = f(x) - t ||c||, so no trial needs a pass over x: every
// workgroup opens the phase from the partials (the same sums in the same
// order) and runs the reduction steps' trials on those values; workgroup 0
// publishes the state.  Returns whether the accepted step s v is to be added.
constexpr int kPhaseSums = 2; // the totals a phase opens from
// What the fused kernels hold beside z and y: block_sum's words, and the phase's
// totals, state and steps.
static_assert(sizeof(double) * (kFusedBlock / 64 + kPhaseSums) + sizeof(SliceState) + sizeof(StepWindow) <=
                  kFusedStaticLds,
              "the fused pass's limit on n leaves this much");
template <int BS>
__device__ inline bool linear_phase(SliceState &sS, const SliceState *__restrict__ st_in, const PertParams &pp,
                                   const double *__restrict__ part, int s, int nt, double *tot,
                                   SliceState *__restrict__ st_out)
{
    __shared__ StepWindow win;
    derive_state<BS>(sS, st_in, pp, 1, part, s, nt, tot, win);
    if (threadIdx.x < 64) (void)line_trials<OBJ_LINEAR>(sS, pp, win, tot[1], tot[0], 0.0, 0);
    __syncthreads();
    const bool apply = must_apply(sS);
    publish_state(sS, st_out, s, apply);
    return apply;
}

// The linear phase in one launch: each workgroup adds the step to its own
// part of x.
__global__ __launch_bounds__(kBlock) void k_trial_linear(float *__restrict__ x, const float *__restrict__ c,
                                                         const SliceState *__restrict__ st_in,
                                                         SliceState *__restrict__ st_out, PertParams pp,
                                                         const double *__restrict__ part_phase)
{
    __shared__ double tot[kPhaseSums];
    __shared__ SliceState sS;
    const int s = blockIdx.y, B = pp.B, nt = gridDim.x;
    if (linear_phase<kBlock>(sS, st_in, pp, part_phase, s, nt, tot, st_out)) {
        const double inv_gn = 1.0 / sS.gn, s_acc = sS.s_acc;
        for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < pp.n; j += (long long)gridDim.x * kBlock)
            x[j * B + s] = linear_step_point(x[j * B + s], c[j], s_acc, inv_gn);
    }
}

// The phase of the squared norm or the L1 norm in one launch after the
// direction launch (k_phase_flat with part_min, which also left a copy xc of
// x): the trials valued along the line (line_trials); where ||x||_1 is not
// known there it is summed over xc, trials in batches as in k_phase_small,
// by every workgroup alike.  So each workgroup takes the same decisions in
// the same order, adds the accepted step to its own part of x, reading xc
// (another workgroup may have moved its part of x already), and workgroup 0
// publishes the state.  The chain this replaces took up to two launches a
// reduction step: on n = 16,384 with four steps ten launches, 80 us, against
// 14.5 us for these two.
template <int OBJ>
__global__ __launch_bounds__(kTrialBlock) void k_trial_line(float *__restrict__ x, const float *__restrict__ xc,
                                                            const SliceState *__restrict__ st_in,
                                                            SliceState *__restrict__ st_out, PertParams pp,
                                                            const double *__restrict__ part,
                                                            const double *__restrict__ part_min, int nt)
{
    constexpr int BS = kTrialBlock, T = kSmallTrials;
    __shared__ double tot[kTrialChunk];
    __shared__ double lds[(BS / 64) * T];
    __shared__ double coef[T];
    __shared__ SliceState sS;
    __shared__ StepWindow win;
    __shared__ int summed; // trials the next batch sums over xc (0: decided in closed form)
    const int s = blockIdx.y, B = pp.B;
    const int n = (int)pp.n;
    double least = INFINITY; // wave 0: least nonzero |x_j|
    if (OBJ == OBJ_L1 && threadIdx.x < 64) {
        for (int b = threadIdx.x; b < nt; b += 64) least = fmin(least, part_min[(long long)s * nt + b]);
        for (int off = 32; off > 0; off >>= 1) least = fmin(least, __shfl_xor(least, off, 64));
    }
    derive_state<BS>(sS, st_in, pp, 1, part, s, nt, tot, win);
    const double gsq = tot[0], f0 = tot[1];
    phase_rounds(
        threadIdx.x < 64, summed, [&] { return line_trials<OBJ>(sS, pp, win, f0, gsq, least, T); },
        [&](int ntr) {
            if (threadIdx.x < ntr) coef[threadIdx.x] = sS.s_acc + step_of(win, pp, sS, sS.ell + threadIdx.x);
            __syncthreads();
            const double inv_gn = 1.0 / sS.gn;
            double acc[T], cw[T];
#pragma unroll
            for (int w = 0; w < T; ++w) {
                acc[w] = 0.0;
                cw[w] = w < ntr ? coef[w] : 0.0;
            }
#pragma unroll 4
            for (int j = threadIdx.x; j < n; j += BS) {
                const double xj = (double)xc[(long long)j * B + s];
                const double vj = xj > 0.0 ? -inv_gn : (xj < 0.0 ? inv_gn : 0.0);
#pragma unroll
                for (int w = 0; w < T; ++w) acc[w] += fabs(xj + cw[w] * vj);
            }
            sum_and_record<T, BS>(sS, pp, win, acc, ntr, lds);
        },
        [] { __syncthreads(); });
    const bool apply = must_apply(sS);
    publish_state(sS, st_out, s, apply);
    if (apply) {
        const double inv_gn = 1.0 / sS.gn, s_acc = sS.s_acc;
        for (int j = blockIdx.x * BS + threadIdx.x; j < n; j += gridDim.x * BS) {
            const float xf = xc[(long long)j * B + s];
            const double gj = OBJ == OBJ_SQNORM ? 2.0 * (double)xf : (xf > 0.f ? 1.0 : (xf < 0.f ? -1.0 : 0.0));
            x[(long long)j * B + s] = (float)((double)xf + s_acc * (-gj * inv_gn));
        }
    }
}

// Compare-exchange stage of a bitonic sort of 1,024 keys, four consecutive ones
// a thread of a 256-thread workgroup (key i = 4 thread + e): partners `stride`
// apart, runs of `size`.  ex (LDS, 1,024 words) for partners in other waves.
template <int SIZE, int STRIDE>
__device__ inline void sort_stage(unsigned (&k)[4], unsigned *ex)
{
    const int i0 = (int)threadIdx.x * 4;
    const bool up = (i0 & SIZE) == 0; // SIZE >= 4: the same for a thread's keys
    if constexpr (STRIDE < 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((e & STRIDE) == 0) {
                const bool asc = SIZE < 4 ? (e & SIZE) == 0 : up;
                const unsigned lo = min(k[e], k[e ^ STRIDE]), hi = max(k[e], k[e ^ STRIDE]);
                k[e] = asc ? lo : hi;
                k[e ^ STRIDE] = asc ? hi : lo;
            }
    } else {
        const bool low = (i0 & STRIDE) == 0;
        unsigned o[4];
        if constexpr (STRIDE < 256) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = __shfl_xor(k[e], STRIDE / 4, 64);
        } else {
            __syncthreads(); // the previous stage's reads of ex are over
#pragma unroll
            for (int e = 0; e < 4; ++e) ex[e * kBlock + threadIdx.x] = k[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = ex[e * kBlock + (threadIdx.x ^ (STRIDE / 4))];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) k[e] = low == up ? min(k[e], o[e]) : max(k[e], o[e]);
    }
}
template <int SIZE, int STRIDE>
__device__ inline void sort_merge(unsigned (&k)[4], unsigned *ex)
{
    sort_stage<SIZE, STRIDE>(k, ex);
    if constexpr (STRIDE > 1) sort_merge<SIZE, STRIDE / 2>(k, ex);
}
template <int SIZE>
__device__ inline void sort_chunk(unsigned (&k)[4], unsigned *ex)
{
    if constexpr (SIZE > 2) sort_chunk<SIZE / 2>(k, ex);
    sort_merge<SIZE, SIZE / 2>(k, ex);
}

// Direction launch of the L1 norm for k_trial_sorted (one slice, a workgroup a
// chunk of kLineChunk entries): k_phase_flat's partials of ||g||^2 (the nonzero
// entries), f(x) and the least nonzero |x_j|, and the chunk's |x_j| sorted, as
// bit patterns, which order as the nonnegative numbers do; zeros, NaN and what
// lies past n become infinities, which no trial reaches.
__global__ __launch_bounds__(kBlock) void k_phase_sorted(const float *__restrict__ x, int n,
                                                         const SliceState *__restrict__ st, LineSorted L,
                                                         double *__restrict__ partials, double *__restrict__ part_min)
{
    static_assert(kLineChunk == 4 * kBlock && kLineBucket % 4 == 0, "four keys a thread");
    __shared__ unsigned ex[kLineChunk];
    __shared__ double lds[4 * 2];
    const int b = blockIdx.x, nt = gridDim.x, j0 = b * kLineChunk + (int)threadIdx.x * 4;
    const bool live = st[0].live != 0; // the same in every thread
    float xf[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) xf[e] = 0.f;
    if (live) {
        if (j0 + 4 <= n) {
            const float4 v4 = *reinterpret_cast<const float4 *>(x + j0);
            xf[0] = v4.x; xf[1] = v4.y; xf[2] = v4.z; xf[3] = v4.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j0 + e < n) xf[e] = x[j0 + e];
        }
    }
    double v[2] = {0.0, 0.0}, least = INFINITY;
    unsigned k[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = fabsf(xf[e]);
        const bool nz = a > 0.f; // not a NaN
        v[0] += nz ? 1.0 : 0.0;
        v[1] += (double)a;
        if (nz) least = fmin(least, (double)a);
        k[e] = __float_as_uint(nz ? a : INFINITY);
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        partials[b] = v[0];
        partials[nt + b] = v[1];
    }
    for (int off = 32; off > 0; off >>= 1) least = fmin(least, __shfl_xor(least, off, 64));
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) lds[wid] = least;
    __syncthreads();
    if (threadIdx.x == 0) part_min[b] = fmin(fmin(lds[0], lds[1]), fmin(lds[2], lds[3]));
    if (!live) return;
    sort_chunk<kLineChunk>(k, ex);
    double sum = 0.0; // of the thread's finite keys, then of all before them
    float f[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[e] = __uint_as_float(k[e]);
        if (isfinite(f[e])) sum += (double)f[e];
    }
    double incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    double before = __shfl_up(incl, 1, 64);
    if (lane == 0) before = 0.0;
    if (lane == 63) lds[4 + wid] = incl;
    __syncthreads();
    for (int w = 0; w < wid; ++w) before += lds[4 + w];
    *reinterpret_cast<float4 *>(L.key + j0) = make_float4(f[0], f[1], f[2], f[3]);
    if (threadIdx.x % (kLineBucket / 4) == 0) {
        const int q = j0 / kLineBucket;
        L.pivot[q] = f[0];
        L.below[q] = before;
    }
}

// The L1 norm's phase in one launch after k_phase_sorted, as k_trial_line; past
// a change of sign
//   ||x + t v||_1 = f0 - t gsq/||g|| + 2 sum over 0 < |x_j| < tau of (tau - |x_j|),
// tau = t/||g||, and thread (trial, chunk) finds its chunk's count and sum of
// keys below tau: a search of the pivots (in LDS from the phase's first such
// batch on) and one bucket of keys, loaded at once.  Every workgroup takes the
// same decisions from the same sums, and adds the step to its part of x, which
// no other workgroup reads.  A batch is a chain of two loads out of L2 and two
// barriers, ~5 us whatever n; summed over x by every workgroup it was 15 us at n
// = 32,761 and 45 at 131,044 (an iteration of four steps there 207 us, now 69).
__global__ __launch_bounds__(kTrialBlock) void k_trial_sorted(float *__restrict__ x,
                                                              const SliceState *__restrict__ st_in,
                                                              SliceState *__restrict__ st_out, PertParams pp,
                                                              const double *__restrict__ part,
                                                              const double *__restrict__ part_min, LineSorted L,
                                                              int nt)
{
    constexpr int BS = kTrialBlock, T = kSmallTrials, Q = kLineMaxN / kLineChunk, P = kLineChunk / kLineBucket;
    static_assert(Q * T == BS && Q % 64 == 0, "a thread a trial and chunk, a wave of one trial");
    __shared__ float pivot[Q * P];
    __shared__ double below[Q * P];
    __shared__ double tot[kPhaseSums];
    __shared__ double wsum[BS / 64];
    __shared__ double coef[T];
    __shared__ SliceState sS;
    __shared__ StepWindow win;
    __shared__ int summed; // trials the next batch sums (0: the phase is over)
    double least = INFINITY; // wave 0: least nonzero |x_j|
    if (threadIdx.x < 64) {
        for (int b = threadIdx.x; b < nt; b += 64) least = fmin(least, part_min[b]);
        for (int off = 32; off > 0; off >>= 1) least = fmin(least, __shfl_xor(least, off, 64));
    }
    derive_state<BS>(sS, st_in, pp, 1, part, 0, nt, tot, win);
    const double gsq = tot[0], f0 = tot[1];
    const int w = threadIdx.x / Q, q = threadIdx.x % Q;
    bool staged = false;
    phase_rounds(
        threadIdx.x < 64, summed, [&] { return line_trials<OBJ_L1>(sS, pp, win, f0, gsq, least, T); },
        [&](int ntr) {
            if (!staged) { // the same in every thread
                for (int i = threadIdx.x; i < nt * P; i += BS) {
                    pivot[i] = L.pivot[i];
                    below[i] = L.below[i];
                }
                staged = true;
            }
            if (threadIdx.x < ntr) coef[threadIdx.x] = sS.s_acc + step_of(win, pp, sS, sS.ell + threadIdx.x);
            __syncthreads();
            double ex[1] = {0.0};
            if (w < ntr && q < nt) {
                const double tau = coef[w] / sS.gn;
                const float *pv = pivot + q * P;
                int c = 0; // pivots below tau
#pragma unroll
                for (int h = P / 2; h > 0; h >>= 1)
                    if ((double)pv[c + h - 1] < tau) c += h;
                if ((double)pv[c] < tau) ++c;
                if (c > 0) { // the keys before bucket c - 1 are below tau, and some of its own
                    const int bk = q * P + c - 1;
                    const float4 *key = reinterpret_cast<const float4 *>(L.key + (size_t)bk * kLineBucket);
                    float4 a[kLineBucket / 4];
#pragma unroll
                    for (int h = 0; h < kLineBucket / 4; ++h) a[h] = key[h];
                    double cnt = (double)((c - 1) * kLineBucket), sum = below[bk];
#pragma unroll
                    for (int h = 0; h < kLineBucket / 4; ++h) {
                        const float f[4] = {a[h].x, a[h].y, a[h].z, a[h].w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if ((double)f[e] < tau) {
                                cnt += 1.0;
                                sum += (double)f[e];
                            }
                    }
                    ex[0] = cnt * tau - sum;
                }
            }
            wave_sum<1>(ex);
            if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ex[0];
            __syncthreads();
            if (threadIdx.x == 0) {
                int acc = -1;
                double fa = 0.0;
                for (int t = 0; t < ntr && acc < 0; ++t) {
                    double e2 = 0.0;
                    for (int h = 0; h < Q / 64; ++h) e2 += wsum[t * (Q / 64) + h];
                    const double ft = f0 - coef[t] * (gsq / sS.gn) + 2.0 * e2;
                    if (ft <= sS.f_cur) {
                        acc = t;
                        fa = ft;
                    }
                }
                record_decision(sS, pp, ntr, acc, fa, acc >= 0 ? step_of(win, pp, sS, sS.ell + acc) : 0.0);
            }
        },
        [] { __syncthreads(); });
    const bool apply = must_apply(sS);
    publish_state(sS, st_out, 0, apply);
    if (apply) {
        const double inv_gn = 1.0 / sS.gn, s_acc = sS.s_acc;
        const int n = (int)pp.n;
        for (int j = blockIdx.x * BS + threadIdx.x; j < n; j += gridDim.x * BS) {
            const float xf = x[j];
            const double gj = xf > 0.f ? 1.0 : (xf < 0.f ? -1.0 : 0.0);
            x[j] = (float)((double)xf + s_acc * (-gj * inv_gn));
        }
    }
}

// Trial launch for the squared norm and the linear objective (flat vectors).
__global__ __launch_bounds__(kBlock) void k_trial_flat(float *__restrict__ x, const float *__restrict__ g,
                                                       const SliceState *__restrict__ st_in,
                                                       SliceState *__restrict__ st_out, PertParams pp, int first,
                                                       int after, const double *__restrict__ part_prev,
                                                       double *__restrict__ part_out)
{
    __shared__ double coef[1024];
    __shared__ double lds[4 * kTrialChunk];
    __shared__ double tot[kTrialChunk];
    __shared__ SliceState sS;
    __shared__ StepWindow win;
    const int s = blockIdx.y, B = pp.B, nt = gridDim.x;
    const bool lin = pp.obj == OBJ_LINEAR;
    derive_state<kBlock>(sS, st_in, pp, first, part_prev, s, nt, tot, win, after);
    const SliceState &S = sS; // read from LDS (a register copy of the struct spills)
    if (must_apply(S)) {
        const double inv_gn = 1.0 / S.gn;
        for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < pp.n; j += (long long)gridDim.x * kBlock) {
            const double gj = lin ? (double)g[j] : (double)g[j * B + s];
            x[j * B + s] = (float)((double)x[j * B + s] + S.s_acc * (-gj * inv_gn));
        }
        publish_state(S, st_out, s, true);
        return;
    }
    publish_state(S, st_out, s, false);
    // the same in every lane: in a scalar register the trials' conditions are branches, not masks (L1, 20M
    // unknowns, the first batch 201 us without)
    const int ntr = __builtin_amdgcn_readfirstlane(trial_width(S, pp, after));
    if (ntr == 0) return;
    const long long nslots = (long long)B * nt, slot = (long long)s * nt + blockIdx.x;
    const double inv_gn = 1.0 / S.gn;
    for (int t = threadIdx.x; t < ntr; t += kBlock) coef[t] = S.s_acc + step_of(win, pp, S, S.ell + t);
    __syncthreads();
    for (int t0 = 0; t0 < ntr; t0 += kTrialChunk) {
        double acc[kTrialChunk];
#pragma unroll
        for (int w = 0; w < kTrialChunk; ++w) acc[w] = 0.0;
        for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < pp.n; j += (long long)gridDim.x * kBlock) {
            const double xj = (double)x[j * B + s];
            const double gj = lin ? (double)g[j] : (double)g[j * B + s];
            const double vj = -gj * inv_gn;
#pragma unroll
            for (int w = 0; w < kTrialChunk; ++w) {
                if (t0 + w < ntr) {
                    const double z = xj + coef[t0 + w] * vj;
                    acc[w] += lin ? gj * z : (pp.obj == OBJ_L1 ? fabs(z) : z * z);
                }
            }
        }
        block_sum<kTrialChunk>(acc, lds);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 0; w < kTrialChunk; ++w)
                if (t0 + w < ntr) part_out[(long long)(t0 + w) * nslots + slot] = acc[w];
        }
    }
}

// The whole perturbation phase of a flat objective in one launch, for short
// vectors (n <= kSmallPhaseMaxN): one workgroup per slice copies its entries
// of x and of the direction into LDS (float32, 8n bytes), forms ||g||^2 and
// f(x^k), opens the phase, values the trials along the line (line_trials;
// L1 trials past a change of sign are summed from LDS, in batches of
// kSmallTrials), and adds the accepted step to x.  One workgroup is a latency
// chain, so every thread issues all of its U loads of x (and c) before using
// any.  Reads state st_in[s], writes st_out[s].
template <int OBJ, int U>
__global__ __launch_bounds__(kSmallPhaseBlock) void k_phase_small(float *__restrict__ x,
                                                                  const float *__restrict__ lin_c,
                                                                  const SliceState *__restrict__ st_in,
                                                                  SliceState *__restrict__ st_out, PertParams pp)
{
    constexpr int BS = kSmallPhaseBlock, T = kSmallTrials;
    extern __shared__ __align__(16) unsigned char phase_lds[];
    __shared__ double lds[(BS / 64) * T];
    __shared__ double coef[T];
    __shared__ double open[3]; // sum g^2, f(x^k), least nonzero |x_j|
    __shared__ SliceState sS;
    __shared__ StepWindow win;
    __shared__ int summed;
    const int s = blockIdx.y, B = pp.B, n = (int)pp.n;
    float *xs = reinterpret_cast<float *>(phase_lds);
    float *gs = xs + n;
    if (threadIdx.x == 0) sS = st_in[s];
    double v[2] = {0.0, 0.0}, least = INFINITY; // sum g^2, f(x^k)
    if (n < BS) form_steps<BS>(win, pp, st_in[s], 1); // else between the last wave's loads and their use
    for (int j0 = threadIdx.x; j0 < n; j0 += U * BS) {
        float xf[U], cf[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(j0 + u * BS, n - 1);
            xf[u] = x[(long long)j * B + s];
            if constexpr (OBJ == OBJ_LINEAR) cf[u] = lin_c[j];
        }
        if (n >= BS && j0 < BS) form_steps<BS>(win, pp, st_in[s], 1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * BS;
            if (j >= n) break;
            const double xj = (double)xf[u];
            float gf;
            if constexpr (OBJ == OBJ_SQNORM) {
                v[1] += xj * xj;
                gf = (float)(2.0 * xj);
            } else if constexpr (OBJ == OBJ_L1) { // subgradient sign(x), 0 at 0
                v[1] += fabs(xj);
                gf = xj > 0.0 ? 1.f : (xj < 0.0 ? -1.f : 0.f);
                if (gf != 0.f) least = fmin(least, fabs(xj));
            } else {
                gf = cf[u];
                v[1] += (double)gf * xj;
            }
            v[0] += (double)gf * (double)gf;
            xs[j] = xf[u];
            gs[j] = gf;
        }
    }
    if constexpr (OBJ == OBJ_L1) {
        for (int off = 32; off > 0; off >>= 1) least = fmin(least, __shfl_xor(least, off, 64));
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = least;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int w = 1; w < BS / 64; ++w) least = fmin(least, lds[w]);
        __syncthreads();
    }
    block_sum<2, BS>(v, lds); // its barriers also publish xs and gs
    if (threadIdx.x == 0) {
        open_phase_state(sS, pp, v[0], v[1]);
        open[0] = v[0];
        open[1] = v[1];
        open[2] = least;
    }
    __syncthreads();
    phase_rounds(
        threadIdx.x < 64, summed, [&] { return line_trials<OBJ>(sS, pp, win, open[1], open[0], open[2], T); },
        [&](int ntr) { // L1 only
            if (threadIdx.x < ntr) coef[threadIdx.x] = sS.s_acc + step_of(win, pp, sS, sS.ell + threadIdx.x);
            __syncthreads();
            const double inv_gn = 1.0 / sS.gn;
            double acc[T], cw[T];
#pragma unroll
            for (int w = 0; w < T; ++w) {
                acc[w] = 0.0;
                cw[w] = w < ntr ? coef[w] : 0.0;
            }
#pragma unroll 4
            for (int j = threadIdx.x; j < n; j += BS) {
                const double xj = (double)xs[j], vj = -(double)gs[j] * inv_gn;
#pragma unroll
                for (int w = 0; w < T; ++w) acc[w] += fabs(xj + cw[w] * vj);
            }
            sum_and_record<T, BS>(sS, pp, win, acc, ntr, lds);
        },
        [] { __syncthreads(); });
    const bool apply = must_apply(sS);
    if (apply) {
        const double inv_gn = 1.0 / sS.gn;
#pragma unroll 4
        for (int j = threadIdx.x; j < n; j += BS)
            x[(long long)j * B + s] = (float)((double)xs[j] + sS.s_acc * (-(double)gs[j] * inv_gn));
    }
    if (threadIdx.x == 0) {
        SliceState o = sS;
        if (apply) o.applied = 1;
        st_out[s] = o;
    }
}

// ---------------------------------------------------------------------------
// setup kernels
// ---------------------------------------------------------------------------

template <typename VT>
__device__ inline float stored_value(const void *val, long long p);
template <>
__device__ inline float stored_value<float>(const void *val, long long p) { return static_cast<const float *>(val)[p]; }
template <>
__device__ inline float stored_value<Bf16Tag>(const void *val, long long p)
{
    return __uint_as_float((uint32_t) static_cast<const uint16_t *>(val)[p] << 16);
}
template <>
__device__ inline float stored_value<F16Tag>(const void *val, long long p)
{
    return __half2float(__ushort_as_half(static_cast<const uint16_t *>(val)[p]));
}
template <>
__device__ inline float stored_value<Bf16PTag>(const void *val, long long p)
{
    return bf16_lo(static_cast<const uint32_t *>(val)[p]);
}
template <>
__device__ inline float stored_value<F16PTag>(const void *val, long long p)
{
    return f16_lo(static_cast<const uint32_t *>(val)[p]);
}

// q_i = ||a_i||^2 in float64 from the stored (possibly rounded) values; one wave per row
template <typename VT>
__global__ __launch_bounds__(kBlock) void k_rownorm(SpView A, double *__restrict__ q)
{
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (row >= A.rows) return;
    const int beg = A.ptr[row], end = A.ptr[row + 1];
    double s = 0.0;
    for (int p = beg + lane; p < end; p += 64) {
        const double a = (double)stored_value<VT>(A.val, p) * (double)A.vscale_inv;
        s += a * a;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) q[row] = s;
}

__global__ void k_make_D(const double *__restrict__ q, const double *__restrict__ w, float *__restrict__ D, long long m)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (long long)gridDim.x * blockDim.x)
        D[i] = q[i] > 0.0 ? (float)(w[i] / q[i]) : 0.f;
}

__global__ void k_to_bf16(const float *__restrict__ src, uint16_t *__restrict__ dst, long long count)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
        dst[i] = __bfloat16_as_ushort(__float2bfloat16(src[i]));
}

__global__ void k_to_f16(const float *__restrict__ src, uint16_t *__restrict__ dst, long long count, float scale)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
        dst[i] = __half_as_ushort(__float2half_rn(src[i] * scale));
}

__global__ void k_pack16u(const uint16_t *__restrict__ val16, const uint16_t *__restrict__ idx16,
                          uint32_t *__restrict__ packed, long long count)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
        packed[i] = (uint32_t)val16[i] | ((uint32_t)idx16[i] << 16);
}

__global__ void k_pack16(const uint16_t *__restrict__ val16, const int32_t *__restrict__ idx,
                         uint32_t *__restrict__ packed, long long count)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
        packed[i] = (uint32_t)val16[i] | ((uint32_t)idx[i] << 16);
}

__global__ void k_fill(float *__restrict__ p, float v, long long count)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_init_state(SliceState *st, int B, StopParams sp)
{
    const int s = threadIdx.x;
    if (s >= B) return;
    SliceState S;
    S.f_cur = S.f_start = __longlong_as_double(0x7ff8000000000000LL);
    S.gn = 0.0;
    S.s_acc = 0.0;
    S.prox = __longlong_as_double(0x7ff8000000000000LL);
    S.k = 0;
    S.k_end = 0x7fffffffffffffffLL;
    S.ell = 0;
    S.restarts = 0;
    S.trials = S.accepts = S.cap_hits = 0;
    S.n_done = 0;
    S.phase = 0;
    S.step_tried = 0;
    S.trials_it = S.accepts_it = 0;
    S.live = 1;
    S.applied = 0;
    S.enabled = 1;
    S.nonfinite = 0;
    S.need_last = 0;
    S.stop_on = sp.on;
    S.stop_n = sp.n;
    S.stop_max = sp.max_iters;
    S.stop_prox = sp.prox;
    S.stop_dprox = sp.dprox;
    S.stop_dobj = sp.dobj;
    S.stop_var = sp.var;
    S.stop_reason = STOP_NONE;
    S.dp_run = S.feas_ok = S.ran = 0;
    S.p_last = S.f_last = S.f_ref = __longlong_as_double(0x7ff8000000000000LL);
    S.beta_ad = 0.0;
    S.var_n = S.var_mean = S.var_m2 = 0.0;
    st[s] = S;
}

// Column s of a slice-interleaved [rows x B] array, in or out.
__global__ void k_put_column(float *__restrict__ dst, const float *__restrict__ src, long long rows, int B, int s)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < rows; i += (long long)gridDim.x * blockDim.x)
        dst[i * B + s] = src[i];
}

// Validation of a slot's bands staged on the device.  flag[0] collects bit 0
// for a NaN bound and bit 1 for lower > upper, flag[1] the lowest row with
// either; k_slot_flag_clear sets them to {0, 0xffffffff} first.
__global__ void k_slot_flag_clear(unsigned *flag)
{
    if (threadIdx.x == 0) {
        flag[0] = 0u;
        flag[1] = 0xffffffffu;
    }
}

__global__ void k_check_bands(const float *__restrict__ lo, const float *__restrict__ up, long long m,
                              unsigned *__restrict__ flag)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (long long)gridDim.x * blockDim.x) {
        const float a = lo[i], b = up[i];
        const unsigned bits = (isnan(a) || isnan(b)) ? 1u : (a > b ? 2u : 0u);
        if (bits) {
            atomicOr(&flag[0], bits);
            atomicMin(&flag[1], (unsigned)i);
        }
    }
}

__global__ void k_get_column(float *__restrict__ dst, const float *__restrict__ src, long long rows, int B, int s)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < rows; i += (long long)gridDim.x * blockDim.x)
        dst[i] = src[i * B + s];
}

// Slot s starts afresh: k = ell = restarts = 0, counters 0, `budget`
// iterations to run (0 disables the slot).
__global__ void k_reset_slot(SliceState *st, int s, long long budget)
{
    if (threadIdx.x != 0) return;
    SliceState S = st[s];
    S.f_cur = S.f_start = __longlong_as_double(0x7ff8000000000000LL);
    S.gn = 0.0;
    S.s_acc = 0.0;
    S.prox = __longlong_as_double(0x7ff8000000000000LL);
    S.k = 0;
    S.k_end = budget;
    S.ell = 0;
    S.restarts = 0;
    S.trials = S.accepts = S.cap_hits = 0;
    S.n_done = 0;
    S.phase = 0;
    S.step_tried = 0;
    S.trials_it = S.accepts_it = 0;
    S.enabled = budget > 0 ? 1 : 0;
    S.live = S.enabled;
    S.applied = 0;
    S.nonfinite = 0;
    S.need_last = 0;
    S.stop_reason = STOP_NONE;
    S.dp_run = S.feas_ok = S.ran = 0;
    S.p_last = S.f_last = S.f_ref = __longlong_as_double(0x7ff8000000000000LL);
    S.beta_ad = 0.0;
    S.var_n = S.var_mean = S.var_m2 = 0.0;
    st[s] = S;
}

__global__ void k_disable_slot(SliceState *st, int s)
{
    if (threadIdx.x != 0) return;
    st[s].enabled = 0;
    st[s].live = 0;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned grid_for(long long work, int per_block, unsigned cap)
{
    long long g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

hipError_t launch_rownorm(const SpView &A, int vk, double *q, hipStream_t s)
{
    const unsigned grid = grid_for(A.rows, kBlock / 64, 1u << 30);
    switch (vk) {
    case VK_F32: hipLaunchKernelGGL(k_rownorm<float>, dim3(grid), dim3(kBlock), 0, s, A, q); break;
    case VK_BF16: hipLaunchKernelGGL(k_rownorm<Bf16Tag>, dim3(grid), dim3(kBlock), 0, s, A, q); break;
    case VK_F16: hipLaunchKernelGGL(k_rownorm<F16Tag>, dim3(grid), dim3(kBlock), 0, s, A, q); break;
    case VK_BF16P: hipLaunchKernelGGL(k_rownorm<Bf16PTag>, dim3(grid), dim3(kBlock), 0, s, A, q); break;
    case VK_F16P: hipLaunchKernelGGL(k_rownorm<F16PTag>, dim3(grid), dim3(kBlock), 0, s, A, q); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_make_D(const double *q, const double *w, float *D, int64_t m, hipStream_t s)
{
    hipLaunchKernelGGL(k_make_D, dim3(grid_for(m, kBlock, 4096)), dim3(kBlock), 0, s, q, w, D, (long long)m);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *src, uint16_t *dst, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_to_bf16, dim3(grid_for(count, kBlock, 8192)), dim3(kBlock), 0, s, src, dst, (long long)count);
    return hipGetLastError();
}

hipError_t launch_to_f16(const float *src, uint16_t *dst, int64_t count, float scale, hipStream_t s)
{
    hipLaunchKernelGGL(k_to_f16, dim3(grid_for(count, kBlock, 8192)), dim3(kBlock), 0, s, src, dst, (long long)count,
                       scale);
    return hipGetLastError();
}

hipError_t launch_pack16u(const uint16_t *val16, const uint16_t *idx16, uint32_t *packed, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack16u, dim3(grid_for(count, kBlock, 8192)), dim3(kBlock), 0, s, val16, idx16, packed,
                       (long long)count);
    return hipGetLastError();
}

hipError_t launch_pack16(const uint16_t *val16, const int32_t *idx, uint32_t *packed, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack16, dim3(grid_for(count, kBlock, 8192)), dim3(kBlock), 0, s, val16, idx, packed,
                       (long long)count);
    return hipGetLastError();
}

hipError_t launch_fill(float *p, float v, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill, dim3(grid_for(count, kBlock, 4096)), dim3(kBlock), 0, s, p, v, (long long)count);
    return hipGetLastError();
}

hipError_t launch_put_column(float *dst, const float *src, int64_t rows, int B, int slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_put_column, dim3(grid_for(rows, kBlock, 2048)), dim3(kBlock), 0, s, dst, src, (long long)rows, B,
                       slot);
    return hipGetLastError();
}

hipError_t launch_check_bands(const float *lo, const float *up, int64_t m, unsigned *flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_slot_flag_clear, dim3(1), dim3(64), 0, s, flag);
    hipLaunchKernelGGL(k_check_bands, dim3(grid_for(m, kBlock, 2048)), dim3(kBlock), 0, s, lo, up, (long long)m, flag);
    return hipGetLastError();
}

hipError_t launch_get_column(float *dst, const float *src, int64_t rows, int B, int slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_get_column, dim3(grid_for(rows, kBlock, 2048)), dim3(kBlock), 0, s, dst, src, (long long)rows, B,
                       slot);
    return hipGetLastError();
}

hipError_t launch_reset_slot(SliceState *st, int slot, int64_t budget, hipStream_t s)
{
    hipLaunchKernelGGL(k_reset_slot, dim3(1), dim3(64), 0, s, st, slot, (long long)budget);
    return hipGetLastError();
}

hipError_t launch_disable_slot(SliceState *st, int slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_disable_slot, dim3(1), dim3(64), 0, s, st, slot);
    return hipGetLastError();
}

hipError_t launch_init_state(SliceState *st, int B, StopParams sp, hipStream_t s)
{
    hipLaunchKernelGGL(k_init_state, dim3(1), dim3(64), 0, s, st, B, sp);
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass1_vec(const PassCfg &cfg, const SpView &A, const float *x, const float *lower,
                            const float *upper, RowW w, float *c, const SliceState *st, int query,
                            double *partials, hipStream_t s)
{
    const dim3 grid(cfg.grid), block(kBlock);
    if constexpr (VEC == 1) { // interleaved lanes: 8 to 64 lanes per row
        switch (cfg.lpr) {
        case 8: hipLaunchKernelGGL((k_pass1<8, 1, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
        case 16: hipLaunchKernelGGL((k_pass1<16, 1, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
        case 32: hipLaunchKernelGGL((k_pass1<32, 1, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
        case 64: hipLaunchKernelGGL((k_pass1<64, 1, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (cfg.lpr) {
    case 2: hipLaunchKernelGGL((k_pass1<2, VEC, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case 4: hipLaunchKernelGGL((k_pass1<4, VEC, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case 8: hipLaunchKernelGGL((k_pass1<8, VEC, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case 16: hipLaunchKernelGGL((k_pass1<16, VEC, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case 32: hipLaunchKernelGGL((k_pass1<32, VEC, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case 64: hipLaunchKernelGGL((k_pass1<64, VEC, VT>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass1_stream(const PassCfg &cfg, const SpView &A, const RowBlocks &RB, const float *x,
                               const float *lower, const float *upper, RowW w, float *c,
                               const SliceState *st, int query, double *partials, hipStream_t s)
{
    hipLaunchKernelGGL((k_pass1_stream<VEC, VT>), dim3(cfg.grid), dim3(kBlock), 0, s, A, RB, x, lower, upper, w, c,
                       st, query, partials);
    return hipGetLastError();
}

template <typename VT, int VEC, int B>
static hipError_t pass1_mm(const PassCfg &cfg, const SpView &A, const float *x, const float *lower,
                           const float *upper, RowW w, float *c, const SliceState *st, int query,
                           double *partials, hipStream_t s)
{
    const dim3 grid(cfg.grid), block(kBlock);
    constexpr int L0 = mm_lanes(B, 0), L1 = mm_lanes(B, 1), L2 = mm_lanes(B, 2);
    switch (cfg.lpr) {
    case L0: hipLaunchKernelGGL((k_pass1_mm<L0, VEC, VT, B>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case L1: hipLaunchKernelGGL((k_pass1_mm<L1, VEC, VT, B>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    case L2: hipLaunchKernelGGL((k_pass1_mm<L2, VEC, VT, B>), grid, block, 0, s, A, x, lower, upper, w, c, st, query, partials); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass1_mm_b(const PassCfg &cfg, const SpView &A, const float *x, const float *lower,
                             const float *upper, RowW w, float *c, const SliceState *st, int B, int query,
                             double *partials, hipStream_t s)
{
    switch (B) {
    case 2: return pass1_mm<VT, VEC, 2>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    case 4: return pass1_mm<VT, VEC, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    case 8: return pass1_mm<VT, VEC, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    case 16: return pass1_mm<VT, VEC, 16>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    case 32: return pass1_mm<VT, VEC, 32>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename VT, int VEC, int LPR>
static hipError_t pass1_lds_go(const PassCfg &cfg, const SpView &A, const float *x, const float *lower,
                               const float *upper, RowW w, float *c, const SliceState *st, int query,
                               double *partials, int prepare, hipStream_t s)
{
    auto kern = k_pass1_lds<LPR, VEC, VT>;
    if (prepare)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)(sizeof(float) * kLdsPassFloats));
    const size_t shm = sizeof(float4) * size_t((cfg.xlds + 3) / 4);
    hipLaunchKernelGGL(kern, dim3(cfg.grid), dim3(kLdsPassBlock), shm, s, A, x, cfg.xlds, lower, upper, w, c, st,
                       query, partials);
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass1_lds(const PassCfg &cfg, const SpView &A, const float *x, const float *lower,
                            const float *upper, RowW w, float *c, const SliceState *st, int query, double *partials,
                            int prepare, hipStream_t s)
{
    switch (cfg.lpr) {
    case 4: return pass1_lds_go<VT, VEC, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case 8: return pass1_lds_go<VT, VEC, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case 16: return pass1_lds_go<VT, VEC, 16>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case 32: return pass1_lds_go<VT, VEC, 32>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename VT>
static hipError_t pass1_lds_v(const PassCfg &cfg, const SpView &A, const float *x, const float *lower,
                              const float *upper, RowW w, float *c, const SliceState *st, int query, double *partials,
                              int prepare, hipStream_t s)
{
    if (cfg.vec == 8) return pass1_lds<VT, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    if (cfg.vec == 4) return pass1_lds<VT, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    return hipErrorInvalidValue;
}

static hipError_t pass1_lds_kind(const PassCfg &cfg, int vk, const SpView &A, const float *x, const float *lower,
                                 const float *upper, RowW w, float *c, const SliceState *st, int query,
                                 double *partials, int prepare, hipStream_t s)
{
    switch (vk) {
    case VK_F32U16: return pass1_lds_v<F32U16Tag>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case VK_F32: return pass1_lds_v<float>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case VK_BF16: return pass1_lds_v<Bf16Tag>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case VK_BF16P: return pass1_lds_v<Bf16PTag>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case VK_F16: return pass1_lds_v<F16Tag>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    case VK_F16P: return pass1_lds_v<F16PTag>(cfg, A, x, lower, upper, w, c, st, query, partials, prepare, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename VT, int VEC, int LPR>
static hipError_t pass2_lds_go(const PassCfg &cfg, const SpView &At, const float *c, float *x, ColStep cs,
                               const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1, Hist h,
                               int prepare, hipStream_t s)
{
    auto kern = k_pass2_lds<LPR, VEC, VT>;
    if (prepare)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)(sizeof(float) * kLdsPassFloats));
    const size_t shm = sizeof(float4) * size_t((cfg.xlds + 3) / 4);
    hipLaunchKernelGGL(kern, dim3(column_grid(cfg.grid, cs)), dim3(kLdsPassBlock), shm, s, At, c, cfg.xlds, x, cs, st_in, st_out,
                       part1, nparts1, h);
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass2_lds(const PassCfg &cfg, const SpView &At, const float *c, float *x, ColStep cs,
                            const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1, Hist h,
                            int prepare, hipStream_t s)
{
    switch (cfg.lpr) {
    case 4: return pass2_lds_go<VT, VEC, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, prepare, s);
    case 8: return pass2_lds_go<VT, VEC, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, prepare, s);
    case 16: return pass2_lds_go<VT, VEC, 16>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, prepare, s);
    case 32: return pass2_lds_go<VT, VEC, 32>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, prepare, s);
    default: return hipErrorInvalidValue;
    }
}

static hipError_t pass2_lds_kind(const PassCfg &cfg, int vk, const SpView &At, const float *c, float *x, ColStep cs,
                                 const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1, Hist h,
                                 int prepare, hipStream_t s)
{
#define SMX_P2L(VT)                                                                                                    \
    (cfg.vec == 8 ? pass2_lds<VT, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, prepare, s)                 \
                  : (cfg.vec == 4 ? pass2_lds<VT, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, prepare, s) \
                                  : hipErrorInvalidValue))
    switch (vk) {
    case VK_F32U16: return SMX_P2L(F32U16Tag);
    case VK_F32: return SMX_P2L(float);
    case VK_BF16: return SMX_P2L(Bf16Tag);
    case VK_BF16P: return SMX_P2L(Bf16PTag);
    case VK_F16: return SMX_P2L(F16Tag);
    case VK_F16P: return SMX_P2L(F16PTag);
    default: return hipErrorInvalidValue;
    }
#undef SMX_P2L
}

template <typename VT, int VEC, int LPR>
static hipError_t panel_go(const PassCfg &cfg, const SpView &At, const PanelView &PV, const float *c,
                           const SliceState *st_in, int prepare, hipStream_t s)
{
    auto kern = k_pass2_panel<LPR, VEC, VT>;
    if (prepare)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)(sizeof(float) * kLdsPassFloats));
    const int n = (int)At.rows;
    const int chunks = std::max(1, std::min(n, (4 * cfg.grid + PV.np - 1) / PV.np)); // ~4 work items per workgroup
    const int cpt = (n + chunks - 1) / chunks;
    const size_t shm = sizeof(float4) * size_t((PV.P + 3) / 4);
    hipLaunchKernelGGL(kern, dim3(cfg.grid), dim3(kLdsPassBlock), shm, s, At, PV.pp, PV.np, PV.P, PV.m, cpt,
                       (n + cpt - 1) / cpt, PV.local, c, PV.ypanel, st_in);
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t panel_lpr(const PassCfg &cfg, const SpView &At, const PanelView &PV, const float *c,
                            const SliceState *st_in, int prepare, hipStream_t s)
{
    switch (cfg.lpr) {
    case 8: return panel_go<VT, VEC, 8>(cfg, At, PV, c, st_in, prepare, s);
    case 16: return panel_go<VT, VEC, 16>(cfg, At, PV, c, st_in, prepare, s);
    case 32: return panel_go<VT, VEC, 32>(cfg, At, PV, c, st_in, prepare, s);
    case 64: return panel_go<VT, VEC, 64>(cfg, At, PV, c, st_in, prepare, s);
    default: return hipErrorInvalidValue;
    }
}

static hipError_t panel_kind(const PassCfg &cfg, int vk, const SpView &At, const PanelView &PV, const float *c,
                             const SliceState *st_in, int prepare, hipStream_t s)
{
#define SMX_PAN(VT)                                                                                                    \
    (cfg.vec == 8 ? panel_lpr<VT, 8>(cfg, At, PV, c, st_in, prepare, s)                                              \
                  : (cfg.vec == 4 ? panel_lpr<VT, 4>(cfg, At, PV, c, st_in, prepare, s) : hipErrorInvalidValue))
    switch (vk) {
    case VK_F32U16: return SMX_PAN(F32U16Tag);
    case VK_F32: return SMX_PAN(float);
    case VK_BF16: return SMX_PAN(Bf16Tag);
    case VK_BF16P: return SMX_PAN(Bf16PTag);
    case VK_F16: return SMX_PAN(F16Tag);
    case VK_F16P: return SMX_PAN(F16PTag);
    default: return hipErrorInvalidValue;
    }
#undef SMX_PAN
}

hipError_t launch_pass2_panels(const PassCfg &cfg, const SpView &At, const PanelView &PV, int vk, const float *c,
                               float *x, ColStep cs, const SliceState *st_in, SliceState *st_out, const double *part1,
                               int nparts1, Hist h, hipStream_t s)
{
    if (cfg.grid < 1 || cfg.grid > kMaxPassGrid || nparts1 < 1 || nparts1 > kMaxPassGrid) return hipErrorInvalidValue;
    if (PV.np < 1 || PV.P < 1 || PV.P > kLdsPassFloats || PV.P % 4 != 0 || PV.m < 1 ||
        (long long)PV.np * PV.P < PV.m || (long long)(PV.np - 1) * PV.P >= PV.m || !PV.pp || !PV.ypanel)
        return hipErrorInvalidValue;
    const hipError_t e = panel_kind(cfg, vk, At, PV, c, st_in, 0, s);
    if (e != hipSuccess) return e;
    // the column sums in the same grid, so that the ||y||^2 partials of the
    // extrapolated steps number cfg.grid as for the other pass-2 shapes
    hipLaunchKernelGGL(k_pass2_panel_sum, dim3(column_grid(cfg.grid, cs)), dim3(kBlock), 0, s, PV.np, (int)At.rows, PV.ypanel,
                       At.vscale_inv, x, cs, st_in, st_out, part1, nparts1, h);
    return hipGetLastError();
}

hipError_t prepare_lds_passes()
{
    static hipError_t done = hipErrorNotReady;
    if (done == hipSuccess) return done;
    const SpView none{};
    for (int vk : {VK_F32U16, VK_F32, VK_BF16, VK_BF16P, VK_F16, VK_F16P})
        for (int lpr : {4, 8, 16, 32})
            for (int vec : {4, 8}) {
                PassCfg c;
                c.mode = 3;
                c.lpr = lpr;
                c.vec = vec;
                c.grid = 1;
                hipError_t e = pass1_lds_kind(c, vk, none, nullptr, nullptr, nullptr, RowW{}, nullptr, nullptr, 0,
                                              nullptr, 1, nullptr);
                if (e != hipSuccess) return e;
                e = pass2_lds_kind(c, vk, none, nullptr, nullptr, ColStep{}, nullptr, nullptr, nullptr, 0, Hist{}, 1,
                                   nullptr);
                if (e != hipSuccess) return e;
                for (int plpr : {8, 16, 32, 64}) {
                    PassCfg cp = c;
                    cp.lpr = plpr;
                    e = panel_kind(cp, vk, none, PanelView{}, nullptr, nullptr, 1, nullptr);
                    if (e != hipSuccess) return e;
                }
            }
    done = hipSuccess;
    return done;
}

hipError_t launch_pass1(const PassCfg &cfg, const SpView &A, const RowBlocks &RB, int vk, const float *x,
                        const float *lower, const float *upper, RowW w, float *c, const SliceState *st, int B,
                        int query, double *partials, hipStream_t s)
{
    if (cfg.grid < 1 || cfg.grid > kMaxPassGrid) return hipErrorInvalidValue;
    if (cfg.mode == 3) {
        if (B != 1 || cfg.xlds < 1 || cfg.xlds > kLdsPassFloats) return hipErrorInvalidValue;
        return pass1_lds_kind(cfg, vk, A, x, lower, upper, w, c, st, query, partials, 0, s);
    }
    if (B > 1) {
        if (vk == VK_F32U16) return pass1_mm_b<F32U16Tag, 4>(cfg, A, x, lower, upper, w, c, st, B, query, partials, s);
        if (vk == VK_F32) return pass1_mm_b<float, 4>(cfg, A, x, lower, upper, w, c, st, B, query, partials, s);
        if (vk == VK_BF16) return pass1_mm_b<Bf16Tag, 8>(cfg, A, x, lower, upper, w, c, st, B, query, partials, s);
        if (vk == VK_BF16P) return pass1_mm_b<Bf16PTag, 4>(cfg, A, x, lower, upper, w, c, st, B, query, partials, s);
        if (vk == VK_F16P) return pass1_mm_b<F16PTag, 4>(cfg, A, x, lower, upper, w, c, st, B, query, partials, s);
        return pass1_mm_b<F16Tag, 8>(cfg, A, x, lower, upper, w, c, st, B, query, partials, s);
    }
    if (cfg.mode == 1) {
        if (vk == VK_F32U16) return pass1_stream<F32U16Tag, 4>(cfg, A, RB, x, lower, upper, w, c, st, query, partials, s);
        if (vk == VK_F32) return pass1_stream<float, 4>(cfg, A, RB, x, lower, upper, w, c, st, query, partials, s);
        if (vk == VK_BF16) return pass1_stream<Bf16Tag, 8>(cfg, A, RB, x, lower, upper, w, c, st, query, partials, s);
        if (vk == VK_BF16P) return pass1_stream<Bf16PTag, 4>(cfg, A, RB, x, lower, upper, w, c, st, query, partials, s);
        if (vk == VK_F16P) return pass1_stream<F16PTag, 4>(cfg, A, RB, x, lower, upper, w, c, st, query, partials, s);
        return pass1_stream<F16Tag, 8>(cfg, A, RB, x, lower, upper, w, c, st, query, partials, s);
    }
    if (vk == VK_BF16P) {
        if (cfg.vec == 1) return pass1_vec<Bf16PTag, 1>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        if (cfg.vec == 8) return pass1_vec<Bf16PTag, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        return pass1_vec<Bf16PTag, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    }
    if (vk == VK_F16P) {
        if (cfg.vec == 1) return pass1_vec<F16PTag, 1>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        if (cfg.vec == 8) return pass1_vec<F16PTag, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        return pass1_vec<F16PTag, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    }
    if (vk == VK_F32U16) {
        if (cfg.vec == 1) return pass1_vec<F32U16Tag, 1>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        if (cfg.vec == 8) return pass1_vec<F32U16Tag, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        return pass1_vec<F32U16Tag, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    }
    if (vk == VK_F32) {
        if (cfg.vec == 1) return pass1_vec<float, 1>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        if (cfg.vec == 8) return pass1_vec<float, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        return pass1_vec<float, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    }
    if (vk == VK_BF16) {
        if (cfg.vec == 1) return pass1_vec<Bf16Tag, 1>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        if (cfg.vec == 8) return pass1_vec<Bf16Tag, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
        return pass1_vec<Bf16Tag, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    }
    if (cfg.vec == 1) return pass1_vec<F16Tag, 1>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    if (cfg.vec == 8) return pass1_vec<F16Tag, 8>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
    return pass1_vec<F16Tag, 4>(cfg, A, x, lower, upper, w, c, st, query, partials, s);
}

template <typename VT, int VEC>
static hipError_t pass2_vec(const PassCfg &cfg, const SpView &At, const float *c, float *x, ColStep cs,
                            const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1, Hist h,
                            hipStream_t s)
{
    const dim3 grid(column_grid(cfg.grid, cs)), block(kBlock);
#define SMX_P2(L) hipLaunchKernelGGL((k_pass2<L, VEC, VT>), grid, block, 0, s, At, c, x, cs, st_in, st_out, part1, nparts1, h)
    switch (cfg.lpr) {
    case 2: SMX_P2(2); break;
    case 4: SMX_P2(4); break;
    case 8: SMX_P2(8); break;
    case 16: SMX_P2(16); break;
    case 32: SMX_P2(32); break;
    case 64: SMX_P2(64); break;
    default: return hipErrorInvalidValue;
    }
#undef SMX_P2
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass2_stream(const PassCfg &cfg, const SpView &At, const RowBlocks &RB, const float *c, float *x,
                               ColStep cs, const SliceState *st_in, SliceState *st_out, const double *part1,
                               int nparts1, Hist h, hipStream_t s)
{
    hipLaunchKernelGGL((k_pass2_stream<VEC, VT>), dim3(column_grid(cfg.grid, cs)), dim3(kBlock), 0, s, At, RB, c, x, cs,
                       st_in, st_out, part1, nparts1, h);
    return hipGetLastError();
}

template <typename VT, int VEC, int B>
static hipError_t pass2_mm(const PassCfg &cfg, const SpView &At, const float *c, float *x, ColStep cs,
                           const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1, Hist h,
                           hipStream_t s)
{
    const dim3 grid(column_grid(cfg.grid, cs)), block(kBlock);
#define SMX_P2MM(L) hipLaunchKernelGGL((k_pass2_mm<L, VEC, VT, B>), grid, block, 0, s, At, c, x, cs, st_in, st_out, part1, nparts1, h)
    constexpr int L0 = mm_lanes(B, 0), L1 = mm_lanes(B, 1), L2 = mm_lanes(B, 2);
    switch (cfg.lpr) {
    case L0: SMX_P2MM(L0); break;
    case L1: SMX_P2MM(L1); break;
    case L2: SMX_P2MM(L2); break;
    default: return hipErrorInvalidValue;
    }
#undef SMX_P2MM
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass2_mm_b(const PassCfg &cfg, const SpView &At, const float *c, float *x, ColStep cs,
                             const SliceState *st_in, SliceState *st_out, int B, const double *part1, int nparts1,
                             Hist h, hipStream_t s)
{
    switch (B) {
    case 2: return pass2_mm<VT, VEC, 2>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 4: return pass2_mm<VT, VEC, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 8: return pass2_mm<VT, VEC, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 16: return pass2_mm<VT, VEC, 16>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 32: return pass2_mm<VT, VEC, 32>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename VT, int VEC, int B>
static hipError_t pass2_tiles_mm(const PassCfg &cfg, const TileView &T, const float *c, float *x, ColStep cs,
                                 const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1,
                                 Hist h, hipStream_t s)
{
    const dim3 grid(column_grid(cfg.grid, cs)), block(kBlock);
    const size_t shm = sizeof(float) * B * size_t(T.max_rows > 0 ? T.max_rows : 1);
#define SMX_P2TM(L) hipLaunchKernelGGL((k_pass2_tile_mm<L, VEC, VT, B>), grid, block, shm, s, T, c, x, cs, st_in, st_out, part1, nparts1, h)
    constexpr int L0 = mm_lanes(B, 0), L1 = mm_lanes(B, 1), L2 = mm_lanes(B, 2);
    switch (cfg.lpr) {
    case L0: SMX_P2TM(L0); break;
    case L1: SMX_P2TM(L1); break;
    case L2: SMX_P2TM(L2); break;
    default: return hipErrorInvalidValue;
    }
#undef SMX_P2TM
    return hipGetLastError();
}

template <typename VT, int VEC>
static hipError_t pass2_tiles_b(const PassCfg &cfg, const TileView &T, const float *c, float *x, ColStep cs,
                                const SliceState *st_in, SliceState *st_out, int B, const double *part1,
                                int nparts1, Hist h, hipStream_t s)
{
    switch (B) {
    case 2: return pass2_tiles_mm<VT, VEC, 2>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 4: return pass2_tiles_mm<VT, VEC, 4>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 8: return pass2_tiles_mm<VT, VEC, 8>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 16: return pass2_tiles_mm<VT, VEC, 16>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    case 32: return pass2_tiles_mm<VT, VEC, 32>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename VT, int VEC>
hipError_t pass2_tiles(const PassCfg &cfg, const TileView &T, const float *c, float *x, ColStep cs,
                       const SliceState *st_in, SliceState *st_out, const double *part1, int nparts1, Hist h,
                       hipStream_t s)
{
    const dim3 grid(column_grid(cfg.grid, cs)), block(kBlock);
    const size_t shm = sizeof(float) * size_t(T.max_rows > 0 ? T.max_rows : 1);
#define SMX_P2T(L) hipLaunchKernelGGL((k_pass2_tile<L, VEC, VT>), grid, block, shm, s, T, c, x, cs, st_in, st_out, part1, nparts1, h)
    switch (cfg.lpr) {
    case 2: SMX_P2T(2); break;
    case 4: SMX_P2T(4); break;
    case 8: SMX_P2T(8); break;
    case 16: SMX_P2T(16); break;
    default: return hipErrorInvalidValue;
    }
#undef SMX_P2T
    return hipGetLastError();
}

hipError_t launch_pass2_tiles(const PassCfg &cfg, const TileView &T, int vk, const float *c, float *x, ColStep cs,
                              const SliceState *st_in, SliceState *st_out, int B, const double *part1, int nparts1,
                              Hist h, hipStream_t s)
{
    if (cfg.grid < 1 || cfg.grid > kMaxPassGrid || nparts1 < 1 || nparts1 > kMaxPassGrid) return hipErrorInvalidValue;
    if (B < 1 || T.ntiles < 1 || T.max_rows < 0 || !tiles_fit(T.max_rows, B)) return hipErrorInvalidValue;
    const bool v8 = cfg.vec == 8;
    if (B > 1) {
        if (vk == VK_F32) return v8 ? pass2_tiles_b<F32U16Tag, 8>(cfg, T, c, x, cs, st_in, st_out, B, part1, nparts1, h, s)
                                    : pass2_tiles_b<F32U16Tag, 4>(cfg, T, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        if (vk == VK_BF16P) return v8 ? pass2_tiles_b<Bf16PTag, 8>(cfg, T, c, x, cs, st_in, st_out, B, part1, nparts1, h, s)
                                      : pass2_tiles_b<Bf16PTag, 4>(cfg, T, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        if (vk == VK_F16P) return v8 ? pass2_tiles_b<F16PTag, 8>(cfg, T, c, x, cs, st_in, st_out, B, part1, nparts1, h, s)
                                     : pass2_tiles_b<F16PTag, 4>(cfg, T, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        return hipErrorInvalidValue;
    }
    if (vk == VK_F32) return v8 ? pass2_tiles<F32U16Tag, 8>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s)
                                : pass2_tiles<F32U16Tag, 4>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    if (vk == VK_BF16P) return v8 ? pass2_tiles<Bf16PTag, 8>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s)
                                  : pass2_tiles<Bf16PTag, 4>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    if (vk == VK_F16P) return v8 ? pass2_tiles<F16PTag, 8>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s)
                                 : pass2_tiles<F16PTag, 4>(cfg, T, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    return hipErrorInvalidValue;
}

hipError_t launch_pass2(const PassCfg &cfg, const SpView &At, const RowBlocks &RB, int vk, const float *c, float *x,
                        ColStep cs, const SliceState *st_in, SliceState *st_out, int B, const double *part1,
                        int nparts1, Hist h, hipStream_t s)
{
    if (cfg.grid < 1 || cfg.grid > kMaxPassGrid || nparts1 < 1 || nparts1 > kMaxPassGrid) return hipErrorInvalidValue;
    if (cfg.mode == 3) {
        if (B != 1 || cfg.xlds < 1 || cfg.xlds > kLdsPassFloats) return hipErrorInvalidValue;
        return pass2_lds_kind(cfg, vk, At, c, x, cs, st_in, st_out, part1, nparts1, h, 0, s);
    }
    if (B > 1) {
        if (vk == VK_F32U16) return pass2_mm_b<F32U16Tag, 4>(cfg, At, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        if (vk == VK_F32) return pass2_mm_b<float, 4>(cfg, At, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        if (vk == VK_BF16) return pass2_mm_b<Bf16Tag, 8>(cfg, At, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        if (vk == VK_BF16P) return pass2_mm_b<Bf16PTag, 4>(cfg, At, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        if (vk == VK_F16P) return pass2_mm_b<F16PTag, 4>(cfg, At, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
        return pass2_mm_b<F16Tag, 8>(cfg, At, c, x, cs, st_in, st_out, B, part1, nparts1, h, s);
    }
    if (cfg.mode == 1) {
        if (vk == VK_F32U16) return pass2_stream<F32U16Tag, 4>(cfg, At, RB, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        if (vk == VK_F32) return pass2_stream<float, 4>(cfg, At, RB, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        if (vk == VK_BF16) return pass2_stream<Bf16Tag, 8>(cfg, At, RB, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        if (vk == VK_BF16P) return pass2_stream<Bf16PTag, 4>(cfg, At, RB, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        if (vk == VK_F16P) return pass2_stream<F16PTag, 4>(cfg, At, RB, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        return pass2_stream<F16Tag, 8>(cfg, At, RB, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    }
    if (vk == VK_BF16P) {
        if (cfg.vec == 8) return pass2_vec<Bf16PTag, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        return pass2_vec<Bf16PTag, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    }
    if (vk == VK_F16P) {
        if (cfg.vec == 8) return pass2_vec<F16PTag, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        return pass2_vec<F16PTag, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    }
    if (vk == VK_F32U16) {
        if (cfg.vec == 8) return pass2_vec<F32U16Tag, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        return pass2_vec<F32U16Tag, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    }
    if (vk == VK_F32) {
        if (cfg.vec == 8) return pass2_vec<float, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        return pass2_vec<float, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    }
    if (vk == VK_BF16) {
        if (cfg.vec == 8) return pass2_vec<Bf16Tag, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
        return pass2_vec<Bf16Tag, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    }
    if (cfg.vec == 8) return pass2_vec<F16Tag, 8>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
    return pass2_vec<F16Tag, 4>(cfg, At, c, x, cs, st_in, st_out, part1, nparts1, h, s);
}

// Row epilogue of the fused passes with z in LDS (one slice): the row's
// c_i (its step weight times the distance to its band) and its proximity
// term added to pacc; a dose-volume row only stores its value r for the
// ranking and adds nothing here (k_scatter_rows adds its c_i a_i once the
// ranking has set its band).
__device__ inline double fused_epilogue(const RowW &w, long long row, double r, float lo, float up, float d, float sw,
                                        double &pacc)
{
    if (w.dose && row >= w.dose_lo && row < w.dose_hi) {
        w.dose[row - w.dose_lo] = r;
        return 0.0;
    }
    const double t = fmin(fmax(r, (double)lo), (double)up) - r;
    pacc += (double)d * t * t;
    return (double)sw * t;
}

// A workgroup's y as its partial vector, float64 or (out32, or a float32 y)
// float32.
template <typename AccT>
__device__ inline void write_partial(void *ypart, int out32, int n, const AccT *y)
{
    if (out32 || sizeof(AccT) == sizeof(float)) {
        float *out = static_cast<float *>(ypart) + (long long)blockIdx.x * n;
        for (int j = threadIdx.x; j < n; j += kFusedBlock) out[j] = (float)y[j];
    } else {
        double *out = static_cast<double *>(ypart) + (long long)blockIdx.x * n;
        for (int j = threadIdx.x; j < n; j += kFusedBlock) out[j] = (double)y[j];
    }
}

// Fused pass with the gathered vector in LDS.  The plain fused pass gathers
// z_j through the vector memory path once per stored entry, about one
// address per CU per clock, which bounds it on long operators.  Here each
// workgroup (one per CU, 1024 threads) first copies all of z into LDS, beside
// y in float64 where both fit (12n bytes, n up to about 13k) and in float32
// otherwise (8n bytes, n up to about 20k), and runs the rows as
// the LDS-staged pass 1 does (LPR lanes per row, four loads of VEC entries in
// flight per lane, rows strided over the grid), gathering from LDS; a row
// outside its band then reads its entries again (from the cache) and adds
// c_i a_i into y with LDS atomics, each group of a wave starting at another
// chunk so that neighbouring rows, which list the same columns in the same
// order, touch different words at once.  y leaves as one partial vector per
// workgroup; k_fused_apply adds them in float64.  A float64 y costs half
// the adds' time or less: ds_add_f32 takes 192 clocks a wave whatever its
// addresses (3 a lane), ds_add_f64 8 to 16 where they spread over the banks.
template <int LPR, int VEC, typename VT, typename AccT>
__global__ __launch_bounds__(kFusedBlock) void k_fused_zl(SpView A, int n, const float *__restrict__ x,
                                                          const float *__restrict__ lower,
                                                          const float *__restrict__ upper, RowW w,
                                                          const SliceState *__restrict__ st,
                                                          double *__restrict__ partials, void *__restrict__ ypart,
                                                          int out32, LinPhase L)
{
    extern __shared__ __align__(16) unsigned char fused_lds[];
    float *zl = reinterpret_cast<float *>(fused_lds);
    AccT *y = reinterpret_cast<AccT *>(zl + ((n + 3) & ~3));
    __shared__ double lds[kFusedBlock / 64];
    __shared__ double tot[kPhaseSums];
    __shared__ SliceState sS;
    constexpr int RPB = kFusedBlock / LPR;
    constexpr int STEP = LPR * VEC;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const bool step = L.c && linear_phase<kFusedBlock>(sS, st, L.pp, L.part, 0, L.nparts, tot, L.st_out);
    const bool live = (L.c ? sS.live : st[0].live) != 0;
    for (int j = threadIdx.x; j < n; j += kFusedBlock) y[j] = AccT(0);
    double pacc[1] = {0.0};
    if (live) {
        if (step) stage_linear_point<kFusedBlock>(reinterpret_cast<float4 *>(zl), x, L.c, n, sS.s_acc, 1.0 / sS.gn);
        else stage_vector<kFusedBlock>(reinterpret_cast<float4 *>(zl), x, n);
        __syncthreads();
        const long long stride = (long long)gridDim.x * RPB;
        long long row = (long long)blockIdx.x * RPB + grp;
        int beg = 0, end = 0;
        if (row < A.rows) {
            beg = A.ptr[row];
            end = A.ptr[row + 1];
        }
        for (; row < A.rows; row += stride) {
            int nbeg = 0, nend = 0; // the next row's offsets, in flight meanwhile
            if (row + stride < A.rows) {
                nbeg = A.ptr[row + stride];
                nend = A.ptr[row + stride + 1];
            }
            const float lo = lower[row], up = upper[row], d = w.D[row], sw = w.S[row]; // read by every lane
            const double r =
                group_sum<LPR>(row_dot_split<LPR, VEC, VT>(A, beg, end, lane, x, zl, n)) * (double)A.vscale_inv;
            double ct = 0.0;
            if (lane == 0) ct = fused_epilogue(w, row, r, lo, up, d, sw, pacc[0]);
            ct = __shfl(ct, 0, LPR);
            if (ct != 0.0 && end > beg)
                scatter_row<LPR, VEC, VT, AccT>(A, beg, end, lane, grp, ct * (double)A.vscale_inv, y);
            beg = nbeg;
            end = nend;
        }
    }
    block_sum<1, kFusedBlock>(pacc, lds); // its barriers also order the LDS adds before the copy-out
    if (!live) return;
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
    write_partial(ypart, out32, n, y);
}

// k_fused_zl with each row's first CAP chunks (CAP * LPR * VEC entries) held
// in registers between the dot product and the scatter, so a row outside its
// band adds c_i a_i without reading its entries again: on an operator whose
// rows re-read from the cache outgrow L2, part of those re-reads come from
// HBM.  Within a group, lane l holds the chunk slots of lane (l + group) mod
// LPR (fetch_entries), so neighbouring rows, which list the same columns in
// the same order, hit different LDS addresses in one atomic instruction.
// Entries past CAP chunks are read again as in k_fused_zl.
template <int LPR, int VEC, int CAP, typename VT, typename AccT>
__global__ __launch_bounds__(kFusedBlock) void k_fused_zlr(SpView A, int n, const float *__restrict__ x,
                                                           const float *__restrict__ lower,
                                                           const float *__restrict__ upper, RowW w,
                                                           const SliceState *__restrict__ st,
                                                           double *__restrict__ partials, void *__restrict__ ypart,
                                                           int out32, LinPhase L)
{
    extern __shared__ __align__(16) unsigned char fused_lds[];
    float *zl = reinterpret_cast<float *>(fused_lds);
    AccT *y = reinterpret_cast<AccT *>(zl + ((n + 3) & ~3));
    __shared__ double lds[kFusedBlock / 64];
    __shared__ double tot[kPhaseSums];
    __shared__ SliceState sS;
    constexpr int RPB = kFusedBlock / LPR;
    constexpr int STEP = LPR * VEC;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int slot = (lane + grp) & (LPR - 1);
    const bool step = L.c && linear_phase<kFusedBlock>(sS, st, L.pp, L.part, 0, L.nparts, tot, L.st_out);
    const bool live = (L.c ? sS.live : st[0].live) != 0;
    for (int j = threadIdx.x; j < n; j += kFusedBlock) y[j] = AccT(0);
    double pacc[1] = {0.0};
    if (live) {
        if (step) stage_linear_point<kFusedBlock>(reinterpret_cast<float4 *>(zl), x, L.c, n, sS.s_acc, 1.0 / sS.gn);
        else stage_vector<kFusedBlock>(reinterpret_cast<float4 *>(zl), x, n);
        __syncthreads();
        const long long stride = (long long)gridDim.x * RPB;
        long long row = (long long)blockIdx.x * RPB + grp;
        int beg = 0, end = 0;
        if (row < A.rows) {
            beg = A.ptr[row];
            end = A.ptr[row + 1];
        }
        for (; row < A.rows; row += stride) {
            // the row's entries, the next row's offsets (in flight while this row
            // is reduced and scattered, so its entries are requested at once) and
            // the epilogue operands: all requested before any of them is used
            EntryRaw<VT, VEC> raw[CAP];
#pragma unroll
            for (int q = 0; q < CAP; ++q) {
                raw[q].zero();
                const int p = beg + (q * LPR + slot) * VEC;
                if (p < end) raw[q].load(A, p);
            }
            int nbeg = 0, nend = 0;
            if (row + stride < A.rows) {
                nbeg = A.ptr[row + stride];
                nend = A.ptr[row + stride + 1];
            }
            const float lo = lower[row], up = upper[row], d = w.D[row], sw = w.S[row]; // read by every lane
            RowRegs<VEC, CAP> R;
#pragma unroll
            for (int q = 0; q < CAP; ++q) {
                raw[q].decode(R.v[q], R.c[q]);
                if constexpr (sizeof(AccT) == sizeof(double)) spread_entries<VEC>(R.v[q], R.c[q], slot);
            }
            double acc[2] = {0.0, 0.0};
#pragma unroll
            for (int q = 0; q < CAP; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) // padding slots hold value 0 at column 0
                    acc[q & 1] = fma((double)R.v[q][e], (double)zl[R.c[q][e]], acc[q & 1]);
            const bool tail = end - beg > CAP * STEP;
            if (tail) { // one chunk at a time: the held entries keep most registers
                for (int p = beg + CAP * STEP + lane * VEC; p < end; p += STEP) {
                    float v[VEC];
                    int c[VEC];
                    Entries<VT, VEC>::load(A, p, v, c);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[0] = fma((double)v[e], (double)zl[c[e]], acc[0]);
                }
            }
            const double r = group_sum<LPR>(acc[0] + acc[1]) * (double)A.vscale_inv;
            double ct = 0.0;
            if (lane == 0) ct = fused_epilogue(w, row, r, lo, up, d, sw, pacc[0]);
            ct = __shfl(ct, 0, LPR);
            if (ct != 0.0) {
                const double sc = ct * (double)A.vscale_inv;
#pragma unroll
                for (int q = 0; q < CAP; ++q) lds_add_held<VEC>(y, R.c[q], R.v[q], sc);
                if (tail) {
                    for (int p = beg + CAP * STEP + lane * VEC; p < end; p += STEP) {
                        float v[VEC];
                        int c[VEC];
                        Entries<VT, VEC>::load(A, p, v, c);
                        lds_add_entries<VEC>(y, c, v, sc);
                    }
                }
            }
            beg = nbeg;
            end = nend;
        }
    }
    block_sum<1, kFusedBlock>(pacc, lds); // its barriers also order the LDS adds before the copy-out
    if (!live) return;
    if (threadIdx.x == 0) partials[blockIdx.x] = pacc[0];
    write_partial(ypart, out32, n, y);
}

// y += sum of c_i a_i over rows [r_lo, r_hi) with c_i already set (the
// dose-volume rows of a problem taking the fused pass, after their ranking):
// each 1024-thread workgroup adds its share of the rows (strided over the
// grid) into a float64 LDS copy of y and leaves it as one float32 partial
// vector, beside the fused pass's own.  A group has few rows, so a row is a latency
// chain: its LPR lanes request CAP * VEC entries each (256 of the row) at
// once, and the next row's offsets and c_i meanwhile.  (One chunk of 32
// entries at a time, as scatter_row goes, took 36 us for 33k rows of 184
// entries, 36 MB; 9 us so.)  As in k_fused_zlr lane l of a group holds
// the chunk slots of lane (l + group) mod LPR.
template <int LPR, int VEC, int CAP, typename VT>
__global__ __launch_bounds__(kFusedBlock) void k_scatter_rows(SpView A, int n, long long r_lo, long long r_hi,
                                                              const float *__restrict__ c,
                                                              const SliceState *__restrict__ st,
                                                              float *__restrict__ ypart)
{
    extern __shared__ __align__(16) unsigned char scat_lds[];
    double *y = reinterpret_cast<double *>(scat_lds);
    constexpr int RPB = kFusedBlock / LPR, STEP = LPR * VEC;
    const int lane = threadIdx.x & (LPR - 1);
    const int grp = threadIdx.x / LPR;
    const int slot = (lane + grp) & (LPR - 1);
    if (st[0].live == 0) return; // the same in every workgroup: the apply reads nothing then
    const long long stride = (long long)gridDim.x * RPB;
    long long row = r_lo + (long long)blockIdx.x * RPB + grp;
    float ci = 0.f;
    int beg = 0, end = 0;
    if (row < r_hi) {
        ci = c[row];
        beg = A.ptr[row];
        end = A.ptr[row + 1];
    }
    for (int j = threadIdx.x; j < n; j += kFusedBlock) y[j] = 0.0;
    __syncthreads();
    for (; row < r_hi; row += stride) {
        float nci = 0.f;
        int nbeg = 0, nend = 0;
        if (row + stride < r_hi) {
            nci = c[row + stride];
            nbeg = A.ptr[row + stride];
            nend = A.ptr[row + stride + 1];
        }
        if (ci != 0.f) {
            const double sc = (double)ci * (double)A.vscale_inv;
            for (int p = beg; p < end; p += CAP * STEP) {
                RowRegs<VEC, CAP> R;
                fetch_entries<LPR, VEC, CAP, VT>(A, p, end, slot, R);
#pragma unroll
                for (int q = 0; q < CAP; ++q) spread_entries<VEC>(R.v[q], R.c[q], slot);
#pragma unroll
                for (int q = 0; q < CAP; ++q) lds_add_held<VEC>(y, R.c[q], R.v[q], sc);
            }
        }
        ci = nci;
        beg = nbeg;
        end = nend;
    }
    __syncthreads();
    write_partial(ypart, 1, n, y);
}

// Workgroups of that kernel: two rows a group, at most `most`.
int scatter_rows_grid(long long rows, int most)
{
    constexpr int per = 2 * kFusedBlock / 16;
    return (int)std::max(1LL, std::min((rows + per - 1) / per, (long long)most));
}

size_t fused_lds_bytes(int64_t n, int acc64) { return size_t(n) * (acc64 ? sizeof(double) : sizeof(float)); }

size_t fused_zl_lds_bytes(int64_t n, int acc64)
{
    return size_t((n + 3) & ~int64_t(3)) * (sizeof(float) + (acc64 ? sizeof(double) : sizeof(float)));
}

int fused_apply_cols(int64_t n) { return n <= 1024 ? 16 : 64; }
int fused_apply_grid(int64_t n) { return (int)grid_for(n, fused_apply_cols(n), 4096); }

size_t fused_lds_limit()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 0;
    return size_t(v) > kFusedStaticLds ? size_t(v) - kFusedStaticLds : 0;
}

namespace {

struct FusedArgs {
    const SpView *A;
    int64_t n;
    const float *x, *lower, *upper;
    RowW w;
    const SliceState *st;
    double *partials;
    void *ypart;
    LinPhase lp; // lp.c == nullptr: no phase in the pass
};

// prepare != 0: only raise the kernel's dynamic-LDS attribute (done outside
// any stream capture, before the first launch of this shape)
template <int LPR, typename VT, int VEC, typename AccT>
hipError_t fused_zl_go(const FusedCfg &cfg, const FusedArgs &a, int prepare, hipStream_t s)
{
    constexpr int CAP = fused_zl_cap(LPR, VEC);
    if (cfg.cap != 0 && cfg.cap != CAP) return hipErrorInvalidValue;
    auto kern = cfg.cap ? k_fused_zlr<LPR, VEC, CAP, VT, AccT> : k_fused_zl<LPR, VEC, VT, AccT>;
    const size_t bytes = fused_zl_lds_bytes(a.n, sizeof(AccT) == sizeof(double));
    if (prepare)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bytes);
    hipLaunchKernelGGL(kern, dim3(cfg.grid), dim3(kFusedBlock), bytes, s, *a.A, (int)a.n, a.x, a.lower, a.upper, a.w,
                       a.st, a.partials, a.ypart, cfg.out32, a.lp);
    return hipGetLastError();
}

template <int LPR, typename VT, int VEC, typename AccT>
hipError_t fused_go(const FusedCfg &cfg, const FusedArgs &a, int prepare, hipStream_t s)
{
    if (cfg.zl) return fused_zl_go<LPR, VT, VEC, AccT>(cfg, a, prepare, s);
    if (cfg.out32 && cfg.acc64) return hipErrorInvalidValue; // the other shapes' partials are their y's type
    if (a.lp.c) return hipErrorInvalidValue; // the linear phase rides only on the shapes with z in LDS
    auto kern = k_fused<LPR, VEC, VT, AccT>;
    if (cfg.cap > 0) {
        // register-cached shapes hold CAP*LPR*VEC = 256 entries of a row; with
        // fewer than 16 lanes a row that takes more registers than a lane has
        if constexpr (LPR * VEC >= 64 && LPR >= 16) {
            constexpr int CAP = 256 / (LPR * VEC);
            if (cfg.cap != CAP) return hipErrorInvalidValue;
            kern = k_fused_rc<LPR, VEC, CAP, VT, AccT>;
        } else {
            return hipErrorInvalidValue;
        }
    }
    const size_t bytes = fused_lds_bytes(a.n, sizeof(AccT) == sizeof(double));
    if (prepare)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bytes);
    hipLaunchKernelGGL(kern, dim3(cfg.grid), dim3(cfg.cap > 0 ? kFusedRcBlock : kFusedBlock), bytes, s, *a.A,
                       (int)a.n, a.x, a.lower, a.upper, a.w, a.st, a.partials, static_cast<AccT *>(a.ypart));
    return hipGetLastError();
}

template <typename VT, int VEC, typename AccT>
hipError_t fused_lpr(const FusedCfg &cfg, const FusedArgs &a, int prepare, hipStream_t s)
{
    switch (cfg.lpr) {
    case 8: return fused_go<8, VT, VEC, AccT>(cfg, a, prepare, s);
    case 16: return fused_go<16, VT, VEC, AccT>(cfg, a, prepare, s);
    case 32: return fused_go<32, VT, VEC, AccT>(cfg, a, prepare, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename VT, int VEC>
hipError_t fused_acc_v(const FusedCfg &cfg, const FusedArgs &a, int prepare, hipStream_t s)
{
    return cfg.acc64 ? fused_lpr<VT, VEC, double>(cfg, a, prepare, s) : fused_lpr<VT, VEC, float>(cfg, a, prepare, s);
}

template <typename VT>
hipError_t fused_acc(const FusedCfg &cfg, const FusedArgs &a, int prepare, hipStream_t s)
{
    if (cfg.vec == 4) return fused_acc_v<VT, 4>(cfg, a, prepare, s);
    if (cfg.vec == 8) return fused_acc_v<VT, 8>(cfg, a, prepare, s);
    return hipErrorInvalidValue;
}

hipError_t fused_dispatch(const FusedCfg &cfg, int vk, const FusedArgs &a, int prepare, hipStream_t s)
{
    if (cfg.grid < 1 || cfg.grid > kMaxPassGrid || a.n < 1 || a.n > (int64_t(1) << 30)) return hipErrorInvalidValue;
    switch (vk) {
    case VK_F32: return fused_acc<float>(cfg, a, prepare, s);
    case VK_BF16: return fused_acc<Bf16Tag>(cfg, a, prepare, s);
    case VK_F16: return fused_acc<F16Tag>(cfg, a, prepare, s);
    case VK_BF16P: return fused_acc<Bf16PTag>(cfg, a, prepare, s);
    case VK_F16P: return fused_acc<F16PTag>(cfg, a, prepare, s);
    case VK_F32U16: return fused_acc<F32U16Tag>(cfg, a, prepare, s);
    default: return hipErrorInvalidValue;
    }
}

} // namespace

hipError_t prepare_fused(const FusedCfg &cfg, int vk, int64_t n)
{
    SpView none{};
    FusedArgs a{&none, n, nullptr, nullptr, nullptr, RowW{nullptr, nullptr, 0}, nullptr, nullptr, nullptr, LinPhase{}};
    return fused_dispatch(cfg, vk, a, 1, nullptr);
}

hipError_t launch_fused(const FusedCfg &cfg, const SpView &A, int vk, int64_t n, const float *x, const float *lower,
                        const float *upper, RowW w, const SliceState *st, double *partials, void *ypart,
                        hipStream_t s, const LinPhase *lp)
{
    if (w.qform) return hipErrorInvalidValue; // the fused pass makes c, never the quadratic form
    if (lp && (!lp->c || !lp->part || !lp->st_out || lp->pp.obj != OBJ_LINEAR || lp->pp.B != 1 || lp->pp.n != n ||
               lp->nparts < 1 || lp->nparts > 65535 || lp->pp.max_trials < 1 || lp->pp.max_trials > 1024 || !cfg.zl))
        return hipErrorInvalidValue;
    FusedArgs a{&A, n, x, lower, upper, w, st, partials, ypart, lp ? *lp : LinPhase{}};
    return fused_dispatch(cfg, vk, a, 0, s);
}

hipError_t launch_fused_apply(const FusedCfg &cfg, int64_t n, const void *ypart, int nvec, float *x, ColStep cs,
                              const SliceState *st_in, SliceState *st_out, const double *part1, Hist h,
                              hipStream_t s, const float *lin_c, double *lin_part, int lin_z)
{
    const bool wide = cfg.acc64 && !cfg.out32;
    if (cfg.grid < 1 || cfg.grid > kMaxPassGrid || n < 1 || nvec < cfg.grid || nvec > 2 * cfg.grid ||
        (wide && nvec != cfg.grid) || (lin_part && (!lin_c || cs.defer)) || (lin_z && (!lin_c || cs.defer)))
        return hipErrorInvalidValue;
    const dim3 grid(column_grid(fused_apply_grid(n), cs)), block(kApplyBlock);
    auto go = [&](auto kern, auto *vectors) {
        hipLaunchKernelGGL(kern, grid, block, 0, s, vectors, nvec, (int)n, x, cs, st_in, st_out, part1, cfg.grid, h,
                           lin_c, lin_part, lin_z);
    };
    const bool few = fused_apply_cols(n) == 16;
    if (wide) {
        const double *v = static_cast<const double *>(ypart);
        few ? go(k_fused_apply<double, 16>, v) : go(k_fused_apply<double, 64>, v);
    } else {
        const float *v = static_cast<const float *>(ypart);
        few ? go(k_fused_apply<float, 16>, v) : go(k_fused_apply<float, 64>, v);
    }
    return hipGetLastError();
}

hipError_t launch_lin_partials(const float *x, const float *c, int64_t n, double *part, int groups, bool extrap,
                               hipStream_t s)
{
    if (n < 1 || groups < 1 || !x || !c || !part) return hipErrorInvalidValue;
    auto kern = extrap ? k_lin_partials<kBlock, kBlock>
                       : (fused_apply_cols(n) == 16 ? k_lin_partials<16, kApplyBlock> : k_lin_partials<64, kApplyBlock>);
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(extrap ? kBlock : kApplyBlock), 0, s, x, c, (int)n, part);
    return hipGetLastError();
}

namespace {
template <typename VT>
hipError_t scatter_rows_go(int prepare, const SpView &A, int64_t n, long long r_lo, long long r_hi, const float *c,
                           const SliceState *st, float *ypart, int grid, hipStream_t s)
{
    auto kern = k_scatter_rows<16, 8, 2, VT>;
    const size_t bytes = sizeof(double) * size_t(n);
    if (prepare)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bytes);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kFusedBlock), bytes, s, A, (int)n, r_lo, r_hi, c, st, ypart);
    return hipGetLastError();
}

hipError_t scatter_rows_dispatch(int prepare, const SpView &A, int vk, int64_t n, long long r_lo, long long r_hi,
                                 const float *c, const SliceState *st, float *ypart, int grid, hipStream_t s)
{
    if (n < 1 || (!prepare && (grid < 1 || grid > kMaxPassGrid || r_lo < 0 || r_hi > A.rows || r_lo > r_hi)))
        return hipErrorInvalidValue;
    switch (vk) {
    case VK_F32: return scatter_rows_go<float>(prepare, A, n, r_lo, r_hi, c, st, ypart, grid, s);
    case VK_BF16: return scatter_rows_go<Bf16Tag>(prepare, A, n, r_lo, r_hi, c, st, ypart, grid, s);
    case VK_F16: return scatter_rows_go<F16Tag>(prepare, A, n, r_lo, r_hi, c, st, ypart, grid, s);
    case VK_BF16P: return scatter_rows_go<Bf16PTag>(prepare, A, n, r_lo, r_hi, c, st, ypart, grid, s);
    case VK_F16P: return scatter_rows_go<F16PTag>(prepare, A, n, r_lo, r_hi, c, st, ypart, grid, s);
    case VK_F32U16: return scatter_rows_go<F32U16Tag>(prepare, A, n, r_lo, r_hi, c, st, ypart, grid, s);
    default: return hipErrorInvalidValue;
    }
}
} // namespace

hipError_t prepare_scatter_rows(int vk, int64_t n)
{
    SpView none{};
    return scatter_rows_dispatch(1, none, vk, n, 0, 0, nullptr, nullptr, nullptr, 0, nullptr);
}

hipError_t launch_scatter_rows(const SpView &A, int vk, int64_t n, long long r_lo, long long r_hi, const float *c,
                               const SliceState *st, float *ypart, int grid, hipStream_t s)
{
    return scatter_rows_dispatch(0, A, vk, n, r_lo, r_hi, c, st, ypart, grid, s);
}

int step_apply_grid(int64_t n, int B) { return (int)grid_for(n * B, kBlock, 2048); }

hipError_t launch_step_apply(int64_t n, int B, const double *y, float *x, const float *lo, const float *hi,
                             float lambda, int emr, const double *part1, int nparts1, const double *party, int npartsy,
                             const double *partq, int npartsq, const SliceState *st_in, SliceState *st_out, Hist h,
                             hipStream_t s, const float *lin_c, double *lin_part, int lin_z)
{
    if (n < 1 || B < 1 || B > 32 || nparts1 < 1 || npartsy < 1 || (emr && npartsq < 1)) return hipErrorInvalidValue;
    if (lin_c ? (B != 1 || !lin_part) : (lin_part || lin_z)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)step_apply_grid(n, B) + 1; // the last closes the iteration
    hipLaunchKernelGGL(k_step_apply, dim3(grid), dim3(kBlock), 0, s, (int)n, B, y, x, lo, hi, lambda, emr, part1,
                       nparts1, party, npartsy, partq, npartsq, st_in, st_out, h, lin_c, lin_part, lin_z);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Dose-volume constraints (Section 2.3.3): sets in the output space of the
// split problem (eq. Split).  A constraint owns the rows of one structure;
// "at most k of them above d" (k = floor(V N)) or "at least k at or above d"
// (k = ceil(V N)).  Its nearest point keeps (MAX) or raises to d (MIN) the k
// highest values and lowers the other values above d to d (MAX) or keeps them
// (MIN); as bands, the k highest rows get (-inf, inf) / [d, inf) and the
// others (-inf, d] / (-inf, inf).  Rows rank by the float32-rounded value,
// equal values by row.  Pass 1 stores the rows' values; a radix select over
// their order-preserving 32-bit patterns (11, 11 and 10 bits, a launch each)
// finds the k-th highest value, and the band kernel forms c_i and the
// proximity terms; where only some of the rows with exactly that value rank
// high, it counts them in row order.  A round's histogram is made by all the
// constraint's workgroups (integer counts, so their atomic sums are exact) and
// its digit is found by every workgroup of the next launch alike, from the
// same 2,048 counts, while its rows' values are on their way.  Four launches,
// each a latency chain of about six microseconds; with a launch for every
// histogram, digit and sum these were fourteen, 68 us against 29 us on 33k
// rows in three constraints.  (Four launches whose last workgroup, by a
// ticket, took the digit and the sum: 36 us, the ticket's and the counts'
// round trips across the XCDs costing what the saved launches did.)
// ---------------------------------------------------------------------------

__device__ inline int dvc_group(const DvcTable &T, int blk)
{
    int g = 0;
    while (g + 1 < T.n && blk >= T.blk_begin[g + 1]) ++g;
    return g;
}

__device__ inline int dvc_shift(int round) { return round == 0 ? 21 : (round == 1 ? 10 : 0); }
__device__ inline int dvc_bits(int round) { return round < kDvcRounds - 1 ? 11 : 10; }

// Order-preserving pattern of a value rounded to float32 (higher value,
// higher pattern; -0 counts as +0).
__device__ inline unsigned dvc_order(double r)
{
    float f = (float)r;
    if (f == 0.0f) f = 0.0f;
    const unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ inline bool dvc_slice_runs(const SliceState *st, int s, int query) { return query || st[s].live != 0; }

// Selection state of constraint g and slice s after the first `rounds` rounds
// (none: only whether there is anything to select), the same in every
// workgroup: the state the first rounds - 1 left, and the digit of the last
// one's histogram that holds the k-th highest value, from the highest digit
// down.  The selection ends once every row of that digit ranks high (mode 2),
// or after the last round, where a digit is one value, of whose rows the
// first krem rank high (mode 4).  Every thread calls it.
__device__ inline DvcSel dvc_state(const DvcTable &T, const DvcScratch &W, int rounds, int g, int s, int B)
{
    __shared__ long long wsum[kDvcBlock / 64];
    __shared__ DvcSel found;
    const long long N = T.end[g] - T.begin[g], k = T.k[g];
    DvcSel S;
    S.krem = k;
    S.value = 0u;
    S.mode = k <= 0 ? 1 : (k >= N ? 3 : 0);
    if (S.mode != 0 || rounds == 0) return S;
    const int gs = g * B + s, ngs = T.n * B, r = rounds - 1;
    constexpr int PER = kDvcBins / kDvcBlock;
    static_assert(PER == 2, "one 8-byte load a thread");
    const uint2 h2 = reinterpret_cast<const uint2 *>(W.hist + ((size_t)r * ngs + gs) * kDvcBins)[threadIdx.x];
    if (r > 0) S = W.sel[(size_t)(r - 1) * ngs + gs];
    if (S.mode != 0) return S; // the same in every thread
    const unsigned cnt[PER] = {h2.x, h2.y};
    long long tsum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) tsum += cnt[j];
    // incl: counts of bins >= threadIdx.x * PER
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    long long incl = tsum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const long long v = __shfl_down(incl, off, 64);
        if (lane + off < 64) incl += v;
    }
    if (lane == 0) wsum[wid] = incl;
    __syncthreads();
#pragma unroll
    for (int w = 1; w < kDvcBlock / 64; ++w)
        if (w > wid) incl += wsum[w];
    const long long excl = incl - tsum;
    if (excl < S.krem && S.krem <= incl) { // one thread: 0 < krem <= the rows counted
        long long above = excl, kr = 0;
        int dig = 0;
        unsigned c_dig = 0;
#pragma unroll
        for (int j = PER - 1; j >= 0; --j) {
            if (c_dig == 0 && above + (long long)cnt[j] >= S.krem) {
                dig = threadIdx.x * PER + j;
                kr = S.krem - above;
                c_dig = cnt[j];
            }
            above += cnt[j];
        }
        const unsigned v = (S.value << dvc_bits(r)) | (unsigned)dig;
        found.krem = kr;
        const bool all = (long long)c_dig == kr;
        found.mode = all ? 2 : (r == kDvcRounds - 1 ? 4 : 0);
        found.value = all ? v << dvc_shift(r) : v;
    }
    __syncthreads();
    return found;
}

// Clears round r's histogram of (g, s), by the constraint's first workgroup: in
// a launch after the one that read it and before the one that fills it again.
__device__ inline void dvc_clear(const DvcTable &T, const DvcScratch &W, int r, int g, int s, int B)
{
    if ((int)blockIdx.x != T.blk_begin[g]) return;
    unsigned *H = W.hist + ((size_t)r * T.n * B + (g * B + s)) * kDvcBins;
    for (int b = threadIdx.x; b < kDvcBins; b += kDvcBlock) H[b] = 0u;
}

// One round of the selection: the digits of the rows that share the digits
// fixed so far into the round's histogram.  The last round also leaves each
// workgroup's own counts (tie, ncand), from which the band kernel tells a
// row's place among the rows of that value.
__global__ __launch_bounds__(kDvcBlock) void k_dvc_select(DvcTable T, int round, const double *__restrict__ dose,
                                                       DvcScratch W, const SliceState *__restrict__ st, int B,
                                                       int query)
{
    __shared__ unsigned h[kDvcBins];
    __shared__ unsigned cand;
    const int s = blockIdx.y;
    if (!dvc_slice_runs(st, s, query)) return;
    const int g = dvc_group(T, blockIdx.x);
    const long long N = T.end[g] - T.begin[g];
    const long long i0 = (long long)(blockIdx.x - T.blk_begin[g]) * kDvcChunk;
    const long long i1 = i0 + kDvcChunk < N ? i0 + kDvcChunk : N;
    constexpr int PERT = kDvcChunk / kDvcBlock;
    double d[PERT];
#pragma unroll
    for (int q = 0; q < PERT; ++q) { // past the end the last row again, not counted
        const long long i = i0 + q * kDvcBlock + threadIdx.x;
        d[q] = dose[(T.begin[g] + (i < i1 ? i : i1 - 1) - T.lo) * B + s];
    }
    for (int b = threadIdx.x; b < kDvcBins; b += kDvcBlock) h[b] = 0u;
    if (threadIdx.x == 0) cand = 0u;
    const DvcSel S = dvc_state(T, W, round, g, s, B);
    if (round > 0 && (int)blockIdx.x == T.blk_begin[g] && threadIdx.x == 0)
        W.sel[(size_t)(round - 1) * T.n * B + (g * B + s)] = S; // read by the next launch
    // the histogram read two launches ago (round 0: by the last band kernel)
    if (round != 1) dvc_clear(T, W, round == 0 ? kDvcRounds - 1 : 0, g, s, B);
    if (S.mode != 0) return; // the same in every thread
    __syncthreads();
    const int shift = dvc_shift(round), bits = dvc_bits(round), pshift = shift + bits;
    const unsigned mask = (1u << bits) - 1u;
    unsigned mine = 0;
#pragma unroll
    for (int q = 0; q < PERT; ++q) {
        const unsigned o = dvc_order(d[q]);
        if (i0 + q * kDvcBlock + threadIdx.x < i1 && (round == 0 || (o >> pshift) == S.value)) {
            atomicAdd(&h[(o >> shift) & mask], 1u);
            ++mine;
        }
    }
    if (mine) atomicAdd(&cand, mine);
    __syncthreads();
    unsigned *H = W.hist + ((size_t)round * T.n * B + (g * B + s)) * kDvcBins;
    if (cand)
        for (int b = threadIdx.x; b < kDvcBins; b += kDvcBlock)
            if (h[b]) atomicAdd(&H[b], h[b]);
    if (round == kDvcRounds - 1) {
        const size_t wg = (size_t)s * T.nblk + blockIdx.x;
        if (threadIdx.x == 0) W.ncand[wg] = cand;
        if (cand) // at most kDvcChunk a bin: 16 bits
            for (int b = threadIdx.x; b < kDvcTieBins; b += kDvcBlock) W.tie[wg * kDvcTieBins + b] = (uint16_t)h[b];
    }
}

// The bands the selection gives, c_i = S_i t_i and the proximity terms D_i
// t_i^2, which a workgroup adds to pass 1's partial of its own number (the
// grid has at most nparts1 workgroups a slice; each takes chunks of rows
// blockIdx.x, blockIdx.x + gridDim.x, ...).
__global__ __launch_bounds__(kDvcBlock) void k_dvc_bands(DvcTable T, const double *__restrict__ dose, DvcScratch W,
                                                      const float *__restrict__ D, const float *__restrict__ Sw,
                                                      float *__restrict__ c, double *__restrict__ part1, int nparts1,
                                                      const SliceState *__restrict__ st, int B, int query)
{
    __shared__ double lds[kDvcBlock / 64];
    __shared__ unsigned wsum[kDvcBlock / 64];
    __shared__ double total;
    const int s = blockIdx.y;
    if (!dvc_slice_runs(st, s, query)) return;
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double pacc[1] = {0.0};
    for (int blk = blockIdx.x; blk < T.nblk; blk += gridDim.x) {
        const int g = dvc_group(T, blk);
        const long long N = T.end[g] - T.begin[g];
        const long long i0 = (long long)(blk - T.blk_begin[g]) * kDvcChunk;
        const long long i1 = i0 + kDvcChunk < N ? i0 + kDvcChunk : N;
        const double dref = T.dose[g];
        const bool upper_kind = T.sense[g] == 0;
        const DvcSel S = dvc_state(T, W, kDvcRounds, g, s, B);
        if (blk == T.blk_begin[g]) { // the second round's histogram, read by the launch before this one
            unsigned *H = W.hist + ((size_t)1 * T.n * B + (g * B + s)) * kDvcBins;
            for (int b = threadIdx.x; b < kDvcBins; b += kDvcBlock) H[b] = 0u;
        }
        long long before = 0; // mode 4: rows of the value in the constraint's chunks before this one
        if (S.mode == 4) {
            double n0[1] = {0.0};
            const unsigned dig = S.value & (kDvcTieBins - 1);
            for (int b = T.blk_begin[g] + (int)threadIdx.x; b < blk; b += kDvcBlock) {
                const size_t wg = (size_t)s * T.nblk + b;
                if (W.ncand[wg]) n0[0] += (double)W.tie[wg * kDvcTieBins + dig];
            }
            block_sum<1, kDvcBlock>(n0, lds);
            if (threadIdx.x == 0) total = n0[0];
            __syncthreads();
            before = (long long)total;
        }
        for (long long r0 = i0; r0 < i1; r0 += kDvcBlock) { // the same rounds in every thread
            const long long i = r0 + threadIdx.x;
            const bool in = i < i1;
            const long long row = T.begin[g] + (in ? i : i1 - 1);
            const double r = dose[(row - T.lo) * B + s];
            const unsigned o = dvc_order(r);
            bool high = S.mode == 3 || (S.mode == 2 && o >= S.value) || (S.mode == 4 && o > S.value);
            if (S.mode == 4) { // the same in every thread
                const bool tie = in && o == S.value;
                const unsigned long long m = __ballot(tie);
                if (lane == 0) wsum[wid] = (unsigned)__popcll(m);
                __syncthreads();
                long long place = before + __popcll(m & ((1ull << lane) - 1ull));
                for (int w = 0; w < kDvcBlock / 64; ++w) {
                    if (w < wid) place += wsum[w];
                    before += wsum[w];
                }
                if (tie && place < S.krem) high = true;
                __syncthreads();
            }
            if (!in) continue;
            double lo = -INFINITY, up = INFINITY;
            if (upper_kind) {
                if (!high) up = dref;
            } else if (high) {
                lo = dref;
            }
            const double t = fmin(fmax(r, lo), up) - r;
            c[row * B + s] = (float)((double)Sw[row] * t);
            pacc[0] += (double)D[row] * t * t;
        }
        __syncthreads(); // before the next chunk's use of the shared state
    }
    block_sum<1, kDvcBlock>(pacc, lds);
    if (threadIdx.x == 0) part1[(long long)s * nparts1 + blockIdx.x] += pacc[0];
}

hipError_t launch_dvc(const DvcTable &T, const double *dose, const DvcScratch &W, const float *D, const float *S,
                      float *c, double *part1, int nparts1, const SliceState *st, int B, int query, hipStream_t s)
{
    if (T.n < 1 || T.n > kMaxDvc || T.nblk < 1 || B < 1 || B > 32 || nparts1 < 1) return hipErrorInvalidValue;
    const dim3 blk(kDvcBlock);
    for (int r = 0; r < kDvcRounds; ++r)
        hipLaunchKernelGGL(k_dvc_select, dim3(T.nblk, B), blk, 0, s, T, r, dose, W, st, B, query);
    hipLaunchKernelGGL(k_dvc_bands, dim3(std::min(T.nblk, nparts1), B), blk, 0, s, T, dose, W, D, S, c, part1, nparts1,
                       st, B, query);
    return hipGetLastError();
}

hipError_t launch_phase(const PertParams &pp, const float *x, float *g, const float *lin_c, const SliceState *st,
                        int eval_only, double *partials, hipStream_t s, double *part_min)
{
    const dim3 grid(phase_grid(pp), pp.B), block(kBlock);
    if (tv_whole_lines(pp)) {
#define SMX_PTV(NB)                                                                                                    \
    case NB:                                                                                                           \
        if (tv_small_block(pp))                                                                                        \
            hipLaunchKernelGGL((k_phase_tv_mm<NB, kTrialSmallBlock>), dim3(grid.x), dim3(kTrialSmallBlock), 0, s, x,   \
                               g, st, pp, tv_tile_rows(pp), eval_only, partials);                                      \
        else                                                                                                           \
            hipLaunchKernelGGL((k_phase_tv_mm<NB, kTrialBlock>), dim3(grid.x), dim3(kTrialBlock), 0, s, x, g, st, pp,  \
                               tv_tile_rows(pp), eval_only, partials);                                                 \
        break
        switch (pp.B) {
            SMX_PTV(2);
            SMX_PTV(4);
            SMX_PTV(8);
            SMX_PTV(16);
            SMX_PTV(32);
        default: return hipErrorInvalidValue;
        }
#undef SMX_PTV
    } else if (pp.obj == OBJ_TV2D)
        hipLaunchKernelGGL(k_phase_tv, grid, block, 0, s, x, g, st, pp, eval_only, partials);
    else
        hipLaunchKernelGGL(k_phase_flat, grid, block, 0, s, x, g, lin_c, st, pp, eval_only, partials, part_min);
    return hipGetLastError();
}

bool phase_on_line(const PertParams &pp)
{
    // k_trial_line steps an int by its grid's threads: longer vectors take the chain, which counts in 64 bits
    constexpr long long walk = (1LL << 31) - (long long)kFlatPhaseGrid * kTrialBlock;
    if (pp.obj == OBJ_SQNORM) return pp.n <= walk;
    if (pp.obj != OBJ_L1) return false;
    return pp.B == 1 ? pp.n <= kLineMaxN : pp.n <= kLineSumN && phase_grid(pp) * pp.B <= kLineSumGroups;
}

bool phase_sorted(const PertParams &pp)
{
    return pp.obj == OBJ_L1 && pp.B == 1 && pp.n > kLineSumN && pp.n <= kLineMaxN;
}

static size_t line_chunks(const PertParams &pp) { return size_t((pp.n + kLineChunk - 1) / kLineChunk); }

size_t line_sorted_bytes(const PertParams &pp)
{
    return phase_sorted(pp) ? line_chunks(pp) * (sizeof(float) * kLineChunk +
                                                 (sizeof(double) + sizeof(float)) * (kLineChunk / kLineBucket))
                            : 0;
}

LineSorted line_sorted(void *buf, const PertParams &pp)
{
    const size_t chunks = line_chunks(pp), pivots = chunks * (kLineChunk / kLineBucket);
    LineSorted L;
    L.key = static_cast<float *>(buf);
    L.below = reinterpret_cast<double *>(L.key + chunks * kLineChunk);
    L.pivot = reinterpret_cast<float *>(L.below + pivots);
    return L;
}

hipError_t launch_phase_sorted(const PertParams &pp, const float *x, const SliceState *st, const LineSorted &L,
                               double *partials, double *part_min, hipStream_t s)
{
    if (!phase_sorted(pp) || size_t(phase_grid(pp)) != line_chunks(pp)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_phase_sorted, dim3(phase_grid(pp)), dim3(kBlock), 0, s, x, (int)pp.n, st, L, partials,
                       part_min);
    return hipGetLastError();
}

hipError_t launch_trial_sorted(const PertParams &pp, float *x, const SliceState *st_in, SliceState *st_out,
                               const LineSorted &L, const double *part_phase, const double *part_min, hipStream_t s)
{
    if (!phase_sorted(pp) || pp.max_trials < 1 || pp.max_trials > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_trial_sorted, dim3(phase_grid(pp)), dim3(kTrialBlock), 0, s, x, st_in, st_out, pp,
                       part_phase, part_min, L, phase_grid(pp));
    return hipGetLastError();
}

hipError_t launch_trial_line(const PertParams &pp, float *x, const float *xc, const SliceState *st_in,
                             SliceState *st_out, const double *part_phase, const double *part_min, hipStream_t s)
{
    if (!phase_on_line(pp) || pp.max_trials < 1 || pp.max_trials > 1024 || pp.B < 1) return hipErrorInvalidValue;
    const int nt = phase_grid(pp);
    const dim3 grid(nt, pp.B), block(kTrialBlock);
    if (pp.obj == OBJ_SQNORM)
        hipLaunchKernelGGL(k_trial_line<OBJ_SQNORM>, grid, block, 0, s, x, xc, st_in, st_out, pp, part_phase, part_min,
                           nt);
    else
        hipLaunchKernelGGL(k_trial_line<OBJ_L1>, grid, block, 0, s, x, xc, st_in, st_out, pp, part_phase, part_min, nt);
    return hipGetLastError();
}

hipError_t launch_query_out(SliceState *st, const PertParams &pp, const double *part_prox, int nparts,
                            const double *part_obj, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_query_out, dim3(pp.B, part_obj ? 2 : 1), dim3(kBlock), 0, s, st, pp.B, part_prox, nparts,
                       part_obj, part_obj ? phase_grid(pp) : 0, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Variance stopping rule (Section 2.3.2): omega_k = ||x^k - x^{k-1}|| / ||x^k||
// (0 when x^k = 0); the run stops once the sample variance of omega_1 ..
// omega_k (k >= 2) is below the threshold.  Running mean and sum of squared
// deviations (Welford), in float64, per slice.
// ---------------------------------------------------------------------------

__global__ void k_copy(float *__restrict__ dst, const float *__restrict__ src, long long count)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// Per-workgroup partials of ||x - xprev||^2 and ||x||^2 for every slice:
// partials[(s * grid + block) * 2 + {0, 1}].
__global__ __launch_bounds__(kBlock) void k_iter_norms(const float *__restrict__ x, const float *__restrict__ xprev,
                                                       long long n, int B, double *__restrict__ partials)
{
    __shared__ double lds[4 * 2];
    for (int s = 0; s < B; ++s) {
        double v[2] = {0.0, 0.0};
        for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < n; j += (long long)gridDim.x * kBlock) {
            const double a = (double)x[j * B + s], b = (double)xprev[j * B + s];
            v[0] += (a - b) * (a - b);
            v[1] += a * a;
        }
        block_sum<2>(v, lds);
        if (threadIdx.x == 0) {
            partials[((long long)s * gridDim.x + blockIdx.x) * 2 + 0] = v[0];
            partials[((long long)s * gridDim.x + blockIdx.x) * 2 + 1] = v[1];
        }
    }
}

// One workgroup: updates the statistics of the slices that ran the iteration
// just ended and stops those whose variance fell below the threshold (a
// reason already set by the proximity rules takes precedence).  In place on
// the current state buffer (no other workgroup touches it in this launch).
__global__ __launch_bounds__(kBlock) void k_stop_var(SliceState *__restrict__ st, int B,
                                                     const double *__restrict__ partials, int nparts)
{
    __shared__ double lds[4 * 2];
    for (int s = 0; s < B; ++s) {
        double tot[2];
        sum_slots<2>(partials, (long long)s * nparts, nparts, tot, lds);
        if (threadIdx.x == 0) {
            SliceState S = st[s];
            if (S.ran && S.stop_on && S.stop_var > 0.0) {
                const double om = tot[1] > 0.0 ? sqrt(tot[0]) / sqrt(tot[1]) : 0.0;
                S.var_n += 1.0;
                const double delta = om - S.var_mean;
                S.var_mean += delta / S.var_n;
                S.var_m2 += delta * (om - S.var_mean);
                if (S.stop_reason == STOP_NONE && S.var_n >= 2.0 && S.var_m2 / (S.var_n - 1.0) < S.stop_var)
                    S.stop_reason = STOP_VAR;
                S.live = slice_runs(S);
                st[s] = S;
            }
        }
    }
}

hipError_t launch_copy(float *dst, const float *src, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_copy, dim3(grid_for(count, kBlock, 4096)), dim3(kBlock), 0, s, dst, src, (long long)count);
    return hipGetLastError();
}

hipError_t launch_iter_norms(const float *x, const float *xprev, int64_t n, int B, double *partials, int *nparts,
                             hipStream_t s)
{
    const unsigned grid = grid_for(n, kBlock, 256);
    *nparts = (int)grid;
    hipLaunchKernelGGL(k_iter_norms, dim3(grid), dim3(kBlock), 0, s, x, xprev, (long long)n, B, partials);
    return hipGetLastError();
}

hipError_t launch_stop_var(SliceState *st, int B, const double *partials, int nparts, hipStream_t s)
{
    hipLaunchKernelGGL(k_stop_var, dim3(1), dim3(kBlock), 0, s, st, B, partials, nparts);
    return hipGetLastError();
}

bool phase_in_one_launch(const PertParams &pp)
{
    return (pp.obj == OBJ_SQNORM || pp.obj == OBJ_L1 || pp.obj == OBJ_LINEAR) && pp.n >= 1 &&
           pp.n <= kSmallPhaseMaxN;
}

static size_t phase_small_lds(const PertParams &pp) { return 2 * sizeof(float) * size_t(pp.n); }

// Loads a thread keeps in flight, the least of 2, 8 and 20 that takes x in one
// round (20: kSmallPhaseMaxN).
template <typename F>
static hipError_t phase_small_dispatch(int obj, int64_t n, F &&go)
{
    const int u = n <= 2 * kSmallPhaseBlock ? 2 : (n <= 8 * kSmallPhaseBlock ? 8 : 20);
#define SMX_PSM(O)                                                                                                     \
    (u == 2 ? go(k_phase_small<O, 2>) : (u == 8 ? go(k_phase_small<O, 8>) : go(k_phase_small<O, 20>)))
    switch (obj) {
    case OBJ_SQNORM: return SMX_PSM(OBJ_SQNORM);
    case OBJ_L1: return SMX_PSM(OBJ_L1);
    case OBJ_LINEAR: return SMX_PSM(OBJ_LINEAR);
    default: return hipErrorInvalidValue;
    }
#undef SMX_PSM
}
static_assert(20 * kSmallPhaseBlock >= kSmallPhaseMaxN, "one round of loads");

hipError_t prepare_phase_small()
{
    // the largest size any problem asks for: the attribute is the kernel's, not a problem's
    const int bytes = (int)(2 * sizeof(float) * kSmallPhaseMaxN);
    for (int obj : {OBJ_SQNORM, OBJ_L1, OBJ_LINEAR})
        for (int64_t n : {1, 8 * kSmallPhaseBlock, kSmallPhaseMaxN}) {
            const hipError_t e = phase_small_dispatch(obj, n, [&](auto kern) {
                return hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
            });
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t launch_phase_small(const PertParams &pp, float *x, const float *lin_c, const SliceState *st_in,
                              SliceState *st_out, hipStream_t s)
{
    if (!phase_in_one_launch(pp) || pp.max_trials < 1 || pp.max_trials > 1024 || pp.B < 1) return hipErrorInvalidValue;
    return phase_small_dispatch(pp.obj, pp.n, [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(1, pp.B), dim3(kSmallPhaseBlock), phase_small_lds(pp), s, x, lin_c, st_in, st_out,
                           pp);
        return hipGetLastError();
    });
}

hipError_t launch_trial_linear(const PertParams &pp, float *x, const float *c, const SliceState *st_in,
                               SliceState *st_out, const double *part_phase, hipStream_t s, int nt)
{
    if (pp.obj != OBJ_LINEAR || pp.max_trials < 1 || pp.max_trials > 1024) return hipErrorInvalidValue;
    if (nt == 0) nt = phase_grid(pp); // the direction launch's partials
    if (nt < 1 || nt > 65535 || (nt != phase_grid(pp) && pp.B != 1)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_trial_linear, dim3(nt, pp.B), dim3(kBlock), 0, s, x, c, st_in, st_out, pp, part_phase);
    return hipGetLastError();
}

static hipError_t trial_tv_mm(const PertParams &pp, float *x, const float *g, const SliceState *st_in,
                              SliceState *st_out, int first, int after, const double *part_prev, double *part_out,
                              hipStream_t s)
{
#define SMX_TTV(NB)                                                                                                    \
    case NB:                                                                                                           \
        if (tv_small_block(pp))                                                                                        \
            hipLaunchKernelGGL((k_trial_tv_mm<NB, kTrialSmallBlock>), dim3(phase_grid(pp)), dim3(kTrialSmallBlock), 0, \
                               s, x, g, st_in, st_out, pp, tv_tile_rows(pp), first, after, part_prev, part_out);       \
        else                                                                                                           \
            hipLaunchKernelGGL((k_trial_tv_mm<NB, kTrialBlock>), dim3(phase_grid(pp)), dim3(kTrialBlock), 0, s, x, g,  \
                               st_in, st_out, pp, tv_tile_rows(pp), first, after, part_prev, part_out);                \
        break
    switch (pp.B) {
        SMX_TTV(2);
        SMX_TTV(4);
        SMX_TTV(8);
        SMX_TTV(16);
        SMX_TTV(32);
    default: return hipErrorInvalidValue;
    }
#undef SMX_TTV
    return hipGetLastError();
}

hipError_t launch_trial_close(const PertParams &pp, float *x, const float *g, const SliceState *st_in,
                              SliceState *st_out, const double *part_prev, hipStream_t s)
{
    if (pp.max_trials < 1 || pp.max_trials > 1024) return hipErrorInvalidValue;
    if (tv_whole_lines(pp)) return trial_tv_mm(pp, x, g, st_in, st_out, 0, -1, part_prev, nullptr, s);
    const long long g_need = (pp.n + kTrialBlock - 1) / kTrialBlock; // one unknown a thread, at most 256 workgroups
    const unsigned grid = (unsigned)std::max(1LL, std::min(g_need, 256LL));
    hipLaunchKernelGGL(k_trial_close, dim3(grid, pp.B), dim3(kTrialBlock), 0, s, x, g, st_in, st_out, pp,
                       (int)phase_grid(pp), part_prev);
    return hipGetLastError();
}

hipError_t launch_trial(const PertParams &pp, float *x, const float *g, const SliceState *st_in, SliceState *st_out,
                        int first, int after, const double *part_prev, double *part_out, hipStream_t s)
{
    if (pp.max_trials < 1 || pp.max_trials > 1024 || after < 0) return hipErrorInvalidValue;
    if (tv_whole_lines(pp))
        return trial_tv_mm(pp, x, g, st_in, st_out, first, after, part_prev, part_out, s);
    const dim3 grid(phase_grid(pp), pp.B), block(kBlock);
    if (pp.obj == OBJ_TV2D)
        hipLaunchKernelGGL(k_trial_tv, grid, dim3(kTrialBlock), 0, s, x, g, st_in, st_out, pp, first, after,
                           part_prev, part_out);
    else
        hipLaunchKernelGGL(k_trial_flat, grid, block, 0, s, x, g, st_in, st_out, pp, first, after, part_prev,
                           part_out);
    return hipGetLastError();
}

} // namespace smx
