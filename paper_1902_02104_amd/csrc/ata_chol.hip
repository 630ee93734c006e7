// Consumers of the packed product on gfx950: the Cholesky factor of the
// packed lower C (the solves with it are in ata_trsv.hip, A^t b and A X in
// ata_mv.hip); and the transpose that gives the companion product A A^t.
//
// Storage: row-major packed lower triangle, element (i, j), j <= i, at
// i (i + 1) / 2 + j, so a row's entries left of the diagonal are contiguous.
//
// The factorization has two levels of blocks.  Panels of NP = 256 columns are
// factored 64 columns at a time, one launch per 64 columns (k_chol_panel);
// after a panel, k_chol_syrk subtracts its product from the rest, 256 deep, so
// that the trailing matrix is read and written once per 256 columns and its
// tiles run at the rate of the FP64 product tiles.  Its first 256 columns (the
// next panel) go first, on the caller's stream; the rest runs on a helper
// stream beside the next panel's steps, which are a chain: every 64 columns
// wait for the 64 before.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ata.h"
#include "ata_device.h"
#include "ata_internal.h"
#include "ata_kernels.h"

namespace atalib {

namespace {

using detail::ProfScope;

constexpr int NB = 64;       // columns of a step
constexpr int NP = 4 * NB;   // columns of a panel

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef double d2_t __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ T buf_load(rsrc_t r, uint32_t off) {
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ void buf_store(rsrc_t r, uint32_t off, T x) {
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, x), r, (int)off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, x), r, (int)off, 0, 0);
}

// r = 1 / sqrt(d) for d with pivot_in_range: the hardware estimate y (22 bits or
// more) times the first terms of (1 - e)^(-1/2) in its residual e = 1 - d y^2,
// one dependent step of four operations (the chain of columns pays it once
// per column).  Exact where the result is a power of two.
__device__ __forceinline__ double rsqrt_in_range(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = __builtin_fma(-(d * y), y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ float rsqrt_in_range(float d) {
    const float y = __builtin_amdgcn_rsqf(d);
    const float e = __builtin_fmaf(-(d * y), y, 1.0f);
    return __builtin_fmaf(y * e, __builtin_fmaf(0.375f, e, 0.5f), y);
}
template <typename T>
__device__ __forceinline__ bool pivot_in_range(T d) {
    return sizeof(T) == 8 ? d > (T)0x1p-900 && d < (T)0x1p900 : d > (T)0x1p-100 && d < (T)0x1p100;
}

// ---------------------------------------------------------------------------
// Products X Y^T of row slices of the packed matrix.  A stage holds 128 bytes
// of each row (16 doubles or 32 floats of consecutive columns k): eight
// 16-byte chunks, chunk c of row r at position c ^ swz(r), copied by buffer
// loads that write LDS (eight rows an instruction; rows start on any multiple
// of the element size).  A 128-bit operand read gives a lane VK consecutive k
// of one row, one per MFMA; lane group g = lane >> 4 takes chunk 4 half + g,
// so the MFMA for element e sums k = VK (4 half + g) + e over g, the same for
// both operands.  swz sends the eight row pairs to eight positions, first
// telling rows r and r + 2 apart by 64 bytes: the 16 rows of a right operand
// and the 4 rows x 4 chunks of an FP64 left operand fall on distinct banks.
// MFMA forms as in the product tiles: FP64 4 x 16 x 4 (left operand four rows
// repeated), FP32 16 x 16 x 4.
// ---------------------------------------------------------------------------
constexpr int RB = 128;  // bytes of a staged row

__device__ __forceinline__ int swz(int row) {
    const int p = row >> 1;
    return (p & 1) << 2 | (p & 2) | (p >> 2 & 1);
}

template <typename T>
struct Mma;

template <>
struct Mma<double> {
    static constexpr int RM = 4, NE = 1, VK = 2;  // rows of a block, elements per lane, k per 16 bytes
    typedef double acc_t;
    typedef d2_t vec_t;
    __device__ static int arow(int lane) { return lane & 3; }
    __device__ static int orow(int lane, int) { return lane >> 4; }
    __device__ static double get(const acc_t& c, int) { return c; }
    __device__ static void sub(acc_t& c, int, double v) { c = v - c; }
    __device__ static acc_t zero() { return 0.0; }
    __device__ static void mma(double a, double b, acc_t& c) { c = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0); }
};
template <>
struct Mma<float> {
    static constexpr int RM = 16, NE = 4, VK = 4;
    typedef f4_t acc_t;
    typedef f4_t vec_t;
    __device__ static int arow(int lane) { return lane & 15; }
    __device__ static int orow(int lane, int e) { return 4 * (lane >> 4) + e; }
    __device__ static float get(const acc_t& c, int e) { return c[e]; }
    __device__ static void sub(acc_t& c, int e, float v) { c[e] = v - c[e]; }
    __device__ static acc_t zero() { return f4_t{0.f, 0.f, 0.f, 0.f}; }
    __device__ static void mma(float a, float b, acc_t& c) { c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

// acc (NR row blocks x NC column blocks of 16) += X Y^T over one stage; xa
// (first half of the row blocks), xb (second half) and y point to the first
// staged rows of this wave's operands (multiples of 16).
template <typename T, int NR, int NC>
__device__ __forceinline__ void mma_stage(const char* xa, const char* xb, const char* y, int lane,
                                          typename Mma<T>::acc_t (&acc)[NR][NC]) {
    typedef Mma<T> M;
    typedef typename M::vec_t V;
    const int g = lane >> 4;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        constexpr int GR = NR / 2 < 8 ? NR / 2 : 8;  // row blocks read at a time
        V b[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int row = 16 * c + (lane & 15);
            b[c] = *(const V*)(y + row * RB + 16 * ((4 * half + g) ^ swz(row)));
        }
#pragma unroll
        for (int r0 = 0; r0 < NR; r0 += GR) {
            V a[GR];
#pragma unroll
            for (int r = 0; r < GR; ++r) {
                const int row = M::RM * ((r0 + r) % (NR / 2)) + M::arow(lane);
                a[r] = *(const V*)((r0 < NR / 2 ? xa : xb) + row * RB + 16 * ((4 * half + g) ^ swz(row)));
            }
#pragma unroll
            for (int e = 0; e < M::VK; ++e)
#pragma unroll
                for (int r = 0; r < GR; ++r)
#pragma unroll
                    for (int c = 0; c < NC; ++c) M::mma(a[r][e], b[c][e], acc[r0 + r][c]);
        }
    }
}

// ---------------------------------------------------------------------------
// One step: columns [kb, kb + w), w <= 64, of a panel that starts at column
// pb.  Workgroup b owns 64 rows below the diagonal block, from kb + 64 + 64 b.
// Every workgroup also factors the diagonal block (a few microseconds, against
// a launch of its own plus a trip through memory), so a step is one launch:
//  1. The 128 rows (diagonal block, own rows) minus the panel's columns left
//     of kb, by MFMA (a wave: 32 rows x 64 columns), left in registers.
//  2. Sixteen columns at a time.  Wave 0 factors the diagonal block's part
//     with a row per lane; waves 0 and 1 then subtract its product from the
//     rest of the diagonal block.  Beside that chain, one step behind, waves 2
//     and 3 solve the own rows for the 16 columns (a row per lane) and
//     subtract their product from the columns to the right.
//  3. The rows are stored.  The diagonal block goes to `diag` (64 x 64), since
//     other workgroups may still read it in C; the next step's workgroup 0
//     puts it in place (`prev`, null for the first step).  A last block
//     without rows below is stored at once.
// A pivot that is not positive is reported once through `info` (first failing
// column + 1, LAPACK's convention); the factorization carries on.
// SHORT: a matrix of at most 48 columns; the sixteens past its end are left out
// (an instance of its own, which keeps the chain of larger factors as it is: FP64
// n = 8 18.0 -> 12.9 us a call, n = 40 19.4 -> 14.4).
// LDS 79 KB (FP64) and 256 registers: beside one workgroup of the update on the
// same CU.
// Measured alone (MI355X): see potrf_t.
// ---------------------------------------------------------------------------
// Row stride of the factored columns in LDS: 16 rows apart by distinct 16-byte
// bank groups, for 128-bit reads by rows.
template <typename T>
constexpr int kLB = sizeof(T) == 8 ? 66 : 68;
constexpr int SX = 17;  // row stride of the diagonal block's 16 columns handed to the row lanes

// Columns [16 s, 16 s + 16) of the diagonal block, lane = row.  The chain from
// one pivot to the next runs on values every lane holds: with X = D[c+1][c]
// and P = D[c+1][c+1] broadcast a column ahead, the next pivot is P - (X r)^2,
// the operation row c + 1 does itself.  The multipliers of columns beyond the
// next two pass through LDS (mb, two columns of 64) and are used a column
// later, off that chain.  A scaled pivot is its root, to an ulp.  Returns
// false if a pivot is out of the range of rsqrt_in_range.
template <typename T>
__device__ __forceinline__ bool factor16(T (&d)[16], T* mb, int b0, int lane) {
    typedef T v2_t __attribute__((ext_vector_type(2)));
    T piv = lane_bcast(d[0], b0), X = lane_bcast(d[0], b0 + 1), P = lane_bcast(d[1], b0 + 1);
    T r = rsqrt_in_range(piv);
    bool ok = pivot_in_range(piv);
    v2_t mv[7];  // multipliers 2.. of the column before, read while it was scaled
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        // the scheduler fills the chain to the next root with updates; keeping
        // it from reaching further bounds the registers
        __builtin_amdgcn_sched_barrier(0);
        const T rc = r;
        // the column before, for the columns its multipliers came through LDS
        if (c >= 1 && c < 14) {
#pragma unroll
            for (int k = 2; k < 16; ++k)
                if (k >= c + 2) d[k] -= d[c - 1] * mv[k / 2 - 1][k & 1];
        }
        d[c] *= rc;
        if (c < 13) mb[(c & 1) * NB + lane] = d[c];
        if (c < 15) {
            const T l = X * rc;
            piv = P - l * l;
            r = rsqrt_in_range(piv);
            ok = ok && pivot_in_range(piv);
            d[c + 1] -= d[c] * l;
        }
        if (c < 14) {
            d[c + 2] -= d[c] * lane_bcast(d[c], b0 + c + 2);
            X = lane_bcast(d[c + 1], b0 + c + 2);
            P = lane_bcast(d[c + 2], b0 + c + 2);
        }
        if (c < 13) {
            wave_lds_fence();
#pragma unroll
            for (int k = 2; k < 16; k += 2)
                if (k + 1 >= c + 3) mv[k / 2 - 1] = *(const v2_t*)&mb[(c & 1) * NB + b0 + k];
        }
    }
    return ok;
}

// The same columns for any pivot, with the plain square root and reciprocal,
// in place in LDS (sx, a row per lane); reports the first pivot that is not
// positive through info.
template <typename T>
__device__ __noinline__ void factor16_any(T* sx, int b0, int lane, int32_t* info, int64_t kb, int w) {
#pragma clang loop unroll(disable)
    for (int c = 0; c < 16; ++c) {
        const T piv = sx[(b0 + c) * SX + c];
        const T root = sqrt(piv), r = T(1) / root;
        if (info && !(piv > T(0)) && b0 + c < w && lane == 0) atomicCAS(info, 0, (int32_t)(kb + b0 + c + 1));
        const T x = lane == b0 + c ? root : sx[lane * SX + c] * r;
        wave_lds_fence();
        sx[lane * SX + c] = x;
        wave_lds_fence();
#pragma clang loop unroll(disable)
        for (int k = c + 1; k < 16; ++k) {
            const T m = sx[(b0 + k) * SX + c];
            sx[lane * SX + k] -= x * m;
        }
        wave_lds_fence();
    }
}

// Workgroup barrier for LDS data alone.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <typename T, bool SHORT>
__global__ __launch_bounds__(256, 2) void k_chol_panel(T* __restrict__ C, int64_t n, int64_t pb, int64_t kb, int w,
                                                    int32_t* __restrict__ info, T* __restrict__ diag,
                                                    const T* __restrict__ prev) {
    typedef Mma<T> M;
    typedef typename M::vec_t V;
    constexpr int NR = 32 / M::RM, NE = M::NE, KS = RB / (int)sizeof(T), LB = kLB<T>;
    constexpr int NBUF = sizeof(T) == 8 ? 4 : 2;  // stages in flight
    constexpr int NJ = 4 / M::VK;                 // 128-bit reads per row of 16 columns and lane group
    __shared__ __attribute__((aligned(16))) T lb[2 * NB * LB];
    __shared__ T sx[NB * SX];
    __shared__ __attribute__((aligned(16))) T mb[2 * NB];
    __shared__ T rw[2][16];  // reciprocals of the 16 pivots, for each own wave
    static_assert(NBUF * 128 * RB <= sizeof(lb), "stages of 128 rows");
    // on the critical path while the helper stream's update fills the CUs
    __builtin_amdgcn_s_setprio(3);
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t r0 = kb + NB + (int64_t)NB * blockIdx.x;  // first own row
    const bool own = r0 < n;
    // This wave's two groups of 16 of the 128 rows.  Waves 0 and 1 share the
    // lower triangle of the diagonal block: groups 0 and 3, 1 and 2.
    const int ga = wv < 2 ? wv : 2 * wv, gb = wv < 2 ? 3 - wv : 2 * wv + 1;

    // C values of this wave's rows
    typename M::acc_t v[NR][4];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int row = 16 * (r < NR / 2 ? ga : gb) + M::RM * (r % (NR / 2)) + M::orow(lane, e);
                const int64_t i = row < NB ? kb + row : r0 + (row - NB), j = kb + 16 * c + (lane & 15);
                // a short last block is continued by the identity
                T x = i == j ? T(1) : T(0);
                if (i < n && j <= i) x = C[pidx(i, j)];
                if constexpr (NE == 1)
                    v[r][c] = x;
                else
                    v[r][c][e] = x;
            }
    if (kb > pb) {
        // minus the product with the panel's columns [pb, kb)
        char* const st = (char*)lb;
        const int64_t b0 = wv < 2 ? kb : r0;  // rows this wave copies: 32 of the 128
        const int64_t first = b0 < n ? b0 : n - 1;
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(C + pidx(first, pb), (short)0, 0x7fffffff, 0x00020000);
        uint32_t off[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 32 * (wv & 1) + 8 * i + (lane >> 3);  // of the 64 rows from b0
            const int64_t gi = b0 + row < n ? b0 + row : n - 1;
            off[i] = (uint32_t)((pidx(gi, pb) - pidx(first, pb)) * (int64_t)sizeof(T)) +
                     16u * (uint32_t)((lane & 7) ^ swz(row));
        }
        auto copy = [&](int k, int buf) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                lds_copy16(rs, st + (buf * 128 + 32 * wv + 8 * i) * RB, off[i], (uint32_t)(k * RB));
        };
        typename M::acc_t acc[NR][4];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[r][c] = M::zero();
        const int ns = (int)(kb - pb) / KS;  // a multiple of 4 (FP64) or 2 (FP32)
#pragma unroll
        for (int k = 0; k < NBUF - 1; ++k) copy(k, k);
        for (int k = 0; k < ns; ++k) {
            // this wave's copies of stage k have landed (four per stage; up
            // to two later stages stay in flight)
            if (NBUF == 4 && k + 2 < ns)
                asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else if (NBUF == 4 && k + 1 < ns)
                asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            // everyone's have, and the oldest buffer is read (a bare barrier:
            // a fence would wait for the later stages too)
            lds_barrier();
            if (k + NBUF - 1 < ns) copy(k + NBUF - 1, (k + NBUF - 1) % NBUF);
            const char* x = st + (k % NBUF) * 128 * RB;
            mma_stage<T, NR, 4>(x + 16 * ga * RB, x + 16 * gb * RB, x, lane, acc);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[r][c] -= acc[r][c];
        if (w < NB) {
            // rows past the end: the identity again (their copies repeat the last row)
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int e = 0; e < NE; ++e)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int row = 16 * (r < NR / 2 ? ga : gb) + M::RM * (r % (NR / 2)) + M::orow(lane, e);
                        const T x = row == 16 * c + (lane & 15) ? T(1) : T(0);
                        if constexpr (NE == 1)
                            v[r][c] = row >= w ? x : v[r][c];
                        else
                            v[r][c][e] = row >= w ? x : v[r][c][e];
                    }
        }
        lds_barrier();  // the stages are read: lb is free
    }

    // columns [16 s, 16 s + 16) of this wave's rows to p (row stride st, first
    // of the rows row0)
    auto put = [&](int s, T* p, int st, int row0) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int row = 16 * (r < NR / 2 ? ga : gb) + M::RM * (r % (NR / 2)) + M::orow(lane, e);
                p[(row - row0) * st + (lane & 15)] = M::get(v[r][s], e);
            }
    };
    // The factored 16 columns from 16 s: minus the product of this wave's rows
    // with rows 16 c .. of the diagonal block, in its column blocks c > s (of
    // the diagonal block the lower ones).  Lane group g takes the k of one
    // 128-bit read, the same for both operands.
    auto update = [&](int s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int gr = h == 0 ? ga : gb;
            V a[NJ][NR / 2];
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < NR / 2; ++r)
                    a[j][r] = -*(const V*)&lb[(16 * gr + M::RM * r + M::arow(lane)) * LB + 16 * s + (4 * j + g) * M::VK];
#pragma unroll
            for (int c = 1; c < 4; ++c)
                if (c > s && c <= gr)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const V b = *(const V*)&lb[(16 * c + (lane & 15)) * LB + 16 * s + (4 * j + g) * M::VK];
#pragma unroll
                        for (int e = 0; e < M::VK; ++e)
#pragma unroll
                            for (int r = 0; r < NR / 2; ++r) M::mma(a[j][r][e], b[e], v[h * (NR / 2) + r][c]);
                    }
        }
    };
    if (wv < 2) {
        put(0, sx, SX, 0);
        lds_barrier();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (SHORT && 16 * s >= w) break;
            if (wv == 0) {
                T d[16];
#pragma unroll
                for (int c = 0; c < 16; ++c) d[c] = sx[lane * SX + c];
                if (!factor16<T>(d, mb, 16 * s, lane)) {
                    factor16_any<T>(sx, 16 * s, lane, blockIdx.x == 0 ? info : nullptr, kb, w);
#pragma unroll
                    for (int c = 0; c < 16; ++c) d[c] = sx[lane * SX + c];
                }
#pragma unroll
                for (int c = 0; c < 16; ++c) lb[lane * LB + 16 * s + c] = d[c];
            }
            lds_barrier();
            if (s < 3) {
                update(s);
                put(s + 1, sx, SX, 0);
            }
            lds_barrier();
        }
    } else {
        lds_barrier();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (SHORT && 16 * s >= w) break;
            lds_barrier();
            lds_barrier();
            if (SHORT) continue;  // no own rows
            // lanes l and l + 32 both hold own row 32 (wv - 2) + (l & 31)
            put(s, lb + NB * LB + 16 * s, LB, NB);
            if (lane < 16) rw[wv - 2][lane] = T(1) / lb[(16 * s + lane) * LB + 16 * s + lane];
            wave_lds_fence();
            T* const row = &lb[(NB + 32 * (wv - 2) + (lane & 31)) * LB + 16 * s];
            T o[16];
#pragma unroll
            for (int c = 0; c < 16; c += M::VK) {
                const V x = *(const V*)&row[c];
#pragma unroll
                for (int e = 0; e < M::VK; ++e) o[c + e] = x[e];
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const T* lk = &lb[(16 * s + k) * LB + 16 * s];
#pragma unroll
                for (int c = 0; c < 16; c += M::VK)
                    if (c < k) {
                        const V m = *(const V*)&lk[c];
#pragma unroll
                        for (int e = 0; e < M::VK; ++e)
                            if (c + e < k) o[k] -= o[c + e] * m[e];
                    }
                o[k] *= rw[wv - 2][k];
            }
            wave_lds_fence();
#pragma unroll
            for (int c = 0; c < 16; c += M::VK) {
                V x;
#pragma unroll
                for (int e = 0; e < M::VK; ++e) x[e] = o[c + e];
                *(V*)&row[c] = x;
            }
            wave_lds_fence();
            if (s < 3) update(s);
        }
    }
    __syncthreads();

    // rows to memory, a row per wave and pass
    if (own)
        for (int r = wv; r < NB; r += 4)
            if (r0 + r < n) C[pidx(r0 + r, kb + lane)] = lb[(NB + r) * LB + lane];
    if (blockIdx.x == 0) {
        for (int r = wv; r < w; r += 4) {
            const T x = lb[r * LB + lane];
            if (own)
                diag[r * NB + lane] = x;
            else if (lane <= r)
                C[pidx(kb + r, kb + lane)] = x;
            if (prev && lane <= r) C[pidx(kb - NB + r, kb - NB + lane)] = prev[r * NB + lane];
        }
        if (prev)  // rows of the previous block beyond a short one
            for (int r = w + wv; r < NB; r += 4)
                if (lane <= r) C[pidx(kb - NB + r, kb - NB + lane)] = prev[r * NB + lane];
    }
}

// ---------------------------------------------------------------------------
// Trailing update after the panel [pb, pb + NP): C[i][j] -= sum over the panel
// of L[i][k] L[j][k] for s0 <= j <= i < n, s0 = pb + NP, on UT x UT tiles from
// s0.  part 0 takes every tile, part 1 the first NP columns (the next panel),
// part 2 the others.  Four waves of UT/2 x UT/2, one stage ahead; the sum is
// formed first and subtracted once.  UT = 128 (two workgroups per CU) reads
// each operand half as often; UT = 64 gives four times the workgroups, each
// done in a quarter of the time: for the parts on the chain and for smaller
// trailing matrices.
// ---------------------------------------------------------------------------
// Row a and column c of linear index b in a lower triangle of tiles.
__device__ __forceinline__ void tri_decode(int64_t b, int64_t& a, int64_t& c) {
    a = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
    while (a * (a + 1) / 2 > b) --a;
    while ((a + 1) * (a + 2) / 2 <= b) ++a;
    c = b - a * (a + 1) / 2;
}

template <typename T, int UT>
__global__ __launch_bounds__(256, UT == 128 ? 2 : 4) void k_chol_syrk(T* __restrict__ C, int64_t n, int64_t pb,
                                                                    int part) {
    typedef Mma<T> M;
    constexpr int WT = UT / 2, NR = WT / M::RM, NC = WT / 16, NE = M::NE, KS = RB / (int)sizeof(T);
    constexpr int NPT = NP / UT;  // tile columns of the next panel
    constexpr int NI = UT / 16;   // copies of a wave per stage (eight rows each)
    __shared__ __attribute__((aligned(16))) char st[2][2 * UT * RB];
    int64_t ti, tj;
    if (part == 1) {
        // the first NPT tile columns: their triangle, then whole rows of NPT
        const int64_t b = blockIdx.x, tri = NPT * (NPT + 1) / 2;
        if (b < tri) {
            tri_decode(b, ti, tj);
        } else {
            ti = NPT + (b - tri) / NPT;
            tj = (b - tri) % NPT;
        }
    } else {
        tri_decode(blockIdx.x, ti, tj);
        if (part == 2) {
            ti += NPT;
            tj += NPT;
        }
    }
    const int64_t s0 = pb + NP, r0 = s0 + UT * ti, c0 = s0 + UT * tj;
    const bool dg = ti == tj;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wr = wv >> 1, wc = wv & 1;

    // this wave's copies: half of the left rows (waves 0, 1) or right rows
    const int64_t b0 = wv < 2 ? r0 : c0;
    const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(C + pidx(b0, pb), (short)0, 0x7fffffff, 0x00020000);
    uint32_t off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int row = WT * (wv & 1) + 8 * i + (lane >> 3);
        const int64_t gi = b0 + row < n ? b0 + row : n - 1;
        off[i] = (uint32_t)((pidx(gi, pb) - pidx(b0, pb)) * (int64_t)sizeof(T)) + 16u * (uint32_t)((lane & 7) ^ swz(row));
    }
    const bool copies = wv < 2 || !dg;
    auto copy = [&](int k, int buf) {
        if (!copies) return;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            lds_copy16(rs, &st[buf][(UT * (wv >> 1) + WT * (wv & 1) + 8 * i) * RB], off[i], (uint32_t)(k * RB));
    };
    typename M::acc_t acc[NR][NC];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[r][c] = M::zero();
    const bool live = !(dg && wr < wc);  // above the diagonal: copies only
    copy(0, 0);
#pragma clang loop unroll(disable)
    for (int k = 0; k < NP / KS; ++k) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (k + 1 < NP / KS) copy(k + 1, (k + 1) & 1);
        if (!live) continue;
        __builtin_amdgcn_s_setprio(1);
        const char* x = st[k & 1] + WT * wr * RB;
        mma_stage<T, NR, NC>(x, x + WT / 2 * RB, st[k & 1] + ((dg ? 0 : UT) + WT * wc) * RB, lane, acc);
        __builtin_amdgcn_s_setprio(0);
    }
    if (!live) return;
    // C in batches of up to 32 values, the loads of a batch in flight
    // together.  Row k of this wave starts k Ru + k (k + 1) / 2 elements after
    // its first row Ru.
    constexpr int GR = NR < 8 / NE ? NR : 8 / NE;
    const int64_t Ru = r0 + WT * wr, cu = c0 + WT * wc;
    const rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(C + pidx(Ru, cu), (short)0, 0x7fffffff, 0x00020000);
    const bool inside = !dg && r0 + UT <= n;
    uint32_t l0 = lane & 15;
    asm volatile("" : "+v"(l0));  // the offsets are formed here, not kept through the loop
    auto at = [&](int r, int e) {
        const uint32_t k = M::RM * r + M::orow(lane, e);
        return (k * (uint32_t)Ru + k * (k + 1) / 2 + l0) * (uint32_t)sizeof(T);
    };
    auto in = [&](int r, int e, int c) {
        const int64_t i = Ru + M::RM * r + M::orow(lane, e);
        return i < n && cu + 16 * c + (int64_t)l0 <= i;
    };
#pragma unroll
    for (int q = 0; q < NR; q += GR) {
        T cv[GR][NE][NC];
        if (inside) {
#pragma unroll
            for (int r = 0; r < GR; ++r)
#pragma unroll
                for (int e = 0; e < NE; ++e)
#pragma unroll
                    for (int c = 0; c < NC; ++c) cv[r][e][c] = buf_load<T>(rc, at(q + r, e) + 16u * c * (uint32_t)sizeof(T));
#pragma unroll
            for (int r = 0; r < GR; ++r)
#pragma unroll
                for (int e = 0; e < NE; ++e)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        buf_store<T>(rc, at(q + r, e) + 16u * c * (uint32_t)sizeof(T), cv[r][e][c] - M::get(acc[q + r][c], e));
            continue;
        }
#pragma unroll
        for (int r = 0; r < GR; ++r)
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    cv[r][e][c] = in(q + r, e, c) ? buf_load<T>(rc, at(q + r, e) + 16u * c * (uint32_t)sizeof(T)) : T(0);
#pragma unroll
        for (int r = 0; r < GR; ++r)
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (in(q + r, e, c))
                        buf_store<T>(rc, at(q + r, e) + 16u * c * (uint32_t)sizeof(T), cv[r][e][c] - M::get(acc[q + r][c], e));
    }
}

// The factorization on s with a helper stream s2 and two events.  Ordering:
// the rest of the update after panel p waits for the panel (event e); the
// next panel's part of the update after panel p + 1 waits for the rest of the
// update after p (event f), whose tiles it overlaps; s joins s2 at the end.
// Trailing matrices of at most kOneLaunch 64 x 64 tiles take one launch on s:
// it lasts no longer than the next panel's part, and the events cost more
// than the overlap brings.
// Beyond the next panel, trailing matrices of at most kSmallTiles 64 x 64 tiles
// take those tiles and larger ones 128 x 128: a step waits for workgroup slots
// that a 128 x 128 tile holds for 86 us, so the smaller tiles are faster
// wherever the steps are the longer chain (n = 4000 2362 -> 2282 us, 6000 4119
// -> 4031, 10000 10620 -> 10470 us), and slower where the updates are (all of
// n = 10000 on them 11110 us); a line at 3500 or 5500 rows gains less.
// ws: two 64 x 64 blocks (n <= 64: none).
// Measured (FP64): a step alone takes 16 us with no panel columns to its left
// and 6 us more for every 64 (its diagonal block alone took 67 us and the rows
// below 51 us as launches of their own); the first update at n = 10000 takes
// 477 us alone, 50 TFLOP/s.  Factor at n = 10000 25.9 -> 10.5 ms, of which the
// updates are bound by the tiles and, from about 5000 columns on, the rest by
// the chain of steps: n = 2048 3.4 -> 1.0 ms.
constexpr int64_t kOneLaunch = 600, kSmallTiles = 2500;

template <typename T>
hipError_t potrf_t(T* C, int64_t n, int32_t* info, T* ws, hipStream_t s, hipStream_t s2, hipEvent_t e, hipEvent_t f) {
    bool rest_pending = false;
    hipError_t err;
    for (int64_t pb = 0; pb < n; pb += NP) {
        const int64_t pe = n < pb + NP ? n : pb + NP;
        {
            ProfScope ps(ATA_KERNEL_FACTOR_PANEL, s);
            for (int64_t kb = pb; kb < pe; kb += NB) {
                const int w = (int)(n - kb < NB ? n - kb : NB);
                const int64_t rest = n - kb - w, step = kb / NB;
                if (n <= 3 * NB / 4)
                    hipLaunchKernelGGL((k_chol_panel<T, true>), dim3(1), dim3(256), 0, s, C, n, pb, kb, w, info,
                                       (T*)nullptr, (const T*)nullptr);
                else
                    hipLaunchKernelGGL((k_chol_panel<T, false>),
                                       dim3((unsigned)(rest > 0 ? (rest + NB - 1) / NB : 1)), dim3(256), 0, s, C, n,
                                       pb, kb, w, info, ws + (step & 1) * NB * NB,
                                       kb > 0 ? ws + ((step - 1) & 1) * NB * NB : (const T*)nullptr);
                if ((err = hipGetLastError()) != hipSuccess) return err;
            }
        }
        if (pe >= n) break;
        if (rest_pending && (err = hipStreamWaitEvent(s, f, 0)) != hipSuccess) return err;
        rest_pending = false;
        const int64_t t64 = (n - pe + 63) / 64, all = t64 * (t64 + 1) / 2;
        if (all <= kOneLaunch) {
            ProfScope ps(ATA_KERNEL_FACTOR_UPDATE, s);
            hipLaunchKernelGGL((k_chol_syrk<T, 64>), dim3((unsigned)all), dim3(256), 0, s, C, n, pb, 0);
            if ((err = hipGetLastError()) != hipSuccess) return err;
            continue;
        }
        if ((err = hipEventRecord(e, s)) != hipSuccess) return err;
        if ((err = hipStreamWaitEvent(s2, e, 0)) != hipSuccess) return err;
        {
            constexpr int64_t np = NP / 64;
            ProfScope ps(ATA_KERNEL_FACTOR_UPDATE, s);
            hipLaunchKernelGGL((k_chol_syrk<T, 64>), dim3((unsigned)(np * (np + 1) / 2 + (t64 - np) * np)), dim3(256),
                               0, s, C, n, pb, 1);
            if ((err = hipGetLastError()) != hipSuccess) return err;
        }
        {
            ProfScope ps(ATA_KERNEL_FACTOR_UPDATE, s2);
            // tile rows beyond the next panel
            if (all <= kSmallTiles) {
                const int64_t t = t64 - NP / 64;
                hipLaunchKernelGGL((k_chol_syrk<T, 64>), dim3((unsigned)(t * (t + 1) / 2)), dim3(256), 0, s2, C, n, pb,
                                   2);
            } else {
                const int64_t t = (n - pe + 127) / 128 - NP / 128;
                hipLaunchKernelGGL((k_chol_syrk<T, 128>), dim3((unsigned)(t * (t + 1) / 2)), dim3(256), 0, s2, C, n, pb,
                                   2);
            }
            if ((err = hipGetLastError()) != hipSuccess) return err;
        }
        if ((err = hipEventRecord(f, s2)) != hipSuccess) return err;
        rest_pending = true;
    }
    if (rest_pending && (err = hipStreamWaitEvent(s, f, 0)) != hipSuccess) return err;
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Transpose for the companion product A A^t: out (n x m, row stride m) =
// A^t for A (m x n, row stride lda), 64 x 64 tiles through LDS so that both
// the reads of A's rows and the writes of out's rows are contiguous.
// E: element type of 4 or 8 bytes (moved as raw bits).
// ---------------------------------------------------------------------------
template <typename E>
__global__ __launch_bounds__(256) void k_transpose(const E* __restrict__ A, int64_t m, int64_t n, int64_t lda,
                                                   E* __restrict__ out) {
    __shared__ E tile[64][65];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * 64, r0 = (int64_t)blockIdx.y * 64;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int r = wv + 4 * u;
        if (r0 + r < m && c0 + lane < n) tile[r][lane] = A[(r0 + r) * lda + c0 + lane];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int c = wv + 4 * u;
        if (c0 + c < n && r0 + lane < m) out[(c0 + c) * m + r0 + lane] = tile[lane][c];
    }
}

}  // namespace

hipError_t launch_transpose(int elem_bytes, const void* A, int64_t m, int64_t n, int64_t lda, void* out,
                            hipStream_t s) {
    const dim3 grid((unsigned)((n + 63) / 64), (unsigned)((m + 63) / 64));
    if (elem_bytes == 8)
        hipLaunchKernelGGL(k_transpose<uint64_t>, grid, dim3(256), 0, s, (const uint64_t*)A, m, n, lda,
                           (uint64_t*)out);
    else
        hipLaunchKernelGGL(k_transpose<uint32_t>, grid, dim3(256), 0, s, (const uint32_t*)A, m, n, lda,
                           (uint32_t*)out);
    return hipGetLastError();
}

// A single block writes C itself.
size_t potrf_ws_bytes(int64_t n) { return n <= NB ? 0 : 2 * NB * NB * sizeof(double); }

hipError_t launch_potrf(bool f32, void* C, int64_t n, int32_t* info, void* ws, hipStream_t s, hipStream_t s2,
                        hipEvent_t e, hipEvent_t f) {
    return f32 ? potrf_t((float*)C, n, info, (float*)ws, s, s2, e, f)
               : potrf_t((double*)C, n, info, (double*)ws, s, s2, e, f);
}

}  // namespace atalib
