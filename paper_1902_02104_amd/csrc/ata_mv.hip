// A^t B and A X of gfx950 for a few right-hand sides: the right-hand side A^t b
// of the normal equations and the product that applies the projection
// A (A^t A)^-1 A^t (Section 1 names both as uses of A^t A).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ata.h"
#include "ata_internal.h"
#include "ata_kernels.h"

namespace atalib {

namespace {

using detail::ProfScope;

// ---------------------------------------------------------------------------
// A^t B: FP64 partial sums over row chunks, then a pass that adds the chunks.
// Workgroup = 64 columns x one chunk x RC right-hand sides: lane = column;
// tiles of 64 rows, sixteen of them per wave with all their loads in flight.
// The tile's rows of B go through LDS (every lane reads the same entry);
// scalar loads of them came one at a time.  The four waves' sums are added in
// wave order.  Bound by the read of A where that is long (FP64 262144 x 2048,
// one right-hand side: 6.2 TB/s, 860 -> 693 us a call; seven: 1065 -> 735),
// else by the launches; one thread per column with one row in flight took
// 121 us for FP32 20011 x 333 and four right-hand sides, now 11, and read A
// once per eight right-hand sides instead of sixteen.
// ---------------------------------------------------------------------------
template <typename T, int RC>
__global__ __launch_bounds__(256) void k_atb_part(const T* __restrict__ A, int64_t m, int64_t n, int64_t lda,
                                                  const T* __restrict__ B, int64_t nrhs, int64_t ldb, int64_t rows,
                                                  double* __restrict__ part, T* __restrict__ out, int64_t ldo,
                                                  int64_t c0) {
    constexpr int U = 16, BT = 4 * U, BE = (BT * RC + 255) / 256;
    __shared__ __attribute__((aligned(16))) double bs[BT * RC];
    __shared__ double red[4][RC][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j = c0 + (int64_t)blockIdx.x * 64 + lane;
    const int64_t ch = blockIdx.y;
    const int64_t i0 = ch * rows;
    const int64_t i1 = i0 + rows < m ? i0 + rows : m;
    const T* a = A + (j < n ? j : n - 1);
    for (int64_t r0 = (int64_t)blockIdx.z * RC; r0 < nrhs; r0 += (int64_t)gridDim.z * RC) {
        double acc[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) acc[r] = 0.0;
        for (int64_t t = i0; t < i1; t += BT) {
            const int64_t i = t + wave * U;
            T v[U];
            if (i + U <= i1) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = a[(i + u) * lda];
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = i + u < i1 ? a[(i + u) * lda] : T(0);
            }
            T bv[BE];
#pragma unroll
            for (int q = 0; q < BE; ++q) {
                const int e = threadIdx.x + 256 * q;
                const int64_t row = t + e / RC, c = r0 + e % RC;
                bv[q] = e < BT * RC && row < i1 && c < nrhs ? B[row * ldb + c] : T(0);
            }
            __syncthreads();  // the tile before has been read
#pragma unroll
            for (int q = 0; q < BE; ++q)
                if (threadIdx.x + 256 * q < BT * RC) bs[threadIdx.x + 256 * q] = (double)bv[q];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < RC; ++r) acc[r] += (double)v[u] * bs[(wave * U + u) * RC + r];
        }
#pragma unroll
        for (int r = 0; r < RC; ++r) red[wave][r][lane] = acc[r];
        __syncthreads();
        for (int r = wave; r < RC; r += 4)
            if (j < n && r0 + r < nrhs) {
                const double v = (red[0][r][lane] + red[1][r][lane]) + (red[2][r][lane] + red[3][r][lane]);
                if (part)
                    part[(ch * nrhs + r0 + r) * n + j] = v;
                else  // the only chunk
                    out[j * ldo + r0 + r] = (T)v;
            }
        __syncthreads();
    }
}

// Sum over the chunks in a fixed order: 64 consecutive elements per
// workgroup, sixteen waves over the chunks (residues mod 16), then the waves
// in order (FP32 20011 x 333: 79 chunks in one chain 21 us, 313 now 5).  The
// workgroups are a grid of two dimensions: sixteen threads an element reach
// the 2^32 threads of one dimension at 2^28 elements.
template <typename T>
__global__ __launch_bounds__(1024) void k_atb_sum(const double* __restrict__ part, int64_t chunks, int64_t n,
                                                  int64_t nrhs, T* __restrict__ out, int64_t ldo) {
    __shared__ double red[16][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t total = n * nrhs;
    const int64_t e = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 64 + lane;
    double s = 0.0;
    if (e < total)
#pragma unroll 8
        for (int64_t c = g; c < chunks; c += 16) s += part[c * total + e];
    red[g][lane] = s;
    __syncthreads();
    if (g || e >= total) return;
#pragma unroll
    for (int q = 1; q < 16; ++q) s += red[q][lane];
    out[(e % n) * ldo + e / n] = (T)s;
}

// ---------------------------------------------------------------------------
// A X for the projection A (A^t A)^-1 A^t B: four rows of A per wave, lanes
// striding their n entries (contiguous loads), so each entry of X that is
// loaded serves four rows.  The 4 RC sums over the lanes are formed together:
// each step halves the values a lane holds as it halves the lanes that hold
// one, 4 RC - 1 exchanges and a few for the rest instead of six for each.
// A row of X is read RC elements at a time, past nrhs too (kAxPad elements
// follow X; sums of those columns are dropped).
// Bound by the reads of X through the L1s where n is small, else by A: FP32
// 20011 x 333 x 4 38 us with a row per wave and single loads of X, now 12;
// 20000 x 2000 x 8 587 -> 35; FP64 262144 x 2048 x 1 6.2 TB/s.
// ---------------------------------------------------------------------------
// RC consecutive elements at any element address, in loads of up to 16 bytes.
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef double d2u_t __attribute__((ext_vector_type(2), aligned(8)));
template <int RC>
__device__ __forceinline__ void load_run(const float* p, float (&o)[RC]) {
    if constexpr (RC == 1) {
        o[0] = p[0];
    } else if constexpr (RC == 2) {
        const f2u_t v = *(const f2u_t*)p;
        o[0] = v[0];
        o[1] = v[1];
    } else {
#pragma unroll
        for (int q = 0; q < RC; q += 4) {
            const f4u_t v = *(const f4u_t*)(p + q);
#pragma unroll
            for (int k = 0; k < 4; ++k) o[q + k] = v[k];
        }
    }
}
template <int RC>
__device__ __forceinline__ void load_run(const double* p, double (&o)[RC]) {
    if constexpr (RC == 1) {
        o[0] = p[0];
    } else {
#pragma unroll
        for (int q = 0; q < RC; q += 2) {
            const d2u_t v = *(const d2u_t*)(p + q);
            o[q] = v[0];
            o[q + 1] = v[1];
        }
    }
}

template <int HALF, int O, int N>
__device__ __forceinline__ void lane_sums(double (&v)[N], int lane) {
    if constexpr (HALF > 0) {
        const bool up = lane & O;
#pragma unroll
        for (int k = 0; k < HALF; ++k) {
            const double send = up ? v[k] : v[k + HALF], keep = up ? v[k + HALF] : v[k];
            v[k] = keep + __shfl_xor(send, O, 64);
        }
    } else {
        v[0] += __shfl_xor(v[0], O, 64);
    }
    if constexpr (O > 1) lane_sums<HALF / 2, O / 2>(v, lane);
}

template <typename T, int RC>
__global__ __launch_bounds__(256) void k_ax(const T* __restrict__ A, int64_t m, int64_t n, int64_t lda,
                                            const T* __restrict__ X, int64_t nrhs, int64_t ldx, T* __restrict__ out,
                                            int64_t ldo) {
    constexpr int R = 4, N = R * RC;
    static_assert(N <= 64, "");
    const int lane = threadIdx.x & 63;
    const int64_t i = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
    if (i >= m) return;  // whole waves leave; no barrier follows
    const T* a[R];       // the last row again past the end
#pragma unroll
    for (int q = 0; q < R; ++q) a[q] = A + (i + q < m ? i + q : m - 1) * lda;
    for (int64_t r0 = 0; r0 < nrhs; r0 += RC) {
        double acc[N];
#pragma unroll
        for (int k = 0; k < N; ++k) acc[k] = 0.0;
        // UJ x 64 entries of each row at a time, all their loads in flight
        // (twice as many: 22 us against 18 at 20011 x 333 x 4)
        constexpr int UJ = RC <= 4 ? 2 : 1;
        for (int64_t j0 = lane; j0 < n; j0 += 64 * UJ) {
            T v[UJ][R], xv[UJ][RC];
#pragma unroll
            for (int u = 0; u < UJ; ++u) {
                const int64_t j = j0 + 64 * u;
                const bool in = j < n;
#pragma unroll
                for (int q = 0; q < R; ++q) v[u][q] = in ? a[q][j] : T(0);
                if (in)
                    load_run<RC>(X + j * ldx + r0, xv[u]);
                else
#pragma unroll
                    for (int r = 0; r < RC; ++r) xv[u][r] = T(0);
            }
#pragma unroll
            for (int u = 0; u < UJ; ++u)
#pragma unroll
                for (int r = 0; r < RC; ++r)
#pragma unroll
                    for (int q = 0; q < R; ++q) acc[q * RC + r] += (double)v[u][q] * (double)xv[u][r];
        }
        lane_sums<N / 2, 32>(acc, lane);
        const int k = lane / (64 / N);  // the sum this lane holds
        const int q = k / RC, r = k % RC;
        if (lane % (64 / N) == 0 && i + q < m && r0 + r < nrhs) out[(i + q) * ldo + r0 + r] = (T)acc[0];
    }
}

template <typename T, int RC>
void part_rc(const T* A, int64_t m, int64_t n, int64_t lda, const T* B, int64_t nrhs, int64_t ldb, double* part,
             int64_t chunks, T* out, int64_t ldo, hipStream_t s) {
    static_assert(RC <= kAtbPass, "");
    const int64_t rows = (m + chunks - 1) / chunks, passes = (nrhs + RC - 1) / RC;
    // columns in slices of 2^29 (2^31 threads): a grid dimension holds less than 2^32 threads
    constexpr int64_t kSlice = (int64_t)1 << 29;
    for (int64_t c0 = 0; c0 < n; c0 += kSlice) {
        const int64_t w = n - c0 < kSlice ? n - c0 : kSlice;
        const dim3 g((unsigned)((w + 63) / 64), (unsigned)chunks, (unsigned)(passes < 16384 ? passes : 16384));
        hipLaunchKernelGGL((k_atb_part<T, RC>), g, dim3(256), 0, s, A, m, n, lda, B, nrhs, ldb, rows, part, out, ldo,
                           c0);
    }
}

template <typename T>
hipError_t atb_t(const T* A, int64_t m, int64_t n, int64_t lda, const T* B, int64_t nrhs, int64_t ldb, T* out,
                 int64_t ldo, double* part, hipStream_t s) {
    const int64_t ch = part ? atb_chunks(m, n, nrhs) : 1;
    ProfScope ps(ATA_KERNEL_SOLVE, s);
    if (nrhs == 1)
        part_rc<T, 1>(A, m, n, lda, B, nrhs, ldb, part, ch, out, ldo, s);
    else if (nrhs == 2)
        part_rc<T, 2>(A, m, n, lda, B, nrhs, ldb, part, ch, out, ldo, s);
    else if (nrhs <= 4)
        part_rc<T, 4>(A, m, n, lda, B, nrhs, ldb, part, ch, out, ldo, s);
    else if (nrhs <= 8)
        part_rc<T, 8>(A, m, n, lda, B, nrhs, ldb, part, ch, out, ldo, s);
    else
        part_rc<T, kAtbPass>(A, m, n, lda, B, nrhs, ldb, part, ch, out, ldo, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !part) return e;
    const int64_t wgs = (n * nrhs + 63) / 64, gx = wgs < (1 << 20) ? wgs : 1 << 20;
    hipLaunchKernelGGL(k_atb_sum<T>, dim3((unsigned)gx, (unsigned)((wgs + gx - 1) / gx)), dim3(1024), 0, s, part, ch,
                       n, nrhs, out, ldo);
    return hipGetLastError();
}

template <typename T>
hipError_t ax_t(const T* A, int64_t m, int64_t n, int64_t lda, const T* X, int64_t nrhs, int64_t ldx, T* out,
                int64_t ldo, hipStream_t s) {
    ProfScope ps(ATA_KERNEL_SOLVE, s);
    const dim3 g((unsigned)((m + 15) / 16)), b(256);
    if (nrhs == 1)
        hipLaunchKernelGGL((k_ax<T, 1>), g, b, 0, s, A, m, n, lda, X, nrhs, ldx, out, ldo);
    else if (nrhs == 2)
        hipLaunchKernelGGL((k_ax<T, 2>), g, b, 0, s, A, m, n, lda, X, nrhs, ldx, out, ldo);
    else if (nrhs <= 4)
        hipLaunchKernelGGL((k_ax<T, 4>), g, b, 0, s, A, m, n, lda, X, nrhs, ldx, out, ldo);
    else if (nrhs <= 8 || sizeof(T) == 4)
        hipLaunchKernelGGL((k_ax<T, 8>), g, b, 0, s, A, m, n, lda, X, nrhs, ldx, out, ldo);
    else
        // FP64: half the passes over A (180786 x 576 x 9 329 -> 272 us); FP32
        // pays more for the conversions of unused columns (182 -> 216 us)
        hipLaunchKernelGGL((k_ax<T, 16>), g, b, 0, s, A, m, n, lda, X, nrhs, ldx, out, ldo);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_atb(bool f32, const void* A, int64_t m, int64_t n, int64_t lda, const void* B, int64_t nrhs,
                      int64_t ldb, void* out, int64_t ldo, double* part, hipStream_t s) {
    return f32 ? atb_t((const float*)A, m, n, lda, (const float*)B, nrhs, ldb, (float*)out, ldo, part, s)
               : atb_t((const double*)A, m, n, lda, (const double*)B, nrhs, ldb, (double*)out, ldo, part, s);
}

hipError_t launch_ax(bool f32, const void* A, int64_t m, int64_t n, int64_t lda, const void* X, int64_t nrhs,
                     int64_t ldx, void* out, int64_t ldo, hipStream_t s) {
    return f32 ? ax_t((const float*)A, m, n, lda, (const float*)X, nrhs, ldx, (float*)out, ldo, s)
               : ax_t((const double*)A, m, n, lda, (const double*)X, nrhs, ldx, (double*)out, ldo, s);
}

}  // namespace atalib
