// Triangular solves with the packed Cholesky factor on gfx950: L Y = B, then
// L^t X = Y, B row-major n x nrhs.
//
// What bounds a solve is its chain of 64-row diagonal blocks, not the bytes
// of L (400 MB at n = 10000, 0.1 ms each way): a block can only be solved
// after the one before it.  Each direction is one launch of one workgroup per
// block row (forward) or block column (backward) and per group of RC
// right-hand sides.  A workgroup streams its blocks of L into registers ahead
// of use, multiplies each with the solved values as soon as they appear, and
// solves its own diagonal block when the last of them is in.  The chain then
// costs, per two blocks, one trip of the solved values through memory, two
// sums over waves and 126 dependent multiply-adds, instead of two launches.
//
// Solved values pass between workgroups through a buffer that starts filled
// with a signalling-NaN pattern no arithmetic produces.  Each value is
// written and read as one relaxed atomic at agent scope, so a value that is
// seen is whole and needs no further ordering.  Workgroups take their blocks
// from a counter in the order of the chain: whoever holds a block waits only
// for blocks taken earlier, by workgroups that already run, so every wait
// ends whatever the number of resident workgroups.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ata.h"
#include "ata_device.h"
#include "ata_internal.h"
#include "ata_kernels.h"

namespace atalib {

namespace {

using detail::ProfScope;

constexpr int NB = 64;  // rows of a block

template <typename T>
struct Bits;
template <>
struct Bits<double> {
    typedef unsigned long long U;
    static constexpr U kUnset = 0x7FF4A5A5C3C3F00Dull;  // signalling NaN
    static constexpr U kQuiet = 0x7FF8000000000000ull;
};
template <>
struct Bits<float> {
    typedef unsigned int U;
    static constexpr U kUnset = 0x7FA5C3F1u;
    static constexpr U kQuiet = 0x7FC00000u;
};

template <typename T>
__device__ __forceinline__ void publish(T* p, T v) {
    typedef typename Bits<T>::U U;
    U b = __builtin_bit_cast(U, v);
    if (b == Bits<T>::kUnset) b = Bits<T>::kQuiet;
    __hip_atomic_store((U*)p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wait for the RC values at p, p + stride, ...  Next in the chain (near), two
// reads are kept in flight, so that a value is seen at most half a round trip
// after it can be; the others sleep about a microsecond between reads (every
// wave of the launch reads the same few lines, which would otherwise queue).
template <typename T, int RC>
__device__ __forceinline__ void await(const T* p, int64_t stride, T (&v)[RC], bool near) {
    typedef typename Bits<T>::U U;
    U b[2][RC];
    auto issue = [&](U (&x)[RC]) {
#pragma unroll
        for (int r = 0; r < RC; ++r)
            x[r] = __hip_atomic_load((const U*)(p + r * stride), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto ready = [&](const U (&x)[RC]) {
        bool ok = true;
#pragma unroll
        for (int r = 0; r < RC; ++r) ok = ok && x[r] != Bits<T>::kUnset;
        return __all(ok) != 0;
    };
    issue(b[0]);
    if (!near)
        while (!ready(b[0])) {
            __builtin_amdgcn_s_sleep(32);
            issue(b[0]);
        }
    else
        issue(b[1]);
    while (near) {
        if (ready(b[0])) break;
        issue(b[0]);
        if (ready(b[1])) {
#pragma unroll
            for (int r = 0; r < RC; ++r) b[0][r] = b[1][r];
            break;
        }
        issue(b[1]);
    }
#pragma unroll
    for (int r = 0; r < RC; ++r) v[r] = __builtin_bit_cast(T, b[0][r]);
}

template <typename T>
__global__ __launch_bounds__(256) void k_trsv_init(T* __restrict__ buf, int64_t count, int* __restrict__ counter) {
    typedef typename Bits<T>::U U;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e < count) ((U*)buf)[e] = Bits<T>::kUnset;
    if (e < 2) counter[e] = 0;
}

// Substitution with one 64 x 64 diagonal block: x (lane = row).  ld holds the
// block with column c (backward: row c) scaled by 1 / L[c][c] and zeros
// elsewhere, so that a step is one broadcast and one multiply-add, and rows
// already solved subtract zeros.  Where a value overflows or is not finite that
// product is a NaN in rows it must not reach: see solve_block.
template <typename T, bool FWD>
__device__ __forceinline__ T substitute(const T* ld, int lane, T x) {
    constexpr int LS = NB + 1;
    T d[2][16];  // 16 columns at a time, read ahead into registers
    auto cols = [&](int c0, T (&v)[16]) {
#pragma unroll
        for (int c = 0; c < 16; ++c) v[c] = FWD ? ld[lane * LS + c0 + c] : ld[(NB - 1 - c0 - c) * LS + lane];
    };
    cols(0, d[0]);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b < 3) cols(16 * (b + 1), d[(b + 1) & 1]);
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (16 * b + c < NB - 1)  // no row comes after the last
                x -= d[b & 1][c] * lane_bcast(x, FWD ? 16 * b + c : NB - 1 - (16 * b + c));
    }
    return x;
}

// The same steps with rows already solved left out and the block's entries as
// they are in L (first row and column d0, wd of them), for any value.
template <typename T, bool FWD>
__device__ __forceinline__ T column_steps(const T* __restrict__ L, int64_t d0, int wd, const T* rcp, int lane, T x) {
#pragma clang loop unroll(disable)
    for (int k = 0; k < wd; ++k) {
        const int c = FWD ? k : wd - 1 - k;
        const T xc = lane_bcast(x, c) * rcp[c];
        if (lane == c) x = xc;
        if (FWD ? lane > c && lane < wd : lane < c)
            x -= L[FWD ? pidx(d0 + lane, d0 + c) : pidx(d0 + c, d0 + lane)] * xc;
    }
    return x;
}

// Solution of a diagonal block (lane = row; zero past its wd rows).  A value
// that is not finite shows in its own row, so one vote over the finished rows
// finds every block that substitute may have got wrong (40 ns a block on the
// chain, what the step of the last column took).
template <typename T, bool FWD>
__device__ __forceinline__ T solve_block(const T* ld, const T* __restrict__ L, int64_t d0, int wd, const T* rcp,
                                         int lane, T x) {
    T v = substitute<T, FWD>(ld, lane, x) * rcp[lane];
    if (__builtin_expect(__any(lane < wd && !__builtin_isfinite(v)), 0))
        v = column_steps<T, FWD>(L, d0, wd, rcp, lane, x);
    return lane < wd ? v : T(0);
}

// Workgroup: the two neighbouring 64-row diagonal blocks 2 sb and 2 sb + 1
// and right-hand sides [ch RC, ch RC + RC).  Eight waves; the four of a half
// serve one diagonal block, lane = its row (backward: column), and share the
// 64 columns (rows) of every other block, 16 a wave, so that sums stay in one
// register per right-hand side until the four waves add theirs in LDS.
// Backward a wave reads 512-byte row segments of L (FP32: 256).  Forward each
// lane reads 128 bytes (64) of its own row; FP64 with one or two right-hand
// sides, where the stream of L is the bound at large n, reads four 128-byte
// segments a load instead and turns them in LDS (one right-hand side at
// n = 10000: 520 -> 380 us; FP32 and wider FP64 launches, which that LDS
// leaves with one workgroup per CU, are faster without: FP32 486 against 571
// us both ways, 33 FP64 right-hand sides 1.48 against 1.94 ms).  Blocks are
// read two ahead of use.  The half whose block comes first in the chain solves it and passes it
// on through LDS; the other half then applies the block between them and
// solves its own.  (Two blocks a workgroup: the trip through memory is paid
// half as often.)
// in / out: np-strided [rhs][row] buffers of the solved values; the forward
// launch takes its right-hand side from B, the backward one from `in` and
// also stores to B.
template <typename T, int RC, bool FWD>
__global__ __launch_bounds__(512) void k_trsv(const T* __restrict__ L, int64_t n, T* __restrict__ B, int64_t nrhs,
                                              int64_t ldb, int nsb, int nch, const T* __restrict__ in, T* out,
                                              int64_t np, int* __restrict__ counter) {
    constexpr int LS = NB + 1;
    __shared__ T ld[2][NB * LS];
    __shared__ T red[2][4 * NB * RC];
    __shared__ T rcp[2 * NB];
    __shared__ T ys[RC][NB];                                  // first block's solution
    __shared__ __attribute__((aligned(16))) T yw[8][RC][16];  // a wave's 16 values of a solved block
    // FP64, forward, up to two right-hand sides: blocks are turned in LDS
    constexpr bool TURN = FWD && sizeof(T) == 8 && RC <= 2;
    constexpr int TS = 17;  // row stride of a turned block
    __shared__ T tr[TURN ? 8 : 1][TURN ? NB * TS : 1];
    __shared__ int s_ticket;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    if (t == 0) s_ticket = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int tk = __builtin_amdgcn_readfirstlane(s_ticket);
    const int ch = tk % nch, sb = FWD ? tk / nch : nsb - 1 - tk / nch;
    const int64_t d0 = (int64_t)2 * NB * sb;
    const int r0 = ch * RC;
    const int rc = (int)(nrhs - r0 < RC ? nrhs - r0 : RC);
    const int h = wv >> 2, w4 = wv & 3;     // half and wave of the half
    const int64_t hb = d0 + NB * h;         // first row of this half's diagonal block
    const int wd = (int)(n - hb < 0 ? 0 : n - hb < NB ? n - hb : NB);
    const bool second = FWD ? h == 1 : h == 0;  // this half's block comes second in the chain
    const int last = (int)((n + NB - 1) / NB) - 1;  // last block with rows
    const int nj = FWD ? 2 * sb : (last >= 2 * sb + 2 ? last - 2 * sb - 1 : 0);
    const T* xin = out + (int64_t)r0 * np;  // solved values of the other blocks

    // This wave's 16 columns (rows) of the block of rows rb and columns cb.
    // Rows past the end repeat the last row forward (their sums are not stored)
    // and are zero backward, as their solved values are.
    T lv[2][16];
    auto load = [&](int64_t rb, int64_t cb, T (&v)[16]) {
        if (FWD && !TURN) {
            const int64_t i = rb + lane < n ? rb + lane : n - 1;
            const T* p = L + pidx(i, cb + 16 * w4);
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = p[u];
        } else if (FWD) {
            // four rows of 16 columns at a time: row 4 u + lane / 16
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int64_t r = rb + 4 * u + (lane >> 4), i = r < n ? r : n - 1;
                v[u] = L[pidx(i, cb + 16 * w4 + (lane & 15))];
            }
        } else {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int64_t i = rb + 16 * w4 + u;
                v[u] = i < n ? L[pidx(i, cb + lane)] : T(0);
            }
        }
    };
    // The loaded block turned so that lane = row, v[u] = column u
    // (through this wave's own LDS, while the solved values are on their way).
    auto turn = [&](T (&v)[16]) {
        if constexpr (TURN) {
            T* w = &tr[wv][0];
#pragma unroll
            for (int u = 0; u < 16; ++u) w[(4 * u + (lane >> 4)) * TS + (lane & 15)] = v[u];
            wave_lds_fence();
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = w[lane * TS + u];
            wave_lds_fence();
        }
    };
    auto load_q = [&](int q, T (&v)[16]) {
        if (FWD)
            load(hb, (int64_t)NB * q, v);
        else
            load((int64_t)NB * (last - q), hb, v);
    };
    if (nj > 0) load_q(0, lv[0]);
    if (nj > 1) load_q(1, lv[1]);

    // diagonal blocks, and this wave's right-hand sides
    if (t < 2 * NB) rcp[t] = d0 + t < n ? T(1) / L[pidx(d0 + t, d0 + t)] : T(1);
    T x = T(0);
    if (w4 < rc && lane < wd) x = FWD ? B[(hb + lane) * ldb + r0 + w4] : in[(int64_t)(r0 + w4) * np + hb + lane];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int row = 4 * u + w4;
        const T v = (row < wd && lane < row) ? L[pidx(hb + row, hb + lane)] : T(0);
        ld[h][row * LS + lane] = v * rcp[NB * h + (FWD ? lane : row)];
    }

    T acc[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r) acc[r] = T(0);
    // the block v times the solved values y (lane = row of the solved block)
    auto apply = [&](const T (&y)[RC], const T (&v)[16]) {
        if ((lane >> 4) == w4)
#pragma unroll
            for (int r = 0; r < RC; ++r) yw[wv][r][lane & 15] = y[r];
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            T s[4] = {T(0), T(0), T(0), T(0)};  // four chains
#pragma unroll
            for (int u = 0; u < 16; ++u) s[u & 3] += v[u] * yw[wv][r][u];
            acc[r] += (s[0] + s[1]) + (s[2] + s[3]);
        }
        wave_lds_fence();
    };
    auto use = [&](int q, T (&v)[16]) {
        T y[RC];
        turn(v);
        await<T, RC>(xin + (int64_t)NB * (FWD ? q : last - q) + lane, np, y, q + 4 >= nj);
        apply(y, v);
    };
#pragma clang loop unroll(disable)
    for (int q = 0; q < nj; q += 2) {
        use(q, lv[0]);
        if (q + 2 < nj) load_q(q + 2, lv[0]);
        if (q + 1 < nj) {
            use(q + 1, lv[1]);
            if (q + 3 < nj) load_q(q + 3, lv[1]);
        }
    }
    // The block between the two diagonal blocks, for the half that needs it
    // (where there is a second block).
    if (second && d0 + NB < n) {
        load(d0 + NB, d0, lv[0]);
        turn(lv[0]);
    }

    // this half's sums into LDS
    auto reduce = [&]() {
#pragma unroll
        for (int r = 0; r < RC; ++r) red[h][(w4 * RC + r) * NB + lane] = acc[r];
    };
    // solve this half's diagonal block, publish it (and keep it in ys)
    auto solve = [&]() {
        if (w4 >= RC) return;
        x -= (red[h][w4 * NB + lane] + red[h][(RC + w4) * NB + lane]) +
             (red[h][(2 * RC + w4) * NB + lane] + red[h][(3 * RC + w4) * NB + lane]);
        const T v = solve_block<T, FWD>(ld[h], L, hb, wd, rcp + NB * h, lane, x);
        publish(out + (int64_t)(r0 + w4) * np + hb + lane, v);
        if (!second) ys[w4][lane] = v;
        if (!FWD && w4 < rc && lane < wd) B[(hb + lane) * ldb + r0 + w4] = v;
    };
    static_assert(RC <= 4, "a wave solves at most one right-hand side");
    if (!second) reduce();
    __syncthreads();
    if (!second) solve();
    __syncthreads();
    if (second) {
        if (d0 + NB < n) {
            T y[RC];
#pragma unroll
            for (int r = 0; r < RC; ++r) y[r] = ys[r][lane];
            apply(y, lv[0]);
        }
        reduce();
    }
    __syncthreads();
    if (second) solve();
}

// Both substitutions for n <= NB: one diagonal block, a wave per right-hand
// side (lane = row), no values to pass between workgroups.  Same arithmetic as
// k_trsv.  Bound by its launch: FP32 n = 24, two right-hand sides 23 us a call
// with the general launches and their workspace, now 14 (18 as two launches of
// one wave).
template <typename T>
__global__ __launch_bounds__(512) void k_trsv_one(const T* __restrict__ L, int n, T* __restrict__ B, int64_t nrhs,
                                                  int64_t ldb) {
    constexpr int LS = NB + 1;
    __shared__ T lf[NB * LS], lb[NB * LS];
    __shared__ T rcp[NB];
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t r = (int64_t)blockIdx.x * 8 + wv;
    if (t < NB) rcp[t] = t < n ? T(1) / L[pidx(t, t)] : T(1);
    T x = T(0);
    if (r < nrhs && lane < n) x = B[lane * ldb + r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NB / 8; ++u) {
        const int row = 8 * u + wv;
        const T v = (row < n && lane < row) ? L[pidx(row, lane)] : T(0);
        lf[row * LS + lane] = v * rcp[lane];
        lb[row * LS + lane] = v * rcp[row];
    }
    __syncthreads();
    if (r >= nrhs) return;
    x = solve_block<T, true>(lf, L, 0, n, rcp, lane, x);
    x = solve_block<T, false>(lb, L, 0, n, rcp, lane, x);
    if (lane < n) B[lane * ldb + r] = x;
}

constexpr int64_t kPass = 128;  // right-hand sides solved together (bounds the workspace)

template <typename T, int RC>
hipError_t potrs_t(const T* L, int64_t n, T* B, int64_t nrhs, int64_t ldb, void* ws, hipStream_t s) {
    const int nsb = (int)((n + 2 * NB - 1) / (2 * NB)), nch = (int)((nrhs + RC - 1) / RC);
    const int64_t np = (int64_t)2 * NB * nsb, count = np * nch * RC;
    int* counter = (int*)ws;
    T* y = (T*)((char*)ws + 256);
    T* x = y + count;
    hipLaunchKernelGGL(k_trsv_init<T>, dim3((unsigned)((2 * count + 255) / 256)), dim3(256), 0, s, y, 2 * count,
                       counter);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_trsv<T, RC, true>), dim3((unsigned)(nsb * nch)), dim3(512), 0, s, L, n, B, nrhs, ldb, nsb,
                       nch, (const T*)nullptr, y, np, counter);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_trsv<T, RC, false>), dim3((unsigned)(nsb * nch)), dim3(512), 0, s, L, n, B, nrhs, ldb, nsb,
                       nch, (const T*)y, x, np, counter + 1);
    return hipGetLastError();
}

// Right-hand sides a workgroup takes.  Each group is a chain of its own that
// streams L, so wide groups pay at large n (FP64, n = 10000, 33 right-hand
// sides: four 1.48 ms, two 1.98 ms) though their chain is longer (n = 1000:
// 96 against 83 us).
int rhs_group(int64_t nrhs) { return nrhs == 1 ? 1 : nrhs == 2 ? 2 : 4; }

template <typename T>
hipError_t potrs_passes(const T* L, int64_t n, T* B, int64_t nrhs, int64_t ldb, void* ws, hipStream_t s) {
    ProfScope ps(ATA_KERNEL_SOLVE, s);
    if (n <= NB) {
        // right-hand sides in slices: 64 threads each, less than 2^32 threads a launch
        constexpr int64_t kSlice = (int64_t)1 << 25;
        for (int64_t r = 0; r < nrhs; r += kSlice) {
            const int64_t k = nrhs - r < kSlice ? nrhs - r : kSlice;
            hipLaunchKernelGGL(k_trsv_one<T>, dim3((unsigned)((k + 7) / 8)), dim3(512), 0, s, L, (int)n, B + r, k, ldb);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    for (int64_t r = 0; r < nrhs; r += kPass) {
        const int64_t k = nrhs - r < kPass ? nrhs - r : kPass;
        const int rc = rhs_group(k);
        const hipError_t e = rc == 1   ? potrs_t<T, 1>(L, n, B + r, k, ldb, ws, s)
                             : rc == 2 ? potrs_t<T, 2>(L, n, B + r, k, ldb, ws, s)
                                       : potrs_t<T, 4>(L, n, B + r, k, ldb, ws, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

size_t potrs_ws_bytes(bool f32, int64_t n, int64_t nrhs) {
    if (n <= NB) return 0;
    const int64_t k = nrhs < kPass ? nrhs : kPass, rc = rhs_group(k), np = (n + 2 * NB - 1) / (2 * NB) * (2 * NB);
    return 256 + (size_t)(2 * np * ((k + rc - 1) / rc * rc)) * (f32 ? 4 : 8);
}

hipError_t launch_potrs(bool f32, const void* L, int64_t n, void* B, int64_t nrhs, int64_t ldb, void* ws,
                        hipStream_t s) {
    return f32 ? potrs_passes((const float*)L, n, (float*)B, nrhs, ldb, ws, s)
               : potrs_passes((const double*)L, n, (double*)B, nrhs, ldb, ws, s);
}

}  // namespace atalib
