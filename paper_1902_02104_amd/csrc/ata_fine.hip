// Fine-tile classical product of gfx950: lower(A^t A) in 64 x 64 or 32 x 32
// tiles with the K range split over the waves of a workgroup and over
// workgroups, for products with too few 128 x 128 tiles to fill the chip.
//
// What bounds these products is parallelism: n = 509 has ten 128 x 128
// tiles.  Splitting K over workgroups alone pays for every part with a
// partial tile in memory, so a workgroup here splits K over its four waves
// first: each wave owns the whole tile for every fourth stage of the
// workgroup's rows, copies its own stages into its own LDS (no workgroup
// barrier in the loop) and the four results are summed in LDS in wave order.
// Only then are rows split over workgroups (parts), whose FP64 partial tiles
// k_fine_sum adds in part order.  A whole-tile wave also reads each staged
// operand once per 64 (32) columns of the other side, half the LDS reads of
// four waves sharing a tile.
//
// Layout of a stage: 4 KB per operand, KS = 4096 / (TB sizeof(T)) rows of
// the tile's TB columns, moved by four 16-byte-per-lane buffer loads that
// write LDS.  FP64 chunks (16 bytes) of row r sit at chunk position
// c ^ ((r & 3) << 2), so the four k rows an MFMA step reads fall in different
// 64-byte bank groups; FP32 rows are read whole (16 lanes cover a row).
// MFMA forms and operand slots are those of the 128 x 128 tile kernels: FP64
// 4x4x4 with slot (block 2q + h, row i) holding column 8q + 2i + h on the
// left and slot (block 2u + h, column j) column 32u + 2j + h on the right;
// FP32 16x16x4 with slot (block h, j) holding column NB j + h on both sides
// (NB blocks of 16 per tile side).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ata.h"
#include "ata_device.h"
#include "ata_internal.h"
#include "ata_kernels.h"

namespace atalib {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef double d2_t __attribute__((ext_vector_type(2)));
constexpr uint32_t kOOB = 0x80000000u;  // an offset past every record count used here
constexpr int KFLUSH = 512;             // FP32 rows between adds into FP64

// Row a and column c of linear index b in a lower triangle of tiles.
__device__ __forceinline__ void tri_decode(int b, int& a, int& c) {
    a = (int)((sqrtf(8.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
    while (a * (a + 1) / 2 > b) --a;
    while ((a + 1) * (a + 2) / 2 <= b) ++a;
    c = b - a * (a + 1) / 2;
}

// Workgroup b of tiles x parts: with parts a multiple of eight the tiles of
// one part (which read the same rows of A) run on one XCD (workgroups go
// round-robin over the eight XCDs).
__device__ __forceinline__ void decode_block(int b, int tiles, int parts, int& tile, int& part) {
    if ((parts & 7) == 0) {
        const int j = b >> 3;
        part = (b & 7) + 8 * (j / tiles);
        tile = j % tiles;
    } else {
        part = b / tiles;
        tile = b % tiles;
    }
}

template <typename T, int TB>
struct Acc;

// FP64: TB / 4 row blocks x TB / 16 column blocks, one element per lane each.
template <int TB>
struct Acc<double, TB> {
    static constexpr int NQ = TB / 8, NU = TB / 32;
    double a[2 * NQ][2 * NU];
    __device__ void zero() {
#pragma unroll
        for (int i = 0; i < 2 * NQ; ++i)
#pragma unroll
            for (int j = 0; j < 2 * NU; ++j) a[i][j] = 0.0;
    }
    // One MFMA step (four k rows) on row kr.. of the planes.
    __device__ void step(const double* xp, const double* yp, int ks, int lane) {
        const int g = lane >> 4, sw = g << 2;
        const double* xr = xp + (ks * 4 + g) * TB;
        const double* yr = yp + (ks * 4 + g) * TB;
        d2_t bv[NU], av[NQ];
#pragma unroll
        for (int u = 0; u < NU; ++u) bv[u] = *(const d2_t*)&yr[2 * ((16 * u + (lane & 15)) ^ sw)];
#pragma unroll
        for (int q = 0; q < NQ; ++q) av[q] = *(const d2_t*)&xr[2 * ((4 * q + (lane & 3)) ^ sw)];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < 2 * NU; ++c)
                    a[2 * q + h][c] =
                        __builtin_amdgcn_mfma_f64_4x4x4f64(av[q][h], bv[c >> 1][c & 1], a[2 * q + h][c], 0, 0, 0);
    }
    __device__ void flush() {}
    // Add (ADD) or store the accumulators to a TB x TB FP64 tile.
    template <bool ADD>
    __device__ void to_lds(double* d, int lane) {
        const int g = lane >> 4;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    d2_t* p = (d2_t*)&d[(8 * q + 2 * g + h) * TB + 32 * u + 2 * (lane & 15)];
                    d2_t v{a[2 * q + h][2 * u], a[2 * q + h][2 * u + 1]};
                    if (ADD) v += *p;
                    *p = v;
                }
    }
};

// FP32: NB x NB blocks of 16 x 16, flushed into FP64 every KFLUSH rows.
template <int TB>
struct Acc<float, TB> {
    static constexpr int NB = TB / 16;
    f4_t a[NB][NB];
    double w[NB][NB][4];
    __device__ void zero() {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                a[i][j] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e) w[i][j][e] = 0.0;
            }
    }
    __device__ void step(const float* xp, const float* yp, int ks, int lane) {
        typedef typename std::conditional<NB == 4, f4_t, f2_t>::type v_t;
        const int o = (ks * 4 + (lane >> 4)) * TB + NB * (lane & 15);
        const v_t x = *(const v_t*)&xp[o], y = *(const v_t*)&yp[o];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) a[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[j], a[i][j], 0, 0, 0);
    }
    __device__ void flush() {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[i][j][e] += (double)a[i][j][e];
                a[i][j] = f4_t{0.f, 0.f, 0.f, 0.f};
            }
    }
    // block (i, j), lane, element e: row NB (4 (lane >> 4) + e) + i, column NB (lane & 15) + j
    template <bool ADD>
    __device__ void to_lds(double* d, int lane) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < NB; j += 2) {
                    d2_t* p = (d2_t*)&d[(NB * (4 * (lane >> 4) + e) + i) * TB + NB * (lane & 15) + j];
                    d2_t v{w[i][j][e], w[i][j + 1][e]};
                    if (ADD) v += *p;
                    *p = v;
                }
    }
};

// The same on operands whose staged rows are tile rows with k along them
// (A A^t): rows of RBY = 4096 / TB bytes, chunk c of row r at chunk position
// c ^ row_swz(r), which puts the sixteen lanes an LDS read serves together (0-3,
// 12-15 and 20-27, or the others of a half wave) in different 16-byte groups
// of the bank row.  A 16-byte read holds VK consecutive k of one row, one for
// each of VK MFMA steps.  Against a transpose and the column form: FP32 1000 x
// 20011 224 -> 193 us, FP64 700 x 60000 680 -> 540.
template <int TB>
__device__ __forceinline__ int row_swz(int r) {
    return TB == 64 ? (0 - (r >> 2)) & 3 : (r >> 1) & 7;
}

// Clear k kv.. of a stage (the last of a part, where what follows the row in
// memory was staged).
template <typename T, int TB>
__device__ __forceinline__ void clear_tail(T* p, int kv, int lane) {
    constexpr int RBY = 4096 / TB, KS = RBY / (int)sizeof(T), VK = 16 / (int)sizeof(T);
    const int row = lane % TB;
    for (int k = kv; k < KS; ++k) p[row * KS + VK * ((k / VK) ^ row_swz<TB>(row)) + k % VK] = T(0);
}

template <typename T, int TB>
struct AccRows;

template <int TB>
struct AccRows<double, TB> {
    static constexpr int RBY = 4096 / TB, KS = RBY / 8, NR = TB / 4, NC = TB / 16;
    double a[NR][NC];
    __device__ void zero() {
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) a[i][j] = 0.0;
    }
    __device__ void stage(const double* xp, const double* yp, int lane) {
        const int g = lane >> 4;
#pragma unroll
        for (int half = 0; half < RBY / 64; ++half) {
            const int ch = 4 * half + g;
            auto rd = [&](const double* p, int row) {
                return *(const d2_t*)((const char*)p + row * RBY + 16 * (ch ^ row_swz<TB>(row)));
            };
            d2_t b[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) b[c] = rd(yp, 16 * c + (lane & 15));
#pragma unroll
            for (int r0 = 0; r0 < NR; r0 += 4) {
                d2_t x[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] = rd(xp, 4 * (r0 + r) + (lane & 3));
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            a[r0 + r][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(x[r][e], b[c][e], a[r0 + r][c], 0, 0, 0);
            }
        }
    }
    __device__ void flush() {}
    template <bool ADD>
    __device__ void to_lds(double* d, int lane) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double* p = &d[(4 * r + (lane >> 4)) * TB + 16 * c + (lane & 15)];
                *p = ADD ? *p + a[r][c] : a[r][c];
            }
    }
};

template <int TB>
struct AccRows<float, TB> : Acc<float, TB> {
    typedef Acc<float, TB> B;
    static constexpr int RBY = 4096 / TB, KS = RBY / 4, NB = B::NB;
    __device__ void stage(const float* xp, const float* yp, int lane) {
        const int g = lane >> 4;
#pragma unroll
        for (int half = 0; half < RBY / 64; ++half) {
            const int ch = 4 * half + g;
            auto rd = [&](const float* p, int row) {
                return *(const f4_t*)((const char*)p + row * RBY + 16 * (ch ^ row_swz<TB>(row)));
            };
            f4_t y[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) y[i] = rd(yp, 16 * i + (lane & 15));
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const f4_t x = rd(xp, 16 * i + (lane & 15));
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        this->a[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[j][e], this->a[i][j], 0, 0, 0);
            }
        }
    }
    template <bool ADD>
    __device__ void to_lds(double* d, int lane) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    double* p = &d[(16 * i + 4 * (lane >> 4) + e) * TB + 16 * j + (lane & 15)];
                    *p = ADD ? *p + this->w[i][j][e] : this->w[i][j][e];
                }
    }
};

// One workgroup: tile `tile` of rows [part * rows, min(K, (part + 1) * rows)).
// ROWS: A holds the operand columns as rows of K elements (A A^t).  LONG: the
// sums of rows may pass 2^31.  (An instance of its own: the few scalar
// instructions that differ move the loop in the instruction cache, and that
// alone took FP32 A A^t of 1400 x 21319 from 352 to 399 us and FP64 1341 x 2280
// from 137 to 162.)
template <typename T, typename OUT, int TB, bool ROWS, bool LONG>
__global__ void __launch_bounds__(256, 2) k_fine(const T* __restrict__ A, int64_t lda, int K, int n, int tiles,
                                                int parts, int rows, OUT* __restrict__ C, int beta,
                                                double* __restrict__ part_out) {
    constexpr int PLANE = 4096 / (int)sizeof(T);  // elements of one operand's stage
    constexpr int KS = PLANE / TB;                // rows of a stage
    constexpr int RB = TB * (int)sizeof(T);       // bytes of a staged row
    constexpr int RPC = 1024 / RB;                // rows per copy instruction
    constexpr int CH = RB / 16;                   // 16-byte chunks per row
    __shared__ __attribute__((aligned(16))) T lds[4][2][2][PLANE];  // [wave][buffer][operand]

    int tile, part, ti, tj;
    decode_block(blockIdx.x, tiles, parts, tile, part);
    tri_decode(tile, ti, tj);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool diag = ti == tj;
    const int ra = part * rows;
    int rb, nst;
    if constexpr (LONG) {
        rb = part_end(K, ra, rows);
        nst = part_stages(rb - ra, KS);
    } else {
        rb = ra + rows < K ? ra + rows : K;
        nst = rb > ra ? (rb - ra + KS - 1) / KS : 0;
    }
    const int64_t row_bytes = lda * (int64_t)sizeof(T);

    // This lane's chunk of a copy: row lane / CH of the copy's RPC rows,
    // chunk position lane % CH; it holds the chunk the swizzle puts there.
    // Row residues repeat every four rows, so RPC = 2 needs two offsets.
    const int lr = lane / CH, lp = lane % CH;
    constexpr int NOFF = (sizeof(T) == 8 && RPC == 2) ? 2 : 1;
    uint32_t xo[NOFF], yo[NOFF];
#pragma unroll
    for (int q = 0; q < NOFF; ++q) {
        const int r = RPC * q + lr;
        const int c = sizeof(T) == 8 ? lp ^ ((r & 3) << 2) : lp;
        const int el = c * (16 / (int)sizeof(T));  // first column of the chunk
        xo[q] = ti * TB + el < n ? (uint32_t)((ti * TB + el) * (int)sizeof(T)) : kOOB;
        yo[q] = tj * TB + el < n ? (uint32_t)((tj * TB + el) * (int)sizeof(T)) : kOOB;
    }
    // Copies of the stage at row r0: rows below rb; the records end with the
    // last valid column of the last valid row, the rest reads as zero.
    // ROWS: lane / CHR is the row of a copy's RPR, lane % CHR the position.
    constexpr int CHR = 4096 / TB / 16, RPR = 64 / CHR;
    auto copy_rows = [&](int st, int buf) {
        const int64_t k0 = ra + st * KS;
        const int lrr = lane / CHR;
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (side && diag) break;
            const int t0 = (side ? tj : ti) * TB;
            const int nv = n - t0 < TB ? n - t0 : TB;
            const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(A + (int64_t)t0 * lda + k0), (short)0,
                                                                (int)((nv - 1) * row_bytes + (K - k0) * (int64_t)sizeof(T)),
                                                                0x00020000);
            T* d = lds[wave][buf][side];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = i * RPR + lrr;
                lds_copy16(rs, d + i * (1024 / (int)sizeof(T)),
                           (uint32_t)(row * row_bytes) + 16u * (uint32_t)((lane % CHR) ^ row_swz<TB>(row)));
            }
        }
    };
    auto copy = [&](int st, int buf) {
        if constexpr (ROWS) {
            copy_rows(st, buf);
            return;
        }
        const int r0 = ra + st * KS;
        const int nv = rb - r0 < KS ? rb - r0 : KS;
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(A + (int64_t)r0 * lda), (short)0,
                                                            (int)((nv - 1) * row_bytes + n * (int64_t)sizeof(T)),
                                                            0x00020000);
        T* x = lds[wave][buf][0];
        T* y = lds[wave][buf][1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t ro = (uint32_t)((i * RPC + lr) * row_bytes);
            lds_copy16(rs, x + i * (1024 / (int)sizeof(T)), ro + xo[i % NOFF]);
        }
        if (!diag) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t ro = (uint32_t)((i * RPC + lr) * row_bytes);
                lds_copy16(rs, y + i * (1024 / (int)sizeof(T)), ro + yo[i % NOFF]);
            }
        }
    };

    typename std::conditional<ROWS, AccRows<T, TB>, Acc<T, TB>>::type acc;
    acc.zero();
    if (wave < nst) copy(wave, 0);
    int done = 0;  // stages of this wave since the last flush
    for (int st = wave, it = 0; st < nst; st += 4, ++it) {
        const int buf = it & 1;
        // this wave's copies of stage st have landed; its reads of stage
        // st - 4 have returned, so their buffer can be filled again
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        if (st + 4 < nst) copy(st + 4, buf ^ 1);
        const T* xp = lds[wave][buf][0];
        const T* yp = diag ? xp : lds[wave][buf][1];
        if constexpr (ROWS) {
            const int kv = rb - (ra + st * KS);
            if (kv < KS) {
                clear_tail<T, TB>(lds[wave][buf][0], kv, lane);
                if (!diag) clear_tail<T, TB>(lds[wave][buf][1], kv, lane);
            }
            acc.stage(xp, yp, lane);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS / 4; ++ks) acc.step(xp, yp, ks, lane);
        }
        if (++done == KFLUSH / KS) {
            acc.flush();
            done = 0;
        }
    }
    acc.flush();

    // Sum of the four waves: (w0 + w1) + (w2 + w3), two tiles of LDS.
    __syncthreads();
    double* red = (double*)&lds[0][0][0][0];
    static_assert(sizeof(lds) >= 2 * TB * TB * sizeof(double), "two FP64 tiles");
    double* mine = red + (wave >> 1) * TB * TB;
    if (wave & 1) acc.template to_lds<false>(mine, lane);
    __syncthreads();
    if (!(wave & 1)) acc.template to_lds<true>(mine, lane);
    __syncthreads();
    if (part_out) {
        d2_t* po = (d2_t*)(part_out + ((int64_t)tile * parts + part) * TB * TB);
#pragma unroll
        for (int u = 0; u < TB * TB / 512; ++u) {
            const int e = u * 256 + threadIdx.x;
            po[e] = ((const d2_t*)red)[e] + ((const d2_t*)(red + TB * TB))[e];
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < TB * TB / 256; ++u) {
        const int e = u * 256 + threadIdx.x;
        const int gi = ti * TB + e / TB, gj = tj * TB + e % TB;
        if (gi < n && gj <= gi) store_c(C + pidx(gi, gj), beta, red[e] + red[TB * TB + e]);
    }
}

// Sum of the parts in a fixed order (group g of G adds parts g, g + G, ...,
// then the groups in order): 64 consecutive elements of one tile per
// workgroup, one element per lane, G waves.
template <typename OUT, int TB, int G>
__global__ void __launch_bounds__(64 * G) k_fine_sum(const double* __restrict__ part, int parts, int n,
                                                    OUT* __restrict__ C, int beta) {
    __shared__ double red[G][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    int ti, tj;
    tri_decode(blockIdx.x, ti, tj);
    const int e = blockIdx.y * 64 + lane;
    const double* p = part + (int64_t)blockIdx.x * parts * (TB * TB) + e;
    double s = 0.0;
#pragma unroll 8
    for (int k = g; k < parts; k += G) s += p[(int64_t)k * (TB * TB)];
    if (G > 1) {
        red[g][lane] = s;
        __syncthreads();
        if (g) return;
#pragma unroll
        for (int k = 1; k < G; ++k) s += red[k][lane];
    }
    const int gi = ti * TB + e / TB, gj = tj * TB + e % TB;
    if (gi < n && gj <= gi) store_c(C + pidx(gi, gj), beta, s);
}

template <typename T, typename OUT, int TB, bool ROWS>
hipError_t fine_t(const T* A, int64_t lda, int K, int n, int parts, int rows, OUT* C, int beta, double* part,
                  hipStream_t s) {
    const int t = (n + TB - 1) / TB, tiles = t * (t + 1) / 2;
    double* const po = parts > 1 ? part : nullptr;
    const dim3 grid(tiles * parts), block(256);
    // rows of A^t fit 32 bits (their bytes do)
    if (!ROWS && long_rows(parts, rows))
        hipLaunchKernelGGL((k_fine<T, OUT, TB, false, true>), grid, block, 0, s, A, lda, K, n, tiles, parts, rows, C, beta,
                           po);
    else
        hipLaunchKernelGGL((k_fine<T, OUT, TB, ROWS, false>), grid, block, 0, s, A, lda, K, n, tiles, parts, rows, C,
                           beta, po);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || parts <= 1) return e;
    const dim3 g(tiles, TB * TB / 64);
    if (parts <= 8)
        hipLaunchKernelGGL((k_fine_sum<OUT, TB, 1>), g, dim3(64), 0, s, part, parts, n, C, beta);
    else if (parts <= 32)
        hipLaunchKernelGGL((k_fine_sum<OUT, TB, 4>), g, dim3(256), 0, s, part, parts, n, C, beta);
    else
        hipLaunchKernelGGL((k_fine_sum<OUT, TB, 16>), g, dim3(1024), 0, s, part, parts, n, C, beta);
    return hipGetLastError();
}

template <bool ROWS>
hipError_t fine_any(bool f32, bool out_f64, int tb, const void* A, int64_t lda, int K, int n, int parts, int rows,
                    void* C, int beta, double* part, hipStream_t s) {
    const double* Ad = (const double*)A;
    const float* Af = (const float*)A;
    double* Cd = (double*)C;
    float* Cf = (float*)C;
    if (!f32)
        return tb == 64 ? fine_t<double, double, 64, ROWS>(Ad, lda, K, n, parts, rows, Cd, beta, part, s)
                        : fine_t<double, double, 32, ROWS>(Ad, lda, K, n, parts, rows, Cd, beta, part, s);
    if (out_f64)
        return tb == 64 ? fine_t<float, double, 64, ROWS>(Af, lda, K, n, parts, rows, Cd, beta, part, s)
                        : fine_t<float, double, 32, ROWS>(Af, lda, K, n, parts, rows, Cd, beta, part, s);
    return tb == 64 ? fine_t<float, float, 64, ROWS>(Af, lda, K, n, parts, rows, Cf, beta, part, s)
                    : fine_t<float, float, 32, ROWS>(Af, lda, K, n, parts, rows, Cf, beta, part, s);
}

}  // namespace

hipError_t launch_fine(bool f32, bool out_f64, int tb, const void* A, int64_t lda, int K, int n, int parts, int rows,
                       void* C, int beta, double* part, hipStream_t s, bool by_rows) {
    if (K <= 0 || n <= 0 || parts < 1 || (parts > 1 && !part)) return hipErrorInvalidValue;
    return by_rows ? fine_any<true>(f32, out_f64, tb, A, lda, K, n, parts, rows, C, beta, part, s)
                   : fine_any<false>(f32, out_f64, tb, A, lda, K, n, parts, rows, C, beta, part, s);
}

}  // namespace atalib
