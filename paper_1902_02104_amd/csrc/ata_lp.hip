// Reduced-precision classical tiles of gfx950 on 16-byte direct-to-LDS
// copies: the products of the transposed converted copies (bfloat16 hi and lo
// planes, or e4m3) whose segment windows lie on 16 bytes of the copy.
//
// What bounds them: the matrix cores, the LDS reads that feed them (64 x 64
// bfloat16-pair waves read 128 KB per 256 x 128 x 32 stage, 1000 cycles of LDS
// under 1536 of MFMA; e4m3 waves of 128 x 64 read 96 KB per 256 x 256 x 64
// stage, as many cycles as its MFMAs take) and, at sizes that keep every CU
// busy, the power budget: the bfloat16-pair tiles of 8192 x 8192 run at
// 1.2 PFLOP/s with the clock down at 1.7 GHz.  So:
//  - eight waves a workgroup, two per SIMD, whose accumulators (64 FP32 and 128
//    registers of FP64 sums for bfloat16, 128 FP32 for e4m3) stay in
//    architectural registers.  One wave per SIMD with twice the registers had
//    the compiler move every accumulator to and from the accumulation
//    registers in each stage, and nothing to run while it read LDS.
//  - workgroup tiles of 256 rows: a quarter (bfloat16) and half (e4m3) less
//    staged data per product than 128 x 128 tiles.
//  - stages of 64-byte rows in a ring of three or four LDS buffers.  A wave
//    waits for its own copies of the stage it needs by count, two or three
//    stages after issuing them, and one barrier per stage publishes them.
//  - row records bound each copy (16 rows, those that exist), so the loop has
//    no row checks, and past the last stage the copies still run, out of
//    range, to keep the count.
// Chunk c (16 bytes) of row r sits at chunk position c ^ (-(r / 4) mod 4):
// the sixteen lanes that a 16-byte LDS read serves at a time are 0-3, 12-15
// and 20-27 (or the rest of a half wave), and this puts them in sixteen
// different 16-byte groups of the 256-byte bank row, for the 16-row operands
// of bfloat16 and the 32-row ones of e4m3 (SQ_LDS_BANK_CONFLICT is 0).
//
// Measured, C in float, per call with the conversions (before: 128 x 128
// tiles of four waves): bfloat16 pairs 8192 x 8192 1955 -> 1615 us, 3001 x
// 4000 217 -> 175 us, 262144 x 300 374 -> 342 us; e4m3 8192 x 8192 503 -> 384
// us, 3001 x 4000 122 -> 84 us, 262144 x 300 502 -> 235 us (the last two and
// half of the first by the conversion passes).
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
typedef float f16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef int i8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u4_t __attribute__((ext_vector_type(4)));
constexpr uint32_t kOOB = 0x80000000u;  // an offset past every record count used here
constexpr int KFLUSH = 512;             // FP32 rows between adds into FP64

// Geometry of a workgroup tile: WM x WN waves of RB x CB result blocks of BS.
// The 128 x 128 tiles, for launches with too few wide ones: eight waves for
// bfloat16 (four waves of 64 x 64, two workgroups per CU: 4096 x 1024 61 us
// against 55), four for e4m3.
template <int MODE_, int WM_, int WN_, int RB_, int CB_, int RING_>
struct Geo {
    static constexpr int MODE = MODE_, WM = WM_, WN = WN_, RB = RB_, CB = CB_, RING = RING_;
    static constexpr int BS = MODE == 0 ? 16 : 32;  // MFMA 16x16x32 bf16, 32x32x64 e4m3
    static constexpr int EB = MODE == 0 ? 2 : 1, PL = MODE == 0 ? 2 : 1;
    static constexpr int KT = 64 / EB;  // k of a stage: 64-byte tile rows
    static constexpr int TM = WM * RB * BS, TN = WN * CB * BS;
    static constexpr int NW = WM * WN, NT = 64 * NW;
    static constexpr int BLKS = (TM + TN) / 16;  // 1 KB copies (16 rows) per plane and stage
    static constexpr int NB = BLKS / NW;         // ... of one wave
    static constexpr int PLANE = BLKS * 1024, STAGE = PL * PLANE;
    static_assert(BLKS % NW == 0 && KFLUSH % KT == 0, "");
};

typedef Geo<0, 4, 2, 4, 4, 3> GeoB0;  // bf16: 256 x 128, eight waves of 64 x 64
typedef Geo<0, 2, 4, 4, 2, 3> GeoT0;  // bf16: 128 x 128, eight waves of 64 x 32
typedef Geo<1, 2, 4, 4, 2, 4> GeoB1;  // e4m3: 256 x 256, eight waves of 128 x 64
typedef Geo<1, 2, 2, 2, 2, 4> GeoT1;  // e4m3: 128 x 128, four waves of 64 x 64
static_assert(GeoB0::TM == kWideRows && GeoB0::TN == 128 && GeoB1::TM == kWideRows && GeoB1::TN == 256, "");

// Chunk position of logical 16-byte chunk c in row r of a block of 64-byte
// rows.
__device__ __forceinline__ int chunk_at(int r, int c) { return c ^ ((0 - (r >> 2)) & 3); }

// Items [0, nmain) are whole tiles; with SPLIT the items after them (`tail`)
// are parts (slot mod nparts) of K-split tiles, whose results go to slot of
// `part`.
template <typename G, typename OUT, bool SPLIT>
__global__ void __launch_bounds__(G::NT, 2) k_lp_tile(const uint8_t* __restrict__ T0, const uint8_t* __restrict__ T1,
                                                      int ldt, const float* __restrict__ scale,
                                                      const DevTask* __restrict__ tasks,
                                                      const DevTerm* __restrict__ terms,
                                                      const int32_t* __restrict__ segs,
                                                      const WorkItem* __restrict__ items, int nmain,
                                                      const WorkItem* __restrict__ tail, OUT* __restrict__ C,
                                                      double* __restrict__ W, int nparts, void* __restrict__ part) {
    constexpr int MODE = G::MODE, RB = G::RB, CB = G::CB, BS = G::BS, KT = G::KT, PL = G::PL, NB = G::NB;
    constexpr int TM = G::TM, TN = G::TN, RING = G::RING;
    __shared__ __attribute__((aligned(16))) uint8_t lds[RING][G::STAGE];

    const int bid = blockIdx.x;
    const bool split = SPLIT && bid >= nmain;
    const WorkItem w = split ? tail[bid - nmain] : items[bid];
    const DevTask t = tasks[w.task];
    const DevTerm tx = terms[t.term_off];
    const DevTerm ty = terms[t.term_off + 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / G::WN, wn = wave % G::WN;
    const int i0 = w.ti * TM, j0 = w.tj * TN;
    const int stride = kSegHdr + 2 * (t.nx + t.ny);
    const bool syrk = t.kind == TK_SYRK;
    // waves of a diagonal tile whose part lies above the diagonal only copy
    // (the other wave on their SIMD gets the MFMA unit)
    const bool idle = syrk && j0 + wn * CB * BS > i0 + wm * RB * BS + RB * BS - 1;

    // Copies of this wave: row blocks wave NB + i of the TM / 16 left and
    // TN / 16 right ones; lane L fetches row L / 4, chunk position L % 4.
    const int64_t rowb = (int64_t)ldt * G::EB;
    const int kl = chunk_at(lane >> 2, lane & 3) * (16 / G::EB);  // first k of the lane's chunk
    const uint32_t vo = (uint32_t)((lane >> 2) * rowb) + (uint32_t)(kl * G::EB);
    rsrc_t rs[NB][PL];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int blk = wave * NB + i;
        const bool x = blk < TM / 16;
        const int row = x ? tx.col + i0 + 16 * blk : ty.col + j0 + 16 * (blk - TM / 16);
        const int nv = (x ? tx.cvend : ty.cvend) - row;  // rows of the block that exist
        const int rec = __builtin_amdgcn_readfirstlane((nv < 0 ? 0 : nv < 16 ? nv : 16) * (int)rowb);
#pragma unroll
        for (int p = 0; p < PL; ++p)
            rs[i][p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>((p == 0 ? T0 : T1) + row * rowb),
                                                         (short)0, rec, 0x00020000);
    }

    int ntiles = 0;
    for (int s = 0; s < t.nseg; ++s)
        ntiles += (segs[t.seg_off + s * stride + 2] - segs[t.seg_off + s * stride + 1] + KT - 1) / KT;
    int seg = 0;
    int k0 = t.nseg > 0 ? segs[t.seg_off + 1] : 0;
    int kend = t.nseg > 0 ? segs[t.seg_off + 2] : 0;  // window end
    int krow = t.nseg > 0 ? segs[t.seg_off + kSegHdr] : 0;
    auto advance = [&]() {
        k0 += KT;
        if (k0 >= kend) {
            ++seg;
            if (seg < t.nseg) {
                k0 = segs[t.seg_off + seg * stride + 1];
                kend = segs[t.seg_off + seg * stride + 2];
                krow = segs[t.seg_off + seg * stride + kSegHdr];
            }
        }
    };
    if (split) {  // its share of the stages
        const int tp = w.slot % nparts;
        const int s0 = (int)((int64_t)ntiles * tp / nparts), s1 = (int)((int64_t)ntiles * (tp + 1) / nparts);
        for (int u = 0; u < s0; ++u) advance();
        ntiles = s1 - s0;
    }

    // Copies of the stage at k0 into buffer `buf`; past the last stage every
    // lane is out of range (zeros into a spare buffer), so that the number of
    // copies in flight at a wait does not depend on the stage.
    int left = ntiles;
    auto copy_stage = [&](int buf) {
        const int krem = left > 0 ? kend - k0 : 0;
        const uint32_t off = kl < krem ? vo : kOOB;
        const int so = (krow + k0) * G::EB;
        uint8_t* dst = &lds[buf][wave * NB * 1024];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int p = 0; p < PL; ++p)
                lds_copy16(rs[i][p], dst + p * G::PLANE + i * 1024, off, so);
        if (--left > 0) advance();
    };

    typedef std::conditional_t<MODE == 0, f4_t, f16_t> acc_t;
    constexpr int NE = MODE == 0 ? 4 : 16;
    acc_t acc[RB][CB];
    double acc64[MODE == 0 ? RB : 1][MODE == 0 ? CB : 1][MODE == 0 ? NE : 1];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) {
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[a][b][e] = 0.0f;
            if constexpr (MODE == 0)
#pragma unroll
                for (int e = 0; e < NE; ++e) acc64[a][b][e] = 0.0;
        }

    // byte offset of the lane's first chunk in a block of BS rows
    const int lr = lane & (BS - 1), lk = lane / BS;
    const int c0 = MODE == 0 ? chunk_at(lr, lk) : chunk_at(lr, 2 * lk);
    const int abase = wm * RB * BS * 64 + lr * 64, bbase = TM * 64 + wn * CB * BS * 64 + lr * 64;

    // MFMA operands of a 32-row block of e4m3 stage `st`: chunks 2 lk and
    // 2 lk + 1 of the lane's row, at positions c0 and c0 ^ 1
    auto frag = [&](const uint8_t* st, int base) {
        const u4_t lo = *(const u4_t*)(st + base + c0 * 16);
        const u4_t hi = *(const u4_t*)(st + base + (c0 ^ 1) * 16);
        return i8_t{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    };

    // e4m3 operands run one row block ahead of the MFMAs, also over the end of
    // a stage, so a stage has to be in LDS one iteration before it is
    // multiplied.
    constexpr int AHEAD = MODE == 1 ? 1 : 0;
#pragma unroll
    for (int s = 0; s < RING - 1; ++s) copy_stage(s);
    i8_t bq[MODE == 1 ? CB : 1], aq{};
    if constexpr (MODE == 1) {
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((RING - 2) * NB * PL) : "memory");
        if (!idle) {
#pragma unroll
            for (int b = 0; b < CB; ++b) bq[b] = frag(lds[0], bbase + b * BS * 64);
            aq = frag(lds[0], abase);
        }
    }
    int buf = 0, done = 0;
    for (int it = 0; it < ntiles; ++it) {
        // this wave's copies of stage `it` + AHEAD have landed and its reads of
        // stage it - 1 have returned; past the barrier that holds for every wave
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((RING - 2 - AHEAD) * NB * PL) : "memory");
        copy_stage(buf == 0 ? RING - 1 : buf - 1);
        const uint8_t* st = lds[buf];
        buf = buf + 1 == RING ? 0 : buf + 1;
        if (!idle) {
            if constexpr (MODE == 0) {
                const uint8_t* ap = st + abase + c0 * 16;
                const uint8_t* bp = st + bbase + c0 * 16;
                bf8_t bh[CB], bl[CB];
#pragma unroll
                for (int b = 0; b < CB; ++b) {
                    bh[b] = *(const bf8_t*)(bp + b * BS * 64);
                    bl[b] = *(const bf8_t*)(bp + G::PLANE + b * BS * 64);
                }
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int a = 0; a < RB; ++a) {
                    const bf8_t ah = *(const bf8_t*)(ap + a * BS * 64);
                    const bf8_t al = *(const bf8_t*)(ap + (PL - 1) * G::PLANE + a * BS * 64);
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[b], acc[a][b], 0, 0, 0);
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[b], acc[a][b], 0, 0, 0);
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[b], acc[a][b], 0, 0, 0);
                }
                __builtin_amdgcn_s_setprio(0);
            } else {
                const uint8_t* sn = lds[buf];  // the next stage
                i8_t bn[CB];
#pragma unroll
                for (int a = 0; a < RB; ++a) {
                    const i8_t an = a + 1 < RB ? frag(st, abase + (a + 1) * BS * 64) : frag(sn, abase);
                    if (a + 1 == RB)
#pragma unroll
                        for (int b = 0; b < CB; ++b) bn[b] = frag(sn, bbase + b * BS * 64);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        acc[a][b] =
                            __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aq, bq[b], acc[a][b], 0, 0, 0, 0, 0, 0);
                    aq = an;
                }
#pragma unroll
                for (int b = 0; b < CB; ++b) bq[b] = bn[b];
            }
        }
        if constexpr (MODE == 0) {
            if (++done == KFLUSH / KT || it + 1 == ntiles) {
                done = 0;
#pragma unroll
                for (int a = 0; a < RB; ++a)
#pragma unroll
                    for (int b = 0; b < CB; ++b)
#pragma unroll
                        for (int e = 0; e < NE; ++e) {
                            acc64[a][b][e] += (double)acc[a][b][e];
                            acc[a][b][e] = 0.0f;
                        }
            }
        }
    }
    // no copy may land after the workgroup's LDS is released
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    // Result rows of block a, element e: 16 x 16 blocks hold rows
    // 4 (lane / 16) + e, 32 x 32 blocks rows 8 (e / 4) + 4 (lane / 32) + e % 4.
    auto row_of = [&](int a, int e) {
        return (wm * RB + a) * BS + (MODE == 0 ? 4 * lk + e : 8 * (e / 4) + 4 * lk + (e & 3));
    };
    if (SPLIT && split) {
        // a part: FP64 sums of bfloat16 (zero past the valid extent, where
        // the copies read as zero), FP32 accumulators of e4m3 as they are
        typedef std::conditional_t<MODE == 0, double, float> part_t;
        if (idle) return;
        part_t* pt = (part_t*)part + (int64_t)w.slot * TM * TN + wn * CB * BS + lr;
#pragma unroll
        for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int b = 0; b < CB; ++b) {
                    if constexpr (MODE == 0)
                        pt[row_of(a, e) * TN + b * BS] = acc64[a][b][e];
                    else
                        pt[row_of(a, e) * TN + b * BS] = acc[a][b][e];
                }
        return;
    }
    // reciprocals of the (power-of-two) scales of the tile's rows and columns
    double* rsc = (double*)&lds[0][0];
    if constexpr (MODE == 1) {
        __syncthreads();
        for (int i = threadIdx.x; i < TM + TN; i += G::NT) {
            const int gi = i < TM ? i0 + i : j0 + i - TM;
            rsc[i] = gi < (i < TM ? t.dM : t.dN) ? 1.0 / (double)scale[(i < TM ? tx.col : ty.col) + gi] : 0.0;
        }
        __syncthreads();
    }
    if (idle) return;
    const int ljw = wn * CB * BS + lr;  // this lane's column of block 0
    double sj[CB];
    if constexpr (MODE == 1)
#pragma unroll
        for (int b = 0; b < CB; ++b) sj[b] = rsc[TM + ljw + b * BS];
    auto value = [&](int a, int b, int e, double si) {
        if constexpr (MODE == 0)
            return acc64[a][b][e];
        else
            return (double)acc[a][b][e] * si * sj[b];  // exact de-scale
    };
    if (t.dst == 0 && !t.beta && i0 + TM <= t.dM && j0 + TN <= t.dN && !(syrk && j0 + TN - 1 > i0)) {
        // tiles inside the block: no bounds, no diagonal
#pragma unroll
        for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int li = row_of(a, e);
                OUT* row = C + pidx((int64_t)t.r0 + i0 + li, t.q0 + j0 + ljw);
                const double si = MODE == 1 ? rsc[li] : 1.0;
#pragma unroll
                for (int b = 0; b < CB; ++b) row[b * BS] = (OUT)value(a, b, e, si);
            }
        return;
    }
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int li = row_of(a, e), gi = i0 + li;
            if (gi >= t.dM) continue;
            OUT* row = C + pidx((int64_t)t.r0 + gi, t.q0);
            const double si = MODE == 1 ? rsc[li] : 1.0;
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int gj = j0 + ljw + b * BS;
                if (gj >= t.dN || (syrk && gj > gi)) continue;
                const double v = value(a, b, e, si);
                if (t.dst == 0)
                    store_c(row + gj, t.beta, v);
                else
                    W[t.ws_off + (int64_t)gi * t.N + gj] = v;
            }
        }
}

// Sum of the K parts of the split tiles (FP64, in part order), stored as
// k_lp_tile stores: block (li, q) covers row li of tail tile q, one thread
// per column.  e4m3 parts are raw FP32 accumulators, de-scaled here.
template <typename G, typename OUT>
__global__ void __launch_bounds__(G::TN) k_lp_part_sum(const float* __restrict__ scale,
                                                       const DevTask* __restrict__ tasks,
                                                       const DevTerm* __restrict__ terms,
                                                       const WorkItem* __restrict__ tail, int nparts,
                                                       const void* __restrict__ part, OUT* __restrict__ C,
                                                       double* __restrict__ W) {
    typedef std::conditional_t<G::MODE == 0, double, float> part_t;
    const int q = blockIdx.y, li = blockIdx.x, lj = threadIdx.x;
    const WorkItem w = tail[q * nparts];
    const DevTask t = tasks[w.task];
    const int gi = w.ti * G::TM + li, gj = w.tj * G::TN + lj;
    if (gi >= t.dM || gj >= t.dN || (t.kind == TK_SYRK && gj > gi)) return;
    const part_t* pt = (const part_t*)part;
    double v = 0.0;
    for (int p = 0; p < nparts; ++p) v += (double)pt[((int64_t)(q * nparts + p) * G::TM + li) * G::TN + lj];
    if (G::MODE == 1) {
        const DevTerm tx = terms[t.term_off];
        const DevTerm ty = terms[t.term_off + 1];
        v = v * (1.0 / (double)scale[tx.col + gi]) / (double)scale[ty.col + gj];  // exact power-of-two de-scale
    }
    if (t.dst == 0)
        store_c(C + pidx((int64_t)t.r0 + gi, t.q0) + gj, t.beta, v);
    else
        W[t.ws_off + (int64_t)gi * t.N + gj] = v;
}

template <typename G, typename OUT>
hipError_t run(const LpCopy& cp, const DevTables& tb, const WorkItem* items, int nmain, const WorkItem* tail, int ntail,
               int nparts, void* part, void* C, double* W, hipStream_t s) {
    const uint8_t* t0 = (const uint8_t*)cp.t0;
    const uint8_t* t1 = (const uint8_t*)(cp.t1 ? cp.t1 : cp.t0);
    const dim3 b(G::NT);
    if (nmain <= 0 && ntail <= 0) return hipSuccess;
    if (ntail <= 0) {
        hipLaunchKernelGGL((k_lp_tile<G, OUT, false>), dim3(nmain), b, 0, s, t0, t1, cp.ldt, cp.scale, tb.tasks,
                           tb.terms, tb.segs, items, nmain, tail, (OUT*)C, W, 1, nullptr);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_lp_tile<G, OUT, true>), dim3(nmain + ntail), b, 0, s, t0, t1, cp.ldt, cp.scale, tb.tasks,
                       tb.terms, tb.segs, items, nmain, tail, (OUT*)C, W, nparts, part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_lp_part_sum<G, OUT>), dim3(G::TM, ntail / nparts), dim3(G::TN), 0, s, cp.scale, tb.tasks,
                       tb.terms, tail, nparts, (const void*)part, (OUT*)C, W);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lp_tile16(int mode, bool out_f64, bool wide, const LpCopy& cp, const DevTables& tb,
                            const WorkItem* items, int nmain, const WorkItem* tail, int ntail, int nparts, void* part,
                            void* C, double* W, hipStream_t s) {
    if (wide) {
        if (mode == 0)
            return out_f64 ? run<GeoB0, double>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s)
                           : run<GeoB0, float>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s);
        return out_f64 ? run<GeoB1, double>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s)
                       : run<GeoB1, float>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s);
    }
    if (mode == 0)
        return out_f64 ? run<GeoT0, double>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s)
                       : run<GeoT0, float>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s);
    return out_f64 ? run<GeoT1, double>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s)
                   : run<GeoT1, float>(cp, tb, items, nmain, tail, ntail, nparts, part, C, W, s);
}

}  // namespace atalib
