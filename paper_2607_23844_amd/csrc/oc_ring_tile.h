// Ring-buffered LDS-DMA MFMA tile engine for gfx950, one to three blocks per
// compute unit: C[b][a] = sum_k A[a][k] * B[b][k] over a BA x BB tile, WA x WB waves,
// 32x32 accumulators of v_mfma_f32_32x32x16_{bf16,f16}, K in steps of 64.
//
// What bounds a projection here: a step moves (BA + BB) x 128 bytes from L2 to
// LDS for BA x BB x 64 products.  Small tiles (128 x 128, two blocks per unit)
// need 64 bytes per clock and unit from L2 at the full matrix rate, all it can
// give; and a step whose loads are issued one MFMA phase before they are read
// waits for them.  So tiles are as large as the shape allows, the operands
// travel through a ring of NST LDS stages, and inside a step everything is
// interleaved by hand (scheduling fences): the fragments of the next 16 k are
// read while the current ones feed the MFMAs; the barrier that publishes the
// next stage stands before the step's last 16 k, whose MFMAs cover the first
// reads of that stage and the DMA that refills the stage just freed, a whole
// ring ahead.  Standalone, 256 tiles of 256 x 192: 1241 TFLOP/s at K = 1536
// (the MFMAs alone, without loads, 1652: the clock drops under load), 128 x
// 128 with four stages 857.
//
// An LDS row is the 128 bytes of one operand row's step; its 16-byte chunk c
// sits in slot c ^ ((row >> 1) & 7): two rows fill the 64 banks, so the
// fragment reads of 16 consecutive rows hit distinct banks.  DMA instruction i
// of wave w covers the 8 rows 8 (w + i NW) .. + 7 of its operand, 8 lanes
// each, as raw buffer loads: a uniform base per instruction, a 32-bit offset
// per lane, the step in a scalar.  K need only be a multiple of 8: in the
// last step the lanes past K get an offset past the end of the buffer, which
// reads as zero.
#pragma once
#include "oc_mfma_tile.h"
#include "oc_launch.h"
#include <type_traits>

namespace oc {

constexpr uint32_t RING_RECORDS = 0xFFFFFFF0u;   // bytes behind a base; this offset and up read as zero

// Rows of one operand as the DMA instructions of a wave read them.  In the one
// instruction of a tile that spans two bases (mix), the lanes in alt read
// behind base2.
template <int N, int NW>
struct RingRows {
    const uint16_t *base[N], *base2;
    uint32_t off[N];         // bytes from the base: row and swizzled chunk
    unsigned mix, alt;       // bit i: instruction i (mix uniform, alt per lane)
    // row of the tile that this lane reads in instruction i, and the first row of the instruction
    __device__ __forceinline__ static int row(int i) { return (threadIdx.x + 64 * NW * i) >> 3; }
    __device__ __forceinline__ static int row8(int i) {
        return 8 * (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) + NW * i);
    }
    // this lane's 16-byte chunk of a step (the same in every instruction: NW is a multiple of 4)
    __device__ __forceinline__ static int chunk() { return (threadIdx.x & 7) ^ ((threadIdx.x >> 4) & 7); }
};

template <int BA_, int BB_, int WA, int WB, int NST, bool F16 = false>
struct RingTile {
    static constexpr int BA = BA_, BB = BB_, BK = 64, NW = WA * WB, NT = NW * 64;
    static constexpr int WTA = BA / WA, WTB = BB / WB, TA = WTA / 32, TB = WTB / 32;
    static constexpr int CA = BA / (8 * NW), CB = BB / (8 * NW), IPT = CA + CB;   // DMA instructions per wave and step
    static constexpr int STAGE = (BA + BB) * BK;                                  // halves per stage
    static constexpr size_t RING_BYTES = (size_t)NST * STAGE * 2;
    // the epilogue's staged rows (and a table of one int2 per row) reuse the ring
    static constexpr size_t EPI_BYTES = (size_t)BB * (BA + 8) * 2 + (size_t)BA * 8;
    static constexpr size_t LDS_BYTES = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
    static_assert(NW % 4 == 0 && WTA % 32 == 0 && WTB % 32 == 0, "wave tiles of whole accumulators");
    static_assert(CA * 8 * NW == BA && CB * 8 * NW == BB, "whole DMA instructions");
    static_assert((NST - 1) * IPT < 64 && LDS_BYTES <= 160 * 1024, "counters and LDS");
    typedef typename std::conditional<F16, f16x8, bf16x8>::type frag;
    typedef RingRows<CA, NW> RowsA;
    typedef RingRows<CB, NW> RowsB;

    f32x16 acc[TA][TB];

    __device__ __forceinline__ static f32x16 mma(frag a, frag b, f32x16 c) {
        if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    template <typename R>
    __device__ __forceinline__ static void dma(const R &r, int i, uint16_t *dst, int koff, uint32_t oob) {
        const int off = (int)(r.off[i] | oob);
        if (__builtin_expect((r.mix >> i) & 1u, 0)) {
            if ((r.alt >> i) & 1u) buffer_load_lds(buffer_rsrc(r.base2, (int)RING_RECORDS), (lds_vp)dst, 16, off, koff, 0, 0);
            else buffer_load_lds(buffer_rsrc(r.base[i], (int)RING_RECORDS), (lds_vp)dst, 16, off, koff, 0, 0);
        } else {
            buffer_load_lds(buffer_rsrc(r.base[i], (int)RING_RECORDS), (lds_vp)dst, 16, off, koff, 0, 0);
        }
    }

    // rows without data (past the operand) may repeat any valid row: their
    // accumulators are garbage and must be discarded
    __device__ __forceinline__ void run(uint16_t *lds, const RowsA &ra, const RowsB &rb, int K) {
        const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
        const int wa = wave / WB, wb = wave % WB, lr = lane & 31, lh = lane >> 5;
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j) acc[i][j] = f32x16{};
        const int nk = (K + BK - 1) / BK;
        // in the last step this lane's chunk may lie past K
        const uint32_t tail = (nk - 1) * BK + RowsA::chunk() * 8 < K ? 0u : RING_RECORDS;
        auto issue = [&](int d, uint16_t *st, int kt, uint32_t oob) {
            if (d < CA) dma(ra, d, st + (wave + NW * d) * 512, kt * BK * 2, oob);
            else dma(rb, d - CA, st + BA * BK + (wave + NW * (d - CA)) * 512, kt * BK * 2, oob);
        };
        // fragment offsets (halves) of this lane inside a stage, per 16-wide k step
        int oa[4], ob[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c = ((ks * 2 + lh) ^ ((lr >> 1) & 7)) << 3;
            oa[ks] = (wa * WTA + lr) * BK + c;
            ob[ks] = BA * BK + (wb * WTB + lr) * BK + c;
        }
        frag fa[2][TA], fb[2][TB];
        constexpr int NR = TA + TB, NM = TA * TB;
        // read r of the fragments of one k step: A row block 0, the B blocks, the other A blocks
        auto read = [&](int r, const uint16_t *st, int ks, int s) {
            if (r == 0) fa[s][0] = *reinterpret_cast<const frag *>(st + oa[ks]);
            else if (r <= TB) fb[s][r - 1] = *reinterpret_cast<const frag *>(st + ob[ks] + (r - 1) * 32 * BK);
            else if (r < NR) fa[s][r - TB] = *reinterpret_cast<const frag *>(st + oa[ks] + (r - TB) * 32 * BK);
        };
        // the MFMAs of fragments s with the reads of the next 16 k (nks of
        // stage nst) and, when go, the DMA of step kt into dst between them
        auto phase = [&](int s, const uint16_t *nst, int nks, uint16_t *dst, bool go, int kt, uint32_t oob) {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
#pragma unroll
                for (int r = m * NR / NM; r < (m + 1) * NR / NM; ++r) read(r, nst, nks, s ^ 1);
                acc[m / TB][m % TB] = mma(fa[s][m / TB], fb[s][m % TB], acc[m / TB][m % TB]);
                if (dst != nullptr && go) {
#pragma unroll
                    for (int d = m * IPT / NM; d < (m + 1) * IPT / NM; ++d) issue(d, dst, kt, oob);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
#pragma unroll
        for (int q = 0; q < NST; ++q)
            if (q < nk) {
#pragma unroll
                for (int d = 0; d < IPT; ++d) issue(d, lds + q * STAGE, q, q + 1 < nk ? 0u : tail);
            }
        if (nk >= NST) {
            OC_WAIT_VMCNT((NST - 1) * IPT);
        } else {
            OC_WAIT_VMCNT(0);
        }
        barrier_lds();
#pragma unroll
        for (int r = 0; r < NR; ++r) read(r, lds, 0, 0);
        uint16_t *st = lds;
        for (int kt = 0; kt < nk; ++kt) {
            uint16_t *const ot = st + STAGE == lds + NST * STAGE ? lds : st + STAGE;
            phase(0, st, 1, nullptr, false, 0, 0);
            phase(1, st, 2, nullptr, false, 0, 0);
            phase(0, st, 3, nullptr, false, 0, 0);
            // this wave's loads of step kt+1 have landed (steps up to kt+NST-1 are in flight)
            if (kt + NST - 1 < nk) {
                OC_WAIT_VMCNT((NST - 2) * IPT);
            } else {
                OC_WAIT_VMCNT(0);
            }
            barrier_lds();   // ... and every wave's, and every wave has read stage kt
            // (after the last step the fragments read here are not used)
            phase(1, ot, 0, st, kt + NST < nk, kt + NST, kt + NST + 1 < nk ? 0u : tail);
            st = ot;
        }
        __syncthreads();   // the epilogue may reuse the ring
    }

    // Several tiles along A against the same B rows, back to back in one
    // pipeline (the ring is not drained between tiles): load_a(rows, u) fills
    // the rows of tile u, and after tile u's last step epi(u) consumes acc.
    // Neither may touch the ring or leave global loads in flight (the waits
    // below count the ring's loads only).  seg_len > 0 (a multiple of 64 that
    // divides K): a row is K / seg_len segments, sub_stride elements apart.
    template <typename LoadA, typename Epi>
    __device__ __forceinline__ void run_tiles(uint16_t *lds, LoadA load_a, RowsB rb, int K, int seg_len,
                                              long sub_stride, int n_tiles, Epi epi) {
        const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
        const int wa = wave / WB, wb = wave % WB, lr = lane & 31, lh = lane >> 5;
        const int seg_k = seg_len > 0 ? seg_len : K, n_seg = K / seg_k;
        const int sps = (seg_k + BK - 1) / BK, nk = sps * n_seg, ns = nk * n_tiles;   // steps per segment, tile and call
        const uint32_t tail = (sps - 1) * BK + RowsA::chunk() * 8 < seg_k ? 0u : RING_RECORDS;
        RowsA ra;
        load_a(ra, 0);
        int iu = 0, isg = 0, ik = 0;   // tile, segment and its step of the next loads
        auto issue = [&](int d, uint16_t *st, uint32_t oob) {
            if (d < CA) dma(ra, d, st + (wave + NW * d) * 512, ik * BK * 2, oob);
            else dma(rb, d - CA, st + BA * BK + (wave + NW * (d - CA)) * 512, ik * BK * 2, oob);
        };
        auto advance = [&]() {
            if (++ik < sps) return;
            ik = 0;
            long by = sub_stride;
            if (++isg == n_seg) {
                isg = 0;
                by = -(long)(n_seg - 1) * sub_stride;
                if (++iu < n_tiles) load_a(ra, iu);
            } else {
#pragma unroll
                for (int i = 0; i < CA; ++i) ra.base[i] += by;
            }
#pragma unroll
            for (int i = 0; i < CB; ++i) rb.base[i] += by;
        };
        int oa[4], ob[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c = ((ks * 2 + lh) ^ ((lr >> 1) & 7)) << 3;
            oa[ks] = (wa * WTA + lr) * BK + c;
            ob[ks] = BA * BK + (wb * WTB + lr) * BK + c;
        }
        frag fa[2][TA], fb[2][TB];
        constexpr int NR = TA + TB, NM = TA * TB;
        auto read = [&](int r, const uint16_t *st, int ks, int s) {
            if (r == 0) fa[s][0] = *reinterpret_cast<const frag *>(st + oa[ks]);
            else if (r <= TB) fb[s][r - 1] = *reinterpret_cast<const frag *>(st + ob[ks] + (r - 1) * 32 * BK);
            else if (r < NR) fa[s][r - TB] = *reinterpret_cast<const frag *>(st + oa[ks] + (r - TB) * 32 * BK);
        };
        // as in run(); fresh: the tile's first products (the accumulators start at zero)
        auto phase = [&](auto fresh, int s, const uint16_t *nst, int nks, uint16_t *dst, bool go, uint32_t oob) {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
#pragma unroll
                for (int r = m * NR / NM; r < (m + 1) * NR / NM; ++r) read(r, nst, nks, s ^ 1);
                f32x16 &c = acc[m / TB][m % TB];
                c = mma(fa[s][m / TB], fb[s][m % TB], decltype(fresh)::value ? f32x16{} : c);
                if (dst != nullptr && go) {
#pragma unroll
                    for (int d = m * IPT / NM; d < (m + 1) * IPT / NM; ++d) issue(d, dst, oob);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
#pragma unroll
        for (int q = 0; q < NST; ++q)
            if (q < ns) {
#pragma unroll
                for (int d = 0; d < IPT; ++d) issue(d, lds + q * STAGE, ik + 1 < sps ? 0u : tail);
                advance();
            }
        if (ns >= NST) {
            OC_WAIT_VMCNT((NST - 1) * IPT);
        } else {
            OC_WAIT_VMCNT(0);
        }
        barrier_lds();
#pragma unroll
        for (int r = 0; r < NR; ++r) read(r, lds, 0, 0);
        uint16_t *st = lds;
        int kt = 0, u = 0;
        for (int s = 0; s < ns; ++s) {
            uint16_t *const ot = st + STAGE == lds + NST * STAGE ? lds : st + STAGE;
            if (kt == 0) phase(std::true_type{}, 0, st, 1, nullptr, false, 0);
            else phase(std::false_type{}, 0, st, 1, nullptr, false, 0);
            phase(std::false_type{}, 1, st, 2, nullptr, false, 0);
            phase(std::false_type{}, 0, st, 3, nullptr, false, 0);
            if (s + NST - 1 < ns) {
                OC_WAIT_VMCNT((NST - 2) * IPT);
            } else {
                OC_WAIT_VMCNT(0);
            }
            barrier_lds();
            phase(std::false_type{}, 1, ot, 0, st, s + NST < ns, ik + 1 < sps ? 0u : tail);
            if (s + NST < ns) advance();
            st = ot;
            if (++kt == nk) {
                epi(u);
                kt = 0;
                ++u;
            }
        }
        __syncthreads();   // the caller may reuse the ring
    }

    __device__ __forceinline__ static int a_of(int i, int g) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        return (wave / WB) * WTA + i * 32 + 8 * g + 4 * (lane >> 5);
    }
    __device__ __forceinline__ static int b_of(int j) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        return (wave % WB) * WTB + j * 32 + (lane & 31);
    }
};

// Rows r0 + row of a contiguous [n, K] matrix (rows past n repeat the last)
template <int N, int NW>
__device__ __forceinline__ void ring_rows(RingRows<N, NW> &w, const uint16_t *m, int n, int K, int r0) {
    w.base2 = m;
    w.mix = w.alt = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        w.base[i] = m + (long)r0 * K;
        w.off[i] = (uint32_t)min(w.row(i), n - 1 - r0) * (uint32_t)(K * 2) + (uint32_t)w.chunk() * 16;
    }
}

// Rows a0 + row of up to three stacked [hd, K] matrices, n rows in all (hd
// and n multiples of 8: the 8 rows of an instruction lie in one of them)
template <int N, int NW>
__device__ __forceinline__ void ring_rows3(RingRows<N, NW> &w, const uint16_t *m0, const uint16_t *m1,
                                           const uint16_t *m2, int hd, int n, int K, int a0) {
    w.base2 = m0;
    w.mix = w.alt = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int a8 = min(a0 + w.row8(i), n - 8), which = a8 / hd;
        w.base[i] = (which == 0 ? m0 : which == 1 ? m1 : m2) + (long)(a8 - which * hd) * K;
        w.off[i] = ((threadIdx.x & 63) >> 3) * (uint32_t)(K * 2) + (uint32_t)w.chunk() * 16;
    }
}

// Tile shapes of the GEMM-shaped kernels, and what a launch of each costs:
// `units` tiles run on each compute unit, `resident` of them at a time, a
// batch of k resident tiles taking fixed + nk * step[k - 1] us for nk steps of
// 64 (prologue, epilogue and the pipeline's fill in `fixed`).  The figures are
// a least-squares fit to the Q/K/V and output projections of 45 layers (256 to
// 230400 rows, C = 64 to 1536) measured with every shape; the shape picked
// from them was within 2.5% of the fastest one on the average, 18% at worst.
// Large tiles move the fewest bytes per product and win where they fill the
// chip in whole rounds; a small tile's shorter prologue and epilogue, and two
// or three of them on a unit, win on small layers and short K.
struct RingShapeCost { int BA, BB, resident; float fixed, step[3]; };
constexpr RingShapeCost RING_SHAPES[] = {
    {256, 256, 1, 5.56f, {1.198f}},        {256, 192, 1, 4.72f, {0.926f}},
    {256, 128, 1, 3.32f, {0.727f}},        {128, 192, 1, 4.33f, {0.609f}},
    {96, 128, 1, 1.42f, {0.487f}},         {128, 128, 2, 1.48f, {0.602f, 0.973f}},
    {128, 192, 2, 2.68f, {0.709f, 1.323f}}, {160, 128, 2, 2.32f, {0.665f, 1.232f}},
    {64, 64, 3, 1.75f, {0.213f, 0.276f, 0.503f}}, {128, 64, 2, 2.26f, {0.277f, 0.537f}},
};
constexpr int N_RING_SHAPES = sizeof(RING_SHAPES) / sizeof(RING_SHAPES[0]);
template <int ID, bool F16> struct RingShape;
template <bool F16> struct RingShape<0, F16> { using Tile = RingTile<256, 256, 4, 2, 2, F16>; };
template <bool F16> struct RingShape<1, F16> { using Tile = RingTile<256, 192, 4, 2, 2, F16>; };
template <bool F16> struct RingShape<2, F16> { using Tile = RingTile<256, 128, 4, 2, 3, F16>; };
template <bool F16> struct RingShape<3, F16> { using Tile = RingTile<128, 192, 2, 2, 3, F16>; };
template <bool F16> struct RingShape<4, F16> { using Tile = RingTile<96, 128, 1, 4, 5, F16>; };
template <bool F16> struct RingShape<5, F16> { using Tile = RingTile<128, 128, 2, 2, 2, F16>; };
template <bool F16> struct RingShape<6, F16> { using Tile = RingTile<128, 192, 2, 2, 2, F16>; };
template <bool F16> struct RingShape<7, F16> { using Tile = RingTile<160, 128, 1, 4, 2, F16>; };
template <bool F16> struct RingShape<8, F16> { using Tile = RingTile<64, 64, 2, 2, 3, F16>; };
template <bool F16> struct RingShape<9, F16> { using Tile = RingTile<128, 64, 2, 2, 3, F16>; };
template <int ID> constexpr int RING_THREADS = RingShape<ID, false>::Tile::NT;
template <int ID> constexpr size_t RING_LDS = RingShape<ID, false>::Tile::RING_BYTES;

// us for `blocks` blocks of nk steps each, with `epi` us of other work per block
inline float ring_cost(const RingShapeCost &c, int nk, long blocks, float epi = 0.f) {
    const long units = (blocks + 255) / 256, full = units / c.resident;
    const int rest = (int)(units % c.resident);
    float t = (float)full * (c.fixed + nk * c.step[c.resident - 1] + epi * c.resident);
    if (rest > 0) t += c.fixed + nk * c.step[rest - 1] + epi * rest;
    return t;
}

// The shape with the lowest cost for K elements; tiles(BA, BB): tiles of the
// launch.  Not more threads than a grid holds (the narrow shapes, on half a
// billion rows of few columns); room for the blocks that convert weights.
template <typename Tiles>
inline int ring_pick(int K, Tiles tiles) {
    constexpr int threads[N_RING_SHAPES] = {RING_THREADS<0>, RING_THREADS<1>, RING_THREADS<2>, RING_THREADS<3>,
                                            RING_THREADS<4>, RING_THREADS<5>, RING_THREADS<6>, RING_THREADS<7>,
                                            RING_THREADS<8>, RING_THREADS<9>};
    const int nk = (K + 63) / 64;
    int best = 0;
    float best_t = 0.f;
    for (int i = 0; i < N_RING_SHAPES; ++i) {
        const long n = tiles(RING_SHAPES[i].BA, RING_SHAPES[i].BB);
        if (i > 0 && (n + 1024) * threads[i] >= MAX_GRID_THREADS) continue;
        const float t = ring_cost(RING_SHAPES[i], nk, n);
        if (i == 0 || t < best_t) {
            best = i;
            best_t = t;
        }
    }
    return best;
}

// f(std::integral_constant<int, id>) for a shape known at run time
template <typename F>
inline auto ring_dispatch(int id, F f) {
    switch (id) {
        case 0: return f(std::integral_constant<int, 0>{});
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        default: return f(std::integral_constant<int, 9>{});
    }
}

}  // namespace oc
