// LDS-DMA MFMA tile engine for gfx950: the same block tile as MfmaTile
// (C[b][a] = sum_k A[a][k] * B[b][k], 256 threads = 4 wave64s arranged
// WA x WB, 32x32 accumulators of v_mfma_f32_32x32x16_bf16), but the
// operands travel global -> LDS with global_load_lds (16 bytes per lane, no
// staging registers).
//
// K is walked in steps of 64 through two LDS stages (small enough for two or
// more blocks per CU): step kt+1 is loaded while step kt's MFMAs run.  An LDS
// row is the 128 bytes of one operand row's step, unpadded; its 16-byte chunk
// c sits in slot c ^ ((row >> 1) & 7): two rows fill the 64 LDS banks, so the
// fragment reads of 16 consecutive rows hit distinct banks.  DMA instruction i
// of a wave fills the 64 slots (wave + 4i)*64 .. +63 of the
// operand's stage, that is rows chunk_row(i) of MfmaTile: callers pass the
// same per-thread row bases.  Rows without data (nullptr) read the fallback
// row instead; their accumulators are garbage and must be discarded.
// Requirements: K % 64 == 0, 16-byte aligned row bases.
#pragma once
#include "oc_mfma_tile.h"

namespace oc {

template <int BA, int BB, int WA, int WB>
struct DmaTile {
    static constexpr int BK = 64;
    static constexpr int WTA = BA / WA, WTB = BB / WB;
    static constexpr int TA = WTA / 32, TB = WTB / 32;
    static constexpr int CA = BA / 32, CB = BB / 32;   // DMA instructions per wave and step
    static constexpr int STAGE = (BA + BB) * BK;       // halves per stage
    static constexpr size_t LDS_BYTES = (size_t)2 * STAGE * 2;
    static_assert(WA * WB == 4, "4 waves");
    static_assert(TA >= 1 && TB >= 1 && WTA % 32 == 0 && WTB % 32 == 0, "wave tile must be a multiple of 32");
    static_assert(BA % 32 == 0 && BB % 32 == 0, "tile rows per DMA instruction");
    typedef bf16x8 frag;

    f32x16 acc[TA][TB];

    __device__ __forceinline__ static int slot(int r, int c) { return r * BK + ((c ^ ((r >> 1) & 7)) << 3); }

    // MFMA fragments of one step: [ks][i] for A, [ks][j] for B
    struct Frags {
        frag a[4][TA], b[4][TB];
    };

    __device__ __forceinline__ static void read_frags(const uint16_t *st, Frags &f) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int wa = wave / WB, wb = wave % WB;
        const int lr = lane & 31, lh = lane >> 5;
        const uint16_t *As = st, *Bs = st + BA * BK;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c = ks * 2 + lh;
#pragma unroll
            for (int i = 0; i < TA; ++i) f.a[ks][i] = *reinterpret_cast<const frag *>(As + slot(wa * WTA + i * 32 + lr, c));
#pragma unroll
            for (int j = 0; j < TB; ++j) f.b[ks][j] = *reinterpret_cast<const frag *>(Bs + slot(wb * WTB + j * 32 + lr, c));
        }
    }

    __device__ __forceinline__ void mfmas(const Frags &f) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ks][i], f.b[ks][j], acc[i][j], 0, 0, 0);
    }

    // Full K loop.  rowsA[i] / rowsB[i]: this thread's row bases for
    // chunk_row(i) (nullptr: use the fallback row).
    __device__ __forceinline__ void run(uint16_t *lds, const uint16_t *const *rowsA, const uint16_t *const *rowsB,
                                        const uint16_t *fallbackA, const uint16_t *fallbackB, int K) {
        const int t = threadIdx.x, wave = t >> 6;
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j) acc[i][j] = f32x16{};
        // this lane's source chunk of each instruction: slot t&7 of its row
        const uint16_t *pa[CA], *pb[CB];
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int r = chunk_row(i);
            pa[i] = (rowsA[i] ? rowsA[i] : fallbackA) + (((t & 7) ^ ((r >> 1) & 7)) << 3);
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int r = chunk_row(i);
            pb[i] = (rowsB[i] ? rowsB[i] : fallbackB) + (((t & 7) ^ ((r >> 1) & 7)) << 3);
        }
        const int nk = K / BK;
        auto issue = [&](int kt) {
            const int off = kt * BK;
            uint16_t *st = lds + (kt & 1) * STAGE;
#pragma unroll
            for (int i = 0; i < CA; ++i)
                __builtin_amdgcn_global_load_lds((glb_vp)(pa[i] + off), (lds_vp)(st + (wave + 4 * i) * 512), 16, 0, 0);
#pragma unroll
            for (int i = 0; i < CB; ++i)
                __builtin_amdgcn_global_load_lds((glb_vp)(pb[i] + off), (lds_vp)(st + BA * BK + (wave + 4 * i) * 512),
                                                 16, 0, 0);
        };
        // the MFMAs of step kt overlap the DMA of step kt+1; the fragments of
        // kt+1 are read after the barrier that publishes it (two blocks per CU
        // hide that latency)
        issue(0);
        OC_WAIT_VMCNT(0);
        barrier_lds();
        Frags f;
        read_frags(lds, f);
        for (int kt = 0; kt < nk; ++kt) {
            if (kt + 1 < nk) issue(kt + 1);   // its stage was last read before the previous barrier
            mfmas(f);
            if (kt + 1 < nk) {
                OC_WAIT_VMCNT(0);
                barrier_lds();
                read_frags(lds + ((kt + 1) & 1) * STAGE, f);
            }
        }
        OC_WAIT_VMCNT(0);
        __syncthreads();   // the epilogue may reuse the LDS
    }

    __device__ __forceinline__ static int a_of(int i, int g) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        return (wave / WB) * WTA + i * 32 + 8 * g + 4 * (lane >> 5);
    }
    __device__ __forceinline__ static int b_of(int j) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        return (wave % WB) * WTB + j * 32 + (lane & 31);
    }
    // Row of the tile that DMA instruction i of this thread loads (as MfmaTile).
    __device__ __forceinline__ static int chunk_row(int i) { return (threadIdx.x + 256 * i) >> 3; }
};

}  // namespace oc
