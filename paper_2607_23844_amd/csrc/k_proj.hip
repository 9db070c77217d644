// Projections of the reduced attention layer on the ring-buffered MFMA tiles.
//
// x, weights and y are bf16; products of bf16 inputs are exact and
// accumulate in fp32.  The attention intermediates Q, K, V and O are stored
// in fp16 (three more mantissa bits than bf16, same MFMA rate): Q is stored
// pre-multiplied by log2(e)/sqrt(head_dim) so that the attention kernel's
// scores are already in the log2 domain.
//   k_proj_qkv: [rows, C] x [3*H*dh, C]^T -> Q, K [rows, H*dh] and
//               Vt [H][seq][dh][Lpad], keys contiguous per (head, d),
//               quads 1 and 2 of every 16-key block swapped (vt_key_of_pos)
//   k_proj_out: O [rows, H*dh] (fp16) x wo [C, H*dh] -> y rows, written
//               straight to their positions (row -> out_idx[row]) or to the
//               context output
// Rows r < n_main come from x (through row_idx when given); rows after them
// are the uncached context tokens of a single sequence.
//
// Bounded by the operands' way from L2 to LDS and by the matrix units' rate
// under load (oc_ring_tile.h); the tile shape follows from the cost of each
// (ring_pick).  Against 128 x 128 tiles, two per compute unit, whose loads
// were issued one step ahead: 2381 rows of C = 1536 47.0 -> 36.8 us (Q/K/V)
// and 20.6 -> 17.8 (output), 4429 rows 79.5 -> 73.4 and 40.9 -> 27.4, 3072
// rows of C = 1152 33.8 -> 28.9, 256 rows of C = 1536 22.2 -> 12.9.
// Epilogues go through LDS: the tile is staged as whole output rows and
// written in 16-byte chunks, so every store is a contiguous run of a row (Vt
// rows included).
//
// Tile order: blocks are remapped so that each XCD runs a contiguous range
// of logical tiles, and logical tiles are grouped GA weight tiles wide, so
// one XCD's L2 sees a few weight tiles and a few token tiles instead of all.
#include "oc_internal.h"
#include "oc_launch.h"
#include "oc_device.h"
#include "oc_attn_common.h"
#include "oc_gemm_epi.h"
#include "oc_ring_tile.h"
#include <algorithm>

namespace oc {

// Batch rows r0 + row of a projection: the index loads of all instructions go
// out together, then the offsets follow without branches (a listed row behind
// x, an unlisted one behind its tile's first row, a context row behind the
// tile's first context row).
template <int N, int NW>
__device__ __forceinline__ void ring_batch_rows(RingRows<N, NW> &w, const RowMap &rm, int r0) {
    const bool listed = rm.row_idx != nullptr || rm.tF > 0;
    const int c0 = max(r0 - rm.n_main, 0);
    const uint16_t *xb = listed || rm.x == nullptr ? rm.x : rm.x + (long)r0 * rm.C;
    w.base2 = rm.ctx + (long)c0 * rm.C;
    w.mix = w.alt = 0;
    int tok[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int r = max(min(r0 + w.row(i), rm.n_main - 1), 0);
        tok[i] = listed ? (int)batch_token(r, rm.row_idx, rm.tF, rm.tN) : r - r0;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int r = min(r0 + w.row(i), rm.n_rows - 1);
        const bool alt = r >= rm.n_main;
        const unsigned long long b = __builtin_amdgcn_ballot_w64(alt);
        w.off[i] = (uint32_t)(alt ? r - rm.n_main - c0 : tok[i]) * (uint32_t)(rm.C * 2) + (uint32_t)w.chunk() * 16;
        w.base[i] = b == ~0ull ? w.base2 : xb;
        if (b != 0 && b != ~0ull) w.mix |= 1u << i;
        if (alt) w.alt |= 1u << i;
    }
}

// bf16 -> fp16 (exact in the fp16 normal range, saturating outside), chunks i,
// i + step, ... of 8 elements, four loads in flight
__device__ __forceinline__ void to_f16(const uint4 *__restrict__ src, long n8, uint4 *__restrict__ dst, long i,
                                       long step) {
    for (; i < n8; i += 4 * step) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[min(i + u * step, n8 - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * step < n8) dst[i + u * step] = bf16x8_to_f16x8(v[u]);
    }
}

// ---------------------------------------------------------------------------
// Q, K and V in one launch.  The first n_qk tiles are row tiles: a in [0,
// nw*hd) are rows of wq, wk (and wv when nw = 3), b = batch rows, staged as
// rows of Q, K (and of V, row-major [rows, H*dh], for short sequences, whose
// attention reads V by rows).  With nw = 2 the rest are V tiles with the roles
// swapped: a = batch rows, b in [0, hd) = rows of wv, so that a staged row is
// a row of Vt[h][s][d][pos].  V tiles whose rows are a 16-aligned run of one
// sequence (a single sequence, or L a multiple of the tile) are written as Vt
// rows: the positions of the tile's tokens, zero for positions past the end
// (the key padding up to lpad), in whole chunks.  Otherwise they are stored in
// quads of tokens and the key padding is zeroed separately where the attention
// reads it (zero_pad, vt_padding_read).  The blocks past
// the tiles convert wo for the output projection where no earlier launch of
// the call has (the uncached layer and the attention entry point: a launch of
// its own took 4.5 us of 263 on the SD3-like layer, 4.4 of 220 by stages).
// ---------------------------------------------------------------------------
template <int ID>
__global__ __launch_bounds__(RING_THREADS<ID>) void k_proj_qkv(
    RowMap rm, const uint16_t *__restrict__ wq, const uint16_t *__restrict__ wk, const uint16_t *__restrict__ wv,
    int hd, int dh, float qscale, int nw, int n_qk_at, int n_bt, int n_v_at, int n_v_bt, int n_seq, int L, int lpad,
    int zero_pad, const int32_t *__restrict__ seq_off, uint16_t *__restrict__ Q, uint16_t *__restrict__ K,
    uint16_t *__restrict__ Vt, const uint4 *__restrict__ wo, long n8, uint4 *__restrict__ wo16) {
    using T = typename RingShape<ID, false>::Tile;
    constexpr int BA = T::BA, BB = T::BB, NT = T::NT;
    extern __shared__ __align__(16) uint16_t lds[];
    const int n_qk = n_qk_at * n_bt, total = n_qk + n_v_at * n_v_bt;
    if ((int)blockIdx.x >= total) {
        to_f16(wo, n8, wo16, (long)(blockIdx.x - total) * NT + threadIdx.x, (long)(gridDim.x - total) * NT);
        return;
    }
    const int lid = xcd_remap(blockIdx.x, total);
    typename T::RowsA ra;
    typename T::RowsB rb;
    T t;
    if (lid < n_qk) {
        int at, bt;
        tile_order(lid, n_qk_at, n_bt, at, bt);
        const int a0 = at * BA, b0 = bt * BB;
        ring_rows3(ra, wq, wk, wv, hd, nw * hd, rm.C, a0);
        ring_batch_rows(rb, rm, b0);
        t.run(lds, ra, rb, rm.C);
        stage_rows<BA>(t, lds, [&](float v, int a) { return f2h_bits(a0 + a < hd ? v * qscale : v); },
                       [](int a) { return a; });
        __syncthreads();
        write_rows<BA, BB, NT>(lds, min(BA, nw * hd - a0), [&](int b, int c0) -> uint16_t * {
            const int r = b0 + b, a = a0 + c0;
            if (r >= rm.n_rows) return nullptr;
            return a < hd ? Q + (long)r * hd + a
                 : a < 2 * hd ? K + (long)r * hd + (a - hd)
                              : Vt + (long)r * hd + (a - 2 * hd);
        });
        return;
    }
    // V tile: at over batch rows, bt over features
    int at, bt;
    tile_order(lid - n_qk, n_v_at, n_v_bt, at, bt);
    const int r0 = at * BA, f0 = bt * BB;
    ring_batch_rows(ra, rm, r0);
    ring_rows3(rb, wv, wv, wv, hd, hd, rm.C, f0);
    t.run(lds, ra, rb, rm.C);
    const int Lk = n_seq == 1 ? rm.n_rows : L;
    if (seq_off == nullptr && vt_whole_rows(n_seq, L, BA)) {
        const int s = n_seq == 1 ? 0 : r0 / L, j0 = r0 - s * L;   // j0 is a multiple of BA
        const int end = vt_tile_end(j0, BA, Lk, lpad);
        stage_rows<BA>(t, lds, [&](float v, int a) { return (uint16_t)(j0 + a < Lk ? f2h_bits(v) : 0); },
                       [](int a) { return vt_key_of_pos(a); });
        __syncthreads();
        const auto vt_at = [&](int b, int c0) -> uint16_t * {
            const int f = f0 + b;
            if (f >= hd) return nullptr;
            const int h = f / dh, d = f - h * dh;
            return Vt + (((long)h * n_seq + s) * dh + d) * lpad + j0 + c0;
        };
        write_rows<BA, BB, NT>(lds, min(BA, end - j0), vt_at);
        if constexpr (BA % 64 != 0) {
            // the key padding past the tile of a sequence's last one
            const int zc = max(end - j0 - BA, 0) >> 3;
            for (int c = threadIdx.x; c < BB * zc; c += NT) {
                uint16_t *const at8 = vt_at(c / zc, BA + c % zc * 8);
                if (at8 != nullptr) *reinterpret_cast<uint4 *>(at8) = make_uint4(0, 0, 0, 0);
            }
        }
        return;
    }
    // Tiles that cross sequences (or sequences whose starts are not multiples
    // of the tile): staged as rows of features too, then stored in quads of
    // tokens, lanes over consecutive tokens.  A quad inside one sequence that
    // starts at a multiple of 4 is 8 contiguous bytes of a Vt row.  (Each lane
    // storing its accumulators one by one, a stride of lpad apart, took 110 us
    // for the whole launch on 16 frames of 16 x 16 tokens of 16 heads of 72
    // that keep varying numbers of tokens; 34 us this way.)
    stage_rows<BA>(t, lds, [](float v, int) { return f2h_bits(v); }, [](int a) { return a; });
    int2 *const where = reinterpret_cast<int2 *>(lds + BB * (BA + 8));   // (sequence, position) per token
    for (int a = threadIdx.x; a < BA; a += NT) {
        int s = -1, jj = 0;
        if (r0 + a < rm.n_rows) seq_pos(r0 + a, n_seq, L, s, jj, seq_off);
        where[a] = make_int2(s, jj);
    }
    __syncthreads();
    constexpr int QPR = BA / 4;
    for (int u = threadIdx.x; u < BB * QPR; u += NT) {
        const int b = u / QPR, a = (u - b * QPR) * 4, f = f0 + b;
        if (f >= hd) break;   // (b rises with u)
        const int h = f / dh, d = f - h * dh;
        const uint16_t *src = lds + b * (BA + 8) + a;
        uint16_t *const row = Vt + ((long)h * n_seq * dh + d) * lpad;   // sequence s: s * dh * lpad further
        const int2 w0 = where[a], w3 = where[a + 3];
        if (w0.x >= 0 && w0.x == w3.x && (w0.y & 3) == 0) {
            *reinterpret_cast<u16x4 *>(row + (long)w0.x * dh * lpad + vt_key_of_pos(w0.y)) =
                *reinterpret_cast<const u16x4 *>(src);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int2 w = where[a + e];
                if (w.x >= 0) row[(long)w.x * dh * lpad + vt_key_of_pos(w.y)] = src[e];
            }
        }
    }
    // zero the padded key positions [Lk, lpad) of this block's features, for
    // the sequences s = at, at + n_v_at, ...
    const int npad = lpad - Lk;
    if (zero_pad && npad > 0) {
        for (int sq = at; sq < n_seq; sq += n_v_at)
            for (int idx = threadIdx.x; idx < BB * npad; idx += NT) {
                const int f = f0 + idx / npad, jj = Lk + idx % npad;
                if (f >= hd) continue;
                const int h = f / dh, d = f - h * dh;
                Vt[(((long)h * n_seq + sq) * dh + d) * lpad + vt_key_of_pos(jj)] = 0;
            }
    }
}

hipError_t launch_proj_qkv(const Plan &p, const RowMap &rm, const AttnArgs &a, hipStream_t st) {
    const float qscale = (float)(1.4426950408889634 / sqrt((double)p.dh));
    StageScope _stage(st, "proj_qkv");
    const int Lk = a.n_seq == 1 ? rm.n_rows : a.L;
    // short sequences: V rows from the Q/K tiles (nw = 3), no V tiles
    const int nw = a.seq_off == nullptr && attn_short(Lk) ? 3 : 2;
    const int zero_pad = vt_padding_read(p, a, Lk) ? 1 : 0;
    const auto v_at = [&](int BA) { return nw == 3 ? 0 : cdiv(rm.n_rows, BA); };
    const long n8 = a.wo16_ready ? 0 : (long)p.C * p.hd / 8;
    const int id = ring_pick(p.C, [&](int BA, int BB) {
        return (long)cdiv(nw * p.hd, BA) * cdiv(rm.n_rows, BB) + (long)v_at(BA) * cdiv(p.hd, BB);
    });
    return ring_dispatch(id, [&](auto c) -> hipError_t {
        constexpr int ID = decltype(c)::value;
        using T = typename RingShape<ID, false>::Tile;
        const hipError_t e = allow_lds(k_proj_qkv<ID>, T::LDS_BYTES);
        if (e != hipSuccess) return e;
        const int n_qk_at = cdiv(nw * p.hd, T::BA), n_bt = cdiv(rm.n_rows, T::BB);
        const int n_v_at = v_at(T::BA), n_v_bt = nw == 3 ? 0 : cdiv(p.hd, T::BB);
        const int cvt_blocks = (int)std::min<long>((n8 + 4 * T::NT - 1) / (4 * T::NT), N_CUS);
        launch_k(k_proj_qkv<ID>, n_qk_at * n_bt + n_v_at * n_v_bt + cvt_blocks, T::NT, T::LDS_BYTES, st, rm,
                 (const uint16_t *)a.wq, (const uint16_t *)a.wk, (const uint16_t *)a.wv, p.hd, p.dh, qscale, nw,
                 n_qk_at, n_bt, n_v_at, n_v_bt, a.n_seq, a.L, a.lpad, zero_pad, a.seq_off, (uint16_t *)a.q, (uint16_t *)a.k,
                 (uint16_t *)a.vt, (const uint4 *)a.wo, n8, (uint4 *)a.wo16);
        return hipGetLastError();
    });
}

// ---------------------------------------------------------------------------
// Output projection: a in [0, C) = rows of wo (fp16); b = batch rows of O.
// y[out row][a].
// ---------------------------------------------------------------------------
template <int ID>
__global__ __launch_bounds__(RING_THREADS<ID>) void k_proj_out(
    const uint16_t *__restrict__ O, int n_rows, int hd, const uint16_t *__restrict__ wo, int C, int n_main,
    const int32_t *__restrict__ out_idx, int tF, int tN, int n_at, int n_bt, uint16_t *__restrict__ y,
    uint16_t *__restrict__ y_ctx) {
    using T = typename RingShape<ID, true>::Tile;
    constexpr int BA = T::BA, BB = T::BB;
    extern __shared__ __align__(16) uint16_t lds[];
    int at, bt;
    tile_order(xcd_remap(blockIdx.x, n_at * n_bt), n_at, n_bt, at, bt);
    const int a0 = at * BA, b0 = bt * BB;
    typename T::RowsA ra;
    typename T::RowsB rb;
    ring_rows(ra, wo, C, hd, a0);
    ring_rows(rb, O, n_rows, hd, b0);
    T t;
    t.run(lds, ra, rb, hd);
    stage_rows<BA>(t, lds, [](float v, int) { return f2bf(v); }, [](int a) { return a; });
    __syncthreads();
    write_rows<BA, BB, T::NT>(lds, min(BA, C - a0), [&](int b, int c0) -> uint16_t * {
        const int r = b0 + b;
        if (r >= n_rows) return nullptr;
        uint16_t *yrow = r < n_main ? y + batch_token(r, out_idx, tF, tN) * C : y_ctx + (long)(r - n_main) * C;
        return yrow + a0 + c0;
    });
}

__global__ void k_to_f16(const uint4 *__restrict__ src, long n8, uint4 *__restrict__ dst) {
    to_f16(src, n8, dst, (long)blockIdx.x * blockDim.x + threadIdx.x, (long)gridDim.x * blockDim.x);
}

hipError_t launch_proj_out(const Plan &p, int n_rows, const AttnArgs &a, hipStream_t st) {
    const long n8 = (long)p.C * p.hd / 8;
    if (!a.wo16_ready) {
        StageScope _stage(st, "wo_f16");
        const long blocks = (n8 + 255) / 256;
        launch_k(k_to_f16, (unsigned)(blocks < 2048 ? blocks : 2048), 256, 0, st, (const uint4 *)a.wo, n8,
                                                                            (uint4 *)a.wo16);
    }
    StageScope _stage(st, "proj_out");
    const int id = ring_pick(p.hd, [&](int BA, int BB) { return (long)cdiv(p.C, BA) * cdiv(n_rows, BB); });
    return ring_dispatch(id, [&](auto c) -> hipError_t {
        constexpr int ID = decltype(c)::value;
        using T = typename RingShape<ID, true>::Tile;
        const hipError_t e = allow_lds(k_proj_out<ID>, T::LDS_BYTES);
        if (e != hipSuccess) return e;
        const int n_at = cdiv(p.C, T::BA), n_bt = cdiv(n_rows, T::BB);
        launch_k(k_proj_out<ID>, n_at * n_bt, T::NT, T::LDS_BYTES, st, (const uint16_t *)a.o, n_rows, p.hd,
                 (const uint16_t *)a.wo16, p.C, a.n_main, a.out_idx, a.tF, a.tN, n_at, n_bt, (uint16_t *)a.y,
                 (uint16_t *)a.y_ctx);
        return hipGetLastError();
    });
}

}  // namespace oc
