// Matching kernels: descriptor inverse norms and the similarity tile GEMM
// with a fused row arg-max (OmniCache §3.2.1-§3.2.3 cosine-similarity
// matching, patch-local per §3.3).  Group members come from GroupMap.
#include "oc_internal.h"
#include "oc_launch.h"
#include "oc_groups.h"
#include "oc_device.h"
#include "oc_mfma_tile.h"
#include "oc_dma_tile.h"
#include "oc_ring_tile.h"
#include "oc_f32_tile.h"
#include "oc_attn_common.h"
#include <algorithm>

namespace oc {

// ----------------------------------------------------------------------------
// inverse L2 norms of item descriptors: one wave per item, or one block per
// item for descriptors made of several segments (blocks: a position over all
// frames); blocks past the norm blocks convert the output-projection weights
// bf16 -> fp16 (exact in the fp16 normal range, saturating outside), 8
// elements per thread
// ----------------------------------------------------------------------------
// lanes per item for rows of `chunks` 16-byte chunks: the largest power of
// two not above chunks, between 8 and 64
__host__ __device__ inline int lanes_per_item(int chunks) {
    int l = 8;
    while (l < 64 && 2 * l <= chunks) l *= 2;
    return l;
}

template <typename T>
__global__ void k_inv_norm(const T *__restrict__ x, float *__restrict__ inv, int n_items, int n_sub,
                           long sub_stride, int C, int norm_blocks, unsigned long long *__restrict__ pack,
                           long n_pack, const uint4 *__restrict__ wo, long n8, uint4 *__restrict__ wo16) {
    if ((int)blockIdx.x >= norm_blocks) {
        const long nb = gridDim.x - norm_blocks;
        for (long i = (long)(blockIdx.x - norm_blocks) * blockDim.x + threadIdx.x; i < n8; i += nb * blockDim.x)
            wo16[i] = bf16x8_to_f16x8(wo[i]);
        return;
    }
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n_pack; i += (long)norm_blocks * blockDim.x)
        pack[i] = 0ull;
    constexpr int VEC = 16 / sizeof(T);
    const int lane = threadIdx.x & (WAVE - 1);
    if (n_sub > 1) {
        // block per item: the segments' 16-byte chunks spread over the block,
        // partial sums reduced in a fixed order
        __shared__ float wsum[4];
        const int item = blockIdx.x;
        const int cpr = C / VEC;
        float ss = 0.f;
        const int nq = n_sub * cpr;
        // four chunks' loads in flight before their sums (same order of
        // accumulation as one chunk at a time)
        for (int q0 = threadIdx.x; q0 < nq; q0 += 4 * blockDim.x) {
            // (a chunk past the end re-reads the last one, unbranched, and
            // its sum is dropped)
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = min(q0 + u * (int)blockDim.x, nq - 1);
                const int sg = q / cpr, c = (q - sg * cpr) * VEC;
                v[u] = *reinterpret_cast<const uint4 *>(x + sg * sub_stride + (long)item * C + c);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const T *e = reinterpret_cast<const T *>(&v[u]);
                float part = ss;
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    const float f = Elem<T>::ld(e + j);
                    part = fmaf(f, f, part);
                }
                ss = q0 + u * (int)blockDim.x < nq ? part : ss;
            }
        }
        ss = wave_sum(ss);
        if (lane == 0) wsum[threadIdx.x / WAVE] = ss;
        __syncthreads();
        if (threadIdx.x == 0) {
            const float t = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
            inv[item] = t > 0.f ? (float)(1.0 / sqrt((double)t)) : 0.f;
        }
        return;
    }
    // LPI lanes per item (a power of two up to 64, about one 16-byte chunk
    // per lane for short rows): 256 / LPI items per block
    const int lpi = lanes_per_item(C / VEC);
    const int sub = threadIdx.x & (lpi - 1);
    const int item = blockIdx.x * (blockDim.x / lpi) + threadIdx.x / lpi;
    if (item >= n_items) return;   // (whole lane groups: the reduction below stays inside one)
    const T *row = x + (long)item * C;
    float ss = 0.f;
    // up to four chunks' loads in flight before their sums (same order of
    // accumulation as one chunk at a time)
    const int step = lpi * VEC;
    for (int c0 = sub * VEC; c0 < C; c0 += 4 * step) {
        // (a chunk past the end re-reads the last one, unbranched, and its
        // sum is dropped)
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = *reinterpret_cast<const uint4 *>(row + min(c0 + u * step, C - VEC));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T *e = reinterpret_cast<const T *>(&v[u]);
            float part = ss;
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const float f = Elem<T>::ld(e + j);
                part = fmaf(f, f, part);
            }
            ss = c0 + u * step < C ? part : ss;
        }
    }
    for (int o = lpi >> 1; o > 0; o >>= 1) ss += __shfl_xor(ss, o, WAVE);
    if (sub == 0) inv[item] = ss > 0.f ? (float)(1.0 / sqrt((double)ss)) : 0.f;
}

hipError_t launch_inv_norm(const Plan &p, const void *x, float *inv, unsigned long long *node_pack, long n_pack,
                           const void *wo, void *wo16, long n_wo, hipStream_t st) {
    StageScope _stage(st, "inv_norm");
    const int n_items = p.kind == KIND_BLOCK ? p.N : p.F * p.N;
    const int n_sub = p.kind == KIND_BLOCK ? p.F : 1;
    const long sub = (long)p.N * p.C;
    const int chunks = p.C / (p.bf16 ? 8 : 4);
    const int blocks = n_sub > 1 ? n_items : cdiv(n_items, 256 / lanes_per_item(chunks));
    const long n8 = (wo && wo16 && p.bf16) ? n_wo / 8 : 0;
    const int cvt_blocks = n8 > 0 ? (int)std::min<long>((n8 + 255) / 256, 1024) : 0;
    if (p.bf16)
        launch_k(k_inv_norm<uint16_t>, blocks + cvt_blocks, 256, 0, st, (const uint16_t *)x, inv, n_items, n_sub, sub, p.C,
                                                                 blocks, node_pack, n_pack, (const uint4 *)wo, n8,
                                                                 (uint4 *)wo16);
    else
        launch_k(k_inv_norm<float>, blocks, 256, 0, st, (const float *)x, inv, n_items, n_sub, sub, p.C, blocks, node_pack,
                                                  n_pack, nullptr, 0, nullptr);
    return hipGetLastError();
}

// Frame Cache on patches: one block per (frame, patch) tile, the sum of
// squares of its ph rows of pw*C elements (16-byte chunks spread over the
// block, wave partials added in a fixed order), stored at the tile's
// top-left token; the blocks past the tiles clear pack and convert wo.
// There are fewer tiles than compute units (64 of 147 KB on a Latte-like
// layer), so a tile takes sixteen waves with four loads each in flight
// (14.2 us with four waves and one load, 6.1 us this way).
template <typename T>
__global__ __launch_bounds__(1024) void k_tile_norm(const T *__restrict__ x, float *__restrict__ inv, int F, int N, int W, int k, int ph,
                            int pw, int C, int norm_blocks, unsigned long long *__restrict__ pack, long n_pack,
                            const uint4 *__restrict__ wo, long n8, uint4 *__restrict__ wo16) {
    if ((int)blockIdx.x >= norm_blocks) {
        const long nb = gridDim.x - norm_blocks;
        for (long i = (long)(blockIdx.x - norm_blocks) * blockDim.x + threadIdx.x; i < n8; i += nb * blockDim.x)
            wo16[i] = bf16x8_to_f16x8(wo[i]);
        return;
    }
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n_pack; i += (long)norm_blocks * blockDim.x)
        pack[i] = 0ull;
    constexpr int VEC = 16 / sizeof(T);
    __shared__ float wsum[16];
    const int kk = k * k, f = blockIdx.x / kk, g = blockIdx.x - f * kk;
    const long tl = (long)f * N + (long)(g / k) * ph * W + (g % k) * pw;
    const int cpr = pw * C / VEC, n_q = ph * cpr;   // 16-byte chunks per tile row and tile
    float ss = 0.f;
    for (int q0 = threadIdx.x; q0 < n_q; q0 += 4 * blockDim.x) {
        // (a chunk past the end re-reads the last one, unbranched, and its
        // sum is dropped)
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = min(q0 + u * (int)blockDim.x, n_q - 1);
            const int row = q / cpr, c = (q - row * cpr) * VEC;
            v[u] = *reinterpret_cast<const uint4 *>(x + (tl + (long)row * W) * C + c);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T *e = reinterpret_cast<const T *>(&v[u]);
            float part = ss;
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const float fv = Elem<T>::ld(e + j);
                part = fmaf(fv, fv, part);
            }
            ss = q0 + u * (int)blockDim.x < n_q ? part : ss;
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & (WAVE - 1)) == 0) wsum[threadIdx.x / WAVE] = ss;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < (int)(blockDim.x / WAVE); ++w) t += wsum[w];
        inv[tl] = t > 0.f ? (float)(1.0 / sqrt((double)t)) : 0.f;
    }
}

hipError_t launch_tile_norm(const Plan &p, const void *x, float *inv, unsigned long long *node_pack, long n_pack,
                            const void *wo, void *wo16, long n_wo, hipStream_t st) {
    StageScope _stage(st, "inv_norm");
    const int blocks = p.F * p.k * p.k;
    const long n8 = (wo && wo16 && p.bf16) ? n_wo / 8 : 0;
    const int threads = (long)p.ph * p.pw * p.C * p.esz >= 64 << 10 ? 1024 : 256;   // (four loads each over 64 KB)
    const int cvt_blocks = n8 > 0 ? (int)std::min<long>((n8 + threads - 1) / threads, 1024) : 0;
    if (p.bf16)
        launch_k(k_tile_norm<uint16_t>, blocks + cvt_blocks, threads, 0, st, (const uint16_t *)x, inv, p.F, p.N, p.W, p.k,
                 p.ph, p.pw, p.C, blocks, node_pack, n_pack, (const uint4 *)wo, n8, (uint4 *)wo16);
    else
        launch_k(k_tile_norm<float>, blocks, threads, 0, st, (const float *)x, inv, p.F, p.N, p.W, p.k, p.ph, p.pw, p.C,
                 blocks, node_pack, n_pack, nullptr, 0, nullptr);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// similarity + arg-max, bf16 MFMA
// ----------------------------------------------------------------------------
// Block (candidate tile bt, representative tile at, group g), in an
// XCD-aware order: t = dot(src_b, dst_a) * inv(dst_a); per candidate the
// largest t over this block's representatives (smallest position on ties)
// is merged into node_pack[g][b] with one 64-bit atomic maximum of the
// packed pair, so the representative tiles need no second pass.  The
// representative norm is applied before the arg-max, the candidate's own
// norm (a positive constant per row) when unpacking.
// Frame tiles (at most 16 representatives) and blocks whose channels are no
// whole K steps.
template <int BA, int BB, int WA, int WB>
__global__ __launch_bounds__(256) void k_match_mfma(const uint16_t *__restrict__ x, const float *__restrict__ inv,
                                                     GroupMap gm, int G, int S, int D,
                                                     int K, int seg_len, long sub_stride, long item_stride,
                                                     int n_bt, int n_at,
                                                     unsigned long long *__restrict__ node_pack) {
    using T = MfmaTile<BA, BB, WA, WB>;
    extern __shared__ __align__(16) uint16_t lds[];
    const int total = n_bt * n_at * G;
    const int lid = xcd_remap(blockIdx.x, total);
    // consecutive logical blocks: the representative tiles of one candidate tile
    const int at = lid % n_at, bt = (lid / n_at) % n_bt, g = lid / (n_at * n_bt);
    const GroupMap::Grp gr = gm.group(g);
    if (bt * BB >= gr.nsrc) return;   // past this group's candidates (groups of one call differ in size)
    const uint16_t *rowsA[T::CA], *rowsB[T::CB];
#pragma unroll
    for (int i = 0; i < T::CA; ++i) {
        const int a = at * BA + T::chunk_row(i);
        const int id = a < D ? gm.dst_id(gr, a) : -1;
        rowsA[i] = id >= 0 ? x + (long)id * item_stride : nullptr;
    }
#pragma unroll
    for (int i = 0; i < T::CB; ++i) {
        const int b = bt * BB + T::chunk_row(i);
        const int id = b < S ? gm.src_id(gr, b) : -1;
        rowsB[i] = id >= 0 ? x + (long)id * item_stride : nullptr;
    }
    T tile;
    // rows without an item read zeros; their results are discarded below
    tile.run(lds, rowsA, rowsB, K, seg_len, sub_stride);

    // representative norms of this tile (0 for padding, which never wins)
    float *sinv = reinterpret_cast<float *>(lds);
    float *sv = sinv + BA;
    int *si = reinterpret_cast<int *>(sv + WA * BB);
    for (int a = threadIdx.x; a < BA; a += 256) {
        const int ga = at * BA + a;
        const int id = ga < D ? gm.dst_id(gr, ga) : -1;
        sinv[a] = id >= 0 ? inv[id] : -1.f;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wa = wave / WB;
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        float bv = -INFINITY;
        int bi = -1;
#pragma unroll
        for (int i = 0; i < T::TA; ++i)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int al = T::a_of(i, g4) + e;
                    const float w = sinv[al];
                    if (w >= 0.f) argmax_merge(bv, bi, tile.acc[i][j][4 * g4 + e] * w, at * BA + al);
                }
        const float v2 = __shfl_xor(bv, 32, WAVE);
        const int i2 = __shfl_xor(bi, 32, WAVE);
        argmax_merge(bv, bi, v2, i2);
        if (lane < 32) {
            const int bl = T::b_of(j);
            sv[wa * BB + bl] = bv;
            si[wa * BB + bl] = bi;
        }
    }
    __syncthreads();
    // merge the WA waves that share a candidate range, in ascending a order
    for (int bl = threadIdx.x; bl < BB; bl += 256) {
        float v = sv[bl];
        int ix = si[bl];
        for (int w = 1; w < WA; ++w) argmax_merge(v, ix, sv[w * BB + bl], si[w * BB + bl]);
        const int b = bt * BB + bl;
        if (b < S && ix >= 0) atomicMax(&node_pack[(long)g * S + b], pack_argmax(v, ix));
    }
}

// Token groups, and blocks whose channels are whole K steps (a position's
// descriptor is a segment per frame): ring-buffered tiles of
// representatives (a) by candidates (b).  A block takes one candidate tile of
// one group and n_at / n_part of its representative tiles, back to back in
// one pipeline; it keeps each candidate's best (value, position) in registers
// and merges it into node_pack once, by the packed atomic maximum.  The
// block's representatives (offset and inverse norm) are tabled in LDS first.
//
// The grid holds the tiles that exist and no others: t_one candidate tiles
// per patch of an unpaired unit, t_pair per patch of a frame pair, and a block
// finds its group by counting through the units.  (A grid of the largest
// group's tiles for every group, in contiguous ranges per XCD, left the XCDs
// whose range held few pairs idle for much of the launch.)
//
// Bounded by the MFMA rate at the clock the load leaves (248 of 290 us with
// the arg-max between the tiles reduced to a maximum).  Parts of one candidate
// tile are adjacent, so they share its rows in one XCD's L2.  25 frames of 72
// x 128 tokens of 320 channels, 5 pairs: 654 us on 128 x 128 tiles and the
// full grid, 290 us this way; 12 pairs matched in 4 x 4 patches 91 -> 71;
// 3072 x 1024 x 1536: 20.5 -> 19.8; 1024 tokens of C = 160 13.2 -> 8.4; blocks
// of 25 frames of 320 channels, 16 groups of 432 x 144: 78 -> 62.
template <int ID>
__global__ __launch_bounds__(RING_THREADS<ID>) void k_match_ring(const uint16_t *__restrict__ x,
                                                                 const float *__restrict__ inv, GroupMap gm,
                                                                 int n_units, int S, int D, int K, int seg_len,
                                                                 long sub_stride, long item_stride, int t_one,
                                                                 int t_pair, int n_at, int n_part, int total,
                                                                 unsigned long long *__restrict__ node_pack) {
    using T = typename RingShape<ID, false>::Tile;
    constexpr int BA = T::BA, BB = T::BB, NT = T::NT, WA = BA / T::WTA;
    extern __shared__ __align__(16) uint16_t lds[];
    float *const snorm = reinterpret_cast<float *>(lds + T::RING_BYTES / 2);
    const int lid = xcd_remap(blockIdx.x, total);
    const int part = lid % n_part, kk = gm.k * gm.k;
    const int u0 = part * n_at / n_part, u1 = (part + 1) * n_at / n_part;   // this block's representative tiles
    uint32_t *const soff = reinterpret_cast<uint32_t *>(snorm + (u1 - u0) * BA);
    int tl = lid / n_part, unit = 0, t_g = t_one;
    if (gm.units == nullptr) {
        unit = tl / (kk * t_one);
        tl -= unit * kk * t_one;
    } else {
        int at = 0, first = 0;
        unit = -1;
        for (int u = 0; u < n_units; ++u) {
            const int t_u = gm.group(u * kk).pair ? t_pair : t_one;
            if (tl >= at && tl < at + kk * t_u) {
                unit = u;
                t_g = t_u;
                first = at;
            }
            at += kk * t_u;
        }
        tl -= first;
        if (unit < 0) return;   // (a unit table with fewer pairs than planned)
    }
    const int g = unit * kk + tl / t_g, b0 = tl % t_g * BB;
    const GroupMap::Grp gr = gm.group(g);
    for (int a = threadIdx.x; a < (u1 - u0) * BA; a += NT) {
        const int id = u0 * BA + a < D ? gm.dst_id(gr, u0 * BA + a) : -1;
        snorm[a] = id >= 0 ? inv[id] : -1.f;                 // padding never wins
        soff[a] = (uint32_t)max(id, 0) * (uint32_t)(item_stride * 2);
    }
    typename T::RowsB rb;
    rb.base2 = x;
    rb.mix = rb.alt = 0;
#pragma unroll
    for (int i = 0; i < T::CB; ++i) {
        const int b = b0 + rb.row(i), id = b < S ? gm.src_id(gr, b) : -1;
        rb.base[i] = x;
        rb.off[i] = (uint32_t)max(id, 0) * (uint32_t)(item_stride * 2) + (uint32_t)rb.chunk() * 16;
    }
    __syncthreads();
    float bv[T::TB];
    int bi[T::TB];
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        bv[j] = -INFINITY;
        bi[j] = -1;
    }
    T tile;
    auto load_a = [&](typename T::RowsA &ra, int u) {
        ra.base2 = x;
        ra.mix = ra.alt = 0;
#pragma unroll
        for (int i = 0; i < T::CA; ++i) {
            ra.base[i] = x;
            ra.off[i] = soff[u * BA + ra.row(i)] + (uint32_t)ra.chunk() * 16;
        }
    };
    // per tile: scale by the representative norms, take the maximum of 16
    // accumulators (four quads of consecutive positions), and only when it
    // beats the running best find its smallest position, the first quad that
    // holds it and then the first in the quad (positions rise with the tiles,
    // so a later equal value never replaces an earlier one); lane halves and
    // waves are merged at the end
    auto epi = [&](int u) {
        const bool full = (u0 + u + 1) * BA <= D;
#pragma unroll
        for (int i = 0; i < T::TA; ++i) {
            float w[16];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const float4 v = *reinterpret_cast<const float4 *>(&snorm[u * BA + T::a_of(i, g4)]);
                w[4 * g4] = v.x;
                w[4 * g4 + 1] = v.y;
                w[4 * g4 + 2] = v.z;
                w[4 * g4 + 3] = v.w;
            }
            const int base = (u0 + u) * BA + T::a_of(i, 0);
#pragma unroll
            for (int j = 0; j < T::TB; ++j) {
                float t[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) t[k] = tile.acc[i][j][k] * w[k];
                if (!full) {
                    // (padding: a NaN, which no maximum takes and no comparison finds)
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        if (w[k] < 0.f) t[k] = __builtin_nanf("");
                }
                float m4[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    m4[q] = fmaxf(fmaxf(fmaxf(t[4 * q], t[4 * q + 1]), t[4 * q + 2]), t[4 * q + 3]);
                const float m = fmaxf(fmaxf(fmaxf(m4[0], m4[1]), m4[2]), m4[3]);
                if (m >= bv[j]) {
                    float s0 = t[12], s1 = t[13], s2 = t[14];
                    int ix = base + 24;
#pragma unroll
                    for (int q = 2; q >= 0; --q) {
                        const bool here = m4[q] == m;
                        s0 = here ? t[4 * q] : s0;
                        s1 = here ? t[4 * q + 1] : s1;
                        s2 = here ? t[4 * q + 2] : s2;
                        ix = here ? base + 8 * q : ix;
                    }
                    ix += s0 == m ? 0 : s1 == m ? 1 : s2 == m ? 2 : 3;
                    // (an equal value replaces none but the start: products of -inf only)
                    bi[j] = m > bv[j] || bi[j] < 0 ? ix : bi[j];
                    bv[j] = m;
                }
            }
        }
    };
    tile.run_tiles(lds, load_a, rb, K, seg_len, sub_stride, u1 - u0, epi);
    const int lane = threadIdx.x & 63, wa = (threadIdx.x >> 6) / (BB / T::WTB);
    float *const sv = reinterpret_cast<float *>(lds);   // the ring, free now
    int *const si = reinterpret_cast<int *>(sv + WA * BB);
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        argmax_merge(bv[j], bi[j], __shfl_xor(bv[j], 32, WAVE), __shfl_xor(bi[j], 32, WAVE));
        if (lane < 32) {
            sv[wa * BB + T::b_of(j)] = bv[j];
            si[wa * BB + T::b_of(j)] = bi[j];
        }
    }
    __syncthreads();
    for (int bl = threadIdx.x; bl < BB; bl += NT) {
        float v = sv[bl];
        int ix = si[bl];
#pragma unroll
        for (int w = 1; w < WA; ++w) argmax_merge(v, ix, sv[w * BB + bl], si[w * BB + bl]);
        if (b0 + bl < gr.nsrc && b0 + bl < S && ix >= 0)
            atomicMax(&node_pack[(long)g * S + b0 + bl], pack_argmax(v, ix));
    }
}

// Split-K variant for long descriptors and few tiles (Block Cache: a
// position's descriptor spans all frames): block (tile, split) computes the
// raw dot products over its K range (whole 64-steps inside one segment) and
// stores them to part[split][g][b][a]; k_match_part_reduce sums the splits in
// order, applies the representative norms and takes the arg-max.
template <int BA, int BB, int WA, int WB>
__global__ __launch_bounds__(256) void k_match_part(const uint16_t *__restrict__ x, GroupMap gm, int G, int S, int D,
                                                     int kc, int seg_len, long sub_stride, long item_stride,
                                                     int n_bt, int n_at, int n_split, float *__restrict__ part) {
    using T = DmaTile<BA, BB, WA, WB>;
    extern __shared__ __align__(16) uint16_t lds[];
    const int total = n_bt * n_at * G * n_split;
    const int lid = xcd_remap(blockIdx.x, total);
    const int sp = lid % n_split, tl = lid / n_split;
    const int at = tl % n_at, bt = (tl / n_at) % n_bt, g = tl / (n_at * n_bt);
    const GroupMap::Grp gr = gm.group(g);
    if (bt * BB >= gr.nsrc) return;
    // K range of this split: inside one segment
    const long k0 = (long)sp * kc;
    const long off = seg_len > 0 ? (k0 / seg_len) * sub_stride + (k0 % seg_len) : k0;
    const uint16_t *rowsA[T::CA], *rowsB[T::CB];
#pragma unroll
    for (int i = 0; i < T::CA; ++i) {
        const int a = at * BA + T::chunk_row(i);
        const int id = a < D ? gm.dst_id(gr, a) : -1;
        rowsA[i] = id >= 0 ? x + (long)id * item_stride + off : nullptr;
    }
#pragma unroll
    for (int i = 0; i < T::CB; ++i) {
        const int b = bt * BB + T::chunk_row(i);
        const int id = b < S ? gm.src_id(gr, b) : -1;
        rowsB[i] = id >= 0 ? x + (long)id * item_stride + off : nullptr;
    }
    T tile;
    tile.run(lds, rowsA, rowsB, x, x, kc);   // (rows without an item read x's first row)
    float *pp = part + ((long)sp * G + g) * S * D;
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        const int b = bt * BB + T::b_of(j);
        if (b >= S) continue;
#pragma unroll
        for (int i = 0; i < T::TA; ++i)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int a = at * BA + T::a_of(i, g4) + e;
                    if (a < D) pp[(long)b * D + a] = tile.acc[i][j][4 * g4 + e];
                }
    }
}

// One block per (group, candidate): wave q sums the splits q, q+4, ... of
// representatives a = lane + 64c, wave 0 adds the four partial sums in order,
// applies the representative norm and keeps the arg-max.
__global__ __launch_bounds__(256) void k_match_part_reduce(const float *__restrict__ part, int n_split, int G, int S,
                                                            int D, const float *__restrict__ inv, GroupMap gm,
                                                            unsigned long long *__restrict__ node_pack) {
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int g = blockIdx.x / S, b = blockIdx.x - g * S;
    const GroupMap::Grp gr = gm.group(g);
    if (gm.src_id(gr, b) < 0) return;
    float bv = -INFINITY;
    int bi = -1;
    for (int a0 = 0; a0 < D; a0 += 64) {
        const int a = a0 + lane;
        float sum = 0.f;
        if (a < D) {
            // splits q, q+4, ... added in ascending order; the loads of eight
            // of them are issued before the first is added
            const long stride = 4L * G * S * D;
            const float *pp = part + (((long)q * G + g) * S + b) * D + a;
            for (int sp0 = q; sp0 < n_split; sp0 += 32, pp += 8 * stride) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = sp0 + 4 * u < n_split ? pp[u * stride] : 0.f;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (sp0 + 4 * u < n_split) sum += v[u];
            }
        }
        red[q][lane] = sum;
        __syncthreads();
        if (q == 0 && a < D) {
            const int id = gm.dst_id(gr, a);
            const float dot = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
            if (id >= 0) argmax_merge(bv, bi, dot * inv[id], a);
        }
        __syncthreads();
    }
    if (q != 0) return;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) argmax_merge(bv, bi, __shfl_xor(bv, o, WAVE), __shfl_xor(bi, o, WAVE));
    if (lane == 0 && bi >= 0) node_pack[(long)g * S + b] = pack_argmax(bv, bi);
}

// fp32 similarity + arg-max: tiles of representatives (a) by candidates (b),
// each candidate's best merged by the packed atomic maximum as above (one
// thread per candidate, its dot products one after the other, took 8030 us at
// 768 x 256 x 320 on 12 blocks; the tiles take 8.1).
template <typename T, int BA, int BB>
__global__ __launch_bounds__(256) void k_match_f32(const float *__restrict__ x, const float *__restrict__ inv,
                                                   GroupMap gm, int G, int S, int D, int K, int seg_len,
                                                   long sub_stride, long item_stride, int n_bt, int n_at,
                                                   unsigned long long *__restrict__ node_pack) {
    extern __shared__ __align__(16) float ldsf[];
    __shared__ float sinv[BA], sv[2][BB];
    __shared__ int si[2][BB];
    const int id = (int)folded_block(), at = id % n_at, bt = (id / n_at) % n_bt, g = id / (n_at * n_bt);
    if (g >= G) return;
    const GroupMap::Grp gr = gm.group(g);
    if (bt * BB >= gr.nsrc) return;
    const float *rowsA[T::NA], *rowsB[T::NB];
#pragma unroll
    for (int i = 0; i < T::NA; ++i) {
        const int a = at * BA + T::load_row(i), id = a < D ? gm.dst_id(gr, a) : -1;
        rowsA[i] = id >= 0 ? x + (long)id * item_stride : nullptr;
    }
#pragma unroll
    for (int i = 0; i < T::NB; ++i) {
        const int b = bt * BB + T::load_row(i), id = b < S ? gm.src_id(gr, b) : -1;
        rowsB[i] = id >= 0 ? x + (long)id * item_stride : nullptr;
    }
    // representative norms (-1 for padding, which never wins)
    for (int a = threadIdx.x; a < BA; a += 256) {
        const int id = at * BA + a < D ? gm.dst_id(gr, at * BA + a) : -1;
        sinv[a] = id >= 0 ? inv[id] : -1.f;
    }
    T t;
    t.run(ldsf, rowsA, rowsB, K, seg_len, sub_stride);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        float bv = -INFINITY;
        int bi = -1;
#pragma unroll
        for (int i = 0; i < T::TA; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int al = T::a_of(i) + e;
                const float w = sinv[al];
                if (w >= 0.f) argmax_merge(bv, bi, t.acc[i][j][e] * w, at * BA + al);
            }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) argmax_merge(bv, bi, __shfl_xor(bv, o, WAVE), __shfl_xor(bi, o, WAVE));
        if (lane < 16) {
            sv[wave >> 1][T::b_of(j)] = bv;
            si[wave >> 1][T::b_of(j)] = bi;
        }
    }
    __syncthreads();
    for (int bl = threadIdx.x; bl < BB; bl += 256) {
        float v = sv[0][bl];
        int ix = si[0][bl];
        argmax_merge(v, ix, sv[1][bl], si[1][bl]);
        const int b = bt * BB + bl;
        if (b < S && ix >= 0) atomicMax(&node_pack[(long)g * S + b], pack_argmax(v, ix));
    }
}

// Unpack the best pair, convert the winning position to a global id and
// apply the candidate's norm.
__global__ void k_match_unpack(const unsigned long long *__restrict__ node_pack, int G, int S,
                               const float *__restrict__ inv, GroupMap gm, float *__restrict__ node_max,
                               int32_t *__restrict__ node_idx) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long)G * S) return;
    const int g = (int)(i / S);
    const GroupMap::Grp gr = gm.group(g);
    const int sid = gm.src_id(gr, (int)(i - (long)g * S));
    if (sid < 0) {
        node_max[i] = -INFINITY;
        node_idx[i] = -1;
        return;
    }
    float v;
    int ix;
    unpack_argmax(node_pack[i], v, ix);
    node_max[i] = v * inv[sid];
    node_idx[i] = ix >= 0 ? gm.dst_id(gr, ix) : -1;
}

template <typename KernelPtr>
static hipError_t allow_lds(KernelPtr k, size_t lds) {
    return raise_lds_limit((const void *)k, lds);
}

template <int BA, int BB, int WA, int WB>
static hipError_t go_match(const Plan &p, const uint16_t *x, const float *inv, const GroupMap &gm, const MatchGeom &mg,
                           unsigned long long *node_pack, hipStream_t st) {
    using T = MfmaTile<BA, BB, WA, WB>;
    const int G = p.n_groups, S = p.n_src_max, D = p.n_dst_max;
    const int n_bt = cdiv(S, BB), n_at = cdiv(D, BA);
    const size_t lds = T::LDS_BYTES;
    hipError_t e = allow_lds(k_match_mfma<BA, BB, WA, WB>, lds);
    if (e != hipSuccess) return e;
    launch_k(k_match_mfma<BA, BB, WA, WB>, n_bt * n_at * G, 256, lds, st, x, inv, gm, G, S, D, mg.K, mg.seg_len,
             mg.sub_stride, mg.item_stride, n_bt, n_at, node_pack);
    return hipGetLastError();
}

// Tile shape and parts per candidate tile with the lowest cost: each block
// pays a shape's fixed part once and, per representative tile, its steps and
// the arg-max (2.7e-5 us per product on its own unit: three to four vector
// instructions each).
constexpr size_t MATCH_LDS = 160 * 1024;   // of a compute unit
struct MatchPick { int id, n_part; };
static MatchPick match_pick(const Plan &p, int K, int n_units, int n_pairs) {
    const int kk = p.k * p.k, D = p.n_dst_max, nk = cdiv(K, 64);
    constexpr size_t ring[N_RING_SHAPES] = {RING_LDS<0>, RING_LDS<1>, RING_LDS<2>, RING_LDS<3>, RING_LDS<4>,
                                            RING_LDS<5>, RING_LDS<6>, RING_LDS<7>, RING_LDS<8>, RING_LDS<9>};
    MatchPick best{-1, 1};
    float best_t = 0.f;
    for (int i = 0; i < N_RING_SHAPES; ++i) {
        const RingShapeCost &c = RING_SHAPES[i];
        const int n_at = cdiv(D, c.BA);
        const long bts = (long)kk * ((long)(n_units - n_pairs) * cdiv(p.np_src, c.BB) +
                                     (long)n_pairs * cdiv(p.np + p.np_src, c.BB));
        for (int parts = 1; parts <= n_at; ++parts) {
            const int per = cdiv(n_at, parts);   // representative tiles of the longest block
            if (parts > 1 && per == cdiv(n_at, parts - 1)) continue;
            if ((ring[i] + (size_t)per * c.BA * 8) * c.resident > MATCH_LDS) continue;
            const float t = ring_cost(c, nk * per, bts * parts, 2.7e-5f * c.BA * c.BB * per);
            if (best.id < 0 || t < best_t) {
                best = MatchPick{i, parts};
                best_t = t;
            }
        }
    }
    return best;
}

static hipError_t go_ring(const Plan &p, const uint16_t *x, const float *inv, const GroupMap &gm, const MatchGeom &mg,
                          unsigned long long *node_pack, hipStream_t st) {
    const int n_pairs = gm.units != nullptr ? p.R_f : 0, kk = p.k * p.k;
    const int n_units = p.kind == KIND_BLOCK ? 1 : p.n_units;   // (blocks: one group per patch)
    const MatchPick pick = match_pick(p, mg.K, n_units, n_pairs);
    return ring_dispatch(pick.id, [&](auto c) -> hipError_t {
        constexpr int ID = decltype(c)::value;
        using T = typename RingShape<ID, false>::Tile;
        const int n_at = cdiv(p.n_dst_max, T::BA);
        const int t_one = cdiv(p.np_src, T::BB), t_pair = cdiv(p.np + p.np_src, T::BB);
        const int total = kk * ((n_units - n_pairs) * t_one + n_pairs * t_pair) * pick.n_part;
        const size_t lds = T::RING_BYTES + (size_t)cdiv(n_at, pick.n_part) * T::BA * 8;
        const hipError_t e = raise_lds_limit((const void *)k_match_ring<ID>, MATCH_LDS);
        if (e != hipSuccess) return e;
        launch_k(k_match_ring<ID>, total, T::NT, lds, st, x, inv, gm, n_units, p.n_src_max, p.n_dst_max, mg.K,
                 mg.seg_len, mg.sub_stride, mg.item_stride, t_one, t_pair, n_at, pick.n_part, total, node_pack);
        return hipGetLastError();
    });
}

template <int BA, int BB, int WA, int WB>
static hipError_t go_split(const Plan &p, const MatchSplit &ms, const uint16_t *x, const float *inv,
                           const GroupMap &gm, const MatchGeom &mg, float *part, unsigned long long *node_pack,
                           hipStream_t st) {
    using T = DmaTile<BA, BB, WA, WB>;
    const int G = p.n_groups, S = p.n_src_max, D = p.n_dst_max;
    const int n_bt = cdiv(S, BB), n_at = cdiv(D, BA);
    const size_t lds = T::LDS_BYTES;
    hipError_t e = allow_lds(k_match_part<BA, BB, WA, WB>, lds);
    if (e != hipSuccess) return e;
    launch_k(k_match_part<BA, BB, WA, WB>, n_bt * n_at * G * ms.n_split, 256, lds, st, x, gm, G, S, D, ms.kc, mg.seg_len,
             mg.sub_stride, mg.item_stride, n_bt, n_at, ms.n_split, part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_k(k_match_part_reduce, (unsigned)((long)G * S), 256, 0, st, (const float *)part, ms.n_split, G, S, D, inv,
             gm, node_pack);
    return hipGetLastError();
}

template <typename T, int B>
static hipError_t go_match_f32(const Plan &p, const float *x, const float *inv, const GroupMap &gm,
                               const MatchGeom &mg, unsigned long long *node_pack, hipStream_t st) {
    const int S = p.n_src_max, D = p.n_dst_max, n_bt = cdiv(S, B), n_at = cdiv(D, B);
    const hipError_t e = allow_lds(k_match_f32<T, B, B>, T::LDS_BYTES);
    if (e != hipSuccess) return e;
    const long blocks = (long)n_bt * n_at * p.n_groups;
    if (blocks >= (1L << 30)) return hipErrorInvalidValue;   // (2^28 tokens in the largest groups give a quarter)
    launch_k(k_match_f32<T, B, B>, folded_grid(blocks, 256), 256, T::LDS_BYTES, st, x, inv, gm, p.n_groups, S, D,
             mg.K, mg.seg_len, mg.sub_stride, mg.item_stride, n_bt, n_at, node_pack);
    return hipGetLastError();
}

hipError_t launch_match(const Plan &p, const void *x, const float *inv, const int32_t *units,
                        unsigned long long *node_pack, float *part, float *node_max, int32_t *node_idx,
                        hipStream_t st) {
    const GroupMap gm = group_map(p, units);
    const int G = p.n_groups, S = p.n_src_max, D = p.n_dst_max;
    const MatchGeom mg = match_geom(p);
    {
        StageScope _stage(st, "match");
        if (p.bf16) {
            const uint16_t *xb = (const uint16_t *)x;
            const MatchSplit ms = match_split(p);
            const bool steps = mg.K % 64 == 0 && mg.seg_len % 64 == 0;   // (of 64, whole in every segment)
            hipError_t e;
            if (ms.n_split > 1) {
                // long descriptors, few tiles: split K (64-row tiles)
                e = go_split<64, 64, 2, 2>(p, ms, xb, inv, gm, mg, part, node_pack, st);
            } else if (p.kind == KIND_TOKEN || (p.kind == KIND_BLOCK && steps)) {
                e = go_ring(p, xb, inv, gm, mg, node_pack, st);
            } else if (D > 64) {
                // representative tile height by group size: 128, 64 or 32
                e = go_match<128, 64, 2, 2>(p, xb, inv, gm, mg, node_pack, st);
            } else if (D > 32) {
                e = go_match<64, 64, 2, 2>(p, xb, inv, gm, mg, node_pack, st);
            } else {
                e = go_match<32, 128, 1, 4>(p, xb, inv, gm, mg, node_pack, st);
            }
            if (e != hipSuccess) return e;
        } else {
            const hipError_t e =
                f32_big(D, S, G) ? go_match_f32<F32Big, 64>(p, (const float *)x, inv, gm, mg, node_pack, st)
                                 : go_match_f32<F32Small, 32>(p, (const float *)x, inv, gm, mg, node_pack, st);
            if (e != hipSuccess) return e;
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || node_max == nullptr) return e;   // no outputs: the selection unpacks node_pack
    const long n = (long)G * S;
    {
        StageScope _stage(st, "match_unpack");
        launch_k(k_match_unpack, (unsigned)cdiv((int)n, 256), 256, 0, st, node_pack, G, S, inv, gm, node_max, node_idx);
    }
    return hipGetLastError();
}

}  // namespace oc
