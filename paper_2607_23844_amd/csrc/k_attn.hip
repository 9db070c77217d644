// Reduced-token attention dispatcher (OmniCache §3.2.3: the layer runs on
// the retained tokens only; cached tokens are neither queries nor
// keys/values), its workspace layout, and the fp32 path for small layers.
//
// bf16 layers: QKV projection (k_proj.hip) -> flash attention (k_flash.hip)
// -> output projection written straight to the output positions.
// fp32 layers: the same dataflow on fp32 MFMA (below).
#include "oc_attn_common.h"
#include "oc_f32_tile.h"
#include "oc_launch.h"

namespace oc {

struct RowMapF {
    const float *x; const int32_t *row_idx; int n_main;
    const float *ctx; int n_rows; int C;
    int tF, tN;
    __device__ __forceinline__ const float *row(int r) const {
        if (r < n_main) return x + batch_token(r, row_idx, tF, tN) * C;
        return ctx + (long)(r - n_main) * C;
    }
};

// Q/K/V[r][f] for f in [0, 3*hd): a = rows of wq, wk, wv, b = batch rows.
// (One output per thread, each its own dot product from memory, took 676 us
// on 512 rows of C = hd = 320; the tiles take 9.7.)
template <typename T, int BA, int BB>
__global__ __launch_bounds__(256) void k_proj_f32(RowMapF rm, const float *__restrict__ wq,
                                                  const float *__restrict__ wk, const float *__restrict__ wv, int hd,
                                                  int n_at, float *__restrict__ Q, float *__restrict__ K,
                                                  float *__restrict__ V) {
    extern __shared__ __align__(16) float ldsf[];
    const int at = blockIdx.x % n_at, bt = blockIdx.x / n_at;
    const float *rowsA[T::NA], *rowsB[T::NB];
#pragma unroll
    for (int i = 0; i < T::NA; ++i) {
        const int f = at * BA + T::load_row(i), which = f / hd, c = f - which * hd;
        rowsA[i] = f < 3 * hd ? (which == 0 ? wq : which == 1 ? wk : wv) + (long)c * rm.C : nullptr;
    }
#pragma unroll
    for (int i = 0; i < T::NB; ++i) {
        const int r = bt * BB + T::load_row(i);
        rowsB[i] = r < rm.n_rows ? rm.row(r) : nullptr;
    }
    T t;
    t.run(ldsf, rowsA, rowsB, rm.C, 0, 0);
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        const int r = bt * BB + T::b_of(j);
        if (r >= rm.n_rows) continue;
#pragma unroll
        for (int i = 0; i < T::TA; ++i) {
            // four consecutive features (hd is a multiple of 8: never across Q, K, V)
            const int f = at * BA + T::a_of(i), which = f / hd, c = f - which * hd;
            if (f < 3 * hd)
                *reinterpret_cast<f32x4 *>((which == 0 ? Q : which == 1 ? K : V) + (long)r * hd + c) = t.acc[i][j];
        }
    }
}

// y rows: a = rows of wo, b = rows of O (161 us for 512 rows of C = hd = 320
// by one thread per output, 5.3 by tiles)
template <typename T, int BA, int BB>
__global__ __launch_bounds__(256) void k_out_f32(const float *__restrict__ O, int n_rows, int hd,
                                                 const float *__restrict__ wo, int C, int n_main,
                                                 const int32_t *__restrict__ out_idx, int tF, int tN, int n_at,
                                                 float *__restrict__ y, float *__restrict__ y_ctx) {
    extern __shared__ __align__(16) float ldsf[];
    const int at = blockIdx.x % n_at, bt = blockIdx.x / n_at;
    const float *rowsA[T::NA], *rowsB[T::NB];
#pragma unroll
    for (int i = 0; i < T::NA; ++i) {
        const int a = at * BA + T::load_row(i);
        rowsA[i] = a < C ? wo + (long)a * hd : nullptr;
    }
#pragma unroll
    for (int i = 0; i < T::NB; ++i) {
        const int r = bt * BB + T::load_row(i);
        rowsB[i] = r < n_rows ? O + (long)r * hd : nullptr;
    }
    T t;
    t.run(ldsf, rowsA, rowsB, hd, 0, 0);
#pragma unroll
    for (int j = 0; j < T::TB; ++j) {
        const int r = bt * BB + T::b_of(j);
        if (r >= n_rows) continue;
        float *row = r < n_main ? y + batch_token(r, out_idx, tF, tN) * C : y_ctx + (long)(r - n_main) * C;
#pragma unroll
        for (int i = 0; i < T::TA; ++i) {
            const int a = at * BA + T::a_of(i);
            if (a < C) *reinterpret_cast<f32x4 *>(row + a) = t.acc[i][j];
        }
    }
}

// Attention of fp32 layers on v_mfma_f32_16x16x4_f32: one block per (16
// queries, head, sequence); its waves take every n_waves-th run of 32 keys,
// each with its own running maximum, sum and output (online softmax), merged
// through LDS at the end.  Per run: S^T = K Q^T (K rows are the A operand, 16
// bytes per lane from memory, the queries stay in registers), so a lane holds
// one query and the keys 4 (lane / 16) + e of each 16; P = exp(s - m) is then
// the B operand of O^T += V^T P as it lies, V read by rows.  K and V come
// straight from L2: a small layer has too few queries to share them through
// LDS, and splitting the keys over the waves is what fills the chip (one
// thread per (query, head) over all keys took 8368 us at 512 keys and 5 heads
// of 64, on 20 blocks; this takes 15.1 on 160 blocks of 8 waves).
constexpr int FA_WAVES = 8, FA_KEYS = 32, FA_LD = 20;
template <int NKS>   // 16-element steps of the head dim
__global__ __launch_bounds__(FA_WAVES * 64) void k_attn_f32(const float *__restrict__ Q, const float *__restrict__ K,
                                                            const float *__restrict__ V, float *__restrict__ O,
                                                            int heads, int dh, int n_seq, int L, int Lk, int n_qt,
                                                            float scale,
                                                            const int32_t *__restrict__ seq_off) {
    constexpr int MAXW = NKS <= 4 ? FA_WAVES : FA_WAVES / 2;   // (the launch uses at most these)
    __shared__ float so[MAXW * NKS * 16 * FA_LD];
    __shared__ float sm[MAXW][16], sl[MAXW][16];
    const int id = (int)folded_block(), qt = id % n_qt, hs = id / n_qt, h = hs % heads, s = hs / heads;
    if (s >= n_seq) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int hd = heads * dh;
    long row0 = (long)s * L;
    if (seq_off != nullptr) {
        row0 = seq_off[s];
        Lk = seq_off[s + 1] - seq_off[s];
    }
    if (qt * 16 >= Lk) return;   // (the whole block)
    const int q = qt * 16 + lr;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 qf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        const int d = ks * 16 + lg * 4;
        qf[ks] = q < Lk && d < dh ? *reinterpret_cast<const f32x4 *>(Q + (row0 + q) * hd + h * dh + d) : zero;
    }
    f32x4 o[NKS];
#pragma unroll
    for (int db = 0; db < NKS; ++db) o[db] = zero;
    float m = -INFINITY, l = 0.f;
    for (int k0 = wave * FA_KEYS; k0 < Lk; k0 += n_waves * FA_KEYS) {
        f32x4 kf[2][NKS];
        float vf[2][NKS][4];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int key = k0 + t * 16 + lr;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const int d = ks * 16 + lg * 4;
                kf[t][ks] = key < Lk && d < dh ? *reinterpret_cast<const f32x4 *>(K + (row0 + key) * hd + h * dh + d)
                                               : zero;
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int key = k0 + t * 16 + lg * 4 + j;
#pragma unroll
                for (int db = 0; db < NKS; ++db) {
                    const int d = db * 16 + lr;
                    vf[t][db][j] = key < Lk && d < dh ? V[(row0 + key) * hd + h * dh + d] : 0.f;
                }
            }
        f32x4 sc[2] = {zero, zero};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    sc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][ks][e], qf[ks][e], sc[t], 0, 0, 0);
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[t][e] = k0 + t * 16 + lg * 4 + e < Lk ? sc[t][e] * scale : -INFINITY;
                mx = fmaxf(mx, sc[t][e]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m, mx), al = expf(m - mn);   // (key k0 is valid: mn is a score)
        m = mn;
        l *= al;
#pragma unroll
        for (int db = 0; db < NKS; ++db) o[db] *= al;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[t][e] = expf(sc[t][e] - mn);
                l += sc[t][e];
            }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int db = 0; db < NKS; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][db][j], sc[t][j], o[db], 0, 0, 0);
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    // this wave's part: rows d of 16 queries, padded to keep the four lane groups in different banks
    float *mine = so + wave * NKS * 16 * FA_LD;
#pragma unroll
    for (int db = 0; db < NKS; ++db)
#pragma unroll
        for (int e = 0; e < 4; ++e) mine[(db * 16 + lg * 4 + e) * FA_LD + lr] = o[db][e];
    if (lg == 0) {
        sm[wave][lr] = m;
        sl[wave][lr] = l;
    }
    __syncthreads();
    // merge: thread -> (query, feature), features contiguous over the lanes
    for (int i = threadIdx.x; i < 16 * dh; i += blockDim.x) {
        const int qq = i / dh, d = i - qq * dh;
        if (qt * 16 + qq >= Lk) continue;
        float mm = -INFINITY;
        for (int w = 0; w < n_waves; ++w) mm = fmaxf(mm, sm[w][qq]);
        float num = 0.f, den = 0.f;
        for (int w = 0; w < n_waves; ++w) {
            if (sl[w][qq] == 0.f) continue;   // a wave without keys
            const float f = expf(sm[w][qq] - mm);
            den += f * sl[w][qq];
            num += f * so[(w * NKS * 16 + d) * FA_LD + qq];
        }
        O[(row0 + qt * 16 + qq) * hd + h * dh + d] = num / den;
    }
}

template <typename T, int B>
static hipError_t go_proj_f32(const Plan &p, const AttnArgs &a, const RowMapF &rm, hipStream_t st) {
    const hipError_t e = raise_lds_limit((const void *)k_proj_f32<T, B, B>, T::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int n_at = cdiv(3 * p.hd, B);
    launch_k(k_proj_f32<T, B, B>, (unsigned)(n_at * cdiv(rm.n_rows, B)), 256, T::LDS_BYTES, st, rm,
             (const float *)a.wq, (const float *)a.wk, (const float *)a.wv, p.hd, n_at, (float *)a.q, (float *)a.k,
             (float *)a.vt);
    return hipGetLastError();
}

template <typename T, int B>
static hipError_t go_out_f32(const Plan &p, const AttnArgs &a, int n_rows, hipStream_t st) {
    const hipError_t e = raise_lds_limit((const void *)k_out_f32<T, B, B>, T::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int n_at = cdiv(p.C, B);
    launch_k(k_out_f32<T, B, B>, (unsigned)(n_at * cdiv(n_rows, B)), 256, T::LDS_BYTES, st, (const float *)a.o,
             n_rows, p.hd, (const float *)a.wo, p.C, a.n_main, a.out_idx, a.tF, a.tN, n_at, (float *)a.y,
             (float *)a.y_ctx);
    return hipGetLastError();
}

template <int NKS>
static hipError_t go_attn_f32(const Plan &p, const AttnArgs &a, int Lk, hipStream_t st) {
    // waves: one per 32 keys, up to eight (four for the widest heads, whose parts fill more LDS)
    const int most = NKS <= 4 ? FA_WAVES : FA_WAVES / 2;
    int nw = 1;
    while (nw < most && nw * FA_KEYS < Lk) nw *= 2;
    const int n_qt = cdiv(Lk, 16);
    const long blocks = (long)n_qt * p.heads * a.n_seq;
    if (blocks >= (1L << 31)) return hipErrorInvalidValue;
    launch_k(k_attn_f32<NKS>, folded_grid(blocks, nw * 64), nw * 64, 0, st, (const float *)a.q, (const float *)a.k,
             (const float *)a.vt, (float *)a.o, p.heads, p.dh, a.n_seq, a.L, Lk, n_qt,
             (float)(1.0 / sqrt((double)p.dh)), a.seq_off);
    return hipGetLastError();
}

static hipError_t launch_attn_f32(const Plan &p, const AttnArgs &a, int Lk, hipStream_t st) {
    switch (cdiv(p.dh, 16)) {
        case 1: return go_attn_f32<1>(p, a, Lk, st);
        case 2: return go_attn_f32<2>(p, a, Lk, st);
        case 3: return go_attn_f32<3>(p, a, Lk, st);
        case 4: return go_attn_f32<4>(p, a, Lk, st);
        case 5: return go_attn_f32<5>(p, a, Lk, st);
        case 6: return go_attn_f32<6>(p, a, Lk, st);
        case 7: return go_attn_f32<7>(p, a, Lk, st);
        case 8: return go_attn_f32<8>(p, a, Lk, st);
        default: return hipErrorInvalidValue;
    }
}

AttnWs attn_ws(const Plan &p, int n_seq, int L, size_t base) {
    AttnWs w;
    const long rows = (long)n_seq * L + p.n_ctx;
    const int Lk = L + (n_seq == 1 ? p.n_ctx : 0);
    w.lpad = cdiv(Lk > 0 ? Lk : 1, 64) * 64;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t e = p.esz == 2 ? 2 : 4;   // fp16 intermediates for bf16 layers
    const size_t m = al((size_t)rows * p.hd * e);
    w.q = base;
    w.k = w.q + m;
    w.o = w.k + m;
    w.v = w.o + m;
    // Vt (or, for short sequences, V rows: never more than m)
    const size_t vt = al((size_t)p.heads * n_seq * p.dh * w.lpad * e);
    const size_t vb = p.bf16 ? (vt > m ? vt : m) : m;
    w.wo16 = w.v + vb;
    const size_t wb = p.bf16 ? al((size_t)p.C * p.hd * 2) : 0;
    w.bytes = w.wo16 + wb - base;
    return w;
}

bool attn_head_dim_supported(int dh) {
    switch (dh) {
        case 16: case 32: case 48: case 64: case 72: case 80: case 96: case 128: return true;
        default: return false;
    }
}

hipError_t launch_attention(const Plan &p, const AttnArgs &a, hipStream_t st) {
    const int n_rows = a.seq_off != nullptr ? a.n_main : a.n_seq * a.L + a.n_ctx;
    const int Lk = a.L + (a.n_seq == 1 ? a.n_ctx : 0);
    if (n_rows == 0) return hipSuccess;
    if (p.bf16) {
        const RowMap rm{(const uint16_t *)a.x, a.row_idx, a.n_main, (const uint16_t *)a.ctx, n_rows, p.C, a.tF, a.tN};
        hipError_t e;
        if (qkv_attn_short_applies(p, a)) {
            if ((e = launch_qkv_attn_short(p, rm, a, st)) != hipSuccess) return e;
            return launch_proj_out(p, n_rows, a, st);
        }
        e = launch_proj_qkv(p, rm, a, st);   // (converts wo when no earlier launch has)
        if (e != hipSuccess) return e;
        if ((e = launch_flash(p, a, Lk, st)) != hipSuccess) return e;
        AttnArgs o = a;
        o.wo16_ready = 1;
        return launch_proj_out(p, n_rows, o, st);
    }
    const RowMapF rm{(const float *)a.x, a.row_idx, a.n_main, (const float *)a.ctx, n_rows, p.C, a.tF, a.tN};
    hipError_t e;
    {
        StageScope _stage(st, "proj_f32");
        e = f32_big(3 * p.hd, n_rows, 1) ? go_proj_f32<F32Big, 64>(p, a, rm, st)
                                         : go_proj_f32<F32Small, 32>(p, a, rm, st);
        if (e != hipSuccess) return e;
    }
    {
        StageScope _stage(st, "attn_f32");
        if ((e = launch_attn_f32(p, a, Lk, st)) != hipSuccess) return e;
    }
    StageScope _stage(st, "out_f32");
    return f32_big(p.C, n_rows, 1) ? go_out_f32<F32Big, 64>(p, a, n_rows, st)
                                   : go_out_f32<F32Small, 32>(p, a, n_rows, st);
}

}  // namespace oc
