// Feed-forward sublayer under the attention's selection (the SD3 experiments
// cache attention and FFN layers alike): y[row] = GELU(x[row] W1^T) W2^T for
// the retained rows only, on the ring-buffered MFMA tiles (bf16 operands, fp32
// accumulation; the tile shape by ring_pick).  Bounded by the matrix units'
// rate under load; 2048 rows of C = 1536, hidden 6144, against double-buffered
// 128-wide tiles: the sublayer 128.7 -> 99.0 us (up about 53 -> 47, down 64 ->
// 47, where 96 x 128 tiles are the largest that fill the chip).
//   k_ffn_up:   [rows, C] x [hidden, C]^T -> H [rows, hidden] fp16, the
//               batch rows gathered from x through kept_idx in the operand
//               load (no separate gather), GELU applied in the epilogue;
//               the launch's extra blocks convert W2 to fp16 meanwhile;
//   k_ffn_down: H x [C, hidden]^T (fp16 MFMA) -> y rows (bf16), written
//               straight to their token positions (restoration in place:
//               cached rows are never touched) or to a compact [rows, C]
//               buffer.
// H is fp16 rather than bf16: three more significant bits for the one
// intermediate that every output sums 'hidden' terms of (bf16 measured
// 0.93% of the output RMS at the SD3 shape beyond the output's own rounding).
// GELU is the tanh form, evaluated as v / (1 + exp(-2 z)) with
// z = sqrt(2/pi) (v + 0.044715 v^3), which equals 0.5 v (1 + tanh z).
#include "oc_gemm_epi.h"
#include "oc_attn_common.h"
#include "oc_ring_tile.h"

namespace oc {

namespace {

__device__ __forceinline__ float gelu_tanh_f(float v) {
    const float z = 0.7978845608028654f * fmaf(0.044715f * v, v * v, v);
    // (exp and reciprocal to 1 ulp of fp32; H is stored in fp16, and its error
    // against 64 bits is that rounding's, 2.08e-4 of the 2-norm, as with a
    // correctly rounded division: 2.0821e-4 either way at C = 1536)
    return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-2.8853900817779268f * z));
}

// Batch rows r0 + row of x through idx; a row past the batch or with an index
// outside [0, FN) reads some row of x: its results are never stored
template <int N, int NW>
__device__ __forceinline__ void ring_ffn_rows(RingRows<N, NW> &w, const uint16_t *x, const int32_t *idx, int n_rows,
                                              int FN, int C, int r0) {
    w.base2 = x;
    w.mix = w.alt = 0;
    int tok[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int r = min(r0 + w.row(i), n_rows - 1);
        tok[i] = idx != nullptr ? idx[r] : r;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        w.base[i] = x;
        w.off[i] = (uint32_t)min(max(tok[i], 0), FN - 1) * (uint32_t)(C * 2) + (uint32_t)w.chunk() * 16;
    }
}

// up: a = rows of w1 (hidden), b = batch rows
template <int ID>
__global__ __launch_bounds__(RING_THREADS<ID>) void k_ffn_up(const uint16_t *__restrict__ x,
                                                const int32_t *__restrict__ idx,
                                                int n_rows, int FN, int C, const uint16_t *__restrict__ w1,
                                                int hidden, int n_at, int n_bt, uint16_t *__restrict__ H,
                                                const uint4 *__restrict__ w2, long n8, uint4 *__restrict__ w2h) {
    using T = typename RingShape<ID, false>::Tile;
    constexpr int BA = T::BA, BB = T::BB;
    extern __shared__ __align__(16) uint16_t lds[];
    const int n_tiles = n_at * n_bt;
    if ((int)blockIdx.x >= n_tiles) {
        // W2 -> fp16 for the down-projection, 8 elements per thread, four loads in flight
        const long step = (long)(gridDim.x - n_tiles) * T::NT;
        for (long i = (long)(blockIdx.x - n_tiles) * T::NT + threadIdx.x; i < n8; i += 4 * step) {
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = w2[min(i + u * step, n8 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u * step < n8) w2h[i + u * step] = bf16x8_to_f16x8(v[u]);
        }
        return;
    }
    int at, bt;
    tile_order(xcd_remap(blockIdx.x, n_tiles), n_at, n_bt, at, bt);
    const int a0 = at * BA, b0 = bt * BB;
    typename T::RowsA ra;
    typename T::RowsB rb;
    ring_rows(ra, w1, hidden, C, a0);
    ring_ffn_rows(rb, x, idx, n_rows, FN, C, b0);
    T t;
    t.run(lds, ra, rb, C);
    stage_rows<BA>(t, lds, [](float v, int) { return f2h_bits(gelu_tanh_f(v)); }, [](int a) { return a; });
    __syncthreads();
    write_rows<BA, BB, T::NT>(lds, min(BA, hidden - a0), [&](int b, int c0) -> uint16_t * {
        const int r = b0 + b;
        return r < n_rows ? H + (long)r * hidden + a0 + c0 : nullptr;
    });
}

// down: a = rows of w2 (fp16, C), b = rows of H; row r goes to y row idx[r]
// (scatter) or r, and nowhere when its token index was outside [0, FN)
template <int ID>
__global__ __launch_bounds__(RING_THREADS<ID>) void k_ffn_down(const uint16_t *__restrict__ H, int n_rows, int hidden,
                                                  const uint16_t *__restrict__ w2, int C,
                                                  const int32_t *__restrict__ idx, int scatter, int FN, int n_at,
                                                  int n_bt, uint16_t *__restrict__ y) {
    using T = typename RingShape<ID, true>::Tile;
    constexpr int BA = T::BA, BB = T::BB;
    extern __shared__ __align__(16) uint16_t lds[];
    int at, bt;
    tile_order(xcd_remap(blockIdx.x, n_at * n_bt), n_at, n_bt, at, bt);
    const int a0 = at * BA, b0 = bt * BB;
    typename T::RowsA ra;
    typename T::RowsB rb;
    ring_rows(ra, w2, C, hidden, a0);
    ring_rows(rb, H, n_rows, hidden, b0);
    T t;
    t.run(lds, ra, rb, hidden);
    stage_rows<BA>(t, lds, [](float v, int) { return f2bf(v); }, [](int a) { return a; });
    __syncthreads();
    write_rows<BA, BB, T::NT>(lds, min(BA, C - a0), [&](int b, int c0) -> uint16_t * {
        const int r = b0 + b;
        if (r >= n_rows) return nullptr;
        const long tok = idx != nullptr ? (long)idx[r] : (long)r;
        if (tok < 0 || tok >= FN) return nullptr;          // the row was never read
        return y + (scatter ? tok : (long)r) * C + a0 + c0;
    });
}

}  // namespace

size_t ffn_h_bytes(int n_rows, int hidden) { return ((size_t)n_rows * hidden * 2 + 255) & ~(size_t)255; }
size_t ffn_workspace_bytes(int n_rows, int hidden, int C) {
    if (n_rows == 0) return 0;   // nothing is launched
    return ffn_h_bytes(n_rows, hidden) + (((size_t)C * hidden * 2 + 255) & ~(size_t)255);
}

hipError_t launch_ffn(const FfnArgs &a, hipStream_t st) {
    if (a.n_rows == 0) return hipSuccess;
    if (a.C % 64 || a.hidden % 64) return hipErrorInvalidValue;
    uint16_t *h = (uint16_t *)a.h;
    uint16_t *w2h = (uint16_t *)((char *)a.h + ffn_h_bytes(a.n_rows, a.hidden));
    const long n8 = (long)a.C * a.hidden / 8;
    {
        StageScope _stage(st, "ffn_up");
        const int id = ring_pick(a.C, [&](int BA, int BB) { return (long)cdiv(a.hidden, BA) * cdiv(a.n_rows, BB); });
        const hipError_t e = ring_dispatch(id, [&](auto c) -> hipError_t {
            constexpr int ID = decltype(c)::value;
            using T = typename RingShape<ID, false>::Tile;
            const hipError_t el = allow_lds(k_ffn_up<ID>, T::LDS_BYTES);
            if (el != hipSuccess) return el;
            const int n_at = cdiv(a.hidden, T::BA), n_bt = cdiv(a.n_rows, T::BB);
            const int cvt_blocks = (int)std::min<long>((n8 + T::NT - 1) / T::NT, 256);
            launch_k(k_ffn_up<ID>, (unsigned)(n_at * n_bt + cvt_blocks), T::NT, T::LDS_BYTES, st,
                     (const uint16_t *)a.x, a.idx, a.n_rows, a.FN, a.C, (const uint16_t *)a.w1, a.hidden, n_at, n_bt, h,
                     (const uint4 *)a.w2, n8, (uint4 *)w2h);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
    }
    StageScope _stage(st, "ffn_down");
    const int id = ring_pick(a.hidden, [&](int BA, int BB) { return (long)cdiv(a.C, BA) * cdiv(a.n_rows, BB); });
    return ring_dispatch(id, [&](auto c) -> hipError_t {
        constexpr int ID = decltype(c)::value;
        using T = typename RingShape<ID, true>::Tile;
        const hipError_t e = allow_lds(k_ffn_down<ID>, T::LDS_BYTES);
        if (e != hipSuccess) return e;
        const int n_at = cdiv(a.C, T::BA), n_bt = cdiv(a.n_rows, T::BB);
        launch_k(k_ffn_down<ID>, (unsigned)(n_at * n_bt), T::NT, T::LDS_BYTES, st, h, a.n_rows, a.hidden, w2h, a.C,
                 a.idx, a.scatter, a.FN, n_at, n_bt, (uint16_t *)a.y);
        return hipGetLastError();
    });
}

}  // namespace oc
