// fp32 tile engine for gfx950: C[b][a] = sum_k A[a][k] * B[b][k] in fp32 on
// v_mfma_f32_16x16x4_f32 (full fp32 products and sums, twice the rate of
// scalar fp32 FMAs), operands K-contiguous rows, for the layers kept in fp32.
//
// 256 threads = 4 waves arranged 2 x 2 over a BA x BB tile.  K is walked in
// chunks of KC through two LDS buffers, one barrier per chunk; the next
// chunk's global loads (16 bytes per thread and load) are in flight during
// the MFMAs of the current one.  An fp32 layer is small (a 32 x 32 grid of
// C = 320 is 0.9 GFLOP), so latency bounds it: chunks are long (few
// barriers), and the 32 x 32 tile is taken until 64 x 64 ones fill the chip.
//
// Operand layout (16x16x4): lane l feeds row (or column) l % 16 and k = l /
// 16.  The contraction order is free, so lane group g = l / 16 reads the four
// consecutive k of chunk 16 s + 4 g with one 16-byte LDS read and MFMA j of
// the step takes element j of it from both operands.  Rows are padded by 16
// bytes: the 16 rows of one lane group then start in 16 different 16-byte
// columns of the banks.  The result lane holds column b = l % 16 and rows a =
// 4 (l / 16) + e.
#pragma once
#include "oc_device.h"

namespace oc {

template <int BA, int BB, int KC>
struct F32Tile {
    static constexpr int LD = KC + 4;
    static constexpr int WTA = BA / 2, WTB = BB / 2, TA = WTA / 16, TB = WTB / 16;
    static constexpr int CPR = KC / 4;                       // 16-byte chunks per row
    static constexpr int NA = BA * CPR / 256, NB = BB * CPR / 256;
    static constexpr int BUF = (BA + BB) * LD;               // floats per buffer
    static constexpr size_t LDS_BYTES = (size_t)2 * BUF * 4;
    static_assert(NA >= 1 && NB >= 1 && KC % 16 == 0, "tile too small for 256 threads");

    f32x4 acc[TA][TB];

    // row of the tile that load i of this thread belongs to
    __device__ __forceinline__ static int load_row(int i) { return (threadIdx.x + 256 * i) / CPR; }
    __device__ __forceinline__ static int a_of(int i) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        return (wave >> 1) * WTA + i * 16 + 4 * (lane >> 4);
    }
    __device__ __forceinline__ static int b_of(int j) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        return (wave & 1) * WTB + j * 16 + (lane & 15);
    }

    // This thread's chunks of the K chunk at k0 (zero for a null row and past
    // K, a multiple of 4); rows are segments as in the 16-bit engines.
    template <int N>
    __device__ __forceinline__ static void load(const float *const *rows, int k0, int K, int seg_len, long sub_stride,
                                                float4 *v) {
        const int k = k0 + (threadIdx.x % CPR) * 4;
        long off = k;
        if (seg_len > 0) {
            const int s = k / seg_len;
            off = (long)s * sub_stride + (k - s * seg_len);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (rows[i] != nullptr && k < K) v[i] = *reinterpret_cast<const float4 *>(rows[i] + off);
        }
    }
    template <int N>
    __device__ __forceinline__ static void store(float *lds, const float4 *v) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            *reinterpret_cast<float4 *>(lds + load_row(i) * LD + (threadIdx.x % CPR) * 4) = v[i];
    }
    __device__ __forceinline__ void compute(const float *buf) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
        const float *As = buf + ((wave >> 1) * WTA + lr) * LD + lg * 4;
        const float *Bs = buf + (BA + (wave & 1) * WTB + lr) * LD + lg * 4;
#pragma unroll
        for (int ks = 0; ks < KC; ks += 16) {
            f32x4 a[TA], b[TB];
#pragma unroll
            for (int i = 0; i < TA; ++i) a[i] = *reinterpret_cast<const f32x4 *>(As + i * 16 * LD + ks);
#pragma unroll
            for (int j = 0; j < TB; ++j) b[j] = *reinterpret_cast<const f32x4 *>(Bs + j * 16 * LD + ks);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TA; ++i)
#pragma unroll
                    for (int j = 0; j < TB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
        }
    }
    __device__ __forceinline__ void run(float *lds, const float *const *rowsA, const float *const *rowsB, int K,
                                        int seg_len, long sub_stride) {
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        float4 va[NA], vb[NB];
        const int nk = cdiv(K, KC);
        auto fetch = [&](int kt) {
            load<NA>(rowsA, kt * KC, K, seg_len, sub_stride, va);
            load<NB>(rowsB, kt * KC, K, seg_len, sub_stride, vb);
        };
        auto put = [&](int kt) {
            float *b = lds + (kt & 1) * BUF;
            store<NA>(b, va);
            store<NB>(b + BA * LD, vb);
        };
        fetch(0);
        put(0);
        if (nk > 1) fetch(1);
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            compute(lds + (kt & 1) * BUF);
            // the other buffer was last read before the barrier that ended step kt-1
            if (kt + 1 < nk) put(kt + 1);
            if (kt + 2 < nk) fetch(kt + 2);
            __syncthreads();
        }
    }
};

// 64 x 64 tiles once they give every compute unit one, else 32 x 32
using F32Big = F32Tile<64, 64, 64>;
using F32Small = F32Tile<32, 32, 128>;
inline bool f32_big(long n_a, long n_b, long batch) { return ((n_a + 63) / 64) * ((n_b + 63) / 64) * batch >= 256; }

}  // namespace oc
