// Attention for grids that cannot fill the chip: few queries and heads over
// long sequences (one head of 2640 keys is 83 tiles of 32 queries for 1024
// SIMDs).  The long-sequence kernel gives every wave 32 queries and walks all
// keys with it, so such a call takes as long as one wave needs for the whole
// sequence.  Here a block holds one tile of 32 queries and its waves share
// out the key tiles, each with its own running maximum, sum and output; the
// parts are merged through LDS at the end.
//
// A wave stages its own tiles of 32 keys: the global loads of the next tile
// (whole rows: 8 cache lines per instruction) travel in registers while the
// current one is computed from the wave's own LDS area, so no barrier is
// needed before the merge.  (Fragments read straight from memory, 32 rows of
// 32 bytes per instruction, were bound by the address path: 32 us for
// one head of 4096 keys of 64, 21 us this way.)
//
// Layouts, precision and the log2 domain are those of k_flash.hip: fp16
// operands, fp32 accumulation, P = exp2(s - m) rounded to fp16 for both the
// product and the running sum; m is the running maximum itself.
#include "oc_attn_common.h"
#include "oc_launch.h"
#include "oc_mfma_tile.h"
#include <algorithm>

namespace oc {

namespace {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

template <int DH>
struct SplitCfg {
    static constexpr int NKS = (DH + 15) / 16, DV = (DH + 31) / 32 * 32, NDB = DV / 32, KT = 32;
    // K rows (features, zero-padded to 16) and V rows (32 keys) of an odd
    // number of 16-byte chunks: fragment reads of 16 rows hit distinct banks
    static constexpr int LDK = NKS * 16 + 8, LDV = KT + 8;
    static constexpr int KCPR = NKS * 2;                       // 16-byte chunks of a K row
    static constexpr int IK = (KT * KCPR + 63) / 64, IV = (DH * 4 + 63) / 64;   // loads per lane and tile
    static constexpr int WAVE_HALVES = KT * LDK + DV * LDV;
    static constexpr int LDO = DV + 4;   // floats per query of a wave's part (16 rows in 16 different bank groups)
    static constexpr size_t lds(int waves) {
        const size_t stage = (size_t)waves * WAVE_HALVES * 2, merge = (size_t)waves * 32 * (LDO + 2) * 4;
        return stage > merge ? stage : merge;
    }
};

}  // namespace

constexpr int SPLIT_WAVES = 8;

template <int DH, bool VARLEN>
__global__ __launch_bounds__(SPLIT_WAVES * 64) void k_flash_split(const uint16_t *__restrict__ Q,
                                                                  const uint16_t *__restrict__ K,
                                                                  const uint16_t *__restrict__ Vt,
                                                                  uint16_t *__restrict__ O, int hd, int heads,
                                                                  int n_seq, int L, int Lk, int lpad, int n_qt,
                                                                  const int32_t *__restrict__ seq_off) {
    using C = SplitCfg<DH>;
    constexpr int NKS = C::NKS, NDB = C::NDB, KT = C::KT, LDK = C::LDK, LDV = C::LDV, LDO = C::LDO;
    constexpr int IK = C::IK, IV = C::IV;
    extern __shared__ __align__(16) float part[];
    const int n_waves = blockDim.x >> 6;
    float *const sm = part + n_waves * 32 * LDO, *const sl = sm + n_waves * 32;

    const int lid = xcd_remap(blockIdx.x, n_qt * heads * n_seq);
    const int qt = lid % n_qt, hs = lid / n_qt, h = hs % heads, s = hs / heads;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ln = lane & 31, lg = lane >> 5;
    long row0 = (long)s * L;
    if constexpr (VARLEN) {
        row0 = seq_off[s];
        Lk = seq_off[s + 1] - seq_off[s];
        if (qt * 32 >= Lk) return;   // (the whole block)
    }
    const uint16_t *kbase = K + row0 * hd + h * DH;
    const uint16_t *vbase = Vt + ((long)h * n_seq + s) * DH * lpad;
    auto ld = [](const uint16_t *p, bool ok) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (ok) v = *reinterpret_cast<const uint4 *>(p);
        return __builtin_bit_cast(f16x8, v);
    };
    f16x8 qf[NKS];
    {
        const int q = qt * 32 + ln;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            const int d0 = ks * 16 + lg * 8;
            qf[ks] = ld(Q + (row0 + q) * hd + h * DH + d0, q < Lk && d0 < DH);
        }
    }
    uint16_t *const Ks = reinterpret_cast<uint16_t *>(part) + wave * C::WAVE_HALVES, *const Vs = Ks + KT * LDK;
    // this lane's chunks of a tile: K (key, 8 features; zero past the head
    // dim) and Vt (feature, 8 key positions; the rows past the head dim only
    // feed outputs that are not stored, and stay as they are)
    // (K chunk i of a lane: rows RS apart where a row's chunks divide 64,
    // so that the offsets of all chunks follow from the first)
    constexpr bool LIN = 64 % C::KCPR == 0;
    constexpr int RS = LIN ? 64 / C::KCPR : 1, NO = LIN ? 1 : IK;
    int kkey0[NO], koff0[NO], klds0[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const int u = lane + 64 * i, r = u / C::KCPR, c = u % C::KCPR;
        kkey0[i] = c < DH / 8 ? r : 0x40000000;   // (no key)
        koff0[i] = r * hd + c * 8;
        klds0[i] = r < KT ? r * LDK + c * 8 : -1;
    }
    auto kkey = [&](int i) { return LIN ? kkey0[0] + i * RS : kkey0[LIN ? 0 : i]; };
    auto koff = [&](int i) { return LIN ? koff0[0] + i * RS * hd : koff0[LIN ? 0 : i]; };
    auto klds = [&](int i) { return LIN ? klds0[0] + i * RS * LDK : klds0[LIN ? 0 : i]; };
    const int vpos = (lane & 3) * 8, voff0 = (lane >> 2) * lpad + vpos, vlds0 = (lane >> 2) * LDV + vpos;
    auto vrow = [&](int i) { return DH % 16 == 0 || (lane >> 2) + 16 * i < DH; };
    uint4 kr[IK], vr[IV];
    auto load = [&](int k0) {
        const uint16_t *kp = kbase + (long)k0 * hd, *vp = vbase + k0;
#pragma unroll
        for (int i = 0; i < IK; ++i) {
            kr[i] = make_uint4(0, 0, 0, 0);
            if (klds(i) >= 0 && k0 + kkey(i) < Lk) kr[i] = *reinterpret_cast<const uint4 *>(kp + koff(i));
        }
        // (Vt rows are lpad positions long, lpad a multiple of 64: the whole tile is inside)
#pragma unroll
        for (int i = 0; i < IV; ++i) {
            vr[i] = make_uint4(0, 0, 0, 0);
            if (vrow(i)) vr[i] = *reinterpret_cast<const uint4 *>(vp + (voff0 + i * 16 * lpad));
        }
    };
    auto store = [&](int k0) {
#pragma unroll
        for (int i = 0; i < IK; ++i)
            if (klds(i) >= 0) *reinterpret_cast<uint4 *>(Ks + klds(i)) = kr[i];
#pragma unroll
        for (int i = 0; i < IV; ++i) {
            if (!vrow(i)) continue;
            // the projection zeroes the padded key positions, except for
            // sequences of varying length, which are masked here
            if (VARLEN && k0 + KT > Lk) {
                uint16_t e[8];
                *reinterpret_cast<uint4 *>(e) = vr[i];
                const int blk = vpos & ~15, p0 = vpos & 15;
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (k0 + blk + vt_key_of_pos(p0 + t) >= Lk) e[t] = 0;
                vr[i] = *reinterpret_cast<const uint4 *>(e);
            }
            *reinterpret_cast<uint4 *>(Vs + vlds0 + i * 16 * LDV) = vr[i];
        }
    };
    const f16x2 ones = {(_Float16)1.f, (_Float16)1.f};
    f32x16 o[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] = f32x16{};
    float m = -INFINITY, l0 = 0.f, l1 = 0.f;
    const int step = n_waves * KT;
    int k0 = wave * KT;
    if (k0 < Lk) load(k0);
    for (; k0 < Lk; k0 += step) {
        // (the previous tile's fragments have been consumed: its last MFMA waited for them)
        __builtin_amdgcn_wave_barrier();
        store(k0);
        if (k0 + step < Lk) load(k0 + step);
        __builtin_amdgcn_wave_barrier();
        f32x16 sc = f32x16{};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            sc = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                *reinterpret_cast<const f16x8 *>(Ks + ln * LDK + (ks * 2 + lg) * 8), qf[ks], sc, 0, 0, 0);
        f16x8 vf[NDB][2];
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
                vf[db][k2] = *reinterpret_cast<const f16x8 *>(Vs + (db * 32 + ln) * LDV + (k2 * 2 + lg) * 8);
        if (k0 + KT > Lk) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (k0 + 8 * (i >> 2) + 4 * lg + (i & 3) >= Lk) sc[i] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
            // (key k0 is valid, so the maximum is a score)
            const float mn = fmaxf(m, mx), al = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l0 *= al;
            l1 *= al;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= al;
        }
        f16x8 pf[2];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            f16x8 f;
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = (_Float16)__builtin_amdgcn_exp2f(sc[8 * hf + e] - m);
            pf[hf] = f;
            l0 = __builtin_amdgcn_fdot2(f.s01, ones, l0, false);
            l1 = __builtin_amdgcn_fdot2(f.s23, ones, l1, false);
            l0 = __builtin_amdgcn_fdot2(f.s45, ones, l0, false);
            l1 = __builtin_amdgcn_fdot2(f.s67, ones, l1, false);
        }
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[db][k2], pf[k2], o[db], 0, 0, 0);
    }
    __syncthreads();   // the parts reuse the staging areas
    // this wave's part: lane holds query ln, d = db*32 + 8*g4 + 4*lg + e
    float lt = l0 + l1;
    lt += __shfl_xor(lt, 32, 64);
    if (lg == 0) {
        sm[wave * 32 + ln] = m;
        sl[wave * 32 + ln] = lt;
    }
    float *mine = part + (wave * 32 + ln) * LDO;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4 v = {o[db][4 * g4], o[db][4 * g4 + 1], o[db][4 * g4 + 2], o[db][4 * g4 + 3]};
            *reinterpret_cast<f32x4 *>(mine + db * 32 + 8 * g4 + 4 * lg) = v;
        }
    __syncthreads();
    // merge: thread -> (query, 8 features)
    constexpr int CPQ = DH / 8;
    for (int i = threadIdx.x; i < 32 * CPQ; i += blockDim.x) {
        const int qq = i / CPQ, c = (i - qq * CPQ) * 8, q = qt * 32 + qq;
        if (q >= Lk) continue;
        float mm = sm[qq];   // (wave 0 always has a key tile)
        for (int w = 1; w < n_waves; ++w) mm = fmaxf(mm, sm[w * 32 + qq]);
        float den = 0.f, num[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) num[e] = 0.f;
        for (int w = 0; w < n_waves; ++w) {
            const float lw = sl[w * 32 + qq];
            if (lw == 0.f) continue;   // a wave without keys
            const float f = __builtin_amdgcn_exp2f(sm[w * 32 + qq] - mm);
            den += f * lw;
            const float *pw = part + (w * 32 + qq) * LDO + c;
#pragma unroll
            for (int e = 0; e < 8; ++e) num[e] += f * pw[e];
        }
        const float inv = 1.f / den;
        uint16_t r[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = f2h_bits(num[e] * inv);
        *reinterpret_cast<uint4 *>(O + (row0 + q) * hd + h * DH + c) = *reinterpret_cast<const uint4 *>(r);
    }
}

template <int DH, bool VARLEN>
static hipError_t go_split(const Plan &p, const AttnArgs &a, int Lk, hipStream_t st) {
    using C = SplitCfg<DH>;
    const int nw = std::min(SPLIT_WAVES, cdiv(Lk, C::KT)), n_qt = cdiv(Lk, 32);
    const size_t lds = C::lds(nw);
    const hipError_t e = raise_lds_limit((const void *)k_flash_split<DH, VARLEN>, C::lds(SPLIT_WAVES));
    if (e != hipSuccess) return e;
    launch_k(k_flash_split<DH, VARLEN>, n_qt * p.heads * a.n_seq, nw * 64, lds, st, (const uint16_t *)a.q,
             (const uint16_t *)a.k, (const uint16_t *)a.vt, (uint16_t *)a.o, p.hd, p.heads, a.n_seq, a.L, Lk, a.lpad,
             n_qt, a.seq_off);
    return hipGetLastError();
}

template <int DH>
static hipError_t go_len(const Plan &p, const AttnArgs &a, int Lk, hipStream_t st) {
    return a.seq_off != nullptr ? go_split<DH, true>(p, a, Lk, st) : go_split<DH, false>(p, a, Lk, st);
}

// Where the keys are split: by the number T of 32-query tiles, one block of
// eight waves per compute unit.  Measured both ways over head dims 32-128, 100
// to 4096 keys and T = 4 to 2000 (µs, walking all keys / split): T <= 256 wins
// throughout, more so the longer the sequence (dh 64: 256 keys 10.5 / 6.3, 1024
// 20.6 / 10.8, 4096 63.9 / 23.2).  T <= 512, two rounds of blocks, still wins
// up to head dim 64 (dh 64: 256 keys 10.0 / 9.5, 1024 20.7 / 17.5, 4096 66.2 /
// 42.6) and for wide heads over 1024 keys or more (dh 128: 1024 33.7 / 32.7;
// but dh 96 at 256 keys 11.8 / 13.9).  T <= 768 wins for head dims up to 32 and
// 1024 keys or more (dh 32: 1024 17.7 / 17.2, 4096 54.4 / 38.5; 256 8.5 / 9.3).
bool flash_splits(const Plan &p, const AttnArgs &a, int Lk) {
    if (a.seq_off == nullptr && attn_short(Lk)) return false;   // (one wave holds the whole sequence)
    const long T = (long)cdiv(Lk, 32) * p.heads * a.n_seq;
    if (T <= N_CUS) return true;
    if (T <= 2 * N_CUS) return p.dh <= 64 || Lk >= 1024;
    return T <= 3 * N_CUS && p.dh <= 32 && Lk >= 1024;
}

hipError_t launch_flash_split(const Plan &p, const AttnArgs &a, int Lk, hipStream_t st) {
    switch (p.dh) {
        case 16: return go_len<16>(p, a, Lk, st);
        case 32: return go_len<32>(p, a, Lk, st);
        case 48: return go_len<48>(p, a, Lk, st);
        case 64: return go_len<64>(p, a, Lk, st);
        case 72: return go_len<72>(p, a, Lk, st);
        case 80: return go_len<80>(p, a, Lk, st);
        case 96: return go_len<96>(p, a, Lk, st);
        case 128: return go_len<128>(p, a, Lk, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace oc
