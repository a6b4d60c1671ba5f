// attn_f32.hip -- split-KV partial attention on matrix cores in fp32 (gfx950).
//
// Serves head_dim 64 (bf16 or fp8 K/V with bf16 queries) and fp32 K/V (head_dim
// 64 and 128, fp32 or bf16 queries).  Probabilities, values and accumulators
// keep their fp32 values: fp32 K/V run both products on v_mfma_f32_16x16x4_f32;
// bf16 and fp8 keys meet bf16 queries on v_mfma_f32_16x16x32_bf16, whose
// products are exact and whose sums are fp32.
//
// One wave is one worker of the stream-K partition (spire_internal.h), which
// the kernel computes itself; a unit is a KV head x up to 16 NB rows.  Per tile
// of 16 KG keys (lane l, n16 = l & 15, j = l >> 4):
//   * S^T = K Q^T, A = K: lane l holds 16-byte chunks of key 16g + n16 (chunk c
//     covers bytes 64c + 16j), so a load instruction reads 64 bytes of 16 rows;
//     the reduction index may be any permutation of the head dims as long as Q
//     is laid out alike, so no shuffles.  C: lane l holds keys 16g + 4j + i,
//     row n16.
//   * O^T += V^T P^T, one product per i: its 4 reduction indices are the keys
//     16g + 4j + i, one per lane group, so the B operand is the probability the
//     lane already holds and the A operand is the value element of key
//     16g + 4j + i the lane loaded: each V load reads 4 whole rows, and nothing
//     is transposed.
// 16- and 8-bit values instead take every probability as three bf16 terms whose
// sum is the fp32 value exactly (split3) on v_mfma_f32_16x16x32_bf16: the fp32
// instruction needs 1024 matrix-core cycles per 16 rows and 32 keys of 64 dims,
// the three bf16 products 192, and the sums stay fp32.  There the value operands
// are transposed in registers (8 keys x 4 dims, byte permutes).
//
// Bound by HBM up to five row blocks of 16-/8-bit keys and two of fp32 keys.
// Measured on MI355X, 64 sequences of log-uniform 512-8192 keys, 8 KV heads,
// 20 rows (k = 4, 4 queries per KV head), head_dim 64, paged bf16 (0.37 GB):
// 2.88 ms on the generic vector kernel, 90 us with fp32 products, 70 us with the
// split (5.2 TB/s, of which the start of the launch is 6-8 us); fp32 K/V at
// head_dim 128, 512-2048 keys (0.58 GB): 120 us.
#include <type_traits>

#include "mfma_common.h"

namespace spire {

// words of a lane's share of one V row (D * ES / 16 bytes)
template <int ES, int D, int KG> struct Tile32 {
    static constexpr int NKC = D * ES / 64;  // 16-byte K chunks per lane and key
    static constexpr int VW = D * ES / 64;   // 32-bit V words per lane and key
    u32x4 k[KG][NKC];
    uint32_t v[KG][4][VW];
};

template <int W> __device__ __forceinline__ void ld_words(uint32_t (&d)[W], const uint8_t *p) {
    if constexpr (W == 1) {
        d[0] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p));
    } else if constexpr (W == 2) {
        const u32x2 v = ld8(p);
        d[0] = v.x; d[1] = v.y;
    } else {
        // 8 words: dims 4 n16 .. +3 of each half row, so that 16 lanes read 256 contiguous bytes
#pragma unroll
        for (int h = 0; h < W / 4; ++h) {
            const u32x4 v = ld16(p + 256 * h);
            d[4 * h] = v.x; d[4 * h + 1] = v.y; d[4 * h + 2] = v.z; d[4 * h + 3] = v.w;
        }
    }
}

template <int ES, int D, int KG, int MODE, bool KNT = true>
__device__ __forceinline__ void load_tile32(Tile32<ES, D, KG> &T, const SegAddr &a, int tile, int lane) {
    using TT = Tile32<ES, D, KG>;
    const int n16 = lane & 15, j = lane >> 4;
    const int key0 = tile * 16 * KG;
    constexpr int VB = TT::VW >= 4 ? 16 : 4 * TT::VW;  // bytes between lanes
#pragma unroll
    for (int g = 0; g < KG; ++g) {
        const int64_t base = group_base<MODE>(a, key0 + 16 * g);
        if (MODE == MODE_PAGED || base >= 0) {  // one contiguous run of 16 rows
            const uint32_t tb = (uint32_t)a.tok_bytes;
            const uint8_t *kp = a.kseq + base + (uint32_t)(n16 * tb + 16 * j);
#pragma unroll
            for (int c = 0; c < TT::NKC; ++c) T.k[g][c] = ld16k<KNT>(kp + 64 * c);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                ld_words(T.v[g][i], a.vseq + base + (uint32_t)((4 * j + i) * tb + VB * n16));
            continue;
        }
        // per-lane rows: contiguous tails past the capacity, ring wrap, sinks
        const int kk = key0 + 16 * g + n16;
        const uint8_t *kp = MODE == MODE_DRAFT ? draft_row(a, kk, false)
                                               : a.kseq + (int64_t)min(kk, a.cap - 1) * a.tok_bytes;
#pragma unroll
        for (int c = 0; c < TT::NKC; ++c) T.k[g][c] = ld16k<KNT>(kp + 16 * j + 64 * c);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int vk = key0 + 16 * g + 4 * j + i;
            const uint8_t *vp = MODE == MODE_DRAFT ? draft_row(a, vk, true)
                                                   : a.vseq + (int64_t)min(vk, a.cap - 1) * a.tok_bytes;
            ld_words(T.v[g][i], vp + VB * n16);
        }
    }
}

// the D/16 value elements a lane holds of one key, as fp32
template <int ES, int D> __device__ __forceinline__ void value_f32(const uint32_t (&w)[D * ES / 64], float (&v)[D / 16]) {
#pragma unroll
    for (int x = 0; x < D * ES / 64; ++x) {
        if constexpr (ES == 4) {
            v[x] = __uint_as_float(w[x]);
        } else if constexpr (ES == 2) {
            v[2 * x] = __uint_as_float(w[x] << 16);
            v[2 * x + 1] = __uint_as_float(w[x] & 0xFFFF0000u);
        } else {
            const auto lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[x], 1.0f, false);
            const auto hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[x], 1.0f, true);
            v[4 * x] = lo[0]; v[4 * x + 1] = lo[1]; v[4 * x + 2] = hi[0]; v[4 * x + 3] = hi[1];
        }
    }
}

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Wait until the matrix results x can be read by vector instructions.  A
// v_mfma_f32_16x16x4_f32 takes 8 passes and nothing but independent instructions
// keeps a reader from seeing sums that lack the last products: 10 wait states,
// which the compiler counts and fills.  Where the reader follows a short branch
// around a few instructions (the mask of a range's last tile, the end of a range), it
// takes the count along the branch for the direct way as well and inserts nothing:
// the row maxima were then taken from partial dot products, and a reference off by
// more than 126 (scores of hundreds) lost its row's tile.  The 4-pass bf16
// instruction needs 8, which every way here has.  tests/test_matrix_waits.py counts
// the wait states of every way in the built library.
template <int N> __device__ __forceinline__ void settle(f32x4 (&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));  // issued before the wait ...
    asm volatile("s_nop 9");
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));  // ... and read after it
}
template <int M, int N> __device__ __forceinline__ void settle(f32x4 (&x)[M][N]) {
    settle(reinterpret_cast<f32x4(&)[M * N]>(x));
}

// Query fragments of NB row blocks: bf16 MFMA operands (16-bit keys) or the
// fp32 elements matching the lane's key chunks.
template <int ES, int D, int NB> struct Q32 {
    static constexpr int N = ES == 4 ? D / 16 : D / 32;
    u32x4 r[NB][N];
};

template <int D, int NB> struct State32 {
    f32x4 acc[D / 16][NB];
    float l[NB], msub[NB], thr[NB];
    int lim[NB];
    // what a range calls for the careful form by (needs_care)
    float top;           // infinite: a reference of kFastReference or more; 32-bit values: the largest magnitude
    f16x2 vmax, vmin;    // 16-bit values, both halves of their words
};

// Two forms of the softmax.  The fast one (lazy_softmax) takes the exact product
// s * sc less a rounded reference, so the probability at the maximum is 2^(rounding
// error of the reference): near 1 below 2^20 (half an ulp is 2^-5), 0 or infinite
// from 2^31 on.  Its reference lags the maximum, so that sums of values near the end
// of the range overflow; a probability below 2^-126 is dropped, which such a value
// would make up for; and an infinite value times a zero lower term of its probability
// is NaN where the product with the whole probability is infinite.  A range with a
// reference of 2^20 or more, or a value of 2^65 or more (infinities and NaN
// included), is therefore computed again by the careful form.
// The values are looked at in half an instruction per 32-bit word, and in one per
// word of two 16-bit ones: as fp16 patterns, whose order is that of the bits, so
// that 2^65 is 512 and what is NaN there is larger still (the maximum and minimum
// keep NaN).  64 sequences, 20 rows, us a call in a graph without and with both
// checks: bf16 73.4 / 73.9, fp8 60.2 / 60.6, fp32 head_dim 64 75.3 / 77.8, 128
// 128.9 / 132.3.
constexpr float kFastReference = 0x1p20f, kFastValue = 0x1p65f;
template <int ES, int D, int NB, int N>
__device__ __forceinline__ void note_values(State32<D, NB> &st, const uint32_t (&w)[N]) {
    static_assert(N % 2 == 0 || ES == 1, "words in pairs");
    if constexpr (ES == 1) return;  // 448 at most
#pragma unroll
    for (int x = 0; x + 1 < N; x += 2) {
        if constexpr (ES == 4) {
            st.top = max3n(st.top, fabsf(__uint_as_float(w[x])), fabsf(__uint_as_float(w[x + 1])));
        } else {
            const f16x2 a = __builtin_bit_cast(f16x2, w[x]), b = __builtin_bit_cast(f16x2, w[x + 1]);
            st.vmax = __builtin_elementwise_maximum(__builtin_elementwise_maximum(st.vmax, a), b);
            st.vmin = __builtin_elementwise_minimum(__builtin_elementwise_minimum(st.vmin, a), b);
        }
    }
}
template <int ES, int D, int NB> __device__ __forceinline__ bool needs_care(const State32<D, NB> &st) {
    bool care = !(st.top < kFastValue);
    if constexpr (ES == 2) {
        const _Float16 most = (_Float16)512.f;  // bits 0x6000: 2^65 in bf16
        care |= !(st.vmax.x < most) || !(st.vmax.y < most) || !(st.vmin.x > -most) || !(st.vmin.y > -most);
    }
    return __any(care);
}

// V^T operands of dim block mb (dims 4m + mb) for the bf16 PV product: element t
// = 4g + i of lane (m, j) is key 16g + 4j + i.
template <int ES>
__device__ __forceinline__ void value_bf16(const uint32_t (&v)[2][4][ES], u32x4 (&a)[4]) {
#pragma unroll
    for (int y = 0; y < 4; ++y) {  // keys t = 2y, 2y + 1
        const int g = y >> 1, i = 2 * (y & 1);
        if constexpr (ES == 2) {
#pragma unroll
            for (int mb = 0; mb < 4; ++mb)
                a[mb][y] = __builtin_amdgcn_perm(v[g][i + 1][mb >> 1], v[g][i][mb >> 1], (mb & 1) ? 0x07060302u : 0x05040100u);
        } else {
            // bytes (t, t+1) of two dim blocks per permute, then exact conversion
            const uint32_t lo = __builtin_amdgcn_perm(v[g][i + 1][0], v[g][i][0], 0x05010400u);
            const uint32_t hi = __builtin_amdgcn_perm(v[g][i + 1][0], v[g][i][0], 0x07030602u);
            a[0][y] = fp8x2_to_bf16x2<false>(lo);
            a[1][y] = fp8x2_to_bf16x2<true>(lo);
            a[2][y] = fp8x2_to_bf16x2<false>(hi);
            a[3][y] = fp8x2_to_bf16x2<true>(hi);
        }
    }
}

// A probability in three bf16 terms, hi + mid + lo == p exactly (8 + 8 + 8
// significant bits, each the truncation of what is left).
__device__ __forceinline__ void split3(float p, uint32_t &hi, uint32_t &mid, uint32_t &lo) {
    hi = __float_as_uint(p);
    const float r1 = p - __uint_as_float(hi & 0xFFFF0000u);
    mid = __float_as_uint(r1);
    lo = __float_as_uint(r1 - __uint_as_float(mid & 0xFFFF0000u));
}
// the upper halves of two words
__device__ __forceinline__ uint32_t upper2(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }

// The careful softmax of a tile: products s * sc rounded before the reference is
// subtracted (exactly 0 at the maximum), the reference the maximum of all keys so
// far, denormal probabilities kept, and accumulators that hold the weighted mean
// of the values so far in place of their weighted sum, which no finite value can
// make overflow.  l: the whole row sum, on every lane.
template <int D, int NB, int KG>
__device__ __forceinline__ void careful_softmax(f32x4 (&s)[KG][NB], State32<D, NB> &st, float sc) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float mx = -INFINITY;
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[g][nb][i] = mul_rounded(s[g][nb][i], sc);
                mx = fmaxf(mx, s[g][nb][i]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mold = st.thr[nb] == -INFINITY ? -INFINITY : st.msub[nb];
        const float mnew = fmaxf(mold, mx);
        const float msub = mnew == -INFINITY ? 0.f : mnew;
        float l = 0.f;
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[g][nb][i] = exp2f(s[g][nb][i] - msub);
                l += s[g][nb][i];
            }
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const float old = st.l[nb] * exp2f(mold - msub);
        l += old;
        // l == 0: no visible key; l NaN: a NaN key or a +inf score was visible
        const float inv = l > 0.f ? 1.f / l : l;
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[g][nb][i] *= inv;
#pragma unroll
        for (int mb = 0; mb < D / 16; ++mb) st.acc[mb][nb] *= old * inv;
        st.l[nb] = l;
        st.msub[nb] = msub;
        st.thr[nb] = mnew == -INFINITY ? -INFINITY : 0.f;  // a reference exists
    }
}

// The online softmax of a tile with a lazy reference maximum, as compute_tile
// (mfma_common.h).  l: this lane's part of the row sum.
template <int D, int NB, int KG>
__device__ __forceinline__ void lazy_softmax(f32x4 (&s)[KG][NB], State32<D, NB> &st, float sc) {
    float lmax[NB];
    bool over = false;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        if constexpr (KG == 2) {
            lmax[nb] = max8(s[0][nb], s[1][nb]);
        } else {
            lmax[nb] = __builtin_elementwise_maximum(s[0][nb][0], max3n(s[0][nb][1], s[0][nb][2], s[0][nb][3]));
        }
        over |= lmax[nb] > st.thr[nb];
    }
    if (__any(over)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float mx = fmaxf(lmax[nb], __shfl_xor(lmax[nb], 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            mx *= sc;  // sc > 0
            const float mold = st.thr[nb] == -INFINITY ? -INFINITY : st.msub[nb];
            const float mnew = mx > mold + kRescaleLog2 ? mx : mold;
            const float msub = mnew == -INFINITY ? 0.f : mnew;
            const float alpha = fast_exp2(mold - msub);  // 1 when unchanged, 0 from -inf
            st.msub[nb] = msub;
            st.top = fabsf(msub) < kFastReference ? st.top : INFINITY;
            st.thr[nb] = mnew == -INFINITY ? -INFINITY : fmaxf((mnew + kRescaleLog2) / sc, -FLT_MAX);
#pragma unroll
            for (int mb = 0; mb < D / 16; ++mb) st.acc[mb][nb] *= alpha;
            st.l[nb] *= alpha;
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float l = 0.f;
#pragma unroll
        for (int g = 0; g < KG; ++g) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[g][nb][i] = fast_exp2(fmaf(s[g][nb][i], sc, -st.msub[nb]));
            l += (s[g][nb][0] + s[g][nb][1]) + (s[g][nb][2] + s[g][nb][3]);
        }
        st.l[nb] += l;
    }
}

// FAST: the lazy reference maximum (careful_softmax otherwise), and for 16- and
// 8-bit values the PV product on the bf16 instruction, every probability as its
// three bf16 terms; else on the fp32 instruction.
template <int ES, int D, int NB, int KG, bool FAST>
__device__ __forceinline__ void compute_tile32(Tile32<ES, D, KG> &T, const Q32<ES, D, NB> &q, State32<D, NB> &st,
                                               int tile, int n, int full_lim, float sc, int lane) {
    using TT = Tile32<ES, D, KG>;
    const int j = lane >> 4;
    const int key0 = tile * 16 * KG;
    // fp32 products: two sums of half the terms each, with less rounding than one (the
    // second in the registers of the keys the first is done with)
    f32x4 s[KG][NB], s1[KG][NB];
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) s[g][nb] = s1[g][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < TT::NKC; ++c) {
        if constexpr (ES == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int g = 0; g < KG; ++g)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        f32x4 &sum = 2 * c >= TT::NKC ? s1[g][nb] : s[g][nb];
                        sum = mfma_f32(__uint_as_float(T.k[g][c][e]), __uint_as_float(q.r[nb][c][e]), sum);
                    }
        } else if constexpr (ES == 2) {
#pragma unroll
            for (int g = 0; g < KG; ++g)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) s[g][nb] = mfma_bf16(T.k[g][c], q.r[nb][c], s[g][nb]);
        } else {
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                const u32x4 lo = fp8x8_to_bf16x8(T.k[g][c].x, T.k[g][c].y);
                const u32x4 hi = fp8x8_to_bf16x8(T.k[g][c].z, T.k[g][c].w);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    s[g][nb] = mfma_bf16(lo, q.r[nb][2 * c], s[g][nb]);
                    s[g][nb] = mfma_bf16(hi, q.r[nb][2 * c + 1], s[g][nb]);
                }
            }
        }
    }
    if constexpr (ES == 4) {
        settle(s);
        settle(s1);
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) s[g][nb] += s1[g][nb];
    }
    if (key0 + 16 * KG > full_lim) {  // uniform: only tiles reaching past a row's last visible key
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int g = 0; g < KG; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (key0 + 16 * g + 4 * j + i >= st.lim[nb]) s[g][nb][i] = -INFINITY;
    }
    if constexpr (FAST) lazy_softmax<D, NB, KG>(s, st, sc);
    else careful_softmax<D, NB, KG>(s, st, sc);
    if (key0 + 16 * KG > n) {  // uniform: storage of keys beyond the segment end may hold anything
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (key0 + 16 * g + 4 * j + i >= n) {
#pragma unroll
                    for (int x = 0; x < TT::VW; ++x) T.v[g][i][x] = 0u;
                }
    }
    if constexpr (FAST) {
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            if constexpr (TT::VW == 1) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) note_values<ES>(st, T.v[g][i]);
        }
    }
    if constexpr (FAST && ES <= 2) {
        static_assert(D == 64 && KG == 2, "32 keys of 64 dims, 16-bit or 8-bit values");
        u32x4 a[4];
        value_bf16<ES>(T.v, a);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            u32x4 t[3];
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                uint32_t h0, m0, l0, h1, m1, l1;
                split3(s[y >> 1][nb][2 * (y & 1)], h0, m0, l0);
                split3(s[y >> 1][nb][2 * (y & 1) + 1], h1, m1, l1);
                t[0][y] = upper2(l0, l1);
                t[1][y] = upper2(m0, m1);
                t[2][y] = upper2(h0, h1);
            }
#pragma unroll
            for (int x = 0; x < 3; ++x)
#pragma unroll
                for (int mb = 0; mb < 4; ++mb) st.acc[mb][nb] = mfma_bf16(a[mb], t[x], st.acc[mb][nb]);
        }
    } else {
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v[D / 16];
                value_f32<ES, D>(T.v[g][i], v);
#pragma unroll
                for (int mb = 0; mb < D / 16; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) st.acc[mb][nb] = mfma_f32(v[mb], s[g][nb][i], st.acc[mb][nb]);
            }
    }
}

// Load the queries of rows r0 .. r0 + 16 NB - 1 and reset their state.
template <int ES, int D, int NB>
__device__ __forceinline__ void begin_rows32(const Problem &p, int b, int h, int n, int r0, Q32<ES, D, NB> &q,
                                             State32<D, NB> &st, int lane) {
    const int n16 = lane & 15, j = lane >> 4;
    st.top = 0.f;
    st.vmax = st.vmin = f16x2{(_Float16)0.f, (_Float16)0.f};
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int r = r0 + 16 * nb + n16;
        st.l[nb] = 0.f;
        st.msub[nb] = 0.f;
        st.thr[nb] = -INFINITY;
        st.lim[nb] = r < p.R ? visible_limit(p, n, r) : n;
#pragma unroll
        for (int mb = 0; mb < D / 16; ++mb) st.acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int64_t off = r < p.R ? row_offset(p, b, h, r) : 0;
#pragma unroll
        for (int c = 0; c < Q32<ES, D, NB>::N; ++c) {
            u32x4 v = u32x4{0u, 0u, 0u, 0u};
            if constexpr (ES == 4) {  // dims 16 c + 4 j .. +3
                if (r < p.R) {
                    if (p.q_dtype == SPIRE_F32) {
                        v = *reinterpret_cast<const u32x4 *>(p.q + (off + 16 * c + 4 * j) * 4);
                    } else {
                        const u32x2 w = *reinterpret_cast<const u32x2 *>(p.q + (off + 16 * c + 4 * j) * 2);
                        v = u32x4{w.x << 16, w.x & 0xFFFF0000u, w.y << 16, w.y & 0xFFFF0000u};
                    }
                }
            } else {
                const int d0 = ES == 1 ? 64 * (c >> 1) + 16 * j + 8 * (c & 1) : 32 * c + 8 * j;
                if (r < p.R) v = *reinterpret_cast<const u32x4 *>(p.q + (off + d0) * 2);
            }
            q.r[nb][c] = v;
        }
    }
}

// Lane l owns, for every i, the 4-dim groups at dim32(i, x) of its rows.
template <int ES, int D> __device__ __forceinline__ int dim32(int i, int x, int j) {
    if (D == 64) return 16 * j + 4 * i;
    return ES == 4 ? 64 * x + 16 * j + 4 * i : 32 * j + 8 * i + 4 * x;
}

// Final rows (whole) or a partial into workspace slot `slot` of the unit whose
// rows start at u0.  MEAN: the accumulators hold means (stream32_careful).
template <int ES, int D, int NB, bool MEAN>
__device__ __forceinline__ void end_rows32(const Problem &p, const Plan &pl, State32<D, NB> &st, int b, int h, int r0,
                                           int u0, bool whole, int64_t slot, int lane) {
    const int n16 = lane & 15, j = lane >> 4;
    const float vs = ES == 1 ? uload(p.kv.v_scale, h) : 1.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float l = st.l[nb];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int r = r0 + 16 * nb + n16;
        if (r >= p.R) continue;
        // l == 0: no visible key; l NaN: a NaN key or a +inf score was visible
        const float inv = l > 0.f ? (MEAN ? vs : vs / l) : (l == 0.f ? 0.f : l);
        const float lse2 = l > 0.f ? st.msub[nb] + log2f(l) : (l == 0.f ? -INFINITY : l);
        const int64_t off = row_offset(p, b, h, r);
        float *part = pl.part_o + (slot * pl.rows + (r - u0)) * (int64_t)D;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int x = 0; x < D / 64; ++x) {
                const f32x4 o = f32x4{st.acc[4 * x][nb][i], st.acc[4 * x + 1][nb][i], st.acc[4 * x + 2][nb][i],
                                      st.acc[4 * x + 3][nb][i]} * inv;
                const int d = dim32<ES, D>(i, x, j);
                if (!whole)
                    *reinterpret_cast<f32x4 *>(part + d) = o;
                else if (p.out_dtype == SPIRE_BF16)
                    *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(p.out) + off + d) =
                        u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
                else
                    *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(p.out) + off + d) = o;
            }
        if (j == 0) {
            if (!whole) pl.part_lse[slot * pl.rows + (r - u0)] = lse2;
            else if (p.lse != nullptr) p.lse[lse_index(p, b, h, r)] = lse2 * 0.69314718055994531f;
        }
    }
}

// The tile's key registers hold nothing from here on (no instruction; without it
// the compiler keeps them where no next tile is loaded).  fp32 drafts of many short
// segments run three waves per SIMD with it (162 registers, 170 without: 2400
// segments of 64 keys 20.3 us, 21.3).
template <int ES, int D, int KG> __device__ __forceinline__ void forget_keys(Tile32<ES, D, KG> &T) {
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int c = 0; c < Tile32<ES, D, KG>::NKC; ++c) asm volatile("" : "=v"(T.k[g][c]));
}

// Tiles [first, last] through NBUF register buffers, NBUF - 1 tiles in flight:
// three, and five of the 4 KB fp8 tiles while they fit (64 sequences of 512-8192
// fp8 keys, 20 rows: 57.6 -> 52.4 us; bf16 within 1 % from two to five).
template <int ES, int D, int NB, int KG, int MODE, bool KNT = true>
__device__ __forceinline__ void stream32(const SegAddr &a, const Q32<ES, D, NB> &q, State32<D, NB> &st, int first,
                                         int last, int n, int full_lim, float sc, int lane) {
    constexpr int NBUF = ES == 1 && NB <= 3 ? 5 : 3;
    Tile32<ES, D, KG> T[NBUF];
#pragma unroll
    for (int x = 0; x < NBUF - 1; ++x)
        if (first + x <= last) load_tile32<ES, D, KG, MODE, KNT>(T[x], a, first + x, lane);
    int tt = first;
    while (true) {
#pragma unroll
        for (int x = 0; x < NBUF; ++x) {
            if (tt + NBUF - 1 <= last)
                load_tile32<ES, D, KG, MODE, KNT>(T[(x + NBUF - 1) % NBUF], a, tt + NBUF - 1, lane);
            else if constexpr (ES == 4 && MODE == MODE_DRAFT)
                forget_keys(T[(x + NBUF - 1) % NBUF]);
            compute_tile32<ES, D, NB, KG, true>(T[x], q, st, tt, n, full_lim, sc, lane);
            if (++tt > last) {
                if constexpr (ES == 4) settle(st.acc);
                return;
            }
        }
    }
}

// Rows r0 .. r0 + 15 over the same tiles by the careful form, one tile at a time
// (rare): the accumulators are left as means, the row sums on one lane group.
template <int ES, int D, int KG, int MODE>
__device__ __forceinline__ void stream32_careful(const Problem &p, const SegAddr &a, State32<D, 1> &st, int b, int h,
                                                 int r0, int first, int last, int n, int full_lim, float sc, int lane) {
    Q32<ES, D, 1> q;
    begin_rows32<ES, D, 1>(p, b, h, n, r0, q, st, lane);
#pragma nounroll
    for (int tt = first; tt <= last; ++tt) {
        Tile32<ES, D, KG> T;
        load_tile32<ES, D, KG, MODE>(T, a, tt, lane);
        compute_tile32<ES, D, 1, KG, false>(T, q, st, tt, n, full_lim, sc, lane);
        settle(st.acc);
    }
    if ((lane >> 4) != 0) st.l[0] = 0.f;
}

template <int ES, int D, int NB, int MODE>
__global__ __launch_bounds__(64 * kMfmaWavesPerWG, 1) void f32_partial_kernel(Problem p, Plan pl) {
    constexpr int KG = f32_tile(ES) / 16;
    __shared__ int32_t s_pre[kPlanMaxB + 1];
    __shared__ int32_t s_sum[kMfmaWavesPerWG];
    plan_in_kernel<64 * kMfmaWavesPerWG>(p, pl, s_pre, s_sum);
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(blockIdx.x * kMfmaWavesPerWG + (threadIdx.x >> 6));
    if (wid >= pl.workers) return;
    const int64_t T = (int64_t)s_pre[p.B] * pl.units;
    int64_t pos = worker_begin(wid, T, pl.workers);
    const int64_t end = worker_begin(wid + 1, T, pl.workers);
    if (pos >= end) {
        if (lane == 0) pl.wstart[2 * wid] = -1;
        return;
    }
    int seg, tile;
    locate(s_pre, p.B, pl.units, pos, seg, tile);
    seg = __builtin_amdgcn_readfirstlane(seg);
    tile = __builtin_amdgcn_readfirstlane(tile);
    if (lane == 0) {  // recorded like the plan kernel's output
        pl.wstart[2 * wid] = seg;
        pl.wstart[2 * wid + 1] = tile;
    }
    const int64_t begin = pos;
    const int nrb = pl.units / p.Hkv;  // units per KV head
    while (pos < end) {
        const int b = seg / pl.units;
        const int u = seg - b * pl.units;
        const int h = u / nrb;
        const int r0 = (u - h * nrb) * pl.rows;
        const int span = __builtin_amdgcn_readfirstlane(s_pre[b + 1] - s_pre[b]);
        const int tiles_b = span - pl.seg_cost;
        const int64_t left = end - pos;
        const int te = left < (int64_t)(span - tile) ? tile + (int)left : span;
        if (tile < tiles_b) {  // else phantom positions only
            const int t1 = te < tiles_b ? te : tiles_b;
            const int n = effective_keys(p, b);
            const SegAddr a = make_seg_addr<MODE>(p, b, h, n);
            Q32<ES, D, NB> q;
            State32<D, NB> st;
            begin_rows32<ES, D, NB>(p, b, h, n, r0, q, st, lane);
            float sc = p.sm_scale_log2;
            if (ES == 1) sc *= uload(p.kv.k_scale, h);
            const int full_lim = p.draft ? n : n - p.k;
            const bool whole = tile == 0 && t1 == tiles_b;
            const int64_t slot = 2 * (int64_t)wid + (pos == begin ? 0 : 1);
            if (n > 0) stream32<ES, D, NB, KG, MODE>(a, q, st, tile, t1 - 1, n, full_lim, sc, lane);
            if (!needs_care<ES>(st)) {
                end_rows32<ES, D, NB, false>(p, pl, st, b, h, r0, r0, whole, slot, lane);
            } else {
#pragma nounroll
                for (int r = r0; r < r0 + 16 * NB && r < p.R; r += 16) {
                    State32<D, 1> one;
                    stream32_careful<ES, D, KG, MODE>(p, a, one, b, h, r, tile, t1 - 1, n, full_lim, sc, lane);
                    end_rows32<ES, D, 1, true>(p, pl, one, b, h, r, r0, whole, slot, lane);
                }
            }
        }
        pos += te - tile;
        ++seg;
        tile = 0;
    }
}

// Short draft segments of up to 16 rows, whole: G = 1, 2 or 4 waves of one
// workgroup per segment, as in attn_mfma.hip (the limits are the host's): no
// partition, no partials, no combine launch.  The waves split the tiles; beyond
// one they leave their accumulators in LDS and each merges and writes its share
// of the head-dim slices, on the reference maxima.  MI355X, 8 KV heads of 4
// queries, in a graph: 13 sequences of 256 bf16 keys at head_dim 64 12.8 -> 6.4 us,
// of 512 fp32 keys 16.6 -> 13.6; 64 of 256 fp32 keys 22.2 -> 14.3.
template <int ES, int D, int G>
__global__ __launch_bounds__(64 * kMfmaWavesPerWG, 1) void f32_draft_whole_kernel(Problem p) {
    constexpr int KG = f32_tile(ES) / 16;
    constexpr int SPW = kMfmaWavesPerWG / G;  // segments per workgroup
    constexpr int NS = D / 16, PER = NS / G;  // slices of four dims, and each wave's share
    __shared__ f32x4 s_o[SPW][G > 1 ? G : 1][G > 1 ? NS : 1][64];
    __shared__ float s_l[SPW][G][16];
    __shared__ float s_m[SPW][G][16];  // reference maximum; -inf: none
    __shared__ bool s_mean[SPW][G];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n16 = lane & 15, j = lane >> 4;
    const int slot = wave / G, part = wave - (wave / G) * G;
    const int seg = (int)blockIdx.x * SPW + slot;
    const bool valid = seg < p.B * p.Hkv;
    const int b = valid ? seg / p.Hkv : 0;
    const int h = valid ? seg - b * p.Hkv : 0;
    // what a wave found: the rows themselves (G = 1), or its part in LDS
    auto leave = [&](State32<D, 1> &st, auto mean_tag) {
        constexpr bool MEAN = decltype(mean_tag)::value;
        if constexpr (G == 1) {
            end_rows32<ES, D, 1, MEAN>(p, Plan{}, st, b, h, 0, 0, true, 0, lane);
        } else {
            float l = st.l[0];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            if (j == 0) {
                s_l[slot][part][n16] = l;
                s_m[slot][part][n16] = st.thr[0] == -INFINITY ? -INFINITY : st.msub[0];
                if (n16 == 0) s_mean[slot][part] = MEAN;
            }
#pragma unroll
            for (int y = 0; y < NS; ++y) {
                const int i = y & 3, x = y >> 2;
                s_o[slot][part][y][lane] = f32x4{st.acc[4 * x][0][i], st.acc[4 * x + 1][0][i], st.acc[4 * x + 2][0][i],
                                                 st.acc[4 * x + 3][0][i]};
            }
        }
    };
    if (valid) {
        const int n = effective_keys(p, b);
        const int T = (n + 16 * KG - 1) / (16 * KG);
        const int t0 = part * T / G, t1 = (part + 1) * T / G;
        State32<D, 1> st;
        Q32<ES, D, 1> q;
        begin_rows32<ES, D, 1>(p, b, h, n, 0, q, st, lane);
        st.lim[0] = n;  // a draft's rows see every key: uniform
        float sc = p.sm_scale_log2;
        if (ES == 1) sc *= uload(p.kv.k_scale, h);
        const SegAddr a = make_seg_addr<MODE_DRAFT>(p, b, h, n);
        // a segment with a CU to itself: ordinary K loads (ld16k; bf16, head_dim 64, 104
        // segments of 1024 keys 13.9 -> 12.8 us; the 64-sequence verify call loses 3 %)
        if (t0 < t1) stream32<ES, D, 1, KG, MODE_DRAFT, G != 4>(a, q, st, t0, t1 - 1, n, n, sc, lane);
        if (!needs_care<ES>(st)) {
            leave(st, std::false_type{});
        } else {
            State32<D, 1> one;
            stream32_careful<ES, D, KG, MODE_DRAFT>(p, a, one, b, h, 0, t0, t1 - 1, n, n, sc, lane);
            leave(one, std::true_type{});
        }
    }
    if constexpr (G > 1) {
        __syncthreads();
        if (!valid || n16 >= p.R) return;
        float m[G], l[G];
#pragma unroll
        for (int w = 0; w < G; ++w) {
            m[w] = s_m[slot][w][n16];
            l[w] = s_l[slot][w][n16];
        }
        RowMerge<G> mr = merge_row<G>(m, l, ES == 1 ? uload(p.kv.v_scale, h) : 1.f);
        bool mean = false;
#pragma unroll
        for (int w = 0; w < G; ++w) mean |= s_mean[slot][w];
        if (mean) {  // a mean's weight takes its sum, the division first: no term beyond the largest value
#pragma unroll
            for (int w = 0; w < G; ++w) mr.w[w] *= mr.inv * (s_mean[slot][w] ? l[w] : 1.f);
            mr.inv = 1.f;
        }
        const int64_t off = row_offset(p, b, h, n16);
#pragma unroll
        for (int z = 0; z < PER; ++z) {
            const int y = part * PER + z;
            f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < G; ++w) o += s_o[slot][w][y][lane] * mr.w[w];
            o *= mr.inv;
            const int d = dim32<ES, D>(y & 3, y >> 2, j);
            if (p.out_dtype == SPIRE_BF16)
                *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(p.out) + off + d) =
                    u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
            else
                *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(p.out) + off + d) = o;
        }
        if (part == 0 && j == 0 && p.lse != nullptr) p.lse[lse_index(p, b, h, n16)] = mr.lse2 * 0.69314718055994531f;
    }
}

template <int ES, int D>
static hipError_t launch_whole_d(const Problem &p, int g, hipStream_t st) {
    const unsigned segs = (unsigned)(p.B * p.Hkv);
    const dim3 block(64 * kMfmaWavesPerWG);
    switch (g) {
    case 1: hipLaunchKernelGGL((f32_draft_whole_kernel<ES, D, 1>), dim3((segs + 3) / 4), block, 0, st, p); break;
    case 2: hipLaunchKernelGGL((f32_draft_whole_kernel<ES, D, 2>), dim3((segs + 1) / 2), block, 0, st, p); break;
    case 4: hipLaunchKernelGGL((f32_draft_whole_kernel<ES, D, 4>), dim3(segs), block, 0, st, p); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_f32_draft_whole(const Problem &p, int g, hipStream_t st) {
    if (!p.draft || p.R > 16 || p.B * p.Hkv <= 0) return hipErrorInvalidValue;
    if (p.kv_dtype == SPIRE_F32) return p.D == 64 ? launch_whole_d<4, 64>(p, g, st) : launch_whole_d<4, 128>(p, g, st);
    if (p.D != 64 || p.q_dtype != SPIRE_BF16) return hipErrorInvalidValue;
    return p.kv_dtype == SPIRE_BF16 ? launch_whole_d<2, 64>(p, g, st) : launch_whole_d<1, 64>(p, g, st);
}

template <int ES, int D, int NB>
static hipError_t launch_f32_nb(const Problem &p, const Plan &pl, hipStream_t st) {
    const dim3 grid((pl.workers + kMfmaWavesPerWG - 1) / kMfmaWavesPerWG), block(64 * kMfmaWavesPerWG);
    if (p.draft)
        hipLaunchKernelGGL((f32_partial_kernel<ES, D, NB, MODE_DRAFT>), grid, block, 0, st, p, pl);
    else if (p.kv.page_size > 0)
        hipLaunchKernelGGL((f32_partial_kernel<ES, D, NB, MODE_PAGED>), grid, block, 0, st, p, pl);
    else
        hipLaunchKernelGGL((f32_partial_kernel<ES, D, NB, MODE_CONTIG>), grid, block, 0, st, p, pl);
    return hipGetLastError();
}

template <int ES, int D>
static hipError_t launch_f32_d(const Problem &p, const Plan &pl, int nb, hipStream_t st) {
    switch (nb) {
    case 1: return launch_f32_nb<ES, D, 1>(p, pl, st);
    case 2: return launch_f32_nb<ES, D, 2>(p, pl, st);
    case 3: if constexpr (f32_blocks(ES, D) >= 3) return launch_f32_nb<ES, D, 3>(p, pl, st); break;
    case 4: if constexpr (f32_blocks(ES, D) >= 4) return launch_f32_nb<ES, D, 4>(p, pl, st); break;
    case 5: if constexpr (f32_blocks(ES, D) >= 5) return launch_f32_nb<ES, D, 5>(p, pl, st); break;
    }
    return hipErrorInvalidValue;
}

hipError_t launch_f32_partial(const Problem &p, const Plan &pl, int nb, hipStream_t st) {
    if (p.kv_dtype == SPIRE_F32)
        return p.D == 64 ? launch_f32_d<4, 64>(p, pl, nb, st) : launch_f32_d<4, 128>(p, pl, nb, st);
    if (p.D != 64 || p.q_dtype != SPIRE_BF16) return hipErrorInvalidValue;
    return p.kv_dtype == SPIRE_BF16 ? launch_f32_d<2, 64>(p, pl, nb, st) : launch_f32_d<1, 64>(p, pl, nb, st);
}

}  // namespace spire
