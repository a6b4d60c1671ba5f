// feedback_memory.hip -- feedback-memory mixing of the draft's activations (gfx950).
//
// The draft is a Feedback Transformer (paper Sec. 3.3): its attention reads
// memory vectors, one per draft layer i, each a convex mix of the token's
// activations after every layer (layer 0 the embedding):
//     m^i = sum_l exp(w_il) x^l / sum_l exp(w_il).
// x is [L+1, B*d], m is [n_out, B*d].  Every workgroup first turns the n_out
// rows of weights into mixing weights (row maximum subtracted, fp32) in LDS;
// every thread then reads E consecutive elements of each layer once and produces
// all n_out outputs from them, so x is read once and m written once.
//
// Bound by HBM and by the start of the launch.  Vector path (aligned rows): at
// most kFmGroups workgroups walk the elements, so the weights are formed and the
// waves launched once per several chunks (one chunk per thread took 4096
// workgroups for 512 x 8192), the first layers of the next chunk are requested
// before the current one is stored, and a thread's accumulators are only as many
// as the call's outputs, rounded up to 1, 2, 4 or 8 (with room for 8 and two
// used, wider loads halved the waves per SIMD and lost what they gained).
// MI355X, 512 x 8192 bf16, 3 layers, 2 outputs (42 MB): 10.5 -> 9.3 us a call.
#include "spire_internal.h"

namespace spire {

constexpr int kFmThreads = 256;

// Rows off those boundaries: four elements per thread, one by one.
template <int XDT, int MDT>
__global__ __launch_bounds__(kFmThreads) void feedback_memory_kernel(FeedbackArgs a) {
    __shared__ float s_w[kFmMaxOut * kFmMaxLayers];
    if ((int)threadIdx.x < a.n_out) {
        const int i = threadIdx.x;
        float top = -INFINITY;
        for (int l = 0; l < a.Lp1; ++l) top = fmaxf(top, a.w[i * a.Lp1 + l]);
        float sum = 0.f;
        for (int l = 0; l < a.Lp1; ++l) {
            const float e = expf(a.w[i * a.Lp1 + l] - top);
            s_w[i * a.Lp1 + l] = e;
            sum += e;
        }
        const float inv = 1.f / sum;
        for (int l = 0; l < a.Lp1; ++l) s_w[i * a.Lp1 + l] *= inv;
    }
    __syncthreads();
    const int64_t e0 = ((int64_t)blockIdx.x * kFmThreads + threadIdx.x) * 4;
    if (e0 >= a.Bd) return;
    float acc[kFmMaxOut][4];
#pragma unroll
    for (int i = 0; i < kFmMaxOut; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[i][c] = 0.f;
    for (int l = 0; l < a.Lp1; ++l) {
        float xv[4];
        const int64_t base = (int64_t)l * a.Bd + e0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            xv[c] = 0.f;
            if (e0 + c < a.Bd)
                xv[c] = XDT == SPIRE_F32 ? static_cast<const float *>(a.x)[base + c]
                                         : bf16_to_f32(static_cast<const uint16_t *>(a.x)[base + c]);
        }
#pragma unroll
        for (int i = 0; i < kFmMaxOut; ++i) {
            if (i < a.n_out) {
                const float wl = s_w[i * a.Lp1 + l];
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[i][c] = fmaf(wl, xv[c], acc[i][c]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kFmMaxOut; ++i) {
        if (i >= a.n_out) break;
        const int64_t o = (int64_t)i * a.Bd + e0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (e0 + c >= a.Bd) break;
            if (MDT == SPIRE_F32) static_cast<float *>(a.m)[o + c] = acc[i][c];
            else static_cast<uint16_t *>(a.m)[o + c] = f32_to_bf16_rne(acc[i][c]);
        }
    }
}

// E elements of one layer as they are stored
template <int XDT, int E> struct FmRaw { uint32_t v[XDT == SPIRE_F32 ? E : E / 2]; };
template <int XDT, int E> __device__ __forceinline__ FmRaw<XDT, E> fm_load(const void *x, int64_t at) {
    FmRaw<XDT, E> r;
    constexpr int W = XDT == SPIRE_F32 ? E : E / 2;
    const uint32_t *p = static_cast<const uint32_t *>(x) + (XDT == SPIRE_F32 ? at : at / 2);
    if constexpr (W == 4) {
        const uint4 q = *reinterpret_cast<const uint4 *>(p);
        r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
    } else {
        const uint2 q = *reinterpret_cast<const uint2 *>(p);
        r.v[0] = q.x; r.v[1] = q.y;
    }
    return r;
}

constexpr int kFmAhead = 4;      // layers requested before their chunk's turn
constexpr int kFmGroups = 2048;  // workgroups of a launch: eight per CU

template <int XDT, int MDT, int NOUT, int E>
__global__ __launch_bounds__(kFmThreads) void feedback_memory_vec_kernel(FeedbackArgs a) {
    __shared__ float s_w[kFmMaxOut * kFmMaxLayers];
    const int64_t stride = (int64_t)gridDim.x * kFmThreads * E;
    int64_t e0 = ((int64_t)blockIdx.x * kFmThreads + threadIdx.x) * E;
    FmRaw<XDT, E> ahead[kFmAhead];
    auto request = [&](int64_t e) {
#pragma unroll
        for (int l = 0; l < kFmAhead; ++l)
            if (l < a.Lp1 && e < a.Bd) ahead[l] = fm_load<XDT, E>(a.x, (int64_t)l * a.Bd + e);
    };
    request(e0);
    for (int i = threadIdx.x; i < a.n_out * a.Lp1; i += kFmThreads) s_w[i] = a.w[i];
    __syncthreads();
    if ((int)threadIdx.x < a.n_out) {
        float *w = s_w + threadIdx.x * a.Lp1;
        float top = -INFINITY;
        for (int l = 0; l < a.Lp1; ++l) top = fmaxf(top, w[l]);
        float sum = 0.f;
        for (int l = 0; l < a.Lp1; ++l) {
            const float e = expf(w[l] - top);
            w[l] = e;
            sum += e;
        }
        const float inv = 1.f / sum;
        for (int l = 0; l < a.Lp1; ++l) w[l] *= inv;
    }
    __syncthreads();
    for (; e0 < a.Bd; e0 += stride) {
        float acc[NOUT][E];
#pragma unroll
        for (int i = 0; i < NOUT; ++i)
#pragma unroll
            for (int c = 0; c < E; ++c) acc[i][c] = 0.f;
        auto mix = [&](int l, const FmRaw<XDT, E> &r) {
            float xv[E];
#pragma unroll
            for (int c = 0; c < E; ++c) {
                if constexpr (XDT == SPIRE_F32) xv[c] = __uint_as_float(r.v[c]);
                else xv[c] = __uint_as_float(c & 1 ? r.v[c / 2] & 0xFFFF0000u : r.v[c / 2] << 16);
            }
#pragma unroll
            for (int i = 0; i < NOUT; ++i) {
                if (i < a.n_out) {
                    const float wl = s_w[i * a.Lp1 + l];
#pragma unroll
                    for (int c = 0; c < E; ++c) acc[i][c] = fmaf(wl, xv[c], acc[i][c]);
                }
            }
        };
#pragma unroll
        for (int l = 0; l < kFmAhead; ++l)
            if (l < a.Lp1) mix(l, ahead[l]);
        for (int l = kFmAhead; l < a.Lp1; ++l) mix(l, fm_load<XDT, E>(a.x, (int64_t)l * a.Bd + e0));
        request(e0 + stride);
#pragma unroll
        for (int i = 0; i < NOUT; ++i) {
            if (i >= a.n_out) break;
            const int64_t o = (int64_t)i * a.Bd + e0;
#pragma unroll
            for (int c = 0; c < E; c += 4) {
                if (MDT == SPIRE_F32) {
                    *reinterpret_cast<float4 *>(static_cast<float *>(a.m) + o + c) =
                        make_float4(acc[i][c], acc[i][c + 1], acc[i][c + 2], acc[i][c + 3]);
                } else if (E == 8) {
                    if (c == 0) {
                        uint32_t q[4];
#pragma unroll
                        for (int d = 0; d < 4; ++d)
                            q[d] = f32_to_bf16_rne(acc[i][2 * d]) | ((uint32_t)f32_to_bf16_rne(acc[i][2 * d + 1]) << 16);
                        *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(a.m) + o) = make_uint4(q[0], q[1], q[2], q[3]);
                    }
                } else {
                    const uint32_t lo = f32_to_bf16_rne(acc[i][0]) | ((uint32_t)f32_to_bf16_rne(acc[i][1]) << 16);
                    const uint32_t hi = f32_to_bf16_rne(acc[i][2]) | ((uint32_t)f32_to_bf16_rne(acc[i][3]) << 16);
                    *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(a.m) + o) = make_uint2(lo, hi);
                }
            }
        }
    }
}

template <int XDT, int MDT, int NOUT, int E>
static void launch_fm_vec(const FeedbackArgs &a, hipStream_t st) {
    const int64_t chunks = (a.Bd / E + kFmThreads - 1) / kFmThreads;
    const dim3 grid((unsigned)(chunks < kFmGroups ? chunks : kFmGroups)), block(kFmThreads);
    hipLaunchKernelGGL((feedback_memory_vec_kernel<XDT, MDT, NOUT, E>), grid, block, 0, st, a);
}

template <int XDT, int MDT>
static void launch_fm_dt(const FeedbackArgs &a, bool vec, bool wide, hipStream_t st) {
    if (!vec) {
        const dim3 grid((unsigned)((a.Bd + 4LL * kFmThreads - 1) / (4LL * kFmThreads))), block(kFmThreads);
        hipLaunchKernelGGL((feedback_memory_kernel<XDT, MDT>), grid, block, 0, st, a);
        return;
    }
    // eight 16-bit elements (16 bytes) per thread and layer where their
    // accumulators are few
    if constexpr (XDT == SPIRE_BF16) {
        if (wide && a.n_out <= 4) {
            if (a.n_out == 1) launch_fm_vec<XDT, MDT, 1, 8>(a, st);
            else if (a.n_out == 2) launch_fm_vec<XDT, MDT, 2, 8>(a, st);
            else launch_fm_vec<XDT, MDT, 4, 8>(a, st);
            return;
        }
    }
    if (a.n_out == 1) launch_fm_vec<XDT, MDT, 1, 4>(a, st);
    else if (a.n_out == 2) launch_fm_vec<XDT, MDT, 2, 4>(a, st);
    else if (a.n_out <= 4) launch_fm_vec<XDT, MDT, 4, 4>(a, st);
    else launch_fm_vec<XDT, MDT, 8, 4>(a, st);
}

hipError_t launch_feedback_memory(const FeedbackArgs &a, hipStream_t st) {
    // vector loads and stores need B*d % 4 == 0 and 16-byte (f32) / 8-byte (bf16)
    // bases, eight elements at a time B*d % 8 == 0 and 16-byte bases
    const uintptr_t xa = a.x_dtype == SPIRE_F32 ? 15u : 7u, ma = a.m_dtype == SPIRE_F32 ? 15u : 7u;
    const bool vec = (a.Bd % 4) == 0 && ((uintptr_t)a.x & xa) == 0 && ((uintptr_t)a.m & ma) == 0;
    const bool wide = vec && (a.Bd % 8) == 0 && ((uintptr_t)a.x & 15u) == 0 && ((uintptr_t)a.m & 15u) == 0;
    if (a.x_dtype == SPIRE_F32) {
        if (a.m_dtype == SPIRE_F32) launch_fm_dt<SPIRE_F32, SPIRE_F32>(a, vec, wide, st);
        else launch_fm_dt<SPIRE_F32, SPIRE_BF16>(a, vec, wide, st);
    } else {
        if (a.m_dtype == SPIRE_F32) launch_fm_dt<SPIRE_BF16, SPIRE_F32>(a, vec, wide, st);
        else launch_fm_dt<SPIRE_BF16, SPIRE_BF16>(a, vec, wide, st);
    }
    return hipGetLastError();
}

}  // namespace spire
