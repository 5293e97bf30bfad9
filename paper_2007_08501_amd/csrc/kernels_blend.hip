// kernels_blend.hip -- silhouette blend (paper, Section 3.2, Algorithm 1),
// softmax blend (Algorithm 2) and their backwards, for gfx950: both spread a
// pixel's slots over a group of lanes.
//
// Silhouette:
//   prob_k = sigmoid(-d_k / sigma) where the slot holds a face, else 0
//   alpha  = 1 - prod_k (1 - prob_k)
//   d alpha / d d_k = -(1/sigma) prob_k (1 - prob_k) prod_{j != k} (1 - prob_j)
// 1 - prob_k is evaluated as sigmoid(+d_k / sigma) so that it keeps its
// relative accuracy where prob_k is close to 1 (deep inside a face).
#include "device.hpp"
#include "launch.hpp"

namespace rast {

// sigmoid(x) and sigmoid(-x), 1 / (1 + e) and e / (1 + e) with e = exp(-|x|),
// which does not overflow: one exponential and no branch for both signs.
// Evaluated by a branch on the sign (two exponentials and two divisions
// wherever a wave holds both signs, and again for -x) this bound the silhouette
// blend, with its loads in branches that waited for each other: 20 x
// 128 x 128 pixels, K = 50 took 43 us forward and 53 us backward, now 29 and 43
// (bound by memory: 65 MB of ids read, and in the backward 65 MB written).
__device__ __forceinline__ float sigmoidf(float x) {
    const float e = expf(-fabsf(x));
    return (x >= 0.0f ? 1.0f : e) / (1.0f + e);
}
__device__ __forceinline__ void sigmoid_pair(float x, float& pos, float& neg) {
    const float e = expf(-fabsf(x)), den = 1.0f + e;
    pos = (x >= 0.0f ? 1.0f : e) / den;
    neg = (x <= 0.0f ? 1.0f : e) / den;
}

// A pixel's K slots are spread over L lanes of a wave, four consecutive slots
// per lane (L the power of two with 4 L >= K, 64 / L pixels per wave), so
// that consecutive lanes read consecutive words: each lane combines its own
// slots and only the per-lane products cross lanes (segmented scans of
// log2(L) steps).  One lane per pixel walking its K words would make every
// load instruction touch 64 different rows (a 200-byte stride at K = 50).
constexpr int kBlendQ = 4;  // consecutive slots per lane
// four words at 4-byte alignment (a pixel's slots start at any word)
typedef int bi32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float bf32x4 __attribute__((ext_vector_type(4), aligned(4)));

// A lane's slots of one pixel: whether each holds a face, and d / sigma.  The
// distances are read only by lanes that hold a face.  TAIL: slots or pixels
// may lie beyond the arrays' ends; without it a lane whose slots run past its
// pixel's reads the next pixel's words and drops them, so that no load sits in
// a branch and the loads of all groups are in flight together.
struct BlendSlots {
    bool on[kBlendQ];
    float x[kBlendQ];
    bool any;

    template <bool TAIL>
    __device__ __forceinline__ void load_ids(const int32_t* __restrict__ p2f, int64_t p, int64_t P, int K, int sub) {
        const int64_t o = p * K + kBlendQ * sub;
        if constexpr (TAIL) {
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i) on[i] = p < P && kBlendQ * sub + i < K && p2f[o + i] >= 0;
        } else {
            const bi32x4 vi = *reinterpret_cast<const bi32x4*>(p2f + o);
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i) on[i] = kBlendQ * sub + i < K && vi[i] >= 0;
        }
        any = false;
#pragma unroll
        for (int i = 0; i < kBlendQ; ++i) any = any || on[i];
    }

    template <bool TAIL>
    __device__ __forceinline__ void load_dists(const float* __restrict__ d, int64_t p, int K, int sub,
                                               float inv_sigma) {
        const int64_t o = p * K + kBlendQ * sub;
        bf32x4 vd{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (TAIL) {
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i)
                if (on[i]) vd[i] = d[o + i];
        } else {
            if (any) vd = *reinterpret_cast<const bf32x4*>(d + o);
        }
#pragma unroll
        for (int i = 0; i < kBlendQ; ++i) x[i] = vd[i] * inv_sigma;
    }
};

// pixel groups that a wave has in flight (their loads are issued together):
// 1 group 32 + 44 us at the size above, 2 groups 29 + 43, 4 groups 27 + 44
constexpr int kBlendU = 2;

// whether all words that a wave's groups at p0 touch without TAIL exist
template <int L>
__device__ __forceinline__ bool blend_inside(int64_t p0, int64_t P, int K) {
    return (p0 + kBlendU * (64 / L) - 1) * K + kBlendQ * L <= P * K;
}

// A wave's groups: the ids of all, then the distances of all.
template <int L, bool TAIL>
__device__ __forceinline__ void blend_load(const int32_t* __restrict__ p2f, const float* __restrict__ d, int64_t p,
                                           int64_t P, int K, int sub, float inv_sigma, BlendSlots (&sl)[kBlendU]) {
#pragma unroll
    for (int u = 0; u < kBlendU; ++u) sl[u].load_ids<TAIL>(p2f, p + u * (64 / L), P, K, sub);
#pragma unroll
    for (int u = 0; u < kBlendU; ++u) sl[u].load_dists<TAIL>(d, p + u * (64 / L), K, sub, inv_sigma);
}

template <int L>
__device__ __forceinline__ float blend_seg_prod(float v) {
#pragma unroll
    for (int m = L / 2; m >= 1; m >>= 1) v *= __shfl_xor(v, m, L);
    return v;
}

// product over the lower / the higher lanes of the segment (1 for none)
template <int L>
__device__ __forceinline__ float blend_excl_prefix(float t, int sub) {
#pragma unroll
    for (int m = 1; m < L; m <<= 1) {
        const float u = __shfl_up(t, m, L);
        if (sub >= m) t *= u;
    }
    const float e = __shfl_up(t, 1, L);
    return sub == 0 ? 1.0f : e;
}
template <int L>
__device__ __forceinline__ float blend_excl_suffix(float t, int sub) {
#pragma unroll
    for (int m = 1; m < L; m <<= 1) {
        const float u = __shfl_down(t, m, L);
        if (sub + m < L) t *= u;
    }
    const float e = __shfl_down(t, 1, L);
    return sub == L - 1 ? 1.0f : e;
}

template <int L>
__global__ __launch_bounds__(256) void blend_fwd_kernel(const int32_t* __restrict__ p2f, const float* __restrict__ d,
                                                        int64_t P, int K, float inv_sigma, float* __restrict__ alpha) {
    constexpr int PPW = 64 / L;
    const int lane = threadIdx.x & 63, sub = lane & (L - 1), grp = lane / L;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t p0 = wave * (PPW * kBlendU); p0 < P; p0 += nwaves * (PPW * kBlendU)) {
        BlendSlots sl[kBlendU];
        if (blend_inside<L>(p0, P, K)) {
            blend_load<L, false>(p2f, d, p0 + grp, P, K, sub, inv_sigma, sl);
        } else {
            blend_load<L, true>(p2f, d, p0 + grp, P, K, sub, inv_sigma, sl);
        }
#pragma unroll
        for (int u = 0; u < kBlendU; ++u) {
            float t = 1.0f;  // product of 1 - prob_k over the lane's slots
            if (__any(sl[u].any)) {
#pragma unroll
                for (int i = 0; i < kBlendQ; ++i)
                    t *= sl[u].on[i] ? sigmoidf(sl[u].x[i]) : 1.0f;
                t = blend_seg_prod<L>(t);
            }
            const int64_t p = p0 + u * PPW + grp;
            if (sub == 0 && p < P) alpha[p] = 1.0f - t;
        }
    }
}

// d alpha / d d_k = -(1/sigma) prob_k (1 - prob_k) prod_{j<k} (1 - prob_j)
// prod_{j>k} (1 - prob_j): the products of the other slots come from the
// lane's own prefix and suffix and the exclusive scans of the lane products
// (no division by 1 - prob_k, which underflows deep inside a face).
template <int L>
__global__ __launch_bounds__(256) void blend_bwd_kernel(const int32_t* __restrict__ p2f, const float* __restrict__ d,
                                                        const float* __restrict__ ga, int64_t P, int K, float inv_sigma,
                                                        float* __restrict__ gd) {
    constexpr int PPW = 64 / L;
    const int lane = threadIdx.x & 63, sub = lane & (L - 1), grp = lane / L;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t p0 = wave * (PPW * kBlendU); p0 < P; p0 += nwaves * (PPW * kBlendU)) {
        BlendSlots sl[kBlendU];
        float g[kBlendU];
        if (blend_inside<L>(p0, P, K)) {
#pragma unroll
            for (int u = 0; u < kBlendU; ++u) g[u] = ga[p0 + u * PPW + grp];
            blend_load<L, false>(p2f, d, p0 + grp, P, K, sub, inv_sigma, sl);
        } else {
#pragma unroll
            for (int u = 0; u < kBlendU; ++u) g[u] = p0 + u * PPW + grp < P ? ga[p0 + u * PPW + grp] : 0.0f;
            blend_load<L, true>(p2f, d, p0 + grp, P, K, sub, inv_sigma, sl);
        }
#pragma unroll
        for (int u = 0; u < kBlendU; ++u) {
            float out[kBlendQ];
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i) out[i] = 0.0f;
            if (__any(sl[u].any)) {
                float om[kBlendQ];  // 1 - prob_k (1 for an empty slot)
                float pr[kBlendQ];  // prob_k
                float t = 1.0f;
#pragma unroll
                for (int i = 0; i < kBlendQ; ++i) {
                    om[i] = 1.0f;
                    pr[i] = 0.0f;
                    // (uniform; without it 3,000,000 pixels of one slot took
                    // 23 us, 16 with a branch on every slot as with this)
                    if (L == 1 && i >= K) continue;
                    sigmoid_pair(sl[u].x[i], om[i], pr[i]);
                    if (!sl[u].on[i]) om[i] = 1.0f;
                    t *= om[i];
                }
                float pre = blend_excl_prefix<L>(t, sub);
                const float lsuf = blend_excl_suffix<L>(t, sub);
#pragma unroll
                for (int i = 0; i < kBlendQ; ++i) {
                    float suf = lsuf;
#pragma unroll
                    for (int j = i + 1; j < kBlendQ; ++j) suf *= om[j];
                    if (sl[u].on[i]) out[i] = -g[u] * inv_sigma * pr[i] * om[i] * pre * suf;
                    pre *= om[i];
                }
            }
            const int64_t p = p0 + u * PPW + grp, o = p * K + kBlendQ * sub;
            if (p < P && kBlendQ * (sub + 1) <= K) {
                *reinterpret_cast<bf32x4*>(gd + o) = bf32x4{out[0], out[1], out[2], out[3]};
            } else {
#pragma unroll
                for (int i = 0; i < kBlendQ; ++i)
                    if (p < P && kBlendQ * sub + i < K) gd[o + i] = out[i];
            }
        }
    }
}

// Softmax blend: prob_k = sigmoid(-d_k / sigma), zinv_k = (zfar - z_k) / (zfar - znear),
// w_k = prob_k exp((zinv_k - max_j zinv_j) / gamma), image = sum_k w_k c_k / sum_k w_k.
// Empty slots take no part; a pixel whose weights sum to 0 is 0.
// The exponent is evaluated as (min_j z_j - z_k) / ((zfar - znear) gamma),
// which equals (zinv_k - max zinv) / gamma: forming zinv first would round
// zfar - z (about zfar) and then divide that rounding by a small gamma.
//
// Bound by HBM (12 + 4 C bytes read a slot, in the backward up to as many
// written again), so the slots are spread over lanes as in the silhouette
// blend: a lane reads its four slots' ids, depths, distances and 4 C colours
// as 16-byte words, consecutive lanes consecutive words, and only the
// minimum, the weight sum and the C colour sums cross lanes.  Lanes whose four
// slots are all empty read no depths, distances or colours.  With one lane
// per pixel every load instruction touched 64 rows K C words apart and the
// loads of one slot waited for the last one's: a forward and backward of
// 4 x 512 x 512 pixels, K = 8, C = 3 took 534 us (87 + 435 in the kernels),
// now 103 us (the start of its reads still lies in the last-level cache).
struct SoftmaxArgs {
    const int32_t* p2f;
    const float* z;
    const float* d;
    const float* col;
    int64_t P;
    int K, C;
    float inv_sigma;
    float zscale;  // 1 / ((zfar - znear) gamma)
};

// Smallest value and sum over the lanes of a segment.
template <int L>
__device__ __forceinline__ float blend_seg_min(float v) {
#pragma unroll
    for (int m = L / 2; m >= 1; m >>= 1) v = fminf(v, __shfl_xor(v, m, L));
    return v;
}
template <int L>
__device__ __forceinline__ float blend_seg_sum(float v) {
#pragma unroll
    for (int m = L / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, L);
    return v;
}

// A lane's slots of one pixel and the pixel's blend.  CB: the channel count
// if EXACT, else a bound on it.
template <int L, int CB, bool EXACT>
struct SoftmaxLane {
    bool on[kBlendQ];
    float x[kBlendQ];          // d / sigma
    float w[kBlendQ];          // weights (0 for an empty slot)
    float col[kBlendQ * CB];   // colours, slot-major (C channels a slot)
    float out[CB];             // the pixel's blended colour
    float W;                   // the pixel's weight sum

    __device__ __forceinline__ void eval(const SoftmaxArgs& a, int64_t p, int sub) {
        const int C = EXACT ? CB : a.C;
        const int64_t o = p * a.K + kBlendQ * sub;
        const bool full = p < a.P && kBlendQ * (sub + 1) <= a.K;
        float z[kBlendQ];
        bool any = false;
        if (full) {
            const bi32x4 vi = *reinterpret_cast<const bi32x4*>(a.p2f + o);
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i) on[i] = vi[i] >= 0;
        } else {
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i) on[i] = p < a.P && kBlendQ * sub + i < a.K && a.p2f[o + i] >= 0;
        }
#pragma unroll
        for (int i = 0; i < kBlendQ; ++i) {
            any = any || on[i];
            z[i] = x[i] = 0.0f;
        }
#pragma unroll
        for (int c = 0; c < kBlendQ * CB; ++c) col[c] = 0.0f;
        if (any) {
            if (full) {
                const bf32x4 vz = *reinterpret_cast<const bf32x4*>(a.z + o);
                const bf32x4 vd = *reinterpret_cast<const bf32x4*>(a.d + o);
#pragma unroll
                for (int i = 0; i < kBlendQ; ++i) {
                    z[i] = vz[i];
                    x[i] = vd[i] * a.inv_sigma;
                }
                if constexpr (EXACT) {
#pragma unroll
                    for (int c = 0; c < CB; ++c) {  // 4 C words: C loads of four
                        const bf32x4 v = *reinterpret_cast<const bf32x4*>(a.col + o * CB + 4 * c);
#pragma unroll
                        for (int j = 0; j < 4; ++j) col[4 * c + j] = v[j];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < kBlendQ; ++i)
#pragma unroll
                        for (int c = 0; c < CB; ++c)
                            if (c < C) col[i * CB + c] = a.col[(o + i) * C + c];
                }
            } else {
#pragma unroll
                for (int i = 0; i < kBlendQ; ++i) {
                    if (!on[i]) continue;
                    z[i] = a.z[o + i];
                    x[i] = a.d[o + i] * a.inv_sigma;
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        if (c < C) col[i * CB + c] = a.col[(o + i) * C + c];
                }
            }
        }
        // smallest depth over the pixel's filled slots (the largest zinv); 0 when there are none
        float m = INFINITY;
#pragma unroll
        for (int i = 0; i < kBlendQ; ++i)
            if (on[i]) m = fminf(m, z[i]);
        m = blend_seg_min<L>(m);
        if (m == INFINITY) m = 0.0f;
        W = 0.0f;
#pragma unroll
        for (int c = 0; c < CB; ++c) out[c] = 0.0f;
#pragma unroll
        for (int i = 0; i < kBlendQ; ++i) {
            w[i] = 0.0f;
            if (!on[i]) continue;
            w[i] = sigmoidf(-x[i]) * expf((m - z[i]) * a.zscale);
            W += w[i];
#pragma unroll
            for (int c = 0; c < CB; ++c) out[c] = fmaf(w[i], col[i * CB + c], out[c]);
        }
        W = blend_seg_sum<L>(W);
        const float inv = W > 0.0f ? 1.0f / W : 0.0f;
#pragma unroll
        for (int c = 0; c < CB; ++c)
            if (EXACT || c < C) out[c] = blend_seg_sum<L>(out[c]) * inv;
    }
};

template <int L, int CB, bool EXACT>
__global__ __launch_bounds__(256) void softmax_fwd_kernel(SoftmaxArgs a, float* __restrict__ img) {
    constexpr int PPW = 64 / L;
    const int C = EXACT ? CB : a.C;
    const int lane = threadIdx.x & 63, sub = lane & (L - 1), grp = lane / L;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t p0 = wave * PPW; p0 < a.P; p0 += nwaves * PPW) {
        const int64_t p = p0 + grp;
        SoftmaxLane<L, CB, EXACT> s;
        s.eval(a, p, sub);
        if (sub == 0 && p < a.P) {
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (EXACT || c < C) img[p * C + c] = s.out[c];
        }
    }
}

// With G_k = sum_c g_c (c_kc - image_c) / W:
//   dL/dd_k = -G_k w_k (1 - prob_k) / sigma, dL/dz_k = -G_k w_k / (gamma (zfar - znear)),
//   dL/dc_kc = g_c w_k / W.  The max-zinv shift cancels in the normalised weights.
template <int L, int CB, bool EXACT>
__global__ __launch_bounds__(256) void softmax_bwd_kernel(SoftmaxArgs a, const float* __restrict__ gimg,
                                                          float* __restrict__ gz, float* __restrict__ gd,
                                                          float* __restrict__ gc) {
    constexpr int PPW = 64 / L;
    const int C = EXACT ? CB : a.C;
    const int lane = threadIdx.x & 63, sub = lane & (L - 1), grp = lane / L;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t p0 = wave * PPW; p0 < a.P; p0 += nwaves * PPW) {
        const int64_t p = p0 + grp;
        float g[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) g[c] = (p < a.P && (EXACT || c < C)) ? gimg[p * C + c] : 0.0f;
        SoftmaxLane<L, CB, EXACT> s;
        s.eval(a, p, sub);
        const float inv = s.W > 0.0f ? 1.0f / s.W : 0.0f;
        float od[kBlendQ], oz[kBlendQ], oc[kBlendQ * CB];
#pragma unroll
        for (int i = 0; i < kBlendQ; ++i) {
            float w = 0.0f, G = 0.0f, om = 0.0f;
            if (s.on[i] && s.W > 0.0f) {
                w = s.w[i];
                om = sigmoidf(s.x[i]);
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    if (EXACT || c < C) G = fmaf(g[c], s.col[i * CB + c] - s.out[c], G);
                G *= inv;
            }
            od[i] = -G * w * om * a.inv_sigma;
            oz[i] = -G * w * a.zscale;
#pragma unroll
            for (int c = 0; c < CB; ++c) oc[i * CB + c] = g[c] * w * inv;
        }
        const int64_t o = p * a.K + kBlendQ * sub;
        if (p < a.P && kBlendQ * (sub + 1) <= a.K) {
            if (gd) *reinterpret_cast<bf32x4*>(gd + o) = bf32x4{od[0], od[1], od[2], od[3]};
            if (gz) *reinterpret_cast<bf32x4*>(gz + o) = bf32x4{oz[0], oz[1], oz[2], oz[3]};
            if (gc) {
                if constexpr (EXACT) {
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        *reinterpret_cast<bf32x4*>(gc + o * CB + 4 * c) =
                            bf32x4{oc[4 * c], oc[4 * c + 1], oc[4 * c + 2], oc[4 * c + 3]};
                } else {
#pragma unroll
                    for (int i = 0; i < kBlendQ; ++i)
#pragma unroll
                        for (int c = 0; c < CB; ++c)
                            if (c < C) gc[(o + i) * C + c] = oc[i * CB + c];
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < kBlendQ; ++i) {
                if (!(p < a.P && kBlendQ * sub + i < a.K)) continue;
                if (gd) gd[o + i] = od[i];
                if (gz) gz[o + i] = oz[i];
                if (gc) {
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        if (EXACT || c < C) gc[(o + i) * C + c] = oc[i * CB + c];
                }
            }
        }
    }
}

static SoftmaxArgs softmax_args(const int32_t* p2f, const float* z, const float* d, const float* col, int64_t P,
                                int K, int C, float sigma, float gamma, float znear, float zfar) {
    SoftmaxArgs a;
    a.p2f = p2f;
    a.z = z;
    a.d = d;
    a.col = col;
    a.P = P;
    a.K = K;
    a.C = C;
    a.inv_sigma = 1.0f / sigma;
    a.zscale = (float)(1.0 / (((double)zfar - (double)znear) * (double)gamma));
    return a;
}

// lanes per pixel: the power of two L with 4 L >= K (K <= 64)
static int blend_lanes(int K) {
    int L = 1;
    while (kBlendQ * L < K) L <<= 1;
    return L;
}

static unsigned blend_grid(int64_t P, int L, int groups = 1) {
    const int64_t per = (int64_t)(64 / L) * groups;  // pixels a wave takes at a time
    const int64_t waves = (P + per - 1) / per;
    int64_t blocks = (waves + 3) / 4;
    if (blocks > 65536) blocks = 65536;
    return (unsigned)(blocks > 0 ? blocks : 1);
}

template <int CB, bool EXACT>
static hipError_t softmax_launch(const SoftmaxArgs& a, bool bwd, float* img, const float* gimg, float* gz, float* gd,
                                 float* gc, hipStream_t s) {
    const int L = blend_lanes(a.K);
    const dim3 grid(blend_grid(a.P, L));
#define RAST_SOFTMAX(LL)                                                                                            \
    case LL:                                                                                                        \
        if (bwd)                                                                                                    \
            hipLaunchKernelGGL((softmax_bwd_kernel<LL, CB, EXACT>), grid, dim3(256), 0, s, a, gimg, gz, gd, gc);    \
        else                                                                                                        \
            hipLaunchKernelGGL((softmax_fwd_kernel<LL, CB, EXACT>), grid, dim3(256), 0, s, a, img);                 \
        break;
    switch (L) {
        RAST_SOFTMAX(1) RAST_SOFTMAX(2) RAST_SOFTMAX(4) RAST_SOFTMAX(8) RAST_SOFTMAX(16)
        default: return hipErrorInvalidValue;
    }
#undef RAST_SOFTMAX
    return hipGetLastError();
}

// Channel counts 1 to 4 have instances of their own, whose colours move as
// 16-byte words; the others move them a word at a time, in the registers of
// eight channels (two channels that way, 2,000,000 pixels of one slot: 18 us
// forward and 29 backward, now 15 and 19).
static hipError_t softmax_dispatch(const SoftmaxArgs& a, bool bwd, float* img, const float* gimg, float* gz,
                                   float* gd, float* gc, hipStream_t s) {
    switch (a.C) {
        case 1: return softmax_launch<1, true>(a, bwd, img, gimg, gz, gd, gc, s);
        case 2: return softmax_launch<2, true>(a, bwd, img, gimg, gz, gd, gc, s);
        case 3: return softmax_launch<3, true>(a, bwd, img, gimg, gz, gd, gc, s);
        case 4: return softmax_launch<4, true>(a, bwd, img, gimg, gz, gd, gc, s);
        default: return softmax_launch<8, false>(a, bwd, img, gimg, gz, gd, gc, s);
    }
}

hipError_t launch_softmax_fwd(const int32_t* p2f, const float* z, const float* d, const float* col, int64_t P, int K,
                              int C, float sigma, float gamma, float znear, float zfar, float* img, hipStream_t s) {
    if (P == 0) return hipSuccess;
    const SoftmaxArgs a = softmax_args(p2f, z, d, col, P, K, C, sigma, gamma, znear, zfar);
    return softmax_dispatch(a, false, img, nullptr, nullptr, nullptr, nullptr, s);
}

hipError_t launch_softmax_bwd(const int32_t* p2f, const float* z, const float* d, const float* col, int64_t P, int K,
                              int C, float sigma, float gamma, float znear, float zfar, const float* gimg, float* gz,
                              float* gd, float* gc, hipStream_t s) {
    if (P == 0) return hipSuccess;
    const SoftmaxArgs a = softmax_args(p2f, z, d, col, P, K, C, sigma, gamma, znear, zfar);
    return softmax_dispatch(a, true, nullptr, gimg, gz, gd, gc, s);
}

hipError_t launch_blend_fwd(const int32_t* p2f, const float* d, int64_t P, int K, float sigma, float* alpha,
                            hipStream_t s) {
    if (P == 0) return hipSuccess;
    const int L = blend_lanes(K);
    const dim3 grid(blend_grid(P, L, kBlendU));
#define RAST_BLEND_FWD(LL) \
    case LL: hipLaunchKernelGGL(blend_fwd_kernel<LL>, grid, dim3(256), 0, s, p2f, d, P, K, 1.0f / sigma, alpha); break;
    switch (L) {
        RAST_BLEND_FWD(1) RAST_BLEND_FWD(2) RAST_BLEND_FWD(4) RAST_BLEND_FWD(8) RAST_BLEND_FWD(16)
        default: return hipErrorInvalidValue;
    }
#undef RAST_BLEND_FWD
    return hipGetLastError();
}

hipError_t launch_blend_bwd(const int32_t* p2f, const float* d, const float* ga, int64_t P, int K, float sigma,
                            float* gd, hipStream_t s) {
    if (P == 0) return hipSuccess;
    const int L = blend_lanes(K);
    const dim3 grid(blend_grid(P, L, kBlendU));
#define RAST_BLEND_BWD(LL)                                                                                       \
    case LL:                                                                                                     \
        hipLaunchKernelGGL(blend_bwd_kernel<LL>, grid, dim3(256), 0, s, p2f, d, ga, P, K, 1.0f / sigma, gd); \
        break;
    switch (L) {
        RAST_BLEND_BWD(1) RAST_BLEND_BWD(2) RAST_BLEND_BWD(4) RAST_BLEND_BWD(8) RAST_BLEND_BWD(16)
        default: return hipErrorInvalidValue;
    }
#undef RAST_BLEND_BWD
    return hipGetLastError();
}

}  // namespace rast
