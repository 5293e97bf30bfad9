// kernels_bwd.hip -- backward of the rasterizer for gfx950.
//
// The forward stores only the face ids (paper, Section 3.2: the cached
// Fragment data avoid recomputing face-pixel intersections); the backward
// recomputes barycentrics, z and the nearest edge of every filled slot and
// sums the chain rule into the nine vertex coordinates of its face.  Two
// forms.  The binned form (the forward's bins): one workgroup per cell of
// pixels, the cell's faces in LDS, FP64 sums per face (described with its
// kernels below).  The per-face form (no bins): a group of lanes scans the pixels
// of face f's blur-grown bounding box (the only pixels whose slots the
// forward can fill with f), find the slot holding f in each and sum in
// registers -- no atomics per slot; a workgroup then merges its faces'
// contributions per vertex in an LDS hash table and issues one float
// atomic per (vertex, coordinate).  Faces whose box exceeds kBigArea pixels
// are handed to a second kernel in which a whole workgroup scans one face's
// box.
//
// Derivatives (pixel p fixed, R_j = v_j - p, cross(u,v) = u.x v.y - u.y v.x):
//   e0 = cross(R1,R2), e1 = cross(R2,R0), e2 = cross(R0,R1), E = e0+e1+e2,
//   w_i = e_i / E.  With G_i = gbary_i + gzbuf * z_i and Gw = sum_i G_i w_i,
//   dL/dv_j(xy) = sum_i (G_i - Gw)/E * de_i/dv_j   (uses dE/dv = sum_i de_i/dv)
//   dL/dz_j     = gzbuf * w_j
//   dists = s d2 (s = -1 inside, +1 outside); on the nearest edge (s0, t) with
//   nearest point Q = R_s0 + u (R_t - R_s0) (relative to p):
//   d d2/d s0 = 2 (1-u) Q,  d d2/d t = 2 u Q.
#include <algorithm>

#include "../../include/rast.h"
#include "device.hpp"
#include "launch.hpp"

namespace rast {

constexpr int kBwdBlock = 256;
constexpr int kHash = 1024;     // LDS hash entries per workgroup (>= 3 * kBwdBlock)
constexpr int kBigArea = 256;   // faces with larger pixel boxes go to the cooperative kernel

struct BwdArgs {
    const float* verts;
    const int32_t* faces;
    const int64_t* first;
    const int64_t* nf;
    const int32_t* p2f;
    const float* gz;
    const float* gb;
    const float* gd;
    float* grad;
    int* hdr;
    int* big;      // list of faces with large boxes
    int64_t V, F;
    int N, H, W, K;
    float rb;      // sqrt(blur_radius)
    int opts;      // rasterizer options (kOpt*)
    // binned form
    const FaceRec* recs;
    const int* counts;
    const int* lists;
    float* partial;    // (F, 4, 9): a face's nine coordinate sums in the i-th cell of its range
    unsigned char* pmask;  // (F, 4): partial row written by this call (the binned form; shares big's memory)
    int bs, nby, nbx, M;
    int* crowded;          // cells left to the second kernel (shares the forward's tile order's memory)
    float inv_k;           // 1 / K
    int lgw, lgh;          // the binned form's cells: log2 of their width and height in pixels
    int ncy, ncx;          // rows and columns of cells per image
    int max_rep;           // log2 of the rows of sums per face at most (replicas)
    int cross;             // the bins are not a multiple of the cells: a cell touches up to four
    int reuse;         // records and bins come from the forward: check its signature first
    BinSig sig;        // the signature this call expects
};

// False (and the status flagged) when a backward that reuses the forward's
// bins finds another call's signature in the workspace.  Every thread of a
// workgroup reads the same words, so the answer is uniform.
__device__ __forceinline__ bool bins_usable(const BwdArgs& a) {
    if (!a.reuse) return true;
    bool same = true;
#pragma unroll
    for (int i = 0; i < kSigWords; ++i) same = same && (a.hdr[kHdrSig + i] == a.sig.w[i]);
    if (!same && threadIdx.x == 0) atomicOr(&a.hdr[kHdrStatus], kStatReuse);
    return same;
}

struct FaceGrad {
    float gx[3], gy[3], gzv[3];
};

// Upstream gradients of slot s (zero for an absent array).  They and the
// slots' face ids are read once, so the binned pass loads them non-temporally
// (the "nt" hint), leaving L2 to the face records that neighbouring bins share.
struct SlotUp {
    float gz, gb0, gb1, gb2, gd;
};
__device__ __forceinline__ SlotUp load_up(const BwdArgs& a, int64_t s) {
    SlotUp u;
    u.gz = a.gz ? __builtin_nontemporal_load(a.gz + s) : 0.0f;
    u.gb0 = u.gb1 = u.gb2 = 0.0f;
    if (a.gb) {
        u.gb0 = __builtin_nontemporal_load(a.gb + 3 * s + 0);
        u.gb1 = __builtin_nontemporal_load(a.gb + 3 * s + 1);
        u.gb2 = __builtin_nontemporal_load(a.gb + 3 * s + 2);
    }
    u.gd = a.gd ? __builtin_nontemporal_load(a.gd + s) : 0.0f;
    return u;
}

// Adds the contribution of a slot of face R at pixel p, with upstream gradients up, to g.
// kOpts = false compiles out the options' barycentrics (for calls without them).
template <class Rec, bool kOpts = true>
__device__ __forceinline__ void slot_grad_up(const BwdArgs& a, const Rec& R, const float (&vz)[3], const Pix& p,
                                             const SlotUp& up, FaceGrad& g) {
    Eval ev;
    eval_full(R, p, ev);
    const float gzs = up.gz, gb0 = up.gb0, gb1 = up.gb1, gb2 = up.gb2, gds = up.gd;
    // dL/dw for the output barycentrics; z = sum_i w_i z_i adds gz z_i
    float G0 = gb0 + gzs * vz[0];
    float G1 = gb1 + gzs * vz[1];
    float G2 = gb2 + gzs * vz[2];
    if (kOpts && (a.opts & (kOptPersp | kOptClip))) {
        // the outputs are the options' barycentrics: carry dL/dw back through
        // the clipping and the correction to the raw ones (and to the depths)
        const float w[3] = {ev.w0, ev.w1, ev.w2};
        float wp[3] = {w[0], w[1], w[2]}, D = 1.0f;
        if (a.opts & kOptPersp) {
            const float u0 = w[0] / vz[0], u1 = w[1] / vz[1], u2 = w[2] / vz[2];
            D = u0 + u1 + u2;
            wp[0] = u0 / D;
            wp[1] = u1 / D;
            wp[2] = u2 / D;
        }
        float wf[3] = {wp[0], wp[1], wp[2]}, M = 1.0f;
        if (a.opts & kOptClip) {
            const float m0 = fmaxf(wp[0], 0.0f), m1 = fmaxf(wp[1], 0.0f), m2 = fmaxf(wp[2], 0.0f);
            M = m0 + m1 + m2;
            wf[0] = m0 / M;
            wf[1] = m1 / M;
            wf[2] = m2 / M;
        }
        g.gzv[0] += gzs * wf[0];
        g.gzv[1] += gzs * wf[1];
        g.gzv[2] += gzs * wf[2];
        if (a.opts & kOptClip) {
            const float S = G0 * wf[0] + G1 * wf[1] + G2 * wf[2];
            G0 = wp[0] > 0.0f ? (G0 - S) / M : 0.0f;
            G1 = wp[1] > 0.0f ? (G1 - S) / M : 0.0f;
            G2 = wp[2] > 0.0f ? (G2 - S) / M : 0.0f;
        }
        if (a.opts & kOptPersp) {
            const float S = G0 * wp[0] + G1 * wp[1] + G2 * wp[2];
            const float q0 = (G0 - S) / D, q1 = (G1 - S) / D, q2 = (G2 - S) / D;
            G0 = q0 / vz[0];
            G1 = q1 / vz[1];
            G2 = q2 / vz[2];
            g.gzv[0] -= q0 * w[0] / (vz[0] * vz[0]);
            g.gzv[1] -= q1 * w[1] / (vz[1] * vz[1]);
            g.gzv[2] -= q2 * w[2] / (vz[2] * vz[2]);
        }
    } else {
        g.gzv[0] += gzs * ev.w0;
        g.gzv[1] += gzs * ev.w1;
        g.gzv[2] += gzs * ev.w2;
    }
    float Gw = G0 * ev.w0 + G1 * ev.w1 + G2 * ev.w2;
    float invE = R.invE;
    float H0 = (G0 - Gw) * invE, H1 = (G1 - Gw) * invE, H2 = (G2 - Gw) * invE;
    // vertex positions relative to the pixel
    float Rx[3], Ry[3];
    Rx[0] = -ev.sx;
    Ry[0] = -ev.sy;
    Rx[1] = Rx[0] + (float)R.ab.x;
    Ry[1] = Ry[0] + (float)R.ab.y;
    Rx[2] = Rx[0] + (float)R.ac.x;
    Ry[2] = Ry[0] + (float)R.ac.y;
    // de0/dR1 = (R2.y, -R2.x), de0/dR2 = (-R1.y, R1.x)
    // de1/dR2 = (R0.y, -R0.x), de1/dR0 = (-R2.y, R2.x)
    // de2/dR0 = (R1.y, -R1.x), de2/dR1 = (-R0.y, R0.x)
    g.gx[0] += H1 * (-Ry[2]) + H2 * Ry[1];
    g.gy[0] += H1 * Rx[2] + H2 * (-Rx[1]);
    g.gx[1] += H0 * Ry[2] + H2 * (-Ry[0]);
    g.gy[1] += H0 * (-Rx[2]) + H2 * Rx[0];
    g.gx[2] += H0 * (-Ry[1]) + H1 * Ry[0];
    g.gy[2] += H0 * Rx[1] + H1 * (-Rx[0]);
    if (gds != 0.0f) {
        int e = ev.edge;
        int js = e, jt = e == 2 ? 0 : e + 1;
        float u = ev.u;
        float Rsx = js == 0 ? Rx[0] : (js == 1 ? Rx[1] : Rx[2]);
        float Rsy = js == 0 ? Ry[0] : (js == 1 ? Ry[1] : Ry[2]);
        float Rtx = jt == 0 ? Rx[0] : (jt == 1 ? Rx[1] : Rx[2]);
        float Rty = jt == 0 ? Ry[0] : (jt == 1 ? Ry[1] : Ry[2]);
        float Qx = Rsx + u * (Rtx - Rsx);
        float Qy = Rsy + u * (Rty - Rsy);
        float sg = ev.inside ? -gds : gds;
        float cs = 2.0f * (1.0f - u) * sg, ct = 2.0f * u * sg;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            float k = (j == js) ? cs : ((j == jt) ? ct : 0.0f);
            g.gx[j] += k * Qx;
            g.gy[j] += k * Qy;
        }
    }
}

template <class Rec, bool kOpts = true>
__device__ __forceinline__ void slot_grad(const BwdArgs& a, const Rec& R, const float (&vz)[3], const Pix& p,
                                          int64_t s, FaceGrad& g) {
    slot_grad_up<Rec, kOpts>(a, R, vz, p, load_up(a, s), g);
}

// Scans the K slots of pixel (n, r, c) for face f and accumulates every match.
__device__ __forceinline__ void scan_pixel(const BwdArgs& a, const FaceRec& R, const float (&vz)[3], int f, int n,
                                           int r, int c, FaceGrad& g) {
    const int64_t pix = ((int64_t)n * a.H + r) * a.W + c;
    const int32_t* row = a.p2f + pix * a.K;
    int first_k = -1;
    bool more = false;
    if ((a.K & 3) == 0) {
        const int4* row4 = reinterpret_cast<const int4*>(row);
        for (int k = 0; k < a.K; k += 4) {
            int4 v = row4[k >> 2];
            int h = (int)(v.x == f) + (int)(v.y == f) + (int)(v.z == f) + (int)(v.w == f);
            if (h > 0) {
                int hit = v.x == f ? 0 : (v.y == f ? 1 : (v.z == f ? 2 : 3));
                more = more || first_k >= 0 || h > 1;
                if (first_k < 0) first_k = k + hit;
            }
        }
    } else {
        for (int k = 0; k < a.K; ++k) {
            if (row[k] == f) {
                more = more || first_k >= 0;
                if (first_k < 0) first_k = k;
            }
        }
    }
    if (first_k < 0) return;
    Pix p = make_pix(r, c, a.H, a.W);
    slot_grad(a, R, vz, p, pix * a.K + first_k, g);
    if (more) {
        // the same face in several slots of one pixel cannot come from the
        // forward, but every slot is still honoured
        for (int kk = first_k + 1; kk < a.K; ++kk)
            if (row[kk] == f) slot_grad(a, R, vz, p, pix * a.K + kk, g);
    }
}

// Face f's record (with its pixel ranges), its vertex ids and depths.
__device__ __forceinline__ bool load_face(const BwdArgs& a, int64_t f, FaceRec& R, int (&vi)[3], float (&vz)[3],
                                          int& n) {
    vi[0] = a.faces[3 * f];
    vi[1] = a.faces[3 * f + 1];
    vi[2] = a.faces[3 * f + 2];
    if (vi[0] < 0 || vi[0] >= a.V || vi[1] < 0 || vi[1] >= a.V || vi[2] < 0 || vi[2] >= a.V) {
        vi[0] = vi[1] = vi[2] = -1;
        return false;
    }
    n = find_mesh(a.first, a.nf, a.N, f);
    if (n < 0) return false;
    const float* P0 = a.verts + 3 * (int64_t)vi[0];
    const float* P1 = a.verts + 3 * (int64_t)vi[1];
    const float* P2 = a.verts + 3 * (int64_t)vi[2];
    R = make_rec(P0[0], P0[1], P0[2], P1[0], P1[1], P1[2], P2[0], P2[1], P2[2], a.rb, a.H, a.W, n,
                 a.opts);
    vz[0] = P0[2];
    vz[1] = P1[2];
    vz[2] = P2[2];
    return R.ok();
}

// Sixteen consecutive vertices keep their order in the table (the faces of a
// workgroup mostly share runs of vertices), so that the flush's atomics of
// neighbouring lanes fall into the same lines.
__device__ __forceinline__ uint32_t vhash(int v) {
    return (((((uint32_t)v >> 4) * 2654435761u) >> (32 - 6)) << 4) | ((uint32_t)v & 15u);
}
static_assert(kHash == 1 << 10, "vhash yields 10 bits");
// A run that meets another's entries goes on in the next run's, and a step that
// is odd visits the whole table: by single entries such runs walked through each
// other up to sixteen entries a vertex (40,960 faces, 8 meshes: the face sum 11.7
// us, 8.6 before vertices were kept in runs, now 6.5).
constexpr int kHashStep = 17;

// Merges (vertex, grad3) into the workgroup's LDS table; falls back to a global
// atomic when the table is full.  The sums are FP64: LDS has FP64 atomics in
// hardware, FP32 ones are a compare-and-swap loop (measured over random words:
// 2.66 ms for 537 M FP32 adds, 0.29 ms for as many FP64 ones).
__device__ __forceinline__ void lds_add(int* keys, double* vals, float* grad, int v, float x, float y, float z) {
    uint32_t h = vhash(v);
    for (int probe = 0; probe < kHash; ++probe) {
        int prev = atomicCAS(&keys[h], -1, v);
        if (prev == -1 || prev == v) {
            atomicAdd(&vals[3 * h + 0], (double)x);
            atomicAdd(&vals[3 * h + 1], (double)y);
            atomicAdd(&vals[3 * h + 2], (double)z);
            return;
        }
        h = (h + kHashStep) & (kHash - 1);
    }
    atomicAdd(grad + 3 * (int64_t)v + 0, x);
    atomicAdd(grad + 3 * (int64_t)v + 1, y);
    atomicAdd(grad + 3 * (int64_t)v + 2, z);
}

__device__ __forceinline__ void clear_table(int* keys, double* vals) {
    for (int i = threadIdx.x; i < kHash; i += kBwdBlock) keys[i] = -1;
    for (int i = threadIdx.x; i < 3 * kHash; i += kBwdBlock) vals[i] = 0.0;
}

// Adds the table to grad_verts: one atomic per (vertex, coordinate), lanes
// running over the words of the table's rows, so that the atomics of a wave
// fall into few lines (three adds per lane, a row apart each, cost 2.6 times
// as much: 0.50 against 0.19 ms for 10 M adds to random rows).
__device__ __forceinline__ void flush_table(float* grad, const int* keys, const double* vals) {
    for (int i = threadIdx.x; i < 3 * kHash; i += kBwdBlock) {
        const int h = (int)((uint32_t)i / 3u);
        const int v = keys[h];
        if (v >= 0) atomicAdd(grad + 3 * (int64_t)v + (i - 3 * h), (float)vals[i]);
    }
}

// A face's box is scanned by kLanes lanes side by side (consecutive pixels of
// a row: consecutive id lists), whose sums meet in a butterfly; a group of
// lanes takes `per` faces in turn, a workgroup 256 / kLanes * per of them, and
// `per` is chosen so that small meshes still fill the chip.  Bound by the
// latency of the id lists' reads where boxes are large or faces few, by the
// faces' records, which every lane of a group builds, where boxes are small:
// four lanes there, else sixteen (launch_backward has the rule).  With one lane
// per face 2,880 faces were 12 workgroups and each lane walked its 80 or so
// pixels alone: 330 us, now 26 (three meshes of up to 1,280 faces, 130 x 75
// pixels, K = 5).
constexpr int64_t kManyFaces = 16384;
constexpr int kFaceMax = kBwdBlock;  // faces of a workgroup at most: their 3 x 256 vertices fit the table
static_assert(3 * kFaceMax <= kHash, "a workgroup's vertices fit its table");

template <int kLanes>
__global__ __launch_bounds__(kBwdBlock) void bwd_faces_kernel(BwdArgs a, int per) {
    constexpr int kGroups = kBwdBlock / kLanes;
    __shared__ int keys[kHash];
    __shared__ double vals[3 * kHash];
    clear_table(keys, vals);
    __syncthreads();
    const int sub = threadIdx.x & (kLanes - 1), grp = threadIdx.x / kLanes;
    for (int it = 0; it < per; ++it) {
        const int64_t f = ((int64_t)blockIdx.x * per + it) * kGroups + grp;
        FaceRec R;
        int vi[3];
        float vz[3];
        int n;
        if (f >= a.F || !load_face(a, f, R, vi, vz, n)) continue;  // (uniform over the group)
        const int c0 = R.px.x, c1 = R.px.y, r0 = R.px.z, r1 = R.px.w;
        if (c1 < c0 || r1 < r0) continue;
        const int w = c1 - c0 + 1;
        const int64_t area = (int64_t)w * (r1 - r0 + 1);
        if (area > kBigArea) {
            if (sub == 0) a.big[atomicAdd(&a.hdr[kHdrBigCount], 1)] = (int)f;
            continue;
        }
        FaceGrad g;
#pragma unroll
        for (int j = 0; j < 3; ++j) g.gx[j] = g.gy[j] = g.gzv[j] = 0.0f;
        const float inv_w = 1.0f / (float)w;
        for (int q = sub; q < (int)area; q += kLanes) {
            const int dr = stage_pixel(q, inv_w);  // q / w (q <= kBigArea: the estimate is exact)
            scan_pixel(a, R, vz, (int)f, n, r0 + dr, c0 + q - dr * w, g);
        }
#pragma unroll
        for (int o = kLanes / 2; o > 0; o >>= 1) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                g.gx[j] += __shfl_xor(g.gx[j], o, kLanes);
                g.gy[j] += __shfl_xor(g.gy[j], o, kLanes);
                g.gzv[j] += __shfl_xor(g.gzv[j], o, kLanes);
            }
        }
        if (sub < 3) {
            const int v = sub == 0 ? vi[0] : (sub == 1 ? vi[1] : vi[2]);
            const float x = sub == 0 ? g.gx[0] : (sub == 1 ? g.gx[1] : g.gx[2]);
            const float y = sub == 0 ? g.gy[0] : (sub == 1 ? g.gy[1] : g.gy[2]);
            const float z = sub == 0 ? g.gzv[0] : (sub == 1 ? g.gzv[1] : g.gzv[2]);
            lds_add(keys, vals, a.grad, v, x, y, z);
        }
    }
    __syncthreads();
    flush_table(a.grad, keys, vals);
}

// Faces with large boxes: each workgroup takes the next listed face and its
// 256 threads share the pixel scan; the nine sums are reduced in LDS.  Every
// workgroup leaves once the list is exhausted.
__global__ __launch_bounds__(kBwdBlock) void bwd_big_faces_kernel(BwdArgs a) {
    __shared__ float red[9][kBwdBlock / 64];
    __shared__ int item_s;
    const int count = a.hdr[kHdrBigCount];
    for (;;) {
        if (threadIdx.x == 0) item_s = atomicAdd(&a.hdr[kHdrBigNext], 1);
        __syncthreads();
        const int item = item_s;
        __syncthreads();
        if (item >= count) break;
        const int f = a.big[item];
        FaceRec R;
        int vi[3] = {-1, -1, -1};
        float vz[3];
        int n;
        FaceGrad g;
#pragma unroll
        for (int j = 0; j < 3; ++j) g.gx[j] = g.gy[j] = g.gzv[j] = 0.0f;
        bool ok = load_face(a, f, R, vi, vz, n);
        if (ok) {
            const int c0 = R.px.x, c1 = R.px.y, r0 = R.px.z, r1 = R.px.w;
            const int w = c1 - c0 + 1;
            const int64_t area = (c1 >= c0 && r1 >= r0) ? (int64_t)w * (r1 - r0 + 1) : 0;
            for (int64_t q = threadIdx.x; q < area; q += kBwdBlock) {
                int r = r0 + (int)(q / w), c = c0 + (int)(q % w);
                scan_pixel(a, R, vz, f, n, r, c, g);
            }
        }
        float t[9] = {g.gx[0], g.gy[0], g.gzv[0], g.gx[1], g.gy[1], g.gzv[1], g.gx[2], g.gy[2], g.gzv[2]};
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            float v = t[j];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if ((threadIdx.x & 63) == 0) red[j][threadIdx.x >> 6] = v;
        }
        __syncthreads();
        if (threadIdx.x < 9 && ok) {
            float s = 0.0f;
            for (int w4 = 0; w4 < kBwdBlock / 64; ++w4) s += red[threadIdx.x][w4];
            int j = threadIdx.x / 3, x = threadIdx.x % 3;
            atomicAdd(a.grad + 3 * (int64_t)vi[j] + x, s);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Binned form.  Pass 1: one workgroup per cell of pixels reads the slots of
// the cell's pixels (coalesced reads of pix_to_face and the gradients), maps
// each slot's face to a chunk index through an LDS hash table, and accumulates
// the nine coordinate sums per face in LDS in FP64.  LDS adds FP64 in
// hardware (FP32 adds are a compare-and-swap loop: 2.3 ms for the pass at
// 4 x 1024 x 1024 pixels, K = 16), and an FP64 sum of FP32 terms needs no scale
// and no range: 64-bit fixed point cost three more instructions a term, a
// range check a slot, a recorded maximum and a second launch for gradients too
// small for the grid.  A face's nine sums from a cell go to its own row
// partial[f][i] for the i-th cell of its range (no global atomic), and the
// row's byte in an (F, 4) mask is set.  Pass 2: the rows that the mask names
// are added per face and merged per vertex in LDS; one float atomic per
// (vertex, coordinate) per workgroup.  Faces spanning more than four cells
// go to grad_verts directly.
//
// Cells are 8, 16 or 32 pixels wide and high: the largest whose slots the
// workgroup holds at once (1,024) and that divides the bins, or, for bins that
// are an odd multiple of 8, that is no larger than a bin (such a cell reaches
// into up to four bins).  Larger bins as cells had their slots scanned once per
// 160 listed faces, on too few workgroups; cells of 8 in bins of 24 were four
// times the workgroups (4 x 578 x 706 pixels, K = 1, backward: 83 us, now 42).
// ---------------------------------------------------------------------------
constexpr int kP1Threads = 256;
constexpr int kP1Chunk = 160;    // faces staged in LDS per pass over a cell's slots
constexpr int kP1Rows = 184;     // rows of sums in LDS (at least kP1Chunk)
constexpr int kP1Table = 512;    // LDS hash entries (>= 2 * kP1Chunk)
constexpr int kP1Probe = 64;     // entries probed before a cell is left to the listed way
constexpr int kP1Unroll = 4;     // slots per thread in one group of the cell's slots
constexpr int kP1Group = kP1Unroll * kP1Threads;  // slots the workgroup holds at once
constexpr int kAgainGrid = 1024;  // workgroups that walk the crowded cells
constexpr int kMaxPartials = 4;  // (the row masks are read as one uchar4)

__device__ __forceinline__ uint32_t fhash(int f) { return ((uint32_t)f * 2654435761u) >> (32 - 9); }
static_assert(kP1Table == 512, "fhash yields 9 bits");

// A face as the slot recomputation reads it (FaceRec without the mesh id and
// the pixel ranges).
struct SlotRec {
    double2 pa, ab, ac;
    double E;
    float az, dz1, dz2, invE, il0, il1, il2;
    int face;  // the face's id
};

// A chunk's faces in LDS, 64 bytes each as four arrays of 16-byte words (one
// face's words a power of two apart would fall into few banks).  The vertices
// are kept as the FP32 coordinates they are; the FP64 offsets from vertex a
// are exact differences of them and come back bit for bit.
struct ChunkRecs {
    float4 q[4][kP1Chunk];
    __device__ __forceinline__ void put(int j, const FaceRec& R, int f) {
        const double bx = R.pa.x + R.ab.x, by = R.pa.y + R.ab.y, cx = R.pa.x + R.ac.x, cy = R.pa.y + R.ac.y;
        q[0][j] = make_float4((float)R.pa.x, (float)R.pa.y, (float)bx, (float)by);
        q[1][j] = make_float4((float)cx, (float)cy, __int_as_float(__double2loint(R.E)),
                              __int_as_float(__double2hiint(R.E)));
        q[2][j] = make_float4(R.az, R.dz1, R.dz2, R.invE);
        q[3][j] = make_float4(R.il0, R.il1, R.il2, __int_as_float(f));
    }
    __device__ __forceinline__ int face(int j) const { return __float_as_int(q[3][j].w); }
    __device__ __forceinline__ SlotRec get(int j) const {
        const float4 u = q[0][j], v = q[1][j], w = q[2][j], x = q[3][j];
        SlotRec R;
        R.pa = make_double2(u.x, u.y);
        R.ab = make_double2((double)u.z - R.pa.x, (double)u.w - R.pa.y);
        R.ac = make_double2((double)v.x - R.pa.x, (double)v.y - R.pa.y);
        R.E = __hiloint2double(__float_as_int(v.w), __float_as_int(v.z));
        R.az = w.x;
        R.dz1 = w.y;
        R.dz2 = w.z;
        R.invE = w.w;
        R.il0 = x.x;
        R.il1 = x.y;
        R.il2 = x.z;
        R.face = __float_as_int(x.w);
        return R;
    }
};

// Slot q of a cell in its slot order (pixel-major, k fastest): row, column
// and slot within the pixel.  A cell has at most 4,096 slots (64 pixels of K =
// 64), for which the quotients by a float reciprocal are exact.
struct SlotPlace {
    int k, pr, pc;
    __device__ __forceinline__ SlotPlace(int q, int K, int cols, float inv_k, float inv_cols) {
        const int pl = stage_pixel(q, inv_k);
        k = q - pl * K;
        pr = stage_pixel(pl, inv_cols);
        pc = pl - pr * cols;
    }
};

// The nine coordinate terms of one slot of face R at pixel (row, col), added
// to a row of its sums.
template <bool kOpts>
__device__ __forceinline__ void add_slot(const BwdArgs& a, const SlotRec& R, int row, int col, double dW, double rW,
                                         double dH, double rH, const SlotUp& up, double* acc) {
    const float vz[3] = {R.az, R.az + R.dz1, R.az + R.dz2};
    FaceGrad g;
#pragma unroll
    for (int jj = 0; jj < 3; ++jj) g.gx[jj] = g.gy[jj] = g.gzv[jj] = 0.0f;
    Pix p;
    p.x = pix_coord_rcp(col, dW, rW);
    p.y = pix_coord_rcp(row, dH, rH);
    slot_grad_up<SlotRec, kOpts>(a, R, vz, p, up, g);
    const float g9[9] = {g.gx[0], g.gy[0], g.gzv[0], g.gx[1], g.gy[1], g.gzv[1], g.gx[2], g.gy[2], g.gzv[2]};
#pragma unroll
    for (int x = 0; x < 9; ++x) atomicAdd(&acc[x], (double)g9[x]);
}

// Where face f's sums from cell (cx, cy) go: its partial row f * 4 + i (i the
// cell's place in the face's range), -1 (to the vertices: the range spans more
// than kMaxPartials cells) or -2 (nowhere: the face never counts, or the cell
// lies outside its range).
__device__ __forceinline__ int partial_row(const BwdArgs& a, const FaceRec& G, int f, int cx, int cy) {
    if (!G.ok() || G.px.y < G.px.x || G.px.w < G.px.z) return -2;
    const int cx0 = G.px.x >> a.lgw, cx1 = G.px.y >> a.lgw, cy0 = G.px.z >> a.lgh, cy1 = G.px.w >> a.lgh;
    const int64_t nc = (int64_t)(cx1 - cx0 + 1) * (cy1 - cy0 + 1);
    if (nc > kMaxPartials) return -1;
    if (cx < cx0 || cx > cx1 || cy < cy0 || cy > cy1) return -2;
    return f * kMaxPartials + (cy - cy0) * (cx1 - cx0 + 1) + (cx - cx0);
}

// The LDS of a cell's workgroup.
struct CellLds {
    ChunkRecs rec;
    double acc[kP1Rows * 9];  // a face's sums, in replicas() rows
    int key[kP1Table];   // face ids (-1: free)
    unsigned char val[kP1Table];  // the key's chunk index
    int dst[kP1Chunk];            // partial_row of each chunk face
    int count, fail;
};
static_assert(kP1Chunk <= 256, "chunk indices are bytes");
static_assert(sizeof(CellLds) <= 21 * 1280, "six workgroups share a compute unit's LDS");

// Lanes that add to one LDS word go one after the other (64 lanes on one
// FP64 word: 64 times as long as on 64 words), and neighbouring pixels name
// the same faces, the more so the larger the faces are and the fewer a cell
// names.  So a chunk of m faces has as many rows per face as there is room for,
// 1 << replicas(m) of them, and a slot adds to the one of its pixel's column.
// But no more than the pixels that a wave holds need (64 / K of them, of which
// a face is in part): a row is cleared and summed whether it is used or not.
// Four meshes of 1,280 faces, 578 x 706 pixels, backward, bins of 16, for eight /
// four / two / one row at most: K = 1 38 / 39 / 45 / 55 us, K = 4 60 / 58 / 62 / 76, K =
// 8 113 / 97 / 92 / 97, K = 16 217 / 178 / 164 / 156; 4 of 327,680 at 1024 x 1024, K =
// 16 650 / 648 / 652 / 604.
// (kOne: the call has one row per face, known to the compiler)
template <bool kOne>
__device__ __forceinline__ int replicas(const BwdArgs& a, int m) {
    if (kOne) return 0;
    const int room = 8 * m <= kP1Rows ? 3 : (4 * m <= kP1Rows ? 2 : (2 * m <= kP1Rows ? 1 : 0));
    return min(room, a.max_rep);
}

// Coordinate sum x of face j of a chunk (over its rows).
__device__ __forceinline__ double face_sum(const CellLds& L, int j, int rep, int x) {
    double v = L.acc[9 * (j << rep) + x];
    for (int i = 1; i < 1 << rep; ++i) v += L.acc[9 * ((j << rep) + i) + x];
    return v;
}

// Writes the sums of the chunk's m faces, lanes running over a face's nine
// words, to their partial rows, and marks those; the sums of a face without
// rows go to its vertices, three neighbouring atomics each.
template <bool kOne>
__device__ __forceinline__ void flush_faces(const BwdArgs& a, const CellLds& L, int m) {
    const int rep = replicas<kOne>(a, m);
    for (int i = threadIdx.x; i < 9 * m; i += kP1Threads) {
        const int j = stage_pixel(i, 1.0f / 9.0f), x = i - 9 * j;
        const int dst = L.dst[j];
        if (dst == -2) continue;
        const float v = (float)face_sum(L, j, rep, x);
        if (dst >= 0) {
            a.partial[(int64_t)dst * 9 + x] = v;
            if (x == 0) a.pmask[dst] = 1;
        } else if (v != 0.0f) {
            const int c = x >= 6 ? 2 : (x >= 3 ? 1 : 0);
            const int vtx = a.faces[3 * (int64_t)L.rec.face(j) + c];
            if (vtx >= 0 && vtx < a.V) atomicAdd(a.grad + 3 * (int64_t)vtx + x - 3 * c, v);
        }
    }
}

// A slot's face into the table; the lane that inserts a face numbers it.
__device__ __forceinline__ void name_face(CellLds& L, int f) {
    uint32_t h = fhash(f);
    for (int probe = 0; probe < kP1Probe; ++probe) {
        const int prev = atomicCAS(&L.key[h], -1, f);
        if (prev == f) return;
        if (prev == -1) {
            const int j = atomicAdd(&L.count, 1);
            L.val[h] = (unsigned char)min(j, kP1Chunk - 1);  // (more than kP1Chunk: not read)
            return;
        }
        h = (h + 1) & (kP1Table - 1);
    }
    L.fail = 1;  // (a crowded table: the listed way takes the cell)
}

__device__ __forceinline__ double* acc_row(CellLds& L, int j, int col, int rep) {
    return &L.acc[9 * ((j << rep) + (col & ((1 << rep) - 1)))];
}

// Chunk index of face f, or -1.
__device__ __forceinline__ int find_face(const CellLds& L, int f) {
    uint32_t h = fhash(f);
    for (int probe = 0; probe < kP1Table; ++probe) {
        const int key = L.key[h];
        if (key == f) return L.val[h];
        if (key == -1) return -1;
        h = (h + 1) & (kP1Table - 1);
    }
    return -1;
}

// Records of the table's faces, one thread per entry, and where their sums
// go; zeroed sums.  A face of another image or one that never counts is marked
// by its id.
template <bool kOne>
__device__ __forceinline__ void gather_named(const BwdArgs& a, CellLds& L, int n, int cx, int cy, int m) {
    for (int i = threadIdx.x; i < 9 * (m << replicas<kOne>(a, m)); i += kP1Threads) L.acc[i] = 0.0;
    for (int i = threadIdx.x; i < kP1Table; i += kP1Threads) {
        const int f = L.key[i];
        if (f < 0) continue;
        const int j = L.val[i];
        const FaceRec& G = a.recs[f];
        const bool ok = G.ok() && G.mesh() == n;
        L.rec.put(j, G, ok ? f : -1);
        L.dst[j] = ok ? partial_row(a, G, f, cx, cy) : -2;
    }
}

// A cell's place: slot (pr, pc, k) is pix_to_face[sbase + (pr * W + pc) * K + k].
struct CellGeo {
    int n, cx, cy, r0, c0, cols, nslots;
    float inv_cols;
    int64_t sbase;
    int64_t bin;   // the forward's bin of the cell's first pixel
    int bx, by;    // its column and row
    int nbx, nby;  // columns and rows of bins that the cell touches
    __device__ __forceinline__ CellGeo(const BwdArgs& a, int64_t cell) {
        const int per_img = a.ncy * a.ncx;
        n = (int)(cell / per_img);
        const int rem = (int)(cell - (int64_t)n * per_img);
        cy = rem / a.ncx;
        cx = rem - cy * a.ncx;
        r0 = cy << a.lgh;
        c0 = cx << a.lgw;
        cols = min(1 << a.lgw, a.W - c0);
        const int rows = min(1 << a.lgh, a.H - r0);
        nslots = rows * cols * a.K;
        inv_cols = 1.0f / (float)cols;
        sbase = (((int64_t)n * a.H + r0) * a.W + c0) * a.K;
        by = r0 / a.bs;
        bx = c0 / a.bs;
        bin = ((int64_t)n * a.nby + by) * a.nbx + bx;
        nbx = nby = 1;
        if (a.cross) {  // (uniform)
            nby += (r0 + rows - 1) / a.bs - by;
            nbx += (c0 + cols - 1) / a.bs - bx;
        }
    }
    // No face reaches the cell's bins.
    __device__ __forceinline__ bool empty(const BwdArgs& a) const {
        int any = a.counts[bin];
        if (a.cross)
            for (int i = 1; i < nbx * nby; ++i) any |= a.counts[bin + (int64_t)(i / nbx) * a.nbx + i % nbx];
        return any == 0;
    }
};

// Ways through a cell.  The direct way (its slots name at most kP1Chunk
// distinct faces, nearly every cell): the distinct ids go into the LDS hash
// table as they arrive, only those faces' records are gathered, and every slot
// is recomputed once.  A crowded cell (silhouettes) then costs no more than a
// quiet one, and no list is read.  Slot ids outside [0, F), of a face that
// never counts or of another image are ignored.  The listed way (any other
// cell): the lists of the cell's bins are taken in chunks of kP1Chunk faces, each
// chunk's records and hash table built, and every slot of the cell looked up
// in it; a face listed in several of the bins counts in the first of them.
//
// This kernel takes cells of at most kP1Group slots the direct way, ids and
// gradients in registers, the gradients in flight while the records are
// gathered, and leaves the others to bwd_cells_again_kernel, whose code would
// cost it registers.  kOpts: the call has perspective-correct or clipped
// barycentrics (an instance of its own, so that their register needs do not
// lower the occupancy of the plain one); kOne: one row of sums per face.
//
// Bound by latency and vector issue about alike: two dependent round trips
// per cell (ids, then records; ids, then gradients), overlapped by the six
// workgroups per compute unit that the LDS block (26.6 KB) allows and that the
// registers (80) are held to, at the price of a few spilled (20 bytes a lane, 24
// with options, none without options where kOne holds); with five of each the
// kernel took 711 us instead of 681 (4 x 1024 x 1024 pixels, K = 16; by one row of
// sums a face and a cheaper hash step since then 520) and 448 instead of 419 (32 x
// 512 x 512, K = 8).  The whole backward, replayed: 895 -> 609 us (K = 16), 430 ->
// 401 (K = 8, bins of 16 pixels), 53 -> 51 (8 x 256 x 256, K = 8, bins of 16) and 80
// -> 41 (K = 4, bins of 32), against bins as cells with fixed-point sums and a
// second, rescue pass.
template <bool kOpts, bool kOne>
__global__ __launch_bounds__(kP1Threads) __attribute__((amdgpu_waves_per_eu(6, 8)))
void bwd_cells_kernel(BwdArgs a) {
    __shared__ CellLds L;
    if (!bins_usable(a)) return;
    // each XCD takes a contiguous range of cells (neighbouring cells gather
    // mostly the same face records)
    const int64_t cell = xcd_item(blockIdx.x, (int64_t)a.N * a.ncy * a.ncx);
    const CellGeo c(a, cell);
    if (c.empty(a)) return;  // no slot to read
    const double dW = (double)a.W, dH = (double)a.H, rW = 1.0 / dW, rH = 1.0 / dH;
    const int t = threadIdx.x;
    int fq[kP1Unroll], rq[kP1Unroll], cq[kP1Unroll];
    int64_t sq[kP1Unroll];
#pragma unroll
    for (int u = 0; u < kP1Unroll; ++u) {
        const int q = u * kP1Threads + t;
        const SlotPlace w(q, a.K, c.cols, a.inv_k, c.inv_cols);
        rq[u] = c.r0 + w.pr;
        cq[u] = c.c0 + w.pc;
        sq[u] = c.sbase + (int64_t)(w.pr * a.W + w.pc) * a.K + w.k;
        int f = -1;
        if (q < c.nslots) f = __builtin_nontemporal_load(a.p2f + sq[u]);
        fq[u] = (f >= 0 && f < a.F) ? f : -1;
    }
    for (int i = t; i < kP1Table; i += kP1Threads) L.key[i] = -1;
    if (t == 0) L.count = L.fail = 0;
    SlotUp up[kP1Unroll];
#pragma unroll
    for (int u = 0; u < kP1Unroll; ++u) {
        up[u] = SlotUp{0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (fq[u] >= 0) up[u] = load_up(a, sq[u]);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kP1Unroll; ++u)
        if (fq[u] >= 0) name_face(L, fq[u]);
    __syncthreads();
    const int U = L.count;
    if (U == 0) return;  // no slot is filled
    if (U > kP1Chunk || L.fail) {
        if (t == 0) a.crowded[atomicAdd(&a.hdr[kHdrCrowded], 1)] = (int)cell;
        return;
    }
    gather_named<kOne>(a, L, c.n, c.cx, c.cy, U);
    __syncthreads();
    const int rep = replicas<kOne>(a, U);
#pragma unroll
    for (int u = 0; u < kP1Unroll; ++u) {
        if (fq[u] < 0) continue;
        const int j = find_face(L, fq[u]);  // (every named face was placed)
        const SlotRec R = L.rec.get(j);
        if (R.face >= 0)
            add_slot<kOpts>(a, R, rq[u], cq[u], dW, rW, dH, rH, up[u], acc_row(L, j, cq[u], rep));
    }
    __syncthreads();
    flush_faces<kOne>(a, L, U);
}

// Cells that are read again: those the first kernel left (kAll false; a grid
// smaller than the list walks it), or all cells where a cell has more than
// kP1Group slots (K above 16): the direct way with ids and gradients read group
// by group, else the listed way.
template <bool kOpts, bool kAll>
__global__ __launch_bounds__(kP1Threads) __attribute__((amdgpu_waves_per_eu(5, 8)))
void bwd_cells_again_kernel(BwdArgs a) {
    constexpr bool kOne = kAll;  // (K above 16)
    __shared__ CellLds L;
    if (!bins_usable(a)) return;
    const double dW = (double)a.W, dH = (double)a.H, rW = 1.0 / dW, rH = 1.0 / dH;
    const int t = threadIdx.x;
    const int ncell = kAll ? 1 : a.hdr[kHdrCrowded];
    for (int i = kAll ? 0 : (int)blockIdx.x; i < ncell; i += gridDim.x) {
        const CellGeo c(a, kAll ? xcd_item(blockIdx.x, (int64_t)a.N * a.ncy * a.ncx) : (int64_t)a.crowded[i]);
        if (c.empty(a)) continue;
        bool named = false;
        // (a list that fits one chunk and is the cell's own needs no naming)
        if (kAll && !(a.bs == kTile && a.counts[c.bin] <= kP1Chunk)) {
            for (int q = t; q < kP1Table; q += kP1Threads) L.key[q] = -1;
            if (t == 0) L.count = L.fail = 0;
            __syncthreads();
            for (int q = t; q < c.nslots; q += kP1Threads) {
                const SlotPlace w(q, a.K, c.cols, a.inv_k, c.inv_cols);
                const int f = a.p2f[c.sbase + (int64_t)(w.pr * a.W + w.pc) * a.K + w.k];
                if (f >= 0 && f < a.F && !L.fail) name_face(L, f);
            }
            __syncthreads();
            named = L.count <= kP1Chunk && !L.fail;
            if (named) {
                if (L.count == 0) return;  // no slot is filled
                gather_named<kOne>(a, L, c.n, c.cx, c.cy, L.count);
            }
        }
        // (named: the faces are in the table, in one chunk)
        for (int bi = 0; bi < (named ? 1 : c.nbx * c.nby); ++bi) {
            const int ox = bi % c.nbx, oy = bi / c.nbx;
            const int64_t bin = c.bin + (int64_t)oy * a.nbx + ox;
            const int* list = a.lists + bin * a.M;
            const int cnt = named ? L.count : min(a.counts[bin], a.M);
            for (int base = 0; base < cnt; base += kP1Chunk) {
                const int m = min(kP1Chunk, cnt - base), rep = replicas<kOne>(a, m);
                __syncthreads();  // (the last chunk is flushed, count and fail are read)
                if (!named) {
                    for (int q = t; q < kP1Table; q += kP1Threads) L.key[q] = -1;
                    for (int q = t; q < 9 * (m << rep); q += kP1Threads) L.acc[q] = 0.0;
                    __syncthreads();
                    if (t < m) {
                        const int f = list[base + t];
                        const FaceRec& G = a.recs[f];
                        L.rec.put(t, G, f);
                        // a face listed in several of the cell's bins counts in its first
                        if (max(G.px.x / a.bs, c.bx) == c.bx + ox && max(G.px.z / a.bs, c.by) == c.by + oy) {
                            L.dst[t] = partial_row(a, G, f, c.cx, c.cy);
                            uint32_t h = fhash(f);
                            for (int probe = 0; probe < kP1Table; ++probe) {
                                if (atomicCAS(&L.key[h], -1, f) == -1) {
                                    L.val[h] = (unsigned char)t;
                                    break;
                                }
                                h = (h + 1) & (kP1Table - 1);
                            }
                        } else {
                            L.dst[t] = -2;
                        }
                    }
                    __syncthreads();
                }
                for (int q0 = 0; q0 < c.nslots; q0 += kP1Group) {
                    int64_t sq[kP1Unroll];
                    int fq[kP1Unroll], rq[kP1Unroll], cq[kP1Unroll];
#pragma unroll
                    for (int u = 0; u < kP1Unroll; ++u) {
                        const int q = q0 + u * kP1Threads + t;
                        const SlotPlace w(q, a.K, c.cols, a.inv_k, c.inv_cols);
                        rq[u] = c.r0 + w.pr;
                        cq[u] = c.c0 + w.pc;
                        sq[u] = c.sbase + ((int64_t)(w.pr * a.W + w.pc) * a.K + w.k);
                        fq[u] = q < c.nslots ? a.p2f[sq[u]] : -1;
                    }
#pragma unroll
                    for (int u = 0; u < kP1Unroll; ++u) {
                        if (fq[u] < 0) continue;
                        const int j = find_face(L, fq[u]);
                        if (j < 0) continue;
                        const SlotRec R = L.rec.get(j);
                        if (R.face >= 0)
                            add_slot<kOpts>(a, R, rq[u], cq[u], dW, rW, dH, rH, load_up(a, sq[u]),
                                            acc_row(L, j, cq[u], rep));
                    }
                }
                __syncthreads();
                flush_faces<kOne>(a, L, m);
            }
        }
        __syncthreads();  // (the next cell clears the tables)
    }
}

// Pass 2: one thread per face adds the partial rows this call wrote for it
// and merges the result per vertex in an LDS hash table (FP64 sums); the
// table's rows then go out with one float atomic per coordinate.
__global__ __launch_bounds__(kBwdBlock) void bwd_face_sum_kernel(BwdArgs a) {
    __shared__ int keys[kHash];
    __shared__ double vals[3 * kHash];
    if (!bins_usable(a)) return;
    clear_table(keys, vals);
    __syncthreads();
    const int64_t f = (int64_t)blockIdx.x * kBwdBlock + threadIdx.x;
    const bool overflowed = (a.hdr[kHdrStatus] & kStatOverflow) != 0;
    if (f < a.F && !overflowed) {
        // the rows this call wrote (none for a face whose sums went to the
        // vertices directly, or that no slot names)
        const uchar4 mk = *reinterpret_cast<const uchar4*>(a.pmask + f * kMaxPartials);
        if (mk.x | mk.y | mk.z | mk.w) {
            const bool wr[kMaxPartials] = {mk.x != 0, mk.y != 0, mk.z != 0, mk.w != 0};
            float g9[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            const float* src = a.partial + f * kMaxPartials * 9;
#pragma unroll
            for (int i = 0; i < kMaxPartials; ++i) {
                if (!wr[i]) continue;
#pragma unroll
                for (int x = 0; x < 9; ++x) g9[x] += src[9 * i + x];
            }
            const int32_t* fv = a.faces + 3 * f;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int v = fv[j];
                if (v >= 0 && v < a.V) lds_add(keys, vals, a.grad, v, g9[3 * j], g9[3 * j + 1], g9[3 * j + 2]);
            }
        }
    }
    __syncthreads();
    flush_table(a.grad, keys, vals);
}

// Zeroes grad_verts (n3v floats), nmask words (the row masks, or the header)
// and the count of crowded cells.
__global__ void bwd_prep_kernel(float* __restrict__ grad, int64_t n3v, int* __restrict__ mask, int64_t nmask,
                                int* __restrict__ hdr) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < n3v; i += stride) grad[i] = 0.0f;
    for (int64_t i = i0; i < nmask; i += stride) mask[i] = 0;
    if (i0 == 0) hdr[kHdrCrowded] = 0;
}
static hipError_t launch_prep(float* grad, int64_t n3v, int* mask, int64_t nmask, int* hdr, hipStream_t s) {
    const int64_t n = std::max(n3v, nmask);
    const unsigned g = (unsigned)std::min<int64_t>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(bwd_prep_kernel, dim3(g > 0 ? g : 1), dim3(256), 0, s, grad, n3v, mask, nmask, hdr);
    return hipGetLastError();
}

hipError_t launch_backward(const float* verts, int64_t V, const int32_t* faces, int64_t F, const int64_t* first,
                           const int64_t* nf, int N, int H, int W, int K, float blur, int opts, int bs, int M,
                           const int32_t* p2f, const float* gz, const float* gb, const float* gd, float* grad,
                           int* hdr, FaceRec* recs, int* counts, int* lists, int* order, float* partial,
                           int* big, bool reuse, const BinSig& sig, hipStream_t s, hipEvent_t eb, hipEvent_t ee) {
    reuse = reuse && bs > 0;
    hipError_t e = hipSuccess;
    // the binned form clears grad_verts together with its row masks (below);
    // the per-face form clears it with the header, in one launch
    if (bs == 0 || F == 0) {
        e = launch_prep(grad, V * 3, hdr, reuse ? 0 : kHdrWords, hdr, s);
        if (e != hipSuccess) return e;
    }
    if (F == 0) return hipSuccess;
    BwdArgs a;
    a.verts = verts;
    a.faces = faces;
    a.first = first;
    a.nf = nf;
    a.p2f = p2f;
    a.gz = gz;
    a.gb = gb;
    a.gd = gd;
    a.grad = grad;
    a.hdr = hdr;
    a.big = big;
    a.V = V;
    a.F = F;
    a.N = N;
    a.H = H;
    a.W = W;
    a.K = K;
    a.rb = sqrtf(blur);
    a.opts = opts;
    a.recs = recs;
    a.counts = counts;
    a.lists = lists;
    a.partial = partial;
    a.pmask = reinterpret_cast<unsigned char*>(big);
    a.bs = bs;
    a.nby = bs > 0 ? (H + bs - 1) / bs : 0;
    a.nbx = bs > 0 ? (W + bs - 1) / bs : 0;
    a.M = M;
    a.inv_k = 1.0f / (float)K;
    a.crowded = order;
    a.lgw = a.lgh = a.ncy = a.ncx = a.cross = a.max_rep = 0;
    a.reuse = reuse ? 1 : 0;
    a.sig = sig;
    if (bs > 0) {
        // the same face setup and binning as the forward (unless the forward's
        // are reused), then the two passes
        if (!reuse) {
            e = launch_header_init(hdr, BinSig{}, counts, (int64_t)N * a.nby * a.nbx, s);
            if (e != hipSuccess) return e;
            e = launch_face_setup(verts, V, faces, F, first, nf, N, H, W, a.rb, opts, recs, hdr, bs, M, counts, lists,
                                  s);
            if (e != hipSuccess) return e;
        }
        // grad_verts and the row masks (no partial row is written yet: F x 4
        // mask bytes = F words), in one launch
        e = launch_prep(grad, V * 3, big, F, hdr, s);
        if (e != hipSuccess) return e;
        // the largest cell that divides the bins (or, in bins of an odd multiple
        // of 8, is no larger than one) and whose slots fit a workgroup's registers, wider before higher (K = 16: 8 x 8, K = 8: 16 x
        // 8, K = 1: 32 x 32); 8 x 8 where none does.  Half the size at K = 8
        // took 611 us instead of 448 (32 x 512 x 512 pixels), twice the size on
        // 512 threads 495.
        a.lgw = a.lgh = 3;
        while ((int64_t)K << (a.lgw + a.lgh + 1) <= kP1Group && a.lgh < 5) {
            int& lg = a.lgw == a.lgh ? a.lgw : a.lgh;
            if (bs % 16 != 0 ? (2 << lg) > bs : bs % (2 << lg) != 0) break;
            ++lg;
        }
        // rows of sums per face: eight for K = 1 and 2, four to 7, two to 15, then one
        a.max_rep = K < 4 ? 3 : (K < 8 ? 2 : (K < 16 ? 1 : 0));
        a.cross = bs % (1 << a.lgw) != 0 ? 1 : 0;
        a.ncy = (H + (1 << a.lgh) - 1) >> a.lgh;
        a.ncx = (W + (1 << a.lgw) - 1) >> a.lgw;
        if (eb) (void)hipEventRecord(eb, s);
        const bool o = (opts & (kOptPersp | kOptClip)) != 0;
        const int64_t ncells = (int64_t)N * a.ncy * a.ncx;
        if ((int64_t)K << (a.lgw + a.lgh) <= kP1Group) {
            auto cells = a.max_rep == 0 ? (o ? bwd_cells_kernel<true, true> : bwd_cells_kernel<false, true>)
                                        : (o ? bwd_cells_kernel<true, false> : bwd_cells_kernel<false, false>);
            auto again = o ? bwd_cells_again_kernel<true, false> : bwd_cells_again_kernel<false, false>;
            hipLaunchKernelGGL(cells, dim3((unsigned)ncells), dim3(kP1Threads), 0, s, a);
            hipLaunchKernelGGL(again, dim3((unsigned)std::min<int64_t>(ncells, kAgainGrid)), dim3(kP1Threads), 0, s, a);
        } else {
            auto again = o ? bwd_cells_again_kernel<true, true> : bwd_cells_again_kernel<false, true>;
            hipLaunchKernelGGL(again, dim3((unsigned)ncells), dim3(kP1Threads), 0, s, a);
        }
        hipLaunchKernelGGL(bwd_face_sum_kernel, dim3((unsigned)((F + kBwdBlock - 1) / kBwdBlock)), dim3(kBwdBlock), 0,
                           s, a);
        if (ee) (void)hipEventRecord(ee, s);
        return hipGetLastError();
    }
    if (eb) (void)hipEventRecord(eb, s);
    // Lanes a face: four for many faces with fewer than two pixels each, else
    // sixteen.  One / four / sixteen lanes, backward alone, K = 4: 20,480 faces
    // on 64 images of 128 x 128 pixels 437 / 139 / 91 us, on 4 of 64 x 64 33 / 21 /
    // 25; 40,960 on 8 of 256 x 256 260 / 88 / 80, of 96 x 96 43 / 26 / 35; 81,920 on 4
    // of 64 x 64 29 / 27 / 42; 163,840 on 2 of 512 x 512 321 / 210 / 211; 327,680 on
    // one of 256 x 256 84 / 85 / 143.  And the
    // faces a group of lanes takes in turn: as many as merge in one table once
    // there are workgroups enough (1,024, four a compute unit).
    const int lanes = F >= kManyFaces && (int64_t)N * H * W < 2 * F ? 4 : 16, groups = kBwdBlock / lanes;
    const int per = (int)std::min<int64_t>(std::max<int64_t>(F / (1024 * groups), 1), kFaceMax / groups);
    const int64_t fpw = (int64_t)per * groups;
    auto scan = lanes == 16 ? bwd_faces_kernel<16> : bwd_faces_kernel<4>;
    hipLaunchKernelGGL(scan, dim3((unsigned)((F + fpw - 1) / fpw)), dim3(kBwdBlock), 0, s, a, per);
    hipLaunchKernelGGL(bwd_big_faces_kernel, dim3(512), dim3(kBwdBlock), 0, s, a);
    if (ee) (void)hipEventRecord(ee, s);
    return hipGetLastError();
}

}  // namespace rast
