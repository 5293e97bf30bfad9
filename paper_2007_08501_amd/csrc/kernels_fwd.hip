// kernels_fwd.hip -- forward rasterization kernels for gfx950.
//
//   face_setup      one thread per face: mesh id, 112-byte record, pixel
//                   ranges; with bins, the face appended to every bin that its
//                   ranges touch (counting only when lists == nullptr) and the
//                   largest bin count -> workspace header, overflow flag
//   raster_tiles    one wave per 8x8 pixel tile: loop over candidate faces
//                   (all faces of the tile's mesh, or the tile's bin list),
//                   cull per tile, test per pixel, keep the K nearest in
//                   registers, write the fragments
//
// The paper's rasterizer (Section 3.2) first works on image tiles to drop
// faces and then on pixels, keeping per-pixel queues of the K nearest faces;
// this is that scheme laid out for 64-wide waves.
#include "../../include/rast.h"
#include "device.hpp"
#include "launch.hpp"
#include "tile_layout.hpp"

namespace rast {

__global__ void fill_i32_kernel(int* __restrict__ p, int64_t n, int v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void fill_f32_kernel(float* __restrict__ p, int64_t n, float v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

static int grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_fill_i32(int* p, int64_t n, int v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// Clears the workspace header, stamps the binning signature and clears the
// nbins bin counts, in one launch.
__global__ void header_init_kernel(int* __restrict__ hdr, BinSig sig, int* __restrict__ counts, int64_t nbins) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    if (i0 < kHdrWords) hdr[i0] = (i0 >= kHdrSig && i0 < kHdrSig + kSigWords) ? sig.w[i0 - kHdrSig] : 0;
    for (int64_t i = i0; i < nbins; i += stride) counts[i] = 0;
}

hipError_t launch_header_init(int* hdr, const BinSig& sig, int* counts, int64_t nbins, hipStream_t s) {
    hipLaunchKernelGGL(header_init_kernel, dim3(grid_for(nbins / 4, 256)), dim3(256), 0, s, hdr, sig, counts, nbins);
    return hipGetLastError();
}

// The header's status bits as a rast_status code (the same precedence as
// rast_query_status) and its largest bin count, for a caller without a workspace.
__global__ void status_out_kernel(const int* __restrict__ hdr, int32_t* __restrict__ out) {
    if (threadIdx.x == 0) {
        const int h = hdr[kHdrStatus];
        out[0] = (h & kStatMesh) ? RAST_EMESH : ((h & kStatOverflow) ? RAST_EOVERFLOW : RAST_OK);
        out[1] = hdr[kHdrMaxCount];
    }
}

hipError_t launch_status_out(const int* hdr, int32_t* out, hipStream_t s) {
    hipLaunchKernelGGL(status_out_kernel, dim3(1), dim3(64), 0, s, hdr, out);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_f32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// Binning of a workgroup's faces.  The workgroup's 256 consecutive faces
// (usually neighbours on the mesh, sharing bins) first count their appends per
// distinct bin in an LDS hash table; one global atomic per distinct bin then
// reserves room for all of the workgroup's appends to it, and a second walk
// over the ranges hands out the positions.  An append whose bin finds the
// table full reserves its own position with a global atomic, and so does one
// whose bin is not within kBinProbe slots of its hash position (both walks
// probe the same slots, so they agree on which bins the table holds): a
// workgroup of large faces, touching thousands of bins, then costs at most
// kBinProbe probes per append.  The workgroup also records the largest count
// it leaves in any of its bins (the last reservation in a bin ends at its
// final count, so the maximum over workgroups is the largest bin count) and
// flags a count above the capacity M.
constexpr int kSetupBlock = 256;
constexpr int kBinHash = 1024;  // LDS hash entries of the binning workgroup
constexpr int kBinProbe = 32;   // slots probed per append
__device__ __forceinline__ uint32_t bin_hash(int64_t b) {
    return ((uint32_t)b * 2654435761u ^ (uint32_t)(b >> 32)) >> (32 - 10);
}
static_assert(kBinHash == 1024, "bin_hash yields 10 bits");

struct BinArgs {
    int bs, nby, nbx, M;
    int* counts;
    int* lists;  // nullptr: count only
};

struct BinTable {
    unsigned long long key[kBinHash];  // bin + 1 (0: empty)
    int cnt[kBinHash];                 // appends per bin, then the next rank to hand out
    int base[kBinHash];                // the workgroup's reserved start in the bin
    int wmax[kSetupBlock / 64];
};

// Appends face f of image n, if it has any pixels (px), to its bins.
__device__ __forceinline__ void bin_face(const BinArgs& a, BinTable& T, bool ok, int n, const int4 px, int f,
                                         int* __restrict__ hdr) {
    for (int i = threadIdx.x; i < kBinHash; i += kSetupBlock) {
        T.key[i] = 0ull;
        T.cnt[i] = 0;
    }
    int bx0 = 0, by0 = 0, bx1, by1, nbw = 1, nb = 0;
    if (ok && face_bins_of_px(px, a.bs, bx0, bx1, by0, by1)) {
        nbw = bx1 - bx0 + 1;
        nb = nbw * (by1 - by0 + 1);
    }
    __syncthreads();
    // 1. count per distinct bin
    {
        int ri = 0, rj = 0;
        for (int i = 0; i < nb; ++i) {
            const long long bin = ((int64_t)n * a.nby + by0 + ri) * a.nbx + bx0 + rj;
            if (++rj == nbw) {
                rj = 0;
                ++ri;
            }
            const unsigned long long key = (unsigned long long)bin + 1ull;
            uint32_t h = bin_hash(bin);
            for (int probe = 0; probe < kBinProbe; ++probe) {
                const unsigned long long prev = atomicCAS(&T.key[h], 0ull, key);
                if (prev == 0ull || prev == key) {
                    atomicAdd(&T.cnt[h], 1);
                    break;
                }
                h = (h + 1) & (kBinHash - 1);
            }
        }
    }
    __syncthreads();
    // 2. one reservation per distinct bin
    int top = 0;  // largest count this thread leaves in a bin
    for (int i = threadIdx.x; i < kBinHash; i += kSetupBlock) {
        const unsigned long long key = T.key[i];
        if (key != 0ull) {
            T.base[i] = atomicAdd(&a.counts[key - 1], T.cnt[i]);
            top = max(top, T.base[i] + T.cnt[i]);
            T.cnt[i] = 0;
        }
    }
    __syncthreads();
    // 3. positions
    {
        int ri = 0, rj = 0;
        for (int i = 0; i < nb; ++i) {
            const long long bin = ((int64_t)n * a.nby + by0 + ri) * a.nbx + bx0 + rj;
            if (++rj == nbw) {
                rj = 0;
                ++ri;
            }
            const unsigned long long want = (unsigned long long)bin + 1ull;
            uint32_t h = bin_hash(bin);
            int pos = -1;
            for (int probe = 0; probe < kBinProbe; ++probe) {
                const unsigned long long key = T.key[h];
                if (key == want) {
                    pos = T.base[h] + atomicAdd(&T.cnt[h], 1);
                    break;
                }
                if (key == 0ull) break;
                h = (h + 1) & (kBinHash - 1);
            }
            if (pos < 0) {
                pos = atomicAdd(&a.counts[bin], 1);  // (not in the table)
                top = max(top, pos + 1);
            }
            if (a.lists != nullptr && pos < a.M) a.lists[bin * a.M + pos] = f;
        }
    }
    // the workgroup's largest count: one word per wave, then one read and, only
    // if larger, one atomic per workgroup (same-address atomics serialise)
    top = wave_max(top);
    if ((threadIdx.x & 63) == 0) T.wmax[threadIdx.x >> 6] = top;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kSetupBlock / 64; ++w) top = max(top, T.wmax[w]);
        if (top > __hip_atomic_load(&hdr[kHdrMaxCount], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&hdr[kHdrMaxCount], top);
        if (a.M > 0 && top > a.M) atomicOr(&hdr[kHdrStatus], kStatOverflow);
    }
}

// One thread per face builds the face's record (make_rec: mesh id, exact FP64
// edge vectors, pixel ranges); the workgroup's 256 records are staged in LDS
// and stored with coalesced 16-byte writes (a lane storing its own 112 bytes
// leaves each store instruction scattered over 64 lines).  The threads below
// N also check the mesh ranges.  kBin: the faces are binned at once, over the
// staging's LDS; as a kernel of its own the binning read every record's
// ranges back, two lines a face: setup and binning of 4 meshes of 327,680 faces
// at 1024 x 1024 took 97 us, now 78.
template <bool kBin>
__global__ __launch_bounds__(kSetupBlock) void face_setup_kernel(const float* __restrict__ verts, int64_t V,
                                                                 const int32_t* __restrict__ faces, int64_t F,
                                                                 const int64_t* __restrict__ first,
                                                                 const int64_t* __restrict__ nf, int N, int H, int W,
                                                                 float rb, int opts, FaceRec* __restrict__ recs,
                                                                 int* __restrict__ hdr, BinArgs bin) {
    __shared__ union {
        FaceRec rec[kSetupBlock];
        BinTable table;
    } L;
    const int64_t f0 = (int64_t)blockIdx.x * kSetupBlock;
    int64_t f = f0 + threadIdx.x;
    if (first != nullptr && f < N) {
        // mesh range check: inside [0, F] and ascending without overlap
        int64_t a = first[f], c = nf[f];
        bool bad = a < 0 || c < 0 || a + c > F;
        if (f > 0) bad = bad || a < first[f - 1] + nf[f - 1];
        if (bad) atomicOr(&hdr[kHdrStatus], kStatMesh);
    }
    if (f0 >= F) return;  // (uniform over the workgroup)
    bool ok = false;
    int image = 0;
    int4 px = make_int4(0, -1, 0, -1);
    if (f < F) {
        int mesh = first != nullptr ? find_mesh(first, nf, N, f) : 0;
        int i0 = faces[3 * f + 0], i1 = faces[3 * f + 1], i2 = faces[3 * f + 2];
        bool idx_ok = i0 >= 0 && i0 < V && i1 >= 0 && i1 < V && i2 >= 0 && i2 < V;
        if (!idx_ok) {
            atomicOr(&hdr[kHdrStatus], kStatMesh);
            mesh = -1;
            i0 = i1 = i2 = 0;
        }
        FaceRec R;
        if (V == 0) {
            R = make_rec(0, 0, 0, 0, 0, 0, 0, 0, 0, rb, H, W, -1);
        } else {
            const float* a = verts + 3 * (int64_t)i0;
            const float* b = verts + 3 * (int64_t)i1;
            const float* c = verts + 3 * (int64_t)i2;
            R = make_rec(a[0], a[1], a[2], b[0], b[1], b[2], c[0], c[1], c[2], rb, H, W, mesh, opts);
        }
        ok = R.ok();
        image = R.mesh();
        px = R.px;
        L.rec[threadIdx.x] = R;
    }
    __syncthreads();
    // the workgroup's records are contiguous: coalesced 16-byte stores
    const int n = (int)min((int64_t)kSetupBlock, F - f0);
    const float4* src = reinterpret_cast<const float4*>(L.rec);
    float4* dst = reinterpret_cast<float4*>(recs + f0);
    constexpr int W4 = sizeof(FaceRec) / sizeof(float4);
    for (int i = threadIdx.x; i < n * W4; i += kSetupBlock) dst[i] = src[i];
    if constexpr (kBin) {
        __syncthreads();
        bin_face(bin, L.table, ok, image, px, (int)f, hdr);
    }
}

hipError_t launch_face_setup(const float* verts, int64_t V, const int32_t* faces, int64_t F, const int64_t* first,
                             const int64_t* nf, int N, int H, int W, float rb, int opts, FaceRec* recs, int* hdr,
                             int bs, int M, int* counts, int* lists, hipStream_t s) {
    int64_t n = F > N ? F : N;
    if (n <= 0) return hipSuccess;
    const BinArgs b{bs, bs > 0 ? (H + bs - 1) / bs : 0, bs > 0 ? (W + bs - 1) / bs : 0, M, counts, lists};
    auto setup = bs > 0 ? face_setup_kernel<true> : face_setup_kernel<false>;
    hipLaunchKernelGGL(setup, dim3((unsigned)((n + kSetupBlock - 1) / kSetupBlock)), dim3(kSetupBlock), 0, s, verts, V,
                       faces, F, first, nf, N, H, W, rb, opts, recs, hdr, b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fine pass.  One 64-thread workgroup = one wave = one 8x8 tile of image n.
// Faces come either from the whole mesh (BINNED = false) or from the list of
// the bin that contains the tile.  Every face is first culled against the
// tile's extent (a wave-uniform branch) and then tested by each lane for its
// own pixel; winners go through the register top-K.
// ---------------------------------------------------------------------------
struct FineArgs {
    const FaceRec* recs;
    const int64_t* first;
    const int64_t* nf;
    const int* counts;
    const int* lists;
    int64_t F;
    int N, H, W, K;
    float blur;
    float rg, sx, sy;  // edge_radius(), 2 / W, 2 / H (for the edge masks)
    int opts;          // rasterizer options (kOpt*)
    int bs, nby, nbx, M;
    int tiles_x, tiles_y;
    int32_t* p2f;
    float* zbuf;
    float* bary;
    float* dists;
};

// LDS of one tile's wave: a block of up to 64 candidate faces that overlap the
// tile (the gather gives every lane one list entry and the transpose one
// record), reused at the end to stage one output array at a time.
constexpr int kChunk = tile_layout::kChunk;

// A face as the tile pass keeps it in LDS: the geometry the pixel tests read
// (the fields of FaceRec that the evaluation uses), the face id, and the
// tile's pixels in the face's pixel ranges, as a 64-bit mask
// (bit r*8 + c), which replaces the box.
struct TileRec {
    double2 pa, ab, ac;
    double E;
    float az, dz1, dz2, invE, il0, il1, il2;
    int fid;
    uint64_t mask;
};
static_assert(sizeof(TileRec) == tile_layout::kTileRecBytes, "tile record layout");

union TileLds {
    TileRec rec[kChunk];
    float stage[tile_layout::kBlockBytes / 4];
};
static_assert(sizeof(TileLds) == tile_layout::kBlockBytes, "tile LDS layout");

// Writes the tile's fragments from the per-lane queues.  Values are staged in
// LDS per pixel and then stored by consecutive lanes to consecutive
// addresses, so every store instruction writes whole contiguous runs (one
// tile row of pix_to_face is 8*K contiguous words) instead of 64 scattered
// words; written slot by slot, each cache line would be completed by K
// separate instructions with loads in between and could be evicted half
// written.  Ids and depths come straight from the keys; barycentrics and
// distances are recomputed from the face records.  One array is staged at a
// time: the block then is no larger than the candidate faces need (6.4 KB),
// so that the registers and not the LDS bound the waves of a compute unit.
constexpr int kStageG1 = tile_layout::kStageG1;  // slots per pass for ids and depths
constexpr int kStageG2 = tile_layout::kStageG2;  // slots per pass for barycentrics and distances

// Stores of four consecutive words.  For a queue of K = KB slots (K a multiple
// of 4, 16-byte aligned outputs) the ids and depths are streamed past the
// caches (the "nt" hint): those passes write whole lines, and streaming them
// leaves L2 to the face records the tile waves share; the barycentric and
// distance passes write part lines per pass and are stored normally, so that
// L2 completes their lines.  Other K start a pixel's run at any word.
typedef float nt_f4 __attribute__((ext_vector_type(4)));
typedef float f4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool ALIGNED, bool STREAM>
__device__ __forceinline__ void store4(float* p, float x, float y, float z, float w) {
    if constexpr (ALIGNED && STREAM)
        __builtin_nontemporal_store(nt_f4{x, y, z, w}, reinterpret_cast<nt_f4*>(p));
    else if constexpr (ALIGNED)
        *reinterpret_cast<nt_f4*>(p) = nt_f4{x, y, z, w};
    else
        *reinterpret_cast<f4_a4*>(p) = f4_a4{x, y, z, w};
}

// The tile's place in an output array of n words a slot.
struct TileOut {
    int K, rowK;     // slots a pixel, slots an image row
    int rows, cols;  // of the tile inside the image
};

// Stores G slots from slot g0 of every pixel of the tile, staged at
// stage[pixel * S ...], n words each: quads of four words, one a lane.
template <int G, int S, int n, bool ALIGNED, bool STREAM>
__device__ __forceinline__ void store_staged(float* __restrict__ out, const float* stage, const TileOut& t, int g0) {
    constexpr int Q = n * G / 4;  // quads a pixel
    const int lane = threadIdx.x & 63;
    const int left = n * (t.K - g0);  // words of the pass
    int px = lane / Q, q = lane - px * Q;
#pragma unroll
    for (int e0 = 0; e0 < 64 * Q; e0 += 64) {
        const int r = px >> 3, c = px & 7;
        if (r < t.rows && c < t.cols) {
            const float* src = stage + px * S + 4 * q;
            float* dst = out + (n * (r * t.rowK + c * t.K + g0) + 4 * q);
            if (ALIGNED || 4 * q + 4 <= left) {
                store4<ALIGNED, STREAM>(dst, src[0], src[1], src[2], src[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (4 * q + i < left) dst[i] = src[i];
            }
        }
        px += 64 / Q;
        q += 64 % Q;
        if (64 % Q != 0 && q >= Q) {
            q -= Q;
            ++px;
        }
    }
}

// Fills the tile's runs of an array of n words a slot with one value (a tile
// that no face reaches).
template <int KB, int n, bool ALIGNED>
__device__ __forceinline__ void fill_rows(float* __restrict__ out, const TileOut& t, float v) {
    const int lane = threadIdx.x & 63;
    if constexpr (ALIGNED) {
        constexpr int Q = n * KB * kTile / 4;  // quads of a full row
        const int nq = n * KB * t.cols / 4;
#pragma unroll
        for (int e0 = 0; e0 < kTile * Q; e0 += 64) {
            const int e = e0 + lane;
            const int r = e / Q, q = e - r * Q;
            if (e < kTile * Q && r < t.rows && q < nq)
                store4<true, true>(out + (n * r * t.rowK + 4 * q), v, v, v, v);
        }
    } else {
        const int w = n * t.cols * t.K;
        for (int r = 0; r < t.rows; ++r) {
            float* dst = out + n * r * t.rowK;
            for (int i = 4 * lane; i < w; i += 256) {
                if (i + 4 <= w) {
                    store4<false, false>(dst + i, v, v, v, v);
                } else {
                    for (int j = i; j < w; ++j) dst[j] = v;
                }
            }
        }
    }
}

// Barycentrics and signed distance of the face of a key at pixel p (-1 for an empty slot).
template <bool OPT>
__device__ __forceinline__ void slot_values(const FineArgs& a, uint64_t key, const Pix& p, float& w0, float& w1,
                                            float& w2, float& d) {
    w0 = w1 = w2 = d = -1.0f;
    if (key != kEmptyKey) {
        const FaceRec R = a.recs[(uint32_t)key];
        Eval ev;
        eval_full(R, p, ev);
        w0 = ev.w0;
        w1 = ev.w1;
        w2 = ev.w2;
        if (OPT) {
            float zf;
            apply_opts(a.opts, R.az, R.dz1, R.dz2, w0, w1, w2, zf);
        }
        d = ev.inside ? -ev.d2 : ev.d2;
    }
}
__device__ __forceinline__ int key_id(uint64_t key) { return key == kEmptyKey ? -1 : (int)(uint32_t)key; }
__device__ __forceinline__ float key_z(uint64_t key) {
    return key == kEmptyKey ? -1.0f : __uint_as_float((uint32_t)(key >> 32));
}

// EXACT: K equals the queue size KB, so every group width, stride and index
// below is a compile-time constant (the common case); otherwise K < KB is a
// run-time value.  Addresses are 32-bit offsets from the tile's first
// fragment, a wave-uniform base.
// OPT: the rasterizer options that change barycentrics and depth are on
// (a separate instantiation, so that the default path carries no test for them).
template <int KB, bool EXACT, bool OPT>
__device__ __forceinline__ void write_fragments(const FineArgs& a, TileLds& L, const TopK<KB>& top, const Pix& p,
                                                int n, int tx, int ty) {
    const int lane = threadIdx.x & 63;
    const TileOut t{EXACT ? KB : a.K, a.W * (EXACT ? KB : a.K), min(kTile, a.H - ty * kTile),
                    min(kTile, a.W - tx * kTile)};
    const int64_t slot0 = (((int64_t)n * a.H + ty * kTile) * a.W + tx * kTile) * t.K;
    float* const p2f_t = reinterpret_cast<float*>(a.p2f) + slot0;  // (ids move as bit patterns)
    float* const zbuf_t = a.zbuf + slot0;
    float* const dist_t = a.dists + slot0;
    float* const bary_t = a.bary + 3 * slot0;
    if constexpr (KB < 4) {
        // one or two slots: a lane's own few words, no staging
        if ((lane >> 3) < t.rows && (lane & 7) < t.cols) {
            const int o = (lane >> 3) * t.rowK + (lane & 7) * KB;
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                float w0, w1, w2, d;
                slot_values<OPT>(a, top.q[k], p, w0, w1, w2, d);
                p2f_t[o + k] = __int_as_float(key_id(top.q[k]));
                zbuf_t[o + k] = key_z(top.q[k]);
                dist_t[o + k] = d;
                bary_t[3 * (o + k) + 0] = w0;
                bary_t[3 * (o + k) + 1] = w1;
                bary_t[3 * (o + k) + 2] = w2;
            }
        }
    } else {
        // (for EXACT the launcher has checked that the four outputs are 16-byte aligned)
        static_assert(KB % 4 == 0, "queues of four or more slots are multiples of four");
        if (__ballot(top.q[0] != kEmptyKey) == 0ull) {
            fill_rows<KB, 1, EXACT>(p2f_t, t, __int_as_float(-1));
            fill_rows<KB, 1, EXACT>(zbuf_t, t, -1.0f);
            fill_rows<KB, 3, EXACT>(bary_t, t, -1.0f);
            fill_rows<KB, 1, EXACT>(dist_t, t, -1.0f);
            return;
        }
        float* const st = L.stage;
        // ids, then depths
        {
            constexpr int G = tile_layout::stage_slots(KB, kStageG1);
            constexpr int S = tile_layout::stage_stride(1, G);
            static_assert(64 * S * 4 <= (int)sizeof(TileLds), "id/depth staging exceeds the tile LDS");
#pragma unroll
            for (int g0 = 0; g0 < KB; g0 += G) {
                if (g0 >= t.K) continue;  // K is uniform: the whole wave skips
#pragma unroll
                for (int k = 0; k < G; ++k) st[lane * S + k] = __int_as_float(key_id(top.q[g0 + k]));
                __syncthreads();
                store_staged<G, S, 1, EXACT, true>(p2f_t, st, t, g0);
                __syncthreads();
#pragma unroll
                for (int k = 0; k < G; ++k) st[lane * S + k] = key_z(top.q[g0 + k]);
                __syncthreads();
                store_staged<G, S, 1, EXACT, true>(zbuf_t, st, t, g0);
                __syncthreads();
            }
        }
        // barycentrics and signed distances
        {
            constexpr int G = tile_layout::stage_slots(KB, kStageG2);
            constexpr int SB = tile_layout::stage_stride(3, G), SD = tile_layout::stage_stride(1, G);
            static_assert(64 * SB * 4 <= (int)sizeof(TileLds), "bary staging exceeds the tile LDS");
#pragma unroll
            for (int g0 = 0; g0 < KB; g0 += G) {
                if (g0 >= t.K) continue;
                float d[G];
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    float w0, w1, w2;
                    slot_values<OPT>(a, top.q[g0 + k], p, w0, w1, w2, d[k]);
                    st[lane * SB + 3 * k + 0] = w0;
                    st[lane * SB + 3 * k + 1] = w1;
                    st[lane * SB + 3 * k + 2] = w2;
                }
                __syncthreads();
                store_staged<G, SB, 3, EXACT, false>(bary_t, st, t, g0);
                __syncthreads();
#pragma unroll
                for (int k = 0; k < G; ++k) st[lane * SD + k] = d[k];
                __syncthreads();
                store_staged<G, SD, 1, EXACT, false>(dist_t, st, t, g0);
                __syncthreads();
            }
        }
    }
}

// Transpose of the 64x64 bit matrix whose row i is lane i's word: bit i of
// lane p's result is bit p of lane i's word.  Six butterfly stages: at stage
// j the lanes i and i ^ j exchange the off-diagonal j x j blocks of their
// 2j x 2j block (the lane with bit j clear keeps its low groups of j bits
// and takes the partner's low groups into its high ones, the other keeps its
// high groups and takes the partner's high groups into its low ones).  All in
// vector registers: stages 32 and 16 are the half-wave and half-row swaps,
// the others fetch the partner's words with DPP; about 30 instructions,
// where shuffles through the LDS took 70 and twelve LDS operations.
struct Transpose64 {
    uint32_t sel8;          // byte selector of stage 8
    uint32_t keep[3];       // stages 4, 2, 1: the bits a lane keeps
    uint32_t rot[3];        // and the rotation that brings the partner's bits
    __device__ __forceinline__ void init(int lane) {
        // v_perm bytes: 0-3 from the lane's own word, 4-7 from the partner's
        sel8 = (lane & 8) ? 0x03070105u : 0x06020400u;
        const uint32_t low[3] = {0x0f0f0f0fu, 0x33333333u, 0x55555555u};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int j = 4 >> i;
            keep[i] = (lane & j) ? ~low[i] : low[i];
            rot[i] = (lane & j) ? (uint32_t)j : 32u - (uint32_t)j;
        }
    }
    template <int kCtrl>
    static __device__ __forceinline__ uint32_t dpp(uint32_t v) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
    }
    __device__ __forceinline__ uint32_t mix(uint32_t x, uint32_t y, int i) const {
        const uint32_t t = __builtin_amdgcn_alignbit(y, y, rot[i]);
        return (x & keep[i]) | (t & ~keep[i]);
    }
    __device__ __forceinline__ uint64_t operator()(uint64_t v) const {
        uint32_t x = (uint32_t)v, y = (uint32_t)(v >> 32);
        // 32: the upper half-wave's low words against the lower half-wave's high words
        const auto s32 = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = s32[0];
        y = s32[1];
        // 16: the same for 16-bit halves between the rows of a half-wave
        const uint32_t lo = __builtin_amdgcn_perm(y, x, 0x05040100u), hi = __builtin_amdgcn_perm(y, x, 0x07060302u);
        const auto s16 = __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
        x = __builtin_amdgcn_perm(s16[1], s16[0], 0x05040100u);
        y = __builtin_amdgcn_perm(s16[1], s16[0], 0x07060302u);
        // 8: partner lane ^ 8 (a rotation of the row by 8)
        x = __builtin_amdgcn_perm(dpp<0x128>(x), x, sel8);
        y = __builtin_amdgcn_perm(dpp<0x128>(y), y, sel8);
        // 4: lane ^ 4 is the half-row mirror (^ 7) of the quad mirror (^ 3)
        x = mix(x, dpp<0x141>(dpp<0x1b>(x)), 0);
        y = mix(y, dpp<0x141>(dpp<0x1b>(y)), 0);
        // 2 and 1: quad permutations
        x = mix(x, dpp<0x4e>(x), 1);
        y = mix(y, dpp<0x4e>(y), 1);
        x = mix(x, dpp<0xb1>(x), 2);
        y = mix(y, dpp<0xb1>(y), 2);
        return ((uint64_t)y << 32) | x;
    }
};

// One wave rasterizes one 8x8 tile:
//  1. where the list is longer than the tile needs (a bin of several tiles, or
//     a whole mesh), read only the pixel ranges of its faces, a wave-wide chunk
//     at a time, and push the ids of those that reach the tile together into
//     full lanes (each lane's place from a ballot, moved by ds_permute);
//  2. gather the records of up to 64 such faces, one a lane, narrow each one's
//     pixels by its edge lines, and append those that keep a pixel to the LDS
//     block, each with its 64-bit mask of such pixels;
//  3. when the block is full (64 records) or the list ends, transpose the kept
//     faces' masks across the wave (lane j holds record j's mask), so that
//     lane p holds the faces that may cover pixel p;
//  4. every lane walks only its own faces, runs the full test and inserts
//     the faces that count into its register top-K.
// Step 4 is where the arithmetic is; gathering each pixel's candidates first
// keeps lanes from idling on faces that miss their pixel, and steps 1 and 3
// keep the lanes of the edge masks and the rounds of step 4 full (a tile of
// a 16-pixel bin needs a third of the bin's list).  Faces that no longer fit
// the block are gathered again after the test: holding their records in
// registers across it would cost a wave per SIMD.
__device__ __forceinline__ double first_lane(double v) {
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
    return __hiloint2double(hi, lo);
}

template <int KB, bool OPT>
__device__ __forceinline__ void test_kept(const FineArgs& a, const TileLds& L, const Transpose64& T, TopK<KB>& top,
                                          const Pix& p, int m) {
    const int lane = threadIdx.x & 63;
    __syncthreads();
    uint64_t mine = T(lane < m ? L.rec[lane].mask : 0ull);
    constexpr int NB = queue_batch(KB);
    // NB candidates per round; the round count is the wave's longest
    // list, so the loop is uniform and the queue stays in place across rounds
    const int nmax = wave_max(__popcll(mine));
    for (int i0 = 0; i0 < nmax; i0 += NB) {
        uint64_t b[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            uint64_t key = kEmptyKey;
            if (mine != 0ull) {
                const int j = __ffsll((unsigned long long)mine) - 1;
                mine &= mine - 1;
                float z;
                if (face_counts_in_box(L.rec[j], p, a.blur, z, OPT ? a.opts : 0)) key = make_key(z, L.rec[j].fid);
            }
            b[u] = key;
        }
        top.push(b);
    }
    __syncthreads();
}

template <int KB, bool BINNED, bool EXACT, bool OPT>
__device__ __forceinline__ void raster_tile(const FineArgs& a, TileLds& L, int n, int tx, int ty) {
    const int lane = threadIdx.x & 63;
    const int x0 = tx * kTile, y0 = ty * kTile;
    const Pix p = make_pix(y0 + (lane >> 3), x0 + (lane & 7), a.H, a.W);
    // the tile's first pixel centre (lane 0's), for the edge masks
    const double px0 = first_lane(p.x), py0 = first_lane(p.y);
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    Transpose64 T;
    T.init(lane);

    TopK<KB> top;
    top.init();

    const int* list = nullptr;
    int64_t base = 0, cnt = 0;
    if (BINNED) {
        int bx = (tx * kTile) / a.bs, by = (ty * kTile) / a.bs;
        int64_t bin = ((int64_t)n * a.nby + by) * a.nbx + bx;
        cnt = min(a.counts[bin], a.M);
        list = a.lists + bin * a.M;
    } else {
        int64_t lo = a.first[n], hi = a.first[n] + a.nf[n];
        lo = lo < 0 ? 0 : lo;
        hi = hi > a.F ? a.F : hi;
        base = lo;
        cnt = hi > lo ? hi - lo : 0;
    }
    int64_t c0 = 0;       // list entries read
    int pend = 0, np = 0; // ids waiting to be gathered: lane i < np holds the i-th
    int batch = 0;        // the lane's id of the present batch
    uint64_t todo = 0ull; // lanes of the batch still to be gathered
    bool last = cnt == 0; // nothing comes after this batch
    int m = 0;            // records in the block
    while (cnt > 0) {
        if (todo == 0ull) {
            // 1. the next batch of ids
            int over = 0;  // ids past the 64th
            if (BINNED && a.bs == kTile) {
                pend = c0 + lane < cnt ? list[c0 + lane] : 0;
                np = (int)min((int64_t)kChunk, cnt - c0);
                c0 += kChunk;
            } else {
                while (np < kChunk && c0 < cnt) {
                    const int64_t e = c0 + lane;
                    const int id = e < cnt ? (BINNED ? list[e] : (int)(base + e)) : -1;
                    bool hit = false;
                    if (id >= 0) {
                        const int4 q = a.recs[id].px;
                        hit = q.x < x0 + kTile && q.y >= x0 && q.z < y0 + kTile && q.w >= y0 && q.x <= q.y && q.z <= q.w;
                    }
                    const uint64_t hits = __ballot(hit);
                    const int add = __popcll(hits);
                    // every hit goes to its place (modulo 64), the other lanes
                    // to the first place after them, which is not read
                    const int to = (np + (hit ? __popcll(hits & lt_mask) : add)) & (kChunk - 1);
                    const int v = __builtin_amdgcn_ds_permute(4 * to, id);
                    if (lane >= np && lane < np + add) pend = v;
                    if (lane < np + add - kChunk) over = v;
                    np += add;
                    c0 += kChunk;
                }
            }
            batch = pend;
            const int nb = min(np, kChunk);
            todo = nb == kChunk ? ~0ull : (1ull << nb) - 1ull;
            np -= nb;
            pend = over;
            last = c0 >= cnt && np == 0;
        }
        // 2. gather and compact the faces that overlap the tile
        const bool mine = (todo >> lane) & 1ull;
        uint64_t pm = 0ull;
        // the record as seven 16-byte words (pa | ab | ac | E, a.z, mesh |
        // dz1, dz2, 1/E, il0 | il1, il2, pad | pixel ranges)
        static_assert(sizeof(FaceRec) == 7 * sizeof(float4), "face record layout");
        const float4* rsrc = reinterpret_cast<const float4*>(a.recs + (mine ? batch : 0));
        const float4 rv0 = rsrc[0], rv1 = rsrc[1], rv2 = rsrc[2], rv3 = rsrc[3], rv4 = rsrc[4], rv5 = rsrc[5];
        if (mine) pm = tile_mask(reinterpret_cast<const int4*>(rsrc)[6], x0, y0);
        if (pm != 0ull) {
            // narrow the ranges' pixels to those near or inside the triangle
            const EdgeGeo G{f4_as_d2(rv0), f4_as_d2(rv1), f4_as_d2(rv2), f4_as_d2(rv3).x};
            pm &= edge_mask(G, a.rg, px0, py0, a.sx, a.sy);
        }
        const uint64_t kept = __ballot(pm != 0ull);
        const int dst = m + __popcll(kept & lt_mask);
        if (pm != 0ull && dst < kChunk) {
            float4* rdst = reinterpret_cast<float4*>(&L.rec[dst]);
            rdst[0] = rv0;
            rdst[1] = rv1;
            rdst[2] = rv2;
            rdst[3] = make_float4(rv3.x, rv3.y, rv3.z, rv4.x);  // E | a.z, dz1
            rdst[4] = make_float4(rv4.y, rv4.z, rv4.w, rv5.x);  // dz2, 1/E, il0, il1
            rdst[5] = make_float4(rv5.y, __int_as_float(batch), __uint_as_float((uint32_t)pm),
                                  __uint_as_float((uint32_t)(pm >> 32)));  // il2, id, mask
        }
        m += __popcll(kept);
        // a full block leaves the rest of the batch for after the test
        todo = m > kChunk ? kept & __ballot(dst >= kChunk) : 0ull;
        const bool end = todo == 0ull && last;
        if (m > kChunk || (end && m > 0)) {  // (uniform)
            test_kept<KB, OPT>(a, L, T, top, p, min(m, kChunk));
            m = 0;
        }
        if (end) break;
    }
    write_fragments<KB, EXACT, OPT>(a, L, top, p, n, tx, ty);
}

// EXACT: faces_per_pixel equals the queue size KB (chosen at launch).
// The grid's workgroups are taken as tiles in image-major raster order, each
// XCD a contiguous range of them (xcd_item).
template <int KB, bool BINNED, bool EXACT, bool OPT>
__global__ __launch_bounds__(64) void raster_tiles_kernel(FineArgs a) {
    __shared__ TileLds L;
    const int64_t per_img = (int64_t)a.tiles_x * a.tiles_y;
    const int64_t wg = blockIdx.x + (int64_t)gridDim.x * (blockIdx.y + (int64_t)gridDim.y * blockIdx.z);
    const int64_t t = xcd_item(wg, per_img * a.N);
    const int n = (int)(t / per_img);
    const int rem = (int)(t - n * per_img);
    const int ty = rem / a.tiles_x;
    raster_tile<KB, BINNED, EXACT, OPT>(a, L, n, rem - ty * a.tiles_x, ty);
}

// Persistent form: a device-sized grid; each wave pulls the next tile id from
// a counter in the workspace header.  order[] lists tile ids (image-major
// linear ids) most-loaded bins first.  Every wave leaves when the counter
// passes the number of tiles.
// One tile of the persistent form, kept out of line: inlined into the work
// loop, the tile's loop-invariant address arithmetic is hoisted out of it and
// held live across tiles, far beyond the register file.
template <int KB, bool EXACT, bool OPT>
__device__ __noinline__ void raster_tile_persistent(const FineArgs& a, TileLds& L, int n, int tx, int ty) {
    raster_tile<KB, true, EXACT, OPT>(a, L, n, tx, ty);
}

template <int KB, bool EXACT, bool OPT>
__global__ __launch_bounds__(64) void raster_persistent_kernel(FineArgs a, const int* __restrict__ order,
                                                               int* __restrict__ hdr, int total) {
    __shared__ TileLds L;
    for (;;) {
        int item = 0;
        if ((threadIdx.x & 63) == 0) item = atomicAdd(&hdr[kHdrWorkNext], 1);
        item = __shfl(item, 0);
        if (item >= total) break;
        int t = order[item];
        int per_img = a.tiles_x * a.tiles_y;
        int n = t / per_img;
        int rem = t - n * per_img;
        int ty = rem / a.tiles_x;
        int tx = rem - ty * a.tiles_x;
        raster_tile_persistent<KB, EXACT, OPT>(a, L, n, tx, ty);
    }
}

// order[]: tiles sorted by the count of their bin, descending, using a
// counting sort over count buckets (64 buckets of width ceil((M+1)/64)), with
// one global atomic per distinct bucket of a wave (per-thread atomics on the
// 64 counters serialised: about 1 ms at 32 images of 512 x 512 pixels).
__device__ __forceinline__ int tile_bucket(const int* __restrict__ counts, int t, int tiles_x, int tiles_y, int bs,
                                           int nby, int nbx, int M) {
    const int per_img = tiles_x * tiles_y;
    const int n = t / per_img;
    const int rem = t - n * per_img;
    const int ty = rem / tiles_x, tx = rem - ty * tiles_x;
    const int64_t bin = ((int64_t)n * nby + (ty * kTile) / bs) * nbx + (tx * kTile) / bs;
    const int cnt = min(counts[bin], M);
    const int width = (M + 64) / 64;
    return 63 - min(cnt / width, 63);  // bucket 0 = heaviest
}

__global__ __launch_bounds__(256) void order_hist_kernel(const int* __restrict__ counts, int N, int tiles_x,
                                                         int tiles_y, int bs, int nby, int nbx, int M,
                                                         int* __restrict__ hist) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)N * tiles_x * tiles_y;
    (void)wave_bucket_slot(hist, t < total ? tile_bucket(counts, (int)t, tiles_x, tiles_y, bs, nby, nbx, M) : -1);
}

__global__ __launch_bounds__(256) void order_scatter_kernel(const int* __restrict__ counts, int N, int tiles_x,
                                                            int tiles_y, int bs, int nby, int nbx, int M,
                                                            int* __restrict__ hist_off, int* __restrict__ order) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)N * tiles_x * tiles_y;
    const int pos =
        wave_bucket_slot(hist_off, t < total ? tile_bucket(counts, (int)t, tiles_x, tiles_y, bs, nby, nbx, M) : -1);
    if (t < total) order[pos] = (int)t;
}

// exclusive scan of the 64 bucket sizes, in place; also arms the work counter
__global__ void order_scan_kernel(int* __restrict__ hist, int* __restrict__ hdr, int total) {
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int i = 0; i < 64; ++i) {
            int v = hist[i];
            hist[i] = acc;
            acc += v;
        }
        hdr[kHdrWorkNext] = 0;
        hdr[kHdrWorkTotal] = total;
    }
}

template <int KB, bool EXACT, bool OPT>
static hipError_t launch_fine_k(const FineArgs& a, bool binned, int sched, int* order, int* hist, int* hdr,
                                int n_workers, hipStream_t s, hipEvent_t eb, hipEvent_t ee) {
    if (binned && sched == 1) {
        int total = a.N * a.tiles_x * a.tiles_y;
        hipError_t e = launch_fill_i32(hist, 64, 0, s);
        if (e != hipSuccess) return e;
        unsigned g = (unsigned)((total + 255) / 256);
        hipLaunchKernelGGL(order_hist_kernel, dim3(g), dim3(256), 0, s, a.counts, a.N, a.tiles_x, a.tiles_y, a.bs,
                           a.nby, a.nbx, a.M, hist);
        hipLaunchKernelGGL(order_scan_kernel, dim3(1), dim3(64), 0, s, hist, hdr, total);
        hipLaunchKernelGGL(order_scatter_kernel, dim3(g), dim3(256), 0, s, a.counts, a.N, a.tiles_x, a.tiles_y, a.bs,
                           a.nby, a.nbx, a.M, hist, order);
        int workers = n_workers < total ? n_workers : total;
        if (eb) (void)hipEventRecord(eb, s);
        hipLaunchKernelGGL((raster_persistent_kernel<KB, EXACT, OPT>), dim3(workers), dim3(64), 0, s, a, order, hdr,
                           total);
        if (ee) (void)hipEventRecord(ee, s);
        return hipGetLastError();
    }
    dim3 grid(a.tiles_x, a.tiles_y, a.N);
    if (eb) (void)hipEventRecord(eb, s);
    if (binned)
        hipLaunchKernelGGL((raster_tiles_kernel<KB, true, EXACT, OPT>), grid, dim3(64), 0, s, a);
    else
        hipLaunchKernelGGL((raster_tiles_kernel<KB, false, EXACT, OPT>), grid, dim3(64), 0, s, a);
    if (ee) (void)hipEventRecord(ee, s);
    return hipGetLastError();
}

hipError_t launch_fine(const FaceRec* recs, const int64_t* first, const int64_t* nf, const int* counts,
                       const int* lists, int64_t F, int N, int H, int W, int K, float blur, int opts, int bs, int M,
                       int sched,
                       int* order, int* hist, int* hdr, int n_workers, int32_t* p2f, float* zbuf, float* bary,
                       float* dists, hipStream_t s, hipEvent_t eb, hipEvent_t ee) {
    FineArgs a;
    a.recs = recs;
    a.first = first;
    a.nf = nf;
    a.counts = counts;
    a.lists = lists;
    a.F = F;
    a.N = N;
    a.H = H;
    a.W = W;
    a.K = K;
    a.blur = blur;
    a.rg = edge_radius(blur, H, W);
    a.sx = 2.0f / (float)W;
    a.sy = 2.0f / (float)H;
    a.opts = opts;
    a.bs = bs > 0 ? bs : kTile;
    a.nby = bs > 0 ? (H + bs - 1) / bs : 0;
    a.nbx = bs > 0 ? (W + bs - 1) / bs : 0;
    a.M = M;
    a.tiles_x = (W + kTile - 1) / kTile;
    a.tiles_y = (H + kTile - 1) / kTile;
    a.p2f = p2f;
    a.zbuf = zbuf;
    a.bary = bary;
    a.dists = dists;
    bool binned = bs > 0;
    // queue sizes are powers of two; K equal to one gets the compile-time-K
    // kernels, which store four slots at a time and so need 16-byte aligned
    // outputs
    const bool aligned = (((uintptr_t)p2f | (uintptr_t)zbuf | (uintptr_t)bary | (uintptr_t)dists) & 15) == 0;
#define RAST_FINE_BUCKET(KB)                                                                          \
    if (K <= KB) {                                                                                    \
        if (opt) return launch_fine_k<KB, false, true>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee); \
        if (K == KB && aligned)                                                                         \
            return launch_fine_k<KB, true, false>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee); \
        return launch_fine_k<KB, false, false>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee); \
    }
    // options that change barycentrics and depth take the runtime-K form with their per-pixel work
    const bool opt = (opts & (kOptPersp | kOptClip)) != 0;
    if (K <= 1 && opt) return launch_fine_k<1, true, true>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee);
    if (K <= 2 && opt) return launch_fine_k<2, true, true>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee);
    if (K <= 1) return launch_fine_k<1, true, false>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee);
    if (K <= 2) return launch_fine_k<2, true, false>(a, binned, sched, order, hist, hdr, n_workers, s, eb, ee);
    RAST_FINE_BUCKET(4)
    RAST_FINE_BUCKET(8)
    RAST_FINE_BUCKET(16)
    RAST_FINE_BUCKET(32)
    RAST_FINE_BUCKET(64)
#undef RAST_FINE_BUCKET
    return hipErrorInvalidValue;
}

}  // namespace rast
