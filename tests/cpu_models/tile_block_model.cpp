// tile_block_model.cpp -- bounds-checked CPU model of how the mesh fine pass
// (csrc/kernels_fwd.hip) fills, tests and reuses its LDS block, one 64-lane wave
// per 8x8 tile, with the sizes of tile_layout.hpp that the kernel uses.
//
// The first part replays a tile's loop: ids of a list packed into full batches
// (a place in the batch from the lanes before that hit, modulo the wave, those
// past the 64th held over), records appended to the block by rank among the
// lanes that keep one, the lanes left over when the block is full gathered again
// after the test.  Every place is checked, no lane reads a place that no hit
// was moved to, and every face that hits and keeps a pixel is tested exactly once.
// The second part replays the write-out: staging of ids, depths, barycentrics
// and distances, one array at a time, and the fill of empty tiles, for every
// queue size, every K and every tile cut by an image's edge.  Every word of every
// fragment is written exactly once, with its own value, and nothing else.
//
//   tile_block_model [bytes]   bytes: of the block (default: the kernel's)
// Exit status 0: all checks hold; 1: one does not (printed).
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../../paper_2007_08501_amd/csrc/tile_layout.hpp"

namespace tl = rast::tile_layout;

static std::mt19937_64 rng(4711);
static int fails(const char* what, long long a, long long b) {
    std::printf("FAILED: %s (%lld, %lld)\n", what, a, b);
    return 1;
}

// ---------------------------------------------------------------- the loop

struct Tile {
    std::vector<unsigned char> block;  // the LDS block
    std::vector<char> hit, keep;       // per list entry: reaches the tile; keeps a pixel
    std::vector<int> tested;
    int bytes;
};

static bool put_record(Tile& T, int place, int id) {
    const size_t at = (size_t)place * tl::kTileRecBytes;
    if (place < 0 || at + tl::kTileRecBytes > T.block.size()) return false;
    for (int i = 0; i < tl::kTileRecBytes; ++i) T.block.at(at + i) = (unsigned char)(id >> (8 * (i & 3)));
    return true;
}
static int get_record(const Tile& T, int place) {
    const size_t at = (size_t)place * tl::kTileRecBytes;
    return T.block.at(at) | T.block.at(at + 1) << 8 | T.block.at(at + 2) << 16;
}

static int test_kept(Tile& T, int m) {
    if (m > tl::kLanes) return fails("records tested at once", m, tl::kLanes);
    for (int lane = 0; lane < m; ++lane) T.tested.at(get_record(T, lane))++;
    return 0;
}

// own: the list is the tile's own bin and is taken as it is
static int run_tile(Tile& T, bool own) {
    const int N = tl::kLanes, cnt = (int)T.hit.size(), kNone = -2;
    std::vector<int> pend(N, 0), over(N, 0), batch(N, 0);
    long long c0 = 0;
    int np = 0, m = 0;
    uint64_t todo = 0;
    bool last = cnt == 0;
    for (int guard = 0; cnt > 0; ++guard) {
        if (guard > 4 * cnt + 8) return fails("the loop does not end", guard, cnt);
        if (todo == 0) {
            over.assign(N, 0);
            if (own) {
                for (int l = 0; l < N; ++l) pend[l] = c0 + l < cnt ? (int)(c0 + l) : 0;
                np = (int)std::min<long long>(tl::kChunk, cnt - c0);
                c0 += tl::kChunk;
            } else {
                while (np < tl::kChunk && c0 < cnt) {
                    uint64_t hits = 0;
                    for (int l = 0; l < N; ++l)
                        if (c0 + l < cnt && T.hit[c0 + l]) hits |= 1ull << l;
                    const int add = __builtin_popcountll(hits);
                    std::vector<int> moved(N, kNone);
                    for (int l = 0; l < N; ++l) {
                        const uint64_t below = l == 0 ? 0 : ~0ull >> (64 - l);
                        const bool h = (hits >> l) & 1;
                        const int to = (np + (h ? __builtin_popcountll(hits & below) : add)) & (tl::kChunk - 1);
                        if (h) {
                            if (moved[to] >= 0) return fails("two hits moved to one place", to, l);
                            moved[to] = (int)(c0 + l);
                        } else if (moved[to] >= 0) {
                            return fails("a lane without a hit moved over one", to, l);
                        } else {
                            moved[to] = -1;
                        }
                    }
                    for (int l = 0; l < N; ++l) {
                        if (l >= np && l < np + add) {
                            if (moved[l] < 0) return fails("a place nothing was moved to is read", l, np);
                            pend[l] = moved[l];
                        }
                        if (l < np + add - tl::kChunk) {
                            if (moved[l] < 0) return fails("a held place nothing was moved to is read", l, np);
                            over[l] = moved[l];
                        }
                    }
                    np += add;
                    c0 += tl::kChunk;
                }
            }
            batch = pend;
            const int nb = std::min(np, tl::kChunk);
            todo = nb == tl::kChunk ? ~0ull : (1ull << nb) - 1;
            np -= nb;
            if (np > tl::kChunk) return fails("ids held over", np, tl::kChunk);
            pend = over;
            last = c0 >= cnt && np == 0;
        }
        uint64_t kept = 0, beyond = 0;
        for (int l = 0; l < N; ++l)
            if (((todo >> l) & 1) && T.keep.at(batch[l]) && (own ? T.hit.at(batch[l]) : true)) kept |= 1ull << l;
        for (int l = 0; l < N; ++l) {
            const uint64_t below = l == 0 ? 0 : ~0ull >> (64 - l);
            const int dst = m + __builtin_popcountll(kept & below);
            if (dst >= tl::kChunk) beyond |= 1ull << l;
            if (((kept >> l) & 1) && dst < tl::kChunk && !put_record(T, dst, batch[l]))
                return fails("record place", dst, T.bytes);
        }
        m += __builtin_popcountll(kept);
        todo = m > tl::kChunk ? kept & beyond : 0;
        const bool end = todo == 0 && last;
        if (m > tl::kChunk || (end && m > 0)) {
            if (test_kept(T, std::min(m, (int)tl::kChunk))) return 1;
            m = 0;
        }
        if (end) break;
    }
    for (int i = 0; i < cnt; ++i)
        if (T.tested[i] != (T.hit[i] && T.keep[i] ? 1 : 0)) return fails("times a face is tested", i, T.tested[i]);
    return 0;
}

// ------------------------------------------------------------- the write-out

// An output array of n words a slot; every word is written once with its tag.
struct Out {
    int n, H, W, K;
    std::vector<int64_t> word;
    Out(int n_, int H_, int W_, int K_) : n(n_), H(H_), W(W_), K(K_), word((size_t)n_ * H_ * W_ * K_, -1) {}
};
// the tag of word x of slot k of the tile's pixel
static int64_t tag(int pixel, int k, int x) { return ((int64_t)pixel * 64 + k) * 4 + x; }

static int put(Out& o, long long at, int64_t v) {
    if (at < 0 || at >= (long long)o.word.size()) return fails("output word", at, (long long)o.word.size());
    if (o.word[at] >= 0) return fails("output word written twice", at, v);
    o.word[at] = v;
    return 0;
}

// One staged pass (store_staged): G slots from g0 on, n words each, pixel stride S words.
static int store_staged(Out& o, const std::vector<int64_t>& stage, long long base, int rows, int cols, int g0, int G,
                        int S, bool aligned) {
    const int n = o.n, Q = n * G / 4, left = n * (o.K - g0);
    if (n * G % 4) return fails("words of a pass", n, G);
    for (int lane = 0; lane < tl::kLanes; ++lane) {
        int px = lane / Q, q = lane - px * Q;
        for (int e0 = 0; e0 < 64 * Q; e0 += 64) {
            const int r = px >> 3, c = px & 7;
            if (px < 0 || px >= 64 || q < 0 || q >= Q) return fails("staged quad", px, q);
            if (r < rows && c < cols) {
                const long long dst = base + (long long)n * (r * (o.W * o.K) + c * o.K + g0) + 4 * q;
                if (aligned && dst % 4) return fails("alignment of a store", dst, 4);
                const int words = aligned || 4 * q + 4 <= left ? 4 : 3;
                for (int i = 0; i < words; ++i)
                    if (words == 4 || 4 * q + i < left)
                        if (put(o, dst + i, stage.at(px * S + 4 * q + i))) return 1;
            }
            px += 64 / Q;
            q += 64 % Q;
            if (64 % Q != 0 && q >= Q) {
                q -= Q;
                ++px;
            }
        }
    }
    return 0;
}

static int fill_rows(Out& o, int KB, long long base, int rows, int cols, bool aligned, int64_t v) {
    const int n = o.n;
    for (int lane = 0; lane < tl::kLanes; ++lane) {
        if (aligned) {
            const int Q = n * KB * 8 / 4, nq = n * KB * cols / 4;
            for (int e0 = 0; e0 < 8 * Q; e0 += 64) {
                const int e = e0 + lane, r = e / Q, q = e - r * Q;
                if (e < 8 * Q && r < rows && q < nq)
                    for (int i = 0; i < 4; ++i)
                        if (put(o, base + (long long)n * r * (o.W * o.K) + 4 * q + i, v)) return 1;
            }
        } else {
            const int w = n * cols * o.K;
            for (int r = 0; r < rows; ++r)
                for (int i = 4 * lane; i < w; i += 256)
                    for (int j = i; j < std::min(i + 4, w); ++j)
                        if (put(o, base + (long long)n * r * (o.W * o.K) + j, v)) return 1;
        }
    }
    return 0;
}

static int write_out(int bytes, int KB, int K, int H, int W, int ty, int tx, bool empty) {
    const bool aligned = K == KB;
    const int rows = std::min(8, H - 8 * ty), cols = std::min(8, W - 8 * tx);
    for (int array = 0; array < 4; ++array) {  // ids, depths, barycentrics, distances
        const int n = array == 2 ? 3 : 1;
        Out o(n, H, W, K);
        const long long base = n * (((long long)8 * ty * W + 8 * tx) * K);
        if (empty) {
            if (fill_rows(o, KB, base, rows, cols, aligned, 0)) return 1;
        } else {
            const int G = tl::stage_slots(KB, array < 2 ? tl::kStageG1 : tl::kStageG2);
            const int S = tl::stage_stride(n, G);
            for (int g0 = 0; g0 < KB; g0 += G) {
                if (g0 >= K) continue;
                std::vector<int64_t> stage(bytes / 4, -1);
                for (int lane = 0; lane < tl::kLanes; ++lane)
                    for (int k = 0; k < G; ++k)
                        for (int x = 0; x < n; ++x) {
                            const int at = lane * S + n * k + x;
                            if (at >= (int)stage.size()) return fails("staged word", at, (long long)stage.size());
                            stage[at] = tag(lane, g0 + k, x);
                        }
                if (store_staged(o, stage, base, rows, cols, g0, G, S, aligned)) return 1;
            }
        }
        long long written = 0;
        for (int r = 0; r < H; ++r)
            for (int c = 0; c < W; ++c)
                for (int k = 0; k < K; ++k)
                    for (int x = 0; x < n; ++x) {
                        const int64_t v = o.word[(size_t)n * (((long long)r * W + c) * K + k) + x];
                        const int lr = r - 8 * ty, lc = c - 8 * tx;
                        const bool in = lr >= 0 && lr < rows && lc >= 0 && lc < cols;
                        const int64_t want = !in ? -1 : (empty ? 0 : tag(8 * lr + lc, k, x));
                        if (v != want) return fails("value of an output word", v, want);
                        written += in;
                    }
        if (written != (long long)rows * cols * K * n) return fails("words written", written, rows * cols * K * n);
    }
    return 0;
}

int main(int argc, char** argv) {
    const int bytes = argc > 1 ? std::atoi(argv[1]) : tl::kBlockBytes;
    const int counts[] = {0, 1, 2, 63, 64, 65, 100, 127, 128, 129, 191, 192, 500, 1000};
    const double share[] = {0.0, 0.02, 0.3, 0.7, 0.98, 1.0};
    for (int own = 0; own < 2; ++own)
        for (int cnt : counts)
            for (double ph : share)
                for (double pk : share)
                    for (int rep = 0; rep < 3; ++rep) {
                        Tile T;
                        T.bytes = bytes;
                        T.block.assign(bytes, 0);
                        T.tested.assign(cnt, 0);
                        std::bernoulli_distribution h(ph), k(pk);
                        for (int i = 0; i < cnt; ++i) {
                            T.hit.push_back(h(rng));
                            T.keep.push_back(k(rng));
                        }
                        if (run_tile(T, own != 0)) return 1;
                    }
    for (int KB : {4, 8, 16, 32, 64})
        for (int K = KB / 2 + 1; K <= KB; ++K)
            for (int empty = 0; empty < 2; ++empty)
                for (int cut = 1; cut <= 8; ++cut)
                    if (write_out(bytes, KB, K, 16, 8 + cut, 1, 1, empty != 0) ||
                        write_out(bytes, KB, K, 8 + cut, 16, 1, 1, empty != 0) ||
                        write_out(bytes, KB, K, cut, 9 - cut, 0, 0, empty != 0))
                        return 1;
    std::printf("ok: block of %d bytes\n", bytes);
    return 0;
}
