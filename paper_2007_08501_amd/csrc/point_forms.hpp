// point_forms.hpp -- which form the point backward takes, and the chunk size
// of its slot-major form, from the sizes of a call.  Plain C++ (no HIP types):
// the launcher (kernels_points.hip) and the CPU test of the rule both use it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace rast {

constexpr int kPtTile = 8;                        // pixels a side of a tile
constexpr int kSlotCapMin = 7, kSlotCapMax = 10;  // log2 of the points per chunk
constexpr size_t kSlotLdsMax = 64 * 1024;
constexpr int kSlotGroups = 7;                    // workgroups of a compute unit, by the kernel's registers
constexpr size_t kSlotLdsShare = 23040;           // LDS of each of them
constexpr int64_t kBoxLdsMax = 64 * 1024;

// Pixel columns (or rows) a disc reaches past its first: at most
// floor(r size + 0.03), the ranges being widened by 0.01 pixel at each end.
inline int pt_span(float radius, int size) {
    return (int)std::fmin(std::floor((double)radius * size + 0.05), (double)size);
}

// The slot-major form's chunk: log2 of its points and of its table's entries,
// and its LDS bytes (table entries of 8, a place and the cells of each point).
// lg_cap 0: the cells of the smallest chunk do not fit.
//
// The capacity is the smallest that holds about twice the points of a covered
// tile's mean (half of the tiles taken as covered), or more where kSlotGroups
// workgroups a compute unit have the room: a tile takes a table by its own
// points, so that the room costs nothing, and a cloud that covers a part of the
// image has tiles far above the mean.  The table is at most half full, a
// quarter where there is room for that too (4 clouds of 20,000 points on 77 x
// 77 pixels, 36 cells, K = 8: 31 us half full, 24 a quarter; on 16 x 16 pixels,
// 9 cells, K = 50: 58 and 31).
struct PtSlots {
    int lg_cap, lg_table;
    size_t bytes;
};
inline size_t pt_slot_bytes(int lg_cap, int lg_table, int64_t ncell) {
    const size_t cap = (size_t)1 << lg_cap;
    return ((size_t)8 << lg_table) + 4 * cap + ((cap * (size_t)ncell + 3) & ~(size_t)3);
}
inline PtSlots pt_slots(int64_t P, int64_t T, int64_t ncell) {
    int lg = kSlotCapMin;
    while (lg < kSlotCapMax && 4 * P > T << lg) ++lg;
    while (lg < kSlotCapMax && pt_slot_bytes(lg + 1, lg + 2, ncell) <= kSlotLdsShare) ++lg;
    while (lg >= kSlotCapMin && pt_slot_bytes(lg, lg + 1, ncell) > kSlotLdsMax) --lg;
    if (lg < kSlotCapMin) return PtSlots{0, 0, 0};
    const int lt = pt_slot_bytes(lg, lg + 2, ncell) <= kSlotLdsShare ? lg + 2 : lg + 1;
    return PtSlots{lg, lt, pt_slot_bytes(lg, lt, ncell)};
}

// LDS bytes of the box-staged form (a tile's pixel box with its ids and up to
// two gradients), or 0 when it does not fit.
inline size_t pt_box_bytes(int H, int W, int K, int span_x, int span_y, bool gz, bool gd) {
    const int64_t bw = std::min(kPtTile + span_x, W), bh = std::min(kPtTile + span_y, H);
    const int64_t bytes = bw * bh * ((K + 3) & ~3) * 4 * (1 + (gz ? 1 : 0) + (gd ? 1 : 0));
    return bytes <= kBoxLdsMax ? (size_t)bytes : 0;
}

enum PtBwdForm { kPtBwdSlots, kPtBwdBox, kPtBwdPoints };
inline PtBwdForm pt_bwd_form(int N, int H, int W, int K, int64_t P, float radius, bool gz, bool gd) {
    const int sx = pt_span(radius, W), sy = pt_span(radius, H);
    const int64_t T = (int64_t)N * ((H + kPtTile - 1) / kPtTile) * ((W + kPtTile - 1) / kPtTile);
    if (pt_slots(P, T, (int64_t)(sx + 1) * (sy + 1)).lg_cap > 0) return kPtBwdSlots;
    return pt_box_bytes(H, W, K, sx, sy, gz, gd) > 0 ? kPtBwdBox : kPtBwdPoints;
}

}  // namespace rast
