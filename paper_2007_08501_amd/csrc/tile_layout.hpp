// tile_layout.hpp -- sizes of the mesh fine pass's LDS block, shared by the
// kernel (kernels_fwd.hip) and the bounds-checked CPU models of its index
// arithmetic (tests/cpu_models/tile_block_model.cpp, tile_lds_model.cpp).  Plain
// C++: no HIP types.
//
// One 64-lane wave rasterizes one 8x8 tile.  It gathers up to 64 faces at a
// time, one a lane, and appends those that may cover a pixel to the block, as
// tile records of kTileRecBytes; a full block (kChunk records) or the last faces
// are tested: lane j reads record j's pixel mask and a bit transpose across the
// wave gives every lane the records that may cover its pixel (bit j = record
// j).  After the last test the same block stages the fragments for coalesced
// stores, one output array at a time: kStageG1 slots a pixel of ids or depths,
// kStageG2 slots of barycentrics or distances, per pass.
#pragma once

namespace rast {
namespace tile_layout {

constexpr int kLanes = 64;         // wave width, one lane per tile pixel
constexpr int kChunk = 64;         // records of a block: the transpose takes one per lane
constexpr int kTileRecBytes = 96;  // a face as the tile pass keeps it
constexpr int kStageG1 = 16;       // slots per staging pass for ids and depths
constexpr int kStageG2 = 8;        // slots per staging pass for barycentrics and distances
constexpr int kRecBytes = kChunk * kTileRecBytes;

static_assert(kChunk == kLanes, "the gather gives every lane one face, and the transpose one record per lane");

// Slots a pixel of one staging pass for a queue of kb, and the words from one
// pixel's to the next one's for n words a slot: odd, so that lanes writing their
// own pixels hit distinct banks.
constexpr int stage_slots(int kb, int most) { return kb < most ? kb : most; }
constexpr int stage_stride(int n, int slots) { return n * slots + 1; }

// The block: the staging never takes more than the records plus one word a lane
// (three barycentrics of kStageG2 slots).
constexpr int kBlockBytes = kRecBytes + 4 * kLanes;
static_assert(4 * kLanes * stage_stride(1, kStageG1) <= kBlockBytes, "id or depth staging exceeds the block");
static_assert(4 * kLanes * stage_stride(3, kStageG2) <= kBlockBytes, "barycentric staging exceeds the block");

// A larger block that stages two arrays side by side, which the kernel does not
// use: tile_lds_model.cpp replays the gather of one chunk, the transpose and such
// a staging in it.
constexpr int kSpareBytes = 4096;
constexpr int kLdsBytes = kRecBytes + kSpareBytes;
constexpr int stage_words_g1(int kb) { return 2 * kLanes * stage_stride(1, stage_slots(kb, kStageG1)); }
constexpr int stage_words_g2(int kb) {
    return kLanes * (stage_stride(3, stage_slots(kb, kStageG2)) + stage_stride(1, stage_slots(kb, kStageG2)));
}
static_assert(4 * stage_words_g1(64) <= kLdsBytes && 4 * stage_words_g2(64) <= kLdsBytes, "two arrays exceed it");

}  // namespace tile_layout
}  // namespace rast
