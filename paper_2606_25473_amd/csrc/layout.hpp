// layout.hpp -- host-side mask handling (C++17, no HIP dependency).
#pragma once

#include <stdint.h>

#include <string>

#include "attn_jvp.h"
#include "schedule.hpp"

namespace attn {

// Validate `layout` against the sequence length L and derive its query-group
// table (ranges of each group sorted, empty ones dropped, touching ones merged).
// Returns false and fills *err on an invalid layout.
bool build_groups(const attn_chunk_layout* layout, int L, GroupTable* gt, std::string* err);

// Admissible (query, key) pairs of the mask, one (batch, head).
int64_t count_pairs(const GroupTable& gt);

// Pairs evaluated by a kernel with (uncut) br-row query tiles and bc-key blocks.
int64_t count_computed_pairs(const GroupTable& gt, int L, int br, int bc);

// Key splits per query tile of the bf16 forward and JVP kernels (1: none, 128- and 256-row
// tiles; 2 or 4: tiles of 256 / splits rows) for nbh (batch, head) pairs, and of the backward's
// query-tile pass.
int choose_ksplit(const GroupTable& gt, int L, int nbh, int D = 128);
int choose_bwd_ksplit(const GroupTable& gt, int L, int nbh, int D);

// Query splits per key tile of the bf16 backward's key-tile pass (1: 128-key tiles; else
// kBwdQuerySplits, 64-key tiles).
int choose_qsplit(const GroupTable& gt, int L, int nbh, int D = 128);

// Tile size of an fp32 kernel: 1 for 128 rows (keys), 2 for 64.  kQueryTiles: the JVP and the
// backward's query-tile pass; kKeyTiles: its key-tile pass.
enum class F32Kernel { kForward, kQueryTiles, kKeyTiles };
int choose_f32_tiles(const GroupTable& gt, int L, int nbh, int D, F32Kernel kernel);

// Work-group -> query-tile order for the layout (heaviest tiles first).
TileOrder make_tile_order(const attn_chunk_layout* layout, int L, int br);

// Tile order when the rows below t0 carry no tangent (their tiles need the primal
// only): the tiles wholly below t0 and the others, each heaviest first, merged by
// estimated cost (mode 3; mode 2 beyond kMaxMergeTiles tiles).
TileOrder make_tile_order_zero_clean(const GroupTable& gt, int L, int br, int bc, int t0,
                                     const TileOrder* cuts = nullptr);

// Cut the tiles of `o` (br rows) at the group bounds where that adds few of them.
void cut_tiles(TileOrder* o, const GroupTable& gt, int L, int br);

}  // namespace attn
