// Device execution tables of a chunk-scheduled GEMM, built on the host from the
// chunk-ordered tile list: the work units in execution order (one sub-list per die),
// each unit's chunk list, and the chunk copy items of the kernel copy backend. Plans
// upload them to memory they own; the allocation-free entry point writes them into the
// library's static scratch.
#pragma once

#include <cstdint>
#include <vector>

#include "kernels.hpp"
#include "planner.hpp"

namespace csg {

struct ExecOptions {
  bool consumer = true;     // AG / grouped (units wait for remote chunks) vs producer (units signal chunks)
  int64_t K = 0;
  int64_t in_bytes = 2;     // bytes per element of A
  int32_t bk = 64;
  int32_t split_k = 1;      // K-slices of every tile
  int32_t tail_split = 0;   // K-slices of the tiles on the critical path (0/1: none)
  int32_t tail_chunks = 0;  // ... those reading one of the last (consumers) / first (producer) chunks
  int32_t tail_taper = 0;   // 1: the tail split tapers from tail_split (the last / first chunk) to 1
  int32_t tile_dispatch = 0;  // 2: one plain list (dealt statically, die-major), else per-die sub-lists
  int32_t grid = 0;         // persistent workgroups (round-robin over the dies)
  int32_t tail_wave = 0;    // > 1: K-slices (at most) for each die's last partial wave of tiles
  int32_t slots = 0;        // co-resident workgroups that take units; when every unit has one of its
                            // own, units are dealt statically (0: never)
};

struct ExecTables {
  std::vector<TileDesc> units;       // execution order
  std::vector<int32_t> list_ptr;     // [units + 1]
  std::vector<int32_t> list_ids;     // consumers: remote chunks a unit waits for; producer: chunks it writes
  std::vector<int32_t> raster;       // raster id per unit
  std::vector<int32_t> need;         // per chunk: units reading it (consumers) / tiles writing it (producer)
  std::vector<int32_t> list_begin;   // [kXcdLists + 1]: die x runs units [list_begin[x], list_begin[x + 1])
  int32_t ws_slices = 0;             // partial-sum buffers of split tiles
  int32_t tail_begin = 0;            // static dispatch, consumers: first unit of the trailing
                                     // critical tiles, dealt from a shared ticket (0: none)
  bool one_shot = false;             // every unit has a workgroup: unit i goes to static slot i
  bool lines_aligned = true;         // every chunk of A starts on a 128-byte line
};

// Execution tables of a tile map. A tile goes to die (row-tile index mod kXcdLists),
// so tiles sharing A rows share an L2; every sub-list keeps the chunk order.
void build_exec_tables(const Schedule& s, const TileMap& m, const ExecOptions& o, ExecTables* out);

// The tiles a kernel runs a tile map's rows in, and their K-slices.
struct Geometry {
  int32_t bm = 0, bn = 0, split = 1;
};

// Geometry of a plan that names neither tile shape nor split: bf16, 256 x 256 tiles
// unless they would leave most of the device's `slots` workgroups (one per CU) idle, and
// then the tile shape and the number of K-slices with the shortest estimated kernel; fp32,
// 64 x 64 tiles, in K-slices where they would.
//   group_rows: rows per group (one entry where nothing is grouped)
//   min_bn: narrowest tiles; may_split: slices may be used; ws_bytes: partial sums they may take
Geometry choose_geometry(bool bf16, const std::vector<int64_t>& group_rows, int64_t N, int64_t K, int32_t slots,
                         int32_t min_bn, bool may_split, int64_t ws_bytes);

// Copy items of the kernel copy backend: every chunk of `moved` (chunk ids, in the
// order the copy workgroups move them) cut into slabs of at most `slab` bytes of
// rows of `row_bytes`; parts[i] = the items of moved[i].
void build_copy_items(const Schedule& s, const std::vector<int32_t>& moved, int64_t row_bytes, int64_t slab,
                      std::vector<CopyItem>* items, std::vector<int32_t>* parts);

}  // namespace csg
