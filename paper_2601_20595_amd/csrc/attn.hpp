// Interface between the host runtime and the ring-attention kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace csg {

constexpr int kAttnHeadDim = 128;  // head dimension the kernel is built for
constexpr int kAttnBlockQ = 128;   // query rows per work unit
constexpr int kAttnBlockKV = 64;   // key rows per inner step (chunks are multiples of it)

// Key slices per (query block, head) for `whole` of them and n_blocks key blocks, on a
// device with `slots` co-resident workgroups. A wave spends about 2.1 us per block with one
// or with two waves on its SIMD, so slices are added until every slot has a unit; writing
// and merging partial results costs about 8 us, and a slice keeps at least six blocks.
inline int32_t attn_slices(int64_t whole, int32_t n_blocks, int32_t slots) {
  int32_t s = 1;
  while (s < 8 && whole * (s + 1) <= slots && n_blocks >= 6 * (s + 1)) ++s;
  return s;
}

struct AttnArgs {
  const uint16_t* Q;          // [Sq][H][D] bf16
  const uint16_t* K;          // [S][Hkv][D] bf16, the landing buffer
  const uint16_t* V;          // [S][Hkv][D] bf16, the landing buffer
  uint16_t* O;                // [Sq][H][D] bf16
  float* LSE;                 // [H][Sq] natural-log log-sum-exp of the scaled scores
  int32_t Sq, H, Hkv;
  int32_t n_units;            // work units: ceil(Sq / kAttnBlockQ) * H * slices
  int32_t slices;             // key slices per (query block, head); 1: not split
  int32_t n_blocks;           // key blocks of kAttnBlockKV rows, all chunks together
  float* ws;                  // slices > 1: partial results, kAttnPartBytes per unit
  uint32_t* slot_count;       // slices > 1: finished slices per (query block, head)
  int32_t n_chunks;
  const int32_t* arrival;     // [n_chunks]: chunk id at each arrival position
  const int32_t* chunk_rows;  // [2 * n_chunks] by chunk id: key row begin, end
  const int32_t* first_block; // [n_chunks + 1] by arrival position: key blocks of the chunks before it
  const int32_t* need;        // [n_chunks] by chunk id: units that read it, 0 if it is local (slices > 1)
  const int64_t* const* ready;  // per chunk id: 0 once its keys and values have landed
  int64_t* const* relay;        // [n_chunks]: word in device memory that a unit which saw the value 0 clears
                                // (a local chunk's: a word that reads 0)
  uint32_t* counters;         // per chunk id: units done reading it
  uint32_t* out_flags;        // per chunk id: the call number once every unit has read it
  uint32_t* ticket;           // [kXcdLists] work-unit tickets, one per die's range of units
  DeviceDiag* diag;
  uint64_t timeout_ticks;
  uint32_t epoch;
  float scale_log2;           // softmax scale times log2(e)
  // the next call's state set, cleared by workgroup 0 at the start (null: not here)
  uint32_t* next_ticket;
  uint32_t* next_counters;
  DeviceDiag* next_diag;
  uint32_t* next_slot_count;  // (null where slices is 1)
  int64_t* next_relay;        // relay words of the next call's set, set to 1
  int32_t n_relay;            // remote chunks
};

// A slice's partial results: per thread its 64 output accumulators, its row's reference
// and its share of the row sum.
constexpr int64_t kAttnPartBytes = 256 * (64 + 2) * 4;

int32_t attn_threads();
hipError_t launch_ring_attn(const AttnArgs& args, int32_t grid, hipStream_t stream, hipEvent_t start, hipEvent_t stop);
// Co-resident workgroups of the attention kernel on `device`.
hipError_t attn_grid(int device, int32_t* grid);

}  // namespace csg
