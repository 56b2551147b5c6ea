// The launch that opens a pass (see PassSetup in misc_kernels.h): block 0 reserves cache blocks and places the rows in them,
// block 1 builds the attention's task table, block 2 marks the rows whose logits are dumped, the next ceil(T / 32) blocks
// fill the row metadata and the rest gather the embeddings and run the first norm.
// Latency bound: as six to eight launches these took 2 to 60 us each and one after the other (one token: 22 us; 64 tokens
// of 64 sequences: 85 us, 57 of them the task table).
#pragma once

#include "attn_mfma.h"
#include "misc_kernels.h"

namespace hsd {

constexpr int kSetupFixedBlocks = 3, kSetupMetaRows = 32, kSetupEmbedRows = 16;   // rows per block of 1024 threads
inline int setup_blocks(int total_q) {
  return kSetupFixedBlocks + (total_q + kSetupMetaRows - 1) / kSetupMetaRows + (total_q + kSetupEmbedRows - 1) / kSetupEmbedRows;
}

// grid: setup_blocks(total_q) blocks of 1024 threads
template <typename T>
__global__ void __launch_bounds__(1024) k_pass_setup(PassSetup ps) {
  static_assert(kAttnTilesLds >= HSD_MAX_SEQ + 18, "one LDS array for both single-block parts");
  __shared__ __attribute__((aligned(8))) int lds[kAttnTilesLds];
  const int b = static_cast<int>(blockIdx.x) - kSetupFixedBlocks, t = threadIdx.x;
  if (b == -3) {
    kv_reserve_block(ps, lds);
  } else if (b == -2) {
    if (ps.n_wg > 0) attn_tiles_block(ps, lds);
  } else if (b == -1) {
    if (ps.n_dump > 0) dump_slots_block(ps);
  } else {
    const int n_meta = (ps.total_q + kSetupMetaRows - 1) / kSetupMetaRows;
    if (b < n_meta) {
      const int r = b * kSetupMetaRows + (t >> 5);
      if (r < ps.total_q) row_meta(ps, r, t & 31);
    } else {
      const int r = (b - n_meta) * kSetupEmbedRows + (t >> 6);
      if (r < ps.total_q) embed_norm_row<T>(ps, r, t & 63);
    }
  }
}

}  // namespace hsd
