// Plain descriptor types of a round, shared by the host planner (no HIP needed) and the kernels.
#pragma once

#include <stdint.h>

namespace tdk {

constexpr int kMaxGroup = 32;     // agents that share one read of a master page
constexpr int kBlock = 256;       // threads per workgroup (4 wavefronts of 64)
constexpr int kWaves = kBlock / 64;
constexpr int kHeadDim = 128;
constexpr int kHalf = kHeadDim / 2;

// One unit of work of the page kernels: a master page and a group of agents of its session.
struct WorkItem {
  int32_t session;
  int32_t page;        // master page number
  int32_t ag_begin;    // range in RoundDev::order
  int32_t ag_count;    // 1..kMaxGroup
};

// The same as the page kernels read it: one scalar read gives everything that the item's first accesses depend on.  A chain through
// the item, its session and its agents to the block table is five reads deep, and each of them is a memory latency.
struct alignas(16) ItemDev {
  int64_t row0;        // the page's first row in master_k / master_v
  int32_t page;        // master page number
  int32_t counts;      // agents of the group, and from bit 8 on the page's rows inside the span
  int32_t agent0;      // id of the first agent where the group's agents have consecutive ids, else -1
  int32_t order0;      // the group's place in RoundDev::order
  int32_t flat0;       // the first agent's (agent, page) pair, agents in descriptor order; the next agent's is `pages` later
  int32_t pages;       // pages of the session
  int32_t score0;      // the first agent's (agent, token) pair of the page's first token; the next agent's is `span` later
  int32_t span;        // tokens of the session
  int32_t pad[2];
};

// Where a master page lies in an agent's pool (identity layouts).
struct alignas(16) PlaceDev {
  int32_t pg0;         // physical page of its first token
  int32_t pg1;         // the next logical page's physical page, -1 past the block table
  int32_t off;         // row of the first token in pg0
  int32_t pad;
};

struct SessionDev {
  int64_t master_row0;  // first row of this session in master_k / master_v
  int32_t span;         // S
  int32_t pages;        // ceil(S / T)
  int32_t order_begin;  // its agents are RoundDev::order[order_begin .. order_begin + n_agents)
  int32_t n_agents;
};

struct AgentDev {
  int32_t pos0;         // dst_pos0 (validated < 2^31)
  int32_t bt_off;       // start of this agent's block-table slice in RoundDev::bt
  int32_t lp_first;     // logical page number of slice entry 0 (= pos0 / T)
  int32_t bt_len;       // entries in the slice
  int32_t session;
  int32_t flag_off;     // start of this agent's per-page flags in the flag scratch
  int32_t score_off;    // start of this agent's per-token scores (sum of the spans of earlier agents)
  int32_t diff_rot;     // bit 0: payload K rows of this agent were stored at another position (re-rotate on restore);
                        // bit 1: and every segment of its layout has moved by the same distance
};

// Per (agent, master page) of a round with per-agent block layouts: the rotation tables of the (at most two)
// segments the page meets, which rows use the second, and which of the two runs moved since the stored diff
// was encoded.  Read by the kernels as one 16-byte word.
struct alignas(16) PageTab {
  int32_t x;   // first table
  int32_t y;   // second table (= x if the page lies in one segment)
  int32_t z;   // bit r: row r uses the second table
  int32_t w;   // bit t: table t's run sat at another position when the stored diff was encoded
};

// Grid of the attention launch that holds the master pass and the listed-pages pass.
struct FusedGrid {
  int32_t n_master;      // workgroups of the master pass: heads * (sessions * chunks) * row blocks
  int32_t row_blocks;    // blocks of 128 query rows per session and KV head
  int32_t n_diff0;       // workgroups of the listed-pages pass per piece: agents * head_groups
  int32_t head_groups;   // ceil(heads / 4)
};

}  // namespace tdk
