// The host planner of a round: argument validation, rotation tables, block-table slices, layout tables and the
// work list, as host vectors.  Nothing here touches the GPU or includes HIP, so the whole planner runs (and is
// fuzzed under AddressSanitizer / UBSan) on machines without one; tdk_api.cpp uploads what it returns.
#pragma once

#include <stdint.h>

#include <string>
#include <vector>

#include "tdk.h"
#include "tdk_types.h"

namespace tdk {

struct PlanSession {
  int32_t span = 0, pages = 0;
  int64_t master_pos0 = 0, master_row0 = 0;
  std::vector<int32_t> agents;   // ids of its agents, in descriptor order
};

struct RoundPlan {
  std::vector<PlanSession> sessions;
  // what the device gets
  std::vector<SessionDev> sess;
  std::vector<AgentDev>   agents;
  std::vector<int32_t>    order;      // agent ids grouped by session
  std::vector<int32_t>    bt;         // block-table slices that cover the shared spans, concatenated
  std::vector<float>      tab;        // [n_agents][2][64]: cos then sin of dst_pos0 - master_pos0
  std::vector<float>      tab_diff;   // the same for dst_pos0 - diff_pos0
  bool any_segments = false;          // some agent has its own block layout: the vectors below are filled
  std::vector<int32_t>    rowmap;     // pool row of (agent, master token)
  std::vector<PageTab>    pagetab;    // per (agent, master page)
  std::vector<float>      segtab, segtab_diff;   // one table per (agent, segment)
  std::vector<int32_t>    seg_off, seg_src;      // per agent the range of its segments, their first master tokens
  // totals
  int64_t max_phys_page = -1;         // largest page number any shared span maps to
  int64_t total_pages = 0;            // sum over agents of their session's page count
  int64_t total_master_pages = 0, total_master_rows = 0;
  int64_t total_tokens = 0;           // sum over agents of their session's span
  int32_t max_segments = 1;           // most segments any agent has (1 for identity layouts)
  bool seg_moved = false;             // a segmented agent's stored diff sits at other positions
  bool seg_apart = false;             // and segments of one agent have moved by different distances
  bool diff_moved = false;            // some agent's stored diff sits at other positions (segmented or not)
  size_t work_capacity = 0;           // work items in the worst case (every agent its own group)
};

// Every function returns TDK_OK or the status to hand to the caller, with the reason in `err`.
tdk_status plan_check_model(const tdk_model* m, std::string& err);
tdk_status plan_round(const tdk_model* model, const tdk_session* sessions, int32_t n_sessions,
                      const tdk_agent* agents, int32_t n_agents, RoundPlan& p, std::string& err);

// Work list for `group` agents per item in the order of a static launch (item i runs on XCD i % 8), and the same
// items grouped by that XCD (queue x = queued[q_begin[x] .. q_begin[x + 1])).
void plan_work(const std::vector<PlanSession>& sessions, int group, bool taper, std::vector<WorkItem>& work);
void plan_queues(const std::vector<WorkItem>& work, std::vector<WorkItem>& queued, int32_t (&q_begin)[9]);
// A work list as the kernels read it, added to `items`.  order: agent ids grouped by session; agents: their descriptors, in the caller's order
void plan_items(const std::vector<PlanSession>& sessions, const std::vector<int32_t>& order, const std::vector<AgentDev>& agents, int page_tokens,
                const std::vector<WorkItem>& work, std::vector<ItemDev>& items);
// agents per work item when the caller names none; page_bytes: K and V of one page; planes: written by the call (2, or 1)
int  plan_auto_group(const std::vector<PlanSession>& sessions, bool read_kernels = false, int64_t page_bytes = 64 * 1024,
                     int n_cus = 256, int planes = 2);
// Workgroups that copy listed pages, for at most so many slots: more than one per slot where the kernel shares them out, down to one of
// its batches of accesses per thread.  left: places on the chip that the launch's other workgroups leave
int  plan_copy_workgroups(int slots, int batches, int n_cus, int left);
// Is a launch of the kernels that write long enough for the form that loops?  items, pairs: work items and (agent, page) pairs; rows: accesses
// per page and wavefront; pack: several rows per access; planes: bit 0 = K, bit 1 = V; seg: some agent has a block order of its own
bool plan_loops(int64_t items, int64_t pairs, int n_cus, int rows, bool pack, int planes, bool seg);

// Attention over mirrors that are never restored: what the planner needs to know of a round.
struct AttendShape {
  const std::vector<PlanSession>* sessions = nullptr;
  int32_t n_agents = 0, heads = 1, page_tokens = 16, n_cus = 256, max_segments = 1;
  bool seg = false, seg_moved = false, seg_apart = false;      // as in RoundPlan (any_segments, seg_moved, seg_apart)
  int64_t total_tokens = 0, total_master_rows = 0;
};

constexpr int64_t kMaxBlocks = (int64_t)1 << 31;     // workgroups of one launch: ids are int32

// Shape of the attention pass for a call: tokens per workgroup of the master pass, parts per query row, the launch, and
// the layout of the caller's workspace.
struct AttendPlan {
  int32_t all_chunks = 0;          // chunks that every session with agents and a span has
  int32_t chunk_tokens = 0, n_chunks = 0, n_parts = 0, max_rows = 0, n_pieces = 1, piece_tokens = 0, piece_grid = 1;
  bool    own_rows = false;        // one agent per wavefront (tdk_attend_rows_kernel)
  bool    pipelined = false;       // the shared launch's master pass with pipelined steps
  int32_t max_agents = 0;
  int32_t launch_sessions = 0;     // own_rows: sessions per launch
  int64_t rows = 0;
  int64_t blocks = 0;              // workgroups of the largest launch; the call is refused from kMaxBlocks on
  FusedGrid fused{};               // the shared launch (identity layouts, not own_rows, blocks < kMaxBlocks)
  size_t o_qrot = 0, o_qdiff = 0, o_part_o = 0, o_part_m = 0, o_part_l = 0, bytes = 0;
};
// workspace: bytes that the call brings.  Where the estimates choose the cut, they choose among those that fit; a plan that needs more
// says so in `bytes`.  false: bad arguments
bool attend_plan(const AttendShape& r, int32_t n_q, int32_t n_q_heads, AttendPlan& p, size_t workspace = SIZE_MAX);
size_t attend_workspace_bytes(const AttendShape& r, int32_t n_q, int32_t n_q_heads);     // covers every call of up to n_q query tokens; 0: bad arguments

}  // namespace tdk
