// Host-only driver for the attention planner (attend_plan in csrc/tdk_plan.cpp), built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_attend_plan.py.  Exit code 0 = clean.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "tdk_plan.h"

using namespace tdk;

static uint64_t rng_state = 0x2545F4914F6CDD1Dull;
static uint32_t rnd() {                       // splitmix64, upper half
  uint64_t z = (rng_state += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return (uint32_t)((z ^ (z >> 31)) >> 32);
}
static int64_t between(int64_t lo, int64_t hi) { return lo + (int64_t)(rnd() % (uint32_t)(hi - lo + 1)); }

#define REQUIRE(c) do { if (!(c)) { std::fprintf(stderr, "case %d: requirement failed: %s (line %d)\n", cs, #c, __LINE__); return 1; } } while (0)

struct Made {
  std::vector<PlanSession> sessions;
  AttendShape shape;
  void add(int32_t span, int32_t agents) {
    PlanSession s;
    s.span = span;
    s.pages = (span + shape.page_tokens - 1) / shape.page_tokens;
    for (int32_t i = 0; i < agents; ++i) s.agents.push_back(shape.n_agents + i);
    shape.n_agents += agents;
    shape.total_tokens += (int64_t)span * agents;
    shape.total_master_rows += span;
    sessions.push_back(s);
  }
  const AttendShape& done() { shape.sessions = &sessions; return shape; }
};

static Made draw() {
  Made m;
  m.shape.heads = (int32_t)between(1, 8);
  m.shape.page_tokens = rnd() % 2 ? 16 : 32;
  m.shape.seg = rnd() % 2;
  m.shape.seg_moved = m.shape.seg && rnd() % 2;
  m.shape.seg_apart = m.shape.seg_moved && rnd() % 2;
  m.shape.max_segments = m.shape.seg ? (int32_t)between(1, 40) : 1;
  const int n = (int)between(1, 10);
  const int32_t agents = (int32_t)between(0, 60);
  const int32_t span = rnd() % 4 ? (int32_t)between(1, 26000) : (int32_t)between(0, 70);
  for (int i = 0; i < n; ++i) m.add(rnd() % 2 ? span : (int32_t)between(0, span), rnd() % 3 ? agents : (int32_t)between(0, agents));
  return m;
}

// The launch of a plan, in 128 bits.
static __int128 blocks_of(const AttendShape& s, const AttendPlan& p, int64_t agent_rows) {
  const __int128 sessions = (__int128)s.sessions->size();
  if (p.own_rows) return (__int128)s.heads * (((__int128)p.max_agents * ((agent_rows + 31) / 32) + 3) / 4) * p.launch_sessions * std::max(p.n_chunks, 1);
  const __int128 master = (__int128)s.heads * (((__int128)p.max_rows + 127) / 128) * sessions * p.n_chunks;
  const __int128 lists = s.seg ? (__int128)s.heads * s.n_agents : (__int128)s.n_agents * ((s.heads + 3) / 4);
  return s.seg ? std::max(master, lists * p.piece_grid) : master + lists * p.piece_grid;
}

static int check_grids() {
  int cs = 0;
  for (; cs < 3000; ++cs) {
    Made m = draw();
    const AttendShape& s = m.done();
    const int32_t n_q = rnd() % 2 ? (int32_t)between(1, 9) : (int32_t)between(1, 200), group = (int32_t)between(1, 8);
    AttendPlan p;
    REQUIRE(attend_plan(s, n_q, group * s.heads, p));
    if (s.n_agents == 0) continue;
    REQUIRE((__int128)p.blocks == blocks_of(s, p, (int64_t)n_q * group) && p.blocks < kMaxBlocks);
    REQUIRE(!p.own_rows || p.launch_sessions == (int32_t)s.sessions->size());
    // what the merge reads before it knows a row's session exists in every session (but for empty spans, whose rows have no part)
    for (const auto& hs : m.sessions) REQUIRE(hs.agents.empty() || hs.span == 0 || (int64_t)(p.all_chunks - 1) * p.chunk_tokens < hs.span);
    REQUIRE(p.all_chunks <= p.n_chunks);
    if (!p.own_rows && !s.seg) {
      REQUIRE((int64_t)p.fused.n_master + (int64_t)p.fused.n_diff0 * p.piece_grid == p.blocks);
      REQUIRE(p.fused.n_master == (int64_t)s.heads * p.fused.row_blocks * (int64_t)s.sessions->size() * p.n_chunks);
    }
  }
  // One wide session among very many small ones: the master pass's grid is all sessions times the widest, which does not
  // fit 32 bits although rows, lists and pages do.  The plan says so instead of wrapping around.
  for (int32_t group : {4, 32, 40}) {
    Made m;
    m.shape.heads = 8;
    m.add(600, 8192);
    for (int i = 1; i < 131072; ++i) m.add(16, 0);
    const AttendShape& s = m.done();
    AttendPlan p;
    REQUIRE(attend_plan(s, 1, 8 * group, p));
    REQUIRE((__int128)p.blocks == blocks_of(s, p, group));
    // (40 rows: a wavefront per agent, whose launch takes as many of the sessions as fit)
    REQUIRE((p.blocks >= kMaxBlocks) == (group == 32));
    REQUIRE(group == 4 || p.fused.n_master == 0);
    REQUIRE(group != 40 || (p.own_rows && p.launch_sessions >= 1 && p.launch_sessions < 131072 &&
                            (__int128)p.blocks / p.launch_sessions * (p.launch_sessions + 1) >= kMaxBlocks));
  }
  return 0;
}

// A workspace sized for n_q query tokens serves every shorter call.
static int check_workspace() {
  int cs = 0;
  for (; cs < 400; ++cs) {
    Made m = draw();
    const AttendShape& s = m.done();
    const int32_t group = rnd() % 4 ? (int32_t)between(1, 9) : (int32_t)between(1, 48);
    const int32_t top = (int32_t)between(1, 90);
    size_t before = 0, need = 0;
    for (int32_t n_q = 1; n_q <= top; ++n_q) {
      AttendPlan p;
      REQUIRE(attend_plan(s, n_q, group * s.heads, p));
      need = std::max(need, p.bytes);
      const size_t asked = attend_workspace_bytes(s, n_q, group * s.heads);
      REQUIRE(asked >= need && asked >= before);
      before = asked;
    }
  }
  // 25 agents, 5000 tokens, 40 query heads on 8 KV heads: two query tokens need more than 64
  Made m;
  m.shape.heads = 8;
  m.add(5000, 25);
  AttendPlan two, long_call;
  REQUIRE(attend_plan(m.done(), 2, 40, two) && attend_plan(m.done(), 64, 40, long_call));
  REQUIRE(two.bytes > long_call.bytes && attend_workspace_bytes(m.done(), 64, 40) >= two.bytes);
  REQUIRE(attend_workspace_bytes(m.done(), 0, 40) == 0 && attend_workspace_bytes(m.done(), 1, 41) == 0);
  return 0;
}

// A call that brings less than the plan of its own choice takes is cut coarser: down to what chunks of 512 tokens and more take
// it is served, whatever the estimates prefer.
static int check_small_workspace() {
  int cs = 0, cut = 0;
  for (; cs < 3000; ++cs) {
    Made m;
    if (cs % 3 == 0) {
      m = draw();
    } else {                     // short spans in the master's order
      m.shape.heads = 1 << between(0, 3);
      m.shape.page_tokens = rnd() % 2 ? 16 : 32;
      for (int i = (int)between(1, 4); i > 0; --i) m.add((int32_t)between(1, 2500), (int32_t)between(1, 40));
    }
    const AttendShape& s = m.done();
    const int32_t heads = s.heads * (int32_t)between(1, 9), n_q = (int32_t)between(1, 6);
    AttendPlan free_choice, least, p;
    REQUIRE(attend_plan(s, n_q, heads, free_choice) && attend_plan(s, n_q, heads, least, 0));
    if (s.n_agents == 0) continue;
    // exactly what the free choice takes changes nothing
    REQUIRE(attend_plan(s, n_q, heads, p, free_choice.bytes) && p.own_rows == free_choice.own_rows && p.chunk_tokens == free_choice.chunk_tokens);
    if (least.bytes >= free_choice.bytes) continue;
    ++cut;
    for (size_t bytes : {least.bytes, least.bytes + (free_choice.bytes - least.bytes) / 3, free_choice.bytes - 1}) {
      REQUIRE(attend_plan(s, n_q, heads, p, bytes));
      REQUIRE(p.bytes <= bytes && p.n_parts <= free_choice.n_parts);
      REQUIRE((__int128)p.blocks == blocks_of(s, p, (int64_t)n_q * (heads / s.heads)) && p.blocks < kMaxBlocks);
      REQUIRE(!p.own_rows || p.chunk_tokens <= 16384);
      REQUIRE(p.own_rows || p.chunk_tokens <= std::min(128 * s.page_tokens, 4096));
    }
  }
  REQUIRE(cut > 400);
  // 22 agents x 2 x 493 tokens, one row: chunks of 64 tokens by choice, one chunk and four pieces where that is what fits
  Made m;
  m.shape.heads = 8;
  m.add(493, 22);
  m.add(493, 22);
  AttendPlan p;
  const size_t one_chunk = 352 * (1 + 4) * 520;
  REQUIRE(attend_plan(m.done(), 1, 8, p) && p.bytes > one_chunk);
  REQUIRE(attend_plan(m.done(), 1, 8, p, one_chunk + 512) && p.bytes <= one_chunk + 512);
  return 0;
}

// Own block orders with few rows per agent: a wavefront per agent on both sides of the rule's lines.
static int check_segment_rule() {
  int cs = 0;
  auto own = [](int sessions, int agents, int span, int heads, int group, bool apart, int n_cus) {
    Made m;
    m.shape.heads = heads;
    m.shape.seg = true;
    m.shape.seg_moved = m.shape.seg_apart = apart;
    m.shape.max_segments = 12;
    m.shape.n_cus = n_cus;
    for (int i = 0; i < sessions; ++i) m.add(span, agents);
    AttendPlan p;
    return attend_plan(m.done(), 1, group * heads, p) ? (int)p.own_rows : -1;
  };
  REQUIRE(own(1, 25, 2500, 8, 1, false, 256) == 1 && own(1, 25, 5000, 8, 1, false, 256) == 0 && own(1, 100, 600, 8, 1, false, 256) == 0);
  REQUIRE(own(4, 6, 5000, 8, 5, false, 256) == 1 && own(4, 12, 3000, 8, 5, false, 256) == 0 && own(1, 100, 600, 8, 5, false, 256) == 0);
  REQUIRE(own(20, 4, 300, 8, 1, false, 256) == 1 && own(4, 22, 530, 8, 4, false, 256) == 1 && own(4, 22, 530, 8, 1, false, 256) == 0);
  REQUIRE(own(10, 25, 200, 8, 4, false, 256) == 0 && own(10, 2, 449, 8, 1, true, 256) == 1 && own(2, 34, 483, 8, 1, true, 256) == 0);
  REQUIRE(own(4, 12, 1000, 8, 8, true, 256) == 1 && own(4, 12, 1000, 8, 4, true, 256) == 0);
  REQUIRE(own(1, 25, 9000, 8, 8, false, 256) == 1 && own(4, 22, 3230, 8, 8, false, 256) == 0 && own(10, 25, 600, 8, 16, false, 256) == 0);
  REQUIRE(own(2, 8, 1500, 8, 4, true, 256) == 1 && own(1, 25, 2500, 8, 4, true, 256) == 0 && own(1, 25, 2500, 8, 4, false, 256) == 1);
  REQUIRE(own(10, 25, 600, 8, 17, true, 256) == 1 && own(10, 25, 5000, 8, 20, false, 256) == 1);
  REQUIRE(own(1, 40, 900, 8, 3, true, 256) == 0 && own(1, 5, 700, 2, 3, true, 256) == 1);      // the rounds of the GPU tests
  REQUIRE(own(1, 25, 2500, 8, 1, false, 128) == 0 && own(1, 25, 5000, 8, 1, false, 512) == 1);
  return 0;
}

// Pipelined steps on both sides of their lines; the span a workgroup really walks counts, not the chunk it could.
static int check_pipelined_rule() {
  int cs = 0;
  auto pipe = [](int sessions, int agents, int span, int heads, int group, bool seg = false) {
    Made m;
    m.shape.heads = heads;
    m.shape.seg = seg;
    for (int i = 0; i < sessions; ++i) m.add(span, agents);
    AttendPlan p;
    return attend_plan(m.done(), 1, group * heads, p) ? (int)(p.pipelined && !p.own_rows) : -1;
  };
  REQUIRE(pipe(10, 25, 5000, 8, 5) == 1 && pipe(10, 25, 600, 8, 1) == 1 && pipe(1, 50, 12000, 8, 2) == 1 && pipe(10, 12, 5000, 2, 5) == 1);
  REQUIRE(pipe(1, 25, 5000, 8, 5) == 0 && pipe(1, 50, 2000, 8, 5) == 0 && pipe(1, 40, 5000, 8, 1) == 0);     // too few steps
  REQUIRE(pipe(10, 25, 207, 8, 5) == 0 && pipe(100, 4, 511, 8, 5) == 0 && pipe(100, 4, 512, 8, 5) == 1);       // short spans
  REQUIRE(pipe(10, 6, 2000, 8, 16) == 1 && pipe(10, 6, 2000, 8, 17) == 0 && pipe(10, 25, 5000, 8, 11) == 0);      // 32-row tiles; three row blocks
  REQUIRE(pipe(10, 25, 5000, 8, 5, true) == 0);
  // the rounds of the GPU tests of that form
  REQUIRE(pipe(10, 4, 513, 8, 3) == 1 && pipe(10, 4, 575, 8, 3) == 1 && pipe(10, 4, 577, 8, 3) == 1 && pipe(10, 4, 640, 8, 3) == 1);
  REQUIRE(pipe(2, 12, 5301, 8, 16) == 1);
  return 0;
}

// The master's order with few rows and a pass too short for pipelined steps: what the estimates choose.
static int check_estimates() {
  int cs = 0;
  auto plan = [](int sessions, int agents, int span, int heads, int group, int page_tokens = 16) {
    Made m;
    m.shape.heads = heads;
    m.shape.page_tokens = page_tokens;
    for (int i = 0; i < sessions; ++i) m.add(span, agents);
    AttendPlan p;
    attend_plan(m.done(), 1, group * heads, p);
    return p;
  };
  // the packed launch stays within one workgroup per compute unit where that is near: 200 and 128 of them walk lists
  AttendPlan p = plan(1, 100, 2500, 8, 1);
  REQUIRE(!p.own_rows && p.fused.n_master <= 56);
  p = plan(1, 16, 5000, 8, 1);
  REQUIRE(!p.own_rows && p.fused.n_master <= 128 && p.fused.n_master > 96);
  // large passes: up to 16 rows packed from 2500 tokens on; from 64 steps per compute unit on packed unless much is promised
  REQUIRE(!plan(1, 123, 3289, 8, 16, 32).own_rows && !plan(4, 69, 2550, 8, 16).own_rows && plan(4, 52, 2054, 8, 16, 32).own_rows);
  REQUIRE(!plan(10, 25, 5000, 8, 20).own_rows && plan(10, 25, 5000, 8, 25).own_rows && plan(10, 13, 3466, 8, 20).own_rows);
  // the rounds of the GPU tests, with both page sizes: form and tokens per chunk (sessions, agents, span, heads, rows per agent and KV
  // head)
  auto is = [&](bool own_rows, int sessions, int agents, int span, int heads, int group, int chunk) {
    for (int page_tokens : {16, 32}) {
      const AttendPlan q = plan(sessions, agents, span, heads, group, page_tokens);
      if (q.own_rows != own_rows || q.pipelined || std::min(q.chunk_tokens, (span + 63) / 64 * 64) != chunk) return false;
    }
    return true;
  };
  auto packed = [&](int sessions, int agents, int span, int heads, int group, int chunk) { return is(false, sessions, agents, span, heads, group, chunk); };
  auto rows = [&](int sessions, int agents, int span, int heads, int group, int chunk) { return is(true, sessions, agents, span, heads, group, chunk); };
  REQUIRE(packed(1, 2, 1100, 1, 8, 128) && packed(1, 2, 1100, 1, 18, 128) && packed(10, 2, 900, 2, 16, 192) && packed(1, 25, 900, 1, 32, 192));
  REQUIRE(packed(6, 2, 577, 8, 16, 256) && packed(6, 2, 577, 8, 18, 256) && packed(4, 18, 1100, 8, 2, 384) && packed(20, 2, 389, 8, 1, 448));
  REQUIRE(packed(2, 18, 193, 8, 3, 64) && packed(2, 18, 700, 8, 3, 128) && packed(3, 12, 1500, 8, 18, 512) && packed(2, 18, 600, 8, 3, 128));
  REQUIRE(packed(1, 4, 225, 2, 3, 64) && packed(1, 4, 225, 2, 18, 64));
  REQUIRE(rows(1, 2, 33, 1, 5, 64) && rows(20, 2, 65, 8, 1, 128) && rows(20, 2, 129, 8, 1, 192) && rows(20, 3, 193, 8, 1, 256));
  REQUIRE(rows(20, 3, 450, 8, 1, 256) && rows(20, 3, 2000, 1, 1, 192) && rows(10, 3, 1500, 1, 16, 128) && rows(1, 2, 2000, 8, 20, 128));
  REQUIRE(rows(2, 18, 63, 8, 3, 64) && rows(2, 18, 65, 8, 3, 128));
  return 0;
}

int main() {
  if (check_grids() || check_workspace() || check_small_workspace() || check_segment_rule() || check_pipelined_rule() || check_estimates()) return 1;
  std::printf("attention planner: clean\n");
  return 0;
}
