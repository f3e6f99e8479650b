// Host planner of a round (see tdk_plan.h).  No HIP here.
#include "tdk_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace tdk {

tdk_status plan_check_model(const tdk_model* m, std::string& err) {
  auto refuse = [&](tdk_status st, const char* msg) { err = msg; return st; };
  if (!m) return refuse(TDK_ERR_INVALID_ARG, "model is NULL");
  if (m->num_layers <= 0 || m->num_kv_heads <= 0 || m->head_dim <= 0 || m->page_tokens <= 0)
    return refuse(TDK_ERR_INVALID_ARG, "model: sizes must be positive");
  if (!(m->rope_theta > 0.0) || !std::isfinite(m->rope_theta))
    return refuse(TDK_ERR_INVALID_ARG, "model: rope_theta must be positive and finite");
  if (m->rope_style != TDK_ROPE_HALF && m->rope_style != TDK_ROPE_INTERLEAVED)
    return refuse(TDK_ERR_INVALID_ARG, "model: unknown rope_style");
  if (m->dtype != TDK_BF16) return refuse(TDK_ERR_UNSUPPORTED, "model: only bf16 caches are supported");
  if (m->head_dim != kHeadDim) return refuse(TDK_ERR_UNSUPPORTED, "model: only head_dim 128 is supported");
  if (m->num_kv_heads > 8) return refuse(TDK_ERR_UNSUPPORTED, "model: at most 8 KV heads per device are supported");
  if (m->page_tokens != 16 && m->page_tokens != 32)
    return refuse(TDK_ERR_UNSUPPORTED, "model: page_tokens must be 16 or 32");
  return TDK_OK;
}


tdk_status plan_round(const tdk_model* model, const tdk_session* sessions, int32_t n_sessions,
                      const tdk_agent* agents, int32_t n_agents, RoundPlan& out, std::string& err) {
  auto refuse = [&](tdk_status st, const char* msg) { err = msg; return st; };
  out = RoundPlan();
  tdk_status st = plan_check_model(model, err);
  if (st != TDK_OK) return st;
  if (n_sessions < 0 || n_agents < 0) return refuse(TDK_ERR_INVALID_ARG, "negative session or agent count");
  if ((n_sessions && !sessions) || (n_agents && !agents)) return refuse(TDK_ERR_INVALID_ARG, "sessions / agents is NULL");
  const int T = model->page_tokens;
  out.sess.resize(n_sessions);
  out.agents.resize(n_agents);
  out.tab.resize((size_t)n_agents * 2 * kHalf);
  out.tab_diff.resize((size_t)n_agents * 2 * kHalf);
  out.sessions.resize(n_sessions);
  int64_t row0 = 0;
  for (int32_t s = 0; s < n_sessions; ++s) {
    if (sessions[s].span_tokens < 0) { return refuse(TDK_ERR_INVALID_ARG, "session: negative span_tokens"); }
    if (sessions[s].master_pos0 < 0) { return refuse(TDK_ERR_INVALID_ARG, "session: negative master_pos0"); }
    PlanSession& hs = out.sessions[s];
    hs.span = sessions[s].span_tokens;
    hs.pages = (hs.span + T - 1) / T;
    hs.master_pos0 = sessions[s].master_pos0;
    hs.master_row0 = row0;
    row0 += hs.span;
    out.sess[s] = {hs.master_row0, hs.span, hs.pages, 0, 0};
    out.total_master_pages += hs.pages;
  }
  out.total_master_rows = row0;
  int64_t flag_off = 0, score_off = 0;
  for (int32_t i = 0; i < n_agents; ++i) out.any_segments |= agents[i].n_segments > 0;
  bool seg_moved = false;                  // some segment's stored diff sits at another position
  for (int32_t i = 0; i < n_agents; ++i) {
    const tdk_agent& a = agents[i];
    if (a.session < 0 || a.session >= n_sessions) { return refuse(TDK_ERR_INVALID_ARG, "agent: session index out of range"); }
    if (a.dst_pos0 < 0) { return refuse(TDK_ERR_INVALID_ARG, "agent: negative dst_pos0"); }
    if (a.dst_pos0 >= (int64_t)1 << 31) { return refuse(TDK_ERR_INVALID_ARG, "agent: positions beyond 2^31"); }
    PlanSession& hs = out.sessions[a.session];
    const int64_t S = hs.span;
    if (a.n_segments < 0 || (a.n_segments > 0 && !a.segments)) { return refuse(TDK_ERR_INVALID_ARG, "agent: bad segment list"); }
    // the logical pages the shared span touches: one range for the identity layout, the hull of the
    // segments otherwise
    int64_t pos_lo = a.dst_pos0, pos_hi = a.dst_pos0 + S;   // [lo, hi)
    if (a.n_segments > 0) {
      int64_t next = 0;
      pos_lo = INT64_MAX; pos_hi = 0;
      for (int32_t q = 0; q < a.n_segments; ++q) {
        const tdk_segment& sg = a.segments[q];
        if (sg.diff_pos < 0 || sg.diff_pos >= (int64_t)1 << 31) { return refuse(TDK_ERR_INVALID_ARG, "agent: segment diff_pos out of range"); }
        if (sg.src_tok != next || sg.len <= 0 || sg.dst_pos < 0) { return refuse(TDK_ERR_INVALID_ARG, "agent: segments must be sorted, contiguous in the master and non-empty"); }
        for (int32_t o = 0; o < q; ++o) {
          const tdk_segment& og = a.segments[o];
          if (sg.dst_pos < og.dst_pos + og.len && og.dst_pos < sg.dst_pos + sg.len) { return refuse(TDK_ERR_INVALID_ARG, "agent: segment destinations overlap"); }
        }
        next += sg.len;
        pos_lo = std::min<int64_t>(pos_lo, sg.dst_pos);
        pos_hi = std::max<int64_t>(pos_hi, sg.dst_pos + sg.len);
      }
      if (next != S) { return refuse(TDK_ERR_INVALID_ARG, "agent: segments do not cover the span"); }
    }
    if (pos_hi + T >= (int64_t)1 << 31) { return refuse(TDK_ERR_INVALID_ARG, "agent: positions beyond 2^31"); }
    const int64_t lp_first = S > 0 ? pos_lo / T : a.dst_pos0 / T;
    const int64_t lp_last = S > 0 ? (pos_hi - 1) / T : lp_first - 1;
    if (S > 0) {
      if (!a.block_table) { return refuse(TDK_ERR_INVALID_ARG, "agent: block_table is NULL"); }
      if ((int64_t)a.block_table_len <= lp_last) { return refuse(TDK_ERR_INVALID_ARG, "agent: block_table too short for its span"); }
    }
    AgentDev& ad = out.agents[i];
    ad.pos0 = (int32_t)a.dst_pos0;
    ad.bt_off = (int32_t)out.bt.size();
    ad.lp_first = (int32_t)lp_first;
    ad.bt_len = (int32_t)(lp_last - lp_first + 1);
    ad.session = a.session;
    ad.flag_off = (int32_t)flag_off;
    ad.score_off = (int32_t)score_off;
    if (a.n_segments == 0 && a.diff_pos0 < 0) { return refuse(TDK_ERR_INVALID_ARG, "agent: negative diff_pos0"); }
    ad.diff_rot = a.n_segments ? 0 : a.diff_pos0 != a.dst_pos0;
    for (int32_t q = 0; q < a.n_segments; ++q) ad.diff_rot |= a.segments[q].diff_pos != a.segments[q].dst_pos;
    if (ad.diff_rot) out.diff_moved = true;
    bool together = ad.diff_rot != 0;
    for (int32_t q = 1; q < a.n_segments; ++q)
      together &= a.segments[q].dst_pos - a.segments[q].diff_pos == a.segments[0].dst_pos - a.segments[0].diff_pos;
    if (together) ad.diff_rot |= 2;
    else if (ad.diff_rot) out.seg_apart = true;
    score_off += S;
    {
      // only pages that hold shared tokens count (the hull of a permuted layout may contain others)
      auto touch = [&](int64_t lo, int64_t hi) -> bool {
        for (int64_t lp = lo / T; lp <= (hi - 1) / T; ++lp) {
          if (a.block_table[lp] < 0) return false;
          out.max_phys_page = std::max<int64_t>(out.max_phys_page, a.block_table[lp]);
        }
        return true;
      };
      bool ok = true;
      if (S > 0 && a.n_segments == 0) ok = touch(pos_lo, pos_hi);
      for (int32_t q = 0; q < a.n_segments && ok; ++q) ok = touch(a.segments[q].dst_pos, a.segments[q].dst_pos + a.segments[q].len);
      if (!ok) { return refuse(TDK_ERR_INVALID_ARG, "agent: negative page number in block_table"); }
    }
    for (int64_t lp = lp_first; lp <= lp_last; ++lp) out.bt.push_back(a.block_table[lp]);
    // layout tables (only if some agent of the round has segments)
    if (out.any_segments) {
      tdk_segment whole{0, (int32_t)S, a.dst_pos0, a.diff_pos0};
      const tdk_segment* segs = a.n_segments ? a.segments : &whole;
      const int32_t nseg = a.n_segments ? a.n_segments : (S > 0 ? 1 : 0);
      const int32_t tab0 = (int32_t)(out.segtab.size() / (2 * kHalf));
      out.seg_off.push_back(tab0);
      for (int32_t q = 0; q < nseg; ++q) {
        out.seg_src.push_back(segs[q].src_tok);
        seg_moved |= segs[q].dst_pos != segs[q].diff_pos;
        const double delta = (double)(segs[q].dst_pos - (hs.master_pos0 + segs[q].src_tok));
        for (int j = 0; j < kHalf; ++j) {
          const double inv_freq = std::pow(model->rope_theta, -(double)(2 * j) / (double)model->head_dim);
          out.segtab.push_back((float)std::cos(delta * inv_freq));
        }
        for (int j = 0; j < kHalf; ++j) {
          const double inv_freq = std::pow(model->rope_theta, -(double)(2 * j) / (double)model->head_dim);
          out.segtab.push_back((float)std::sin(delta * inv_freq));
        }
        const double moved = (double)(segs[q].dst_pos - segs[q].diff_pos);
        for (int j = 0; j < kHalf; ++j) {
          const double inv_freq = std::pow(model->rope_theta, -(double)(2 * j) / (double)model->head_dim);
          out.segtab_diff.push_back((float)std::cos(moved * inv_freq));
        }
        for (int j = 0; j < kHalf; ++j) {
          const double inv_freq = std::pow(model->rope_theta, -(double)(2 * j) / (double)model->head_dim);
          out.segtab_diff.push_back((float)std::sin(moved * inv_freq));
        }
        for (int32_t m = segs[q].src_tok; m < segs[q].src_tok + segs[q].len; ++m) {
          const int64_t pos = segs[q].dst_pos + (m - segs[q].src_tok);
          out.rowmap.push_back((int32_t)((int64_t)a.block_table[pos / T] * T + pos % T));
        }
      }
      int32_t q = 0;
      for (int32_t p = 0; p < hs.pages; ++p) {
        const int32_t m_lo = p * T, m_hi = (int32_t)std::min<int64_t>(S, (int64_t)(p + 1) * T);
        while (segs[q].src_tok + segs[q].len <= m_lo) ++q;
        PageTab e{tab0 + q, tab0 + q, 0, 0};
        int32_t q2 = q;
        for (int32_t m = m_lo; m < m_hi; ++m) {
          while (segs[q2].src_tok + segs[q2].len <= m) ++q2;
          if (q2 > q + 1) { return refuse(TDK_ERR_UNSUPPORTED, "agent: a master page meets more than two segments"); }
          if (q2 == q + 1) { e.y = tab0 + q2; e.z |= 1 << (m - m_lo); }
        }
        // which of the two runs sat elsewhere when the stored diff was encoded
        e.w = (segs[e.x - tab0].dst_pos != segs[e.x - tab0].diff_pos ? 1 : 0) |
              (segs[e.y - tab0].dst_pos != segs[e.y - tab0].diff_pos ? 2 : 0);
        out.pagetab.push_back(e);
      }
    }
    flag_off += hs.pages;
    if (flag_off >= (int64_t)1 << 31 || score_off >= (int64_t)1 << 31 || out.bt.size() >= (size_t)1 << 31) { return refuse(TDK_ERR_UNSUPPORTED, "round too large"); }
    hs.agents.push_back(i);

    // rotation tables of this agent: master frame -> its offset, and the frame its stored diff values
    // were encoded in -> its offset.  Angles in double, one rounding to fp32.
    const double deltas[2] = {(double)(a.dst_pos0 - hs.master_pos0), (double)(a.dst_pos0 - a.diff_pos0)};
    float* tabs[2] = {out.tab.data() + (size_t)i * 2 * kHalf, out.tab_diff.data() + (size_t)i * 2 * kHalf};
    for (int which = 0; which < 2; ++which) {
      float* c = tabs[which];
      float* sn = c + kHalf;
      for (int j = 0; j < kHalf; ++j) {
        const double inv_freq = std::pow(model->rope_theta, -(double)(2 * j) / (double)model->head_dim);
        const double phi = deltas[which] * inv_freq;
        c[j] = (float)std::cos(phi);
        sn[j] = (float)std::sin(phi);
      }
    }
  }
  out.total_pages = flag_off;
  if (out.any_segments) out.seg_off.push_back((int32_t)out.seg_src.size());
  out.seg_moved = seg_moved;
  for (int32_t i = 0; out.any_segments && i < n_agents; ++i) out.max_segments = std::max(out.max_segments, out.seg_off[i + 1] - out.seg_off[i]);
  if (out.any_segments && (out.max_phys_page + 1) * T >= (int64_t)1 << 31)
    return refuse(TDK_ERR_UNSUPPORTED, "segmented layouts address pool rows with 32 bits: page numbers too large");
  out.order.reserve(n_agents);
  for (size_t q = 0; q < out.sessions.size(); ++q) {
    const auto& hs = out.sessions[q];
    out.sess[q].order_begin = (int32_t)out.order.size();
    out.sess[q].n_agents = (int32_t)hs.agents.size();
    out.order.insert(out.order.end(), hs.agents.begin(), hs.agents.end());
  }
  out.total_tokens = score_off;

  // worst case for the work list: every agent its own group
  size_t work_cap = 0;
  for (const auto& hs : out.sessions) work_cap += (size_t)hs.pages * hs.agents.size();
  out.work_capacity = work_cap;

  return TDK_OK;
}

// Work list: one item per (master page, agent group).  Items that share a master page are given
// workgroup ids that are congruent modulo 8, so that (with round-robin dispatch of workgroups to
// the 8 XCDs) they run on the same XCD and the re-read of the master page hits that XCD's L2.
// taper: the pages at the end of the list are cut into smaller groups (a third of the group size over
// the last tenth of the work, single agents over the last fiftieth), so that the launch does not end
// with a few long items running on an otherwise idle chip.
void plan_work(const std::vector<PlanSession>& sessions, int group, bool taper, std::vector<WorkItem>& work) {
  work.clear();
  std::vector<int32_t> order_begin(sessions.size(), 0);
  int32_t cursor = 0;
  int64_t total = 0, done = 0;
  for (size_t s = 0; s < sessions.size(); ++s) {
    order_begin[s] = cursor;
    cursor += (int32_t)sessions[s].agents.size();
    total += (int64_t)sessions[s].pages * (int64_t)sessions[s].agents.size();
  }
  for (size_t s = 0; s < sessions.size(); ++s) {
    const int n = (int)sessions[s].agents.size();
    if (!n) continue;
    const int32_t pages = sessions[s].pages;
    for (int32_t q0 = 0; q0 < pages; q0 += 8) {
      const int32_t qn = std::min<int32_t>(8, pages - q0);
      // every block of 8 pages has one group count
      int g_eff = group;
      if (taper && total > 0) {
        if (done * 50 >= total * 49) g_eff = 1;
        else if (done * 10 >= total * 9) g_eff = std::max(1, (group + 2) / 3);
      }
      const int G = (n + g_eff - 1) / g_eff;
      for (int g = 0; g < G; ++g) {
        // balanced split: the first (n % G) groups get one agent more
        const int base = n / G, extra = n % G;
        const int begin = g * base + std::min(g, extra);
        const int cnt = base + (g < extra ? 1 : 0);
        for (int32_t q = 0; q < qn; ++q)
          work.push_back({(int32_t)s, q0 + q, order_begin[s] + begin, cnt});
      }
      done += (int64_t)qn * n;
    }
  }
}

void plan_items(const std::vector<PlanSession>& sessions, const std::vector<int32_t>& order, const std::vector<AgentDev>& agents, int page_tokens,
                const std::vector<WorkItem>& work, std::vector<ItemDev>& items) {
  items.reserve(items.size() + work.size());
  std::vector<int32_t> ascend(order.size());       // agents from this place of the order on whose ids ascend by one
  for (size_t k = order.size(); k-- > 0;) ascend[k] = k + 1 < order.size() && order[k + 1] == order[k] + 1 ? ascend[k + 1] + 1 : 1;
  for (const WorkItem& w : work) {
    const PlanSession& s = sessions[(size_t)w.session];
    const int32_t first = order[(size_t)w.ag_begin], m0 = w.page * page_tokens;
    const bool consecutive = ascend[(size_t)w.ag_begin] >= w.ag_count;
    ItemDev it{};
    it.row0 = s.master_row0 + m0;
    it.page = w.page;
    it.counts = w.ag_count | std::min(page_tokens, s.span - m0) << 8;
    it.agent0 = consecutive ? first : -1;
    it.order0 = w.ag_begin;
    it.flat0 = agents[(size_t)first].flag_off + w.page;
    it.pages = s.pages;
    it.score0 = agents[(size_t)first].score_off + m0;
    it.span = s.span;
    items.push_back(it);
  }
}

int plan_auto_group(const std::vector<PlanSession>& sessions, bool read_kernels, int64_t page_bytes, int n_cus, int planes) {
  // Measured on MI355X: about 9 agents per work item is the best trade between re-reads of the
  // master page (one per work item, served by the XCD's L2) and the number of work items; rounds
  // too small to give ~2800 items that way are split further (a launch of one workgroup per item then runs
  // three to four rounds of the chip's workgroup slots instead of one and a bit: the 25-agent session
  // steps in 15.31 ms with 3 agents per item, 2817 items, against 15.48 ms with 9 agents, 939 items).
  // The kernels that only read have their own list: every item re-reads its master page, which costs them more
  // than the coarser end of their launch (the same session: compare kernel 87 us with 9 agents per item, 91 with 3),
  // so they stop splitting at ~900 items.
  //
  // An item must also be worth its start: about 8 us of dependent reads when these figures were taken (about half of that since one record holds
  // what they depended on), during which the compute unit's other two
  // workgroups have to keep its share of the memory busy (about 64 KB in 3 us each).  So an item that writes takes at
  // least 1.3 x 64 KB of pages, and with fewer than 3 agents the re-reads of the master page weigh as much as the
  // pages.  25 agents x 5000 tokens, collect: 1 KV head (8 KB pages) 23 us with 3 agents per item, 18 with 9; 2 heads,
  // restore 41 us with 3, 31 with 7; 8 heads 112 us with 1, 100 with 3.  48 agents with 32-token pages and their own block
  // orders, restore: 130 us with 1, 110 with 2, 105 with 3.  Writing one plane, an item holds half the bytes and has a list of
  // its own (37 agents x 2999 tokens, 4 heads, both planes stored and restored: 140 us with 3 agents per item, 130 with 6).
  // Reading items are worth 3 agents at most, whatever their pages: the rows of several agents are in flight there anyway
  // (2 heads, 1840 (agent, page) pairs, store of one plane: 12.2 us with 2, 12.4 with 3, 13.5 with 6; 1 head, 3150 pairs, check
  // layer 16.2 with 3, 18.3 with 11; 8 heads, 1260 pairs, store 33.2 with 1, 26.3 with 3).
  //
  // A round too small to fill the chip with such items is cut finer: nothing is saturated there, and an item's pages are
  // written one after another.  The line is one pair per compute unit and agent of an item; for pages above 64 KB as much
  // more as the pages are larger for the kernels that write, for smaller pages half as much again for those that read.
  // 8 heads, 32-token pages, collect of 532 pairs: 14.7 us with 1 agent per item, 17.3 with 2; restore of 1140 pairs: 39.9 with
  // 1, 38.3 with 2, 42.2 with 3; store of 532 pairs 54.0 with 1, 50.0 with 2; check layer of 1180 pairs 33.2 with 1, 29.5 with 3.
  // 16-token pages, restore of 1148 pairs: 20.9 with 1, 18.1 with 3; 1 head, 900 pairs: 8.9 with 1, 6.3 with 3; store of one
  // plane, 702 pairs: 15.2 with 1, 16.0 with 2; four agents x 256 tokens, collect + restore + store: 28.4 with 1, 30.6 with 2.
  const int64_t target = read_kernels ? 900 : 2800;
  int64_t pairs = 0;
  for (const auto& s : sessions) pairs += (int64_t)s.pages * (int64_t)s.agents.size();
  const int64_t item_bytes = std::max<int64_t>(planes == 2 ? page_bytes : page_bytes / 2, 1);
  const int64_t worth = read_kernels ? 3 : std::max<int64_t>(3, (85 * 1024 + item_bytes - 1) / item_bytes);
  const int64_t cus = std::max(n_cus, 1), kLarge = 64 * 1024;
  const int64_t per_agent = read_kernels ? (page_bytes > kLarge ? cus : cus * 3 / 2) : cus * std::max<int64_t>(1, page_bytes / kLarge);
  const int floor = (int)std::min<int64_t>(kMaxGroup, std::max<int64_t>(1, std::min(worth, pairs / per_agent)));
  int best = std::max(9, floor);
  for (int g = best; g >= floor; --g) {
    int64_t items = 0;
    for (const auto& s : sessions) {
      const int n = (int)s.agents.size();
      if (n) items += (int64_t)s.pages * ((n + g - 1) / g);
    }
    best = g;
    if (items >= target) break;
  }
  return best;
}

int plan_copy_workgroups(int slots, int batches, int n_cus, int left) {
  // Slots of two batches have little to gain: where one workgroup per slot fits beside the others, the further ones must fit too, or
  // some wait until the first leave (restores with a fifth listed, 60 agents x 300 tokens, 16 x 1000 and 8 x 1000: 19.7, 18.6 and 12.0
  // us with one per slot, 21.1, 19.5 and 12.7 beyond the chip).  Where even one per slot does not fit, more are no loss (100 x 200, 23.8
  // -> 23.3, 25 x 1000 28.3 -> 27.5), nor with four batches (16 x 1000, pages of 32 tokens: 24.3 with one per slot, 23.6 within the
  // chip, 21.0 beyond it).
  const int64_t most = batches <= 2 && slots <= left ? left : 4 * (int64_t)std::max(n_cus, 1);
  return (int)std::max<int64_t>(slots, std::min<int64_t>((int64_t)slots * std::max(1, batches), most));
}

bool plan_loops(int64_t items, int64_t pairs, int n_cus, int rows, bool pack, int planes, bool seg) {
  // At least four items and 32 pairs (a round cut into many small items, such as one agent per item, is no longer than its pairs) for every
  // workgroup that fits the chip.  Numbers, for K, V and both, of what fitted when the line was measured: asked for at run time it
  // moves with every few registers that a kernel takes, and on the wrong side of it the looping form is slower (120 agents x 5000 tokens, 4 heads,
  // 32-token pages, collect 239.7 us looping and 228.5 with a workgroup per item, restore 260.1 and 244.0).
  constexpr int fit[3][4] = {{8, 5, 4, 2}, {8, 8, 6, 4}, {6, 4, 3, 2}};       // 1, 2, 4, 8 rows
  int n = fit[planes - 1][rows >= 8 ? 3 : rows >= 4 ? 2 : rows - 1];
  if (planes == 2 && rows == 4 && !pack) n = 7;
  if (seg) n = planes == 3 && rows == 4 && pack ? 2 : std::min(n, 4);          // (their tables: four workgroups' LDS fits)
  const int64_t resident = n * (int64_t)std::max(n_cus, 1);
  return items >= 4 * resident && pairs >= 32 * resident;
}

void plan_queues(const std::vector<WorkItem>& work, std::vector<WorkItem>& queued, int32_t (&q_begin)[9]) {
  queued.clear();
  queued.reserve(work.size());
  for (int x = 0; x < 8; ++x) {
    q_begin[x] = (int32_t)queued.size();
    for (size_t i = x; i < work.size(); i += 8) queued.push_back(work[i]);
  }
  q_begin[8] = (int32_t)queued.size();
}

namespace {

int attend_piece_tokens(int64_t lists, int n_cus) {
  // lists = agents x KV heads.  A piece is 512 tokens, unless the round is so small (at most one list per compute
  // unit) that its few wavefronts would each walk ten or more tiles one after another while most
  // of the chip idles: then 128.  (Shorter pieces in larger rounds cost more in start-up than they gain: the
  // 100-agent long round 138 -> 162 us with pieces of 256 tokens.)
  return lists > n_cus ? 512 : 128;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Own block orders, at most 32 rows per agent and KV head: a wavefront per agent, or packed rows?  The packed form needs a
// copy of every row per segment and reloads a tile's queries lane by lane; the wavefronts of one agent walk the span with
// 32-row tiles that are mostly empty, and their lists with them.  From 17 rows on the packed tiles are no emptier (25 agents x
// 5000 tokens, 20 rows 107 against 69 us; 100 agents x 1500 tokens 112 against 97; ten sessions of 25 x 600 tokens 138
// against 88).  With fewer rows the packed form wins once there are enough agents to fill the chip; what decides is the
// work per compute unit (64-token steps over all agents and KV heads) and how many workgroups of four agents share a
// chunk.  Measured over 21 rounds (1 to 10 sessions of 3 to 100 agents, 600 to 9000 tokens, 2 and 8 KV heads, blocks of 64 and
// 200 tokens, 2 to 20 % of the pages listed, diffs that moved together or not), time packed / time per agent:
//   1 row:       up to 32 steps and 3/8 of a workgroup per compute unit 1.0 .. 3.3; 61 steps 0.96, 73 steps and 25/32 0.60
//   2 to 7 rows: up to 60 steps and 3/8                               1.01 .. 3.3; 69 steps 0.94, 110 steps 0.92
//   8 and more:  up to 110 steps and 5/8                              0.99 .. 3.2; 138 steps and 3/4 0.74
// Short spans of many agents leave the packed form as little to do: up to 24 steps (1 row: 12) one workgroup per compute unit is
// still better off with a wavefront per agent (20 sessions of 4 x 300 tokens 1.21 .. 1.81, 100 agents x 300 tokens 1.36 .. 2.16; ten
// sessions of 25 x 200 tokens, 24 steps and 35/16, 0.76).
// Where segments of one agent have moved by different distances since the diff was stored, the lists turn rows per segment:
// up to 28 steps and 1/8 of a workgroup 1.04 .. 2.5, up to 8 steps and 3/8 1.10 .. 1.45; 30 steps and 7/32 0.73, 16 steps and
// 9/16 0.88 (1 row, a fifth of the pages listed).  With 8 rows or more up to 24 steps and 1/2: 0.97 .. 1.7; 18 steps and
// 35/64 0.88.
bool attend_rows_for_segments(const AttendShape& r, int64_t agent_rows) {
  if (agent_rows > 16) return true;
  int64_t wgs = 0;
  for (const auto& hs : *r.sessions) wgs += ((int64_t)hs.agents.size() + kWaves - 1) / kWaves;
  wgs *= r.heads;
  const int64_t steps = r.total_tokens / 64 * r.heads, cus = r.n_cus;
  auto within = [&](int64_t most_steps, int64_t eighths) { return steps <= most_steps * cus && 8 * wgs <= eighths * cus; };
  if (r.seg_apart) return within(28, 1) || within(8, 3) || (agent_rows >= 8 && within(24, 4));
  if (agent_rows == 1) return within(32, 3) || within(12, 8);
  return within(24, 8) || (agent_rows < 8 ? within(60, 3) : within(110, 5));
}

// What a call takes, in microseconds, where nothing is simple: the master's order, at most 32 rows per agent and KV head, and a pass
// too small for pipelined steps.  Both estimates are robust least squares fits (on the logarithm) to 9 000 timed launches of 318
// rounds: 1 to 20 sessions, 2 to 260 agents, 64 to 26 000 tokens, 1 to 8 KV heads, 1 to 32 rows, 2 to 20 % of the pages listed, diffs
// moved or not, both page sizes, both forms, up to 14 chunk sizes; three sets of inputs in turn, so that the caches hold
// what they hold in a program.  They are within 11 and 9 % of the measured times.  (With one set of inputs over and over, 2 to 5 %
// listed pages and short pieces look better than they are: fitted to that, ten sessions of 25 x 5000 tokens lost 6 %.)
// What they miss is a step: up to one workgroup per compute unit the packed launch runs alone there, beyond it some share one (100
// agents x 2500 tokens, 1 row: 56 and 200 workgroups 31 us, 64 and 200 36; 16 x 5000: 128 and 128 22.8, 160 and 128 28.7).  So
// launches beyond it count a tenth more, and the cut that needs no estimate (packed rows, chunks of 512 tokens or more) stays unless
// another promises 3 %.
// Measured over 820 rounds that the fit has not seen, 2 to 20 % listed, every form and cut: 1.28 times as fast as that cut, 1.033
// times the best choice.  16 of them are more than 5 % slower than it, 2 more than 10 % (25, 5 and one of 1.40 with the estimates
// alone): 20 sessions x 2 agents x 420 tokens, 2 rows 22 -> 28 us, 22 agents x 13329 tokens, 2 heads, 5 rows 29 -> 32.  4 x 23 agents x
// 152 tokens with 32 rows take 18 us instead of 41.  71 rounds of 20 to 150 steps per compute unit: 1.34 times as fast, none slower.
// No page, half or all of them listed (the assumed share is far off there), 120 rounds: 1.25 times as fast, 3 more than 10 % slower (2 x
// 43 agents x 557 tokens, 5 rows, half listed 37 -> 49 us; of another 90 rounds 37 agents x 1080 tokens, 8 rows, all listed 55 -> 79).
struct AttendLoad {
  double wgs;        // workgroups of the pass over the master, per compute unit
  double steps;      // 64-token steps of a workgroup
  double parts;      // partial results per row, on average
  double rows;       // query rows, in thousands
  double listed;     // workgroups of the packed form that walk listed pages, per compute unit
};
constexpr double kListedShare = 0.08;       // share of the pages taken to be listed (the lists are on the device)

// pieces of a list, with that share of the pages listed
double pieces_of(int64_t max_span, int piece) { return std::max(1.0, std::ceil(kListedShare * (double)max_span / piece)); }

// microseconds at 6 TB/s for the payload of the listed pages
double listed_us(const AttendShape& r) { return kListedShare * (double)r.total_tokens * r.heads * (4 * kHeadDim) / 6e6; }

// rounds of workgroups, two to a compute unit: a round of at most one per unit counts 1, a fuller one `two`
double rounds_of(double wgs, double two) {
  const double full = std::floor(wgs / 2 + 1e-9), rest = wgs - 2 * full;
  return full * two + (rest < 1e-9 ? 0.0 : rest > 1 ? two : 1.0);
}

// Packed rows and listed pages in one launch, and the merge.  Both kinds of workgroup run at the same time.  At most four
// wavefronts share a list.
double packed_us(const AttendShape& r, AttendLoad l, int64_t max_span, int piece) {
  const double tokens = kListedShare * (double)max_span, pieces = pieces_of(max_span, piece);
  const double tiles = std::ceil(pieces / std::min(4.0, std::ceil((double)max_span / piece))) * std::min((double)piece, std::max(32.0, tokens)) / 32;
  double walk = (0.805 + 1.505 * l.steps) * (0.572 * std::max(1.0, 1.83 * l.wgs) + 0.428 * rounds_of(l.wgs, 0.98));
  double list = 1.37 * tiles + 0.865 * listed_us(r);
  if (l.wgs + l.listed > 1) { walk *= 1.1; list *= 1.1; }
  l.parts += pieces;
  return 8.35 + std::sqrt(walk * walk + list * list) + 0.099 * l.parts + 0.39 * l.rows * l.parts;
}

// A wavefront per agent, and the merge where the span is cut.  A workgroup walks its part of the lists after its steps.
double rows_us(const AttendShape& r, const AttendLoad& l) {
  const double tiles = 2 * kListedShare * l.steps;
  return (9.03 + 1.40 * l.steps + 1.47 * tiles) * (0.638 * std::max(1.0, 0.823 + 0.306 * l.wgs) + 0.362 * rounds_of(l.wgs, 1.16)) +
         0.76 * listed_us(r) + (l.parts > 1 ? 2.6 + 0.175 * l.parts + 0.22 * l.rows * l.parts : 0.0);
}

// Calls f(chunk) for the chunk sizes worth trying, longest first: the span in 1, 2, .. 16 and then ever more equal parts, in
// multiples of 64 tokens up to `most`.
template <class F>
void for_chunks(int64_t max_span, int64_t most, F f) {
  int64_t last = 0;
  for (int64_t k = 1;; k += 1 + k / 16 * 2) {
    const int64_t c = std::max<int64_t>(64, ((max_span + k - 1) / k + 63) / 64 * 64);
    if (c != last && c <= most) f(last = c);
    if (c == 64) break;
  }
}

// bytes of the workspace with the partial results of rows x n_parts
size_t with_parts(size_t off, int64_t rows, int64_t n_parts) {
  const size_t n = (size_t)rows * n_parts;
  return std::max<size_t>(align_up(off + n * kHeadDim * sizeof(float), 256) + 2 * align_up(n * sizeof(float), 256), 256);
}

// the partial results of p.rows x p.n_parts, from byte `off` of the workspace on
void place_parts(AttendPlan& p, size_t off) {
  const size_t n = (size_t)p.rows * p.n_parts;
  p.o_part_o = off;
  p.o_part_m = align_up(off + n * kHeadDim * sizeof(float), 256);
  p.o_part_l = p.o_part_m + align_up(n * sizeof(float), 256);
  p.bytes = with_parts(off, p.rows, p.n_parts);
}

int32_t chunks_of_all(const AttendShape& r, const AttendPlan& p) {
  int64_t least = p.n_chunks;
  for (const auto& hs : *r.sessions)
    if (!hs.agents.empty() && hs.span > 0) least = std::min(least, ((int64_t)hs.span + p.chunk_tokens - 1) / p.chunk_tokens);
  return (int32_t)least;
}

}  // namespace

bool attend_plan(const AttendShape& r, int32_t n_q, int32_t n_q_heads, AttendPlan& p, size_t workspace) {
  if (n_q < 1 || n_q_heads < 1 || n_q_heads % r.heads) return false;
  const int32_t G = n_q_heads / r.heads;
  int64_t max_span = 0, max_agents = 0, max_pages = 0;
  for (const auto& hs : *r.sessions) {
    if (hs.agents.empty()) continue;
    max_pages = std::max<int64_t>(max_pages, hs.pages);
    max_span = std::max<int64_t>(max_span, hs.span);
    max_agents = std::max<int64_t>(max_agents, (int64_t)hs.agents.size());
  }
  const int64_t max_rows = max_agents * n_q * G;
  if (max_rows >= (int64_t)1 << 30) return false;
  p.max_rows = (int32_t)max_rows;
  p.rows = (int64_t)r.n_agents * n_q * n_q_heads;
  const int64_t n_sessions = (int64_t)r.sessions->size();
  auto times = [](int64_t a, int64_t b) { return a > 0 && b > INT64_MAX / a ? INT64_MAX : a * b; };
  p.max_agents = (int32_t)max_agents;
  const int64_t agent_rows = (int64_t)n_q * G;
  // Which kernels: one agent per wavefront, or the rows of a session's agents packed into one block.
  //   Packed rows waste no place in the 32-row tiles, but their listed pages need a pass and partial results of their
  //   own.  From 33 rows on the tiles of one agent are full and packing has nothing to save (40 rows: 94 against 70 us, ten
  //   sessions 575 against 460 us; 320 rows: 462 against 206 us).  Below, in the master's order, the pipelined steps decide
  //   (10 rows, ten sessions: packed) or the estimates above.
  const int64_t lists = (int64_t)r.n_agents * r.heads;
  const int64_t row_blocks = std::max<int64_t>(1, (max_rows + 127) / 128), per_agent = (agent_rows + 31) / 32, cus = r.n_cus;
  const int32_t max_chunk = std::min<int32_t>(128 * r.page_tokens, 4096);
  p.own_rows = agent_rows > 32 || r.total_master_rows == 0 || lists >= ((int64_t)1 << 27) ||
               (r.seg && attend_rows_for_segments(r, agent_rows));
  // the packed form's listed-pages pass: one wavefront takes a piece of an agent's list and every piece has its own partial result
  p.piece_tokens = attend_piece_tokens(lists, r.n_cus);
  p.n_pieces = (int32_t)std::max<int64_t>(1, (max_pages * r.page_tokens + p.piece_tokens - 1) / p.piece_tokens);
  // enough steps for the pipelined form? (see below)
  int64_t steps = 0;
  for (const auto& hs : *r.sessions)
    if (!hs.agents.empty()) steps += ((int64_t)hs.span + 63) / 64;
  steps *= r.heads * row_blocks;
  const bool long_pass = !r.seg && agent_rows <= 16 && row_blocks <= 2 && max_span >= 512 && 4 * steps >= 11 * cus;
  // Tokens per workgroup of the master pass where it fills the chip.  A workgroup walks its chunk in steps of 64 tokens; two
  // workgroups fit a compute unit at a time, so the pass takes about ceil(workgroups / slots) rounds of
  // (steps per chunk + a fixed start-up cost of about two steps).  Of the chunk sizes that the 128-bit page
  // mask per query row can cover, the one with the lowest such cost wins; ties go to the larger chunk
  // (fewer partial results to merge).  Chunks shorter than 512 tokens are not tried here (unless the span is): a workgroup's
  // start-up (page masks, query rotation, first rows) costs about as much as three steps, and every chunk adds a partial
  // result per row for the merge.
  auto fewest_rounds = [&]() {
    const int64_t slots = 2 * cus;
    const int32_t min_chunk = std::max((int32_t)std::min<int64_t>(512, (max_span + 63) / 64 * 64), 64);
    int32_t chunk = min_chunk;
    int64_t best = -1;
    for (int32_t c = max_chunk; c >= min_chunk; c -= 64) {
      int64_t wgs = 0;
      for (const auto& hs : *r.sessions)
        if (!hs.agents.empty()) wgs += ((int64_t)hs.span + c - 1) / c;
      wgs *= r.heads * row_blocks;
      if (wgs == 0) break;
      const int64_t cost = ((wgs + slots - 1) / slots) * (std::min<int64_t>(c, max_span + 63) / 64 + 2);
      if (best < 0 || cost < best) { best = cost; chunk = c; }
    }
    return chunk;
  };
  int32_t chosen = 0;              // the chunk that the estimates chose
  if (!p.own_rows && !r.seg && !long_pass) {
    int64_t with_agents = 0;
    for (const auto& hs : *r.sessions) with_agents += !hs.agents.empty();
    double packed = -1, rows = -1;
    bool first = true, refused = false;
    int64_t packed_chunk = 64, rows_chunk = 64;
    // From three steps per compute unit on the packed form has nothing to gain from other chunks (1.01 times as fast on 62 such
    // rounds, 101 -> 122 us on one), the wavefront per agent 1.3 times.
    const bool only = steps >= 3 * cus;
    // workgroups that walk lists: a piece of four KV heads each, at most four per list
    const double walk_lists = (double)(r.n_agents * (int64_t)((r.heads + kWaves - 1) / kWaves)) *
                              std::min({4.0, (double)p.n_pieces, pieces_of(max_span, p.piece_tokens)}) / (double)cus;
    // The fit has few large passes, and estimates the wavefront per agent too fast there.  With 8 to 16 rows (half of every tile is
    // empty), three steps per compute unit and 2500 tokens or more it won nothing in 17 rounds (time per agent / packed 0.99 .. 1.41,
    // estimated 0.77 .. 1.2), with shorter spans it won 16 of 19 (0.55 .. 0.93): there it counts twice, and is taken where nothing else
    // fits the workspace.  From 64 steps on a promise of less than 15 % does not count (ten sessions of 25 x 5000 tokens, 20 rows 266
    // against 291 us).
    const double doubtful = only && agent_rows <= 16 && max_span >= 2500 ? 2 : 1;
    auto consider = [&](int64_t c, bool in_packed, bool in_rows, double bonus = 1) {
      // chunks of c tokens over all sessions with agents, and the workgroups of the rows kernel in them (both per KV head)
      int64_t chunks = 0, row_wgs = 0, span = -1, n = 0;
      for (const auto& hs : *r.sessions) {
        if (hs.agents.empty()) continue;
        if (hs.span != span) { span = hs.span; n = (span + c - 1) / c; }
        chunks += n;
        row_wgs += n * (((int64_t)hs.agents.size() + kWaves - 1) / kWaves);
      }
      AttendLoad l{(double)(chunks * row_blocks * r.heads) / (double)cus, (double)((std::min(c, max_span) + 63) / 64),
                   (double)chunks / (double)std::max<int64_t>(with_agents, 1), (double)p.rows / 1000, walk_lists};
      // (a packed launch that fits a grid with the first cut tried is not cut so fine that it does not; one that does not is refused,
      // as ever: not to be taken by the other form)
      const int64_t n_chunks = (max_span + c - 1) / c;
      const bool fits = times(times(times(r.heads, row_blocks), n_sessions), n_chunks) < kMaxBlocks - times(lists, 4);
      if (in_packed && first && !fits) refused = true;
      first = first && !in_packed;
      // the partial results have to fit the workspace that the call brings
      in_packed = in_packed && with_parts(0, p.rows, n_chunks + p.n_pieces) <= workspace;
      in_rows = in_rows && with_parts(0, p.rows, n_chunks) <= workspace;
      if (in_packed && (packed < 0 || fits)) {
        const double us = bonus * packed_us(r, l, max_span, p.piece_tokens);
        if (packed < 0 || us < packed) { packed = us; packed_chunk = c; }
      }
      l.wgs = (double)(row_wgs * r.heads) / (double)cus;
      const double us = in_rows ? doubtful * rows_us(r, l) : 0;
      if (in_rows && (rows < 0 || us < rows)) { rows = us; rows_chunk = c; }
    };
    consider(fewest_rounds(), true, false, steps >= 64 * cus ? 0.85 : 0.97);
    for_chunks(max_span, 16384, [&](int64_t c) { consider(c, !only && c <= max_chunk, true); });
    // (neither fits: the cut that needs least, for the caller to compare)
    p.own_rows = !refused && rows > 0 && (packed < 0 || rows < packed);
    if (p.own_rows || packed >= 0) chosen = (int32_t)(p.own_rows ? rows_chunk : packed_chunk);
  }
  if (p.own_rows) {
    // Chunks of the span: workgroups of four wavefronts, two of which share a compute unit (each then takes about
    // 1.6 times as long).  In units of a 64-token step (about 1.2 us): a workgroup starts up in 8, a step with
    // per-agent block orders costs 2 (query reloads at the borders), a second launch to merge costs 6 and the
    // traffic of the partial results.  (More than 32 rows and own block orders; 50 and 192 rounds: 1.02 and 1.05 times the best
    // choice.  16 query tokens, 25 agents: 1, 2, 4, 8 chunks take 104, 74, 68, 79 us without
    // listed pages; per-agent orders, 4 tokens: 1, 4, 8, 12 chunks 252, 87, 70, 85 us.)
    double best = -1;
    if (chosen) p.chunk_tokens = chosen;
    const int k_lo = (int)std::max<int64_t>(1, (max_span + 16383) / 16384);
    for (int k = k_lo; !chosen && k < k_lo + 32; ++k) {
      const int64_t c = std::max<int64_t>(64, ((max_span + k - 1) / k + 63) / 64 * 64);
      if (k > k_lo && c * (k - 1) >= max_span) continue;       // the same chunks as a smaller k
      int64_t wgs = 0;
      for (const auto& hs : *r.sessions)
        if (!hs.agents.empty()) wgs += (((int64_t)hs.span + c - 1) / c) * (((int64_t)hs.agents.size() * per_agent + 3) / 4);
      wgs *= r.heads;
      const double one = (double)(c / 64) * (r.seg ? 2 : 1) + 8;
      const int64_t full = wgs / (2 * cus), rest = wgs % (2 * cus);
      const double cost = one * (1.6 * (double)full + (rest == 0 ? 0.0 : rest > cus ? 1.6 : 1.0)) +
                          (max_span > c ? 6 + (double)p.rows * ((double)max_span / (double)c + 1) * 1024 / 6e6 : 0.0);
      if (best < 0 || cost < best) { best = cost; p.chunk_tokens = (int32_t)c; }
    }
    p.n_chunks = (int32_t)((max_span + p.chunk_tokens - 1) / p.chunk_tokens);
    p.all_chunks = chunks_of_all(r, p);
    p.n_pieces = 0;
    p.piece_tokens = 512;          // (no listed-pages pass: the merge finds no pieces)
    p.n_parts = std::max(p.n_chunks, 1);
    // A launch takes as many sessions as fit a grid: with four wavefronts per workgroup and short chunks it has up to 30
    // times the workgroups of the packed form, and a round that fits that one has to fit this one too.
    p.blocks = times(times(r.heads, (max_agents * per_agent + kWaves - 1) / kWaves), p.n_parts);
    p.launch_sessions = (int32_t)std::min<int64_t>(std::max<int64_t>((kMaxBlocks - 1) / std::max<int64_t>(p.blocks, 1), 1), std::max<int64_t>(n_sessions, 1));
    p.blocks = times(p.blocks, p.launch_sessions);
    place_parts(p, 0);
    return true;
  }
  const int32_t chunk = chosen ? chosen : fewest_rounds();
  p.chunk_tokens = chunk;
  p.n_chunks = (int32_t)((max_span + chunk - 1) / chunk);
  p.all_chunks = chunks_of_all(r, p);
  // Pipelined steps in the master pass (identity layouts; tdk_attend.hip, attend_packed_body).  A workgroup starts up later there
  // (two more tiles and the first scores before the loop), so it needs workgroups of at least 8 steps and at least 2 3/4 steps
  // per compute unit over the whole pass; with three row blocks or more the plain form's calls of coming tiles into L2
  // serve several readers; and 17 rows or more (32-row tiles for the listed pages) lose with many listed pages what
  // they gain with few.  Time plain / pipelined, 1 to 16 rows, 3 and 20 % of the pages listed: ten sessions of 6 x 2000
  // tokens (9.8 steps) 1.04 .. 1.10, four of 12 x 3000 (5.9) 1.04 .. 1.06, ten of 25 x 600 (2.9) 1.00 .. 1.10, 50 agents x 12000 (5.9)
  // 1.01 .. 1.05; one session of 25 x 5000 (2.4) 0.99 .. 1.04, of 50 x 2000 (2.0) 0.99 .. 1.00, two of 36 x 500 (1.0) 0.96 .. 1.02, ten of
  // 25 x 1500 with 2 heads (1.8) 0.95 .. 1.01, two of 25 x 207 (0.2) 0.92 .. 0.99; 20 rows, half of the pages listed, ten sessions of 6 x
  // 2000 tokens 145 against 176 us.
  p.pipelined = long_pass && chunk >= 512;
  p.n_parts = p.n_chunks + p.n_pieces;
  // Most lists are far shorter than a whole session's pages: a few wavefronts per list walk its pieces in turn,
  // instead of one launched wavefront per possible piece (nearly all of which would find nothing).
  p.piece_grid = std::min<int32_t>(p.n_pieces, 4);
  // The launches, in 64 bits: the master pass has every session as wide as the widest one and as long as the longest,
  // so rounds of very many sessions reach the limit of a grid long before their rows do.
  const int64_t master = times(times(times(r.heads, row_blocks), n_sessions), p.n_chunks);
  if (r.seg) {
    p.blocks = std::max(master, times(lists, p.piece_grid));
  } else {
    const int64_t head_groups = (r.heads + kWaves - 1) / kWaves, diff0 = r.n_agents * head_groups;
    p.blocks = master == INT64_MAX ? master : master + diff0 * p.piece_grid;
    if (p.blocks < kMaxBlocks) p.fused = {(int32_t)master, (int32_t)row_blocks, (int32_t)diff0, (int32_t)head_groups};
  }
  size_t off = 0;
  if (r.seg) {                 // copies of every query row per segment
    p.o_qdiff = align_up((size_t)p.rows * r.max_segments * kHeadDim * 2, 256);
    off = p.o_qdiff + align_up((size_t)p.rows * (r.seg_moved ? r.max_segments : 1) * kHeadDim * 2, 256);
  }
  place_parts(p, off);
  return true;
}

// A short call may be cut into more parts than a long one, whose rows fill the chip by themselves, and may need more
// memory; a program that sizes its workspace for its longest call expects it to serve the shorter ones.
size_t attend_workspace_bytes(const AttendShape& r, int32_t n_q, int32_t n_q_heads) {
  AttendPlan p;
  if (!attend_plan(r, n_q, n_q_heads, p)) return 0;
  const int64_t group = n_q_heads / r.heads;
  size_t most = p.bytes;
  for (int64_t n = 1; n < n_q;) {
    AttendPlan one;
    if (!attend_plan(r, (int32_t)n, n_q_heads, one)) return 0;
    // Up to 32 rows per agent and KV head: every length by itself.  Beyond: the lengths with the same number of
    // wavefronts per agent at once, since more rows add only to the cost of further parts and so never get more of them.
    int64_t last = n;
    if (n * group > 32) {
      last = std::min<int64_t>(std::max<int64_t>((n * group + 31) / 32 * 32 / group, n), n_q);
      one.rows = (int64_t)r.n_agents * last * n_q_heads;
      place_parts(one, 0);
    }
    most = std::max(most, one.bytes);
    n = last + 1;
  }
  return most;
}

}  // namespace tdk
