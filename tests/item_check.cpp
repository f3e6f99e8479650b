// Host-only driver for the page kernels' item records (plan_items, csrc/tdk_plan.cpp), built by tests/test_items.py: what a kernel works
// out from a record against the session and agent descriptors it stands for.  Exit code 0 = clean.
#include <cstdio>
#include <vector>

#include "tdk_plan.h"

using namespace tdk;

#define REQUIRE(c) do { if (!(c)) { std::fprintf(stderr, "requirement failed: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

int main() {
  int64_t with_ids = 0, without = 0;
  for (int round = 0; round < 40; ++round) {
    uint32_t x = 77u + (uint32_t)round * 2654435761u;
    auto rnd = [&](int n) { x = x * 1664525u + 1013904223u; return (int)((x >> 8) % (uint32_t)n); };
    const int T = round % 2 ? 16 : 32, n_sessions = 1 + rnd(4), n_agents = rnd(40);
    std::vector<PlanSession> sessions((size_t)n_sessions);
    int64_t row0 = 0;
    for (auto& s : sessions) {
      s.span = rnd(5) ? 1 + rnd(200) : 0;
      s.pages = (s.span + T - 1) / T;
      s.master_row0 = row0;
      row0 += s.span;
    }
    // the caller's order: by session, or mixed
    std::vector<AgentDev> agents;
    int32_t flat = 0, score = 0;
    for (int i = 0; i < n_agents; ++i) {
      const int s = round % 3 == 0 ? i * n_sessions / n_agents : rnd(n_sessions);
      AgentDev ad{};
      ad.session = s; ad.flag_off = flat; ad.score_off = score;
      flat += sessions[(size_t)s].pages;
      score += sessions[(size_t)s].span;
      agents.push_back(ad);
      sessions[(size_t)s].agents.push_back(i);
    }
    std::vector<int32_t> order;
    for (const auto& s : sessions) order.insert(order.end(), s.agents.begin(), s.agents.end());
    std::vector<ItemDev> items;
    for (const int group : {1, 3, 9, 32}) {
      std::vector<WorkItem> work;
      plan_work(sessions, group, round % 5 == 0, work);
      const size_t first = items.size();
      plan_items(sessions, order, agents, T, work, items);
      REQUIRE(items.size() == first + work.size());
      for (size_t k = 0; k < work.size(); ++k) {
        const WorkItem& w = work[k];
        const ItemDev& it = items[first + k];
        const PlanSession& s = sessions[(size_t)w.session];
        REQUIRE((it.counts & 255) == w.ag_count && it.counts >> 8 >= 1 && it.counts >> 8 <= T);
        REQUIRE((it.counts >> 8) == (s.span - w.page * T < T ? s.span - w.page * T : T));
        REQUIRE(it.row0 == s.master_row0 + w.page * T && it.page == w.page && it.order0 == w.ag_begin);
        (it.agent0 >= 0 ? with_ids : without) += w.ag_count > 1;
        for (int g = 0; g < w.ag_count; ++g) {
          const int32_t a = order[(size_t)(w.ag_begin + g)];
          const AgentDev& ad = agents[(size_t)a];
          if (it.agent0 < 0) continue;              // the kernels read the agents' descriptors then
          REQUIRE(it.agent0 + g == a);
          REQUIRE(it.flat0 + g * it.pages == ad.flag_off + w.page);
          REQUIRE(it.score0 + g * it.span == ad.score_off + w.page * T);
        }
        if (w.ag_count == 1) REQUIRE(it.agent0 == order[(size_t)w.ag_begin]);
      }
    }
  }
  REQUIRE(with_ids > 100 && without > 100);
  std::printf("items: clean\n");
  return 0;
}
