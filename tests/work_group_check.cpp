// Host-only driver for the rule that sizes the page kernels' work items (csrc/tdk_plan.cpp), built by
// tests/test_work_groups.py.  Exit code 0 = clean.
#include <cstdio>
#include <vector>

#include "tdk_plan.h"

using namespace tdk;

static std::vector<PlanSession> round_of(int sessions, int agents, int pages) {
  std::vector<PlanSession> v;
  for (int s = 0; s < sessions; ++s) {
    PlanSession p;
    p.pages = pages;
    for (int i = 0; i < agents; ++i) p.agents.push_back(s * agents + i);
    v.push_back(p);
  }
  return v;
}

#define REQUIRE(c) do { if (!(c)) { std::fprintf(stderr, "requirement failed: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

int main() {
  const auto kb = [](int heads, int page_tokens) { return (int64_t)heads * page_tokens * 512; };   // K and V of one page
  // kernels that read: at least three agents per item, whatever the size of their pages
  REQUIRE(plan_auto_group(round_of(2, 25, 63), true, kb(1, 16), 256) == 3);
  REQUIRE(plan_auto_group(round_of(10, 23, 8), true, kb(2, 16), 256) == 3);
  REQUIRE(plan_auto_group(round_of(1, 78, 9), true, kb(8, 16), 256) == 1);        // 702 pairs
  REQUIRE(plan_auto_group(round_of(1, 78, 9), true, kb(8, 32), 256) == 2);        // the same with pages of 128 KB
  // kernels that write, small rounds: one pair per compute unit and agent of an item, two with pages of 128 KB
  REQUIRE(plan_auto_group(round_of(1, 133, 4), false, kb(8, 32), 256) == 1);      // 532
  REQUIRE(plan_auto_group(round_of(10, 19, 6), false, kb(8, 32), 256) == 2);      // 1140
  REQUIRE(plan_auto_group(round_of(10, 19, 6), false, kb(8, 32), 512) == 1);      // the same on a chip twice as wide
  REQUIRE(plan_auto_group(round_of(10, 10, 9), false, kb(1, 16), 256) == 3);      // 900
  // larger ones: what an item is worth, in bytes
  REQUIRE(plan_auto_group(round_of(1, 141, 60), false, kb(1, 16), 256) == 11);
  REQUIRE(plan_auto_group(round_of(1, 25, 313), false, kb(8, 16), 256) == 3);
  REQUIRE(plan_auto_group(round_of(10, 25, 313), false, kb(8, 16), 256) == 9);
  // writing one plane: items of the same worth hold twice the agents
  REQUIRE(plan_auto_group(round_of(1, 37, 188), false, kb(4, 16), 256, 2) == 3);
  REQUIRE(plan_auto_group(round_of(1, 37, 188), false, kb(4, 16), 256, 1) == 6);
  REQUIRE(plan_auto_group(round_of(10, 18, 77), false, kb(8, 16), 256, 1) == 5);
  REQUIRE(plan_auto_group(round_of(4, 11, 154), false, kb(8, 32), 256, 1) == 3);
  REQUIRE(plan_auto_group(round_of(10, 15, 4), false, kb(8, 32), 256, 1) == 1);   // 600
  // listed pages' copies: shared out while places are left
  const int all = 1 << 30;
  REQUIRE(plan_copy_workgroups(10, 4, 256, all) == 40 && plan_copy_workgroups(10, 2, 256, all) == 20 && plan_copy_workgroups(5000, 4, 256, all) == 5000);
  REQUIRE(plan_copy_workgroups(7, 0, 256, all) == 7 && plan_copy_workgroups(0, 4, 256, all) == 0);
  // beside page items, two batches: not beyond the chip where one per slot fits, as far as four per unit where it does not
  REQUIRE(plan_copy_workgroups(308, 2, 256, 312) == 312 && plan_copy_workgroups(138, 2, 256, 164) == 164 && plan_copy_workgroups(28, 2, 256, 164) == 56);
  REQUIRE(plan_copy_workgroups(383, 2, 256, 238) == 766 && plan_copy_workgroups(800, 2, 256, -700) == 1024 && plan_copy_workgroups(1500, 2, 256, -700) == 1500);
  // four batches
  REQUIRE(plan_copy_workgroups(350, 4, 256, 400) == 1024 && plan_copy_workgroups(96, 4, 256, 100) == 384);
  // long launches: four items and 32 pairs per workgroup that fits the chip, by numbers that no build moves
  struct { int rows; bool pack; int planes; bool seg; int64_t fits; } lines[] = {
      {4, false, 3, false, 3}, {8, false, 3, false, 2}, {4, true, 3, false, 3}, {4, true, 3, true, 2}, {2, true, 3, false, 4}, {1, true, 3, false, 6}, {1, true, 3, true, 4},
      {8, false, 3, true, 2}, {4, false, 3, true, 3}, {4, false, 2, false, 7}, {4, true, 2, false, 6}, {8, false, 2, false, 4}, {2, true, 2, false, 8}, {4, false, 2, true, 4},
      {4, true, 1, false, 4}, {8, false, 1, false, 2}, {2, true, 1, false, 5}, {1, true, 1, true, 4}};
  for (const auto& l : lines)
    for (int cus : {64, 256}) {
      const int64_t wg = l.fits * cus;
      REQUIRE(plan_loops(4 * wg, 32 * wg, cus, l.rows, l.pack, l.planes, l.seg));
      REQUIRE(!plan_loops(4 * wg - 1, 32 * wg, cus, l.rows, l.pack, l.planes, l.seg) && !plan_loops(4 * wg, 32 * wg - 1, cus, l.rows, l.pack, l.planes, l.seg));
    }
  std::printf("work groups: clean\n");
  return 0;
}
