// Test harness (CPU only): a count plan's direct items, their order and the room
// of their parts' counters.
#include "host_build.h"

using namespace dbbc;

// out: whether the items are ordered heaviest first, parts, items that are no
// parts, and those of them before the last part.
extern "C" int plan_parts(int32_t n_u, int32_t n_v, int64_t m, const int32_t* u, const int32_t* v, const int8_t* sign,
                          int32_t part_work, int64_t* out) {
  HostGraph g;
  std::string err;
  int rc = build_host_graph(n_u, n_v, m, u, v, sign, 0, g, err);
  if (rc) return rc;
  PlanParams p = default_params(g);
  p.hub_T = 0;
  p.part_work = part_work;
  HostPlan plan;
  rc = make_plan(g, p, plan, err);
  if (rc) return rc;
  out[0] = 1;
  out[1] = out[2] = out[3] = 0;
  const Item* last = nullptr;
  for (const Item& it : plan.direct_items) {
    if (last && direct_order_work(it.work, it.seg_count) > direct_order_work(last->work, last->seg_count)) out[0] = 0;
    last = &it;
    if (it.flags & kItemMultiPart) {
      ++out[1];
      out[3] = out[2];
    } else {
      ++out[2];
    }
  }
  return 0;
}

// The plan with part_room bytes for the parts' counters; out: bytes they take,
// parts, the direct items' wedges, reduces.
extern "C" int plan_room(int32_t n_u, int32_t n_v, int64_t m, const int32_t* u, const int32_t* v, const int8_t* sign,
                         int32_t part_work, int64_t part_room, int64_t* out) {
  HostGraph g;
  std::string err;
  int rc = build_host_graph(n_u, n_v, m, u, v, sign, 0, g, err);
  if (rc) return rc;
  PlanParams p = default_params(g);
  p.hub_T = 0;
  p.part_work = part_work;
  p.part_room = part_room;
  HostPlan plan;
  rc = make_plan(g, p, plan, err, true);
  if (rc) return rc;
  out[0] = static_cast<int64_t>(plan.acc_slots) * plan.acc_width * 4;
  out[1] = 0;
  for (const Item& it : plan.direct_items) out[1] += (it.flags & kItemMultiPart) != 0;
  out[2] = plan.k_wedges[0];
  out[3] = static_cast<int64_t>(plan.reduces.size());
  return 0;
}
