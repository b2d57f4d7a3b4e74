// The split-K planner behind baklava_plan_schedule, with the shorter runs that a context's own schedules take.
#ifndef BAKLAVA_PLAN_H
#define BAKLAVA_PLAN_H

#include <cstdint>

#include "baklava.h"

namespace baklava {

int plan_schedule(const int64_t* off_host, const int32_t* cap_host, int32_t L, int32_t caches_per_layer, int32_t chunk,
                  int32_t target_items, int32_t shortest, int32_t fill_items, int32_t whole_model, int64_t max_items,
                  baklava_work_item* items_out, int64_t* n_items_out);

}  // namespace baklava
#endif
