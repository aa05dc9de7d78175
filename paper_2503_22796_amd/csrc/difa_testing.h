// Views of the library's inner decisions for its tests: exported by the library, no part of its interface (include/difa.h).
#pragma once
#include <stdint.h>

#include "difa.h"

#ifdef __cplusplus
extern "C" {
#endif

// ---- host only, no device needed
// The records of a layer as the bf16 kernel gets them: `rows` query rows each, in the scheduler's order (head by head).
// Two calls as for difa_worklist_build: items == NULL, capacity 0 asks for the count.
difa_status_t difa_testing_records(int32_t batch, int32_t heads, const int32_t* head_plan, const int32_t* window, int32_t n_text,
                                   int32_t n_img, int32_t rows, int32_t head_dim, uint32_t flags, difa_work_item_t* items,
                                   int32_t capacity, int32_t* n_items);
// Their schedule as the library makes it (the kernel's own costs, `n_wg` workgroups on n_xcd dies of the given relative
// speeds; NULL: alike).  die_span: n_xcd predicted finishing times.  tried: plans with cuts that were looked at on the way.
difa_status_t difa_testing_schedule(const difa_work_item_t* items, int32_t n_items, int32_t head_dim, int32_t n_wg, int32_t n_xcd,
                                    const double* die_speed, int64_t* die_span, difa_segment_t* segs, int32_t seg_capacity,
                                    int32_t* wg_begin, int32_t* n_segs, difa_merge_item_t* merges, int32_t merge_capacity,
                                    int32_t* n_merges, int32_t* n_slots, int32_t* tried);
// Query rows per record that the library chooses for a bf16 call on a device of n_cu compute units.
int32_t difa_testing_record_rows(int32_t batch, int32_t heads, int32_t head_dim, const int32_t* head_plan, const int32_t* window,
                                 int32_t n_text, int32_t n_img, uint32_t flags, int32_t n_cu);
// n_launches launches of one memoised schedule, each timed by the next call.  die_ticks[v][n_dies]: what the dies take on its
// version v (the last row for all later ones).  capturing[i]: launch i is recorded into a graph (NULL: none is).  version[i]: the
// version launch i runs; speeds[i][n_dies]: what it was made for.
void difa_testing_trial(int32_t n_dies, const int64_t* die_span, int32_t n_versions, const double* die_ticks, int32_t n_launches,
                        const int32_t* capturing, int32_t* version, double* speeds);
// What a plan object sets aside for schedules: device and pinned host memory, and how many stay resident.
void difa_testing_schedule_memory(int32_t batch, int32_t heads, int32_t dtype, int32_t max_tokens, int32_t n_cu,
                                  int64_t* device_bytes, int64_t* pinned_bytes, int32_t* schedules);
// Chunks of the cached-head copy that shares the launch of a layer's computed heads; -1: refused.
int32_t difa_testing_copy_chunks(int64_t n_tokens, int32_t head_dim, int32_t dtype, int32_t batch, int32_t n_copy);
// Which of n resident schedules gives way to a new one: in use or free, launched by a captured graph, time of its last use.
int32_t difa_testing_victim(int32_t n, const int32_t* valid, const int32_t* held, const int64_t* stamp);

// ---- plan objects
// Query rows per record from the next call on: 128, 256 (head_dim 128), or 0 for the library's own choice.  The plan object
// forgets its schedules.
difa_status_t difa_testing_force_rows(difa_plan_t* plan, int32_t rows);
// The plan object's last bf16 attention call: query rows per record, workgroups the schedule is for, workgroups launched,
// pieces of cut records, whether the launch was asked to report run times.
void difa_testing_last_call(const difa_plan_t* plan, int32_t* rows, int32_t* n_wg, int32_t* grid, int32_t* n_pieces,
                            int32_t* reports);

#ifdef __cplusplus
}
#endif
