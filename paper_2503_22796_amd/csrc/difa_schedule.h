// The scheduler as the library itself calls it (host code only; defined in difa_worklist.cpp).
#pragma once
#include <stdint.h>

#include "difa.h"

namespace difa {

// Cost model of a segment, in eighths of a plain key-tile iteration of the kernel it is for.
struct CostModel {
    int masked;      // extra for an iteration on a tile that needs the element mask
    int whole;       // starting and finishing a whole record
    int piece;       // ... a piece of a cut record, without the fold
    int fold;        // folding one other piece's partial result in (the piece that arrives last pays; who that is is
                     // not known here, so every piece is charged its share)
    int min_piece;   // shortest piece, in key tiles, worth cutting off a record
};
constexpr CostModel kGenericCosts{7, 36, 72, 40, 12};   // what difa_schedule_build prices with

// difa_worklist_build (n_xcd = 1) for a kernel whose records are `rows` query rows, a divisor of the block-granular
// band's block of `band_rows` rows: the key tiles a record visits are then those of the block it lies in.
difa_status_t worklist_for_kernel(int32_t batch, int32_t heads, const int32_t* head_plan, const int32_t* window,
                                  int32_t n_text, int32_t n_img, int32_t rows, int32_t band_rows, int32_t bn,
                                  uint32_t flags, difa_work_item_t* items, int32_t capacity, int32_t* n_items_out,
                                  int32_t* copy_heads, int32_t* n_copy_out);

// difa_schedule_build with three more arguments:
//   m           what a segment costs
//   die_speed   n_xcd relative speeds of the accelerator dies (NULL: all alike).  Under a heavy load the
//               dies of one chip settle at clocks a few percent apart; a die is given work in
//               proportion to its speed.
//   die_span    receives, per die, the predicted finishing time of its slowest workgroup in the
//               scheduler's cost units at speed 1 (NULL: not wanted).  The caller divides it by the die's
//               measured time to learn the speeds.
difa_status_t schedule_for_dies(const CostModel& m, const difa_work_item_t* items, int32_t n_items, int32_t n_wg, int32_t n_xcd,
                                const double* die_speed, int64_t* die_span, difa_segment_t* segs,
                                int32_t seg_capacity, int32_t* wg_begin, int32_t* n_segs_out,
                                difa_merge_item_t* merges, int32_t merge_capacity, int32_t* n_merges_out,
                                int32_t* n_slots_out);

}  // namespace difa
