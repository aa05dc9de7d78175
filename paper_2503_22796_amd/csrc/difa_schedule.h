// The scheduler as the library itself calls it (host code only; defined in difa_worklist.cpp).
#pragma once
#include <stdint.h>

#include <vector>

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
// Measured on MI355X: clock counters around every segment, regressed per workgroup on what its list held (1K and 2K
// layers).  head_dim 128, one workgroup of eight wavefronts on a compute unit: 2950 clocks a plain iteration, 0.5-0.6
// iterations more on a masked tile, 5.9 for starting and finishing a whole record, 6.1 for a piece (9-11 while slots were
// laid out by rows), 2.4 for folding one other slot in; two workgroups of four wavefronts 2900, 0.7, 5.2, 5.7 and 3.0.
// head_dim 64, two workgroups of four wavefronts: 2000 clocks, 1.4, 1-3, 3-5 and 2.7 iterations.
// At head_dim 128 records and pieces are charged less than that (3.3 and 4.5 iterations, 2.4 a fold) and masked tiles more
// (1.0): what a schedule depends on is their difference and the tiles, and a schedule is corrected from its own launches
// besides (difa_trial.h).  Charging {6, 43, 46, 22, 8}, the measured ones, instead: FLUX-like 1K layer 128.8 us (129.1 as it
// is), 2K mixed 993 (1000), all full 2892 (2900), video-like 1312 (1328), w = 128 at 1K 94.0 (94.8), runs of one side differing
// by as much; one set does for both record lengths for the same reason.
// (An iteration is shorter by now, 2350-2650 and 1700-1850 clocks, and records, pieces and folds are more of them: 5.5-7, 5-8 and
// 2.3-2.9 at head_dim 128, 5-6, 5-6 and 2 at 64.  {10, 36, 42, 16, 8} and {8, 44, 50, 20, 8} changed no layer by more than 0.5 %.)
constexpr CostModel kernel_costs(int head_dim) {
    return head_dim == 64 ? CostModel{11, 12, 28, 21, 8} : CostModel{8, 26, 36, 19, 8};
}

// The records of difa_worklist_build, head by head and query tiles in ascending order, for a kernel whose records are
// `rows` query rows, a divisor of the block-granular band's block of `band_rows` rows: the key tiles a record visits
// are then those of the block it lies in.  `recs` is overwritten.  May throw std::bad_alloc, as the next one may.
difa_status_t worklist_for_kernel(int32_t batch, int32_t heads, const int32_t* head_plan, const int32_t* window,
                                  int32_t n_text, int32_t n_img, int32_t rows, int32_t band_rows, int32_t bn,
                                  uint32_t flags, std::vector<difa_work_item_t>& recs, int32_t* copy_heads,
                                  int32_t* n_copy_out);

// difa_schedule_build for records in that order, with three more arguments:
//   m           what a segment costs
//   die_speed   n_xcd relative speeds of the accelerator dies (NULL: all alike).  Under a heavy load the
//               dies of one chip settle at clocks a few percent apart; a die is given work in
//               proportion to its speed.
//   die_span    receives, per die, the predicted finishing time of its slowest workgroup in the
//               scheduler's cost units at speed 1 (NULL: not wanted).  The caller divides it by the die's
//               measured time to learn the speeds.
difa_status_t schedule_for_dies(const CostModel& m, const std::vector<difa_work_item_t>& recs, int32_t n_wg, int32_t n_xcd,
                                const double* die_speed, int64_t* die_span, difa_segment_t* segs,
                                int32_t seg_capacity, int32_t* wg_begin, int32_t* n_segs_out,
                                difa_merge_item_t* merges, int32_t merge_capacity, int32_t* n_merges_out,
                                int32_t* n_slots_out);

}  // namespace difa
