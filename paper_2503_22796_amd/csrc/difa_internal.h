// Internal declarations shared by the host API and the kernel translation unit.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "difa.h"

namespace difa {

constexpr int kBM = 256;  // query rows per block of the block-granular band, and per work record of the fp32 path
constexpr int kBN = 64;   // keys per K/V tile
// bf16 kernel: query rows per work record and workgroup (32 per wavefront).  Either way a SIMD has two wavefronts: they
// belong to one workgroup of 256 rows, or to two workgroups of 128 that know nothing of each other, so that the barriers,
// masks and record ends of one run under the other's arithmetic, records are half as long (easier to share out evenly, and a
// band covers fewer keys outside it), and every K/V tile is written to LDS twice as often.
// head_dim 64 (the softmax's share of an iteration is twice as large): 128 rows throughout.  Clocks per 256 rows x 64 keys on
// MI355X 2050 against 2190-2360; SD3-like 512 px layers 1.13 times as fast, the 1K layer up to 1.05; at 2K (where the clock
// gives way as the loop gets denser) the same.  64 rows per wavefront as well: 2010 clocks, 2K the same, 1K 0.75 times.
// head_dim 128: the loop takes 2350-2450 clocks with records of 128 rows and 2650 with 256, and the second copy of every tile costs
// the power that those clocks save (the chip holds less than 1.7 GHz on such layers; all-full 2K 2800 us with 256 rows, 2885 with
// 128).  Short records earn it back where a band covers noticeably fewer keys for 128 rows than for 256, where records are few tiles
// long, and where the layer is too small to fill the chip otherwise; with heads that see every key, or blocks of 256 rows, there is
// nothing to earn.  256 rows against 128, us
// (one MI355X, 24 heads but where said; "saved": share of the key tiles that the shorter records do not visit):
//   all full              1536 tokens 40.4 / 41.3, 4608 229 / 231, 9216 844 / 860, 13056 1668 / 1702, 16896 2799 / 2885
//   ... of few heads      1536 tokens, 6 heads 37.0 / 25.9, 12 heads 32.5 / 30.9; 2560 tokens, 6 heads 35.5 / 34.7, 12 heads 49.3 / 48.0
//   ... short             768 tokens 24.2 / 17.9, 300 tokens 16.2 / 11.5
//   block-granular band   16896 tokens, w = 2048 845 / 858, 1024 567 / 570, 512 424 / 420, 128 (17 tiles a record) 311 / 306;
//                         mixed plan 913 / 920
//   full and w = N / 16   12 + 12 at 9216 tokens (1.0 % saved) 546 / 547, at 4608 (1.8 %) 169.5 / 167.2;
//                         8 + 16 at 9216 (1.7 %) 454 / 440; 4 + 20 at 16896 (1.8 %) 991 / 959; mixed 2K (1.2 %) 958 / 964
//   all arrow             16896 tokens, w = 4224 (1.3 %, 14.6 M pairs a compute unit) 1404 / 1408, 2112 (2.3 %) 883 / 858,
//                         528 (5.3 %) 458 / 424; pairs of them, w = 2048 (2.4 %, 15.8 M) 1728 / 1748, 1024 (9.5 M) 1166 / 1157
// The lines below were drawn before the row sums moved to the matrix core and are no longer the best ones for this table: by them
// the all-full layers of 2560 tokens and few heads take 256 rows (2.3 and 2.7 % slower), so does the block-granular w = 512 (1 %), and the
// mixed 2K layer takes 128 (0.6 %).  Every other row of it gets its faster form.
constexpr int kRowsShort = 128, kRowsLong = 256;
constexpr double kLongPairsPerCu = 14.0e6;   // head_dim 128, query-key pairs per compute unit: 256 rows above this line,
constexpr double kShortPairsPerCu = 0.13e6;  // 128 below this one; between them 128 where an image record visits fewer
constexpr double kShortKeys = 24 * 64;       // keys than this on average, or where the shorter records save
constexpr double kShortSaves = 0.011;        // ... this share of the visited keys and more
constexpr int wgs_per_cu(int rows) { return 256 / rows; }
constexpr int copy_chunk_vecs(int rows) { return 32 * rows; }   // 16-byte vectors per chunk of the cached-head copy: 16 per thread

constexpr int kF32BlockRows = 16;      // fp32 kernel: query rows per workgroup
constexpr int kF32CopyVecs = 16 * 512; // ... and 16-byte vectors per chunk of its cached-head copy

// The cached-head copy of a layer as chunks of `chunk` 16-byte vectors.
struct CopySplit { int64_t head_vecs, per_head, chunks; };
inline CopySplit copy_split(int64_t n_tokens, int64_t vec_per_row, int64_t chunk, int64_t batch, int64_t n_copy) {
    const int64_t head_vecs = n_tokens * vec_per_row, per_head = (head_vecs + chunk - 1) / chunk;
    return {head_vecs, per_head, batch * n_copy * per_head};
}

// Arguments common to the attention kernels.  Strides are in elements.
struct AttnArgs {
    const void* q;
    const void* k;
    const void* v;
    void* out;
    const difa_work_item_t* items;  // device: one record per kBM query rows (fp32 kernel)
    const difa_segment_t* segs;     // device: segments grouped by workgroup (bf16 kernel)
    const int32_t* wg_begin;        // device: first segment of each workgroup, n_wg + 1 entries; sched_id stands in front of them
    const difa_merge_item_t* merges;  // device: records cut into pieces
    float* part_o;                  // device scratch: [slot][rows of a record][head_dim] unnormalised accumulators
    float* part_ml;                 // device scratch: [slot][rows of a record][2] row reference (log2 domain), row sum
    int32_t* tickets;               // device, one per cut record, zero between launches: pieces finished so far
    const void* residual;           // device, shaped like out: kept differences of the residual-sharing heads (or NULL)
    // cached heads: out[b, h] = copy_src[b, h] for the heads listed in copy_heads
    const void* copy_src;
    const int32_t* copy_heads;      // device, n_copy entries
    int64_t copy_stride_b, copy_stride_h, copy_stride_n;   // in bytes
    int32_t n_copy;
    int32_t copy_chunks;            // batch * n_copy * copy_chunks_per_head; 0: nothing to copy
    int32_t copy_chunks_per_head;
    int64_t copy_head_vecs;         // 16-byte vectors per (batch entry, head): n_tokens << copy_vec_shift (bf16: below 2^27)
    int32_t copy_vec_shift;         // log2(16-byte vectors per token row)
    int64_t stride_b, stride_h, stride_n;
    int32_t heads, n_tokens, n_text;
    int32_t younger_from;  // bf16 kernel: workgroups from this number on share a compute unit with an older one
    int32_t f32_blocks;  // fp32 kernel: workgroups of the computed heads (kBM / kF32BlockRows per record); copy chunks follow
    int32_t text_begin;  // first text token: 0, or n_img when the image tokens come first
    int32_t tile_rot;    // key-tile position u of a record is tile (u + tile_rot) % n_kv_tiles
    int32_t n_kv_tiles;
    float scale;  // softmax scale (natural-log domain)
    // bf16 kernel, optional: workgroup p leaves (launch_tag << 32 | its running time in ticks of the
    // constant-rate 100 MHz counter) in wg_times[p] when it ends (host memory mapped into the device; NULL: off)
    unsigned long long* wg_times;
    uint32_t launch_tag;
    int32_t sched_id;               // bf16 kernel: the schedule the launch was made for
};

struct CopyArgs {
    const void* src;
    void* dst;
    const int32_t* copy_heads;  // device, n_copy entries
    int64_t stride_b, stride_h, stride_n;  // in bytes
    int32_t batch, n_copy, n_tokens, vec_per_row;  // 16-byte vectors per token row
};

// Arguments of the influence-metric kernels.  Strides are in elements.
constexpr int kRseChunks = 64;  // workgroups per (batch, head) of the streaming pass
struct RseArgs {
    const void* y_m;
    const void* y_o;
    double* partial;  // device scratch: [batch * heads][kRseChunks][3]
    float* out;       // device: heads values
    int64_t stride_b, stride_h, stride_n;
    int32_t batch, heads, n_tokens, head_dim;
};

// Launchers (defined in difa_kernels.hip and difa_rse.hip).  All enqueue on `stream` and return the launch status.
hipError_t launch_attn_bf16(const AttnArgs& a, int head_dim, int rows, int n_wg, hipStream_t stream);
hipError_t launch_attn_f32(const AttnArgs& a, int head_dim, int n_items, hipStream_t stream);
hipError_t launch_cache_copy(const CopyArgs& a, hipStream_t stream);
hipError_t launch_head_rse(const RseArgs& a, int dtype, hipStream_t stream);
hipError_t launch_residual_store(const void* o_full, const void* o_arrow, void* residual, int64_t n_elems, int dtype,
                                 hipStream_t stream);

// File-scope device scratch of difa_joint_attention_static (defined beside the kernels that use it).
// static_scratch_init: looks up the array's address on `device`, which must be the current device; once per
// device, later calls return at once.  static_scratch: that address (NULL before init) and the array's size.
hipError_t static_scratch_init(int device);
float* static_scratch(int device, size_t* bytes);

}  // namespace difa
