// gfx950 kernels of the head-wise joint-attention operator (Sec. 3.3 of the paper):
//   attn_bf16_kernel  -- the whole layer in one launch: full / arrow heads with bf16 MFMA and fp32
//                        accumulation, then the cached heads, out[b,h] = cache[b,h] (the cache fill that
//                        ends Alg. 1), copied by whichever workgroups have finished their attention work
//   attn_f32_kernel   -- the fp32 debug path: fp64 contractions on the matrix cores, fp32 exponentials; cached heads too
//   cache_copy_kernel -- a layer with every head cached
#include <mutex>
#include <type_traits>

#include "difa_internal.h"

namespace difa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Maximum / sum of a value over the two halves of a wavefront (lanes l and l^32).
// v_permlane32_swap is a VALU instruction: unlike ds_bpermute it does not queue behind the LDS
// reads in flight.  With both operands equal it returns {low half, low half} and {high half, high half}.
__device__ __forceinline__ float halves_max(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned lo = r[0], hi = r[1];    // copied to scalars first: a bit_cast applied directly to a vector element reads element 0
    return fmaxf(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
}
__device__ __forceinline__ float halves_sum(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned lo = r[0], hi = r[1];
    return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA attention.
//
// A workgroup is BM / 32 wavefronts (eight, or two workgroups of four on a compute unit: two per SIMD) and stays resident: it walks
// the list of segments the host scheduler gave it.  A segment is a BM-row query tile of one (batch, head) together with a
// run of that record's key/value tiles (the whole run for most records; a few records are cut so
// that every workgroup ends at the same time, and their pieces leave fp32 partial results that the
// piece finishing last folds into its own).  Wavefront w owns rows 32*w .. 32*w+31.
// Key/value tiles of 64 keys are written into 4-stage LDS rings by the buffer-load-to-LDS DMA, K three
// tiles and V two tiles ahead of their use (with two workgroups on a compute unit: stages of half a tile, K four and V two
// blocks of 32 keys ahead, a barrier for every block),
// in the order the work record lists them (text tiles,
// then the band tiles), so a tile with no allowed pair is never loaded (Sec. 3.1 / 3.3:
// block-sparse band).  The first tiles and the Q rows of the next segment are requested before
// the current segment's epilogue.
//
// Rows per wavefront: with 64 rows every 16-byte-per-lane LDS operand read would feed two MFMAs,
// but the whole register file would go to one wavefront per SIMD, and a single wavefront does not overlap
// its own vector arithmetic with its own MFMAs: measured, the clocks of the two simply add.  With 32
// rows a wavefront fits in half the register file, two share a SIMD, and one's softmax runs
// under the other's MFMAs; LDS (twice the operand reads) is busy about a third of the time.  (Before the row sums moved to the
// matrix core 32 rows took 16 % fewer clocks a key tile than 64 and 5-19 % less time in the 1K layers, head_dim 64 and narrow windows; at
// the long 2K layers the same time, where the chip runs at its power limit.)
//
// Scores are produced transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: a lane then holds
// 16 keys of ONE query (column = lane % 32), so the softmax row statistics are per-lane scalars
// (a maximum needs one exchange between the wavefront halves, the sums come from the matrix core).  The same register layout is exactly the
// B operand of O^T = V^T P^T, so P never goes through LDS.  V stays row-major [key][feature] in
// LDS and its transposed operand comes from ds_read_b64_tr_b16.
//
// Software pipeline inside a wavefront: a wavefront issues in order, so the loop body is laid
// out by hand as 8 slots per 32-key half-step, each slot one MFMA (S^T of the next block, or
// P V of the previous one) followed by the few vector instructions of the softmax of the block
// in between, an LDS operand read or a DMA request; the vector work runs while the matrix core
// is busy with the slot's MFMA.
// ------------------------------------------------------------------------------------------
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

// LDS transpose read: within each group of 16 lanes, lane i receives element (i % 4) of the four
// 8-byte rows that lanes (i/4), 4+(i/4), 8+(i/4), 12+(i/4) of the group point at.
__device__ __forceinline__ bf16x4 lds_read_tr16(const __bf16* p) {
    const shortx4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (shortx4 __attribute__((address_space(3)))*)(p));
    return __builtin_bit_cast(bf16x4, r);
}

// S^T = K Q^T MFMAs are written as assembly so that the register classes are fixed: the scores
// accumulate in ordinary vector registers, where the softmax arithmetic reads them directly (the
// compiler's own choice for a kernel this size is accumulation registers plus one copy per score),
// and the Q operand sits in accumulation registers, which only matrix instructions read.
// The hardware does not interlock a vector instruction that reads a matrix result too early and the
// compiler does not see through the assembly, so every reader is a full half-step away, preceded by an explicit wait
// (mfma_results_visible, tied to the registers: a wait that names only memory holds back no read of a register), or behind the read
// of a younger matrix instruction's result, one that the compiler knows about and waits for (settled_results).
__device__ __forceinline__ void mfma_s_first(floatx16& d, const bf16x8& k, const bf16x8& q) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(k), "a"(q));
}
__device__ __forceinline__ void mfma_s_acc(floatx16& d, const bf16x8& k, const bf16x8& q) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "a"(q));
}
__device__ __forceinline__ void mfma_results_visible(floatx16& d) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(d) :: "memory"); }
// No wait, only the order: for results of an MFMA that a younger MFMA's result has already been read behind.  (The matrix
// pipe works in order.)
__device__ __forceinline__ void settled_results(floatx16& d) { asm volatile("" : "+v"(d) :: "memory"); }

// Cache-policy operand of the buffer load/store builtins: device scope ("sc1").
constexpr int kDeviceCoherent = 16;
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));

struct RowState {
    float m;       // reference maximum (log2 domain) the weights are expressed against
    float l;       // running sum of the weights
    int lo;        // band of allowed image keys is [lo, lo + span]; text keys are always allowed
    unsigned span;
};

// One chunk of the cached-head copy: 16 vectors of 16 bytes per thread, all in flight together.
template <int THREADS>
__device__ __forceinline__ void copy_vectors(const AttnArgs& ca, int chunk, int tid) {
    constexpr int PER = 16;
    const int per_head = ca.copy_chunks_per_head, n_copy = ca.n_copy, shift = ca.copy_vec_shift;
    const int64_t row_bytes = ca.copy_stride_n;
    const int hh = chunk / per_head, cc = chunk - hh * per_head;
    const int bb = hh / n_copy, head = ca.copy_heads[hh - bb * n_copy];
    // a chunk is whole token rows: its first one is found in 64 bits (a head may hold 2^31 vectors and more), the rest in 32
    const int64_t first = (int64_t)cc * (PER * THREADS), left = ca.copy_head_vecs - first;
    const int vecs = left < PER * THREADS ? (int)left : PER * THREADS;
    const int64_t base = (int64_t)bb * ca.copy_stride_b + (int64_t)head * ca.copy_stride_h + (first >> shift) * row_bytes;
    const char* __restrict__ src = (const char*)ca.copy_src + base;
    char* __restrict__ dst = (char*)ca.out + base;
    uintx4 val[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int vi = u * THREADS + tid;                                     // vector inside the chunk
        const int vr = vi < vecs ? vi : vecs - 1;                             // past the end: reread the last one, store nothing
        val[u] = *(const uintx4*)(src + (vr >> shift) * row_bytes + (vr & ((1 << shift) - 1)) * 16);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int vi = u * THREADS + tid;
        if (vi < vecs) *(uintx4*)(dst + (vi >> shift) * row_bytes + (vi & ((1 << shift) - 1)) * 16) = val[u];
    }
}

template <int D, int BM>                        // BM: query rows per record
__global__ __launch_bounds__(2 * BM, 2) void attn_bf16_kernel(AttnArgs a) {
    constexpr int RW = 32;                  // query rows of a wavefront
    constexpr int NW = BM / RW;             // wavefronts per workgroup
    constexpr int KS = D / 16;              // MFMA k-steps of S^T = K Q^T
    constexpr int DB = D / 32;              // 32-row blocks of O^T
    constexpr int CPR = D / 8;              // 16-byte chunks per K/V row
    // Two workgroups on a compute unit: the rings hold 32-key blocks (half tiles) instead of tiles.  At head_dim 128 whole
    // tiles would not fit twice.  At head_dim 64 they would (measured: SD3-like 512 px refresh 90.5 us against 87.0, 1K 145.6 /
    // 142.3, 2K 1455 / 1441; the smallest call, one tile long, 8.5 / 8.9), but a ring that a tile moves by two stages
    // needs two copies of the loop body instead of four, and two compute units share 64 KB of instruction cache.
    constexpr bool BLK = BM == 128;
    constexpr int RKEYS = BLK ? kBN / 2 : kBN;    // keys per ring stage
    constexpr int TILE = RKEYS * D;         // elements of one ring stage
    constexpr int NS = 4;                   // LDS ring depth, K and V alike: tile p lives in stage p % 4
    constexpr float kTrip = 0x1p40f;        // a block row sum beyond this sends the wavefront to the renormalising side path
    constexpr float kBump = 16.0f;          // ... where a row's reference moves if its block maximum exceeds it by 2^16

    // LDS moves 256 bytes per clock over 64 banks of 4 bytes: a b128 read is served 16 lanes at a time
    // (16 consecutive key rows, one 16-byte chunk each), a transpose read 32 lanes at a time (4 key rows
    // x 8 pieces of 8 bytes out of one group of 4 chunks).  A 256-byte row (D = 128) covers every bank
    // once, a 128-byte row (D = 64) half of them, alternating with the row's parity.  The 16-byte chunk c
    // of row r is therefore stored at chunk c ^ kswz(r) (K) or c ^ vswz(r) (V), chosen so that the
    // lanes served together land in different banks:
    //   K: 16 rows x 1 chunk:  D = 128: r % 16;        D = 64: (r / 2) % 8 (rows of one parity share banks)
    //   V: 4 rows x 4 chunks:  D = 128: 4 * (r % 4);   D = 64: 2 * (r % 4) (the group moves for r % 4 >= 2, the parity does the rest)
    auto kswz = [](int r) { return CPR == 16 ? (r & 15) : ((r >> 1) & 7); };
    auto vswz = [](int r) { return CPR == 16 ? 4 * (r & 3) : 2 * (r & 3); };
    __shared__ __attribute__((aligned(16))) __bf16 Ksm[NS * TILE];
    __shared__ __attribute__((aligned(16))) __bf16 Vsm[NS * TILE];
    __shared__ int ctl_sm[4];                // [0]: a ticket, handed from thread 0 to the workgroup; [2..3]: thread 0's start time
    // The arguments that only the rare paths use (merging a cut record, the cached-head copy) are read
    // from the kernel-argument block where they are needed: named through `a` they would be fetched at
    // kernel entry and held in scalar registers for the whole key loop, which has none to spare.
    auto cold_args = []() __attribute__((always_inline)) {
        unsigned long long kp = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(kp));
        return (const AttnArgs*)kp;
    };

    const int tid = threadIdx.x, wave_v = tid >> 6;
    // How long the workgroup runs is reported to the host, which learns from it how fast each accelerator
    // die is going (their clocks differ by a few percent under load) and shares out later work accordingly.
    // The start time waits in LDS (ctl_sm[2..3]): no register is held for it across the kernel.
    int l32, half;                                          // lane % 32, lane / 32 (set by lane_offsets below)
    const int N = a.n_tokens, n_text = a.n_text;
    // text tokens are [text_begin, text_begin + n_text), image tokens [img0, img1) (the text block sits
    // before or after the image block); a record's key-tile position u is tile (u + tile_rot) % n_kv_tiles
    const int text_begin = a.text_begin;
    const int img0 = text_begin == 0 ? n_text : 0, img1 = text_begin == 0 ? N : text_begin;
    auto tile_at = [&](int u) { const int t = u + a.tile_rot; return t >= a.n_kv_tiles ? t - a.n_kv_tiles : t; };
    const float c = a.scale * 1.44269504088896340736f;      // scores are kept in the log2 domain

    // ---- per-lane offsets: LDS operand reads (elements, within one stage) and the lane's place in a tile load
    int koff[KS];                                           // A operand of S^T: row l32, chunk 2*ks+half
    int voff[DB];                                           // transpose read: row 4*half + s/4, 4 features

    // ---- global -> LDS: K/V tiles are written into the ring by the load itself
    // (buffer_load_dwordx4 ... lds: lane l of a wavefront deposits its 16 bytes at M0 + 16*l), so a
    // tile never occupies registers and needs no ds_write.  One instruction fills RPI consecutive
    // tile rows; the XOR swizzle of the LDS layout is applied by permuting which 16-byte chunk of the
    // row each lane fetches.  One buffer descriptor per tensor for the segment's (batch, head): rows
    // past the last token read as zero (they are masked later).  The loads are outside the compiler's
    // view, so the wait for them is explicit (dma_wait) and sits just before the barrier that
    // publishes the tile.
    constexpr int RPI = 64 / CPR;                           // tile rows per load instruction
    constexpr int NDMA = RKEYS / RPI / NW;                     // load instructions per wavefront, tensor and tile
    const unsigned head_bytes = (unsigned)(((int64_t)(N - 1) * a.stride_n + D) * 2);
    uintx4 krsrc, vrsrc;                                    // descriptors of the head whose tiles are being loaded
    // (Products of the vector form of the wavefront's number, held from segment to segment, came to 28 bytes of scratch a lane in the
    // 256-row kernel, with a reload in each segment's first half-step that waited for every load in flight.  The scalar
    // form in the others as well: the SD3-like 512 px refresh 79.7 us instead of 79.2.)
    const unsigned wave_u = __builtin_amdgcn_readfirstlane(wave_v);
    const int wave = BM == kRowsLong ? (int)wave_u : wave_v;
    unsigned gk[NDMA], gv[NDMA];                            // per-lane byte offsets inside a tile
    // These sixteen-odd registers are derived from the lane number again at the start of every segment,
    // through a copy the compiler cannot see through.  Held for the whole kernel instead, they would be
    // live across the rare, register-hungry paths between segments (merging a cut record, the cached-head
    // copy), and the register allocator would answer by parking some of them in accumulation registers
    // and fetching them back inside the key loop.
    auto lane_offsets = [&]() __attribute__((always_inline)) {
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        l32 = lane & 31;
        half = lane >> 5;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) koff[ks] = l32 * D + 8 * ((2 * ks + half) ^ kswz(l32));
        const int blk = lane >> 4, s16 = lane & 15;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int chunk = 4 * db + 2 * (blk & 1) + ((s16 & 3) >> 1);
            voff[db] = (4 * half + (s16 >> 2)) * D + 8 * (chunk ^ vswz(s16 >> 2)) + 4 * (s16 & 1);
        }
#pragma unroll
        for (int u = 0; u < NDMA; ++u) {
            const int r = (wave * NDMA + u) * RPI + lane / CPR, pc = lane % CPR;   // tile row, chunk slot in LDS
            gk[u] = (unsigned)(r * (int)a.stride_n + 8 * (pc ^ kswz(r))) * 2u;
            gv[u] = (unsigned)(r * (int)a.stride_n + 8 * (pc ^ vswz(r))) * 2u;
        }
    };
    const unsigned tile_bytes = (unsigned)(kBN * (int)a.stride_n) * 2u;
    const unsigned k_lds = (unsigned)(unsigned long long)(__attribute__((address_space(3))) __bf16*)Ksm;
    const unsigned v_lds = (unsigned)(unsigned long long)(__attribute__((address_space(3))) __bf16*)Vsm;
    // One load instruction: part u (0..NDMA-1) of a K (tensor 0) or V (tensor 1) tile.  `tb` is the tile's
    // byte offset inside the head, or an offset beyond the buffer for positions past the end of the
    // segment (those fetch nothing and deposit zeros); `dst` is this wavefront's LDS byte address inside
    // the ring stage.  All per-tile scalars are computed once per iteration by the caller.
    auto dma_part = [&](int tensor, int u, unsigned tb, unsigned dst) __attribute__((always_inline)) {
        if (tensor == 0)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                         :: "s"(dst + (unsigned)(u * RPI * D * 2)), "v"(gk[u] + tb), "s"(krsrc) : "m0");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                         :: "s"(dst + (unsigned)(u * RPI * D * 2)), "v"(gv[u] + tb), "s"(vrsrc) : "m0");
    };
    const unsigned wave_lds = wave_u * (unsigned)(NDMA * RPI * D * 2);     // this wavefront's rows inside a stage
    // all loads done / all but the 2*NDMA youngest (= the tiles issued during the current iteration) done
    auto dma_wait_all = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    auto dma_wait_older = [] { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * NDMA) : "memory"); };

    // What a segment needs before its first block: its K tiles 0..2 and V tiles 0, 1 in the ring (the
    // segment's tile p goes to stage (sb + p) % 4) and its query rows in the Q operand registers.
    // Requested ahead of time: for the first segment at once, for every other one by its predecessor,
    // between the end of its own key loop and its epilogue.
    bf16x8 qf[KS];
    auto first_tiles = [&](const difa_segment_t& sg, int sb) __attribute__((always_inline)) {
        const int b = sg.bh / a.heads, h = sg.bh - b * a.heads;
        const int64_t base = (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
        const unsigned long long ka = (unsigned long long)((const __bf16*)a.k + base);
        const unsigned long long va = (unsigned long long)((const __bf16*)a.v + base);
        krsrc[0] = (unsigned)ka; krsrc[1] = (unsigned)(ka >> 32) & 0xffffu; krsrc[2] = head_bytes; krsrc[3] = 0x00020000u;
        vrsrc[0] = (unsigned)va; vrsrc[1] = (unsigned)(va >> 32) & 0xffffu; vrsrc[2] = head_bytes; vrsrc[3] = 0x00020000u;
        const int n = sg.pos_end - sg.pos_begin;
        if constexpr (BLK) {                                // blocks 0..3 of K, 0 and 1 of V
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int p = sg.pos_begin + t;
                const int tile = tile_at(p < sg.kv0_end ? p : sg.kv1_begin + (p - sg.kv0_end));
                const unsigned tb = t < n ? (unsigned)tile * tile_bytes : 0x80000000u;
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    const unsigned st = (unsigned)(((sb + 2 * t + jb) & 3) * TILE * 2) + wave_lds;
#pragma unroll
                    for (int u = 0; u < NDMA; ++u) {
                        dma_part(0, u, tb + jb * (tile_bytes / 2), k_lds + st);
                        if (t == 0) dma_part(1, u, tb + jb * (tile_bytes / 2), v_lds + st);
                    }
                }
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int p = sg.pos_begin + t;
            const int tile = tile_at(p < sg.kv0_end ? p : sg.kv1_begin + (p - sg.kv0_end));
            const unsigned tb = t < n ? (unsigned)tile * tile_bytes : 0x80000000u;
            const unsigned st = (unsigned)(((sb + t) & 3) * TILE * 2) + wave_lds;
#pragma unroll
            for (int u = 0; u < NDMA; ++u) {
                dma_part(0, u, tb, k_lds + st);
                if (t < 2) dma_part(1, u, tb, v_lds + st);
            }
        }
    };
    constexpr int kFirstTileLoads = (BLK ? 6 : 5) * NDMA;               // load instructions first_tiles issues
    auto query_rows = [&](const difa_segment_t& sg) __attribute__((always_inline)) {
        const int b = sg.bh / a.heads, h = sg.bh - b * a.heads;
        const int64_t base = (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
        const __bf16* qg = (const __bf16*)a.q + base;
        const int i_r = sg.q_tile * BM + wave * RW + l32;
        const int i = i_r < N ? i_r : N - 1;            // rows past the end recompute row N-1
        // B operand of S^T = K Q^T: column = query l32, k-slots 8*half..8*half+7 of each 16-wide step
        const __bf16* qrow = qg + (int64_t)i * a.stride_n + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(qrow + 16 * ks);
    };
    auto first_loads = [&](const difa_segment_t& sg, int sb) __attribute__((always_inline)) {
        first_tiles(sg, sb);
        query_rows(sg);
    };

    // Persistent workgroup: one or two per compute unit, walking the segments the host scheduled for it.
    // The record of the following segment is fetched at the start of the current one.
    // A launch replayed from a graph may find that its schedule has given way to another, for the other record length even: the
    // segments would name scratch slots beyond the end, and half of a record's pieces would leave their ticket standing.  It has
    // nothing to do then.  (All three words are read together; a return up front put a memory latency before every launch: 0.8 us.)
    const bool mine = __builtin_amdgcn_readfirstlane(a.wg_begin[-1]) == a.sched_id;
    const int seg_first = __builtin_amdgcn_readfirstlane(a.wg_begin[blockIdx.x]);
    const int seg_listed = __builtin_amdgcn_readfirstlane(a.wg_begin[blockIdx.x + 1]), seg_end = mine ? seg_listed : seg_first;
    // ---- cached heads (Sec. 3.2; the cache fill that ends Alg. 1): out[b, h] = cache[b, h], bit for bit.
    // HBM-bound work that needs no matrix core.  It is cut into chunks of copy_chunk_vecs(BM) 16-byte vectors of one
    // (batch entry, cached head); workgroup p takes chunks p, p + gridDim.x, ... and moves one after each of
    // its attention segments, when it waits for the next segment's first tiles anyway, so the copy is
    // spread over the launch and runs in the shadow of the other workgroups' arithmetic.
    auto copy_chunk = [&](int chunk) __attribute__((always_inline)) {
        constexpr int PER = copy_chunk_vecs(BM) / (NW * 64);          // vectors per thread and chunk, all in flight together
        const AttnArgs* ca = cold_args();
        const int per_head = ca->copy_chunks_per_head, n_copy = ca->n_copy, shift = ca->copy_vec_shift;
        const int head_vecs = (int)ca->copy_head_vecs;
        const unsigned row_bytes = (unsigned)ca->copy_stride_n;     // (a head spans less than 2 GiB)
        const int hh = chunk / per_head, cc = chunk - hh * per_head;
        const int bb = hh / n_copy, head = ca->copy_heads[hh - bb * n_copy];
        const int64_t base = (int64_t)bb * ca->copy_stride_b + (int64_t)head * ca->copy_stride_h;
        const char* __restrict__ src = (const char*)ca->copy_src + base;
        char* __restrict__ dst = (char*)ca->out + base;
        uintx4 val[PER];
        unsigned off[PER];
        bool live[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            int vi = cc * copy_chunk_vecs(BM) + u * (NW * 64) + tid;                // vector inside the head
            live[u] = vi < head_vecs;
            vi = live[u] ? vi : head_vecs - 1;                            // past the end: reread the last one, store nothing
            off[u] = (unsigned)(vi >> shift) * row_bytes + (unsigned)(vi & ((1 << shift) - 1)) * 16u;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) val[u] = *(const uintx4*)(src + off[u]);
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (live[u]) *(uintx4*)(dst + off[u]) = val[u];
    };
    int next_chunk = mine ? (int)blockIdx.x : 0x7fffffff;
    // Where two workgroups share a compute unit, its SIMDs serve the older wavefront first: left to itself (head_dim 64) the
    // workgroup that was dispatched second ran at 2500 clocks an iteration beside 1735 of the other (before the row sums moved to
    // the matrix core), and the schedule, which gives both the same work, waits for it.  So the younger half of the grid runs every other
    // iteration at the higher priority.  With and without: SD3-like 2K layer 1365 / 1391 us, 1K 132.3 / 136.5; every half-step instead 1377 and 135.8; head_dim
    // 128 the same either way.  (A segment leaves the priority as its last iteration had it: lowering it after the key loop changes nothing.)
    const bool younger = wgs_per_cu(BM) > 1 && (int)blockIdx.x >= a.younger_from;

    difa_segment_t seg_next{};
    int sbase = 0;                                          // ring stage of the current segment's tile 0
    if (seg_first < seg_end) {
        seg_next = a.segs[seg_first];
        lane_offsets();
        first_loads(seg_next, sbase);
        // (the clock is read here, a few hundred clocks into the kernel, rather than on entry: at this point it
        // costs no register that the key loop needs)
        if (tid == 0) {
            const unsigned long long t = wall_clock64();
            ctl_sm[2] = (int)(unsigned)t;
            ctl_sm[3] = (int)(unsigned)(t >> 32);
        }
    }
    for (int seg_idx = seg_first; seg_idx < seg_end; ++seg_idx) {
    lane_offsets();
    // (the record was read with vector loads; moving its fields to scalar registers tells the compiler
    // that everything derived from them is uniform over the wavefront)
    difa_segment_t it;
    it.bh = __builtin_amdgcn_readfirstlane(seg_next.bh);
    it.q_tile = __builtin_amdgcn_readfirstlane(seg_next.q_tile);
    it.kv0_end = __builtin_amdgcn_readfirstlane(seg_next.kv0_end);
    it.nm0_end = __builtin_amdgcn_readfirstlane(seg_next.nm0_end);
    it.kv1_begin = __builtin_amdgcn_readfirstlane(seg_next.kv1_begin);
    it.kv1_end = __builtin_amdgcn_readfirstlane(seg_next.kv1_end);
    it.nm1_begin = __builtin_amdgcn_readfirstlane(seg_next.nm1_begin);
    it.nm1_end = __builtin_amdgcn_readfirstlane(seg_next.nm1_end);
    it.window = __builtin_amdgcn_readfirstlane(seg_next.window);
    it.pos_begin = __builtin_amdgcn_readfirstlane(seg_next.pos_begin);
    it.pos_end = __builtin_amdgcn_readfirstlane(seg_next.pos_end);
    it.part_slot = __builtin_amdgcn_readfirstlane(seg_next.part_slot);
    it.merge_idx = __builtin_amdgcn_readfirstlane(seg_next.merge_idx);
    it.n_parts = __builtin_amdgcn_readfirstlane(seg_next.n_parts);
    it.first_slot = __builtin_amdgcn_readfirstlane(seg_next.first_slot);
    it.flags = __builtin_amdgcn_readfirstlane(seg_next.flags);

    const int b = it.bh / a.heads, h = it.bh - b * a.heads;
    __bf16* __restrict__ og = (__bf16*)a.out + (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
    const int row0 = it.q_tile * BM + wave * RW;           // first query row of this wavefront

    // ---- per-lane query row and its allowed key range
    RowState rs;
    const int i_raw = row0 + l32, i_row = i_raw < N ? i_raw : N - 1;
    {
        int lo, hi;
        if (it.window < 0 || (unsigned)(i_row - text_begin) < (unsigned)n_text) { lo = 0; hi = N - 1; }
        else { lo = i_row - it.window; hi = i_row + it.window < N - 1 ? i_row + it.window : N - 1; }
        rs.lo = lo;
        rs.span = (unsigned)(hi - lo);                      // key j is in the band iff (unsigned)(j-lo) <= span
        rs.m = -1.0e30f;                                    // finite: exp2(-inf - m) must be 0, not NaN
        rs.l = 0.f;
    }

    // A operand of the row sums.  P as it stands (lane l: query l % 32, keys of half l / 32) read as the B operand of a
    // 16x16x32 product has query l % 16 + 16 * (l / 16 % 2) in column l % 16 and key slots 8 * (l / 16) .. + 7: row m of A
    // has ones in the slots of the lane groups whose parity is that of m / 4, so that every lane receives, in
    // register 0, the sum over both halves' keys of its own query's weights.  (Only every fourth row is there, the one register
    // 0 comes from: with ones in the other rows as well the products take more power, 1-1.5 % of the clock.)
    bf16x8 row_ones;
    {
        const int lane = l32 + 32 * half;
#pragma unroll
        for (int e = 0; e < 8; ++e) row_ones[e] = (__bf16)((((lane >> 4) ^ (lane >> 2)) & 1) || (lane & 3) ? 0.f : 1.f);
    }
    floatx16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;

    // The segment covers positions [pos_begin, pos_end) of the record's visiting order; idx counts from
    // the segment's first position.
    const int n_iter = it.pos_end - it.pos_begin;
    auto upos_of = [&](int idx) {                           // key-tile position in the record's rotated order
        const int p = it.pos_begin + (idx < n_iter ? idx : n_iter - 1);   // past the end: reload the last tile (unused)
        return p < it.kv0_end ? p : it.kv1_begin + (p - it.kv0_end);
    };
    auto tile_of = [&](int idx) { return tile_at(upos_of(idx)); };
    auto tile_masked = [&](int idx) {
        const int t = upos_of(idx);
        return it.pos_begin + idx < it.kv0_end ? (t >= it.nm0_end) : (t < it.nm1_begin || t >= it.nm1_end);
    };
    auto tile_offset = [&](int idx) {                       // byte offset of the tile at position idx
        return idx < n_iter ? (unsigned)tile_of(idx) * tile_bytes : 0x80000000u;
    };

    // ---- S^T = K Q^T for one 32-key block jb of a tile: s, register r = key 32*jb + 8*(r/4) + 4*half + r%4
    auto qk_block = [&](int idx, int jb, floatx16& s) {
        const __bf16* kst = BLK ? &Ksm[((2 * idx + jb + sbase) & 3) * TILE] : &Ksm[((idx + sbase) & 3) * TILE + 32 * jb * D];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 ka = *(const bf16x8*)(kst + koff[ks]);
            if (ks == 0) mfma_s_first(s, ka, qf[ks]);
            else mfma_s_acc(s, ka, qf[ks]);
        }
        mfma_results_visible(s);
    };
    // Element mask of one 32-key block whose first key is j0.  The host marks a tile as masked when any
    // of the record's rows has a forbidden key in it; for the rows of one wavefront most such
    // blocks lie entirely inside the band.  Which first keys those are is two intervals of the segment: blocks of text keys, and
    // for a wavefront of image rows the blocks that all its bands cover (of other rows: everything before the end).
    const int row_first = it.q_tile * BM + (int)wave_u * RW < N ? it.q_tile * BM + (int)wave_u * RW : N - 1;   // this wavefront's rows
    const int row_last = row_first + RW - 1 < N - 1 ? row_first + RW - 1 : N - 1;
    int free0 = 0, free_last = N - 32;                                     // a full head, or rows that are all text
    if (it.window >= 0 && row_last >= img0 && row_first < img1) {
        free0 = row_last - it.window > img0 ? row_last - it.window : img0;
        free_last = row_first + it.window < img1 - 1 ? row_first + it.window - 31 : img1 - 32;
        if (row_first < img0 || row_last >= img1) free_last = -1;         // rows of both kinds
    }
    const bool some_free = free_last >= free0, some_text = n_text >= 32;
    const int free_from = some_free ? free0 : -1, text_from = some_text ? text_begin : -1;   // (-1: no block begins there)
    const unsigned free_span = some_free ? (unsigned)(free_last - free0) : 0u, text_span = some_text ? (unsigned)(n_text - 32) : 0u;
    auto mask_block = [&](int j0, floatx16& s) {
        if ((unsigned)(j0 - free_from) <= free_span || (unsigned)(j0 - text_from) <= text_span) return;
        const unsigned ninf = 0xff800000u;
        // Bit r of `keep` says that register r holds the score of an allowed key.  Register r of a lane holds the key at
        // offset 8*(r/4) + r%4 (+ 4*half) of the block, increasing with r, so the keys below some key are the lane's
        // first k registers; the count k comes from that key with a handful of integer instructions.
        auto below = [&](int key) {                                    // registers whose key is < key
            const int e = key - j0 - 4 * half, ec = e < 0 ? 0 : (e > 32 ? 32 : e);
            const int rem = ec & 7;
            return (1u << (4 * (ec >> 3) + (rem < 4 ? rem : 4))) - 1u;
        };
        unsigned keep = below(rs.lo + (int)rs.span + 1) & ~below(rs.lo);
        // text keys in the block (spelled out key by key this was 150 instructions, ten times in the kernel, and pushed the
        // loop out of the instruction cache two compute units share)
        if (j0 < img0 || j0 + 31 >= img1) keep |= below(text_begin + n_text) & ~below(text_begin);
        // Each score then costs a signed one-bit extract (all ones or zero) and a bit-select between the score
        // and -inf, in place.  No compare writes a lane mask that the next instruction would have to wait for
        // (a compare and a select that reads its result cost 20 clocks a pair on this chip, four ordinary
        // instructions 16), and the sixteen registers are not rebuilt elsewhere (a select per score into a
        // fresh set of registers makes the compiler copy all sixteen over and back on every path through
        // here, the one that changes nothing included).
        // (one statement for the block's sixteen scores, written out so that the compiler neither turns
        // the bit-select back into a compare and a select nor pads every score with a wait state)
        float x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = s[r];
        unsigned t0, t1;
        asm volatile("v_bfe_i32 %16, %18, 0, 1\n\tv_bfe_i32 %17, %18, 1, 1\n\tv_bfi_b32 %0, %16, %0, %19\n\tv_bfi_b32 %1, %17, %1, %19\n\tv_bfe_i32 %16, %18, 2, 1\n\tv_bfe_i32 %17, %18, 3, 1\n\tv_bfi_b32 %2, %16, %2, %19\n\tv_bfi_b32 %3, %17, %3, %19\n\tv_bfe_i32 %16, %18, 4, 1\n\tv_bfe_i32 %17, %18, 5, 1\n\tv_bfi_b32 %4, %16, %4, %19\n\tv_bfi_b32 %5, %17, %5, %19\n\tv_bfe_i32 %16, %18, 6, 1\n\tv_bfe_i32 %17, %18, 7, 1\n\tv_bfi_b32 %6, %16, %6, %19\n\tv_bfi_b32 %7, %17, %7, %19\n\tv_bfe_i32 %16, %18, 8, 1\n\tv_bfe_i32 %17, %18, 9, 1\n\tv_bfi_b32 %8, %16, %8, %19\n\tv_bfi_b32 %9, %17, %9, %19\n\tv_bfe_i32 %16, %18, 10, 1\n\tv_bfe_i32 %17, %18, 11, 1\n\tv_bfi_b32 %10, %16, %10, %19\n\tv_bfi_b32 %11, %17, %11, %19\n\tv_bfe_i32 %16, %18, 12, 1\n\tv_bfe_i32 %17, %18, 13, 1\n\tv_bfi_b32 %12, %16, %12, %19\n\tv_bfi_b32 %13, %17, %13, %19\n\tv_bfe_i32 %16, %18, 14, 1\n\tv_bfe_i32 %17, %18, 15, 1\n\tv_bfi_b32 %14, %16, %14, %19\n\tv_bfi_b32 %15, %17, %15, %19"
                     : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]),
                       "+v"(x[8]), "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]), "+v"(x[15]),
                       "=&v"(t0), "=&v"(t1)
                     : "v"(keep), "v"(ninf));
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = x[r];
    };
    // ---- softmax of one 32-key block, cut into 16 pieces of six VALU instructions, one per slot, each
    // split in two halves that sit behind the slot's two MFMAs (a wavefront issues in order:
    // whatever is not behind an MFMA delays the next one; the steady state spends nothing on a running
    // maximum).
    //   piece s: scores 2*(s&7), 2*(s&7)+1 of row block s>>3 -> two weights 2^(score*c - reference) as
    //   bf16 B operands (convert)
    // The reference of a row is NOT the running maximum: it is set from the first block that holds an
    // allowed key and afterwards moves only when a weight outgrows 2^kTrip.  That is detected after
    // the fact, from the block's row sum, and repaired on a rare side path (renormalise() below), so
    // the hot path needs no maximum at all.  Weights are at most 2^kTrip * 16: bf16 has fp32's exponent
    // range, the row sum and O stay below 2^kTrip * N * max|v| < 2^70, far inside fp32, and the
    // common factor cancels in O / l.
    // Each piece ends in an empty volatile asm on its results: that keeps it in its slot (otherwise the
    // optimizer sinks the arithmetic to the block that uses it).
    auto pin = [](float& x) { asm volatile("" : "+v"(x)); };
    auto softmax_a = [&](int s, const floatx16& sc, float mneg, float (&x)[2]) __attribute__((always_inline)) {
        const int r = 2 * s;
        x[0] = __builtin_amdgcn_exp2f(fmaf(sc[r], c, mneg));
        x[1] = fmaf(sc[r + 1], c, mneg);
        pin(x[0]);
        pin(x[1]);
    };
    auto convert = [&](int s, const float (&x)[2], bf16x8 (&pw)[2]) __attribute__((always_inline)) {
        const int r = 2 * s;
        floatx2 pf;
        pf[0] = x[0];
        pf[1] = x[1];
        bf16x2 pr = __builtin_convertvector(pf, bf16x2);
        unsigned bits = __builtin_bit_cast(unsigned, pr);
        asm volatile("" : "+v"(bits));
        pr = __builtin_bit_cast(bf16x2, bits);
        pw[r >> 3][r & 7] = pr[0];
        pw[r >> 3][(r & 7) + 1] = pr[1];
    };
    // Sum of a row's weights in a block from that row's lanes alone (rare paths: see sum_weights for the others).
    auto own_sum = [&](const bf16x8 (&pw)[2]) __attribute__((always_inline)) {
        bf16x2 ones;
        ones[0] = (__bf16)1.0f;
        ones[1] = (__bf16)1.0f;
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            bf16x2 pr;
            pr[0] = pw[r >> 3][r & 7];
            pr[1] = pw[r >> 3][(r & 7) + 1];
            sum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, sum, false);
        }
        return halves_sum(sum);
    };
    // Rare side path, uniform over the wavefront: some row of block g produced a weight beyond 2^kTrip
    // (also a row's first block with an allowed key, if that is not the segment's first).  Every row
    // whose block maximum exceeds its reference by more than 2^kBump takes that maximum as its new
    // reference; the block's weights and row sums are recomputed, the running sums and O are scaled.
    // The accumulators live in accumulation registers and are scaled in place there; the waits cover
    // MFMA results still in flight.
    auto renormalise = [&](const floatx16& sc, float& lb, bf16x8 (&pw)[2]) __attribute__((always_inline)) {
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sc[r]);
        const float t = halves_max(tmax) * c;
        const float m_old = rs.m;
        const float m_new = t > m_old + kBump ? t : m_old;
        const float alpha = __builtin_amdgcn_exp2f(m_old - m_new);
        rs.m = m_new;
        rs.l *= alpha;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            floatx2 pf;
            pf[0] = __builtin_amdgcn_exp2f(fmaf(sc[r], c, -m_new));
            pf[1] = __builtin_amdgcn_exp2f(fmaf(sc[r + 1], c, -m_new));
            const bf16x2 pr = __builtin_convertvector(pf, bf16x2);
            pw[r >> 3][r & 7] = pr[0];
            pw[r >> 3][(r & 7) + 1] = pr[1];
        }
        lb = own_sum(pw);
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float e = o[db][r], t;
                asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                             : "+a"(e), "=&v"(t) : "v"(alpha));
                o[db][r] = e;
            }
        asm volatile("s_nop 7" ::: "memory");
    };
    // ---- O^T += V^T P^T: k-slot e of a lane is key 32*jb + 16*tt + 4*half + (e<4 ? e : e+4)
    // ---- operand fetches from LDS
    auto k_operand = [&](const __bf16* kst, int ks) { return *(const bf16x8*)(kst + koff[ks]); };
    auto v_operand = [&](const __bf16* vst, int i) {          // operand i = 2*db + tt
        const __bf16* vp = vst + 16 * (i & 1) * D + voff[i >> 1];
        const bf16x4 v0 = lds_read_tr16(vp);
        const bf16x4 v1 = lds_read_tr16(vp + 8 * D);
        return (bf16x8)__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    // ---- prologue: tiles 0 and 1 into the ring, S^T of block (tile 0, jb 0)
    dma_wait_all();     // the segment's first tiles and query rows, requested ahead of time
    // The assembly MFMAs read Q from accumulation registers.  If the compiler holds the loaded rows in
    // ordinary registers, this is where it has to move them over: a vector write needs two wait states
    // before a matrix instruction reads it, and only here are those guaranteed.
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[ks]));
    asm volatile("s_nop 1" ::: "memory");
    __syncthreads();

    // The pipeline advances by 32-key blocks g = 2*tile + jb.  One half-step for block g is one basic
    // block of 8 slots; slot s issues
    //     MFMA s of S^T of block g+1   | two pieces of the softmax of block g |   MFMA s of P V of block g-1
    // so that consecutive MFMAs never depend on each other and every MFMA has a few VALU
    // instructions behind it.  LDS operands are fetched three operands ahead, across half-step
    // boundaries.  Two rare side blocks follow and modify registers in place: the rescale of O by the
    // factors the softmax just produced (after P V of block g-1, before P V of block g) and the
    // element mask of the scores of block g+1.  In the last iteration block g+1 is a reload of the
    // last tile whose scores are never used.
    constexpr int NOP = D / 16;             // MFMAs, and LDS operands, per stream and half-step: 8 at D=128, 4 at D=64
    constexpr int NSLOT = 8;                // slots per half-step: one per pair of scores of a lane
    constexpr int AHEAD = 3;                // operands in flight per stream
    // head_dim 64 has half as many MFMAs as slots would take: S^T in the first four slots, P V in the last four (both in the
    // first four: 7 % more clocks), and a pair of weights is converted one slot after its exponentials, whose result the
    // conversion may not read in the very next instruction (at head_dim 128 the same costs 2 %: the MFMAs set the pace there and a
    // slot gets longer by the conversion).  With both SD3-like 1K 141.9 -> 139.3 us, 2K 1426 -> 1406, 512 px refresh 85.2 -> 84.1.
    constexpr int PV0 = NSLOT - NOP;        // slot of the first P V MFMA
    constexpr int kLag = D == 64 ? 1 : 0;
    static_assert(NOP == 8 || NOP == 4, "slot layout assumes head_dim 128 or 64");
    floatx16 s0, s1;                        // scores of the even / odd block in flight
    bf16x8 pa[2], pb[2];                    // weights of the even / odd block in flight
    bf16x8 kq[NOP], vq[NOP];                // LDS operands (entry j = operand j of the stream)

    // Row sums of a block's weights (the rounded ones, which are what P V multiplies), by the matrix core: two 16x16x32
    // products beside the 16 (head_dim 64: 8) of S^T and P V.  v_dot2_f32_bf16, which adds a pair in one vector instruction, runs in
    // the matrix pipe and stalls it: an MFMA with one of them behind it takes 49 clocks of its SIMD where four v_fma cost one
    // (33 instead of 32), and the softmax's mix per MFMA 40.5 with it, 34.5 with the two products, 33.2 with no sum at all
    // (head_dim 64: 52.0, 42.1, 38.3).  2K all-full layer 2955 -> 2839 us (2977 -> 2917 where every pass has
    // other inputs), video-like 1349 -> 1270 (1353 -> 1307), mixed 1021 -> 969, FLUX-like 1K 127.8 -> 122.0 (130.0 -> 126.3);
    // head_dim 64 within 0.5 %.  (v_add on the unrounded weights costs the same and is less exact: 2.0e-3 of
    // the result's norm off instead of 1.75e-3 where few keys carry a row.)
    floatx4 wsum;
    auto sum_weights = [&](int tt, const bf16x8 (&pw)[2]) __attribute__((always_inline)) {
        wsum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row_ones, pw[tt], tt ? wsum : floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    };
    // Closes a block: its row sums are checked (see renormalise) and added to the rows' running sums.
    auto settle = [&](const floatx16& sc, bf16x8 (&pw)[2], bool first) __attribute__((always_inline)) {
        float lb = wsum[0];
        pin(lb);                            // (read here, whatever follows)
        // compared as integers: a row beside one with an infinite weight has the sum NaN (0 x inf), which has to count as large
        const bool large = __builtin_amdgcn_ballot_w64(__builtin_bit_cast(unsigned, lb) > __builtin_bit_cast(unsigned, kTrip)) != 0;
        // In a segment's first block the references are the block's own maxima: the weights are 1 at most (but for what is lost of a
        // reference of 2^24 and more), or not numbers, which stay with their own row.
        if (first) {
            if (__builtin_expect(large, 0)) lb = own_sum(pw);
            rs.l = lb;
            return;
        }
        if (__builtin_expect(large, 0)) renormalise(sc, lb, pw);
        rs.l += lb;
    };
    auto half_step = [&](const floatx16& s_cur, floatx16& s_nxt, const bf16x8 (&p_prev)[2],
                         bf16x8 (&p_cur)[2], const __bf16* kst_nxt, const __bf16* kst_after,
                         const __bf16* vst_prev, const __bf16* vst_cur, bool with_pv, bool mask_nxt,
                         int blk_nxt, int dma_tensor, unsigned dma_tb, unsigned dma_dst,
                         unsigned dma_tb2 = 0, unsigned dma_dst2 = 0) __attribute__((always_inline)) {
        const float mneg = -rs.m;
        float xs[2][2];
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) {
            const int jn = s + AHEAD;              // operand jn is fetched while operand s is used
            float (&x)[2] = xs[s & 1];
            if (s < NOP) {
                if (s == 0) mfma_s_first(s_nxt, kq[s], qf[s]);
                else mfma_s_acc(s_nxt, kq[s], qf[s]);
                if (jn < NOP) kq[jn] = k_operand(kst_nxt, jn);
                else kq[jn - NOP] = k_operand(kst_after, jn - NOP);
            }
            softmax_a(s, s_cur, mneg, x);
            __builtin_amdgcn_sched_barrier(0);
            if (s >= PV0) {
                const int i = s - PV0, in = i + AHEAD;
                if (with_pv)
                    o[i >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vq[i], p_prev[i & 1], o[i >> 1], 0, 0, 0);
                if (in < NOP) { if (with_pv) vq[in] = v_operand(vst_prev, in); }
                else vq[in - NOP] = v_operand(vst_cur, in - NOP);
            }
            x[1] = __builtin_amdgcn_exp2f(x[1]);
            pin(x[1]);
            if (s >= kLag) convert(s - kLag, xs[(s - kLag) & 1], p_cur);
            if (s == 5 + kLag) sum_weights(0, p_cur);
            if (kLag && s == NSLOT - 1) convert(s, x, p_cur);
            if (s == NSLOT - 1) sum_weights(1, p_cur);
            // the loads of a later tile are spread over the slots (a burst of them right after the
            // barrier stalls all wavefronts on the one memory pipe)
            if ((s & 3) == 1 && (s >> 2) < NDMA) dma_part(dma_tensor, s >> 2, dma_tb, dma_dst);
            if (BLK && (s & 3) == 3 && (s >> 2) < NDMA) dma_part(1, s >> 2, dma_tb2, dma_dst2);
            __builtin_amdgcn_sched_barrier(0);
        }
        settle(s_cur, p_cur, !with_pv);
        // block number blk_nxt = 2*position + jb; its first key is only needed on this rare path.  (settle() has read the row sums,
        // which the matrix pipe makes after the last S^T MFMA: the scores are there.  Another 32 wait states here, scalar
        // decisions about each edge of the band and a branch for each cost the SD3-like 512 px refresh 85.5 us instead of 82,
        // the 1K layer 138.3 instead of 134.5.)
        if (__builtin_expect(mask_nxt, 0)) {
            settled_results(s_nxt);
            mask_block(tile_of(blk_nxt >> 1) * kBN + 32 * (blk_nxt & 1), s_nxt);
        }
    };

    // (requested here, and waited for before the key loop: the compiler takes the record to scalar registers as soon as it can)
    seg_next = a.segs[seg_idx + 1 < seg_end ? seg_idx + 1 : seg_idx];
    qk_block(0, 0, s0);
    if (tile_masked(0)) mask_block(tile_of(0) * kBN, s0);   // (before the loop-carried flags exist)
    // The rows' references: the maximum of the first block (a row that sees nothing of it keeps the initial one).  Left to
    // renormalise(), which finds it only after the block's weights have come out infinite, every segment paid for a second
    // set of weights: SD3-like 1K layer 141.8 us against 140.5, 2K 1457 / 1447, FLUX-like 2K mixed 981 / 974.
    {
        float top = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) top = fmaxf(top, s0[r]);
        rs.m = fmaxf(rs.m, halves_max(top) * c);
    }

    if constexpr (BLK) __syncthreads();     // block 0 has been read by everyone: its stage takes block 4
    // Loop-carried scalars (all uniform over the wavefront), advanced once per iteration instead of
    // being recomputed from the position: ring stages of the tiles in use, mask flags, load target.
    // A wavefront issues in order and scalar work delays its next MFMA, so there is as little of it as possible.
    const int m0e = (it.nm0_end < it.kv0_end ? it.nm0_end : it.kv0_end) - it.pos_begin;   // idx in [.., m0e) and
    const int m1b = it.kv0_end + (it.nm1_begin > it.kv1_begin ? it.nm1_begin - it.kv1_begin : 0) - it.pos_begin;
    const int m1e = it.kv0_end + ((it.nm1_end < it.kv1_end ? it.nm1_end : it.kv1_end) - it.kv1_begin) - it.pos_begin;
    auto pos_masked = [&](int idx) { return !(idx < m0e || (idx >= m1b && idx < m1e)); };   // [m1b, m1e) are mask-free
    auto kptr = [&](int off, int jb) { return &Ksm[off + 32 * jb * D]; };
    auto vptr = [&](int off, int jb) { return &Vsm[off + 32 * jb * D]; };
    const unsigned half_tile = tile_bytes / 2;
    auto stage = [&](int blk) { return ((sbase + blk) & 3) * TILE; };                       // (BLK)
    auto dst = [&](unsigned base, int off) { return base + (unsigned)(off * 2) + wave_lds; };
    // ring stages as element offsets: K stages of positions idx, idx+1, idx+3, V stages of idx-1, idx, idx+2
    int k_cur = (sbase & 3) * TILE, k_nxt = ((sbase + 1) & 3) * TILE, k_ld = ((sbase + 3) & 3) * TILE;
    int v_cur = k_cur, v_ld = ((sbase + 2) & 3) * TILE;
    bool msk_cur = pos_masked(0), msk_nxt = pos_masked(1);
    unsigned tb_k = tile_offset(BLK ? 2 : 3), tb_v = tile_offset(BLK ? 1 : 2);  // tiles whose K / V loads the coming iteration issues

    // first tile: its even block has no predecessor whose P V would be due
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) kq[j] = k_operand(BLK ? kptr(stage(1), 0) : kptr(k_cur, 1), j);
    if constexpr (BLK) {
        half_step(s0, s1, pb, pa, kptr(stage(1), 0), kptr(stage(2), 0), vptr(stage(0), 0), vptr(stage(0), 0), false, msk_cur, 1,
                  0, tb_k, dst(k_lds, stage(4)), tb_v, dst(v_lds, stage(2)));
        mfma_results_visible(s1);
        __syncthreads();
        half_step(s1, s0, pa, pb, kptr(stage(2), 0), kptr(stage(3), 0), vptr(stage(0), 0), vptr(stage(1), 0), true, msk_nxt, 2,
                  0, tb_k + half_tile, dst(k_lds, stage(5)), tb_v + half_tile, dst(v_lds, stage(3)));
    } else {
    half_step(s0, s1, pb, pa, kptr(k_cur, 1), kptr(k_nxt, 0), vptr(v_cur, 0), vptr(v_cur, 0), false,
              msk_cur, 1, 0, tb_k, k_lds + (unsigned)(k_ld * 2) + wave_lds);
    mfma_results_visible(s1);  // no P V MFMA separated this block's last S^T MFMA from its first reader
    half_step(s1, s0, pa, pb, kptr(k_nxt, 0), kptr(k_nxt, 1), vptr(v_cur, 0), vptr(v_cur, 1), true,
              msk_nxt, 2, 1, tb_v, v_lds + (unsigned)(v_ld * 2) + wave_lds);
    }
    dma_wait_older();

    // With half-tile stages (BLK) half-step g reads K blocks g+1 and g+2 and V blocks g-1 and g, and issues the loads of
    // K block g+4 into the stage of block g and of V block g+2 into that of block g-2, both read for the last time before
    // the barrier it begins with; they are waited for at the end of half-step g+1, before the barrier of g+2.  A tile
    // moves the ring by two stages, so there are two copies of the loop body.
    // Otherwise: iteration idx works on tiles idx-1 (P V), idx and idx+1 (S^T), issues the loads of K tile idx+3 and
    // V tile idx+2 and, before the next barrier, waits for the loads issued one iteration earlier
    // (K tile idx+2, V tile idx+1).  K tile p is last read in the first half of iteration p, V tile p in
    // the first half of iteration p+1, so both rings are four stages deep.
    // The loop body exists four times, once per ring stage the current tile can sit in: with the stage a
    // compile-time constant the ring offsets become immediate operands of the LDS reads, which saves the
    // two dozen address additions a tile costs when the stage is a run-time value, and the stage
    // bookkeeping itself.  The loop is entered at the copy the segment's second tile needs.
    auto iteration = [&](auto stage_c, int idx) __attribute__((always_inline)) {
        constexpr int P = decltype(stage_c)::value;         // ring stage of tile idx
        constexpr int KC = P * TILE, KN = ((P + 1) & 3) * TILE, KL = ((P + 3) & 3) * TILE;
        constexpr int VP = ((P + 3) & 3) * TILE, VC = P * TILE, VL = ((P + 2) & 3) * TILE;
        if (wgs_per_cu(BM) > 1 && (P & 1) == 0 && younger) __builtin_amdgcn_s_setprio(P == 0 ? 1 : 0);
        msk_cur = msk_nxt;
        msk_nxt = pos_masked(idx + 1);
        tb_v = tb_k;
        tb_k = tile_offset(idx + (BLK ? 2 : 3));
        __syncthreads();    // the tiles waited for last are in LDS for everyone; the stages loaded next are no longer read
        if constexpr (BLK) {
            constexpr int S0 = P * TILE, S1 = (P + 1) * TILE, S2 = ((P + 2) & 3) * TILE, S3 = ((P + 3) & 3) * TILE;   // blocks 2 * idx ..
            half_step(s0, s1, pb, pa, kptr(S1, 0), kptr(S2, 0), vptr(S3, 0), vptr(S0, 0), true, msk_cur, 2 * idx + 1,
                      0, tb_k, dst(k_lds, S0), tb_v, dst(v_lds, S2));
            dma_wait_older();
            __syncthreads();
            half_step(s1, s0, pa, pb, kptr(S2, 0), kptr(S3, 0), vptr(S0, 0), vptr(S1, 0), true, msk_nxt, 2 * idx + 2,
                      0, tb_k + half_tile, dst(k_lds, S1), tb_v + half_tile, dst(v_lds, S3));
            dma_wait_older();
            return;
        }
        half_step(s0, s1, pb, pa, kptr(KC, 1), kptr(KN, 0), vptr(VP, 1), vptr(VC, 0), true,
                  msk_cur, 2 * idx + 1, 0, tb_k, k_lds + (unsigned)(KL * 2) + wave_lds);
        half_step(s1, s0, pa, pb, kptr(KN, 0), kptr(KN, 1), vptr(VC, 0), vptr(VC, 1), true,
                  msk_nxt, 2 * idx + 2, 1, tb_v, v_lds + (unsigned)(VL * 2) + wave_lds);
        dma_wait_older();
    };
    {
        int idx = 1;
        int phase = (sbase + 1) & 3;
        if constexpr (BLK) {                // a tile takes two stages: two copies
            phase = (sbase + 2) & 3;
            while (idx < n_iter) {
                if (phase == 0) {
                    iteration(std::integral_constant<int, 0>(), idx);
                    if (++idx >= n_iter) break;
                }
                iteration(std::integral_constant<int, 2>(), idx);
                ++idx;
                phase = 0;
            }
        } else
        while (idx < n_iter) {
            switch (phase) {
                case 0:
                    iteration(std::integral_constant<int, 0>(), idx);
                    if (++idx >= n_iter) break;
                    [[fallthrough]];
                case 1:
                    iteration(std::integral_constant<int, 1>(), idx);
                    if (++idx >= n_iter) break;
                    [[fallthrough]];
                case 2:
                    iteration(std::integral_constant<int, 2>(), idx);
                    if (++idx >= n_iter) break;
                    [[fallthrough]];
                default:
                    iteration(std::integral_constant<int, 3>(), idx);
                    ++idx;
            }
            phase = 0;
        }
        v_cur = BLK ? stage(2 * n_iter - 1) : ((sbase + n_iter - 1) & 3) * TILE;          // stage of the last tile, for its second block's P V
    }
    // The key loop is over: the K stages and all V stages but the last tile's are free.  Loads past the
    // segment's end may still be depositing zeros, and other wavefronts may still be reading: wait for
    // both, then request what the next segment needs first, so that it arrives during the epilogue.
    dma_wait_all();
    __syncthreads();
    const int sbase_next = (sbase + (BLK ? 2 : 1) * n_iter) & 3;            // keeps clear of the stage the last P V still reads
    if (seg_idx + 1 < seg_end && it.part_slot < 0) first_loads(seg_next, sbase_next);   // (a piece: after its slot stores)
    // P V of the very last block (its first operands are already in flight)
    {
        const __bf16* vst = vptr(v_cur, BLK ? 0 : 1);
#pragma unroll
        for (int i = 0; i < NOP; ++i) {
            if (i + AHEAD < NOP) vq[i + AHEAD] = v_operand(vst, i + AHEAD);
            o[i >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vq[i], pb[i & 1], o[i >> 1], 0, 0, 0);
        }
    }

    // ---- epilogue: O^T register r of block db is feature d = 32*db + 8*(r/4) + 4*half + r%4
    float l_fin = rs.l;
    bool writes_rows = it.part_slot < 0;
    if (it.part_slot >= 0) {
        // A piece of a cut record.  Its unnormalised fp32 accumulators, row reference (log2 domain) and row
        // sum go to the piece's scratch slot; then it takes a ticket of the record.  The piece that draws
        // the last ticket folds the other pieces' slots into its own accumulators,
        //     O = sum_p O_p 2^(m_p - M),  l = sum_p l_p 2^(m_p - M),  M = max_p m_p,
        // in the register layout it already holds them in, writes the record's rows like a whole record
        // and puts the ticket counter back to zero for the next launch.
        // The slot stores and loads are device-coherent ("sc1": written through and read around a stale L2
        // line): another piece may run on another accelerator die, with an L2 of its own, and ordinary
        // accesses would need a device-wide release and acquire, i.e. writing back and invalidating a die's
        // whole L2, the K/V tiles its workgroups share included.
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(a.part_o, 0, 0x7fffffff, 0x00020000);
        const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(a.part_ml, 0, 0x7fffffff, 0x00020000);
        auto slot_bytes = [&](int slot) { return (slot * NW + (int)wave_u) * (32 * D * 4); };
        // A slot holds the accumulators in the order of the registers, 1 KiB per wavefront and store: the piece
        // that folds it in has them in the same registers, so no other order is ever needed.
        const int slot_lane = (half * 32 + l32) * 16;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                floatx4 w4;
#pragma unroll
                for (int e = 0; e < 4; ++e) w4[e] = o[db][4 * g + e];
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, w4), ro, slot_lane + 1024 * (4 * db + g),
                                                       slot_bytes(it.part_slot), kDeviceCoherent);
            }
        if (half == 0) {
            floatx2 ml;
            ml[0] = rs.m;
            ml[1] = l_fin;
            const int rl = it.part_slot * BM + wave * RW + l32;       // row inside the scratch
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, ml), rm, rl * 8, 0, kDeviceCoherent);
        }
        // The slot has to be written before the ticket is taken.  The next segment's query rows and first
        // tiles are requested behind the slot stores, and the tiles are not waited for: memory operations
        // complete in the order they were issued, so "all but the youngest kFirstTileLoads" covers the
        // stores.  (The empty statements keep the compiler from moving a memory operation across them, so
        // that no store is issued among the tile loads; anything it adds there only makes the wait stricter.)
        if (seg_idx + 1 < seg_end) {
            asm volatile("" ::: "memory");
            query_rows(seg_next);
            asm volatile("" ::: "memory");
            first_tiles(seg_next, sbase_next);
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kFirstTileLoads) : "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();                                     // ... by every wavefront
        if (tid == 0) ctl_sm[0] = atomicAdd(cold_args()->tickets + it.merge_idx, 1);
        __syncthreads();
        if (ctl_sm[0] == it.n_parts - 1) {
#pragma unroll 1
            for (int p = 0; p < it.n_parts; ++p) {
                const int slot = it.first_slot + p;
                if (slot == it.part_slot) continue;
                const int rl = slot * BM + wave * RW + l32;
                // (whole vectors are reinterpreted: a bit_cast applied to one vector element reads element 0)
                const floatx2 ml = __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(rm, rl * 8, 0, kDeviceCoherent));
                floatx4 x[DB][4];
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        x[db][g] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                            ro, slot_lane + 1024 * (4 * db + g), slot_bytes(slot), kDeviceCoherent));
                const float m_new = fmaxf(rs.m, ml[0]);
                const float w_mine = __builtin_amdgcn_exp2f(rs.m - m_new), w_other = __builtin_amdgcn_exp2f(ml[0] - m_new);
                rs.m = m_new;
                l_fin = fmaf(ml[1], w_other, l_fin * w_mine);
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            o[db][4 * g + e] = fmaf(x[db][g][e], w_other, o[db][4 * g + e] * w_mine);
            }
            if (tid == 0) atomicExch(cold_args()->tickets + it.merge_idx, 0);
            writes_rows = true;
        }
    }
    if (writes_rows) {
        // A lane holds features 8g + 4*half + (0..3) of its row for g = 0..3 in each block db.  The two
        // halves of the wavefront exchange one quad per pair (g, g+1), after which the lower half holds
        // features 8g..8g+7 and the upper half 8(g+1)..8(g+1)+7: 16-byte stores, half as many of them (with
        // the next segment's loads already in flight, more memory instructions than the 63 the counter
        // can track would stall the wavefront until loads return).
        float inv = 1.0f / l_fin;
        const int64_t row_off = (int64_t)(i_raw < N ? i_raw : N - 1) * a.stride_n;
        __bf16* orow = og + row_off;
        if (it.flags & DIFA_ITEM_ADD_RESIDUAL) {
            // arrow attention with residual sharing: the head's kept difference is added to the
            // normalised result before it is rounded (the lane's features: four in a row per (db, g))
            const __bf16* rrow = (const __bf16*)cold_args()->residual + (og - (__bf16*)a.out) + row_off;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const bf16x4 rv = *(const bf16x4*)(rrow + 32 * db + 8 * g + 4 * half);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o[db][4 * g + e] = fmaf(o[db][4 * g + e], inv, (float)rv[e]);
                }
            inv = 1.0f;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int gp = 0; gp < 2; ++gp) {
                unsigned w[2][2];                        // [g - 2*gp][pair of features]
#pragma unroll
                for (int gg = 0; gg < 2; ++gg)
#pragma unroll
                    for (int e2 = 0; e2 < 2; ++e2) {
                        floatx2 f;
                        f[0] = o[db][4 * (2 * gp + gg) + 2 * e2] * inv;
                        f[1] = o[db][4 * (2 * gp + gg) + 2 * e2 + 1] * inv;
                        w[gg][e2] = __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
                    }
                uintx4 q4;
#pragma unroll
                for (int e2 = 0; e2 < 2; ++e2) {
                    // lower half keeps its quad of g and receives the upper half's; the upper half receives
                    // the lower half's quad of g+1 and keeps its own
                    const auto r = __builtin_amdgcn_permlane32_swap(w[0][e2], w[1][e2], false, false);
                    const unsigned first = r[0], second = r[1];
                    q4[e2] = first;
                    q4[2 + e2] = second;
                }
                if (i_raw < N) *(uintx4*)(orow + 32 * db + 16 * gp + 8 * half) = q4;
            }
    }
    sbase = sbase_next;
    // one chunk of the cached-head copy, while the next segment's first tiles are on their way
    if (next_chunk < cold_args()->copy_chunks) {
        copy_chunk(next_chunk);
        next_chunk += (int)gridDim.x;
    }
    }
    // whatever is left of this workgroup's share of the copy (a layer with every head cached goes to cache_copy_kernel instead)
    {
        const int copy_chunks = cold_args()->copy_chunks;
        for (; next_chunk < copy_chunks; next_chunk += (int)gridDim.x) copy_chunk(next_chunk);
    }
    if (tid == 0) {
        const AttnArgs* ca = cold_args();
        if (ca->wg_times) {
            // (read through a pointer the compiler cannot trace back to the store, or it would carry the value
            // in registers from one end of the kernel to the other)
            const int* ts = ctl_sm;
            asm volatile("" : "+v"(ts));
            const unsigned long long t0 = (unsigned long long)(unsigned)ts[2] | ((unsigned long long)(unsigned)ts[3] << 32);
            const unsigned long long ran = seg_first < seg_end ? wall_clock64() - t0 : 0;   // (no segments: no start time)
            ca->wg_times[blockIdx.x] = ((unsigned long long)ca->launch_tag << 32) | (ran < 0xffffffffull ? ran : 0xffffffffull);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Scratch of difa_joint_attention_static, the entry point for callers that must not allocate: the
// partial results of cut records (what part_o / part_ml point at) live in this file-scope array
// instead of a buffer the plan object allocated.  512 pieces of 256 rows, or 1024 of 128, at head_dim 128:
// 512 * 256 * (128 + 2) floats = 68 157 440 bytes, held by every GPU the library runs on until the
// process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the device
// address is looked up once per device and is what the kernels receive as an argument.
// ------------------------------------------------------------------------------------------
constexpr size_t kStaticScratchFloats = (size_t)512 * kBM * (128 + 2);
static __device__ __align__(256) float scratch[kStaticScratchFloats];
constexpr int kMaxDevices = 64;
static float* g_scratch_ptr[kMaxDevices];      // device address of `scratch` per device ordinal
static std::mutex g_scratch_mutex;

hipError_t static_scratch_init(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return hipSuccess;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));   // of the current device's copy
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = (float*)ptr;
    return hipSuccess;
}

float* static_scratch(int device, size_t* bytes) {
    if (bytes) *bytes = kStaticScratchFloats * sizeof(float);
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[device];
}

hipError_t launch_attn_bf16(const AttnArgs& a, int head_dim, int rows, int n_wg, hipStream_t stream) {
    if (n_wg <= 0) return hipSuccess;
    const dim3 grid(n_wg), threads(2 * rows);
    if (head_dim == 128 && rows == kRowsLong) hipLaunchKernelGGL((attn_bf16_kernel<128, kRowsLong>), grid, threads, 0, stream, a);
    else if (head_dim == 128 && rows == kRowsShort) hipLaunchKernelGGL((attn_bf16_kernel<128, kRowsShort>), grid, threads, 0, stream, a);
    else if (head_dim == 64 && rows == kRowsShort) hipLaunchKernelGGL((attn_bf16_kernel<64, kRowsShort>), grid, threads, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// fp32 debug path.  Scores, weighted sums and row sums in fp64 on the matrix cores (v_mfma_f64_16x16x4_f64: products of
// fp32 data are exact there), weights by the fp32 exponential: with logits of magnitude ~10 an fp32 dot product alone
// costs a few 1e-6 in every weight, which is the whole error budget of this path.  It shares only the work record's
// (batch, head, query tile) with the fast path.
//
// Bound by the fp64 matrix rate (72 TFLOP/s on MI355X, one of these MFMAs per SIMD every 64 clocks) and by the vector
// instructions, none of which runs beside it; the loads come straight from L2.  A workgroup is eight wavefronts on one block
// of 16 query rows, each taking every eighth tile of 16 keys (so that a layer of a few heads still fills the chip), combined through LDS at
// the end.  As in the fast path scores are computed transposed, S^T = K Q^T: the accumulator layout (lane: query
// l % 16, register i: key 4 * i + l / 16) is then the B operand layout of O^T = V^T P^T.  Which four features make up a
// contraction step, and which feature a row of O^T is, is free as long as both operands agree; they are chosen so that a
// lane's part of a K, V or output row is contiguous.
// Measured on MI355X, 5 computed heads of 64 and 1101 tokens, a cached head copied by the same launch: 31.2 us, 34.7 with 270
// instead of 60 vector instructions a tile beside its 32 MFMAs (addresses, masks and maxima of every tile, a library
// exponential, conversions one by one); 12 at the fp64 matrix rate alone: 153 of the 345 blocks see every key, and 60 % of the
// compute units carry them.  6.7 ms with one wavefront per row, scalar dot products and two passes over the
// keys.  Weighted sums on the fp32 matrix rate instead: 36 us against 34, and a larger error (1.0e-7 of the
// result's norm against 64 bits; 3.0e-8 as it is, 8.7e-8 with scalar sums).
// ------------------------------------------------------------------------------------------
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int kF32Rows = kF32BlockRows, kF32Keys = 16, kF32Waves = 8;

// WIDE: 16 token rows span 2 GiB or more (hundreds of thousands of heads in [token, head, feature] order).
template <int D, bool WIDE>
__global__ __launch_bounds__(64 * kF32Waves, D == 64 ? 4 : 2) void attn_f32_kernel(AttnArgs a) {
    constexpr int KF = D / 4;                                // features of a K or Q row per lane
    constexpr int VF = D / 16;                               // features of a V or output row per lane = 16-row blocks of O^T
    const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= (unsigned)a.f32_blocks) {                   // the blocks behind the computed heads' copy the cached heads
        const unsigned chunk = block - (unsigned)a.f32_blocks;
        if (chunk < (unsigned)a.copy_chunks) copy_vectors<64 * kF32Waves>(a, (int)chunk, (int)threadIdx.x);
        return;
    }
    const difa_work_item_t it = a.items[block / (kBM / kF32Rows)];
    if (it.q_tile < 0) return;
    const int N = a.n_tokens, n_text = a.n_text;
    const int i0 = it.q_tile * kBM + (int)(block % (kBM / kF32Rows)) * kF32Rows;
    if (i0 >= N) return;                                     // (uniform over the workgroup)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c16 = lane & 15, g = lane >> 4;
    const int b = it.bh / a.heads, h = it.bh - b * a.heads;
    const int64_t base = (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
    const float* __restrict__ qg = (const float*)a.q + base;
    const float* __restrict__ kg = (const float*)a.k + base;
    const float* __restrict__ vg = (const float*)a.v + base;

    // Keys the block visits, as two ranges [begin0, end0) and [begin1, end1): everything, or the text keys and the part of
    // the image that some row of the block sees.
    const int tb = a.text_begin, img0 = tb == 0 ? n_text : 0, img1 = tb == 0 ? N : tb;
    const int i_last = i0 + kF32Rows - 1 < N - 1 ? i0 + kF32Rows - 1 : N - 1;
    const bool banded = it.window >= 0;
    int begin0 = 0, end0 = N, begin1 = 0, end1 = 0;
    if (banded && i0 >= img0 && i_last < img1) {
        begin0 = tb;
        end0 = tb + n_text;
        begin1 = i0 - it.window > img0 ? i0 - it.window : img0;
        end1 = (i_last < img1 - 1 - it.window ? i_last + it.window : img1 - 1) + 1;
    }
    const int tiles0 = (end0 - begin0 + kF32Keys - 1) / kF32Keys, tiles = tiles0 + (end1 - begin1 + kF32Keys - 1) / kF32Keys;

    // this lane's query: column c16 of S^T and O^T
    const int i = i0 + c16 < N ? i0 + c16 : N - 1;
    const bool text_row = !banded || (unsigned)(i - tb) < (unsigned)n_text;
    const int lo = i - it.window, hi = i < N - 1 - it.window ? i + it.window : N - 1;
    // The block's query rows in fp64, in the order the contraction reads them: held in registers they would leave room for
    // one workgroup on a compute unit at head_dim 64 instead of two.
    __shared__ double q_sm[KF][64];
    if (wave == 0) {
#pragma unroll
        for (int s = 0; s < KF; s += 4) {
            const floatx4 t4 = *(const floatx4*)(qg + (int64_t)i * a.stride_n + 4 * s + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) q_sm[s + e][lane] = (double)t4[e];
        }
    }
    __syncthreads();

    doublex4 o[VF];
#pragma unroll
    for (int f = 0; f < VF; ++f) o[f] = doublex4{0.0, 0.0, 0.0, 0.0};
    double l = 0.0, m = -1.0e30;                             // m: reference in the log2 domain, an integer: rescaling is exact
    const double c = (double)a.scale * 1.44269504088896340736;
    const float c32 = (float)c;

    // Step 4 * s + e of the contraction takes features 16 * s + 4 * g + e, so that the four lanes of a key row read 64
    // bytes of it together.  The next tile's K rows are requested when this one's are converted, its V rows after the
    // last use of this one's: each has the other contraction's time to arrive.  (The last tile is requested again past the
    // end: behind a branch the compiler would have to wait for the younger loads too.)  A lane's place in a tile does not change;
    // where the tile lies is a buffer descriptor of its own, which ends with the sequence: rows past that read as zero.
    floatx4 kc[KF / 4], vc[4][VF / 4];
    const int row_bytes = WIDE ? 0 : (int)a.stride_n * 4;
    const int at_k = c16 * row_bytes + 16 * g;
    int at_v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) at_v[u] = (4 * u + g) * row_bytes + 4 * VF * c16;
    auto first_key = [&](int t_any) {
        const int t = t_any < tiles ? t_any : tiles - 1;
        return t < tiles0 ? begin0 + t * kF32Keys : begin1 + (t - tiles0) * kF32Keys;
    };
    auto tile_rows = [&](const float* head, int t) {
        const int j0 = first_key(t), rows = N - j0 < kF32Keys ? N - j0 : kF32Keys;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(head + (int64_t)j0 * a.stride_n), 0, (rows - 1) * row_bytes + 4 * D, 0x00020000);
    };
    auto fetch_k = [&](int t) {
        if constexpr (WIDE) {
            const int j = first_key(t) + c16;
            const float* kr = kg + (int64_t)(j < N ? j : N - 1) * a.stride_n + 4 * g;
#pragma unroll
            for (int s = 0; s < KF / 4; ++s) kc[s] = *(const floatx4*)(kr + 16 * s);
            return;
        }
        const __amdgpu_buffer_rsrc_t r = tile_rows(kg, t);
#pragma unroll
        for (int s = 0; s < KF / 4; ++s) kc[s] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, at_k + 64 * s, 0, 0));
    };
    auto fetch_v = [&](int t) {
        if constexpr (WIDE) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = first_key(t) + 4 * u + g;
                const float* vr = vg + (int64_t)(j < N ? j : N - 1) * a.stride_n + c16 * VF;
#pragma unroll
                for (int s = 0; s < VF / 4; ++s) vc[u][s] = *(const floatx4*)(vr + 4 * s);
            }
            return;
        }
        const __amdgpu_buffer_rsrc_t r = tile_rows(vg, t);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int s = 0; s < VF / 4; ++s) vc[u][s] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, at_v[u] + 16 * s, 0, 0));
    };
    // An fp64 MFMA and every vector instruction of the SIMD exclude each other, and changing over costs 12 clocks besides (one
    // MFMA 64 clocks, with one conversion behind it 77, with two 80, with eight plain integer instructions 86): as few vector
    // instructions as possible, and conversions in groups, not one before each MFMA.
    constexpr int kGroup = 8;
    auto convert = [](const floatx4 (&x)[2], double (&y)[kGroup]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kGroup; ++i) y[i] = (double)x[i >> 2][i & 3];
#pragma unroll
        for (int i = 0; i < kGroup; ++i) asm volatile("" : "+v"(y[i]));
        __builtin_amdgcn_sched_barrier(0);
    };
    const bool split = banded && i0 >= img0 && i_last < img1;   // text keys and band as two ranges
    fetch_k(wave);
    fetch_v(wave);
    for (int t = wave; t < tiles; t += kF32Waves) {
        const int j0 = first_key(t), j_end = t < tiles0 ? end0 : end1;
        asm volatile("" ::: "memory");                       // (or the compiler reads the query rows once and holds them after all)
        doublex4 s2[2] = {doublex4{0.0, 0.0, 0.0, 0.0}, doublex4{0.0, 0.0, 0.0, 0.0}};   // two chains: neither waits for itself
#pragma unroll
        for (int h8 = 0; h8 < KF / kGroup; ++h8) {
            const floatx4 kx[2] = {kc[2 * h8], kc[2 * h8 + 1]};
            double kd[kGroup];
            convert(kx, kd);
            if (h8 == KF / kGroup - 1) fetch_k(t + kF32Waves);
#pragma unroll
            for (int e = 0; e < kGroup; ++e)
                s2[e & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(kd[e], q_sm[kGroup * h8 + e][lane], s2[e & 1], 0, 0, 0);
        }
        doublex4 sc = s2[0] + s2[1];
        // Does every row of the block see every key of the tile?  (the same for the whole wavefront; most tiles)
        const bool every_pair = j0 + kF32Keys <= j_end &&
                                (!banded || (split && (t < tiles0 || (j0 >= i_last - it.window && j0 + kF32Keys - 1 <= i0 + it.window))));
        if (!every_pair) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + 4 * u + g;
                const bool ok = (j < j_end) & (text_row | ((unsigned)(j - tb) < (unsigned)n_text) | ((j >= lo) & (j <= hi)));
                sc[u] = ok ? sc[u] : -INFINITY;
            }
        }
        // The reference is the maximum so far, rounded up to a whole power of two (which one exactly does not matter: moving it
        // is exact).  Only where some row has outgrown it do the four lanes of a row exchange their maxima.
        const float top = fmaxf(fmaxf((float)sc[0], (float)sc[1]), fmaxf((float)sc[2], (float)sc[3])) * c32;
        if (__builtin_amdgcn_ballot_w64((double)top > m) != 0) {
            float row_top = fmaxf(top, __shfl_xor(top, 16, 64));
            row_top = fmaxf(row_top, __shfl_xor(row_top, 32, 64));
            const double m_new = fmax(m, ceil((double)row_top));
            const double alpha = m < -1.0e29 ? 0.0 : ldexp(1.0, (int)fmax(m - m_new, -2000.0));
            l *= alpha;
#pragma unroll
            for (int f = 0; f < VF; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[f][e] *= alpha;
            m = m_new;
        }
        double p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            p[u] = (double)__builtin_amdgcn_exp2f((float)fma(sc[u], c, -m));
            l += p[u];
        }
#pragma unroll
        for (int h8 = 0; h8 < 4 * VF / kGroup; ++h8) {
            const floatx4* vx = &vc[0][0] + 2 * h8;
            const floatx4 v2[2] = {vx[0], vx[1]};
            double vd[kGroup];
            convert(v2, vd);
            if (h8 == 4 * VF / kGroup - 1) fetch_v(t + kF32Waves);
#pragma unroll
            for (int e = 0; e < kGroup; ++e) {
                const int u = (kGroup * h8 + e) / VF, f = (kGroup * h8 + e) % VF;
                o[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(vd[e], p[u], o[f], 0, 0, 0);
            }
        }
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);

    // ---- the eight wavefronts' parts are added pairwise, upper half into lower half
    __shared__ double part[kF32Waves / 2][4 * VF + 2][64];
#pragma unroll
    for (int n = kF32Waves / 2; n >= 1; n /= 2) {
        __syncthreads();
        if (wave >= n && wave < 2 * n) {
            double (*mine)[64] = part[wave - n];
            mine[4 * VF][lane] = m;
            mine[4 * VF + 1][lane] = l;
#pragma unroll
            for (int f = 0; f < VF; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) mine[4 * f + e][lane] = o[f][e];
        }
        __syncthreads();
        if (wave < n) {
            double (*other)[64] = part[wave];
            const double mo = other[4 * VF][lane], m_new = fmax(m, mo);
            const double wm = m < -1.0e29 ? 0.0 : ldexp(1.0, (int)fmax(m - m_new, -2000.0));
            const double wo = mo < -1.0e29 ? 0.0 : ldexp(1.0, (int)fmax(mo - m_new, -2000.0));
            m = m_new;
            l = l * wm + other[4 * VF + 1][lane] * wo;
#pragma unroll
            for (int f = 0; f < VF; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[f][e] = o[f][e] * wm + other[4 * f + e][lane] * wo;
        }
    }
    if (wave != 0) return;
    const double inv = 1.0 / l;
    double all = l;                                          // not finite if any part of it is
#pragma unroll
    for (int f = 0; f < VF; ++f)
#pragma unroll
        for (int e = 0; e < 4; ++e) all += o[f][e];
    unsigned high = (unsigned)(__builtin_bit_cast(unsigned long long, all) >> 32);
    asm volatile("" : "+v"(high));                           // (the file is compiled on the assumption that there are no NaNs)
    const bool finite = (high >> 20 & 0x7ff) != 0x7ff;
    // The rows whose reference lies outside +-2^24 or whose result is not finite (see below) as a bit mask, the same in
    // every lane.
    unsigned long long exact_rows = __builtin_amdgcn_ballot_w64(!(m > -0x1p24 && m < 0x1p24) || !finite);
    exact_rows = (exact_rows | exact_rows >> 16 | exact_rows >> 32 | exact_rows >> 48) & 0xffff;
    if (i0 + c16 < N && !(exact_rows >> c16 & 1)) {
        // register e of o[f] is feature (4 * e + g) * VF + f of the lane's query
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t at = base + (int64_t)i * a.stride_n + (4 * e + g) * VF;
#pragma unroll
            for (int s = 0; s < VF / 4; ++s) {
                floatx4 w;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    double y = o[4 * s + k][e] * inv;
                    if (it.flags & DIFA_ITEM_ADD_RESIDUAL) y += (double)((const float*)a.residual)[at + 4 * s + k];   // + kept difference
                    w[k] = (float)y;
                }
                *(floatx4*)((float*)a.out + at + 4 * s) = w;
            }
        }
    }
    // The loop above compares maxima in fp32 and scales a score to the log2 domain in one fp64 product: right to 4e-9 of a
    // weight while the largest scaled score is below 2^24, wrong by more with every power of two beyond (from about 2^32 on
    // the weights overflow or all vanish).  Nothing limits the magnitude of the inputs, so those rows are computed once more
    // here, by one wavefront, as the operator is defined: maximum of the fp64 scores, weights from exact differences to it.
    // And the matrix products multiply every key of a visited tile into every row, the forbidden ones with weight 0, which is
    // not enough against an infinity or a NaN in V: a row that came out not finite is computed from its allowed keys alone, so
    // that it stays so only if it sees such a value.
    // (As slow as one wavefront per row is; neither logits of 10^7 nor infinities are what a model has in earnest.)
    for (; exact_rows != 0; exact_rows &= exact_rows - 1) {
        const int r = i0 + __builtin_ctzll(exact_rows);
        if (r >= N) break;
        const bool every = !banded || (unsigned)(r - tb) < (unsigned)n_text;
        auto sees = [&](int j) {
            return j < N && (every || (unsigned)(j - tb) < (unsigned)n_text || (j >= r - it.window && j - it.window <= r));
        };
        auto score = [&](int j) {
            const float* qr = qg + (int64_t)r * a.stride_n;
            const float* kr = kg + (int64_t)j * a.stride_n;
            double s = 0.0;
#pragma unroll 1
            for (int d = 0; d < D; d += 4) {
                const floatx4 x = *(const floatx4*)(qr + d), y = *(const floatx4*)(kr + d);
#pragma unroll
                for (int e = 0; e < 4; ++e) s = fma((double)x[e], (double)y[e], s);
            }
            return s;
        };
        double top = -INFINITY;
        for (int j = lane; j < N; j += 64)
            if (sees(j)) top = fmax(top, score(j));
#pragma unroll
        for (int n = 32; n >= 1; n >>= 1) top = fmax(top, __shfl_xor(top, n, 64));
        double sum = 0.0, acc[D / 64] = {};                  // lane: features lane, lane + 64
        for (int j0 = 0; j0 < N; j0 += 64) {
            const bool mine = sees(j0 + lane);
            const double p = mine ? (double)exp2f((float)((score(j0 + lane) - top) * c)) : 0.0;
            sum += p;
            for (unsigned long long keys = __builtin_amdgcn_ballot_w64(mine); keys != 0; keys &= keys - 1) {
                const int u = __builtin_ctzll(keys);
                const double pu = __shfl(p, u, 64);
                const float* vr = vg + (int64_t)(j0 + u) * a.stride_n;
#pragma unroll
                for (int d = 0; d < D / 64; ++d) acc[d] = fma(pu, (double)vr[lane + 64 * d], acc[d]);
            }
        }
#pragma unroll
        for (int n = 32; n >= 1; n >>= 1) sum += __shfl_xor(sum, n, 64);
#pragma unroll
        for (int d = 0; d < D / 64; ++d) {
            const int64_t at = base + (int64_t)r * a.stride_n + lane + 64 * d;
            double y = acc[d] / sum;
            if (it.flags & DIFA_ITEM_ADD_RESIDUAL) y += (double)((const float*)a.residual)[at];
            ((float*)a.out)[at] = (float)y;
        }
    }
}

hipError_t launch_attn_f32(const AttnArgs& a, int head_dim, int n_items, hipStream_t stream) {
    if (n_items <= 0) return hipSuccess;
    // (a grid dimension holds fewer than 2^32 threads)
    const int64_t blocks = (int64_t)a.f32_blocks + a.copy_chunks, in_x = blocks < (1 << 22) ? blocks : 1 << 22;
    const dim3 grid((unsigned)in_x, (unsigned)((blocks + in_x - 1) / in_x));
    const bool wide = a.stride_n >= ((int64_t)1 << 31) / (4 * kF32Keys);
    const dim3 threads(64 * kF32Waves);
    if (head_dim == 128 && !wide) hipLaunchKernelGGL((attn_f32_kernel<128, false>), grid, threads, 0, stream, a);
    else if (head_dim == 128) hipLaunchKernelGGL((attn_f32_kernel<128, true>), grid, threads, 0, stream, a);
    else if (head_dim == 64 && !wide) hipLaunchKernelGGL((attn_f32_kernel<64, false>), grid, threads, 0, stream, a);
    else if (head_dim == 64) hipLaunchKernelGGL((attn_f32_kernel<64, true>), grid, threads, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Cached heads (Sec. 3.2) by a kernel of their own, for a layer that computes no head at all.  A 16-byte-per-lane copy of the heads' rows; beyond 32768 workgroups a thread takes
// several vectors, four in flight.  HBM bound: 2 * N * D * elem bytes per (batch entry, cached head).
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cache_copy_kernel(CopyArgs c) {
    const int64_t per_head = (int64_t)c.n_tokens * c.vec_per_row;
    const int64_t total = per_head * c.n_copy * c.batch;
    const int64_t stride = (int64_t)gridDim.x * 256;
    const char* __restrict__ src = (const char*)c.src;
    char* __restrict__ dst = (char*)c.dst;
    auto offset_of = [&](int64_t idx) {
        const int64_t hh = idx / per_head, rem = idx - hh * per_head;
        const int bb = (int)(hh / c.n_copy), ch = (int)(hh - (int64_t)bb * c.n_copy);
        const int head = c.copy_heads[ch];
        const int64_t n = rem / c.vec_per_row, vc = rem - n * c.vec_per_row;
        return (int64_t)bb * c.stride_b + (int64_t)head * c.stride_h + n * c.stride_n + vc * 16;
    };
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (; idx + 3 * stride < total; idx += 4 * stride) {
        const int64_t o0 = offset_of(idx), o1 = offset_of(idx + stride);
        const int64_t o2 = offset_of(idx + 2 * stride), o3 = offset_of(idx + 3 * stride);
        const uint4 v0 = *(const uint4*)(src + o0);
        const uint4 v1 = *(const uint4*)(src + o1);
        const uint4 v2 = *(const uint4*)(src + o2);
        const uint4 v3 = *(const uint4*)(src + o3);
        *(uint4*)(dst + o0) = v0;
        *(uint4*)(dst + o1) = v1;
        *(uint4*)(dst + o2) = v2;
        *(uint4*)(dst + o3) = v3;
    }
    for (; idx < total; idx += stride) {
        const int64_t o0 = offset_of(idx);
        *(uint4*)(dst + o0) = *(const uint4*)(src + o0);
    }
}

// ------------------------------------------------------------------------------------------
// Residual sharing, refresh step: residual = o_full - o_arrow, element by element, rounded once to the
// element type.  HBM bound: three tensors pass once.
// ------------------------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void residual_store_kernel(const void* o_full, const void* o_arrow, void* residual,
                                                              int64_t n_vec) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_vec; i += stride) {
        if (BF16) {
            const bf16x8 a = ((const bf16x8*)o_full)[i], b = ((const bf16x8*)o_arrow)[i];
            bf16x8 r;
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = (__bf16)((float)a[e] - (float)b[e]);   // the difference of two bf16 values is exact in fp32
            ((bf16x8*)residual)[i] = r;
        } else {
            const floatx4 a = ((const floatx4*)o_full)[i], b = ((const floatx4*)o_arrow)[i];
            ((floatx4*)residual)[i] = a - b;
        }
    }
}

hipError_t launch_residual_store(const void* o_full, const void* o_arrow, void* residual, int64_t n_elems, int dtype,
                                 hipStream_t stream) {
    if (n_elems <= 0) return hipSuccess;
    const bool bf16 = dtype == DIFA_DTYPE_BF16;
    const int64_t n_vec = n_elems / (bf16 ? 8 : 4);          // (head_dim is a multiple of 64: no remainder)
    int64_t blocks = (n_vec + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    if (bf16) hipLaunchKernelGGL(residual_store_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, stream, o_full, o_arrow, residual, n_vec);
    else hipLaunchKernelGGL(residual_store_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, stream, o_full, o_arrow, residual, n_vec);
    return hipGetLastError();
}

hipError_t launch_cache_copy(const CopyArgs& c, hipStream_t stream) {
    const int64_t total = (int64_t)c.n_tokens * c.vec_per_row * c.n_copy * c.batch;
    if (total <= 0) return hipSuccess;
    // (measured on a 2K layer with every head cached: one vector per thread and as many small workgroups as
    // that takes moves 6.4 TB/s, four per thread in a quarter of the workgroups 5.9)
    int64_t blocks = (total + 255) / 256;
    if (blocks > 256 * 128) blocks = 256 * 128;
    hipLaunchKernelGGL(cache_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, c);
    return hipGetLastError();
}

}  // namespace difa
