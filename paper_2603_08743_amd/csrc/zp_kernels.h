// Kernel-side argument block and launch entry points shared by the HIP sources of libzp.
// Paper sections are cited as in include/zp.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zp {

enum : int {
    STAGE_SCORE = 1,    // compute S from K and the window queries
    STAGE_SELECT = 2,   // fill, top-k_h, ascending list
    STAGE_COMPACT = 4,  // move kept K/V rows
    STAGE_LOAD_SCORES = 8,  // S comes from args.scores_in instead of STAGE_SCORE
    STAGE_LOAD_LIST = 16,   // the kept list comes from args.keep_idx_in / len_in
    STAGE_CHECK_SLOT = 32,  // a launch after the scoring launches of the same call: units they skipped are skipped here too
};

// Score refinements switched on for a launch (appendix "Global Score", "Pooling at the Sequence Dimension",
// "Lightning Redundancy") and how compaction carries the global-score cache along.
enum : int {
    EX_GLOBAL = 1,     // decayed max with the cached history, cache updated
    EX_POOL = 2,       // max pooling along the live sequence
    EX_RED = 4,        // S - lambda * R
    EX_MOVE_F = 8,     // compaction moves F rows read back from global memory (staged call)
    EX_POOL_FIRST = 32,  // pooling only for requests without history
    EX_RED_FUSED = 64,   // redundancy: the similarity tiles of the live prefix come from the key tiles of sweep 2 (row sums at off_R)
    EX_RED_STAGED = 128, // redundancy of large blocks: block by block, rows through LDS (redundancy_staged)
    EX_MOVE_F_LDS = 16 // compaction writes the kept entries' values from the on-chip copy made by EX_GLOBAL (fused call)
};

// Reasons a kernel skips a unit (reported through the context's status words).
enum : int {
    BAD_NUM_BLOCKS = 1, BAD_VALID_LEN = 2, BAD_KEEP = 3, BAD_SLOT = 4, BAD_BLOCK_ID = 5, BAD_KEEP_IDX = 6,
};

struct Args {
    // paged memory (Background, "Pre-allocated memory"; Method, query cache)
    char *k, *v;
    const char *q;
    int layer0, L_slab, N_total, b, h_kv, h_q, d, M, w, dtype;
    // batch
    int B, N_max, max_blocks, L;
    const int *block_table, *dst_table, *num_blocks, *q_slot, *valid_len, *keep;
    // derived on the host
    int G, T_max, budget, row_bytes, b_shift;   // b_shift >= 0 iff b is a power of two
    float scale_log2;                          // log2(e) / sqrt(d)
    int stages;
    int xcd_map;                               // 1: contiguous unit ranges per XCD (see unit_of_block)
    int by_cost;                               // 1: costliest units first (see unit_by_cost)
    // staged inputs / outputs (device pointers, any may be null depending on stages)
    const float *scores_in; int scores_in_stride;
    float *scores_out;                         // [units][T_max]
    const int *keep_idx_in; const int *len_in;
    int *keep_idx_out;                         // [units][budget]
    int *len_out;                              // [units]
    int *status;                               // [8]: flag, first bad unit, reason
    // refinements
    int ex;                                    // EX_* flags
    float *F;                                  // [L_slab][N_total][b][h_kv] global-score cache
    const int *compressed;                     // [B]
    float alpha, lambda, inv_tau_log2, p_thr;  // inv_tau_log2 = log2(e) / tau
    int pool_r;                                // pooling radius (kernel - 1) / 2
    int off_G;                                 // LDS: [T_max] copy of the global scores for EX_MOVE_F_LDS
    int off_R;                                 // LDS: [T_max] redundancy row sums + 96 words per wave for EX_RED_FUSED
    // byte offsets into dynamic LDS
    int off_S, off_tbl, off_dst, off_misc, off_union, lds_bytes;
    int NP;                                    // matrix-core kernel: passes over the keys (padded rows only)
    // few units: several workgroups per unit, one launch per dependency (the rules and their figures: split_pays and pick_parts in zp_api.hip)
    int phase;                                 // matrix-core kernel: 0 whole unit, 1 sweep 1 of a part, 2 sweep 2 of a part
    int parts;                                 // workgroups per unit (phases 1 and 2), each taking whole segments
    float2 *seg;                               // [units][ZP_SEGMENTS][query rows, padded]: (reference, sum) of sweep 1 per segment
    int2 *unit_out; const int2 *unit_in;       // [units]: (live prefix length, keep count) of every unit, written by phase 2, read by the launch after it
    int slices, slice_bytes;                   // row-moving kernel: workgroups per unit, bytes of a row each of them moves
};

// check-only paged decode attention (zp_check.hip)
struct DecodeArgs {
    const char *k, *v, *q;      // pools [L_slab][N_total][b][h_kv][d]; q [B][L_slab][h_q][d]
    float *out;                 // [B][L_slab][h_q][d]
    const int *table, *len;     // [B][table_stride], [B][L_slab][h_kv]
    int *status;
    int B, L_slab, N_total, b, h_kv, h_q, d, dtype, table_stride, row_bytes;
    float scale_log2;
};
hipError_t launch_decode_attention(const DecodeArgs &a, int items, hipStream_t s);

// launchers (host).  Each returns the hipError_t of the launch.
hipError_t launch_unit_generic(const Args &a, int units, hipStream_t s);
hipError_t launch_unit_sliced(const Args &a, int units, hipStream_t s);
// The keys of a unit are cut into at most ZP_SEGMENTS runs of whole tiles, a function of their number alone.  Sweep 1 sums
// every run by itself and the runs are put together in ascending order, whichever workgroups they ran in: a call gives the
// same bits with one workgroup per unit and with several.
// One run costs a maximum over its first 32 keys (FIRST_MAX in zp_mfma.h) or a second look at them, and a merge: between nothing and
// 1.5 % of a launch against one run, most with several blocks per wave.  Four runs where a wave holds several query blocks: such a
// workgroup fills a compute unit, so 64 units have their share with four (384 units of 8208 positions, G 5, w 128, one launch with
// the second look: eight runs cost 0.9 %).
#define ZP_SEGMENTS 8
constexpr __host__ __device__ int segments_of(int RB) { return RB > 1 ? 4 : ZP_SEGMENTS; }
// Runs of a unit with `ntiles` key tiles: as many as allowed of at least three tiles each, of equal length but for one tile; run
// sg starts with tile sg * ntiles / count.
constexpr __host__ __device__ int segment_count(int ntiles, int segments) {
    const int n = (ntiles + 1) / 3;
    return n < 1 ? 1 : (n < segments ? n : segments);
}
// Geometry of the matrix-core kernel for a launch: waves per workgroup, 32-row query blocks per wave, passes over the keys,
// row bytes of the instantiation and whether the pool's rows are shorter than that.
struct MfmaGeo { int NW, RB, NP, rowb; bool pad; };
bool mfma_path_available(const Args &a, MfmaGeo *g);
hipError_t launch_unit_mfma(const Args &a, int units, const MfmaGeo &g, hipStream_t s);
// instantiations by row size and workgroup width, one translation unit each (zp_mfma_*.hip); _ref: with score refinements
#define ZP_DECLARE_MFMA(name) hipError_t name(const Args &a, int units, int NW, int RB, hipStream_t s);
ZP_DECLARE_MFMA(launch_mfma_d64) ZP_DECLARE_MFMA(launch_mfma_d64_wide) ZP_DECLARE_MFMA(launch_mfma_d64_ref) ZP_DECLARE_MFMA(launch_mfma_d64_wide_ref)
ZP_DECLARE_MFMA(launch_mfma_d128) ZP_DECLARE_MFMA(launch_mfma_d128_wide) ZP_DECLARE_MFMA(launch_mfma_d128_ref) ZP_DECLARE_MFMA(launch_mfma_d128_wide_ref)
#undef ZP_DECLARE_MFMA
hipError_t launch_mfma_pad_bf16(const Args &a, int units, int rowb, int NW, hipStream_t s);
hipError_t launch_mfma_pad_bf16_long(const Args &a, int units, int rowb, int NW, hipStream_t s);
hipError_t launch_mfma_pad_f32(const Args &a, int units, int rowb, int NW, hipStream_t s);
// keys per LDS tile of the matrix-core kernel: two 32-key subtiles, one for rows so long that two tiles of 64 would not
// leave room for a second workgroup on the CU
constexpr int mfma_tile_keys(int rowb) { return rowb <= 256 ? 64 : 32; }
size_t mfma_union_bytes(const MfmaGeo &g);

}  // namespace zp
