// How a call is cut into tiles and how many executor blocks run them: pure
// functions of the call, the tuning table and the device's figures.  Host
// logic without HIP.
#pragma once

#include <cstdint>

#include "sparkcl.h"
#include "tuning.h"

namespace sparkcl {

// How a reduce-kind call is cut into tiles: the tuning table's row (batched
// or per-launch) and whether the mixed-batch tile sizes apply.
struct Cut {
    int tm = TM_PER_LAUNCH;
    bool mixed = false;
    // mixed batches: each kernel's tile derived from the batch's totals and
    // the tuned tiles per CU (index kernel id - 1; 0: none derived)
    uint32_t share_tile[3] = {0, 0, 0};
    // small streaming batches: tiles of this many bytes, on a grid of this many
    // executor blocks (0: by the table)
    uint64_t even_bytes = 0;
    uint32_t grid = 0;
};

// A batched call is "mixed" (takes sparkcl_tuning.tile_many) with at least
// this many tasks whose sizes span at least this many log2 buckets.
constexpr uint32_t kMixedMinTasks = 512;
constexpr uint32_t kMixedMinSpan = 4;

// What a cut depends on beside the call.
struct ExecEnv {
    int cus = 0;
    int occ_batch = 1; // batch-executor blocks per CU that fit
    int occ_mc = 1;    // blocks per CU of the Monte-Carlo-only executor
    // autotuner only: Monte-Carlo batches run the shared executor, so that
    // blocks_per_cu[MC_PI] is measured where mixed batches use it
    bool tune_shared_mc = false;
    uint32_t exec_blocks_per_cu = 0; // the caller's; 0: the tuned value
    sparkcl_tuning tuning{};
    // The per-launch rows of the streaming kernels that were tuned on single
    // tasks: the built-in ones, or those that the autotuner or its cache file
    // put in force (0: none).  While they are the table's, small batches are
    // cut by estimated time; rows that the caller set are the cut.  So a table
    // read and set again changes nothing, a tuned context and one that loads
    // its cache file cut alike, and a row changed and changed back counts as
    // unchanged.
    uint32_t tuned_rows[2][SPARKCL_TUNE_BUCKETS] = {};

    void rows_are_tuned(bool tuned);
    bool small_by_time() const;
};

// Input bytes a streaming kernel reads per element (x, and y for FMUL).
uint64_t input_bytes(uint32_t kernel_id);
// The cut of a call: a function of the call and the ExecEnv; allocates
// nothing.
Cut plan_cut(const ExecEnv *ctx, int mode, const sparkcl_task *tasks, uint32_t ntasks,
             bool host_in, uint32_t per_cu = 0);
// The tile size of one task under a cut.
uint32_t cut_tile(const ExecEnv *ctx, const Cut &c, const sparkcl_task &t);
// Persistent-executor grid for a batch holding the kernels in kid_mask
// (bit k-1 for kernel id k) and `ntiles` tiles over `ntasks` tasks.
uint32_t exec_grid(const ExecEnv *ctx, uint32_t kid_mask, uint64_t ntiles = 0,
                   uint64_t ntasks = 0, uint32_t block = 0);
// The executor's threads per block for a batch holding the kernels in
// kid_mask (one kernel: its tuned size; several: the mixed-batch size), and
// the float4 loads in flight per thread for a kernel's streaming loop.
uint32_t exec_block(const ExecEnv *ctx, uint32_t kid_mask);
// Executor blocks per CU that fit for a batch holding the kernels in
// kid_mask (the Monte-Carlo-only instance fits more).
uint32_t exec_occupancy(const ExecEnv *ctx, uint32_t kid_mask);
// Whether a batch holding the kernels in kid_mask runs the Monte-Carlo-only
// executor instance (Monte-Carlo tasks alone).
bool mc_instance(const ExecEnv *ctx, uint32_t kid_mask);
uint32_t kernel_unroll(const sparkcl_tuning &t, uint32_t kid);

} // namespace sparkcl
