// How a call is cut into tiles and how many executor blocks run them (cut.h).
#include "cut.h"

#include <algorithm>
#include <cmath>
#include <cstring>

#include "sparkcl_dev.h"

namespace sparkcl {

uint64_t input_bytes(uint32_t kernel_id)
{
    return kernel_id == SPARKCL_FMUL ? 8ull : 4ull;
}

void ExecEnv::rows_are_tuned(bool tuned)
{
    static_assert(SPARKCL_POLY == 1 && SPARKCL_FMUL == 2, "the first two kernels' rows");
    if (tuned)
        std::memcpy(tuned_rows, tuning.tile[TM_PER_LAUNCH], sizeof(tuned_rows));
    else
        std::memset(tuned_rows, 0, sizeof(tuned_rows));
}

bool ExecEnv::small_by_time() const
{
    return std::memcmp(tuned_rows, tuning.tile[TM_PER_LAUNCH], sizeof(tuned_rows)) == 0;
}

uint32_t exec_block(const ExecEnv *ctx, uint32_t kid_mask)
{
    uint32_t b = ctx->tuning.block_many;
    for (uint32_t k = 0; k < 3; ++k)
        if (kid_mask == (1u << k))
            b = ctx->tuning.block[k];
    return b ? b : (uint32_t)kBlock;
}

uint32_t kernel_unroll(const sparkcl_tuning &t, uint32_t kid)
{
    const uint32_t u = kid >= SPARKCL_POLY && kid <= SPARKCL_MC_PI ? t.unroll[kid - 1] : 0;
    return u ? u : (uint32_t)kUnroll;
}

uint32_t exec_occupancy(const ExecEnv *ctx, uint32_t kid_mask)
{
    return (uint32_t)(mc_instance(ctx, kid_mask) ? ctx->occ_mc : ctx->occ_batch);
}

bool mc_instance(const ExecEnv *ctx, uint32_t kid_mask)
{
    return kid_mask == (1u << (SPARKCL_MC_PI - 1)) && !ctx->tune_shared_mc;
}

uint32_t exec_grid(const ExecEnv *ctx, uint32_t kid_mask, uint64_t ntiles, uint64_t ntasks,
                   uint32_t block)
{
    // a batch of Monte-Carlo tasks alone runs the executor's MC instance,
    // which fits more blocks per CU
    const uint32_t occ = exec_occupancy(ctx, kid_mask);
    uint32_t per_cu = 0;
    if (ctx->exec_blocks_per_cu) {
        per_cu = ctx->exec_blocks_per_cu;
    } else if (kid_mask == (1u << (SPARKCL_MC_PI - 1)) && !ctx->tune_shared_mc) {
        // Monte-Carlo tasks alone: the executor instance of their own
        per_cu = ctx->tuning.blocks_per_cu_mc_only ? ctx->tuning.blocks_per_cu_mc_only : occ;
    } else {
        // the largest tuned value among the kernels in the batch: a
        // compute-bound kernel needs waves to hide instruction latency, a
        // streaming one does best with a few deep streams per CU
        for (uint32_t k = 0; k < 3; ++k)
            if (kid_mask & (1u << k)) {
                const uint32_t v = ctx->tuning.blocks_per_cu[k];
                per_cu = std::max(per_cu, v ? v : occ);
            }
        if (per_cu == 0)
            per_cu = occ;
        // many small tasks: per-tile latency (queue, descriptor, ticket,
        // final combine) has to be hidden by more blocks per CU
        if (ntasks && ntiles < 4 * ntasks) {
            const uint32_t v = ctx->tuning.blocks_per_cu_many;
            per_cu = std::max(per_cu, v ? v : occ);
        }
    }
    // per_cu counts 256-thread blocks (waves per SIMD); larger blocks take
    // their share of them
    const uint32_t waves = std::max(1u, std::min(per_cu, occ));
    if (block == 0)
        block = exec_block(ctx, kid_mask);
    return std::max(1u, waves * (uint32_t)kBlock / block) * (uint32_t)ctx->cus;
}

namespace {

// A call is cut before its tasks are checked: one whose kernel id check_task
// will reject has no row in the tables and takes no part in the cut.
bool known(const sparkcl_task &t)
{
    return t.kernel_id >= SPARKCL_POLY && t.kernel_id <= SPARKCL_MC_PI;
}

// Elements of a tile that moves about `bytes`; a power of two.
uint32_t even_tile(const sparkcl_task &t, uint64_t bytes)
{
    return (uint32_t)(bytes / (t.kernel_id == SPARKCL_POLY && !t.out ? 4 : 8));
}

// The tile size of a batch of streaming tasks too small for the batched
// table's tiles: the per-launch table is tuned on one task at a time and cuts
// such a batch into several times as many tiles as blocks, each with its two
// memory round trips and its queue atomic.  Taken is the size of least
// estimated time: rounds of tiles, each the time of its bytes and of about
// 110 KB more (4 us at a block's share of 7 TB/s; a third of that if no task
// has more than one tile, and so none a ticket); one round alone counts half
// its bytes again, since the blocks that share a CU with another then finish
// last with nothing left to even it out.  One block per CU streams best (the
// caller's count, if it gives one).  Tiles that also write stop at 512 KB:
// 20 tasks of 3e6 elements took 133 us so and 138 at 1 MB.
// Measured on MI355X, per-launch table and this rule: 64 FMUL tasks of 2^20
// elements 125 and 90 us, as a chain of three maps 179 and 126; 48 POLY tasks
// of 300007 41 and 33 (with their values written 44 and 41); 256 of 20001 29
// and 22; 16 of 10^6 with values 56 and 39.  Batches with Monte-Carlo tasks,
// which compute, stay with the table, and so do rows that the caller set.
void even_cut(const ExecEnv *ctx, const sparkcl_task *tasks, uint32_t ntasks, uint32_t mask,
              uint32_t per_cu, Cut *c)
{
    if (mask & (1u << (SPARKCL_MC_PI - 1)))
        return;
    const uint64_t grid = per_cu                    ? (uint64_t)per_cu * ctx->cus
                          : ctx->exec_blocks_per_cu ? exec_grid(ctx, mask)
                                                    : ctx->cus;
    const double fixed = 110e3 * ctx->cus / (double)grid;
    bool writes = false;
    uint64_t table_tiles = 0; // of the per-launch table
    for (uint32_t i = 0; i < ntasks; ++i) {
        if (!known(tasks[i]))
            continue;
        writes |= tasks[i].out != nullptr;
        const uint32_t T = tile_for(ctx->tuning, TM_PER_LAUNCH, tasks[i].kernel_id, tasks[i].n);
        table_tiles += std::max<uint64_t>(1, (tasks[i].n + T - 1) / T);
    }
    double best = 0;
    for (uint64_t bytes = 32u << 10; bytes <= (writes ? 512u : 2048u) << 10; bytes *= 2) {
        uint64_t tiles = 0, largest = 0;
        bool tickets = false;
        for (uint32_t i = 0; i < ntasks; ++i) {
            if (!known(tasks[i]))
                continue;
            const uint64_t T = even_tile(tasks[i], bytes);
            tickets |= tasks[i].n > T;
            tiles += std::max<uint64_t>(1, (tasks[i].n + T - 1) / T);
            largest = std::max(largest, std::min(T, tasks[i].n) *
                                            (input_bytes(tasks[i].kernel_id) +
                                             (tasks[i].out ? 4 : 0)));
        }
        if (tiles > std::max<uint64_t>(table_tiles, 4 * grid))
            continue; // no more workspace than the table's cut, or little
        const uint64_t rounds = (tiles + grid - 1) / grid;
        const double cost = (rounds == 1 ? 1.5 : (double)rounds) * (double)largest +
                            (double)rounds * (tickets ? fixed : fixed / 3);
        if (best == 0 || cost < best) {
            best = cost;
            c->even_bytes = bytes;
        }
    }
    if (c->even_bytes)
        c->grid = (uint32_t)grid;
}

} // namespace

Cut plan_cut(const ExecEnv *ctx, int mode, const sparkcl_task *tasks,
                                uint32_t ntasks, bool host_in, uint32_t per_cu)
{
    // Tile table: the batched one, unless the batch would then give the
    // executor's blocks fewer than two tiles each (a batch of one or a few
    // partitions, where the batched table's large tiles would leave most of
    // the GPU idle, or about one large tile per block, where the time is set
    // by how unevenly the blocks land on the CUs); such a batch is cut by
    // estimated time if it streams, else with the per-launch table.  The
    // choice is a function of the call, so a repeated call is cut the same
    // way.
    Cut c;
    c.tm = mode != SPARKCL_PER_LAUNCH && !host_in ? TM_BATCHED : TM_PER_LAUNCH;
    // A batch of many tasks of widely spread sizes takes the mixed-batch
    // tile sizes instead of the per-bucket table (tuned on batches of one
    // size): one tile size per kernel, so small tasks run whole and large
    // ones in mid-sized interleaved tiles.  On the 4096-task uneven batch one
    // 2^16 tile for the streaming kernels ran it in 515 us against 553 us
    // with the table.  The size is either given (tile_many) or derived from
    // the batch's own total work, cut into a tuned number of tiles per CU:
    // the share, not the size, is what carries over between batches.
    // Streaming work is counted in input bytes, so a POLY tile (4 bytes per
    // element) holds twice the elements of an FMUL tile (8): tiles of equal
    // bytes stream for equal times and carry equal shares of the per-tile
    // set-up (on the uneven batch, 2^16 POLY with 2^15 FMUL elements ran in
    // 461 us against 471 us with 2^16 for both).
    if (c.tm == TM_BATCHED && ntasks >= kMixedMinTasks) {
        uint32_t lo = SPARKCL_TUNE_BUCKETS, hi = 0;
        uint64_t total[2] = {0, 0}; // streaming input bytes, Monte-Carlo samples
        for (uint32_t i = 0; i < ntasks; ++i) {
            const uint32_t b = size_bucket(tasks[i].n);
            lo = std::min(lo, b);
            hi = std::max(hi, b);
            if (tasks[i].kernel_id == SPARKCL_MC_PI)
                total[1] += tasks[i].n;
            else if (tasks[i].kernel_id == SPARKCL_POLY || tasks[i].kernel_id == SPARKCL_FMUL)
                total[0] += tasks[i].n * input_bytes(tasks[i].kernel_id);
        }
        c.mixed = hi >= lo + kMixedMinSpan;
        for (uint32_t kid = SPARKCL_POLY; kid <= SPARKCL_MC_PI && c.mixed; ++kid) {
            const int k = kid == SPARKCL_MC_PI ? 1 : 0;
            const uint32_t q = ctx->tuning.many_tiles_per_cu[k];
            if (q == 0 || total[k] == 0)
                continue;
            const double per_elem = k == 1 ? 1.0 : (double)input_bytes(kid);
            const double want = (double)total[k] / ((double)ctx->cus * q) / per_elem;
            const double l2 = std::rint(std::log2(std::max(want, 1.0)));
            const int e = (int)std::min<double>(kMaxTileLog2, std::max<double>(kMinTileLog2, l2));
            c.share_tile[kid - 1] = 1u << e;
        }
    }
    if (c.tm == TM_BATCHED) {
        uint64_t tiles = 0;
        uint32_t mask = 0;
        for (uint32_t i = 0; i < ntasks; ++i) {
            if (!known(tasks[i]))
                continue;
            const uint32_t T = cut_tile(ctx, c, tasks[i]);
            tiles += std::max<uint64_t>(1, (tasks[i].n + T - 1) / T);
            mask |= 1u << (tasks[i].kernel_id - 1);
        }
        const uint64_t grid =
            per_cu ? per_cu * (uint32_t)ctx->cus : exec_grid(ctx, mask, tiles, ntasks);
        if (tiles < 2 * grid) {
            c.tm = TM_PER_LAUNCH;
            c.mixed = false;
            c.share_tile[0] = c.share_tile[1] = c.share_tile[2] = 0;
            if (ctx->small_by_time())
                even_cut(ctx, tasks, ntasks, mask, per_cu, &c);
        }
    }
    return c;
}

uint32_t cut_tile(const ExecEnv *ctx, const Cut &c, const sparkcl_task &t)
{
    if (c.even_bytes)
        return even_tile(t, c.even_bytes);
    if (c.tm == TM_BATCHED && c.mixed && known(t)) {
        if (ctx->tuning.tile_many[t.kernel_id - 1])
            return ctx->tuning.tile_many[t.kernel_id - 1];
        const uint32_t s = c.share_tile[t.kernel_id - 1];
        if (s)
            return s;
    }
    return tile_for(ctx->tuning, c.tm, t.kernel_id, t.n);
}

} // namespace sparkcl
