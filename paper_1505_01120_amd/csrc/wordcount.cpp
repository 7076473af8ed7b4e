// WordCount (sec. 3.2.3): words of a device-resident byte stream counted under
// their 64-bit FNV-1a key, in per-block LDS tables whose misses go to
// per-partition spill regions; a merge pass counts each partition's keys and
// adds them to one global open-addressing table, which is then compacted into
// the caller's arrays.
#include <algorithm>
#include <cstring>
#include <string>

#include "runtime.h"

using namespace sparkcl;

namespace {

// The scan's geometry: bytes of text per lane and chunk, and blocks.  Equal
// shares for all lanes of kWcPerCu blocks per CU, cut into as few chunks as `most`
// allows (16 steps past each span's end are spent on words that
// cross it); a text too short for 16 bytes per lane takes fewer blocks, whose
// waves share their tables.
void scan_geometry(const sparkcl_ctx *ctx, uint64_t nbytes, uint32_t most, uint32_t *span,
                   uint32_t *grid)
{
    const uint64_t blocks = (uint64_t)kWcPerCu * (uint64_t)ctx->cus;
    const uint64_t lanes = 64ull * kWcWaves * blocks;
    const uint64_t per = std::max<uint64_t>(1, (nbytes + lanes - 1) / lanes);
    const uint64_t sweeps = (per + most - 1) / most;
    *span = (uint32_t)(((per + sweeps - 1) / sweeps + 15) / 16 * 16);
    const uint64_t chunks = std::max<uint64_t>(1, (nbytes + 64ull * *span - 1) / (64ull * *span));
    *grid = (uint32_t)std::min<uint64_t>((chunks + kWcWaves - 1) / kWcWaves, blocks);
}

} // namespace

extern "C" {

int sparkcl_wordcount(sparkcl_ctx *ctx, const uint8_t *text, uint64_t nbytes, uint64_t *keys,
                      uint64_t *counts, uint64_t capacity, uint64_t *ndistinct,
                      uint64_t *nwords, void *stream)
{
    int rc = check_ctx(ctx);
    if (rc != SPARKCL_OK)
        return rc;
    if (!ndistinct || !nwords || (nbytes && !text) || (capacity && (!keys || !counts)))
        return fail(SPARKCL_EINVAL, "NULL argument");
    *ndistinct = 0;
    *nwords = 0;
    if (nbytes == 0)
        return SPARKCL_OK;
    if (nbytes > kMaxN)
        return fail(SPARKCL_ETOOBIG, "text of " + std::to_string(nbytes) +
                                         " bytes exceeds 2^40");
    std::lock_guard<std::mutex> g(ctx->mu);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // open addressing at load <= 1/2: room for capacity + 1 keys (so one key
    // past the capacity is still seen), never more than the text can hold
    uint64_t need = std::min<uint64_t>(capacity + 1, nbytes / 2 + 1);
    uint64_t slots = 1024;
    while (slots < 2 * need)
        slots *= 2;
    uint32_t span, grid;
    scan_geometry(ctx, nbytes, kWcMaxSpan, &span, &grid);
    const uint64_t table_bytes = slots * 16 + 64;
    // Spill regions: room for one spilled word per 16 bytes of each scan
    // block's share of the text (a quarter more for the spread between
    // partitions); words past a full region go to the table directly.  Left
    // out when the arena cannot hold them.
    const uint64_t parts = 1ull << kWcPartBits;
    uint64_t cap = nbytes / ((uint64_t)grid * parts * 16);
    cap = cap + cap / 4 + 16;
    const uint64_t spill_bytes =
        (uint64_t)grid * (parts * (cap * 8 + 4) + kWcSlots * (sizeof(uint64_t) + sizeof(uint32_t)));
    uint64_t bytes = table_bytes + spill_bytes;
    uint64_t off = ctx->arena.alloc(bytes);
    if (off == Arena::kFail) {
        cap = 0;
        bytes = table_bytes;
        off = ctx->arena.alloc(bytes);
    }
    if (off == Arena::kFail)
        return fail(SPARKCL_ENOMEM, "word-count table of " + std::to_string(bytes) +
                                        " bytes does not fit the arena");
    char *base = static_cast<char *>(ctx->dev(off));
    WcArgs a{};
    a.text = text;
    a.n = nbytes;
    a.keys = reinterpret_cast<uint64_t *>(base);
    a.counts = reinterpret_cast<uint64_t *>(base + slots * 8);
    a.ctl = reinterpret_cast<uint64_t *>(base + slots * 16);
    a.mask = slots - 1;
    a.spill_cap = (uint32_t)cap;
    a.span = span;
    // (the second half of the control words' 64 bytes)
    uint8_t *pad = reinterpret_cast<uint8_t *>(a.ctl + 4);
    if (nbytes < 16) {
        a.text = pad;
        a.n = kWcPad;
    }
    if (cap) {
        a.spill = reinterpret_cast<uint64_t *>(base + table_bytes);
        a.table_keys = a.spill + (uint64_t)grid * parts * cap;
        a.table_counts = reinterpret_cast<uint32_t *>(a.table_keys + (uint64_t)grid * kWcSlots);
        a.spill_cnt = a.table_counts + (uint64_t)grid * kWcSlots;
    }
    // (only the table and the counters need clearing: every spill slot read
    // by the merge was written by the scan)
    if ((rc = ensure_pinned(ctx, 1)) == SPARKCL_OK &&
        (rc = launch_zero(base, table_bytes, s)) == SPARKCL_OK &&
        (nbytes >= 16 || (rc = launch_wc_pad(text, nbytes, pad, s)) == SPARKCL_OK) &&
        (rc = launch_wordcount(a, grid, s)) == SPARKCL_OK &&
        (!cap || (rc = launch_wc_merge(a, grid, s)) == SPARKCL_OK) &&
        (rc = launch_wc_compact(a, keys, counts, capacity, s)) == SPARKCL_OK) {
        hipError_t e = hipMemcpyAsync(ctx->pinned, a.ctl, 32, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipStreamSynchronize(s);
        if (e != hipSuccess)
            rc = fail_hip(e, "word count");
    } else if (rc != SPARKCL_OK) {
        (void)hipStreamSynchronize(s);
        rc = fail(rc, "word-count launch failed");
    }
    ctx->arena.release(off);
    if (rc != SPARKCL_OK)
        return rc;
    uint64_t ctl[4];
    std::memcpy(ctl, ctx->pinned, sizeof(ctl));
    *nwords = ctl[0];
    *ndistinct = ctl[3];
    if (ctl[2] || ctl[3] > capacity)
        return fail(SPARKCL_ETOOBIG, "more distinct words than the capacity of " +
                                         std::to_string(capacity));
    return SPARKCL_OK;
}

int sparkcl_wordcount_locate(sparkcl_ctx *ctx, const uint8_t *text, uint64_t nbytes,
                             const uint64_t *keys, uint64_t nkeys, uint64_t *offsets,
                             void *stream)
{
    int rc = check_ctx(ctx);
    if (rc != SPARKCL_OK)
        return rc;
    if ((nbytes && !text) || (nkeys && (!keys || !offsets)))
        return fail(SPARKCL_EINVAL, "NULL argument");
    if (nkeys == 0)
        return SPARKCL_OK;
    if (nbytes > kMaxN)
        return fail(SPARKCL_ETOOBIG, "text of " + std::to_string(nbytes) +
                                         " bytes exceeds 2^40");
    if (nkeys > 0xFFFFFFFFull)
        return fail(SPARKCL_ETOOBIG, "more than 2^32 - 1 keys");
    std::lock_guard<std::mutex> g(ctx->mu);
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint64_t least = 1024; // slots, at a load of 1/3 to 2/3
    while (least < 2 * nkeys)
        least *= 2;
    least = least / 4 * 3;
    uint32_t span, grid;
    // A block's LDS keys settle a word only once one before it has been met, so
    // the spans of a first chunk, which the waves walk side by side, gain
    // little by them: shorter ones while there would be fewer than four chunks
    // (100 MiB: 270 us in two of 192 bytes, 252 in three of 128; 256 MiB: 482 in
    // four of 256, 489 in eight of 128).
    const uint64_t lanes = 64ull * kWcWaves * kWcPerCu * (uint64_t)ctx->cus;
    scan_geometry(ctx, nbytes, nbytes < 4 * kWlMaxSpan * lanes ? kWlMaxSpan / 2 : kWlMaxSpan,
                  &span, &grid);
    // the table, then the control words; a small one (some 2 MiB at most, half
    // an XCD's L2) four times as large where that fits, which keeps the chains
    // of dependent accesses short that a call with few keys waits for
    uint64_t slots = least <= (1u << 15) ? 4 * least : least;
    uint64_t off = ctx->arena.alloc(slots * sizeof(WlSlot) + 64);
    if (off == Arena::kFail && slots != least) {
        slots = least;
        off = ctx->arena.alloc(slots * sizeof(WlSlot) + 64);
    }
    const uint64_t zero_bytes = slots * sizeof(WlSlot) + 64;
    if (off == Arena::kFail)
        return fail(SPARKCL_ENOMEM, "word lookup table of " + std::to_string(zero_bytes) +
                                        " bytes does not fit the arena");
    char *base = static_cast<char *>(ctx->dev(off));
    WlArgs l{};
    l.text = text;
    l.n = nbytes;
    l.keys = keys;
    l.nkeys = nkeys;
    l.offsets = offsets;
    l.table = reinterpret_cast<WlSlot *>(base);
    l.ctl = reinterpret_cast<uint64_t *>(base + slots * sizeof(WlSlot));
    l.slots = slots;
    l.span = span;
    uint8_t *pad = reinterpret_cast<uint8_t *>(l.ctl + 4);
    if (nbytes > 0 && nbytes < 16) {
        l.text = pad;
        l.n = kWcPad;
    }
    if ((rc = ensure_pinned(ctx, 1)) == SPARKCL_OK &&
        (rc = launch_zero(base, zero_bytes, s)) == SPARKCL_OK &&
        (nbytes == 0 || nbytes >= 16 ||
         (rc = launch_wc_pad(text, nbytes, pad, s)) == SPARKCL_OK) &&
        (rc = launch_wordcount_locate(l, grid, s)) == SPARKCL_OK) {
        hipError_t e = hipMemcpyAsync(ctx->pinned, l.ctl, 16, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipStreamSynchronize(s);
        if (e != hipSuccess)
            rc = fail_hip(e, "word locate");
    } else if (rc != SPARKCL_OK) {
        (void)hipStreamSynchronize(s);
        rc = fail(rc, "word-locate launch failed");
    }
    ctx->arena.release(off);
    if (rc != SPARKCL_OK)
        return rc;
    uint64_t ctl[2];
    std::memcpy(ctl, ctx->pinned, sizeof(ctl));
    if (ctl[1])
        return fail(SPARKCL_EINVAL, "a key appears twice in keys");
    return SPARKCL_OK;
}

} // extern "C"
