// Array-valued ReduceCL (sec. 3.1.3; Fig 3; SparkCLVectorAdd, sec. 3.2.2): the
// RDD's elements are float arrays of one length, folded by a two-input
// combiner along a fixed pairwise tree.  Plans (leaf tables, passes and their
// intermediate rows) are cached in the context like the reduce plans.
#include <algorithm>
#include <cstring>
#include <string>

#include "runtime.h"
#include "treeplan.h"

using namespace sparkcl;

namespace {

constexpr uint32_t kTreeMaxK = 1u << 24;

// Array reduces are keyed by kind (2: pointer table, 3: rows of one buffer),
// combiner, shape, output and the leaves (the table, or base and stride).
uint64_t tree_hash(int kind, uint32_t combiner, const float *const *arrays,
                   const float *base, uint64_t stride, uint32_t k, uint64_t len,
                   const float *out)
{
    uint64_t h = 0xCBF29CE484222325ull;
    h = fnv1a(h, &kind, sizeof(kind));
    h = fnv1a(h, &combiner, sizeof(combiner));
    h = fnv1a(h, &k, sizeof(k));
    h = fnv1a(h, &len, sizeof(len));
    h = fnv1a(h, &out, sizeof(out));
    h = fnv1a(h, &base, sizeof(base));
    h = fnv1a(h, &stride, sizeof(stride));
    return arrays ? fnv1a(h, arrays, sizeof(const float *) * k) : h;
}

bool tree_plan_matches(const Plan *p, int kind, uint64_t h, uint32_t combiner,
                       const float *const *arrays, const float *base, uint64_t stride,
                       uint32_t k, uint64_t len, const float *out)
{
    if (p->kind != kind || p->hash != h || p->combiner != combiner || p->len != len ||
        p->user_out != out || p->nleaves != k || p->leaf_base != base ||
        p->leaf_stride != stride)
        return false;
    return !arrays ||
           std::memcmp(p->leaves.data(), arrays, sizeof(const float *) * k) == 0;
}

// Builds the plan along the passes of tree_passes(); `least`: those that need
// the least scratch.
int build_tree_plan(sparkcl_ctx *ctx, uint32_t combiner, const float *const *arrays,
                    const float *base, uint64_t stride, uint32_t k, uint64_t len,
                    float *out, hipStream_t stream, bool least, Plan **res)
{
    std::unique_ptr<Plan> p(new Plan);
    p->kind = arrays ? 2 : 3;
    p->combiner = combiner;
    p->len = len;
    p->user_out = out;
    p->nleaves = k;
    p->leaf_base = base;
    p->leaf_stride = stride;
    if (arrays) {
        p->leaves.assign(arrays, arrays + k);
        for (uint32_t i = 0; i < k; ++i) {
            if (!arrays[i])
                return fail(SPARKCL_EINVAL, "array " + std::to_string(i) + " is NULL");
            if ((uintptr_t)arrays[i] & 3u)
                return fail(SPARKCL_EINVAL, "arrays must be 4-byte aligned");
        }
    }
    const std::vector<TreePass> passes = tree_passes(k, len, (uint32_t)ctx->cus, least);
    for (const TreePass &t : passes) {
        TreeArgs a{};
        a.len = len;
        a.count = t.count;
        a.chunk = t.chunk;
        a.cpt = t.cpt;
        a.threads = t.threads;
        a.groups = t.groups;
        a.cols = t.cols;
        p->passes.push_back(a);
    }

    // scratch: rows of pass 0 in buffer 0, of pass 1 in buffer 1, then alternate
    float *scratch[2] = {nullptr, nullptr};
    for (size_t i = 0; i + 1 < p->passes.size() && i < 2; ++i) {
        const uint64_t bytes = (uint64_t)passes[i].rows * len * 4;
        void *q = nullptr;
        int rc = arena_alloc(ctx, p.get(), std::max<uint64_t>(bytes, 256), &q);
        if (rc != SPARKCL_OK) {
            Plan *raw = p.release();
            free_plan(ctx, raw);
            return rc;
        }
        scratch[i] = static_cast<float *>(q);
    }
    void *dptrs = nullptr;
    if (arrays) {
        int rc = arena_alloc(ctx, p.get(), sizeof(const float *) * k, &dptrs);
        if (rc != SPARKCL_OK) {
            Plan *raw = p.release();
            free_plan(ctx, raw);
            return rc;
        }
    }
    for (size_t i = 0; i < p->passes.size(); ++i) {
        TreeArgs &a = p->passes[i];
        if (i == 0) {
            a.ptrs = static_cast<const float *const *>(dptrs);
            a.base = base;
            a.stride = stride;
        } else {
            a.base = scratch[(i - 1) % 2];
            a.stride = len;
        }
        a.out = (i + 1 == p->passes.size()) ? out : scratch[i % 2];
    }
    if (arrays) {
        hipError_t e = hipMemcpyAsync(dptrs, p->leaves.data(), sizeof(const float *) * k,
                                      hipMemcpyHostToDevice, stream);
        if (e == hipSuccess)
            e = hipStreamSynchronize(stream);
        if (e != hipSuccess) {
            Plan *raw = p.release();
            free_plan(ctx, raw);
            return fail_hip(e, "upload of the array table");
        }
    }
    p->hash = tree_hash(p->kind, combiner, arrays, base, stride, k, len, out);
    *res = p.release();
    return SPARKCL_OK;
}

} // namespace

namespace {

int reduce_tree(sparkcl_ctx *ctx, uint32_t combiner, const float *const *arrays,
                const float *base, uint64_t stride, uint32_t k, uint64_t len, float *out,
                void *stream)
{
    int rc = check_ctx(ctx);
    if (rc != SPARKCL_OK)
        return rc;
    if (combiner != SPARKCL_VADD && combiner != SPARKCL_VMAX)
        return fail(SPARKCL_EINVAL, "combiner " + std::to_string(combiner) +
                                        " is not SPARKCL_VADD or SPARKCL_VMAX");
    if (k == 0 || (!arrays && !base))
        return fail(SPARKCL_EINVAL, "an array reduce needs at least one array");
    if (k > kTreeMaxK)
        return fail(SPARKCL_ETOOBIG, "more than 2^24 arrays");
    if (len > kMaxN)
        return fail(SPARKCL_ETOOBIG, "arrays longer than 2^40 elements");
    if (!arrays && (((uintptr_t)base & 3u) || (k > 1 && stride < len)))
        return fail(SPARKCL_EINVAL, "rows must be 4-byte aligned and row_stride >= len");
    if (len == 0)
        return SPARKCL_OK;
    if (!out)
        return fail(SPARKCL_EINVAL, "out is NULL");
    if ((uintptr_t)out & 3u)
        return fail(SPARKCL_EINVAL, "out must be 4-byte aligned");
    std::lock_guard<std::mutex> g(ctx->mu);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int kind = arrays ? 2 : 3;
    const uint64_t h = tree_hash(kind, combiner, arrays, base, stride, k, len, out);
    Plan *p = nullptr;
    for (auto it = ctx->plans.begin(); it != ctx->plans.end(); ++it)
        if (tree_plan_matches(*it, kind, h, combiner, arrays, base, stride, k, len, out)) {
            p = *it;
            ctx->plans.splice(ctx->plans.begin(), ctx->plans, it);
            break;
        }
    if (!p) {
        if (capturing(s))
            return fail(SPARKCL_EINVAL, "no cached plan for this call on a stream under capture: "
                                        "make the same call once before capturing");
        while (ctx->plans.size() >= kMaxPlans)
            evict_one(ctx);
        // an arena that can't hold the fastest plan's rows may hold the one
        // that leaves the fewest
        rc = build_tree_plan(ctx, combiner, arrays, base, stride, k, len, out, s, false, &p);
        if (rc == SPARKCL_ENOMEM)
            rc = build_tree_plan(ctx, combiner, arrays, base, stride, k, len, out, s, true, &p);
        if (rc != SPARKCL_OK)
            return rc;
        ctx->plans.push_front(p);
    }
    for (const TreeArgs &a : p->passes)
        if ((rc = launch_tree(a, combiner, s)) != SPARKCL_OK)
            return fail(rc, "array reduce launch failed");
    return SPARKCL_OK;
}

} // namespace

extern "C" {

int sparkcl_reduce_arrays(sparkcl_ctx *ctx, uint32_t combiner, const float *const *arrays,
                          uint32_t k, uint64_t len, float *out, void *stream)
{
    if (k && !arrays)
        return fail(SPARKCL_EINVAL, "arrays is NULL");
    return reduce_tree(ctx, combiner, arrays, nullptr, 0, k, len, out, stream);
}

int sparkcl_reduce_rows(sparkcl_ctx *ctx, uint32_t combiner, const float *base,
                        uint64_t row_stride, uint32_t k, uint64_t len, float *out,
                        void *stream)
{
    if (k && !base)
        return fail(SPARKCL_EINVAL, "base is NULL");
    return reduce_tree(ctx, combiner, nullptr, base, row_stride, k, len, out, stream);
}

} // extern "C"
