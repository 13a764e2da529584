// How the library covers one plain launch (plan_gen), for the tests: which kernel, blocks,
// segments and rate a call of these sizes, at this output address, takes; the order a served or
// an API batch runs in (serve_order, batch_order). Host code only.
#include "internal.h"

extern "C" void plan_query(const rngx_launch *cfg, int u32, int star, uint32_t n, uint32_t iters,
                           uint64_t out, int in_place, uint32_t *v)
{
    const rngx::GenPlan p =
        rngx::plan_gen(*cfg, u32 != 0, star != 0, n, iters,
                       reinterpret_cast<const void *>((uintptr_t)out), in_place != 0);
    v[0] = p.cfg.block;
    v[1] = p.cfg.chunks;
    v[2] = p.cfg.nontemporal;
    v[3] = p.cfg.pace_gbs;
    v[4] = p.aligned16;
    v[5] = p.scheduled;
    v[6] = p.shift;
    v[7] = p.segs;
    v[8] = p.seg_rows;
}

extern "C" void serve_order_query(uint64_t values, rngx_batch_cfg *cfg)
{
    *cfg = rngx::serve_order(values);
}

// The API's default configuration; anchors: whether there is memory for the sweep order's.
static const rngx_batch_cfg kDefault{16, 4, 0, 1, 16, 0, 0, 32, 8, 6250};
extern "C" void batch_order_query(uint64_t values, int anchors, rngx_batch_cfg *cfg)
{
    *cfg = rngx::batch_order(kDefault, values, anchors != 0);
}

// One batch, whatever its size, as the default configuration runs a large one without memory for
// anchors; returns when it is done.
extern "C" int batch_without_anchors(const rngx_req *reqs, uint32_t m, uint64_t *out,
                                     uint64_t out_cap)
{
    const rngx_batch_cfg cfg = rngx::batch_order(kDefault, ~(uint64_t)0, false);
    rngx::BatchSlot slot;
    rngx_batch_cfg run;
    uint64_t total = 0;
    int rc = rngx::batch_stage(slot, reqs, m, out, out_cap, cfg, true, &run, &total);
    if (rc == RNGX_OK)
        rc = rngx::batch_launch(slot, run, false, nullptr);
    rngx::release_slot(slot);
    return rc;
}

extern "C" uint64_t anchor_room_query(uint64_t need) { return rngx::anchor_room(need); }

// Every place stage_tail gives for wavefronts of W columns, chunks of E words and lines of L, over
// all columns left in the row and all line offsets: how many lie outside the stage, or are not
// the word that the lane stores.
extern "C" uint32_t stage_tail_faults(uint32_t E, uint32_t L, uint32_t W)
{
    uint32_t faults = 0;
    for (uint32_t cols = 1; cols < W + L; ++cols)
        for (uint32_t d = 0; d < L; ++d)
            for (uint32_t lane = 0; lane < 64; ++lane) {
                const uint32_t lim = d >= cols ? 0 : cols - d;
                const uint32_t at = rngx::stage_tail(d, lim, lane, E, W + L);
                const bool stores = lane < lim % E && lim < W;
                faults += at >= W + L || (stores && at != d + lim - lim % E + lane);
            }
    return faults;
}

extern "C" uint64_t table_chunks_query(uint64_t m) { return rngx::table_chunks(m); }
