// How the library covers one plain launch (plan_gen), for the tests: which kernel, blocks,
// segments and rate a call of these sizes, at this output address, takes; and the order a served
// batch runs in (serve_order). Host code only.
#include "internal.h"

extern "C" void plan_query(const rngx_launch *cfg, int u32, int star, uint32_t n, uint32_t iters,
                           uint64_t out, uint32_t *v)
{
    const rngx::GenPlan p = rngx::plan_gen(*cfg, u32 != 0, star != 0, n, iters,
                                           reinterpret_cast<const void *>((uintptr_t)out));
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
