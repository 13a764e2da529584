// How a plain generate call is covered: which kernel, blocks, segments and rate
// its sizes, its output's alignment and the configured launch come to. Host
// code only; the kernels are in kernels.hip.
#include <algorithm>

#include "internal.h"

namespace rngx {

bool launch_cfg_valid(const rngx_launch &cfg)
{
    return cfg.block >= 64 && cfg.block <= 1024 && cfg.block % 64 == 0 &&
           (cfg.chunks == 1 || cfg.chunks == 2 || cfg.chunks == 4) && cfg.nontemporal <= 1 &&
           (cfg.pace_gbs == 0 || (cfg.pace_gbs >= 1000 && cfg.pace_gbs <= 20000));
}

GenPlan plan_gen(const rngx_launch &cfg, bool u32, bool star, uint32_t n, uint32_t iters,
                 const void *out, bool in_place)
{
    const uint64_t row = (uint64_t)n * (u32 ? 4 : 8), bytes = row * iters;
    const uintptr_t at = reinterpret_cast<uintptr_t>(out) | (iters > 1 ? row : 0);
    // On the lines: rows that start on 128-byte lines or in their middle, as the
    // memory takes halves whole (332,808 x 103 u64 46.6 us, 56.2 staged; u32
    // 19,200,016 x 6 115 and 144).
    const bool lines = at % 64 == 0;
    GenPlan p;
    p.cfg = cfg;
    p.seg_rows = iters;
    p.aligned16 = at % 16 == 0;
    const bool heaviest = u32 && star, heavy = u32 || star;
    const uint64_t waves = (row + 1023) / 1024;
    // Rows off the 128-byte lines are staged where the memory takes the
    // values: stored where it lies, such a row writes its lines in parts
    // (10^6 + 3 states x 256 u64: 6.89 TB/s staged, 4.13 not; 10^6 + 2, 16-byte
    // aligned: 6.9 and 4.3). Below 256 MiB the Infinity Cache puts the parts
    // together and staging only costs (2^22 + 1 x 8: 54.7 us staged, 51.6 not).
    // It still does most of that somewhat above, for rows that are not 16-byte
    // aligned and so take no schedule unstaged: of 4-byte words from 2,304
    // wavefronts on up to 352 MiB, very wide rows up to 416 MiB, of 8-byte
    // words up to 512 MiB in the rows that would be staged in two or three
    // segments (us, where it lies and staged: 179,201 x 216 u64 56.5
    // and 64.9, 332,801 x 116 53.0 and 60.2, but 537,601 x 72 61.0 and 52.3;
    // 7,040,001 x 6 69.0 and 72.0; u32 4,096,001 x 18 56.5 and 64.8; 2,304,001 x
    // 33 57.4 and 63.8, x 46 104.7 and 80.4).
    uint64_t stage_from = kCacheBytes;
    if (!p.aligned16) {
        if (u32)
            stage_from = kCacheBytes / 8 * (waves < 2304 ? 8 : waves < 64000 ? 11 : 13);
        else if (waves >= (star ? 1200 : 900))
            stage_from = kCacheBytes / 8 * (waves < 3072 ? 16 : waves < 24000 ? 8 : 13);
    }
    // Staged calls keep two copies of the states. Where one fits in that cache
    // and two do not, a few iterations are better off in place, to up to 12 of
    // 16-byte aligned rows and 4 of others of 8-byte words, beyond that 2 of the
    // latter (us, in place and staged: 32,000,002 x 3 u64 193 and 259, x 6 332
    // and 403, x 13 742 and 748; 28,160,004 x 6 u32 174 and 217; 25,600,001 x 3
    // u64 193 and 211, x 5 298 and 293).
    const uint64_t states = 8ull * n;
    uint64_t few_rows = 0;
    if (states > kCacheBytes)
        few_rows = p.aligned16 || u32 ? 0 : 2;
    else if (states > kCacheBytes / 2)
        few_rows = p.aligned16 ? 12 : u32 ? 0 : 4;
    stage_from = std::max(stage_from, few_rows * row);
    // Without a schedule the staged kernel needs wide rows to fill the device
    // and outputs well beyond that cache (block 256, 1 chunk, 39,240 x 1,207 u64
    // 307 us staged, 97 not; 512 and 2, 300,001 x 224 114 and 92, x 374 190 and
    // 230).
    if (!cfg.pace_gbs)
        stage_from = waves >= 2048 ? kCacheBytes / 2 * 5 : UINT64_MAX;
    // Narrow rows, below 4 MiB (3 on the lines, where 3.4 MiB x 500 is as fast
    // as configured, but for the heaviest steps): as configured they would leave
    // wavefronts or whole compute units without work, so every lane takes one
    // chunk and blocks are small.
    // Too few wavefronts to fall in with the memory's rate, and at least 64
    // iterations (off the lines 48, scrambled 32, of 4-byte words 28, where both
    // 24; a segment's jump costs about 2.5 us): the iterations are cut into
    // segments of at least 8. (Off the lines, us a call: 1,001 x 28 u64 9.9 in
    // one, 11.6 in three; x 64 13.5 and 11.4; 1,001 x 24 u32 10.9 and 11.8.)
    //
    // How many: an aligned row of 1 KiB takes a wavefront about 55 ns, and at
    // least 480 of them hold the rate; about 755 where its words are 4 bytes,
    // twice the steps, or scrambled, 900 where both; staged, a row takes 220 ns
    // and more. More segments than that are more places written at once, which the
    // memory takes more slowly (4,096 x 10,000 u64: 54 us in 16 segments, 60
    // in 32, 68 in 128, 1,650 in one of 512 x 2; 12,800 x 3,276: 53 in 5, 62 in
    // 6; 65,536 x 640: 51 in two, 63 in one; scrambled 4,096 x 10,000: 73 in
    // 16, 53 in 24, 61 in 32; u32 51,200 x 1,638: 66 in 3, 68 in 5). Outputs
    // that the Infinity Cache takes wait for the rows alone, and run at 1,024
    // (4,096 x 1,000: 9.6 us, 11.4 in half as many); unaligned, they are better
    // off word by word where one segment keeps the device busy (262,273 x 99
    // u64: 34 us, 40 in two staged ones; 65,537 x 399: 65 and 44 in three).
    // Rows off the lines that are stored where they lie run narrow in outputs
    // that the cache holds. Beyond (in place) and where they take no schedule
    // (not 16-byte aligned) they run as configured from 768 to 1,800 wavefronts
    // on: in place, 262,146 x 500 u64 231 us so, 296 narrow; 163,842 x 800 255
    // and 295; 65,538 x 1,000 178 and 121; u32 524,292 x 500 272 and 300;
    // 400,004 x 660 299 and 285.
    const bool bare = !lines && (in_place || bytes <= stage_from);
    const uint32_t wide = !bare ? (lines && !heaviest ? 3072u : 4096u)
                          : p.aligned16 && bytes <= kCacheBytes ? 4096u
                          : u32                                 ? 1800u
                          : star || p.aligned16                 ? 1200u
                                                                : 768u;
    const bool narrow = cfg.pace_gbs && iters >= 2 && waves < wide;
    const bool cached = bytes <= kCacheBytes * 3 / 4;
    const uint32_t least = lines ? 64u : heaviest ? 24u : u32 ? 28u : star ? 32u : 48u;
    if (narrow && !in_place && iters >= least) {
        uint64_t segs = 1;
        if (!lines && !(bytes <= stage_from && waves >= (heavy ? 1800u : 768u)))
            segs = ((u32 && !cached && waves >= 200 && waves < 1600 ? 6144 : 4096) + waves / 2) /
                   waves;
        else if (lines && cached && waves < 512)
            segs = (1024 + waves / 2) / waves;
        else if (lines && !cached && waves < 768)
            segs = std::max<uint64_t>(2, heavy ? ((heaviest ? 900 : 755) + waves / 2) / waves
                                               : (480 + waves - 1) / waves);
        segs = std::min<uint64_t>({segs, iters / 8, kMaxSegs});
        if (segs > 1) {
            p.seg_rows = (uint32_t)((iters + segs - 1) / segs);
            p.segs = (uint32_t)(((uint64_t)iters + p.seg_rows - 1) / p.seg_rows);
        }
    }
    p.shift = !in_place && !lines && iters >= 2 && (bytes > stage_from || p.segs > 1);
    // A few iterations of long rows end before a schedule orders anything;
    // they run as fast without one, or faster, up to 32 bytes a stream and up
    // to 48 where rows are on lines and the output is about the cache's size
    // (2^26 states x 4 u64 578 us free, 600 scheduled; 2^25 x 8 u32 229 and
    // 234; 10^7 x 12 u32 96 and 100, but 2,200,000 x 12 u32 26 and 24, and
    // 3,000,002 x 6 u64, off lines, 36 and 34; 2^24 x 8 u64 201 and 190).
    const bool mid = lines && bytes > kCacheBytes / 2 && bytes <= 2 * kCacheBytes;
    const bool few = !p.shift && !narrow && row / n * iters <= (mid ? 48u : 32u);
    p.scheduled = p.shift || (cfg.pace_gbs && iters >= 2 && p.aligned16 && !few);
    if (narrow && p.scheduled) {
        // Outputs well inside that cache run ahead of HBM's rate, so a
        // schedule only holds them back (131,072 x 100 u64: 5.25 TB/s free,
        // below 5.1 scheduled; 65,536 x 1,000: 5.5 free, 6.5 scheduled): up to
        // 192 MiB, of wide rows in one segment 64 MiB, as more wavefronts write
        // than the cache takes in any order (332,800 x 71 u64, 190 MB, 39.3 us
        // free, 34.3 scheduled; 243,200 x 97 38.9 and 34.5).
        const bool free =
            bytes <= (waves < 1280 || p.segs > 1 ? kCacheBytes / 4 * 3 : kCacheBytes / 4);
        // From 1,536 wavefronts blocks of 512 (262,144 x 1,000 u64: 303 us,
        // 322 with 256; below, 102,400 x 1,000 u32: 122 with 256, 131).
        p.cfg.chunks = 1;
        p.cfg.block =
            std::min(cfg.block, lines && !free && !heaviest && waves >= 1536 ? 512u : 256u);
        // Many segments: at most a rate that they hold, above which they fall
        // behind for good (at 6,000, 6,500 and 7,000 GB/s: 16,387 x 10,000
        // u64, 32 segments, 230, 214, 264 us; 4,099 x 10,000, 124, 66, 73, 79;
        // 131,073 x 2,000, 4, 354, 327, 308; 65,537 x 1,000 u32, 24, 48, 52,
        // 54; 131,073 x 2,000 u32, 12, 179, 166, 189; aligned, at 6,500, 6,750
        // and 7,000: 25,600 x 6,553 u32, 8, 107, 106, 123; 32,768 x 5,120, 6,
        // 107, 104, 104; scrambled u64 12,800 x 6,553, 8, 107, 104, 116).
        const uint32_t pace = cfg.pace_gbs;
        if (free)
            p.cfg.pace_gbs = 0;
        else if (lines && heavy && p.segs > 1)
            p.cfg.pace_gbs = std::min(pace, 6750u);
        else if (!lines && p.segs >= (u32 ? 20u : 64u))
            p.cfg.pace_gbs = std::min(pace, 6000u);
        else if (!lines && p.segs >= (u32 ? 2u : 6u))
            p.cfg.pace_gbs = std::min(pace, 6500u);
    }
    // Neighbouring wavefronts of one chunk share a line of each row off the
    // lines. Normal stores let the caches put it together (300,000 x 100 u64,
    // 16-byte aligned, 41.9 us, 60 non-temporal; with two chunks 54, narrow 42).
    if (p.scheduled && !p.shift && !lines && bytes <= kCacheBytes && p.cfg.chunks == 1)
        p.cfg.nontemporal = 0;
    return p;
}

} // namespace rngx
