// tsf_launch.h -- the strategy and lanes per walk of a walk call that leaves them
// open, and what the autotuner tries and remembers (host code, no HIP).
#pragma once
#include "../../include/tsf.h"
#include "tsf_internal.h"

#include <stddef.h>
#include <vector>

// LDS stride per factor kind: capacity rounded up to even (to a multiple of 4 for
// the indexed strategy, which reads four terms at a time).
inline int lds_stride(int cap, bool ix) { return ix ? (cap + 3) & ~3 : cap + (cap & 1); }

// LDS of a walk: its terms, and for the indexed strategy 3 match masks per term
// (rows of `capacity` masks, not padded).  Factors of at most 16 entries are
// packed there: digits and signs in one 32-bit word.
inline size_t walk_lds(int cap, int max_len, bool ix)
{
    const size_t factor = max_len > 32 ? 16 : ix && max_len <= 16 ? 4 : 8;
    return (size_t)lds_stride(cap, ix) * 3 * factor + (ix ? (size_t)cap * 3 * 8 : 0);
}

// Rounds in which 256 CUs work through n walks of `lanes` lanes each, one
// wavefront per workgroup: a CU has 160 KiB of LDS, handed out in pieces of 1,280
// bytes, and the attempt-parallel kernels' registers let 16 wavefronts in.
inline int64_t launch_rounds(int64_t n, int lanes, size_t lds_per_walk)
{
    const int64_t wave = ((int64_t)(64 / lanes) * (int64_t)lds_per_walk + 1279) / 1280 * 1280;
    const int64_t fit = 160 * 1024 / wave, per_cu = fit < 1 ? 1 : fit > 16 ? 16 : fit;
    const int64_t walks = 256 * per_cu * (64 / lanes);
    return (n + walks - 1) / walks;
}

// Times are us per iteration of the whole batch, rank objective and ternary where
// not said otherwise.
//  * Small batches do not fill the 1,024 SIMDs, and an iteration's latency
//    counts: the fewer walks share a wavefront, the less each waits for the
//    others' branches.  Up to 4,096 walks 32 lanes each ((2,2,2), 256 walks:
//    2.1 with 32 lanes, 2.3 with 8), up to 8,192 walks 16 lanes (capacity 58:
//    3.0 against 3.5); one wavefront per walk with fingerprints where the
//    indexed kernels' masks are long and no SIMD has more than three wavefronts
//    (capacity 58, 1,024 walks: 2.1 against 2.5 with 32 lanes; 3,072 walks 2.5
//    against 2.7; 4,096 walks 2.8 against 2.7), or one, from 33 terms (capacity
//    35, 1,024 walks: 2.0 against 2.1; 26: 2.2 against 2.1).
//  * Beyond 64 terms the indexed kernels end and the attempts of the
//    attempt-parallel ones scan every term: one wavefront per walk is faster
//    until the chip is full (capacity 88: 4,096 walks 2.9 against 7.1 with 16
//    lanes, 12,288 walks 7.2 against 9.6, 32,768 walks 18.8 against 18.7; at
//    16,384 walks 9.6 and 9.7, but with fewer terms in the walks, as in batches
//    of several formats, only the scans become shorter), and always above 96
//    terms, where their partner scans and LDS grow (capacity 108, 65,536 walks:
//    37 against 49).  The additions objective needs no reduction scan, so up to
//    76 terms its attempt-parallel kernels win earlier (capacity 72: 10,752
//    walks 5.3 against 5.6 with 8 lanes, in Z2 4.6 against 4.5; 12,288 walks 5.8
//    against 5.6, in Z2 4.9 against 4.5; capacity 83: 5.8 against 6.7).
//  * Full chips: 8 lanes, or 16 where a walk's LDS leaves a CU too few
//    wavefronts of eight walks (capacity 56, 65,536 walks: 14.3 against 15.0;
//    capacity 88: 36.5 against 38.9; capacity 44: 13.4 against 11.4) -- as long
//    as 16 lanes do not cost one more round of resident wavefronts: a CU holds
//    16 of them, 64 walks, but at 53 terms 9 wavefronts of eight walks, 72
//    (capacity 53, 18,432 walks: 4.0 with 8 lanes, 5.9 with 16; 36,864 walks
//    8.1 and 9.4; capacity 72, 20,480 walks 8.5 and 12.1, 40,960 walks 17.1 and
//    19.8, 49,152 walks, three rounds of either, 22.3 and 22.2).  The additions
//    objective gains nothing from 16 lanes beyond 64 terms (capacity 68, 14,336
//    walks: 5.7 with 8, 6.1 with 16; capacity 88: 7.4 and 7.7; 32,768 walks 15.0
//    and 15.1) but at capacities 80 and 96, where the walks of a wavefront meet
//    in the same LDS banks (capacity 80, 16,384 walks: 8.7 and 8.3).
inline tsf_launch default_launch(const tsf_walk_params *prm, const tsf_walk_batch *b)
{
    const bool wide = b->max_len > 32, rank = prm->objective == TSF_OBJ_RANK;
    const int cap = b->capacity, n = b->n_walks;
    const bool ix = cap <= 64;
    if (ix) {
        if (!wide && cap > 32 && n <= (cap > 40 ? 3072 : 1024)) return tsf_launch{64, 0, 2};
        if (n <= 8192) return tsf_launch{n <= 4096 ? 32 : 16, 0, 3};
    } else if (wide || cap > 96 || n <= (rank || cap > 76 ? 12288 : 11264)) {
        return tsf_launch{64, 0, 2};
    }
    const size_t lds = walk_lds(cap, b->max_len, ix);
    const bool sixteen = (ix ? wide || cap > 48 : rank || (cap % 16 == 0 && n <= 16384)) &&
                         launch_rounds(n, 16, lds) <= launch_rounds(n, 8, lds);
    return tsf_launch{sixteen ? 16 : 8, 0, ix ? 3 : 1};
}

// The shape of a walk call: what its launch names, and the library's choice where it
// leaves the strategy and the lanes open.  With only one of them named: the indexed
// strategy up to 64 terms, the attempt-parallel one up to 128 terms of 32-bit
// factors, the term-parallel one beyond; 8 lanes, 64 of the term-parallel one.
// Checked calls take the shape that an unchecked one takes, or one of the shapes
// whose lanes follow from the strategy: other kernels are not built with the checks.
struct WalkShape {
    int strategy, lanes, waves;
};
inline tsf_status walk_shape(const tsf_walk_params *prm, const tsf_walk_batch *b,
                             const tsf_launch *launch, bool checked, WalkShape &w)
{
    int strategy = launch ? launch->strategy : 0, lanes = launch ? launch->lanes_per_walk : 0;
    const int waves = launch && launch->waves_per_block ? launch->waves_per_block : 1;
    if (strategy < 0 || strategy > 3)
        return tsf_fail(TSF_E_ARG, "strategy %d not in 0..3", strategy);
    const bool open = strategy == 0 && lanes == 0;
    if (open) {
        const tsf_launch d = default_launch(prm, b);
        strategy = d.strategy;
        lanes = d.lanes_per_walk;
    }
    if (strategy == 0)
        strategy = b->capacity <= 64 ? 3 : b->capacity <= 128 && b->max_len <= 32 ? 1 : 2;
    const bool ap = strategy != 2;
    if (strategy == 3 && b->capacity > 64)
        return tsf_fail(TSF_E_CAPACITY, "the indexed strategy needs capacity <= 64");
    if (ap && b->capacity > 128)
        return tsf_fail(TSF_E_CAPACITY, "the attempt-parallel strategy needs capacity <= 128");
    if (lanes == 0) lanes = ap ? 8 : 64;
    if (lanes != 4 && lanes != 8 && lanes != 16 && lanes != 32 && lanes != 64)
        return tsf_fail(TSF_E_ARG, "lanes_per_walk %d not in {4,8,16,32,64}", lanes);
    if (lanes == 4 && !ap)
        return tsf_fail(TSF_E_ARG, "4 lanes per walk only with the attempt-parallel strategies");
    if (ap && lanes == 64)
        return tsf_fail(TSF_E_ARG, "the attempt-parallel strategies use 4 to 32 lanes per walk");
    if (waves < 1 || waves > 4)
        return tsf_fail(TSF_E_ARG, "waves_per_block %d not in 1..4", waves);
    if (checked && !open && lanes != (ap ? 8 : 64))
        return tsf_fail(TSF_E_ARG, "checked walks use %d lanes per walk with this strategy",
                        ap ? 8 : 64);
    w = WalkShape{strategy, lanes, waves};
    return TSF_OK;
}

// What tsf_autotune times: 4 to 16 lanes of the attempt-parallel strategies, 16 to
// 64 of the term-parallel one and the launch that a call without tuning takes, so
// that tuning never ends with a slower one; 1, 2 and 4 wavefronts per workgroup.
inline std::vector<tsf_launch> tune_candidates(const tsf_walk_params *prm, const tsf_walk_batch *b)
{
    const tsf_launch d = default_launch(prm, b);
    std::vector<tsf_launch> c;
    for (int wpb : {1, 2, 4}) {
        const auto add = [&](int lanes, int strategy) {
            if (lanes != d.lanes_per_walk || strategy != d.strategy)
                c.push_back(tsf_launch{lanes, wpb, strategy});
        };
        for (int st : {3, 1})
            if (b->capacity <= (st == 3 ? 64 : 128))
                for (int g : {4, 8, 16}) add(g, st);
        for (int g : {16, 32, 64}) add(g, 2);
        c.push_back(tsf_launch{d.lanes_per_walk, wpb, d.strategy});
    }
    return c;
}

// A tuned launch and the batches that it serves.
struct TuneEntry {
    int32_t capacity, max_len, mode, objective, size_class;
    tsf_launch launch;
    bool used;
};

inline int size_class(int n_walks)
{
    int c = 0;
    while (n_walks > 1 && c < 30) {
        n_walks >>= 1;
        ++c;
    }
    return c;
}

inline TuneEntry tune_entry(const tsf_walk_params *prm, const tsf_walk_batch *b,
                            const tsf_launch &launch)
{
    return TuneEntry{b->capacity,    b->max_len, b->mode, prm->objective, size_class(b->n_walks),
                     launch, true};
}

inline bool tune_serves(const TuneEntry &e, const tsf_walk_params *prm, const tsf_walk_batch *b)
{
    return e.used && e.capacity == b->capacity && e.max_len == b->max_len && e.mode == b->mode &&
           e.objective == prm->objective && e.size_class == size_class(b->n_walks);
}
