// Test shim: the launch choices (tsf_launch.h).
#include "../paper_2511_20317_amd/csrc/tsf_launch.h"

#include <cstring>

tsf_status tsf_fail(tsf_status st, const char *, ...) { return st; }

static void batch(int cap, int max_len, int n, int objective, tsf_walk_params &prm,
                  tsf_walk_batch &b)
{
    std::memset(&prm, 0, sizeof prm);
    std::memset(&b, 0, sizeof b);
    prm.objective = objective;
    b.capacity = cap;
    b.max_len = max_len;
    b.n_walks = n;
}

// the default: 100 * strategy + lanes
extern "C" int shim_default(int cap, int max_len, int n, int objective)
{
    tsf_walk_params prm;
    tsf_walk_batch b;
    batch(cap, max_len, n, objective, prm, b);
    const tsf_launch l = default_launch(&prm, &b);
    return 100 * l.strategy + l.lanes_per_walk;
}

// the autotuner's launches: 1000 * strategy + 10 * lanes + wavefronts per
// workgroup each; returns their number
extern "C" int shim_candidates(int cap, int max_len, int n, int objective, int *out, int room)
{
    tsf_walk_params prm;
    tsf_walk_batch b;
    batch(cap, max_len, n, objective, prm, b);
    int k = 0;
    for (const tsf_launch &l : tune_candidates(&prm, &b)) {
        if (k < room) out[k] = 1000 * l.strategy + 10 * l.lanes_per_walk + l.waves_per_block;
        ++k;
    }
    return k;
}

// whether a launch tuned for one batch serves another
extern "C" int shim_serves(const int *tuned, const int *other)
{
    tsf_walk_params p, q;
    tsf_walk_batch a, b;
    batch(tuned[0], tuned[1], tuned[2], tuned[3], p, a);
    batch(other[0], other[1], other[2], other[3], q, b);
    a.mode = tuned[4];
    b.mode = other[4];
    return tune_serves(tune_entry(&p, &a, tsf_launch{8, 1, 1}), &q, &b);
}

// the shape of a call: 1000 * strategy + 10 * lanes + wavefronts, or its status
extern "C" int shim_shape(int cap, int max_len, int n, int objective, int strategy, int lanes,
                          int waves, int checked)
{
    tsf_walk_params prm;
    tsf_walk_batch b;
    batch(cap, max_len, n, objective, prm, b);
    const tsf_launch l{lanes, waves, strategy};
    WalkShape w;
    const tsf_status st = walk_shape(&prm, &b, &l, checked != 0, w);
    return st ? st : 1000 * w.strategy + 10 * w.lanes + w.waves;
}
