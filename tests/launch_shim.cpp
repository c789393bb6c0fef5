// Test shim: the launch choices (tsf_launch.h).
#include "../paper_2511_20317_amd/csrc/tsf_launch.h"

#include <cstring>

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
