// Test shim: the two ways to a factor's rank (tsf_bits.h).
#include "../paper_2511_20317_amd/csrc/tsf_bits.h"

extern "C" int shim_rank_entries(uint64_t d, uint64_t s, int rows, int cols, int z2)
{
    int32_t M[64];
    return factor_rank(d, s, rows, cols, z2 != 0, M);
}
extern "C" int shim_rank_masks(uint64_t d, uint64_t s, int rows, int cols, int z2)
{
    uint64_t starts = 0;
    for (int r = 0; r < rows; ++r) starts |= 1ull << (r * cols);
    return factor_rank_masks(d, s, rows, cols, z2 != 0, starts, (65536u + cols - 1) / cols);
}
