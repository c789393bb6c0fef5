// walk.hip -- host side of the batched walks: walk-state initialisation,
// batch Brent verification on the GPU, and the launch of the walk kernels
// (walk_kernel.h, instantiated in walk_inst.hip).
#include "walk_kernel.h"
#include "tsf_internal.h"
#include "tsf_launch.h"
#include "tsf_meta.h"

#include <cstring>
#include <mutex>
#include <vector>

namespace tsfk {
KernelFn pick_kernel_w0_z0(int g, int s, int strategy, bool chk);
KernelFn pick_kernel_w0_z1(int g, int s, int strategy, bool chk);
KernelFn pick_kernel_w1_z0(int g, int s, int strategy, bool chk);
KernelFn pick_kernel_w1_z1(int g, int s, int strategy, bool chk);
}  // namespace tsfk

namespace {
using namespace tsfk;

// One wavefront per walk: validate the start scheme, then cur := best :=
// start and clear the walk's state.  A factor's two masks are 16 bytes, so a
// lane moves factors lane, lane+64, ... of the scheme with one load and two
// stores each, all coalesced.  16,384 exploratory walks 83 -> 34 us, 65,536
// walks of the mixed formats 374 -> 147 us (576 MB, 3.9 TB/s); a term per lane,
// whose 8-byte accesses lay 48 bytes apart, wasted most of each access.
__global__ void __launch_bounds__(256) init_kernel(tsf_walk_header *hdr, uint64_t *cur,
                                                   uint64_t *best, const uint64_t *start,
                                                   int32_t n_walks, int32_t cap)
{
    const int64_t walk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (walk >= n_walks) return;
    tsf_walk_header *h = hdr + walk;
    const int m = h->m, n = h->n, p = h->p, r0 = h->start_rank;
    const bool z2 = h->mode == 1;
    bool ok = m >= 1 && n >= 1 && p >= 1 && (h->mode == 0 || h->mode == 1) && r0 >= 0 &&
              r0 <= h->r_cap && h->r_cap <= cap;
    const int len[3] = {m * n, n * p, p * m};
    ok = ok && len[0] <= 64 && len[1] <= 64 && len[2] <= 64;
    const size_t base = (size_t)walk * cap * 6;
    // 16-byte accesses where the buffers allow them
    const bool al = ((reinterpret_cast<uintptr_t>(start) | reinterpret_cast<uintptr_t>(cur) |
                      reinterpret_cast<uintptr_t>(best)) & 15) == 0;
    bool bad = false;
    int nnz = 0;  // non-zero coefficients of the start scheme
    if (ok) {
        int X = lane % 3;
        for (int q = lane; q < 3 * r0; q += 64) {
            ulonglong2 v;
            const size_t o = base + 2 * (size_t)q;
            if (al)
                v = *reinterpret_cast<const ulonglong2 *>(start + o);
            else
                v = make_ulonglong2(start[o], start[o + 1]);
            const uint64_t d = v.x, s = v.y;
            const int L = X == 0 ? len[0] : X == 1 ? len[1] : len[2];
            const uint64_t lim = L == 64 ? ~0ull : ((1ull << L) - 1);
            if (d == 0 || (s & ~d) || (d & ~lim) || (z2 && s)) bad = true;
            if (!z2 && X < 2 && (s & (d & (~d + 1)))) bad = true;  // not normalised
            nnz += __builtin_popcountll(d);
            if (al) {
                *reinterpret_cast<ulonglong2 *>(cur + o) = v;
                *reinterpret_cast<ulonglong2 *>(best + o) = v;
            } else {
                cur[o] = best[o] = d;
                cur[o + 1] = best[o + 1] = s;
            }
            X = X == 2 ? 0 : X + 1;  // 64 mod 3 = 1
        }
    }
    const bool any_bad = __ballot(bad) != 0;
    for (int off = 32; off > 0; off >>= 1) nnz += __shfl_xor(nnz, off);
    if (lane == 0) {
        h->done = (!ok || any_bad) ? -2 : 0;
        h->rank = r0;
        h->best_rank = r0;
        h->n_rec = 0;
        h->best_nnz = nnz;
        h->t = 0;
        h->plateau_start = 0;
        for (int c = 0; c < 12; ++c) h->counters[c] = 0;
        h->params_hash = 0;
        h->reserved = 0;
    }
}

// Brent verification (Eq. 1, C^T form of Sec. 3.1), a wavefront per scheme.
// A lane owns an (a, b) pair of entries of u and v and adds up the row
// sum_l u_l[a] v_l[b] w_l of the tensor for all entries of w at once, in
// bit-sliced two's complement: plane k holds bit k of every entry's sum.  The
// terms of a pair are the intersection of two sets: for every entry of u and v
// the terms that have it, and those that have it negative, are 64-bit words
// built with ballots.  So the work is the number of non-zero u_l[a] v_l[b]; the
// carry steps of a pair's terms bound it.  65,536 schemes of the mixed formats
// take 256 us; building the tensor with LDS atomics, an atomic for every
// non-zero product and two barriers for every entry of u, took 1,292 us.  Ten planes hold the sums of up to
// 512 terms modulo 1,024.  A mask bit that encodes no coefficient (a digit at
// or beyond the factor's length, a sign without its digit, any sign of a Z2
// scheme) counts as one violation of its own and takes no part in the tensor.
// The digits and signs of w take 32-bit words where w has at most 32 entries.
constexpr int kPlanes = 10;
// LDS of a wavefront, per 64 terms: w's masks and the four sets of 64 entries
constexpr size_t kVerifyLds = 64 * 16 + 4 * 64 * 8;

// adds +1 to the entries of `up` and -1 to those of `down`, from plane Z on;
// carries and borrows run on while there are any (in Z2 only plane 0 counts)
template <typename T, int Z>
__device__ __forceinline__ void add_planes(T (&plane)[kPlanes], T up, T down, bool z2)
{
    const T x = plane[Z];
    plane[Z] = x ^ (up | down);
    if constexpr (Z + 1 < kPlanes) {
        up &= x;
        down &= ~x;
        if (!z2 && (up | down) != 0) add_planes<T, Z + 1>(plane, up, down, z2);
    }
}

// violations in the rows of this lane's pairs (a, b)
template <typename T>
__device__ __forceinline__ int verify_pairs(const T *W, const uint64_t *Ud, const uint64_t *Us,
                                            const uint64_t *Vd, const uint64_t *Vs, int all,
                                            int words, int m, int n, int p, bool z2)
{
    const int Lv = n * p, pairs = m * n * Lv;
    int bad = 0;
    for (int pair = threadIdx.x & 63; pair < pairs; pair += 64) {
        const int a = pair / Lv, b = pair - a * Lv;
        T plane[kPlanes];
#pragma unroll
        for (int k = 0; k < kPlanes; ++k) plane[k] = 0;
        for (int k = 0; k < words; ++k) {
            uint64_t terms = Ud[a * all + k] & Vd[b * all + k];
            const uint64_t neg = Us[a * all + k] ^ Vs[b * all + k];
            for (; terms; terms &= terms - 1) {
                const int e = __builtin_ctzll(terms), l = 64 * k + e;
                const T d = W[2 * l];
                // digits of -1 and +1 of this term
                const T sg = W[2 * l + 1] ^ ((neg >> e) & 1 ? d : (T)0);
                add_planes<T, 0>(plane, d & ~sg, sg, z2);
            }
        }
        const int a1 = a / n, a2 = a - a1 * n, b1 = b / p, b2 = b - b1 * p;
        T diff = plane[0] ^ (a2 == b1 ? (T)1 << (b2 * m + a1) : (T)0);
#pragma unroll
        for (int k = 1; k < kPlanes; ++k) diff |= plane[k];
        bad += __builtin_popcountll((uint64_t)diff);
    }
    return bad;
}

// per entry e of a factor the lanes' terms that have it (D) and have it
// negative (S): entry e's words go to lane e, which writes them
__device__ __forceinline__ void entry_sets(uint64_t d, uint64_t s, int L, uint64_t *D, uint64_t *S,
                                           int all)
{
    const int lane = threadIdx.x & 63;
    uint64_t wd = 0, ws = 0;
    for (int half = 0; half < 2; ++half) {
        const uint32_t hd = (uint32_t)(d >> (32 * half)), hs = (uint32_t)(s >> (32 * half));
        const int end = L - 32 * half < 32 ? L - 32 * half : 32;
        for (int e = 0; e < end; ++e) {
            const uint64_t bd = __ballot((hd & (1u << e)) != 0), bs = __ballot((hs & (1u << e)) != 0);
            const bool mine = lane == 32 * half + e;
            wd = mine ? bd : wd;
            ws = mine ? bs : ws;
        }
    }
    if (lane < L) {
        D[lane * all] = wd;
        S[lane * all] = ws;
    }
}

__global__ void __launch_bounds__(256) verify_kernel(const tsf_walk_header *hdr,
                                                     const uint64_t *schemes, int32_t cap,
                                                     int32_t n_walks, int32_t which,
                                                     int64_t *n_violated)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char verify_smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (q >= n_walks) return;
    const tsf_walk_header *h = hdr + q;
    const int m = h->m, n = h->n, p = h->p;
    const int rank = which == 0 ? h->rank : which == 1 ? h->best_rank : h->start_rank;
    const bool z2 = h->mode == 1;
    const int Lu = m * n, Lv = n * p, Lw = p * m;
    if (m < 1 || n < 1 || p < 1 || Lu > 64 || Lv > 64 || Lw > 64 || rank < 0 || rank > cap) {
        if (lane == 0) n_violated[q] = -1;
        return;
    }
    const int words = (rank + 63) / 64, all = (cap + 63) / 64;
    unsigned char *mem = verify_smem + (size_t)wave * all * kVerifyLds;
    uint64_t *Ud = reinterpret_cast<uint64_t *>(mem + (size_t)all * 64 * 16);
    uint64_t *Us = Ud + 64 * all, *Vd = Us + 64 * all, *Vs = Vd + 64 * all;
    uint64_t *W64 = reinterpret_cast<uint64_t *>(mem);  // (digits, signs) of w per term
    uint32_t *W32 = reinterpret_cast<uint32_t *>(mem);
    const uint64_t *sc = schemes + (size_t)q * cap * 6;
    const auto mask = [](int L) { return L == 64 ? ~0ull : (1ull << L) - 1; };
    const uint64_t lims[3] = {mask(Lu), mask(Lv), mask(Lw)};
    const bool narrow = Lw <= 32;
    int bad = 0;
    for (int k = 0; k < words; ++k) {
        const int l = 64 * k + lane;
        uint64_t f[6] = {0, 0, 0, 0, 0, 0};
        if (l < rank)
#pragma unroll
            for (int x = 0; x < 6; ++x) f[x] = sc[(size_t)l * 6 + x];
#pragma unroll
        for (int X = 0; X < 3; ++X) {
            const uint64_t d = f[2 * X] & lims[X], s = f[2 * X + 1];
            bad += __builtin_popcountll(f[2 * X] & ~lims[X]) +
                   __builtin_popcountll(z2 ? s : (s & ~d));
            f[2 * X] = d;
            f[2 * X + 1] = z2 ? 0 : s & d;
        }
        if (narrow) {
            W32[2 * l] = (uint32_t)f[4];
            W32[2 * l + 1] = (uint32_t)f[5];
        } else {
            W64[2 * l] = f[4];
            W64[2 * l + 1] = f[5];
        }
        entry_sets(f[0], f[1], Lu, Ud + k, Us + k, all);
        entry_sets(f[2], f[3], Lv, Vd + k, Vs + k, all);
    }
    wave_lds_sync();
    bad += narrow ? verify_pairs<uint32_t>(W32, Ud, Us, Vd, Vs, all, words, m, n, p, z2)
                  : verify_pairs<uint64_t>(W64, Ud, Us, Vd, Vs, all, words, m, n, p, z2);
    for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
    if (lane == 0) n_violated[q] = bad;
}

// (r, c) of a row-major rows x cols factor -> the new position, or -1 when
// its row or column is dropped (drop_r / drop_c, -1 for none); cols2 is the
// new row length
__device__ __forceinline__ uint64_t remap_mask(uint64_t mask, int cols, int cols2, int drop_r,
                                               int drop_c)
{
    const uint32_t by = div_by(cols);
    uint64_t o = 0;
    for (; mask; mask &= mask - 1) {
        const int e = __builtin_ctzll(mask);
        const int rr = div_entry(e, by), cc = e - rr * cols;
        if (rr == drop_r || cc == drop_c) continue;
        const int r2 = rr - (drop_r >= 0 && rr > drop_r), c2 = cc - (drop_c >= 0 && cc > drop_c);
        o |= 1ull << (r2 * cols2 + c2);
    }
    return o;
}

// One wavefront per walk: project / extend / copy a scheme into a new start.
__global__ void __launch_bounds__(64) meta_kernel(tsf_walk_batch in, int32_t which,
                                                  const int32_t *op, const int32_t *axis,
                                                  const int32_t *index, int32_t r_cap_extra,
                                                  tsf_walk_batch out)
{
    const int64_t walk = blockIdx.x;
    const int lane = threadIdx.x;
    if (walk >= in.n_walks) return;
    const tsf_walk_header *h = in.hdr + walk;
    tsf_walk_header *ho = out.hdr + walk;
    const int m = h->m, n = h->n, p = h->p, mode = h->mode;
    const int rank = which ? h->best_rank : h->rank;
    const int o = op[walk], ax = axis[walk], ix = index[walk];
    const int dims[3] = {m, n, p};
    bool ok = m >= 1 && n >= 1 && p >= 1 && rank >= 0 && rank <= in.capacity && o >= 0 &&
              o <= 2 && (o == 0 || (ax >= 0 && ax <= 2));
    if (ok && o == 1) ok = dims[ax] >= 2 && ix >= 0 && ix < dims[ax];
    const int m2 = m + (ok && ax == 0 ? (o == 1 ? -1 : o == 2 ? 1 : 0) : 0);
    const int n2 = n + (ok && ax == 1 ? (o == 1 ? -1 : o == 2 ? 1 : 0) : 0);
    const int p2 = p + (ok && ax == 2 ? (o == 1 ? -1 : o == 2 ? 1 : 0) : 0);
    ok = ok && m2 * n2 <= 64 && n2 * p2 <= 64 && p2 * m2 <= 64;
    const int extra = (ok && o == 2) ? (ax == 0 ? n * p : ax == 1 ? m * p : m * n) : 0;
    // per factor: columns before/after and the dropped row/column (axis order:
    // U rows i (m) cols j (n); V rows j (n) cols k (p); W rows k (p) cols i (m))
    const int colsU = n, colsV = p, colsW = m;
    const int colsU2 = n2, colsV2 = p2, colsW2 = m2;
    const int dr_u = (o == 1 && ax == 0) ? ix : -1, dc_u = (o == 1 && ax == 1) ? ix : -1;
    const int dr_v = (o == 1 && ax == 1) ? ix : -1, dc_v = (o == 1 && ax == 2) ? ix : -1;
    const int dr_w = (o == 1 && ax == 2) ? ix : -1, dc_w = (o == 1 && ax == 0) ? ix : -1;
    const uint64_t *src = (which ? in.best : in.cur) + (size_t)walk * in.capacity * 6;
    uint64_t *dst = const_cast<uint64_t *>(out.start) + (size_t)walk * out.capacity * 6;
    int count = 0;
    if (ok) {
        for (int base = 0; base < rank; base += 64) {
            const int k = base + lane;
            uint64_t f[6] = {0, 0, 0, 0, 0, 0};
            bool keep = false;
            if (k < rank) {
                f[0] = remap_mask(src[k * 6 + 0], colsU, colsU2, dr_u, dc_u);
                f[1] = remap_mask(src[k * 6 + 1], colsU, colsU2, dr_u, dc_u);
                f[2] = remap_mask(src[k * 6 + 2], colsV, colsV2, dr_v, dc_v);
                f[3] = remap_mask(src[k * 6 + 3], colsV, colsV2, dr_v, dc_v);
                f[4] = remap_mask(src[k * 6 + 4], colsW, colsW2, dr_w, dc_w);
                f[5] = remap_mask(src[k * 6 + 5], colsW, colsW2, dr_w, dc_w);
                keep = f[0] != 0 && f[2] != 0 && f[4] != 0;
                if (mode == 0) {
                    // Sec. 3.6: first non-zero of u, then of v, positive; w absorbs
                    for (int X = 0; X < 2; ++X) {
                        const uint64_t low = f[2 * X] & (~f[2 * X] + 1);
                        if (f[2 * X + 1] & low) {
                            f[2 * X + 1] ^= f[2 * X];
                            f[5] ^= f[4];
                        }
                    }
                }
            }
            const uint64_t mk = __ballot(keep);
            const int pos = count + __builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0));
            if (keep && pos < out.capacity)
                for (int x = 0; x < 6; ++x) dst[pos * 6 + x] = f[x];
            count += __builtin_popcountll(mk);
        }
        // extend: the naive scheme of the new index
        for (int q = lane; q < extra; q += 64) {
            int i, j, k;
            if (ax == 2) { i = q / n; j = q % n; k = p; }
            else if (ax == 0) { i = m; j = q / p; k = q % p; }
            else { i = q / p; j = n; k = q % p; }
            const int pos = count + q;
            if (pos < out.capacity) {
                dst[pos * 6 + 0] = 1ull << (i * n2 + j);
                dst[pos * 6 + 1] = 0;
                dst[pos * 6 + 2] = 1ull << (j * p2 + k);
                dst[pos * 6 + 3] = 0;
                dst[pos * 6 + 4] = 1ull << (k * m2 + i);
                dst[pos * 6 + 5] = 0;
            }
        }
        count += extra;
    }
    if (lane == 0) {
        const bool fits = ok && count <= out.capacity;
        ho->m = fits ? m2 : m;
        ho->n = fits ? n2 : n;
        ho->p = fits ? p2 : p;
        ho->mode = mode;
        ho->target_rank = h->target_rank;
        ho->start_rank = fits ? count : -1;
        const int rc = count + r_cap_extra;
        ho->r_cap = fits ? (rc < out.capacity ? rc : out.capacity) : 0;
    }
}

// Feature rows of the proposal network from log records: a wavefront writes a
// row of 1 KiB with one 16-byte store per lane.  A record is 128 bytes, so the
// kernel is bound by its writes; one row per thread, whose stores went to 64
// different rows at a time, took 14 us for 4,096 rows.  A launch has at most
// 65,536 workgroups, which take further rows in turn: with a workgroup for every
// four rows, launches would end at 2^32 threads, 64 GiB of features.
constexpr int64_t kFeatureBlocks = 65536;
__global__ void __launch_bounds__(256) features_kernel(const tsf_flip_log *log, int64_t n,
                                                       uint16_t *X)
{
    const int lane = threadIdx.x & 63;
    const int b = lane < 48 ? lane >> 3 : 0;
    for (int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); q < n;
         q += (int64_t)gridDim.x * 4) {
        const tsf_flip_log &lg = log[q];
        const int slot = lg.format_slot < 0 || lg.format_slot > 15 ? 15 : lg.format_slot;
        store_feature_piece(X + q * 512, lane,
                            feature_piece(lane, lg.f[2 * b], lg.f[2 * b + 1], slot, lg.rank_before));
    }
}

// Isotropy invariants (Sec. 3.7) of one scheme per wavefront: lane l takes
// factors l, l+64, ... of the scheme (a factor's two masks are one 16-byte
// load).  The rank comes from elimination on the masks (factor_rank_masks);
// where that leaves it open, from elimination modulo 65521 on the entries, which
// every factor took before, in 16 KiB of LDS a wavefront.  65,536 schemes of
// the mixed formats 998 -> 201 us.
__device__ int factor_rank_entries(uint64_t d, uint64_t s, int rows, int cols)
{
    int32_t M[64];
    return factor_rank(d, s, rows, cols, false, M);
}
__global__ void __launch_bounds__(256) invariants_kernel(const tsf_walk_header *hdr,
                                                        const uint64_t *schemes, int32_t cap,
                                                        int32_t n_walks, int32_t which,
                                                        uint8_t *term_ranks, int32_t *rank_sums)
{
    const int64_t walk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (walk >= n_walks) return;
    const tsf_walk_header *h = hdr + walk;
    const int m = h->m, n = h->n, p = h->p;
    const int rank = which == 0 ? h->rank : which == 1 ? h->best_rank : h->start_rank;
    const bool ok = m >= 1 && n >= 1 && p >= 1 && m * n <= 64 && n * p <= 64 && p * m <= 64 &&
                    (h->mode == 0 || h->mode == 1) && rank >= 0 && rank <= cap;
    if (!ok) {
        if (lane < 3) rank_sums[walk * 3 + lane] = -1;
        return;
    }
    const bool z2 = h->mode == 1;
    const uint64_t *sc = schemes + (size_t)walk * cap * 6;
    uint8_t *out = term_ranks + (size_t)walk * cap * 3;
    // per kind: rows, columns, row starts, reciprocal of the columns
    const int rows[3] = {m, n, p}, cols[3] = {n, p, m};
    uint64_t starts[3];
    uint32_t magic[3];
#pragma unroll
    for (int X = 0; X < 3; ++X) {
        starts[X] = 0;
        for (int r = 0; r < rows[X]; ++r) starts[X] |= 1ull << (r * cols[X]);
        magic[X] = (65536u + cols[X] - 1) / cols[X];
    }
    const bool al = (reinterpret_cast<uintptr_t>(sc) & 15) == 0;
    int sum[3] = {0, 0, 0};
    int X = lane % 3;
    for (int q = lane; q < 3 * rank; q += 64) {
        uint64_t d, s;
        if (al) {
            const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(sc + 2 * q);
            d = v.x;
            s = v.y;
        } else {
            d = sc[2 * q];
            s = sc[2 * q + 1];
        }
        const int R = X == 0 ? rows[0] : X == 1 ? rows[1] : rows[2];
        const int Cc = X == 0 ? cols[0] : X == 1 ? cols[1] : cols[2];
        const uint64_t lim = R * Cc == 64 ? ~0ull : (1ull << (R * Cc)) - 1;
        d &= lim;
        s &= d;
        int a = factor_rank_masks(d, s, R, Cc, z2, X == 0 ? starts[0] : X == 1 ? starts[1] : starts[2],
                                  X == 0 ? magic[0] : X == 1 ? magic[1] : magic[2]);
        if (a < 0) a = factor_rank_entries(d, s, R, Cc);
        out[q] = (uint8_t)a;
        sum[0] += X == 0 ? a : 0;
        sum[1] += X == 1 ? a : 0;
        sum[2] += X == 2 ? a : 0;
        X = X == 2 ? 0 : X + 1;  // 64 mod 3 = 1
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        for (int off = 32; off > 0; off >>= 1) sum[k] += __shfl_xor(sum[k], off);
        if (lane == k) rank_sums[walk * 3 + k] = sum[k];
    }
}

// ---------------------------------------------------------------------------
// Population synchronisation and the Resize kernel (Sec. 3.4.1, Algorithm 2)
// ---------------------------------------------------------------------------
__global__ void clear_table_kernel(unsigned long long *keys, unsigned long long *vals, int slots,
                                   int32_t *overflow)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < slots) {
        keys[q] = 0;
        vals[q] = ~0ull;
    }
    if (q == 0) *overflow = 0;
}

// One thread per walk: insert the walk's format into an open-addressing
// table (key = 1 | m << 8 | n << 16 | p << 24) and keep, per format, the
// smallest (best rank << 32 | walk id).
__global__ void best_insert_kernel(const tsf_walk_header *hdr, int32_t n_walks,
                                   unsigned long long *keys, unsigned long long *vals, int slots,
                                   int32_t *overflow)
{
    const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= n_walks) return;
    const tsf_walk_header *h = hdr + w;
    if (h->done < 0 || h->m < 1 || h->m > 64 || h->n < 1 || h->n > 64 || h->p < 1 || h->p > 64)
        return;
    const unsigned long long key = 1ull | ((unsigned long long)h->m << 8) |
                                   ((unsigned long long)h->n << 16) | ((unsigned long long)h->p << 24);
    const unsigned long long val = ((unsigned long long)(uint32_t)h->best_rank << 32) | (uint64_t)w;
    int q = (int)((key * 0x9E3779B97F4A7C15ull) >> 40) % slots;
    for (int probe = 0; probe < slots; ++probe) {
        // (a word read late only looks emptier or larger than it is)
        unsigned long long prev = __atomic_load_n(&keys[q], __ATOMIC_RELAXED);
        if (prev == 0) prev = atomicCAS(&keys[q], 0ull, key);
        if (prev == 0 || prev == key) {
            if (__atomic_load_n(&vals[q], __ATOMIC_RELAXED) > val) atomicMin(&vals[q], val);
            return;
        }
        q = q + 1 == slots ? 0 : q + 1;
    }
    atomicAdd(overflow, 1);
}

// The occupied slots in ascending (m, n, p) order -> table: a slot's position
// is the number of smaller formats.  Every workgroup lists the occupied keys
// (in any order) in its LDS; it places 64 slots, whose smaller formats its
// sixteen wavefronts count over a sixteenth of the list each, four keys per LDS
// read.  A round of 16,384 exploratory walks (about a thousand formats): 5 us;
// one workgroup that counted over every slot, empty ones too, took 1.0 ms.
constexpr int kMaxSlots = 4096;
constexpr int kCompactSlots = 64, kCompactWaves = 16;
__global__ void __launch_bounds__(64 * kCompactWaves)
best_compact_kernel(const unsigned long long *keys, const unsigned long long *vals, int slots,
                    tsf_best_entry *table, int32_t *n_entries, const int32_t *overflow,
                    int32_t *dropped)
{
    __shared__ __attribute__((aligned(16))) uint32_t list[kMaxSlots + 4];
    __shared__ int32_t used, smaller[kCompactSlots];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) used = 0;
    if (threadIdx.x < kCompactSlots) smaller[threadIdx.x] = 0;
    __syncthreads();
    const auto order = [](unsigned long long k) {
        return (uint32_t)(((k >> 8) & 0xFF) << 16 | ((k >> 16) & 0xFF) << 8 | ((k >> 24) & 0xFF));
    };
    for (int q0 = 0; q0 < slots; q0 += 64 * kCompactWaves) {
        const int q = q0 + threadIdx.x;
        const unsigned long long k = q < slots ? keys[q] : 0;
        const uint64_t has = __ballot(k != 0);
        int at = 0;
        if (lane == 0 && has) at = atomicAdd(&used, __builtin_popcountll(has));
        at = __shfl(at, 0) + __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0));
        if (k) list[at] = order(k);
    }
    __syncthreads();
    const int n = used;
    if (threadIdx.x < 4) list[n + threadIdx.x] = 0xFFFFFFFFu;  // smaller than no format
    __syncthreads();
    const int q = blockIdx.x * kCompactSlots + lane;
    const unsigned long long k = q < slots ? keys[q] : 0;
    const uint32_t o = k ? order(k) : 0;
    if (__ballot(k != 0)) {
        const int groups = (n + 3) / 4;
        int less = 0;
        for (int x = wave; x < groups; x += kCompactWaves) {
            const uint4 v = *reinterpret_cast<const uint4 *>(list + 4 * x);
            less += (v.x < o) + (v.y < o) + (v.z < o) + (v.w < o);
        }
        if (less) atomicAdd(&smaller[lane], less);
    }
    __syncthreads();
    if (wave == 0 && k) {
        tsf_best_entry e;
        e.m = (int32_t)((k >> 8) & 0xFF);
        e.n = (int32_t)((k >> 16) & 0xFF);
        e.p = (int32_t)((k >> 24) & 0xFF);
        e.rank = (int32_t)(vals[q] >> 32);
        e.walk = (int64_t)(vals[q] & 0xFFFFFFFFull);
        table[smaller[lane]] = e;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *n_entries = n;
        if (dropped) *dropped = *overflow;
    }
}

// Algorithm 2 on every walk (one wavefront per walk): the walk's current or
// best scheme, after the operators drawn from Philox blocks (round, 0, 3)
// and (round, 1, 3) of its seed, becomes its start scheme in `out`.
// Partners are the best schemes of the table, read from in.best.  Lanes
// handle output terms.
__global__ void __launch_bounds__(64) resize_kernel(tsf_walk_batch in, int32_t which,
                                                    const tsf_best_entry *table,
                                                    const int32_t *n_entries, uint64_t base_seed,
                                                    int64_t first_walk_id, int64_t round,
                                                    uint64_t t_resize, int32_t r_cap_extra,
                                                    tsf_walk_batch out, int32_t *applied_out)
{
    const int64_t walk = blockIdx.x;
    const int lane = threadIdx.x;
    if (walk >= in.n_walks) return;
    const tsf_walk_header *h = in.hdr + walk;
    tsf_walk_header *ho = out.hdr + walk;
    const int m0 = h->m, n0 = h->n, p0 = h->p;
    const int r0 = which ? h->best_rank : h->rank;
    const int nb = *n_entries;
    const bool sane = h->done >= 0 && m0 >= 1 && n0 >= 1 && p0 >= 1 && m0 * n0 <= 64 &&
                      n0 * p0 <= 64 && p0 * m0 <= 64 && r0 >= 1 && r0 <= in.capacity &&
                      r0 <= out.capacity;
    const uint64_t seed = base_seed + (uint64_t)(first_walk_id + walk);
    const Philox4 b0 = walk_block(seed, round, 0, 3), b1 = walk_block(seed, round, 1, 3);
    const uint64_t *src = (which ? in.best : in.cur) + (size_t)walk * in.capacity * 6;
    uint64_t *dst = const_cast<uint64_t *>(out.start) + (size_t)walk * out.capacity * 6;
    const bool swp = sane && b0.x[0] < 0x80000000u;
    // format after the optional swap
    const int m = m0, n = swp ? p0 : n0, p = swp ? n0 : p0;
    auto term = [&](int k, uint64_t (&f)[6]) {
        uint64_t g[6];
        for (int x = 0; x < 6; ++x) g[x] = src[k * 6 + x];
        if (swp)
            term_swap(g, m0, n0, p0, f);
        else
            for (int x = 0; x < 6; ++x) f[x] = g[x];
    };
    int applied = swp ? 1 : 0;
    int op = 0;  // 0 keep, 2 merge, 4 project, 8 product, 16 double, 32 extend
    int axis = 0, pidx = 0, M = m, N = n, P = p, R = r0;
    int64_t partner = -1;
    int pm = 0, pn = 0, pp = 0, pr = 0;
    if (sane && nb > 0) {
        const tsf_best_entry e = table[below(b0.x[1], (uint32_t)nb)];
        const int order[3] = {2, 0, 1};
        for (int q = 0; q < 3 && op == 0; ++q) {
            const int ax = order[q];
            const bool compat = ax == 2 ? (e.m == m && e.n == n) : ax == 0 ? (e.n == n && e.p == p)
                                                                            : (e.m == m && e.p == p);
            const int M2 = ax == 0 ? m + e.m : m, N2 = ax == 1 ? n + e.n : n,
                      P2 = ax == 2 ? p + e.p : p;
            if (compat && M2 * N2 <= 64 && N2 * P2 <= 64 && P2 * M2 <= 64 &&
                r0 + e.rank <= out.capacity) {
                op = 2;
                axis = ax;
                M = M2; N = N2; P = P2; R = r0 + e.rank;
                partner = e.walk;
                pm = e.m; pn = e.n; pp = e.p; pr = e.rank;
            }
        }
    }
    if (sane && op == 0 && (uint64_t)b0.x[2] < t_resize) {
        axis = (int)below(b1.x[1], 3u);
        const int dim = axis == 0 ? m : axis == 1 ? n : p;
        const uint32_t q = b0.x[3];
        if (q < 214748365u) {  // round(0.05 * 2^32): project
            if (dim >= 2) {
                op = 4;
                pidx = (int)below(b1.x[2], (uint32_t)dim);
                M = m - (axis == 0); N = n - (axis == 1); P = p - (axis == 2);
            }
        } else if (q < 2362232013u) {  // round(0.55 * 2^32): product
            if (nb > 0) {
                const tsf_best_entry e = table[below(b1.x[0], (uint32_t)nb)];
                const int M2 = m * e.m, N2 = n * e.n, P2 = p * e.p;
                if (M2 * N2 <= 64 && N2 * P2 <= 64 && P2 * M2 <= 64 &&
                    (int64_t)r0 * e.rank <= out.capacity) {
                    op = 8;
                    M = M2; N = N2; P = P2; R = r0 * e.rank;
                    partner = e.walk;
                    pm = e.m; pn = e.n; pp = e.p; pr = e.rank;
                }
            }
        } else if (q < 3650722202u) {  // round(0.85 * 2^32): double
            const int M2 = axis == 0 ? 2 * m : m, N2 = axis == 1 ? 2 * n : n,
                      P2 = axis == 2 ? 2 * p : p;
            if (M2 * N2 <= 64 && N2 * P2 <= 64 && P2 * M2 <= 64 && 2 * r0 <= out.capacity) {
                op = 16;
                M = M2; N = N2; P = P2; R = 2 * r0;
            }
        } else {  // extend
            const int M2 = m + (axis == 0), N2 = n + (axis == 1), P2 = p + (axis == 2);
            const int extra = axis == 0 ? n * p : axis == 1 ? m * p : m * n;
            if (M2 * N2 <= 64 && N2 * P2 <= 64 && P2 * M2 <= 64 && r0 + extra <= out.capacity) {
                op = 32;
                M = M2; N = N2; P = P2; R = r0 + extra;
            }
        }
    }
    applied |= op;
    const uint64_t *psrc = partner >= 0 ? in.best + (size_t)partner * in.capacity * 6 : nullptr;
    int count = 0;
    if (sane) {
        if (op == 0 || op == 2 || op == 16 || op == 32) {
            // the walk's own terms, embedded (offset 0)
            for (int k = lane; k < r0; k += 64) {
                uint64_t f[6], o[6];
                term(k, f);
                term_embed(f, m, n, p, M, N, P, 0, 0, 0, o);
                for (int x = 0; x < 6; ++x) dst[k * 6 + x] = o[x];
            }
            count = r0;
        }
        if (op == 2) {
            const int oi = axis == 0 ? m : 0, oj = axis == 1 ? n : 0, ok = axis == 2 ? p : 0;
            for (int k = lane; k < pr; k += 64) {
                uint64_t f[6], o[6];
                for (int x = 0; x < 6; ++x) f[x] = psrc[k * 6 + x];
                term_embed(f, pm, pn, pp, M, N, P, oi, oj, ok, o);
                for (int x = 0; x < 6; ++x) dst[(r0 + k) * 6 + x] = o[x];
            }
            count = R;
        } else if (op == 16) {
            const int oi = axis == 0 ? m : 0, oj = axis == 1 ? n : 0, ok = axis == 2 ? p : 0;
            for (int k = lane; k < r0; k += 64) {
                uint64_t f[6], o[6];
                term(k, f);
                term_embed(f, m, n, p, M, N, P, oi, oj, ok, o);
                for (int x = 0; x < 6; ++x) dst[(r0 + k) * 6 + x] = o[x];
            }
            count = R;
        } else if (op == 32) {
            const int extra = R - r0;
            for (int q = lane; q < extra; q += 64) {
                int i, j, k;
                if (axis == 2) { i = q / n; j = q % n; k = p; }
                else if (axis == 0) { i = m; j = q / p; k = q % p; }
                else { i = q / p; j = n; k = q % p; }
                uint64_t *d = dst + (size_t)(r0 + q) * 6;
                d[0] = 1ull << (i * N + j);
                d[1] = 0;
                d[2] = 1ull << (j * P + k);
                d[3] = 0;
                d[4] = 1ull << (k * M + i);
                d[5] = 0;
            }
            count = R;
        } else if (op == 8) {
            for (int q = lane; q < R; q += 64) {
                const int l1 = q / pr, l2 = q % pr;
                uint64_t f[6], g[6], o[6];
                term(l1, f);
                for (int x = 0; x < 6; ++x) g[x] = psrc[l2 * 6 + x];
                term_kron(f, m, n, p, g, pm, pn, pp, o);
                for (int x = 0; x < 6; ++x) dst[q * 6 + x] = o[x];
            }
            count = R;
        } else if (op == 4) {
            // project: drop index pidx of `axis`, keep the non-zero terms in order
            const int cu = n, cv = p, cw = m;
            const int dr_u = axis == 0 ? pidx : -1, dc_u = axis == 1 ? pidx : -1;
            const int dr_v = axis == 1 ? pidx : -1, dc_v = axis == 2 ? pidx : -1;
            const int dr_w = axis == 2 ? pidx : -1, dc_w = axis == 0 ? pidx : -1;
            for (int base = 0; base < r0; base += 64) {
                const int k = base + lane;
                uint64_t f[6], o[6] = {0, 0, 0, 0, 0, 0};
                bool keep = false;
                if (k < r0) {
                    term(k, f);
                    o[0] = remap_mask(f[0], cu, N, dr_u, dc_u);
                    o[1] = remap_mask(f[1], cu, N, dr_u, dc_u);
                    o[2] = remap_mask(f[2], cv, P, dr_v, dc_v);
                    o[3] = remap_mask(f[3], cv, P, dr_v, dc_v);
                    o[4] = remap_mask(f[4], cw, M, dr_w, dc_w);
                    o[5] = remap_mask(f[5], cw, M, dr_w, dc_w);
                    keep = o[0] != 0 && o[2] != 0 && o[4] != 0;
                    normalise_packed(o);
                }
                const uint64_t mk = __ballot(keep);
                const int pos = count + __builtin_amdgcn_mbcnt_hi(
                                            (uint32_t)(mk >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0));
                if (keep)
                    for (int x = 0; x < 6; ++x) dst[pos * 6 + x] = o[x];
                count += __builtin_popcountll(mk);
            }
            R = count;
        }
    }
    if (lane == 0) {
        ho->m = sane ? M : m0;
        ho->n = sane ? N : n0;
        ho->p = sane ? P : p0;
        ho->mode = h->mode;
        ho->target_rank = h->target_rank;
        ho->start_rank = sane ? count : -1;
        const int rc = count + r_cap_extra;
        ho->r_cap = rc < out.capacity ? rc : out.capacity;
        if (applied_out) applied_out[walk] = sane ? applied : -1;
    }
}

// ---------------------------------------------------------------------------
// host side: kernel table and launch
// ---------------------------------------------------------------------------
KernelFn pick_kernel(int g, int s, bool wide, bool z2, int strategy, bool chk)
{
    if (wide) return z2 ? pick_kernel_w1_z1(g, s, strategy, chk) : pick_kernel_w1_z0(g, s, strategy, chk);
    return z2 ? pick_kernel_w0_z1(g, s, strategy, chk) : pick_kernel_w0_z0(g, s, strategy, chk);
}

int slots_for(int cap, int g)
{
    for (int s : {1, 2, 4, 5, 6, 7, 8})
        if (s * g >= cap && (g == 64 || (s & (s - 1)) == 0)) return s;
    return -1;
}

tsf_status check_batch(const tsf_walk_batch *b)
{
    if (!b) return tsf_fail(TSF_E_ARG, "null batch");
    if (b->n_walks < 0) return tsf_fail(TSF_E_ARG, "n_walks %d < 0", b->n_walks);
    if (b->capacity < 1 || b->capacity > 512)
        return tsf_fail(TSF_E_CAPACITY, "capacity %d outside [1, 512]", b->capacity);
    if (b->rec_cap < 0) return tsf_fail(TSF_E_ARG, "rec_cap %d < 0", b->rec_cap);
    if (b->mode != TSF_TERNARY && b->mode != TSF_Z2)
        return tsf_fail(TSF_E_ARG, "batch mode %d", b->mode);
    if (b->max_len < 1 || b->max_len > 64)
        return tsf_fail(TSF_E_FORMAT, "max_len %d outside [1, 64]", b->max_len);
    if (b->n_walks > 0 && (!b->hdr || !b->cur || !b->best || !b->start ||
                           (b->rec_cap > 0 && !b->rec)))
        return tsf_fail(TSF_E_ARG, "null device buffer");
    return TSF_OK;
}

}  // namespace

// A captured sequence of learned iterations, replayed with hipGraphLaunch.
struct GraphEntry {
    unsigned char key[sizeof(KArgs) + 8 * sizeof(void *)];
    hipGraph_t graph;
    hipGraphExec_t exec;
    int64_t chunk;
    bool used;
};

struct tsf_ctx {
    int device;
    int cu_count;
    hipStream_t capture;      // private stream used only to capture graphs
    GraphEntry graphs[8];
    int next_graph;
    TuneEntry tuned[16];
    int next_tuned;
    void *scratch;            // autotuner's copy of a batch
    size_t scratch_bytes;
};

namespace {
const tsf_launch *tuned_launch(const tsf_ctx *ctx, const tsf_walk_params *prm,
                               const tsf_walk_batch *b)
{
    if (!ctx || !prm) return nullptr;
    for (const TuneEntry &e : ctx->tuned)
        if (tune_serves(e, prm, b)) return &e.launch;
    return nullptr;
}

bool launch_is_default(const tsf_launch *l)
{
    return !l || (l->lanes_per_walk == 0 && l->waves_per_block == 0 && l->strategy == 0);
}

// The three launches of the population synchronisation over a table of
// `slots` keys and values and an overflow counter in `work` (2*slots + 1
// words); the clear kernel writes every word the others read, so the table
// may hold anything before.
tsf_status launch_population(const tsf_walk_batch *b, tsf_best_entry *table, int32_t *n_entries,
                             uint64_t *work, int32_t slots, int32_t *dropped, hipStream_t s)
{
    unsigned long long *keys = (unsigned long long *)work, *vals = keys + slots;
    int32_t *overflow = (int32_t *)(vals + slots);
    hipLaunchKernelGGL(clear_table_kernel, dim3((slots + 255) / 256), dim3(256), 0, s, keys, vals,
                       slots, overflow);
    if (b->n_walks > 0)
        hipLaunchKernelGGL(best_insert_kernel, dim3((b->n_walks + 255) / 256), dim3(256), 0, s,
                           b->hdr, b->n_walks, keys, vals, slots, overflow);
    hipLaunchKernelGGL(best_compact_kernel, dim3((slots + kCompactSlots - 1) / kCompactSlots),
                       dim3(64 * kCompactWaves), 0, s, keys, vals, slots, table,
                       n_entries, (const int32_t *)overflow, dropped);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "population launch failed");
    return TSF_OK;
}

// Working memory of tsf_population_best_noalloc: the table at its largest
// size (kMaxSlots keys, kMaxSlots values, the overflow counter), one copy on
// every device the library runs on, for the life of the process.  Host code
// never passes the array's name to a kernel (on the host it only stands for
// the symbol): it uses the device address hipGetSymbolAddress returns, looked
// up once per device.
__device__ __align__(256) uint64_t scratch[2 * kMaxSlots + 1];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
uint64_t *scratch_ptr[kMaxDevices];

// the current device's copy of `scratch`
tsf_status population_scratch(uint64_t **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return tsf_fail(TSF_E_DEVICE, "hipGetDevice failed");
    if (dev < 0 || dev >= kMaxDevices)
        return tsf_fail(TSF_E_DEVICE, "device %d beyond the %d the library supports", dev,
                        kMaxDevices);
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return tsf_fail(TSF_E_DEVICE, "hipGetSymbolAddress(scratch) failed: %s",
                            hipGetErrorString(e));
        scratch_ptr[dev] = (uint64_t *)p;
    }
    *out = scratch_ptr[dev];
    return TSF_OK;
}
}  // namespace

extern "C" {

tsf_status tsf_ctx_create(tsf_ctx **ctx)
{
    if (!ctx) return tsf_fail(TSF_E_ARG, "null ctx pointer");
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return tsf_fail(TSF_E_DEVICE, "hipGetDevice failed");
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return tsf_fail(TSF_E_DEVICE, "hipDeviceGetAttribute failed");
    tsf_ctx *c = new tsf_ctx;
    std::memset(c, 0, sizeof *c);
    c->device = dev;
    c->cu_count = cus;
    if (hipStreamCreateWithFlags(&c->capture, hipStreamNonBlocking) != hipSuccess) {
        delete c;
        return tsf_fail(TSF_E_DEVICE, "cannot create the capture stream");
    }
    *ctx = c;
    return TSF_OK;
}

tsf_status tsf_ctx_destroy(tsf_ctx *ctx)
{
    if (!ctx) return TSF_OK;
    for (GraphEntry &g : ctx->graphs)
        if (g.used) {
            hipGraphExecDestroy(g.exec);
            hipGraphDestroy(g.graph);
        }
    if (ctx->capture) hipStreamDestroy(ctx->capture);
    if (ctx->scratch) hipFree(ctx->scratch);
    delete ctx;
    return TSF_OK;
}

tsf_status tsf_walk_init(tsf_ctx *ctx, const tsf_walk_batch *b, void *hip_stream)
{
    (void)ctx;
    tsf_status st = check_batch(b);
    if (st) return st;
    if (b->n_walks == 0) return TSF_OK;
    hipStream_t s = (hipStream_t)hip_stream;
    hipLaunchKernelGGL(init_kernel, dim3((b->n_walks + 3) / 4), dim3(256), 0, s, b->hdr, b->cur, b->best,
                       b->start, b->n_walks, b->capacity);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "init launch failed");
    return TSF_OK;
}

}  // extern "C"

namespace {

struct Launch {
    KernelFn fn;
    dim3 grid, block;
    size_t lds;
    int g;
    bool ap, ix;
};

// validate a walk call and build its kernel arguments and launch shape
tsf_status prepare_walk(const tsf_walk_params *prm, const tsf_walk_batch *b, int64_t n_iters,
                        const tsf_launch *launch, KArgs &a, Launch &L, bool checked = false,
                        bool learned = false)
{
    tsf_status st = check_batch(b);
    if (st) return st;
    if (!prm) return tsf_fail(TSF_E_ARG, "null params");
    if (prm->flip_tries < 1 || prm->flip_tries > 64)
        return tsf_fail(TSF_E_ARG, "flip_tries %d outside [1, 64]", prm->flip_tries);
    if (prm->t_eq > (1ull << 32) || prm->t_reduce > (1ull << 32) || prm->t_expand > (1ull << 32))
        return tsf_fail(TSF_E_ARG, "a probability threshold exceeds 2^32");
    if (n_iters < 0) return tsf_fail(TSF_E_ARG, "n_iters < 0");
    if (prm->objective != TSF_OBJ_RANK && prm->objective != TSF_OBJ_ADDITIONS)
        return tsf_fail(TSF_E_ARG, "objective %d", prm->objective);
    if (b->log && b->log_cap < 0) return tsf_fail(TSF_E_ARG, "log_cap < 0");
    WalkShape w;
    if ((st = walk_shape(prm, b, launch, checked, w))) return st;
    const bool wide = b->max_len > 32, ix = w.strategy == 3, ap = ix || w.strategy == 1;
    const int g = w.lanes, wpb = w.waves;
    // term slots per lane (term-parallel kernels), or 64-bit words of a
    // partner set (attempt-parallel kernels)
    const int s = ap ? (b->capacity > 64 ? 2 : 1) : slots_for(b->capacity, g);
    if (s < 0)
        return tsf_fail(TSF_E_CAPACITY, "capacity %d needs more than 8 slots at %d lanes/walk",
                        b->capacity, g);
    // factors of at most 16 entries: the indexed kernels keep each factor's
    // digits and signs in one 32-bit LDS word
    const bool pk = ix && !wide && b->max_len <= 16;
    L.fn = pick_kernel(g, s, wide, b->mode == TSF_Z2, learned ? 5 : pk ? 4 : w.strategy, checked);
    if (!L.fn) return tsf_fail(TSF_E_ARG, "no kernel for this configuration");
    const int walks_per_wave = 64 / g;
    const int cap2 = lds_stride(b->capacity, ix);
    const size_t per_walk = walk_lds(b->capacity, b->max_len, ix);
    L.lds = (size_t)wpb * walks_per_wave * per_walk;
    if (L.lds > 160 * 1024)
        return tsf_fail(TSF_E_CAPACITY, "%zu bytes of LDS per workgroup exceed 160 KiB", L.lds);
    std::memset(&a, 0, sizeof a);
    a.base_seed = prm->base_seed;
    a.params_hash = tsf_params_hash(prm);
    a.first_walk_id = prm->first_walk_id;
    a.max_iters = prm->max_iters;
    a.plateau = prm->plateau;
    a.n_iters = n_iters;
    a.t_eq = prm->t_eq;
    a.t_reduce = prm->t_reduce;
    a.t_expand = prm->t_expand;
    a.flip_tries = prm->flip_tries;
    a.restart_from_best = prm->restart_from_best;
    a.objective = prm->objective;
    a.n_walks = b->n_walks;
    a.cap = b->capacity;
    a.rec_cap = b->rec_cap;
    a.mode = b->mode;
    a.max_len = b->max_len;
    a.cap2 = cap2;
    a.capm = b->capacity;
    a.log = b->log;
    a.log_cap = b->log ? b->log_cap : 0;
    a.hdr = b->hdr;
    a.cur = b->cur;
    a.best = b->best;
    a.start = b->start;
    a.rec = b->rec;
    const int64_t walks_per_block = (int64_t)wpb * walks_per_wave;
    const int64_t blocks = (b->n_walks + walks_per_block - 1) / walks_per_block;
    L.grid = dim3((unsigned)blocks);
    L.block = dim3(64 * wpb);
    L.g = g;
    L.ap = ap;
    L.ix = ix;
    if (L.lds > 64 * 1024 &&
        hipFuncSetAttribute((const void *)L.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)L.lds) != hipSuccess)
        return tsf_fail(TSF_E_DEVICE, "cannot raise the LDS limit to %zu bytes", L.lds);
    return TSF_OK;
}

tsf_status run(const Launch &L, const KArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(L.fn, L.grid, L.block, L.lds, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return tsf_fail(TSF_E_DEVICE, "walk launch failed: %s", hipGetErrorString(e));
    return TSF_OK;
}

}  // namespace

extern "C" {

tsf_status tsf_walk(tsf_ctx *ctx, const tsf_walk_params *prm, const tsf_walk_batch *b,
                    int64_t n_iters, const tsf_launch *launch, void *hip_stream)
{
    if (launch_is_default(launch) && b) {
        const tsf_launch *t = tuned_launch(ctx, prm, b);
        if (t) launch = t;
    }
    KArgs a;
    Launch L;
    tsf_status st = prepare_walk(prm, b, n_iters, launch, a, L);
    if (st) return st;
    if (b->n_walks == 0 || n_iters == 0) return TSF_OK;
    return run(L, a, (hipStream_t)hip_stream);
}

tsf_status tsf_walk_checked(tsf_ctx *ctx, const tsf_walk_params *prm, const tsf_walk_batch *b,
                            int64_t n_iters, const tsf_launch *launch, void *hip_stream)
{
    (void)ctx;  // the autotuner's choices are not used: they may name other shapes
    KArgs a;
    Launch L;
    tsf_status st = prepare_walk(prm, b, n_iters, launch, a, L, true);
    if (st) return st;
    if (b->n_walks == 0 || n_iters == 0) return TSF_OK;
    return run(L, a, (hipStream_t)hip_stream);
}

tsf_status tsf_autotune(tsf_ctx *ctx, const tsf_walk_params *prm, const tsf_walk_batch *b,
                        int64_t trial_iters, tsf_launch *chosen, void *hip_stream)
{
    if (!ctx) return tsf_fail(TSF_E_ARG, "null context");
    tsf_status st = check_batch(b);
    if (st) return st;
    if (!prm || trial_iters < 1) return tsf_fail(TSF_E_ARG, "bad params or trial_iters");
    if (b->n_walks == 0) return tsf_fail(TSF_E_ARG, "empty batch");
    const size_t n = (size_t)b->n_walks;
    const size_t sz_hdr = n * sizeof(tsf_walk_header);
    const size_t sz_sch = n * (size_t)b->capacity * 6 * sizeof(uint64_t);
    const size_t sz_rec = n * (size_t)(b->rec_cap > 0 ? b->rec_cap : 1) * sizeof(tsf_record);
    const size_t need = 2 * (sz_hdr + 2 * sz_sch + sz_rec);
    if (ctx->scratch_bytes < need) {
        if (ctx->scratch) hipFree(ctx->scratch);
        ctx->scratch = nullptr;
        ctx->scratch_bytes = 0;
        if (hipMalloc(&ctx->scratch, need) != hipSuccess)
            return tsf_fail(TSF_E_DEVICE, "cannot allocate %zu bytes for the autotuner", need);
        ctx->scratch_bytes = need;
    }
    hipStream_t s = (hipStream_t)hip_stream;
    // snapshot of the batch (first half of the scratch) and the trial copy
    unsigned char *base = (unsigned char *)ctx->scratch;
    unsigned char *snap = base, *trial = base + need / 2;
    auto lay = [&](unsigned char *p, tsf_walk_batch &c) {
        c = *b;
        c.hdr = (tsf_walk_header *)p;
        c.cur = (uint64_t *)(p + sz_hdr);
        c.best = (uint64_t *)(p + sz_hdr + sz_sch);
        c.rec = (tsf_record *)(p + sz_hdr + 2 * sz_sch);
        c.log = nullptr;
        c.log_cap = 0;
    };
    tsf_walk_batch bs, bt;
    lay(snap, bs);
    lay(trial, bt);
    bool ok = hipMemcpyAsync(bs.hdr, b->hdr, sz_hdr, hipMemcpyDeviceToDevice, s) == hipSuccess &&
              hipMemcpyAsync(bs.cur, b->cur, sz_sch, hipMemcpyDeviceToDevice, s) == hipSuccess &&
              hipMemcpyAsync(bs.best, b->best, sz_sch, hipMemcpyDeviceToDevice, s) == hipSuccess;
    if (!ok) return tsf_fail(TSF_E_DEVICE, "autotuner snapshot failed");
    hipEvent_t e0, e1;
    hipEventCreate(&e0);
    hipEventCreate(&e1);
    float best_ms = -1.0f;
    tsf_launch best{0, 0, 0};
    for (const tsf_launch &c : tune_candidates(prm, b)) {
        KArgs a;
        Launch L;
        if (prepare_walk(prm, &bt, trial_iters, &c, a, L) != TSF_OK) continue;
        hipMemcpyAsync(bt.hdr, bs.hdr, sz_hdr, hipMemcpyDeviceToDevice, s);
        hipMemcpyAsync(bt.cur, bs.cur, sz_sch, hipMemcpyDeviceToDevice, s);
        hipMemcpyAsync(bt.best, bs.best, sz_sch, hipMemcpyDeviceToDevice, s);
        hipEventRecord(e0, s);
        if (run(L, a, s) != TSF_OK) continue;
        hipEventRecord(e1, s);
        if (hipEventSynchronize(e1) != hipSuccess) break;
        float ms = 0.0f;
        hipEventElapsedTime(&ms, e0, e1);
        if (best_ms < 0.0f || ms < best_ms) {
            best_ms = ms;
            best = c;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (best_ms < 0.0f) return tsf_fail(TSF_E_CAPACITY, "no launch configuration fits the batch");
    TuneEntry *slot = nullptr;
    for (TuneEntry &e : ctx->tuned)
        if (tune_serves(e, prm, b)) slot = &e;
    if (!slot) {
        slot = &ctx->tuned[ctx->next_tuned];
        ctx->next_tuned = (ctx->next_tuned + 1) % 16;
    }
    *slot = tune_entry(prm, b, best);
    if (chosen) *chosen = best;
    return TSF_OK;
}

tsf_status tsf_walk_learned(tsf_ctx *ctx, const tsf_walk_params *prm, const tsf_walk_batch *b,
                            const tsf_mlp *net, const tsf_learn_ws *ws, int64_t n_iters,
                            const tsf_launch *launch, void *hip_stream)
{
    KArgs a;
    Launch L;
    // the propose and apply phases are kernels of the plain attempt-parallel
    // strategy (the scheme is reloaded by every launch, so an index would be
    // rebuilt each time)
    tsf_launch la = launch ? *launch : tsf_launch{0, 0, 0};
    if (la.strategy == 0) la.strategy = 1;
    if (la.strategy != 1)
        return tsf_fail(TSF_E_ARG, "learned proposals use the attempt-parallel strategy 1");
    if (prm && prm->objective != TSF_OBJ_RANK)
        return tsf_fail(TSF_E_ARG, "learned proposals serve the rank objective only");
    // Lanes per walk where the call leaves them open: an iteration is bound by
    // the latency of one wavefront, which grows with the walks in it (4,096
    // (3,3,3) walks: 32.1 us an iteration with 32 lanes, 33.2 with 16, 38.3 with
    // 8; 16,384 walks 91, 84 and 87).  The attempts scored stay those of 8.
    const int lanes = la.lanes_per_walk;
    if (lanes == 0 && b) la.lanes_per_walk = b->n_walks <= 4096 ? 32 : 16;
    tsf_status st;
    for (;;) {
        st = prepare_walk(prm, b, n_iters, &la, a, L, false, true);
        if (st) return st;
        // the staged feature rows, beside the terms; fewer wavefronts share a
        // workgroup where both do not fit (one always does)
        L.lds += (size_t)(L.block.x / L.g) * 12 * kLearnRows * sizeof(uint64_t);
        if (L.lds <= 160 * 1024 || L.block.x == 64) break;
        la.waves_per_block = (int)L.block.x / 64 - 1;
    }
    if (L.lds > 64 * 1024 &&
        hipFuncSetAttribute((const void *)L.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)L.lds) != hipSuccess)
        return tsf_fail(TSF_E_DEVICE, "cannot raise the LDS limit to %zu bytes", L.lds);
    if (!L.ap)
        return tsf_fail(TSF_E_CAPACITY,
                        "learned proposals use the attempt-parallel strategy (capacity <= 64)");
    const int K = prm->flip_tries;
    const int g = lanes ? L.g : 8;
    if (K > g - 1 || K > kLearnRows)
        return tsf_fail(TSF_E_ARG, "flip_tries %d exceeds the %d attempts scored at %d lanes/walk",
                        K, g - 1 < kLearnRows ? g - 1 : kLearnRows, g);
    if (!net || !ws || !ws->cand || !ws->feat || !ws->h1 || !ws->h2 || !ws->logit)
        return tsf_fail(TSF_E_ARG, "null learned-proposal buffer");
    if (ws->choice && ws->choice_cap < 0) return tsf_fail(TSF_E_ARG, "choice_cap < 0");
    if (b->n_walks == 0 || n_iters == 0) return TSF_OK;
    const int64_t rows = (int64_t)b->n_walks * kLearnRows;
    if (rows > 0x7FFFFFFF) return tsf_fail(TSF_E_CAPACITY, "too many candidate rows");
    a.learn_k = K;
    a.cand = ws->cand;
    a.feat = ws->feat;
    a.logit = ws->logit;
    a.choice = ws->choice;
    a.choice_cap = ws->choice ? ws->choice_cap : 0;
    a.n_iters = 1;
    hipStream_t s = (hipStream_t)hip_stream;
    const auto walks = [&](int phase, hipStream_t on) -> tsf_status {
        a.phase = phase;
        return run(L, a, on);
    };
    // score the proposed candidates, then apply the best and, but in the call's
    // last iteration, propose the next ones: the scheme is loaded once an
    // iteration.  The hidden layers stay in the network's kernel, but for those
    // of the last iteration, which the caller finds beside its rows and scores.
    auto iteration = [&](hipStream_t on, bool last) -> tsf_status {
        const tsf_status e =
            mlp_forward(net, ws->feat, (int32_t)rows, last ? ws->h1 : nullptr,
                        last ? ws->h2 : nullptr, ws->logit, on);
        return e ? e : walks(last ? 2 : 3, on);
    };
    if ((st = walks(1, s))) return st;
    // Every iteration but the last launches the same kernels with the same
    // arguments (the walk state lives in device memory), so a chunk of
    // iterations is captured once into a HIP graph and replayed.
    const int64_t chunk = 16;
    if (!ctx || n_iters <= chunk) {
        for (int64_t it = 0; it < n_iters; ++it)
            if ((st = iteration(s, it + 1 == n_iters))) return st;
        return TSF_OK;
    }
    unsigned char key[sizeof(GraphEntry::key)];
    std::memset(key, 0, sizeof key);
    a.phase = 0;
    std::memcpy(key, &a, sizeof a);
    const void *ptrs[8] = {net->param, net->wbf, ws->cand, ws->feat, ws->logit,
                           (const void *)L.fn};
    std::memcpy(key + sizeof a, ptrs, sizeof ptrs);
    GraphEntry *ge = nullptr;
    for (GraphEntry &g : ctx->graphs)
        if (g.used && g.chunk == chunk && std::memcmp(g.key, key, sizeof key) == 0) ge = &g;
    if (!ge) {
        ge = &ctx->graphs[ctx->next_graph];
        ctx->next_graph = (ctx->next_graph + 1) % 8;
        if (ge->used) {
            hipGraphExecDestroy(ge->exec);
            hipGraphDestroy(ge->graph);
            ge->used = false;
        }
        if (hipStreamBeginCapture(ctx->capture, hipStreamCaptureModeThreadLocal) != hipSuccess)
            return tsf_fail(TSF_E_DEVICE, "stream capture failed to start");
        for (int64_t it = 0; it < chunk; ++it)
            if ((st = iteration(ctx->capture, false))) {
                hipGraph_t dummy;
                hipStreamEndCapture(ctx->capture, &dummy);
                if (dummy) hipGraphDestroy(dummy);
                return st;
            }
        if (hipStreamEndCapture(ctx->capture, &ge->graph) != hipSuccess)
            return tsf_fail(TSF_E_DEVICE, "stream capture failed");
        if (hipGraphInstantiate(&ge->exec, ge->graph, nullptr, nullptr, 0) != hipSuccess) {
            hipGraphDestroy(ge->graph);
            return tsf_fail(TSF_E_DEVICE, "graph instantiation failed");
        }
        std::memcpy(ge->key, key, sizeof key);
        ge->chunk = chunk;
        ge->used = true;
    }
    int64_t done = 0;
    for (; done + chunk < n_iters; done += chunk)
        if (hipGraphLaunch(ge->exec, s) != hipSuccess)
            return tsf_fail(TSF_E_DEVICE, "graph launch failed");
    for (; done < n_iters; ++done)
        if ((st = iteration(s, done + 1 == n_iters))) return st;
    return TSF_OK;
}

tsf_status tsf_meta_batch(const tsf_walk_batch *in, int32_t which, const int32_t *op,
                          const int32_t *axis, const int32_t *index, int32_t r_cap_extra,
                          const tsf_walk_batch *out, void *hip_stream)
{
    tsf_status st = check_batch(in);
    if (st) return st;
    if ((st = check_batch(out))) return st;
    if (in->n_walks != out->n_walks) return tsf_fail(TSF_E_ARG, "batches differ in n_walks");
    if (which < 0 || which > 1) return tsf_fail(TSF_E_ARG, "which %d not in 0..1", which);
    if (r_cap_extra < 0) return tsf_fail(TSF_E_ARG, "r_cap_extra < 0");
    if (in->n_walks == 0) return TSF_OK;
    if (!op || !axis || !index) return tsf_fail(TSF_E_ARG, "null op/axis/index");
    if ((const void *)in->start == (const void *)out->start || in->cur == out->start ||
        in->best == out->start)
        return tsf_fail(TSF_E_ARG, "in and out must not share scheme buffers");
    hipLaunchKernelGGL(meta_kernel, dim3(in->n_walks), dim3(64), 0, (hipStream_t)hip_stream, *in,
                       which, op, axis, index, r_cap_extra, *out);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "meta launch failed");
    return TSF_OK;
}

tsf_status tsf_features_from_log(const tsf_flip_log *log, int64_t n, uint16_t *X, void *hip_stream)
{
    if (n < 0 || (n > 0 && (!log || !X))) return tsf_fail(TSF_E_ARG, "bad feature arguments");
    if (n == 0) return TSF_OK;
    const int64_t blocks = n / 4 + (n % 4 != 0);
    hipLaunchKernelGGL(features_kernel,
                       dim3((unsigned)(blocks < kFeatureBlocks ? blocks : kFeatureBlocks)), dim3(256), 0,
                       (hipStream_t)hip_stream, log, n, X);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "feature launch failed");
    return TSF_OK;
}

tsf_status tsf_population_best(const tsf_walk_batch *b, tsf_best_entry *table, int32_t *n_entries,
                               uint64_t *work, int32_t slots, void *hip_stream)
{
    tsf_status st = check_batch(b);
    if (st) return st;
    if (slots < 1 || slots > kMaxSlots)
        return tsf_fail(TSF_E_ARG, "slots %d outside [1, %d]", slots, kMaxSlots);
    if (!table || !n_entries || !work) return tsf_fail(TSF_E_ARG, "null table or workspace");
    return launch_population(b, table, n_entries, work, slots, nullptr, (hipStream_t)hip_stream);
}

tsf_status tsf_population_best_noalloc(const tsf_walk_batch *b, tsf_best_entry *table,
                                       int32_t *n_entries, int32_t slots, int32_t *dropped,
                                       void *hip_stream)
{
    tsf_status st = check_batch(b);
    if (st) return st;
    if (slots < 1 || slots > kMaxSlots)
        return tsf_fail(TSF_E_ARG, "slots %d outside [1, %d] (the size of the library's table)",
                        slots, kMaxSlots);
    if (!table || !n_entries) return tsf_fail(TSF_E_ARG, "null table or count");
    uint64_t *work = nullptr;
    if ((st = population_scratch(&work))) return st;
    return launch_population(b, table, n_entries, work, slots, dropped, (hipStream_t)hip_stream);
}

tsf_status tsf_resize_batch(const tsf_walk_batch *in, int32_t which, const tsf_best_entry *table,
                            const int32_t *n_entries, const tsf_resize_params *prm,
                            const tsf_walk_batch *out, int32_t *applied, void *hip_stream)
{
    tsf_status st = check_batch(in);
    if (st) return st;
    if ((st = check_batch(out))) return st;
    if (in->n_walks != out->n_walks) return tsf_fail(TSF_E_ARG, "batches differ in n_walks");
    if (which < 0 || which > 1) return tsf_fail(TSF_E_ARG, "which %d not in 0..1", which);
    if (!prm || !table || !n_entries) return tsf_fail(TSF_E_ARG, "null argument");
    if (prm->r_cap_extra < 0 || prm->t_resize > (1ull << 32))
        return tsf_fail(TSF_E_ARG, "bad resize parameters");
    if (in->mode != out->mode) return tsf_fail(TSF_E_ARG, "batches differ in mode");
    if ((const void *)in->start == (const void *)out->start || in->cur == out->start ||
        in->best == out->start)
        return tsf_fail(TSF_E_ARG, "in and out must not share scheme buffers");
    if (in->n_walks == 0) return TSF_OK;
    hipLaunchKernelGGL(resize_kernel, dim3(in->n_walks), dim3(64), 0, (hipStream_t)hip_stream, *in,
                       which, table, n_entries, prm->base_seed, prm->first_walk_id, prm->round,
                       prm->t_resize, prm->r_cap_extra, *out, applied);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "resize launch failed");
    return TSF_OK;
}

tsf_status tsf_invariants_batch(const tsf_walk_batch *b, int32_t which, uint8_t *term_ranks,
                                int32_t *rank_sums, void *hip_stream)
{
    tsf_status st = check_batch(b);
    if (st) return st;
    if (which < 0 || which > 2) return tsf_fail(TSF_E_ARG, "which %d not in 0..2", which);
    if (b->n_walks == 0) return TSF_OK;
    if (!term_ranks || !rank_sums) return tsf_fail(TSF_E_ARG, "null output");
    const uint64_t *src = which == 0 ? b->cur : which == 1 ? b->best : b->start;
    hipLaunchKernelGGL(invariants_kernel, dim3((b->n_walks + 3) / 4), dim3(256), 0, (hipStream_t)hip_stream,
                       b->hdr, src, b->capacity, b->n_walks, which, term_ranks, rank_sums);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "invariants launch failed");
    return TSF_OK;
}

tsf_status tsf_verify_batch(const tsf_walk_batch *b, int32_t which, int64_t *n_violated,
                            void *hip_stream)
{
    tsf_status st = check_batch(b);
    if (st) return st;
    if (which < 0 || which > 2) return tsf_fail(TSF_E_ARG, "which %d not in 0..2", which);
    if (!n_violated && b->n_walks) return tsf_fail(TSF_E_ARG, "null output");
    if (b->n_walks == 0) return TSF_OK;
    const uint64_t *src = which == 0 ? b->cur : which == 1 ? b->best : b->start;
    // four wavefronts (schemes) per workgroup, two where their LDS is large
    const int all = (b->capacity + 63) / 64, waves = all <= 4 ? 4 : 2;
    hipLaunchKernelGGL(verify_kernel, dim3((b->n_walks + waves - 1) / waves), dim3(64 * waves),
                       waves * all * kVerifyLds, (hipStream_t)hip_stream, b->hdr, src, b->capacity,
                       b->n_walks, which, n_violated);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "verify launch failed");
    return TSF_OK;
}

}  // extern "C"
