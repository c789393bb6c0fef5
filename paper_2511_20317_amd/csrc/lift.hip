// lift.hip -- ternary lifting of a Z2 scheme (Sec. 3.10.1) as a parallel
// exhaustive search on the GPU.
//
// The search space and order (a fixed convention, so that the first lifting
// found is unique): per term the first non-zero entry of u and of v is +1 and the other non-zero entries --
// u ascending, then v, then w -- are the term's free signs, bit i of the
// term's pattern x meaning entry i is -1; terms in order, patterns
// ascending; after a term every equation it touches must stay reachable,
// |target - partial sum| <= the number of later terms touching it.  The
// patterns of the first P terms, read as one mixed-radix number (term 0 most
// significant), name a subtree; one wavefront searches one subtree depth first
// with the residuals of all equations in LDS.  At a term the lanes try 64
// patterns at once: each lane walks the term's products, whose equations and
// sign masks come from a table the host lays out (uniform, so scalar loads and
// LDS broadcasts), and a ballot gives the set of patterns that keep every
// equation reachable; the search then takes its members in order, and a term's
// set stays valid until the search leaves that term upwards.  LDS is sized by
// the scheme's equations, so that a CU holds as many wavefronts as it has
// slots.  16,384 subtrees of (2,2,3) schemes, 256 nodes each: 85-190 us a call,
// of which about 60 are its fixed cost (620-8,300 us with a pattern at a time,
// every trial written to LDS and taken back, and 36 KiB of LDS a wavefront);
// with 16,384 nodes each 0.16-2.5 ms (1.5-98 ms).  The first solution in the
// global order is the one in the smallest subtree that has a solution, provided
// every smaller subtree was searched to the end.
#include <hip/hip_runtime.h>

#include "../../include/tsf.h"
#include "tsf_bits.h"
#include "tsf_internal.h"

#include <cstdint>
#include <cstring>
#include <vector>

namespace {

constexpr int kLiftMaxEq = 8192;     // equations (mn)(np)(pm) searched on the GPU
constexpr int kLiftMaxTerms = 512;

// What a search leaves: the smallest subtree with a solution, the smallest that
// ran out of budget, the numbers searched to the end.  Atomics on one address
// wait for each other, so the subtrees count in kCounters lines of memory in
// turn, and only a subtree below them writes the two minima: a search of a
// (2,2,2) scheme with 65,536 subtrees of at most 16 nodes takes 83 us, 1,262 us
// with one counter and every subtree's minimum written.
constexpr int kCounters = 64;
struct LiftOut {
    unsigned long long first, budget;
    struct {
        unsigned long long n, pad[15];
    } exhausted[kCounters];
};

struct LiftArgs {
    const uint64_t *mask;   // per product: the pattern bits whose parity is its sign
    const uint16_t *eq;     // per product: its equation
    const int32_t *off;     // per term: its first product (r + 1 entries)
    const int32_t *nfree;   // per term: its free signs
    const int16_t *rem0;    // per equation: the products that touch it
    int m, n, p, r, P, E;   // format, rank, prefix terms, equations
    int64_t n_sub;          // subtrees
    int64_t max_nodes;      // per subtree
    LiftOut *out;
    int64_t *pat;           // pattern per term of the solution (replay pass)
    int replay;             // search subtree out->first only and write its patterns
};

struct LiftWave {
    const LiftArgs *a;
    int lane;
    int16_t *res, *rem;     // per equation: target - partial sum, later products

    // add (dir -1) or remove (+1) term l's products under pattern x; returns
    // whether every touched equation stays reachable (when adding)
    __device__ bool apply(int l, int64_t x, int dir)
    {
        bool ok = true;
        for (int c = a->off[l] + lane; c < a->off[l + 1]; c += 64) {
            const int e = a->eq[c];
            const int neg = __builtin_popcountll((uint64_t)x & a->mask[c]) & 1;
            const int r2 = res[e] + dir * (neg ? -1 : 1);
            const int m2 = rem[e] + dir;
            res[e] = (int16_t)r2;
            rem[e] = (int16_t)m2;
            if (dir < 0 && (r2 > m2 || -r2 > m2)) ok = false;
        }
        sync();
        return __ballot(!ok) == 0;
    }
    // the patterns of term l in 64 consecutive ones from x0 on that keep every
    // equation reachable
    __device__ uint64_t feasible(int l, int64_t x0) const
    {
        const int64_t x = x0 + lane;
        bool ok = x < (1ll << a->nfree[l]);
        const int end = a->off[l + 1];
        for (int c = a->off[l]; c < end; ++c) {
            const int e = a->eq[c];
            const int r1 = res[e], m2 = rem[e] - 1;
            const int r2 = r1 - 1 + 2 * (__builtin_popcountll((uint64_t)x & a->mask[c]) & 1);
            ok = ok && r2 <= m2 && -r2 <= m2;
        }
        return __ballot(ok);
    }
    __device__ __forceinline__ static void sync()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

// LDS of a search: two counters per equation, a pattern and a set per term
size_t lift_lds(int E, int r) { return (size_t)r * 16 + (size_t)E * 4; }

__global__ void __launch_bounds__(64) lift_kernel(LiftArgs a)
{
    extern __shared__ uint64_t lift_smem[];
    uint64_t *set = lift_smem;                              // per term
    int64_t *pat = reinterpret_cast<int64_t *>(set + a.r);  // per term
    int16_t *res = reinterpret_cast<int16_t *>(pat + a.r), *rem = res + a.E;
    const int lane = threadIdx.x;
    const unsigned long long known = a.replay ? a.out->first : 0;
    if (a.replay && known == ~0ull) return;  // nothing was found
    const int64_t sub = a.replay ? (int64_t)known : (int64_t)blockIdx.x;
    if (sub >= a.n_sub) return;
    LiftWave W{&a, lane, res, rem};
    const int Lv = a.n * a.p, Lw = a.p * a.m;
    // targets and contributor counts
    for (int e = lane; e < a.E; e += 64) {
        const int ea = e / (Lv * Lw), eb = (e / Lw) % Lv, ec = e % Lw;
        const int a1 = ea / a.n, a2 = ea % a.n, b1 = eb / a.p, b2 = eb % a.p, c1 = ec / a.m,
                  c2 = ec % a.m;
        res[e] = (a2 == b1 && b2 == c1 && c2 == a1) ? 1 : 0;
        rem[e] = a.rem0[e];
    }
    // the subtree's prefix: patterns of terms 0..P-1 from the mixed-radix id
    int64_t rest = sub;
    for (int l = a.P - 1; l >= 0; --l) {
        if (lane == 0) pat[l] = rest & ((1ll << a.nfree[l]) - 1);
        rest >>= a.nfree[l];
    }
    LiftWave::sync();
    bool alive = true;
    for (int l = 0; l < a.P && alive; ++l) alive = W.apply(l, pat[l], -1);
    int status = 0;  // 0 searched to the end, 1 found, 2 budget, 3 a smaller subtree has one
    if (alive) {
        int l = a.P;
        int64_t nodes = 0, x = 0;  // x: the next pattern of term l
        bool found = a.P == a.r;
        for (uint32_t turn = 0; !found; ++turn) {
            if (!a.replay && (turn & 63) == 0 &&
                __atomic_load_n(&a.out->first, __ATOMIC_RELAXED) < (unsigned long long)sub) {
                status = 3;
                break;
            }
            const int64_t end = 1ll << a.nfree[l];
            uint64_t s = 0;
            if (x < end) {
                const int64_t block = x & ~63ll;
                if (x == block) {  // entered from above or from the block before
                    s = W.feasible(l, block);
                    if (lane == 0) set[l] = s;
                    LiftWave::sync();
                } else {
                    s = set[l];
                }
                // members from x on; the patterns passed over are nodes too
                s &= ~0ull << (x & 63);
                const int64_t next = s ? block + __builtin_ctzll(s)
                                       : (block + 64 < end ? block + 64 : end);
                nodes += next - x;
                if (s ? nodes >= a.max_nodes : nodes > a.max_nodes) {
                    status = 2;
                    break;
                }
                x = next;
                if (s == 0 && x < end) continue;
            }
            if (s == 0) {
                // this term is exhausted: back to the previous free one
                if (l == a.P) break;
                --l;
                x = pat[l];
                W.apply(l, x, +1);
                ++x;
                continue;
            }
            ++nodes;
            if (lane == 0) pat[l] = x;
            W.apply(l, x, -1);
            ++l;
            x = 0;
            found = l == a.r;
        }
        if (found) status = 1;
    }
    if (a.replay) {
        if (status == 1)
            for (int l = lane; l < a.r; l += 64) a.pat[l] = pat[l];
        return;
    }
    if (lane == 0) {
        // (a minimum read late only looks larger than it is)
        const auto lower = [&](unsigned long long *to) {
            if (__atomic_load_n(to, __ATOMIC_RELAXED) > (unsigned long long)sub)
                atomicMin(to, (unsigned long long)sub);
        };
        if (status == 1) lower(&a.out->first);
        if (status == 2) lower(&a.out->budget);
        if (status <= 1) atomicAdd(&a.out->exhausted[sub % kCounters].n, 1ull);
    }
}

}  // namespace

extern "C" {

tsf_status tsf_lift(const tsf_scheme *z2, int64_t max_nodes, int32_t max_subtrees,
                    tsf_scheme *out, tsf_lift_result *res)
{
    if (!z2 || !out || !res || !z2->U || !z2->V || !z2->W || !out->U || !out->V || !out->W)
        return tsf_fail(TSF_E_ARG, "null argument");
    if (z2->d.mode != TSF_Z2) return tsf_fail(TSF_E_ARG, "the input must be a Z2 scheme");
    if (max_nodes < 1 || max_subtrees < 1) return tsf_fail(TSF_E_ARG, "bad search limits");
    const int m = z2->d.m, n = z2->d.n, p = z2->d.p, r = z2->d.rank;
    if (m < 1 || n < 1 || p < 1 || m * n > 64 || n * p > 64 || p * m > 64)
        return tsf_fail(TSF_E_FORMAT, "format (%d,%d,%d)", m, n, p);
    if ((int64_t)m * n * n * p * p * m > kLiftMaxEq)
        return tsf_fail(TSF_E_CAPACITY, "more than %d Brent equations", kLiftMaxEq);
    if (r < 1 || r > kLiftMaxTerms || r > z2->d.capacity || out->d.capacity < r)
        return tsf_fail(TSF_E_CAPACITY, "rank %d", r);
    const int len[3] = {m * n, n * p, p * m};
    const int8_t *mat[3] = {z2->U, z2->V, z2->W};
    std::vector<uint64_t> d((size_t)r * 3, 0);
    std::vector<int> nfree(r);
    for (int l = 0; l < r; ++l) {
        for (int X = 0; X < 3; ++X)
            for (int e = 0; e < len[X]; ++e) {
                const int8_t c = mat[X][(size_t)l * len[X] + e];
                if (c != 0 && c != 1) return tsf_fail(TSF_E_NOT_TERNARY, "Z2 coefficient %d", c);
                if (c) d[l * 3 + X] |= 1ull << e;
            }
        if (!d[l * 3] || !d[l * 3 + 1] || !d[l * 3 + 2])
            return tsf_fail(TSF_E_ARG, "term %d has a zero factor", l);
        nfree[l] = __builtin_popcountll(d[l * 3]) - 1 + __builtin_popcountll(d[l * 3 + 1]) - 1 +
                   __builtin_popcountll(d[l * 3 + 2]);
        if (nfree[l] > 40) return tsf_fail(TSF_E_CAPACITY, "term %d has %d free signs", l, nfree[l]);
    }
    // prefix terms: as many leading terms as keep the subtrees within the limit
    int P = 0;
    int64_t n_sub = 1;
    while (P < r && n_sub * (1ll << nfree[P]) <= max_subtrees) n_sub *= 1ll << nfree[P++];
    // the products of every term, the contributor counts and the search's
    // results, in one buffer: one allocation, one copy each way
    const int Lv = len[1], Lw = len[2], E = len[0] * Lv * Lw;
    std::vector<uint64_t> mask;
    std::vector<uint16_t> eq;
    std::vector<int32_t> off(1, 0);
    std::vector<int16_t> rem(E, 0);
    for (int l = 0; l < r; ++l) {
        const uint64_t u = d[l * 3], v = d[l * 3 + 1], w = d[l * 3 + 2];
        const int cu = __builtin_popcountll(u), cv = __builtin_popcountll(v);
        int qa = 0;
        for (uint64_t fu = u; fu; fu &= fu - 1, ++qa) {
            int qb = 0;
            for (uint64_t fv = v; fv; fv &= fv - 1, ++qb) {
                int qc = 0;
                for (uint64_t fw = w; fw; fw &= fw - 1, ++qc) {
                    const int e = (__builtin_ctzll(fu) * Lv + __builtin_ctzll(fv)) * Lw +
                                  __builtin_ctzll(fw);
                    eq.push_back((uint16_t)e);
                    mask.push_back((qa ? 1ull << (qa - 1) : 0) |
                                   (qb ? 1ull << (cu - 1 + qb - 1) : 0) |
                                   1ull << (cu - 1 + cv - 1 + qc));
                    ++rem[e];
                }
            }
        }
        off.push_back((int32_t)eq.size());
    }
    const size_t np = eq.size();
    const size_t o_pat = sizeof(LiftOut), o_mask = o_pat + (size_t)r * 8, o_off = o_mask + np * 8,
                 o_free = o_off + (size_t)(r + 1) * 4, o_eq = o_free + (size_t)r * 4,
                 o_rem = o_eq + np * 2, bytes = o_rem + (size_t)E * 2;
    std::vector<unsigned char> blob(bytes);
    const LiftOut none{~0ull, ~0ull, {}};
    std::memcpy(blob.data(), &none, sizeof none);
    std::memset(blob.data() + o_pat, 0, (size_t)r * 8);
    std::memcpy(blob.data() + o_mask, mask.data(), np * 8);
    std::memcpy(blob.data() + o_off, off.data(), off.size() * 4);
    std::memcpy(blob.data() + o_free, nfree.data(), nfree.size() * 4);
    std::memcpy(blob.data() + o_eq, eq.data(), np * 2);
    std::memcpy(blob.data() + o_rem, rem.data(), rem.size() * 2);
    unsigned char *dev = nullptr;
    if (hipMalloc(&dev, bytes) != hipSuccess) return tsf_fail(TSF_E_DEVICE, "lift buffers");
    tsf_status st = TSF_OK;
    LiftArgs a{(const uint64_t *)(dev + o_mask), (const uint16_t *)(dev + o_eq),
               (const int32_t *)(dev + o_off), (const int32_t *)(dev + o_free),
               (const int16_t *)(dev + o_rem), m, n, p, r, P, E, n_sub, max_nodes,
               (LiftOut *)dev, (int64_t *)(dev + o_pat), 0};
    const size_t lds = lift_lds(E, r);
    const bool sent = hipMemcpy(dev, blob.data(), bytes, hipMemcpyHostToDevice) == hipSuccess;
    if (sent) {
        // the search, then the patterns of the smallest subtree that has a
        // solution (no budget: the search found it)
        hipLaunchKernelGGL(lift_kernel, dim3((unsigned)n_sub), dim3(64), lds, 0, a);
        a.replay = 1;
        a.max_nodes = INT64_MAX;
        hipLaunchKernelGGL(lift_kernel, dim3(1), dim3(64), lds, 0, a);
    }
    std::vector<unsigned char> back(o_mask);
    if (!sent || hipGetLastError() != hipSuccess ||
        hipMemcpy(back.data(), dev, o_mask, hipMemcpyDeviceToHost) != hipSuccess) {
        st = tsf_fail(TSF_E_DEVICE, "lift search failed");
    } else {
        LiftOut got;
        std::memcpy(&got, back.data(), sizeof got);
        std::memset(res, 0, sizeof *res);
        res->subtrees = n_sub;
        res->prefix_terms = P;
        for (const auto &c : got.exhausted) res->exhausted += (int64_t)c.n;
        if (got.first != ~0ull) {
            res->status = got.first < got.budget ? 1 : 2;
            res->subtree = (int64_t)got.first;
            const int32_t out_cap = out->d.capacity;   // the caller's buffers
            out->d = z2->d;
            out->d.capacity = out_cap;
            out->d.mode = TSF_TERNARY;
            int8_t *om[3] = {out->U, out->V, out->W};
            for (int X = 0; X < 3; ++X) std::memset(om[X], 0, (size_t)out->d.capacity * len[X]);
            for (int l = 0; l < r; ++l) {
                int64_t x;
                std::memcpy(&x, back.data() + o_pat + (size_t)l * 8, 8);
                // the first entries of u and v are +1, the others as the
                // pattern's bits say
                for (int X = 0; X < 3; ++X) {
                    bool first = X < 2;
                    for (uint64_t f = d[l * 3 + X]; f; f &= f - 1) {
                        int sign = 1;
                        if (!first) {
                            sign = x & 1 ? -1 : 1;
                            x >>= 1;
                        }
                        first = false;
                        om[X][(size_t)l * len[X] + __builtin_ctzll(f)] = (int8_t)sign;
                    }
                }
            }
        } else {
            res->status = got.budget == ~0ull ? 0 : -1;
            res->subtree = -1;
        }
    }
    hipFree(dev);
    return st;
}

}  // extern "C"
