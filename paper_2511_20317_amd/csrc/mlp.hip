// mlp.hip -- the learned flip-proposal network on gfx950: bf16 operands on
// the MFMA matrix cores with fp32 accumulation.
//
//   z1 = X W1 + b1, h1 = bf16(relu(z1)); z2 = h1 W2 + b2, h2 = bf16(relu(z2));
//   logit = h2 . w3 + b3;  loss = mean(softplus(logit) - y logit)
//
// Three kernels carry it.  fwd_kernel runs the whole forward pass of a block
// of rows (two layers on v_mfma_f32_32x32x16_bf16 and the logit) with the
// hidden rows kept in LDS; delta_kernel the loss derivative and the delta of
// the first layer; grad_kernel every weight gradient and the loss.
#include <hip/hip_runtime.h>

#include "../../include/tsf.h"
#include "tsf_internal.h"


namespace {

typedef float v16f32 __attribute__((ext_vector_type(16)));

constexpr int IN = TSF_MLP_IN, HID = TSF_MLP_HID;
// offsets into the fp32 parameter vector
constexpr int O_W1T = 0;                   // W1^T: HID x IN (row n holds W1[:, n])
constexpr int O_B1 = O_W1T + HID * IN;     // HID
constexpr int O_W2T = O_B1 + HID;          // W2^T: HID x HID
constexpr int O_B2 = O_W2T + HID * HID;    // HID
constexpr int O_W3 = O_B2 + HID;           // HID
constexpr int O_B3 = O_W3 + HID;           // 1 (padded to 4)
static_assert(O_B3 + 4 == TSF_MLP_NPARAM, "parameter layout");
// offsets into the bf16 compute copies
constexpr int Q_W1T = 0;                   // HID x IN
constexpr int Q_W2T = Q_W1T + HID * IN;    // HID x HID (W2^T)
constexpr int Q_W2 = Q_W2T + HID * HID;    // HID x HID (W2, for the backward)
constexpr int Q_W3 = Q_W2 + HID * HID;     // HID
static_assert(Q_W3 + HID == TSF_MLP_NBF16, "bf16 layout");

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    // round to nearest, ties to even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef __bf16 v8bf16 __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf16 __attribute__((ext_vector_type(2)));
typedef float v2f32 __attribute__((ext_vector_type(2)));
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));

// two floats to packed bf16, to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const v2f32 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2bf16));
}

// eight consecutive bf16 of global memory; AL: p is 16-byte aligned
template <bool AL>
__device__ __forceinline__ v4u32 load8(const uint16_t *p)
{
    if constexpr (AL) {
        return *reinterpret_cast<const v4u32 *>(p);
    } else {
        return v4u32{p[0] | (uint32_t)p[1] << 16, p[2] | (uint32_t)p[3] << 16,
                     p[4] | (uint32_t)p[5] << 16, p[6] | (uint32_t)p[7] << 16};
    }
}
template <bool AL>
__device__ __forceinline__ void store8(uint16_t *p, v4u32 v)
{
    if constexpr (AL) {
        *reinterpret_cast<v4u32 *>(p) = v;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            p[2 * q] = (uint16_t)v[q];
            p[2 * q + 1] = (uint16_t)(v[q] >> 16);
        }
    }
}

// ---------------------------------------------------------------------------
// A block of 32*RB*WR rows through 256-wide layers: WR groups of four wavefronts,
// 32*RB rows a group; wavefront w of a group owns the output columns
// 64w .. 64w+63 of each of its rows.  The weight
// matrices (256 rows of the output column, k contiguous) stream through LDS 64
// k at a time, double buffered, and kAhead chunks are in flight to registers
// before that.  The rows' activations come from a 64-wide chunk beside it
// (first layer) or from the whole hidden tile in LDS.  LDS rows are padded to
// 72 and 264 entries, so that the 16-byte reads of 32 consecutive rows spread
// over all banks.
// The weights are the matrix instruction's first operand, so a lane's four
// consecutive accumulators are four consecutive output columns of one row and
// go to the tile with one 8-byte write.
// ---------------------------------------------------------------------------
constexpr int BK = 64, LDK = BK + 8, LDT = HID + 8;
constexpr int kWBuf = HID * LDK;  // entries of one weight chunk
constexpr int kAhead = 2;         // chunks in flight: chunk c passes slot and buffer c % 2

template <int RB, int WR>
struct Block {
    static constexpr int R = 32 * RB * WR, kThreads = 256 * WR;
    static constexpr int kXBuf = R * LDK;
    static constexpr int kTile = R * LDT > 2 * kXBuf ? R * LDT : 2 * kXBuf;
    uint16_t *W;     // two weight chunks
    uint16_t *tile;  // R x LDT hidden rows; first two X chunks of R x LDK
    v4u32 wreg[kAhead][8 / WR], xreg[kAhead][RB];
    v16f32 acc[RB][2];

    // this wavefront's first row
    __device__ __forceinline__ static int first_row()
    {
        return WR == 1 ? 0 : 32 * RB * (int)(threadIdx.x >> 8);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[a][b][q] = 0.0f;
    }
    // 64 k from w on of the 256 rows of a matrix (row stride K), on their way to
    // slot q
    template <bool AL>
    __device__ __forceinline__ void load_w(const uint16_t *w, int K, int q)
    {
#pragma unroll
        for (int t = 0; t < 8 / WR; ++t)
            wreg[q][t] =
                load8<AL>(w + ((threadIdx.x >> 3) + 32 * WR * t) * K + (threadIdx.x & 7) * 8);
    }
    __device__ __forceinline__ void store_w(int q, int buf)
    {
#pragma unroll
        for (int t = 0; t < 8 / WR; ++t)
            *reinterpret_cast<v4u32 *>(W + buf * kWBuf + ((threadIdx.x >> 3) + 32 * WR * t) * LDK +
                                       (threadIdx.x & 7) * 8) = wreg[q][t];
    }
    // multiply one weight chunk with 64 k of the rows at `x` (row stride ldx).
    // 32x32x16: lane l holds row l%32 of an operand, k = 8*(l/32) + 0..7
    __device__ __forceinline__ void multiply(int buf, const uint16_t *x, int ldx)
    {
        const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
        const uint16_t *wp = W + buf * kWBuf + (64 * wave + (lane & 31)) * LDK + 8 * (lane >> 5);
        const uint16_t *xp = x + (first_row() + (lane & 31)) * ldx + 8 * (lane >> 5);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            v8bf16 wv[2], xv[RB];
#pragma unroll
            for (int b = 0; b < 2; ++b)
                wv[b] = *reinterpret_cast<const v8bf16 *>(wp + 32 * b * LDK + kk);
#pragma unroll
            for (int a = 0; a < RB; ++a)
                xv[a] = *reinterpret_cast<const v8bf16 *>(xp + 32 * a * ldx + kk);
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv[b], xv[a], acc[a][b], 0, 0, 0);
        }
    }
    // the product of the tile with w, whose first kAhead chunks are on their
    // way already; ends at a barrier.  The loops over chunks stay rolled (two
    // steps, one per slot): straight-line code that runs once waits for its
    // own instructions.
    template <bool AL>
    __device__ __forceinline__ void layer_on_tile(const uint16_t *w)
    {
#pragma unroll 1
        for (int c0 = 0; c0 < HID / BK; c0 += kAhead) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int c = c0 + q;
                store_w(q, q);
                if (c + kAhead < HID / BK) load_w<AL>(w + (c + kAhead) * BK, HID, q);
                __syncthreads();
                multiply(q, tile + c * BK, LDT);
            }
        }
        __syncthreads();
    }
    // accumulator register q of lane l: output column 8*(q/4) + 4*(l/32) + q%4
    // of its 32, row l%32
    __device__ __forceinline__ void to_tile()
    {
        const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = 64 * wave + 32 * b + 8 * g + 4 * (lane >> 5);
#pragma unroll
                for (int a = 0; a < RB; ++a)
                    *reinterpret_cast<uint2 *>(tile + (first_row() + 32 * a + (lane & 31)) * LDT + n) =
                        make_uint2(pack_bf16(acc[a][b][4 * g], acc[a][b][4 * g + 1]),
                                   pack_bf16(acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]));
            }
    }
};

// bias + ReLU + bf16 of the accumulators into the tile
template <int RB, int WR>
__device__ __forceinline__ void relu_to_tile(Block<RB, WR> &B, const float *bias)
{
    const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
    float bv[2][16];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 16; ++q)
            bv[b][q] = bias[64 * wave + 32 * b + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3)];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const float v = B.acc[a][b][q] + bv[b][q];
                B.acc[a][b][q] = v > 0.0f ? v : 0.0f;
            }
    B.to_tile();
}

// the tile's live rows to global memory, 16 bytes a lane
template <int RB, int WR, bool AL>
__device__ __forceinline__ void tile_out(const Block<RB, WR> &B, uint16_t *out, int row0, int M)
{
#pragma unroll
    for (int t = 0; t < 4 * RB; ++t) {
        const int r = (threadIdx.x >> 5) + 8 * WR * t, c = (threadIdx.x & 31) * 8;
        if (row0 + r < M)
            store8<AL>(out + (int64_t)(row0 + r) * HID + c,
                       *reinterpret_cast<const v4u32 *>(B.tile + r * LDT + c));
    }
}

// rows of global memory into the tile, zeros past the end
template <int RB, int WR, bool AL>
__device__ __forceinline__ void tile_in(const Block<RB, WR> &B, const uint16_t *in, int row0, int M)
{
#pragma unroll
    for (int t = 0; t < 4 * RB; ++t) {
        const int r = (threadIdx.x >> 5) + 8 * WR * t, c = (threadIdx.x & 31) * 8;
        v4u32 v = {0, 0, 0, 0};
        if (row0 + r < M) v = load8<AL>(in + (int64_t)(row0 + r) * HID + c);
        *reinterpret_cast<v4u32 *>(B.tile + r * LDT + c) = v;
    }
}

// Sums over the wavefront's lanes, in the order of a butterfly over lane
// distances 32, 16, 8, 4, 2, 1.  The first two steps of four sums share their
// instructions: a swap of the halves (quarters) of two registers leaves one
// register of lower and one of upper halves, and one addition serves both.
__device__ __forceinline__ float swap_add32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// each lane's sum over its 16 lanes; the partner at distance d is reached by a
// rotation by d, since the sums so far repeat every 2d lanes
__device__ __forceinline__ float row_sum(float s)
{
#define TSF_ROR_ADD(n)                                                                          \
    s += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(s),      \
                                                               0x120 + n, 0xF, 0xF, true))
    TSF_ROR_ADD(8);
    TSF_ROR_ADD(4);
    TSF_ROR_ADD(2);
    TSF_ROR_ADD(1);
#undef TSF_ROR_ADD
    return s;
}
__device__ __forceinline__ float wave_sum(float s)
{
    s = swap_add32(s, s);
    return row_sum(swap_add16(s, s));
}
// the sums of a, c, b and d in lanes 0-15, 16-31, 32-47 and 48-63
__device__ __forceinline__ float wave_sum4(float a, float b, float c, float d)
{
    return row_sum(swap_add16(swap_add32(a, b), swap_add32(c, d)));
}

struct FwdArgs {
    const uint16_t *X, *w1t, *w2t, *w3;
    const float *b1, *b2, *b3;
    int M;
    uint16_t *h1, *h2;  // null: not stored
    float *logit;
    int step;           // of a pass in steps
};

// The forward pass of a block of rows.  Layer 1 reads X (1 KiB a row) and W1
// once, its output stays in LDS for layer 2, whose output stays there for the
// logit; h1 and h2 are written where the caller wants them.  32,768 rows move
// 67 MB, 14.6 us at the 4.6 TB/s of a large copy, and take 19.9 us (12.9 us of
// it products and LDS traffic alone); as a GEMM per layer and a kernel for the
// logit they took 38.8 us.  At 4,096 rows the weights through each workgroup
// bound it: 10.1 us, of which 3.7 us are their reads.
// STEPS: one step of the pass, from the buffers of the one before: 0 the first
// layer, 1 the second, 2 the logit.  For calls whose h2 or logit lies over an
// input of an earlier step; a block would overwrite rows that others still read.
template <int RB, int WR, bool AL, bool STEPS = false>
__global__ void __launch_bounds__(256 * WR) fwd_kernel(FwdArgs g)
{
    using Bl = Block<RB, WR>;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * kWBuf + Bl::kTile];
    Bl B;
    B.W = smem;
    B.tile = smem + 2 * kWBuf;
    const int row0 = blockIdx.x * Bl::R;
    if (!STEPS || g.step == 0) {
        // this thread's pieces of an X chunk (rows past the end read the last one)
        const int xr = threadIdx.x >> 3, xc = (threadIdx.x & 7) * 8;
        const uint16_t *xsrc[RB];
#pragma unroll
        for (int t = 0; t < RB; ++t) {
            const int r = row0 + xr + 32 * WR * t;
            xsrc[t] = g.X + (int64_t)(r < g.M ? r : g.M - 1) * IN + xc;
        }
        const auto load_x = [&](int c, int q) {
#pragma unroll
            for (int t = 0; t < RB; ++t) B.xreg[q][t] = load8<AL>(xsrc[t] + c * BK);
        };
        constexpr int C1 = IN / BK;
#pragma unroll
        for (int c = 0; c < kAhead; ++c) {
            B.template load_w<AL>(g.w1t + c * BK, IN, c);
            load_x(c, c);
        }
        B.clear();
#pragma unroll 1
        for (int c0 = 0; c0 < C1; c0 += kAhead) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int c = c0 + q;
                uint16_t *xb = B.tile + q * Bl::kXBuf;
                B.store_w(q, q);
#pragma unroll
                for (int t = 0; t < RB; ++t)
                    *reinterpret_cast<v4u32 *>(xb + (xr + 32 * WR * t) * LDK + xc) = B.xreg[q][t];
                // the chunk two steps on, of W1 or the first ones of W2
                const int cn = c + kAhead;
                const bool more = cn < C1;
                B.template load_w<AL>(more ? g.w1t + cn * BK : g.w2t + (cn - C1) * BK,
                                      more ? IN : HID, q);
                if (more) load_x(cn, q);
                __syncthreads();
                B.multiply(q, xb, LDK);
            }
        }
        __syncthreads();
        relu_to_tile<RB, WR>(B, g.b1);
        __syncthreads();
        if (g.h1) tile_out<RB, WR, AL>(B, g.h1, row0, g.M);
    }
    if constexpr (STEPS) {
        if (g.step == 0) return;
        tile_in<RB, WR, AL>(B, g.step == 1 ? g.h1 : g.h2, row0, g.M);
        if (g.step == 1)
#pragma unroll
            for (int c = 0; c < kAhead; ++c) B.template load_w<AL>(g.w2t + c * BK, HID, c);
    }
    if (!STEPS || g.step == 1) {
        B.clear();
        B.template layer_on_tile<AL>(g.w2t);
        relu_to_tile<RB, WR>(B, g.b2);
        __syncthreads();
        if (g.h2) tile_out<RB, WR, AL>(B, g.h2, row0, g.M);
        if constexpr (STEPS) return;
    }
    if constexpr (STEPS) __syncthreads();
    // logit: lane l sums columns l, l+64, l+128, l+192 of a row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float w3[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w3[q] = from_bf16(g.w3[lane + 64 * q]);
    const float b3 = g.b3[0];
#pragma unroll 2
    for (int i = 0; i < 2 * RB; ++i) {
        const int r = wave * 8 * RB + 4 * i;
        float s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                s[e] += from_bf16(B.tile[(r + e) * LDT + lane + 64 * q]) * w3[q];
        }
        const float v = wave_sum4(s[0], s[2], s[1], s[3]);
        const int out = row0 + r + (lane >> 4);
        if ((lane & 15) == 0 && out < g.M) g.logit[out] = v + b3;
    }
}

// loss derivative of a row with respect to its logit
__device__ __forceinline__ float logit_delta(float z, float y, int M)
{
    const float sig = 1.0f / (1.0f + __expf(-z));
    return (sig - y) / (float)M;
}

struct DeltaArgs {
    const float *logit, *y;
    const uint16_t *h1, *h2, *w2, *w3;
    int M;
    float *d3;
    uint16_t *d2, *d1;
    int step;           // of a pass in steps
};

// delta3 = (sigmoid(logit) - y) / M; delta2 = bf16(delta3 w3 [h2 > 0]);
// delta1 = bf16((delta2 W2^T) [h1 > 0]) for 32*RB*WR rows; delta2 stays in LDS as
// the operand of its product.
// STEPS: one step of the pass: 0 delta3 and delta2, 1 delta1 from them.
template <int RB, int WR, bool AL, bool STEPS = false>
__global__ void __launch_bounds__(256 * WR) delta_kernel(DeltaArgs g)
{
    using Bl = Block<RB, WR>;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * kWBuf + Bl::kTile];
    __shared__ float dz[Bl::R];
    Bl B;
    B.W = smem;
    B.tile = smem + 2 * kWBuf;
    const int row0 = blockIdx.x * Bl::R;
#pragma unroll
    for (int c = 0; c < kAhead; ++c) B.template load_w<AL>(g.w2 + c * BK, HID, c);
    const int c8 = (threadIdx.x & 31) * 8;
    if (!STEPS || g.step == 0) {
        if (threadIdx.x < Bl::R) {
            const int r = row0 + threadIdx.x;
            float d = 0.0f;
            if (r < g.M) {
                d = logit_delta(g.logit[r], g.y[r], g.M);
                g.d3[r] = d;
            }
            dz[threadIdx.x] = d;
        }
        float w3[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) w3[q] = from_bf16(g.w3[c8 + q]);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4 * RB; ++t) {
            const int r = (threadIdx.x >> 5) + 8 * WR * t;
            v4u32 o = {0, 0, 0, 0};
            if (row0 + r < g.M) {
                const v4u32 h = load8<AL>(g.h2 + (int64_t)(row0 + r) * HID + c8);
                const float d = dz[r];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float lo = from_bf16((uint16_t)h[q]), hi = from_bf16((uint16_t)(h[q] >> 16));
                    o[q] = pack_bf16(lo > 0.0f ? d * w3[2 * q] : 0.0f, hi > 0.0f ? d * w3[2 * q + 1] : 0.0f);
                }
                store8<AL>(g.d2 + (int64_t)(row0 + r) * HID + c8, o);
            }
            *reinterpret_cast<v4u32 *>(B.tile + r * LDT + c8) = o;
        }
    } else {
        tile_in<RB, WR, AL>(B, g.d2, row0, g.M);
    }
    if (STEPS && g.step == 0) return;
    B.clear();
    // delta1[m][k] = sum_n delta2[m][n] W2[k][n]
    B.template layer_on_tile<AL>(g.w2);
    B.to_tile();
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4 * RB; ++t) {
        const int r = (threadIdx.x >> 5) + 8 * WR * t;
        if (row0 + r >= g.M) continue;
        const v4u32 h = load8<AL>(g.h1 + (int64_t)(row0 + r) * HID + c8);
        v4u32 d = *reinterpret_cast<const v4u32 *>(B.tile + r * LDT + c8);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!(from_bf16((uint16_t)h[q]) > 0.0f)) d[q] &= 0xFFFF0000u;
            if (!(from_bf16((uint16_t)(h[q] >> 16)) > 0.0f)) d[q] &= 0x0000FFFFu;
        }
        store8<AL>(g.d1 + (int64_t)(row0 + r) * HID + c8, d);
    }
}

struct GradArgs {
    const uint16_t *X, *h1, *h2, *d1, *d2;
    const float *d3, *logit, *y;  // d3 null: taken from the logits (db3, loss)
    int M;
    float *grad, *loss;
    int first;                    // the launch's first block
};

constexpr int kGradWaves = 16;
typedef short v4s16 __attribute__((ext_vector_type(4)));

// Sum of a value per wavefront of the workgroup, in wavefront order
__device__ __forceinline__ float block_sum(float v, float *sh)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kGradWaves; ++w) s += sh[w];
    return s;
}

// Every gradient of the network and the loss, sums over the M rows.  A
// workgroup owns a 32 x 32 tile of dW1^T = delta1^T X or dW2^T = delta2^T h1
// and its sixteen wavefronts take 32 rows each in turn, so the sum over the
// rows needs no atomics and no workspace and its order is fixed.  The rows are
// the contracted dimension, while memory holds them row by row: a wavefront
// stages 32 rows x 32 columns of both operands in its own LDS and reads them
// back transposed (ds_read_b64_tr_b16: 16 lanes read four rows of 16 entries
// and receive a column each).  4,096 rows take 14.7 us, where tiled GEMMs of
// strided operands over 8 and 16 workgroups took 1.5 ms; the reads bound it
// (every tile reads 128 bytes of every row).  The column sums db1 and db2 come from a second
// product with ones in the tiles of the first 32 columns.  dW3 = h2^T delta3
// (fp32 delta3, so no matrix instruction) takes eight workgroups more, db3 and
// the loss one.  Blocks go to the XCDs in turn: one XCD's tiles share their
// columns of X or h1, so its L2 holds an eighth of them.
template <bool AL>
__global__ void __launch_bounds__(1024) grad_kernel(GradArgs g)
{
    __shared__ __attribute__((aligned(16))) uint16_t stage[kGradWaves][2][32 * 32];
    __shared__ float sums[kGradWaves][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int block = g.first + (int)blockIdx.x, x = block & 7, j = block >> 3;
    if (j == 25) {
        // db3 and the loss
        float sd = 0.0f, sl = 0.0f;
        for (int m = threadIdx.x; m < g.M; m += 64 * kGradWaves) {
            const float z = g.logit[m];
            sd += g.d3 ? g.d3[m] : logit_delta(z, g.y[m], g.M);
            // softplus(z) - y z, computed stably
            const float sp = z > 0.0f ? z + log1pf(__expf(-z)) : log1pf(__expf(z));
            sl += (sp - g.y[m] * z) / (float)g.M;
        }
        sd = block_sum(sd, sums[0]);
        sl = block_sum(sl, sums[0]);
        if (threadIdx.x == 0) {
            g.loss[0] = sl;
            g.grad[O_B3] = sd;
            g.grad[O_B3 + 1] = g.grad[O_B3 + 2] = g.grad[O_B3 + 3] = 0.0f;
        }
        return;
    }
    const int pr = lane >> 2, pc = (lane & 3) * 8;  // this lane's piece of 16 rows x 32 columns
    if (j == 24) {
        // dW3 of columns 32x .. 32x+31
        float s[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) s[q] = 0.0f;
        for (int m = wave * 16 + pr; m < g.M; m += 16 * kGradWaves) {
            const v4u32 h = load8<AL>(g.h2 + (int64_t)m * HID + 32 * x + pc);
            const float d = g.d3[m];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s[2 * q] += d * from_bf16((uint16_t)h[q]);
                s[2 * q + 1] += d * from_bf16((uint16_t)(h[q] >> 16));
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            for (int off = 32; off >= 4; off >>= 1) s[q] += __shfl_xor(s[q], off);
            if (lane < 4) sums[wave][pc + q] = s[q];
        }
        __syncthreads();
        if (threadIdx.x < 32) {
            float t = 0.0f;
            for (int w = 0; w < kGradWaves; ++w) t += sums[w][threadIdx.x];
            g.grad[O_W3 + 32 * x + threadIdx.x] = t;
        }
        return;
    }
    const bool first = j < 16;  // dW1^T, else dW2^T
    const uint16_t *A = first ? g.d1 : g.d2, *Bm = first ? g.X : g.h1;
    const int K = first ? IN : HID;
    const int n0 = 32 * (j & 7), k0 = 32 * (first ? (j >> 3) * 8 + x : x);
    const bool colsum = k0 == 0;
    v16f32 acc, one;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = one[q] = 0.0f;
    v8bf16 ones;
#pragma unroll
    for (int q = 0; q < 8; ++q) ones[q] = (__bf16)1.0f;
    uint16_t *sa = stage[wave][0], *sb = stage[wave][1];
    // transposed read: lanes of group l/16 read rows 8*(l/32) + 0..3 (and 4..7)
    // at columns 16*((l/16)%2) + 0..15
    const int tr = (8 * (lane >> 5) + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    v4u32 ra[2], rb[2];
    const uint16_t *pa = A + n0 + pc, *pb = Bm + k0 + pc;
    const auto load = [&](int m0) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int m = m0 + pr + 16 * t;
            const int64_t mc = m < g.M ? m : g.M - 1;
            const uint32_t keep = m < g.M ? ~0u : 0u;  // zeros past the end
            ra[t] = load8<AL>(pa + mc * HID) & keep;
            rb[t] = load8<AL>(pb + mc * K) & keep;
        }
    };
    const auto transposed = [&](const uint16_t *s, int step) {
        typedef __attribute__((address_space(3))) v4s16 lds_v4;
        const v4s16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(s + tr + 16 * 32 * step));
        const v4s16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(s + tr + 16 * 32 * step + 4 * 32));
        return __builtin_bit_cast(v8bf16, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    int m0 = wave * 32;
    if (m0 < g.M) load(m0);
    for (; m0 < g.M; m0 += 32 * kGradWaves) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            *reinterpret_cast<v4u32 *>(sa + (pr + 16 * t) * 32 + pc) = ra[t];
            *reinterpret_cast<v4u32 *>(sb + (pr + 16 * t) * 32 + pc) = rb[t];
        }
        if (m0 + 32 * kGradWaves < g.M) load(m0 + 32 * kGradWaves);
        // the wavefront's own stores are complete before its reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int step = 0; step < 2; ++step) {
            const v8bf16 av = transposed(sa, step), bv = transposed(sb, step);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
            if (colsum) one = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, ones, one, 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // the wavefronts' partial tiles, each in its own 4 KiB of `stage`; register
    // q of lane l: row 8*(q/4) + 4*(l/32) + q%4, column l%32
    float *part = reinterpret_cast<float *>(&stage[0][0][0]);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
        part[wave * 1024 + r * 32 + (lane & 31)] = acc[q];
        if (colsum && (lane & 31) == 0) sums[wave][r] = one[q];
    }
    __syncthreads();
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kGradWaves; ++w) s += part[w * 1024 + threadIdx.x];
    g.grad[(first ? O_W1T : O_W2T) + (n0 + (threadIdx.x >> 5)) * K + k0 + (threadIdx.x & 31)] = s;
    if (colsum && threadIdx.x < 32) {
        float t = 0.0f;
        for (int w = 0; w < kGradWaves; ++w) t += sums[w][threadIdx.x];
        g.grad[(first ? O_B1 : O_B2) + n0 + threadIdx.x] = t;
    }
}
// blocks: dW1 and db1, dW2 and db2, dW3, then one for db3 and the loss
constexpr int kGradW1 = 0, kGradW2 = 8 * 16, kGradB3 = 8 * 25, kGradBlocks = kGradB3 + 1;
// `stage` holds a wavefront's operands and later its partial tile
static_assert(2 * 32 * 32 * sizeof(uint16_t) == 32 * 32 * sizeof(float), "stage size");

// bf16 compute copies of parameter i: W1^T, W2^T, W2, w3
__device__ __forceinline__ void copy_param(int i, float v, uint16_t *q)
{
    const uint16_t h = to_bf16(v);
    if (i < O_B1) {
        q[Q_W1T + i] = h;
    } else if (i >= O_W2T && i < O_B2) {
        const int e = i - O_W2T, n = e / HID, k = e % HID;  // W2[k][n] = W2^T[n][k]
        q[Q_W2T + e] = h;
        q[Q_W2 + k * HID + n] = h;
    } else if (i >= O_W3 && i < O_B3) {
        q[Q_W3 + i - O_W3] = h;
    }
}

// Adam (Kingma & Ba) on the fp32 masters, then their bf16 copies
__global__ void __launch_bounds__(256) adam_kernel(float *p, const float *g, float *m, float *v,
                                                   uint16_t *q, float lr, float b1, float b2,
                                                   float eps, float c1, float c2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= TSF_MLP_NPARAM) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    copy_param(i, pi, q);
}

__global__ void __launch_bounds__(256) sync_kernel(const float *p, uint16_t *q)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < TSF_MLP_NPARAM) copy_param(i, p[i], q);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// whether two arrays of M rows of `a` and `b` bytes share memory
bool overlap(const void *p, int64_t a, const void *q, int64_t b, int64_t M)
{
    const char *x = (const char *)p, *y = (const char *)q;
    return p && q && x < y + M * b && y < x + M * a;
}

// The rows of a workgroup, by what fills the 256 CUs in one turn: 128 rows
// (eight wavefronts) above 16,384 rows, 64 above 8,192, 32 below.  The weights,
// 384 KiB through every workgroup, favour large blocks (32,768 rows: 19.9 us
// with 128 rows, 26.3 us with 64) until CUs are left idle (16,384 rows: 13.4 us
// with 64).
int rows_per_block(int M) { return M > 16384 ? 128 : M > 8192 ? 64 : 32; }

// The most rows that a pass takes: a launch has at most 2^32 threads, eight per
// row with 32-row blocks, and rows are numbered in 32 bits; both are far away.
constexpr int kMaxRows = 65535 * 64;

tsf_status check_net(const tsf_mlp *net)
{
    if (!net || !net->param || !net->wbf) return tsf_fail(TSF_E_ARG, "null network buffers");
    return TSF_OK;
}

}  // namespace

tsf_status mlp_forward(const tsf_mlp *net, const uint16_t *X, int32_t M, uint16_t *h1,
                       uint16_t *h2, float *logit, void *hip_stream)
{
    tsf_status st = check_net(net);
    if (st) return st;
    if (M == 0) return TSF_OK;
    if (M > kMaxRows) return tsf_fail(TSF_E_ARG, "%d rows exceed the %d of a call", M, kMaxRows);
    FwdArgs g{X, net->wbf + Q_W1T, net->wbf + Q_W2T, net->wbf + Q_W3, net->param + O_B1,
              net->param + O_B2, net->param + O_B3, M, h1, h2, logit, 0};
    const bool al = aligned16(X) && aligned16(net->wbf) && aligned16(h1) && aligned16(h2);
    constexpr int kX = 2 * IN, kH = 2 * HID;
    if (h1 && h2 && (overlap(h2, kH, X, kX, M) || overlap(logit, 4, X, kX, M) ||
                     overlap(logit, 4, h1, kH, M))) {
        auto *fn = al ? fwd_kernel<1, 1, true, true> : fwd_kernel<1, 1, false, true>;
        for (g.step = 0; g.step < 3; ++g.step)
            hipLaunchKernelGGL(fn, dim3((M + 31) / 32), dim3(256), 0, (hipStream_t)hip_stream, g);
        if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "forward launch failed");
        return TSF_OK;
    }
    const int rows = al ? rows_per_block(M) : 32;
    auto *fn = !al ? fwd_kernel<1, 1, false> : rows == 128 ? fwd_kernel<2, 2, true>
                                             : rows == 64 ? fwd_kernel<1, 2, true>
                                                          : fwd_kernel<1, 1, true>;
    hipLaunchKernelGGL(fn, dim3((M + rows - 1) / rows), dim3(rows > 32 ? 512 : 256), 0,
                       (hipStream_t)hip_stream, g);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "forward launch failed");
    return TSF_OK;
}

extern "C" {

tsf_status tsf_mlp_sync(const tsf_mlp *net, void *hip_stream)
{
    tsf_status st = check_net(net);
    if (st) return st;
    hipLaunchKernelGGL(sync_kernel, dim3((TSF_MLP_NPARAM + 255) / 256), dim3(256), 0,
                       (hipStream_t)hip_stream, net->param, net->wbf);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "sync launch failed");
    return TSF_OK;
}

tsf_status tsf_mlp_fwd(const tsf_mlp *net, const uint16_t *X, int32_t M, uint16_t *h1,
                       uint16_t *h2, float *logit, void *hip_stream)
{
    tsf_status st = check_net(net);
    if (st) return st;
    if (M < 0 || (M > 0 && (!X || !h1 || !h2 || !logit))) return tsf_fail(TSF_E_ARG, "bad forward arguments");
    return mlp_forward(net, X, M, h1, h2, logit, hip_stream);
}

tsf_status tsf_mlp_bwd(const tsf_mlp *net, const uint16_t *X, const float *y, int32_t M,
                       const uint16_t *h1, const uint16_t *h2, const float *logit, uint16_t *d2,
                       uint16_t *d1, float *d3, float *loss, void *hip_stream)
{
    tsf_status st = check_net(net);
    if (st) return st;
    if (!net->grad) return tsf_fail(TSF_E_ARG, "null gradient buffer");
    if (M <= 0 || !X || !y || !h1 || !h2 || !logit || !d2 || !d1 || !d3 || !loss)
        return tsf_fail(TSF_E_ARG, "bad backward arguments");
    if (M > kMaxRows) return tsf_fail(TSF_E_ARG, "%d rows exceed the %d of a call", M, kMaxRows);
    hipStream_t s = (hipStream_t)hip_stream;
    const bool al = aligned16(X) && aligned16(net->wbf) && aligned16(h1) && aligned16(h2) &&
                    aligned16(d1) && aligned16(d2);
    const int rows = al ? rows_per_block(M) : 32;
    DeltaArgs d{logit, y, h1, h2, net->wbf + Q_W2, net->wbf + Q_W3, M, d3, d2, d1, 0};
    GradArgs g{X, h1, h2, d1, d2, d3, logit, y, M, net->grad, loss, 0};
    auto *gfn = al ? grad_kernel<true> : grad_kernel<false>;
    const auto grads = [&](int from, int to) {
        g.first = from;
        hipLaunchKernelGGL(gfn, dim3(to - from), dim3(64 * kGradWaves), 0, s, g);
    };
    constexpr int kH = 2 * HID;
    if (overlap(d3, 4, logit, 4, M) || overlap(d1, kH, h1, kH, M) || overlap(d1, kH, h2, kH, M) ||
        overlap(d1, kH, logit, 4, M) || overlap(d1, kH, y, 4, M) || overlap(d1, kH, d3, 4, M)) {
        // a workspace over an input: every input is used before it is overwritten
        auto *dfn = al ? delta_kernel<1, 1, true, true> : delta_kernel<1, 1, false, true>;
        const auto delta = [&](int step) {
            d.step = step;
            hipLaunchKernelGGL(dfn, dim3((M + 31) / 32), dim3(256), 0, s, d);
        };
        g.d3 = nullptr;
        grads(kGradB3, kGradBlocks);
        g.d3 = d3;
        delta(0);
        grads(kGradW2, kGradB3);
        delta(1);
        grads(kGradW1, kGradW2);
    } else {
        auto *dfn = !al ? delta_kernel<1, 1, false> : rows == 128 ? delta_kernel<2, 2, true>
                                                    : rows == 64 ? delta_kernel<1, 2, true>
                                                                 : delta_kernel<1, 1, true>;
        hipLaunchKernelGGL(dfn, dim3((M + rows - 1) / rows), dim3(rows > 32 ? 512 : 256), 0, s, d);
        grads(0, kGradBlocks);
    }
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "backward launch failed");
    return TSF_OK;
}

tsf_status tsf_mlp_step(const tsf_mlp *net, float lr, float beta1, float beta2, float eps,
                        int32_t step, void *hip_stream)
{
    tsf_status st = check_net(net);
    if (st) return st;
    if (!net->grad || !net->adam_m || !net->adam_v || step < 1)
        return tsf_fail(TSF_E_ARG, "bad optimiser arguments");
    hipStream_t s = (hipStream_t)hip_stream;
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3((TSF_MLP_NPARAM + 255) / 256), dim3(256), 0, s,
                       net->param, net->grad, net->adam_m, net->adam_v, net->wbf, lr, beta1, beta2,
                       eps, c1, c2);
    if (hipGetLastError() != hipSuccess) return tsf_fail(TSF_E_DEVICE, "adam launch failed");
    return TSF_OK;
}

}  // extern "C"
