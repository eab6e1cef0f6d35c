// hawkes_mlp.hip -- the BF16 surrogate network of the log-likelihood on gfx950.
//
// Network 6 -> 256 -> 256 -> 256 -> 1 with GELU activations (x Phi(x)):
//   h1 = W1 z + b1, a1 = gelu(h1), h2 = W2 a1 + b2, a2 = gelu(h2),
//   h3 = W3 a2 + b3, a3 = gelu(h3), f = w4 . a3 + b4.
// Flat parameter layout (133,633 values): W1 (256x6, out x in), b1, W2
// (256x256), b2, W3 (256x256), b3, w4 (256), b4.
//
// The state buffer holds FP32 master weights, the two Adam moment vectors,
// and BF16 working copies: the small blocks in the flat vector's own layout, and
// W2, W3, W2^T, W3^T twice: packed by row for the one-sample kernels and as
// matrix-core operand fragments (both below) for the batched kernels.
//
// Batched kernels (value and input gradient of many inputs, the training
// pass) run the 256 x 256 products on the matrix cores with
// v_mfma_f32_16x16x32_bf16, features as rows and 16 samples as columns: a
// workgroup of 16 waves per tile of 16 samples and a row tile per wave in
// training, 8 waves of two row tiles for one or two tiles of samples in
// inference.  A product's
// FP32 output sits in the lanes in the k order of the next product's column
// operand, so each wave converts its own outputs and the operands meet in
// LDS.  The weights are exact BF16; each FP32 activation enters as hi + lo
// BF16 parts (x = hi + lo + O(2^-18 |x|)), two products per operand, so the
// result matches FP32 activations times BF16 weights to ~1e-5 relative.
// One-sample kernels (a value and gradient at batch <= 8, a leapfrog
// trajectory) take the matrix-vector form with the weights in registers and
// LDS, whose latency is lower.
//
// Inference: value and input gradient per sample (k_mlp_forward for small
// batches, k_mlp_forward_mfma), or a whole leapfrog trajectory on the
// surrogate posterior in one workgroup (k_mlp_leapfrog, the stage-1 proposal
// of delayed-acceptance HMC).
//
// Training loss (value + gradient matching):
//   L = (1/B) sum_b (f(z_b) - y_b)^2 + lambda |grad_z f(z_b) - g_b|^2.
// Its parameter gradient uses d/dtheta [r . grad_z f] = d/dtheta [D_r f] for
// r = grad_z f - g held fixed: per sample a primal pass, the reverse pass for
// grad_z f, a forward tangent pass along r, and one reverse pass through the
// primal and tangent computations; the per-sample adjoint vectors are then
// contracted over the batch (matrix cores for W2 and W3, fixed-order wave
// reductions for the rest), the same way on every call (deterministic).

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "hawkes.h"
#include "hawkes_common.h"
#include "hawkes_gelu.h"
#include "hawkes_mlp.h"

namespace hawkes {
namespace {

constexpr int H = 256;
constexpr int DZ = 6;
constexpr int64_t P = HAWKES_MLP_PARAMS;
// offsets of the parameter blocks in the flat vector
constexpr int64_t OW1 = 0, OB1 = OW1 + H * DZ, OW2 = OB1 + H, OB2 = OW2 + H * H, OW3 = OB2 + H, OB3 = OW3 + H * H,
                  OW4 = OB3 + H, OB4 = OW4 + H;
static_assert(OB4 + 1 == P, "parameter layout");

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// Working copies of the 256 x 256 matrices, in this order.
enum { F_W2, F_W2T, F_W3, F_W3T };

struct StateLayout {
    size_t master, m, v, wb, pack[4], frag[4], total;
};

StateLayout state_layout()
{
    StateLayout s;
    size_t off = 0;
    s.master = off;
    off = align256(off + sizeof(float) * P);
    s.m = off;
    off = align256(off + sizeof(float) * P);
    s.v = off;
    off = align256(off + sizeof(float) * P);
    s.wb = off;
    off = align256(off + sizeof(uint16_t) * P);
    for (int i = 0; i < 4; ++i) {
        s.pack[i] = off;
        off = align256(off + sizeof(uint16_t) * H * H);
    }
    for (int i = 0; i < 4; ++i) {
        s.frag[i] = off;
        off = align256(off + sizeof(uint16_t) * H * H);
    }
    s.total = off;
    return s;
}

// The one-sample kernels' view.  A packed matrix M (out = M v) holds, for each
// eight consecutive k, the 16 bytes M[j][k..k+7] of every output j in turn.
struct Net {
    const uint16_t *w;      // flat BF16 copy (W1, the biases, w4, b4)
    const uint4 *pack[4];
};
__host__ __device__ inline int pack_index(int j, int k) { return ((k >> 3) * H + j) * 8 + (k & 7); }

Net net_of(const void *state)
{
    const StateLayout L = state_layout();
    const char *b = static_cast<const char *>(state);
    Net n;
    n.w = reinterpret_cast<const uint16_t *>(b + L.wb);
    for (int i = 0; i < 4; ++i)
        n.pack[i] = reinterpret_cast<const uint4 *>(b + L.pack[i]);
    return n;
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) unsigned short u16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// The batched kernels' view: the flat BF16 copy and the four operand copies.
struct MfNet {
    const uint16_t *w;
    const bf16x8 *frag[4];
};

MfNet mfnet_of(const void *state)
{
    const StateLayout L = state_layout();
    const char *b = static_cast<const char *>(state);
    MfNet n;
    n.w = reinterpret_cast<const uint16_t *>(b + L.wb);
    for (int i = 0; i < 4; ++i)
        n.frag[i] = reinterpret_cast<const bf16x8 *>(b + L.frag[i]);
    return n;
}

// Operand fragments.  A product out = M v over 256 features (M[m][k], m the
// output feature) is 16 row tiles x 8 chunks of 32 k; in a chunk, lane l
// (row m = 16 mt + l % 16, lane group q = l / 16) holds 8 consecutive BF16
// values at k = 32 kc + 4q + c (c < 4) and 32 kc + 16 + 4q + (c - 4) (c >= 4).
// That k order is the order in which the FP32 output of the previous product
// sits in the lanes (two 16-row tiles, rows 4q..4q+3 of each), so the output
// becomes the next column operand without leaving the lane; the column
// operand uses the same k order, so every k pairs with itself.  A lane's
// fragment is 16 contiguous bytes: fragment (mt, kc) of lane l at
// ((mt * 8 + kc) * 64 + l) * 8.
__host__ __device__ inline int frag_index(int m, int k)
{
    const int mt = m >> 4, lm = m & 15, kc = k >> 5, r = k & 31;
    const int upper = r >> 4, q = (r & 15) >> 2, c = upper * 4 + (r & 3);
    return ((mt * 8 + kc) * 64 + q * 16 + lm) * 8 + c;
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// round to nearest, ties to even; NaN stays NaN
__device__ inline uint16_t f32_to_bf16(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu))
        return uint16_t((u >> 16) | 0x40u);
    const uint32_t lsb = (u >> 16) & 1u;
    return uint16_t((u + 0x7fffu + lsb) >> 16);
}

// One-sample evaluation: value and input gradient by a workgroup of two groups
// of 256 threads, output feature j per thread.  Group 0 owns layer 2 (W2 and
// W2^T), group 1 layer 3 (W3 and W3^T); each thread keeps its row of the forward
// matrix and half of its row of the transposed one in registers (192 of 256),
// the other halves sit in LDS (128 KB), all of it loaded once.  A product is
// the fma chain over k = 0..255 in order.
// Bound: issue of those four chains by one wave per SIMD, 256 fmas and as many
// unpackings each, at about 8 clocks an instruction (loading the inputs further ahead
// changed nothing).  Reading the 512 KB of weights from L2 through one CU for
// every evaluation (two bytes per lane and load) took 16 us; resident they make
// it 7.5 us per step of a trajectory, and a single evaluation 12.2 us.
constexpr int ONE_WG = 2 * H;
constexpr int NS7 = 7;
struct OneLds {
    uint4 wt[2][H / 16][H];  // k = 128..255 of the transposed matrices
    float4 vec[2][H / 4];    // the product's input: products alternate
    float s2[H];
    float red[NS7][H];
    float sum[8];
};

struct OneWeights {
    uint4 fwd[H / 8], bwd[H / 16];
};

__device__ __forceinline__ void one_load(const Net &net, OneLds &L, OneWeights &W)
{
    const int grp = threadIdx.x >> 8, j = threadIdx.x & (H - 1);
    const uint4 *f = net.pack[grp ? F_W3 : F_W2], *t = net.pack[grp ? F_W3T : F_W2T];
#pragma unroll
    for (int c = 0; c < H / 8; ++c)
        W.fwd[c] = f[c * H + j];
#pragma unroll
    for (int c = 0; c < H / 16; ++c)
        W.bwd[c] = t[c * H + j];
#pragma unroll
    for (int c = 0; c < H / 16; ++c)
        L.wt[grp][c][j] = t[(H / 16 + c) * H + j];  // read by this thread only
}

__device__ __forceinline__ float lo_bf16(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi_bf16(unsigned u) { return __uint_as_float(u & 0xffff0000u); }

// The weights as values of this evaluation: their unpacking is the same in every one, and
// the compiler would otherwise keep it in (twice as many) registers.
__device__ __forceinline__ void renew(uint4 &w)
{
    asm volatile("" : "+v"(w.x), "+v"(w.y), "+v"(w.z), "+v"(w.w));
}

// acc + eight terms of a chain: weights w, inputs a and b
__device__ __forceinline__ float chain8(float acc, const uint4 &w, const float4 &a, const float4 &b)
{
    acc = fmaf(lo_bf16(w.x), a.x, acc);
    acc = fmaf(hi_bf16(w.x), a.y, acc);
    acc = fmaf(lo_bf16(w.y), a.z, acc);
    acc = fmaf(hi_bf16(w.y), a.w, acc);
    acc = fmaf(lo_bf16(w.z), b.x, acc);
    acc = fmaf(hi_bf16(w.z), b.y, acc);
    acc = fmaf(lo_bf16(w.w), b.z, acc);
    acc = fmaf(hi_bf16(w.w), b.w, acc);
    return acc;
}
// acc + the chain over N chunks of 8 with weights in registers; inputs are loaded one
// chunk ahead
template <int N>
__device__ __forceinline__ float chain_reg(float acc, const float4 *v, uint4 (&w)[N])
{
    float4 a = v[0], b = v[1];
#pragma unroll
    for (int c = 0; c < N; ++c) {
        float4 na = a, nb = b;
        if (c + 1 < N) {
            na = v[2 * c + 2];
            nb = v[2 * c + 3];
        }
        renew(w[c]);
        acc = chain8(acc, w[c], a, b);
        asm volatile("" : "+v"(acc));
        a = na;
        b = nb;
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}
// the same with weights in LDS, loaded one chunk ahead too
template <int N>
__device__ __forceinline__ float chain_lds(float acc, const float4 *v, const uint4 (*wt)[H], int j)
{
    float4 a = v[0], b = v[1];
    uint4 w = wt[0][j];
#pragma unroll
    for (int c = 0; c < N; ++c) {
        float4 na = a, nb = b;
        uint4 nw = w;
        if (c + 1 < N) {
            na = v[2 * c + 2];
            nb = v[2 * c + 3];
            nw = wt[c + 1][j];
        }
        acc = chain8(acc, w, a, b);
        asm volatile("" : "+v"(acc));
        a = na;
        b = nb;
        w = nw;
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}
__device__ __forceinline__ float dot_fwd(OneWeights &W, const float4 *v) { return chain_reg(0.0f, v, W.fwd); }
__device__ __forceinline__ float dot_bwd(OneWeights &W, const uint4 (*wt)[H], int j, const float4 *v)
{
    return chain_lds<H / 16>(chain_reg(0.0f, v, W.bwd), v + H / 8, wt, j);
}

// Sum over the wave's 64 values in the pairwise order x[l] += x[l + w], w = 32, 16, ..., 1
// (lane 0's value of that tree, in every lane: an addition's two orders give the same bits)
__device__ __forceinline__ float tree_sum64(float x)
{
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    auto ror = [&](auto c) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x120 + decltype(c)::value, 0xf, 0xf, true));
    };
    x += ror(std::integral_constant<int, 8>{});
    x += ror(std::integral_constant<int, 4>{});
    x += ror(std::integral_constant<int, 2>{});
    x += ror(std::integral_constant<int, 1>{});
    return x;
}

// The small weights a thread needs: its row of W1, its biases and output weight.
struct OneSmall {
    float w1[DZ], b1, bias, w4;
};
__device__ __forceinline__ OneSmall one_small(const uint16_t *__restrict__ w)
{
    const int grp = threadIdx.x >> 8, j = threadIdx.x & (H - 1);
    OneSmall o;
#pragma unroll
    for (int i = 0; i < DZ; ++i)
        o.w1[i] = bf16_to_f32(w[OW1 + j * DZ + i]);
    o.b1 = bf16_to_f32(w[OB1 + j]);
    o.bias = bf16_to_f32(w[(grp ? OB3 : OB2) + j]);
    o.w4 = bf16_to_f32(w[OW4 + j]);
    return o;
}

// Value (without b4) and input gradient of the input sz[DZ] (in LDS, published by the
// caller's barrier) into L.sum[0..6], published by a barrier here.
__device__ __forceinline__ void value_and_grad(OneWeights &W, const OneSmall &o, const float *sz, OneLds &L)
{
    const int grp = threadIdx.x >> 8, j = threadIdx.x & (H - 1);
    float *v0 = reinterpret_cast<float *>(L.vec[0]), *v1 = reinterpret_cast<float *>(L.vec[1]);
    float s1 = 0.0f;
    if (grp == 0) {
        float h1 = o.b1;
#pragma unroll
        for (int i = 0; i < DZ; ++i)
            h1 = fmaf(o.w1[i], sz[i], h1);
        v0[j] = gelu(h1);
        s1 = gelu_d1(h1);
    }
    __syncthreads();
    if (grp == 0) {
        const float h2 = o.bias + dot_fwd(W, L.vec[0]);
        v1[j] = gelu(h2);
        L.s2[j] = gelu_d1(h2);
    }
    __syncthreads();
    if (grp == 1) {
        const float h3 = o.bias + dot_fwd(W, L.vec[1]);
        L.red[0][j] = o.w4 * gelu(h3);  // summed with the input gradient below
        v0[j] = o.w4 * gelu_d1(h3);
    }
    __syncthreads();
    if (grp == 1)
        v1[j] = L.s2[j] * dot_bwd(W, L.wt[1], j, L.vec[0]);  // (W3^T d3)_j
    __syncthreads();
    if (grp == 0) {
        const float d1 = s1 * dot_bwd(W, L.wt[0], j, L.vec[1]);
#pragma unroll
        for (int i = 0; i < DZ; ++i)
            L.red[1 + i][j] = o.w1[i] * d1;
    }
    __syncthreads();
    const int z = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (z < NS7) {
        const float *r = L.red[z];
        const float s = tree_sum64((r[l] + r[l + 128]) + (r[l + 64] + r[l + 192]));
        if (l == 0)
            L.sum[z] = s;
    }
    __syncthreads();
}

// Value and input gradient, one workgroup per sample.
__global__ __launch_bounds__(ONE_WG) void k_mlp_forward(Net net, const float *__restrict__ z, int64_t B,
                                                        float *__restrict__ f_out, float *__restrict__ gz_out)
{
    __shared__ float sz[DZ];
    __shared__ OneLds L;
    OneWeights W;
    const int j = threadIdx.x;
    const int64_t b = blockIdx.x;
    if (j < DZ)
        sz[j] = z[b * DZ + j];
    const OneSmall o = one_small(net.w);
    one_load(net, L, W);
    __syncthreads();
    value_and_grad(W, o, sz, L);
    if (j == 0)
        f_out[b] = L.sum[0] + bf16_to_f32(net.w[OB4]);
    if (gz_out && j < DZ)
        gz_out[b * DZ + j] = L.sum[1 + j];
}

// A leapfrog trajectory on the surrogate posterior in one workgroup (the
// stage-1 proposal of delayed-acceptance HMC): n_steps steps of
// H(z, p) = -s(z) + p' M^-1 p / 2 with
//   s(z) = s_y f((z - m_z) / s_z) + m_y - z.z / (2 prior_var),
// from (z, p) with grad = ds/dz at z: half a momentum step, then per step a
// position step, s and its gradient at the new point, and a full momentum
// step (half a step after the last one).  Position and momentum updates are
// FP64 without contraction, in the operation order of a host-side leapfrog
// written the same way; a step whose s or gradient is not finite ends the
// trajectory (s = -inf, no final half step).  Every wave runs the six
// components' updates in its lanes 0..5 on the same values, so that the
// trajectory needs no barrier beyond the network's.
__global__ __launch_bounds__(ONE_WG) void k_mlp_leapfrog(Net net, hawkes_mlp_leapfrog_io *io, int n)
{
#pragma clang fp contract(off)
    __shared__ float sz[DZ];
    __shared__ OneLds L;
    OneWeights W;
    const int l = threadIdx.x & 63, d = l < DZ ? l : 0;
    const OneSmall o = one_small(net.w);
    one_load(net, L, W);
    const float b4 = bf16_to_f32(net.w[OB4]);
    const double eps = io->eps, m_y = io->m_y, s_y = io->s_y, pv = io->prior_var;
    const double im = io->inv_mass[d], mz = io->m_z[d], szc = io->s_z[d];
    double z = io->z[d], p = io->p[d] + (0.5 * eps) * io->grad[d], g = 0.0, sval = 0.0;
    bool ok = true;
    __syncthreads();  // every wave has read io before any writes it
    for (int step = 0; step < n; ++step) {
        z = z + (eps * im) * p;
        if (threadIdx.x < DZ)
            sz[threadIdx.x] = float((z - mz) / szc);
        __syncthreads();
        value_and_grad(W, o, sz, L);
        g = (double(L.sum[1 + d]) * s_y) / szc - z / pv;
        double zz = 0.0;
        for (int i = 0; i < DZ; ++i) {
            const double zi = __shfl(z, i);
            zz = zz + zi * zi;
        }
        const float f = L.sum[0] + b4;
        sval = (double(f) * s_y + m_y) - (0.5 * zz) / pv;
        ok = isfinite(sval) && __ballot(!isfinite(g)) == 0;
        if (!ok)
            break;
        if (step + 1 < n)
            p = p + eps * g;
    }
    if (ok && n > 0)
        p = p + (0.5 * eps) * g;
    if (threadIdx.x < DZ) {
        io->z[l] = z;
        io->p[l] = p;
        io->grad[l] = g;
    }
    if (threadIdx.x == 0) {
        io->s = ok ? sval : -HUGE_VAL;
        io->status = ok ? 1.0 : 0.0;
    }
}

// ------------------------------------------------------------------ batched kernels (matrix cores)

// Training: a workgroup of 16 waves takes 16 samples.  In every 256-feature product the
// wave w computes row tile w (features 16w..16w+15) for the 16 samples: lane l
// (sample l % 16, lane group q = l / 16) holds v[i] of feature 16 w + 4 q + i
// (i = 0..3).  A product's column operand (all 256 features) is published
// through LDS: wave w converts its 4 values to half of the hi + lo BF16 operands
// of chunk w / 2, every wave then reads all 8 chunks.  One row tile per wave and
// four waves per SIMD: a wave issues a VALU instruction every 8 clocks or so,
// and most instructions here are elementwise (GELUs, operand splits).  Bound:
// those, then the L2 latency of the weights at each of a workgroup's ten serial
// products.  A step at batch 256 47.8 -> 42.0 us against 8 waves of two row tiles, with the
// same bits (then 35.2, see mf_product).  (The inference pass, below, has its own split.)
constexpr int NWAVE = 16;
constexpr int VPL = 4;  // values per lane

__device__ inline int feat(int w, int q, int i) { return 16 * w + 4 * q + i; }

typedef __attribute__((ext_vector_type(8))) float f32x8;
__device__ inline void split8(const float x[8], bf16x8 &hi, bf16x8 &lo)
{
    f32x8 v;
#pragma unroll
    for (int c = 0; c < 8; ++c)
        v[c] = x[c];
    hi = __builtin_convertvector(v, bf16x8);  // round to nearest even, two values an instruction
    lo = __builtin_convertvector(v - __builtin_convertvector(hi, f32x8), bf16x8);
}

// The wave's 8 weight fragments of a product (its row tile x 8 chunks),
// requested ahead of the product: the callers issue them before the elementwise
// work that forms the product's input, which then hides the memory latency.
typedef bf16x8 Frags[8];

__device__ inline void load_frags(const bf16x8 *__restrict__ M, Frags &a)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int kc = 0; kc < 8; ++kc)
        a[kc] = M[(w * 8 + kc) * 64 + l];
    // keep the loads here: the scheduler would otherwise sink each next to its use
    __builtin_amdgcn_sched_barrier(0);
}

// Column operands in LDS: two slots (consecutive products alternate), 8 chunks, hi and lo, 64
// lanes of two halves (row tiles 2 kc and 2 kc + 1).
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4v;
using Operands = bf16x8[2][8][2][64];

// y = M x for the workgroup's 16 samples (M's fragments in a), x given by each wave's
// values.  A fragment's registers take the next product's (null: the same matrix again) as soon
// as it is used, so that reading a matrix from L2 (2048 clocks for one CU) runs beside this
// product's operand reads from LDS (as many): a step at batch 256 42.0 -> 35.2 us against
// loading it between the products.  (The branch on next also parts the chunks' code: taken away, the
// registers spill and the step takes 39.7 us.)  Element c of chunk kc is the value of row tile 2 kc + c / 4, row 4 q + c % 4.
__device__ inline void mf_product(Frags &a, const bf16x8 *__restrict__ next, const float x[VPL], float y[VPL],
                                  Operands &op, int slot)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    // the values as rounded: the compiler would fuse the subtraction below into the product
    // that formed them, and the lo part would belong to another number than hi
    float r[VPL];
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
        r[c] = x[c];
        asm volatile("" : "+v"(r[c]));
    }
    const f32x4v v = {r[0], r[1], r[2], r[3]};
    const bf16x4 hi = __builtin_convertvector(v, bf16x4);  // to nearest even, two values an instruction
    const bf16x4 lo = __builtin_convertvector(v - __builtin_convertvector(hi, f32x4v), bf16x4);
    reinterpret_cast<bf16x4 *>(&op[slot][w >> 1][0][l])[w & 1] = hi;
    reinterpret_cast<bf16x4 *>(&op[slot][w >> 1][1][l])[w & 1] = lo;
    __syncthreads();
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 bh = op[slot][0][0][l], bl = op[slot][0][1][l];
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) {
        // the next chunk's operands are read during this chunk's products, and no further ahead
        const bf16x8 nh = op[slot][kc < 7 ? kc + 1 : kc][0][l], nl = op[slot][kc < 7 ? kc + 1 : kc][1][l];
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kc], bl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kc], bh, acc, 0, 0, 0);
        bh = nh;
        bl = nl;
        if (next)
            a[kc] = next[(w * 8 + kc) * 64 + l];
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r4 = 0; r4 < VPL; ++r4)
        y[r4] = acc[r4];
}

// sum over the four lane groups that hold one sample (every lane gets the same bits)
__device__ inline float group_sum(float x)
{
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    return x;
}

// sum over the wave by a fixed butterfly
__device__ inline float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        x += __shfl_xor(x, o);
    return x;
}

constexpr int NRED = 7;  // per-sample sums: value and input gradient

// Layer-1 weights, biases and output weights in FP32, staged in LDS by each
// workgroup of the batched kernels.
struct SmallW {
    float w1[DZ][H];
    float b1[H], b2[H], b3[H], w4[H];
};

__device__ inline void stage_small(const uint16_t *__restrict__ w, SmallW &sw)
{
    for (int p = threadIdx.x; p < H * DZ; p += blockDim.x)
        sw.w1[p % DZ][p / DZ] = bf16_to_f32(w[OW1 + p]);
    for (int f = threadIdx.x; f < H; f += blockDim.x) {
        sw.b1[f] = bf16_to_f32(w[OB1 + f]);
        sw.b2[f] = bf16_to_f32(w[OB2 + f]);
        sw.b3[f] = bf16_to_f32(w[OB3 + f]);
        sw.w4[f] = bf16_to_f32(w[OW4 + f]);
    }
    __syncthreads();
}

// Value and input gradient, 16 NS samples (NS column tiles) per workgroup of 8 waves, two
// row tiles per wave: wave w holds features 32 w .. 32 w + 31, which are operand chunk w, so a
// lane's 8 values of a sample are one operand entry, and every operand that a wave reads serves
// two row tiles, every weight fragment NS column tiles.  GELU slopes stay in registers; with 74 KB
// of LDS two workgroups share a CU, and one's products (LDS reads, 128 NS KB each) run
// beside the other's GELUs.  Bound: the GELUs' VALU work, then those reads.  Against workgroups of
// 16 waves and 32 samples, one per CU, with the slopes in LDS (all waves in the same phase, twice the
// operand reads): 21,000 samples 43.3 -> 35.7 us, 100,000 181 -> 134 us.
//   NS: two while that fills the chip; the last FWD_RESIDENT tiles or fewer go one to a workgroup,
// which spreads them (a lone workgroup of two tiles takes half as long again): 300 samples 15.0 ->
// 9.3 us, 5,000 15.4 -> 13.4, 17,000 34.6 -> 28.4 (second figures in pairs: 15.5, 16.2, 34.6).
constexpr int64_t FWD_RESIDENT = 512;  // workgroups that the chip's 256 CUs hold at once
constexpr int FWD_WAVES = 8, FWD_ROWS = 2, FWD_VPL = 4 * FWD_ROWS;
template <int NS>
constexpr int FWD_AHEAD = (NS == 1) ? 3 : 1;  // chunks of weight fragments requested ahead
template <int NS>
using FwdOperands = bf16x8[2][NS][8][2][64];
template <int NS>
using FwdFrags = bf16x8[FWD_AHEAD<NS>][FWD_ROWS];

template <int NS>
__device__ inline void fwd_frags(const bf16x8 *__restrict__ M, int kc, FwdFrags<NS> &a)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int t = 0; t < FWD_ROWS; ++t)
        a[kc % FWD_AHEAD<NS>][t] = M[((FWD_ROWS * w + t) * 8 + kc) * 64 + l];
}

// the first chunks of a product's fragments, requested before the elementwise work in front of it
template <int NS>
__device__ inline void fwd_frags_first(const bf16x8 *__restrict__ M, FwdFrags<NS> &a)
{
#pragma unroll
    for (int kc = 0; kc < FWD_AHEAD<NS>; ++kc)
        fwd_frags<NS>(M, kc, a);
    __builtin_amdgcn_sched_barrier(0);
}

// y = M x; x and y may be the same array
template <int NS>
__device__ inline void fwd_product(const bf16x8 *__restrict__ M, FwdFrags<NS> &a, const float (*x)[FWD_VPL],
                                   float (*y)[FWD_VPL], FwdOperands<NS> &op, int slot)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        float r[FWD_VPL];  // the values as rounded, as in mf_product
#pragma unroll
        for (int c = 0; c < FWD_VPL; ++c) {
            r[c] = x[s][c];
            asm volatile("" : "+v"(r[c]));
        }
        bf16x8 hi, lo;
        split8(r, hi, lo);
        op[slot][s][w][0][l] = hi;
        op[slot][s][w][1][l] = lo;
    }
    __syncthreads();
    f32x4 acc[NS][FWD_ROWS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < FWD_ROWS; ++t)
            acc[s][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 ph[NS], pl[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        ph[s] = op[slot][s][0][0][l];
        pl[s] = op[slot][s][0][1][l];
    }
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bf16x8 bh = ph[s], bl = pl[s];
            if (kc < 7) {
                ph[s] = op[slot][s][kc + 1][0][l];
                pl[s] = op[slot][s][kc + 1][1][l];
            }
#pragma unroll
            for (int t = 0; t < FWD_ROWS; ++t) {
                acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kc % FWD_AHEAD<NS>][t], bl, acc[s][t], 0, 0, 0);
                acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kc % FWD_AHEAD<NS>][t], bh, acc[s][t], 0, 0, 0);
            }
        }
        if (kc + FWD_AHEAD<NS> < 8)
            fwd_frags<NS>(M, kc + FWD_AHEAD<NS>, a);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < FWD_ROWS; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                y[s][4 * t + r] = acc[s][t][r];
}

template <int NS>
struct FwdLds {
    SmallW sw;
    FwdOperands<NS> op;
};

// samples b0 .. b0 + 16 NS - 1
template <int NS>
__device__ __forceinline__ void forward_tiles(const MfNet &net, const float *__restrict__ z, int64_t b0, int64_t B,
                                              float *__restrict__ f_out, float *__restrict__ gz_out, FwdLds<NS> &L)
{
    SmallW &sw = L.sw;
    FwdOperands<NS> &op = L.op;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4;
    auto feat = [&](int i) { return 32 * w + 16 * (i >> 2) + 4 * q + (i & 3); };
    FwdFrags<NS> a;
    fwd_frags_first<NS>(net.frag[F_W2], a);
    stage_small(net.w, sw);
    float v[NS][FWD_VPL], s1[NS][FWD_VPL], s2[NS][FWD_VPL];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int64_t b = b0 + 16 * s + (l & 15);
        float zi[DZ];
#pragma unroll
        for (int d = 0; d < DZ; ++d)
            zi[d] = b < B ? z[b * DZ + d] : 0.0f;
#pragma unroll
        for (int i = 0; i < FWD_VPL; ++i) {
            float h = sw.b1[feat(i)];
#pragma unroll
            for (int d = 0; d < DZ; ++d)
                h = fmaf(sw.w1[d][feat(i)], zi[d], h);
            const Gelu g = gelu_all(h);
            v[s][i] = g.a;
            s1[s][i] = g.d1;
        }
    }
    fwd_product<NS>(net.frag[F_W2], a, v, v, op, 0);
    fwd_frags_first<NS>(net.frag[F_W3], a);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < FWD_VPL; ++i) {
            const Gelu g = gelu_all(v[s][i] + sw.b2[feat(i)]);
            v[s][i] = g.a;
            s2[s][i] = g.d1;
        }
    fwd_product<NS>(net.frag[F_W3], a, v, v, op, 1);
    fwd_frags_first<NS>(net.frag[F_W3T], a);
    float acc[NS][NRED] = {};
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < FWD_VPL; ++i) {
            const Gelu g = gelu_all(v[s][i] + sw.b3[feat(i)]);
            const float w4 = sw.w4[feat(i)];
            acc[s][0] = fmaf(w4, g.a, acc[s][0]);
            v[s][i] = w4 * g.d1;
        }
    // input gradient: d2 = s2 (W3^T d3), d1 = s1 (W2^T d2), g = W1^T d1
    fwd_product<NS>(net.frag[F_W3T], a, v, v, op, 0);
    fwd_frags_first<NS>(net.frag[F_W2T], a);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < FWD_VPL; ++i)
            v[s][i] *= s2[s][i];
    fwd_product<NS>(net.frag[F_W2T], a, v, v, op, 1);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < FWD_VPL; ++i) {
            const float d1 = v[s][i] * s1[s][i];
#pragma unroll
            for (int d = 0; d < DZ; ++d)
                acc[s][1 + d] = fmaf(sw.w1[d][feat(i)], d1, acc[s][1 + d]);
        }
    // the sample's sums: lane groups, then the waves in order through LDS (slot 0 of the operands,
    // which every wave finished reading before the last product's barrier), a thread per sum
    auto *red = reinterpret_cast<float (*)[16 * NS][NRED]>(&op[0]);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int k = 0; k < NRED; ++k) {
            const float t = group_sum(acc[s][k]);
            if (l < 16)
                red[w][16 * s + l][k] = t;
        }
    __syncthreads();
    if (threadIdx.x >= 16 * NS * NRED)
        return;
    const int sample = threadIdx.x / NRED, k = threadIdx.x % NRED;
    if (b0 + sample >= B)
        return;
    float t = red[0][sample][k];
#pragma unroll
    for (int ww = 1; ww < FWD_WAVES; ++ww)
        t += red[ww][sample][k];
    if (k == 0)
        f_out[b0 + sample] = t + bf16_to_f32(net.w[OB4]);
    else if (gz_out)
        gz_out[(b0 + sample) * DZ + k - 1] = t;
}

// The first `pairs` workgroups take two sample tiles, the others one.
__global__ __launch_bounds__(64 * FWD_WAVES) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_mlp_forward_mfma(
    MfNet net, const float *__restrict__ z, int64_t B, int pairs, float *__restrict__ f_out,
    float *__restrict__ gz_out)
{
    __shared__ alignas(16) char lds[sizeof(FwdLds<2>)];
    const int block = blockIdx.x;
    if (block < pairs)
        forward_tiles<2>(net, z, int64_t(block) * 32, B, f_out, gz_out, *reinterpret_cast<FwdLds<2> *>(lds));
    else
        forward_tiles<1>(net, z, (int64_t(block) + pairs) * 16, B, f_out, gz_out, *reinterpret_cast<FwdLds<1> *>(lds));
}

// Training pass.  Per-sample vectors of the parameter gradient, feature-major
// for the batch contraction: vec[(v * H + f) * bp + b], bp = batch rounded up
// to 32 (padding samples hold zeros).
struct TrainWs {
    float *vec;    // [12][H][bp]: h1b t1b | h2b t2b a1 u1 | h3b t3b a2 u2 | a3 u3
    float *zr;     // [12][bp]: z (6), r (6)
    float *cf;     // [bp]
    float *loss;   // [bp]
    int64_t bp;
};
constexpr int NV = 12;
enum { V_H1B, V_T1B, V_H2B, V_T2B, V_A1, V_U1, V_H3B, V_T3B, V_A2, V_U2, V_A3, V_U3 };

// a vector's base is uniform and a lane's place in it, in bytes, the same for all twelve (below
// 2^32: bp <= 2^22), so that a store needs no address arithmetic of its own
__device__ inline void put_vec(const TrainWs &ws, int vi, const uint32_t place[VPL], bool valid, const float x[VPL])
{
    char *base = reinterpret_cast<char *>(ws.vec + int64_t(vi) * H * ws.bp);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        uint32_t o = place[i];
        asm volatile("" : "+v"(o));  // widened here, where the store can take it as its 32-bit offset
        *reinterpret_cast<float *>(base + o) = valid ? x[i] : 0.0f;
    }
}

// GELU of a layer's pre-activation h = y + bias: activation, slope and curvature
__device__ inline void layer_primal(const float *bias, int w, int q, const float y[VPL], float a[VPL], float s[VPL],
                                    float c[VPL])
{
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const float h = y[i] + bias[feat(w, q, i)];
        a[i] = gelu(h);
        s[i] = gelu_d1(h);
        c[i] = gelu_d2(h);
    }
}

// Adjoints of one layer's pre-activation from those of its activation (ab) and
// of the activation's tangent (ub): h_b = ab s + ub c t and t_b = ub s, with
// the GELU slope s and curvature c and the tangent t of the layer.
__device__ inline void layer_adjoint(float ab[VPL], float ub[VPL], const float s[VPL], const float c[VPL],
                                     const float t[VPL])
{
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const float hb = fmaf(ab[i], s[i], ub[i] * c[i] * t[i]);  // fused on this side for any code around it
        ub[i] = ub[i] * s[i];
        ab[i] = hb;
    }
}

__global__ __launch_bounds__(64 * NWAVE) void k_mlp_train_mfma(MfNet net, const float *__restrict__ z,
                                                       const float *__restrict__ y, const float *__restrict__ g,
                                                       int64_t B, float lam, TrainWs ws)
{
    __shared__ SmallW sw;
    __shared__ Operands op;
    __shared__ float red[NWAVE / 2][64][NRED], pairs[NWAVE / 2][16][NRED], total[16][NRED];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4;
    const int64_t b = int64_t(blockIdx.x) * 16 + (l & 15);
    const bool valid = b < B;
    stage_small(net.w, sw);
    float zi[DZ], gt[DZ];
#pragma unroll
    for (int d = 0; d < DZ; ++d) {
        zi[d] = valid ? z[b * DZ + d] : 0.0f;
        gt[d] = valid ? g[b * DZ + d] : 0.0f;
    }
    const float yb = valid ? y[b] : 0.0f;
    uint32_t place[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        place[i] = (uint32_t(feat(w, q, i)) * uint32_t(ws.bp) + uint32_t(b)) * 4u;
    float s1[VPL], s2[VPL], s3[VPL], c1[VPL], c2[VPL], c3[VPL], t1[VPL], t2[VPL], t3[VPL];
    float v[VPL], u[VPL], x[VPL];
    Frags a;
    load_frags(net.frag[F_W2], a);
    // primal pass
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const int f = feat(w, q, i);
        float h = 0.0f;
#pragma unroll
        for (int d = 0; d < DZ; ++d)
            h = fmaf(sw.w1[d][f], zi[d], h);
        x[i] = h;
    }
    layer_primal(sw.b1, w, q, x, v, s1, c1);
    put_vec(ws, V_A1, place, valid, v);
    mf_product(a, net.frag[F_W3], v, x, op, 0);
    layer_primal(sw.b2, w, q, x, v, s2, c2);
    put_vec(ws, V_A2, place, valid, v);
    mf_product(a, net.frag[F_W3T], v, x, op, 1);
    layer_primal(sw.b3, w, q, x, v, s3, c3);
    put_vec(ws, V_A3, place, valid, v);
    float acc[NRED] = {};
    float a3[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        a3[i] = v[i];
    // input gradient
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        v[i] = sw.w4[feat(w, q, i)] * s3[i];
    mf_product(a, net.frag[F_W2T], v, x, op, 0);
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        v[i] = x[i] * s2[i];
    mf_product(a, net.frag[F_W2], v, x, op, 1);
    // value and input gradient of the sample: a lane's fma chain runs over the two row tiles of
    // a wave pair (even wave first), then the lane groups and the wave pairs in order
    auto extend = [&]() {
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            const int f = feat(w, q, i);
            acc[0] = fmaf(sw.w4[f], a3[i], acc[0]);
            const float d1 = s1[i] * x[i];
#pragma unroll
            for (int d = 0; d < DZ; ++d)
                acc[1 + d] = fmaf(sw.w1[d][f], d1, acc[1 + d]);
        }
    };
    if (!(w & 1)) {
        extend();
#pragma unroll
        for (int k = 0; k < NRED; ++k)
            red[w >> 1][l][k] = acc[k];
    }
    __syncthreads();
    if (w & 1) {
#pragma unroll
        for (int k = 0; k < NRED; ++k)
            acc[k] = red[w >> 1][l][k];
        extend();
#pragma unroll
        for (int k = 0; k < NRED; ++k)
            acc[k] = group_sum(acc[k]);
        if (l < 16)
#pragma unroll
            for (int k = 0; k < NRED; ++k)
                pairs[w >> 1][l][k] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x < 16 * NRED) {
        const int sample = threadIdx.x / NRED, k = threadIdx.x % NRED;
        float t = pairs[0][sample][k];
#pragma unroll
        for (int p = 1; p < NWAVE / 2; ++p)
            t += pairs[p][sample][k];
        total[sample][k] = t;
    }
    __syncthreads();
    const float *tot = total[l & 15];
    float rr[DZ];
#pragma unroll
    for (int d = 0; d < DZ; ++d)
        rr[d] = valid ? tot[1 + d] - gt[d] : 0.0f;
    const float e = valid ? tot[0] + bf16_to_f32(net.w[OB4]) - yb : 0.0f;
    // tangent pass along r
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const int f = feat(w, q, i);
        float t = 0.0f;
#pragma unroll
        for (int d = 0; d < DZ; ++d)
            t = fmaf(sw.w1[d][f], rr[d], t);
        t1[i] = t;
        v[i] = s1[i] * t;
    }
    put_vec(ws, V_U1, place, valid, v);
    mf_product(a, net.frag[F_W3], v, t2, op, 0);
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        v[i] = s2[i] * t2[i];
    put_vec(ws, V_U2, place, valid, v);
    mf_product(a, net.frag[F_W3T], v, t3, op, 1);
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        v[i] = s3[i] * t3[i];
    put_vec(ws, V_U3, place, valid, v);
    // reverse pass of J = cf f + ct D_r f (v: adjoint of the activation, u: of its tangent)
    const float cf = 2.0f * e / float(B);
    const float ct = 2.0f * lam / float(B);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const float w4 = sw.w4[feat(w, q, i)];
        v[i] = cf * w4;
        u[i] = ct * w4;
    }
    layer_adjoint(v, u, s3, c3, t3);
    put_vec(ws, V_H3B, place, valid, v);
    put_vec(ws, V_T3B, place, valid, u);
    mf_product(a, nullptr, v, x, op, 0);
    mf_product(a, net.frag[F_W2T], u, v, op, 1);
    layer_adjoint(x, v, s2, c2, t2);
    put_vec(ws, V_H2B, place, valid, x);
    put_vec(ws, V_T2B, place, valid, v);
    mf_product(a, nullptr, x, u, op, 0);
    mf_product(a, nullptr, v, x, op, 1);
    layer_adjoint(u, x, s1, c1, t1);
    put_vec(ws, V_H1B, place, valid, u);
    put_vec(ws, V_T1B, place, valid, x);
    if (w == 0 && q == 0) {
        float rn = 0.0f;
#pragma unroll
        for (int d = 0; d < DZ; ++d) {
            ws.zr[d * ws.bp + b] = zi[d];
            ws.zr[(DZ + d) * ws.bp + b] = rr[d];
            rn = fmaf(rr[d], rr[d], rn);
        }
        ws.cf[b] = cf;
        ws.loss[b] = valid ? e * e + lam * rn : 0.0f;
    }
}

// Parameter gradient, contracted over the padded batch, by workgroups of 4 waves:
//   workgroups 0..511: a 16 x 16 tile of dW2 (0..255) or dW3 (256..511) on the
//     matrix cores, sum_b h_b[j] a_b[k] + t_b[j] u_b[k], each FP32 factor split
//     into hi + lo BF16 parts and three products taken (hi hi, hi lo, lo hi;
//     lo lo is below 2^-16 of the product).  The (term, 32-sample chunk) items
//     are dealt to the 4 waves in turn, each wave's partial tile is added in
//     item order, and the 4 partials in wave order;
//   workgroups 512..: 4 rows each (one per wave) of W1 (6 values), b1, b2, b3,
//     w4, then b4 with the loss: lanes take samples lane + 64 i in order, then a
//     fixed butterfly over the wave.
constexpr int WG_TILES = 512;
constexpr int WG_ROWS = 5 * H + 1;
constexpr int WGRAD_WAVES = 4;

// lane group q's 8 values of a 32-sample chunk in the fragment k order
__device__ inline void load8(const float *p, int q, float4 &x0, float4 &x1)
{
    x0 = *reinterpret_cast<const float4 *>(p + 4 * q);
    x1 = *reinterpret_cast<const float4 *>(p + 16 + 4 * q);
}

__device__ inline void split_pair(const float4 &x0, const float4 &x1, bf16x8 &hi, bf16x8 &lo)
{
    const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    split8(x, hi, lo);
}

__global__ __launch_bounds__(64 * WGRAD_WAVES) void k_mlp_wgrad_mfma(TrainWs ws, int64_t B, float ct,
                                                                    float *__restrict__ grad,
                                                                    float *__restrict__ loss_out)
{
    __shared__ f32x4 part[WGRAD_WAVES][64];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4, lm = l & 15;
    const int64_t bp = ws.bp;
    const int wg = blockIdx.x;
    if (wg < WG_TILES) {
        const int mat = wg >> 8, jt = (wg >> 4) & 15, kt = wg & 15;
        const int vh = mat ? V_H3B : V_H2B, vt = mat ? V_T3B : V_T2B, va = mat ? V_A2 : V_A1, vu = mat ? V_U2 : V_U1;
        const int j = 16 * jt + lm, k = 16 * kt + lm;
        const int nchunk = int(bp >> 5), nitems = 2 * nchunk;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        // this wave's items i = w, w + 4, ...: four at a time, all their loads issued before the products
        for (int i0 = w; i0 < nitems; i0 += 4 * WGRAD_WAVES) {
            float4 xa[4][2], xb[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + WGRAD_WAVES * u;
                if (i < nitems) {
                    const int term = (i >= nchunk) ? 1 : 0;
                    const int64_t c0 = 32 * int64_t(i - term * nchunk);
                    load8(ws.vec + (int64_t(term ? vt : vh) * H + j) * bp + c0, q, xa[u][0], xa[u][1]);
                    load8(ws.vec + (int64_t(term ? vu : va) * H + k) * bp + c0, q, xb[u][0], xb[u][1]);
                } else {
                    xa[u][0] = xa[u][1] = xb[u][0] = xb[u][1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i0 + WGRAD_WAVES * u < nitems) {
                    bf16x8 ah, al, bh, bl;
                    split_pair(xa[u][0], xa[u][1], ah, al);
                    split_pair(xb[u][0], xb[u][1], bh, bl);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
                }
            }
        }
        part[w][l] = acc;
        __syncthreads();
        if (w == 0) {
            f32x4 t = part[0][l];
#pragma unroll
            for (int ww = 1; ww < WGRAD_WAVES; ++ww)
                t += part[ww][l];
            const int64_t base = mat ? OW3 : OW2;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                grad[base + int64_t(16 * jt + 4 * q + r) * H + k] = t[r];
        }
        return;
    }
    const int row = (wg - WG_TILES) * WGRAD_WAVES + w;
    if (row >= WG_ROWS)
        return;
    if (row < H) {  // W1[j][:]: sum_b h1b[j] z_b + t1b[j] r_b
        const float *hb = ws.vec + (int64_t(V_H1B) * H + row) * bp;
        const float *tb = ws.vec + (int64_t(V_T1B) * H + row) * bp;
        float acc[DZ] = {};
#pragma unroll 4
        for (int64_t b = l; b < bp; b += 64) {
            const float h = hb[b], t = tb[b];
#pragma unroll
            for (int d = 0; d < DZ; ++d) {
                acc[d] = fmaf(h, ws.zr[d * bp + b], acc[d]);
                acc[d] = fmaf(t, ws.zr[(DZ + d) * bp + b], acc[d]);
            }
        }
#pragma unroll
        for (int d = 0; d < DZ; ++d)
            acc[d] = wave_sum(acc[d]);
        if (l == 0)
#pragma unroll
            for (int d = 0; d < DZ; ++d)
                grad[OW1 + row * DZ + d] = acc[d];
    } else if (row < 4 * H) {  // b1, b2, b3: sum_b h_b[j]
        const int layer = row / H - 1, j = row % H;
        const int vi = layer == 0 ? V_H1B : layer == 1 ? V_H2B : V_H3B;
        const int64_t off = layer == 0 ? OB1 : layer == 1 ? OB2 : OB3;
        const float *hb = ws.vec + (int64_t(vi) * H + j) * bp;
        float acc = 0.0f;
#pragma unroll 4
        for (int64_t b = l; b < bp; b += 64)
            acc += hb[b];
        acc = wave_sum(acc);
        if (l == 0)
            grad[off + j] = acc;
    } else if (row < 5 * H) {  // w4[j]: sum_b cf_b a3_b[j] + ct u3_b[j]
        const int j = row - 4 * H;
        const float *a3 = ws.vec + (int64_t(V_A3) * H + j) * bp;
        const float *u3 = ws.vec + (int64_t(V_U3) * H + j) * bp;
        float acc = 0.0f;
#pragma unroll 4
        for (int64_t b = l; b < bp; b += 64) {
            acc = fmaf(ws.cf[b], a3[b], acc);
            acc = fmaf(ct, u3[b], acc);
        }
        acc = wave_sum(acc);
        if (l == 0)
            grad[OW4 + j] = acc;
    } else {  // b4 and the loss
        float acc = 0.0f, ls = 0.0f;
#pragma unroll 4
        for (int64_t b = l; b < bp; b += 64) {
            acc += ws.cf[b];
            ls += ws.loss[b];
        }
        acc = wave_sum(acc);
        ls = wave_sum(ls);
        if (l == 0) {
            grad[OB4] = acc;
            loss_out[0] = ls / float(B);
        }
    }
}

// The BF16 working copies of a parameter: flat, or for W2 and W3 packed rows and operand
// fragments of the matrix and its transpose.
struct Copies {
    uint16_t *wb, *pack[4], *frag[4];
};

Copies copies_of(void *state)
{
    const StateLayout L = state_layout();
    char *b = static_cast<char *>(state);
    Copies c;
    c.wb = reinterpret_cast<uint16_t *>(b + L.wb);
    for (int i = 0; i < 4; ++i) {
        c.pack[i] = reinterpret_cast<uint16_t *>(b + L.pack[i]);
        c.frag[i] = reinterpret_cast<uint16_t *>(b + L.frag[i]);
    }
    return c;
}

__device__ inline void write_copies(const Copies &c, int64_t p, uint16_t h)
{
    const bool w2 = p >= OW2 && p < OB2, w3 = p >= OW3 && p < OB3;
    if (!w2 && !w3) {
        c.wb[p] = h;
        return;
    }
    const int q = int(p - (w2 ? OW2 : OW3)), j = q / H, k = q % H, i = w2 ? F_W2 : F_W3;
    c.pack[i][pack_index(j, k)] = h;
    c.pack[i + 1][pack_index(k, j)] = h;
    c.frag[i][frag_index(j, k)] = h;
    c.frag[i + 1][frag_index(k, j)] = h;
}

// BF16 working copies from the FP32 master.
__global__ __launch_bounds__(256) void k_mlp_refresh(const float *__restrict__ master, Copies c)
{
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= P)
        return;
    write_copies(c, p, f32_to_bf16(master[p]));
}

__global__ __launch_bounds__(256) void k_mlp_load(const float *__restrict__ src, float *__restrict__ master,
                                                  float *__restrict__ m, float *__restrict__ v)
{
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= P)
        return;
    master[p] = src[p];
    m[p] = 0.0f;
    v[p] = 0.0f;
}

__global__ __launch_bounds__(256) void k_mlp_copy(const float *__restrict__ src, float *__restrict__ dst)
{
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p < P)
        dst[p] = src[p];
}

// Adam (Kingma and Ba, 2015) with bias correction on the FP32 master weights,
// followed by the BF16 working copies of the updated value.
__global__ __launch_bounds__(256) void k_mlp_adam(float *__restrict__ master, float *__restrict__ m,
                                                  float *__restrict__ v, const float *__restrict__ grad, float lr,
                                                  float beta1, float beta2, float eps, float c1, float c2, Copies c)
{
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= P)
        return;
    const float gr = grad[p];
    const float mm = beta1 * m[p] + (1.0f - beta1) * gr;
    const float vv = beta2 * v[p] + (1.0f - beta2) * gr * gr;
    m[p] = mm;
    v[p] = vv;
    const float th = master[p] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    master[p] = th;
    write_copies(c, p, f32_to_bf16(th));
}

struct TrainLayout {
    int64_t bp;
    size_t vec, zr, cf, loss, grad, total;
};

TrainLayout train_layout(int64_t B)
{
    TrainLayout t;
    t.bp = (B + 31) / 32 * 32;
    const size_t bp = size_t(t.bp);
    size_t off = 0;
    t.vec = off;
    off = align256(off + sizeof(float) * bp * NV * H);
    t.zr = off;
    off = align256(off + sizeof(float) * bp * 12);
    t.cf = off;
    off = align256(off + sizeof(float) * bp);
    t.loss = off;
    off = align256(off + sizeof(float) * bp);
    t.grad = off;
    off = align256(off + sizeof(float) * P);
    t.total = off;
    return t;
}

// Batches up to this size take the one-sample kernel (the arithmetic of k_mlp_leapfrog).
constexpr int64_t SMALL_BATCH = 8;
constexpr int64_t MAX_BATCH = int64_t(1) << 22;

bool aligned256(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }

}  // namespace
}  // namespace hawkes

using namespace hawkes;

extern "C" size_t hawkes_mlp_state_bytes(void) { return state_layout().total; }

extern "C" size_t hawkes_mlp_workspace_bytes(int64_t batch)
{
    if (batch < 1 || batch > MAX_BATCH)
        return 0;
    return train_layout(batch).total;
}

extern "C" int hawkes_mlp_load(void *d_state, const float *d_params, void *stream)
{
    if (!d_state || !d_params || !aligned256(d_state)) {
        set_error("mlp_load: null or misaligned pointer");
        return HAWKES_EINVAL;
    }
    const StateLayout L = state_layout();
    char *s = static_cast<char *>(d_state);
    const unsigned blocks = unsigned((P + 255) / 256);
    hipStream_t st = as_stream(stream);
    hipLaunchKernelGGL(k_mlp_load, dim3(blocks), dim3(256), 0, st, d_params, reinterpret_cast<float *>(s + L.master),
                       reinterpret_cast<float *>(s + L.m), reinterpret_cast<float *>(s + L.v));
    hipLaunchKernelGGL(k_mlp_refresh, dim3(blocks), dim3(256), 0, st, reinterpret_cast<const float *>(s + L.master),
                       copies_of(d_state));
    return check_launch("mlp_load");
}

extern "C" int hawkes_mlp_store(const void *d_state, float *d_params, void *stream)
{
    if (!d_state || !d_params || !aligned256(d_state)) {
        set_error("mlp_store: null or misaligned pointer");
        return HAWKES_EINVAL;
    }
    const StateLayout L = state_layout();
    hipLaunchKernelGGL(k_mlp_copy, dim3(unsigned((P + 255) / 256)), dim3(256), 0, as_stream(stream),
                       reinterpret_cast<const float *>(static_cast<const char *>(d_state) + L.master), d_params);
    return check_launch("mlp_store");
}

extern "C" int hawkes_mlp_forward(const void *d_state, const float *d_z, int64_t batch, float *d_f, float *d_gz,
                                  void *stream)
{
    if (!d_state || !d_z || !d_f || !aligned256(d_state) || batch < 1 || batch > MAX_BATCH) {
        set_error("mlp_forward: invalid arguments (batch %lld)", (long long)batch);
        return HAWKES_EINVAL;
    }
    if (batch <= SMALL_BATCH)
        hipLaunchKernelGGL(k_mlp_forward, dim3(unsigned(batch)), dim3(ONE_WG), 0, as_stream(stream), net_of(d_state), d_z,
                           batch, d_f, d_gz);
    else {
        const int64_t tiles = (batch + 15) / 16, rest = tiles % (2 * FWD_RESIDENT);
        const int64_t pairs = (tiles - rest) / 2 + (rest > FWD_RESIDENT ? (rest + 1) / 2 : 0);
        const int64_t ones = rest > FWD_RESIDENT ? 0 : rest;
        hipLaunchKernelGGL(k_mlp_forward_mfma, dim3(unsigned(pairs + ones)), dim3(64 * FWD_WAVES), 0,
                           as_stream(stream), mfnet_of(d_state), d_z, batch, int(pairs), d_f, d_gz);
    }
    return check_launch("mlp_forward");
}

extern "C" int hawkes_mlp_leapfrog(const void *d_state, hawkes_mlp_leapfrog_io *d_io, int64_t n_steps, void *stream)
{
    if (!d_state || !d_io || !aligned256(d_state) || n_steps < 1 || n_steps > 4096) {
        set_error("mlp_leapfrog: invalid arguments (n_steps %lld)", (long long)n_steps);
        return HAWKES_EINVAL;
    }
    hipLaunchKernelGGL(k_mlp_leapfrog, dim3(1), dim3(ONE_WG), 0, as_stream(stream), net_of(d_state), d_io,
                       int(n_steps));
    return check_launch("mlp_leapfrog");
}

extern "C" int hawkes_mlp_loss_grad(const void *d_state, const float *d_z, const float *d_y, const float *d_g,
                                    int64_t batch, float lambda_g, void *ws, size_t ws_bytes, float *d_loss,
                                    float *d_grad, void *stream)
{
    if (!d_state || !d_z || !d_y || !d_g || !d_loss || !aligned256(d_state) || batch < 1 || batch > MAX_BATCH ||
        !(lambda_g >= 0.0f)) {
        set_error("mlp_loss_grad: invalid arguments (batch %lld)", (long long)batch);
        return HAWKES_EINVAL;
    }
    const TrainLayout T = train_layout(batch);
    if (!ws || !aligned256(ws) || ws_bytes < T.total) {
        set_error("mlp_loss_grad: workspace of %zu bytes, need %zu (256-byte aligned)", ws_bytes, T.total);
        return HAWKES_EWORKSPACE;
    }
    char *w = static_cast<char *>(ws);
    TrainWs t{reinterpret_cast<float *>(w + T.vec), reinterpret_cast<float *>(w + T.zr),
              reinterpret_cast<float *>(w + T.cf), reinterpret_cast<float *>(w + T.loss), T.bp};
    float *grad = d_grad ? d_grad : reinterpret_cast<float *>(w + T.grad);
    hipStream_t st = as_stream(stream);
    hipLaunchKernelGGL(k_mlp_train_mfma, dim3(unsigned(T.bp / 16)), dim3(64 * NWAVE), 0, st, mfnet_of(d_state), d_z, d_y, d_g,
                       batch, lambda_g, t);
    hipLaunchKernelGGL(k_mlp_wgrad_mfma, dim3(unsigned(WG_TILES + (WG_ROWS + WGRAD_WAVES - 1) / WGRAD_WAVES)),
                       dim3(64 * WGRAD_WAVES), 0, st, t, batch,
                       2.0f * lambda_g / float(batch), grad, d_loss);
    return check_launch("mlp_loss_grad");
}

extern "C" int hawkes_mlp_adam_step(void *d_state, const float *d_grad, int64_t step, float lr, float beta1,
                                    float beta2, float eps, void *stream)
{
    if (!d_state || !d_grad || !aligned256(d_state) || step < 1 || !(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) ||
        !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f)) {
        set_error("mlp_adam_step: invalid arguments");
        return HAWKES_EINVAL;
    }
    const StateLayout L = state_layout();
    char *s = static_cast<char *>(d_state);
    const float c1 = float(1.0 - std::pow(double(beta1), double(step)));
    const float c2 = float(1.0 - std::pow(double(beta2), double(step)));
    const unsigned blocks = unsigned((P + 255) / 256);
    hipStream_t st = as_stream(stream);
    hipLaunchKernelGGL(k_mlp_adam, dim3(blocks), dim3(256), 0, st, reinterpret_cast<float *>(s + L.master),
                       reinterpret_cast<float *>(s + L.m), reinterpret_cast<float *>(s + L.v), d_grad, lr, beta1, beta2,
                       eps, c1, c2, copies_of(d_state));
    return check_launch("mlp_adam_step");
}
