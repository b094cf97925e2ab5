// md_mlp.hip -- training kernels of the aerodynamic-residual surrogate
// (64 -> 128 -> 128 -> 128 -> 6, SiLU, bfloat16 operands, fp32 accumulation).
//
// A training step is five launches:
//   mlp_forward_kernel  all four layers of 16 samples per workgroup and pass;
//   mlp_dgrad_kernel    loss, output gradient and the chain of data gradients,
//                       16 samples per workgroup and pass;
//   mlp_wgrad_kernel    weight gradients, 32x32 tiles per wave, split over the batch;
//   mlp_reduce_kernel   the split's partial sums, added in a fixed order, so
//                       that gradients are deterministic;
//   adam_kernel         fp32 parameters, and their bfloat16 operands.
// Every product runs on v_mfma_f32_16x16x32_bf16.  The weight operands are
// kept as bfloat16 fragments beside the fp32 parameters (rounded once per
// update instead of on every read), in the order in which a wave loads them:
// one 16-byte read per lane and fragment, 1 KB in line order per wave.
// Master weights, gradients, Adam moments and pre-activations are fp32.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "md.h"
#include "md_mlp.h"

namespace md {
namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

__device__ __forceinline__ float dsilu_f(float z) {
    const float s = __builtin_amdgcn_rcpf(1.f + __expf(-z));
    return s * (1.f + z * (1.f - s));
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Offsets of the flat parameter vector (W row-major [out][in], then b).
constexpr int PW1 = 0, PB1 = 8192, PW2 = 8320, PB2 = 24704, PW3 = 24832, PB3 = 41216, PW4 = 41344, PB4 = 42112;
// Weight operands (bfloat16): Wf, element (k = in, n = out) for the forward
// pass, the 6 output rows padded to 16 with zeros; Wt, element (k = out,
// n = in) for the data gradients of layers 2-4, the 6 padded to 32.
constexpr int WF1 = 0, WF2 = WF1 + MLP_H * MLP_IN, WF3 = WF2 + MLP_H * MLP_H, WF4 = WF3 + MLP_H * MLP_H,
              WF_TOTAL = WF4 + 16 * MLP_H;
constexpr int WT2 = 0, WT3 = WT2 + MLP_H * MLP_H, WT4 = WT3 + MLP_H * MLP_H, WT_TOTAL = WT4 + 32 * MLP_H;
// Place of element (n, k) among fragments of 16 columns n x 32 values of k,
// kcs of them along k: lane n % 16 + 16 ((k % 32) / 8) holds 8 consecutive k.
__host__ __device__ constexpr int frag_at(int n, int k, int kcs) {
    return ((n / 16 * kcs + k / 32) * 64 + n % 16 + 16 * (k % 32 / 8)) * 8 + k % 8;
}

// Rows of the kept activations [row][ldb] (inputs, then three hidden layers)
// and of the gradients dZ [row][ldb] (three hidden layers, then the outputs);
// ldb = the batch in whole 32-sample chunks, the samples past the batch 0.
constexpr int ACT_ROWS = MLP_IN + 3 * MLP_H, DZ_ROWS = 3 * MLP_H + MLP_OUT;
constexpr int NBIAS = 3 * MLP_H + MLP_OUT;
inline long long padded(int B) { return ((long long)B + 31) / 32 * 32; }

// Workgroups of the two chain kernels (each takes every grid-th tile of 16
// samples): two per CU, so that one's barriers overlap the other's products.
constexpr int FWD_MAX_WG = 512, DGRAD_MAX_WG = 512;
// 32-sample chunks per slice of the weight gradients' split over the batch:
// 256 samples (eight products in a row per accumulator, 44 waves a slice),
// longer from 32768 samples on, where 128 slices fill the chip.
constexpr int MAX_SLICES = 128;
inline int slice_chunks(int chunks) { return std::max(8, (chunks + MAX_SLICES - 1) / MAX_SLICES); }
inline int max_slices(int max_batch) {
    return (int)std::min<long long>(MAX_SLICES, (padded(max_batch) / 32 + 7) / 8);
}

constexpr int LDX = MLP_IN + 8, LDH = MLP_H + 8;  // LDS row strides (bf16), 16-byte multiples

struct FwdArgs {
    const float *X;
    bool x16;  // X is 16-byte aligned
    int B, tiles;
    long long ldb;
    const float *norm;
    const bf16 *W;
    const float *P;
    bf16 *act;
    float *Z, *Y, *out;
};

// The whole forward pass: four waves share 16 samples; each wave computes 32
// units of every hidden layer with its weight fragments in registers (read
// once per workgroup), the activations pass from layer to layer through LDS,
// the output layer rotates over the waves.  KEEP: the inputs, activations,
// pre-activations and standardised outputs are stored for the backward pass.
//
// One launch in place of six, and no pass over memory between layers: at the
// batches of training (4096 samples, 256 workgroups) the time is the chain
// weights -> four layers -> store, so the 16-sample tile, the smallest that
// fills an MFMA, spreads it over the most CUs.
// The products run in the order k = 0, 32, ... from 0 with the bias added
// last, samples as rows: the same roundings at every batch size.
template <bool KEEP>
__global__ void __launch_bounds__(256, 2) mlp_forward_kernel(FwdArgs a) {
    __shared__ __attribute__((aligned(16))) bf16 xs[16 * LDX];
    __shared__ __attribute__((aligned(16))) bf16 hs[3][16 * LDH];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    bf16x8 W1[2][2], W2[2][4], W3[2][4], W4[4];
    float bias[3][2];
    auto frag = [&](int off, int tile, int kcs, int kc) {
        return *(const bf16x8 *)(a.W + off + ((tile * kcs + kc) * 64 + lane) * 8);
    };
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int ot = 2 * w + j;
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) W1[j][kc] = frag(WF1, ot, 2, kc);
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            W2[j][kc] = frag(WF2, ot, 4, kc);
            W3[j][kc] = frag(WF3, ot, 4, kc);
        }
        bias[0][j] = a.P[PB1 + 16 * ot + r];
        bias[1][j] = a.P[PB2 + 16 * ot + r];
        bias[2][j] = a.P[PB3 + 16 * ot + r];
    }
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) W4[kc] = frag(WF4, 0, 4, kc);
    const int o = r < MLP_OUT ? r : 0;
    const float b4 = a.P[PB4 + o], ym = a.norm[2 * MLP_IN + o], ys = a.norm[2 * MLP_IN + MLP_OUT + o];
    // this thread's four inputs of the tile: a wave reads 64 bytes of each
    // sample and stores 32 of each kept row
    const int xr = tid & 15, xc = (tid >> 4) * 4;
    float mean[4], inv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        mean[k] = a.norm[xc + k];
        inv[k] = a.norm[MLP_IN + xc + k];
    }
    auto load_x = [&](int tile, float (&x)[4]) {
        const long long b = 16ll * tile + xr;
        if (b < a.B) {
            const float *p = a.X + b * MLP_IN + xc;
            if (a.x16) {
                const f32x4 v = *(const f32x4 *)p;
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = v[k];
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = p[k];
            }
        } else {
            // past the batch: the standardised input 0
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = mean[k];
        }
    };
    float x[4];
    load_x(blockIdx.x, x);
    int it = 0;
    for (int tile = blockIdx.x; tile < a.tiles; tile += gridDim.x, ++it) {
        const int b0 = 16 * tile;
        bf16x4 xb;
#pragma unroll
        for (int k = 0; k < 4; ++k) xb[k] = (bf16)((x[k] - mean[k]) * inv[k]);
        *(bf16x4 *)(xs + xr * LDX + xc) = xb;
        if (KEEP) {
#pragma unroll
            for (int k = 0; k < 4; ++k) a.act[(xc + k) * a.ldb + b0 + xr] = xb[k];
        }
        if (tile + (int)gridDim.x < a.tiles) load_x(tile + gridDim.x, x);
        __syncthreads();
        auto hidden = [&](int l, const bf16 *hin, int ldh, int kcs, const bf16x8 *const (&Wl)[2]) {
            bf16x8 av[4];
#pragma unroll
            for (int kc = 0; kc < kcs; ++kc) av[kc] = *(const bf16x8 *)(hin + r * ldh + 32 * kc + 8 * g);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int unit = 32 * w + 16 * j + r;
                f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < kcs; ++kc) acc = mfma(av[kc], Wl[j][kc], acc);
                f32x4 z;
                bf16x4 h;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    z[t] = acc[t] + bias[l][j];
                    h[t] = (bf16)silu_f(z[t]);
                    if (KEEP && b0 + 4 * g + t >= a.B) h[t] = (bf16)0.f;
                    hs[l][(4 * g + t) * LDH + unit] = h[t];
                }
                if (KEEP) {
                    *(bf16x4 *)(a.act + (MLP_IN + MLP_H * l + unit) * a.ldb + b0 + 4 * g) = h;
                    *(f32x4 *)(a.Z + (((tile * 3ll + l) * 8 + 2 * w + j) * 64 + lane) * 4) = z;
                }
            }
            __syncthreads();
        };
        hidden(0, xs, LDX, 2, {W1[0], W1[1]});
        hidden(1, hs[0], LDH, 4, {W2[0], W2[1]});
        hidden(2, hs[1], LDH, 4, {W3[0], W3[1]});
        if (w == (it & 3)) {
            f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) acc = mfma(*(const bf16x8 *)(hs[2] + r * LDH + 32 * kc + 8 * g), W4[kc], acc);
            if (r < MLP_OUT) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const long long b = b0 + 4 * g + t;
                    if (b >= a.B) continue;
                    const float y = acc[t] + b4;
                    if (KEEP) a.Y[b * MLP_OUT + r] = y;
                    if (a.out) a.out[b * MLP_OUT + r] = y * ys + ym;
                }
            }
        }
    }
}

struct DgradArgs {
    const float *Y, *T;
    int B, tiles;
    long long ldb;
    const float *norm;
    const bf16 *W;
    const float *Z;
    bf16 *dZ;
    float *part_b;
    double *loss_part;
};

// Gradient of the mean squared error over B x OUT standardised targets, and
// the data gradients dZ_l = (dZ_(l+1) W_(l+1)) * SiLU'(Z_l) down to the first
// hidden layer, 16 samples per pass on the forward pass's scheme (32 units per
// wave, weight fragments and pre-activations in registers before the chain
// starts, operands through LDS).  The fp32 gradients are rounded to bfloat16
// once, as operands of the next product and (stored [unit][sample]) of the
// weight gradients; the bias gradients sum the fp32 values, here per
// workgroup, fixed order.  One launch in place of four and no fp32 gradient
// in memory.  4096 samples: 7.4 us, against 4.6 + 3 x 16 us for the loss and
// the tiled products as launches of their own; bound, as the forward pass, by
// the chain of one tile.
__global__ void __launch_bounds__(256, 2) mlp_dgrad_kernel(DgradArgs a) {
    constexpr int LDY = 40;
    __shared__ __attribute__((aligned(16))) bf16 dy[16 * LDY];
    __shared__ __attribute__((aligned(16))) bf16 ds[2][16 * LDH];
    __shared__ float red4[96];
    __shared__ double red[96];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    // the outputs padded to k = 32: the padding alone, since the outputs'
    // elements are written by other threads before the first barrier
    for (int i = tid; i < 16 * LDY; i += 256)
        if (i % LDY >= MLP_OUT) dy[i] = (bf16)0.f;
    bf16x8 W4[2], W3[2][4], W2[2][4];
    auto frag = [&](int off, int tile, int kcs, int kc) {
        return *(const bf16x8 *)(a.W + off + ((tile * kcs + kc) * 64 + lane) * 8);
    };
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        W4[j] = frag(WT4, 2 * w + j, 1, 0);
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            W3[j][kc] = frag(WT3, 2 * w + j, 4, kc);
            W2[j][kc] = frag(WT2, 2 * w + j, 4, kc);
        }
    }
    // this thread's output value: sample yr of the tile, output yo
    const int yr = tid / MLP_OUT, yo = tid % MLP_OUT;
    const bool out_thread = tid < 16 * MLP_OUT;
    const float ym = a.norm[2 * MLP_IN + yo], ys = a.norm[2 * MLP_IN + MLP_OUT + yo];
    const float scale = 2.f / (float)(a.B * MLP_OUT);
    // (squared errors in double: a workgroup's chain grows with the batch)
    double e2 = 0.0;
    float sum4 = 0.f, sums[3][2] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
    for (int tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
        const int b0 = 16 * tile;
        f32x4 z[3][2];
#pragma unroll
        for (int l = 0; l < 3; ++l)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                z[l][j] = *(const f32x4 *)(a.Z + (((tile * 3ll + l) * 8 + 2 * w + j) * 64 + lane) * 4);
        if (out_thread) {
            const long long b = b0 + yr;
            float gy = 0.f;
            if (b < a.B) {
                const float ts = (a.T[b * MLP_OUT + yo] - ym) / ys;
                const float d = a.Y[b * MLP_OUT + yo] - ts;
                gy = d * scale;
                e2 += (double)(d * d);
            }
            sum4 += gy;
            dy[yr * LDY + yo] = (bf16)gy;
            a.dZ[(3 * MLP_H + yo) * a.ldb + b] = (bf16)gy;
        }
        __syncthreads();
        auto chain = [&](int l, const bf16 *in, int ld, int kcs, const bf16x8 *const (&Wl)[2], bf16 *next) {
            bf16x8 av[4];
#pragma unroll
            for (int kc = 0; kc < kcs; ++kc) av[kc] = *(const bf16x8 *)(in + r * ld + 32 * kc + 8 * g);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int unit = 32 * w + 16 * j + r;
                f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < kcs; ++kc) acc = mfma(av[kc], Wl[j][kc], acc);
                bf16x4 h;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float d = b0 + 4 * g + t < a.B ? acc[t] * dsilu_f(z[l][j][t]) : 0.f;
                    sums[l][j] += d;
                    h[t] = (bf16)d;
                    if (next) next[(4 * g + t) * LDH + unit] = h[t];
                }
                *(bf16x4 *)(a.dZ + (MLP_H * l + unit) * a.ldb + b0 + 4 * g) = h;
            }
            if (next) __syncthreads();
        };
        const bf16x8 *const w4[2] = {&W4[0], &W4[1]};
        chain(2, dy, LDY, 1, w4, ds[0]);
        chain(1, ds[0], LDH, 4, {W3[0], W3[1]}, ds[1]);
        chain(0, ds[1], LDH, 4, {W2[0], W2[1]}, nullptr);
    }
    float *pb = a.part_b + (long long)blockIdx.x * NBIAS;
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float s = sums[l][j];
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (g == 0) pb[MLP_H * l + 32 * w + 16 * j + r] = s;
        }
    if (out_thread) {
        red4[tid] = sum4;
        red[tid] = e2;
    }
    __syncthreads();
    if (tid < MLP_OUT) {
        float s = 0.f;
        for (int k = 0; k < 16; ++k) s += red4[k * MLP_OUT + tid];
        pb[3 * MLP_H + tid] = s;
    } else if (tid == 64) {
        double s = 0.0;
        for (int k = 0; k < 96; ++k) s += red[k];
        a.loss_part[blockIdx.x] = s;
    }
}

struct WgradArgs {
    const bf16 *act, *dZ;
    long long ldb;
    int chunks, slice;  // 32-sample chunks in all and per slice (blockIdx.y)
    float *part;
};

// One wave's tile of a weight gradient dW[out][in] = sum_b dZ[out][b] H[in][b]
// over a slice of the batch.  Both operands lie along the batch in memory, so
// a lane's 8 values are one 16-byte read and no LDS or conversion is needed;
// a 32x32 tile reads each operand twice per product pair.  4096 samples, all
// four layers in one launch: 6.8 us and 3.6 us for the partial sums, against
// 4 x (25 + 6 + 7) us when each layer's product, partial sums and bias sums
// were launches of their own with operands converted through LDS.
template <int MT>
__device__ __forceinline__ void wgrad_tile(const bf16 *dz, int rows, const bf16 *h, long long ldb, int c0, int c1,
                                           int lane, float *out, int ldo) {
    const int r = lane & 15, g = lane >> 4;
    f32x4 acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // rows past the gradient's last (the 6 outputs in a 16-row tile) are 0
    const bool on = r < rows;
    const bf16 *pa = dz + (on ? r : 0) * ldb + 8 * g, *pb = h + r * ldb + 8 * g;
    auto load = [&](int c, bf16x8 (&x)[MT], bf16x8 (&y)[2]) {
#pragma unroll
        for (int i = 0; i < MT; ++i) x[i] = *(const bf16x8 *)(pa + 16 * i * ldb + 32ll * c);
#pragma unroll
        for (int j = 0; j < 2; ++j) y[j] = *(const bf16x8 *)(pb + 16 * j * ldb + 32ll * c);
    };
    auto products = [&](bf16x8 (&x)[MT], bf16x8 (&y)[2]) {
        if (MT == 1) {
#pragma unroll
            for (int k = 0; k < 8; ++k) x[0][k] = on ? x[0][k] : (bf16)0.f;
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma(x[i], y[j], acc[i][j]);
    };
    int c = c0;
    for (; c + 4 <= c1; c += 4) {
        bf16x8 x[4][MT], y[4][2];
#pragma unroll
        for (int k = 0; k < 4; ++k) load(c + k, x[k], y[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) products(x[k], y[k]);
    }
    for (; c < c1; ++c) {
        bf16x8 x[MT], y[2];
        load(c, x, y);
        products(x, y);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (16 * i + 4 * g + t < rows) out[(16 * i + 4 * g + t) * ldo + 16 * j + r] = acc[i][j][t];
}

// Jobs of a slice, one per wave: 32x32 tiles of W1 (4 x 2), W2 and W3 (4 x 4
// each), and W4's 6 rows x 32 columns (4).
constexpr int WGRAD_JOBS = 8 + 16 + 16 + 4;

__global__ void __launch_bounds__(256) mlp_wgrad_kernel(WgradArgs a) {
    const int job = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c0 = blockIdx.y * a.slice, c1 = min(a.chunks, c0 + a.slice);
    float *part = a.part + (long long)blockIdx.y * MLP_NPARAMS;
    const bf16 *H[4] = {a.act, a.act + MLP_IN * a.ldb, a.act + (MLP_IN + MLP_H) * a.ldb,
                        a.act + (MLP_IN + 2 * MLP_H) * a.ldb};
    if (job < 8) {
        const int m = 32 * (job >> 1), n = 32 * (job & 1);
        wgrad_tile<2>(a.dZ + m * a.ldb, 32, H[0] + n * a.ldb, a.ldb, c0, c1, lane, part + PW1 + m * MLP_IN + n, MLP_IN);
    } else if (job < 40) {
        const int l = (job - 8) >> 4, m = 32 * (((job - 8) >> 2) & 3), n = 32 * (job & 3);
        wgrad_tile<2>(a.dZ + (MLP_H * (1 + l) + m) * a.ldb, 32, (l ? H[2] : H[1]) + n * a.ldb, a.ldb, c0, c1, lane,
                      part + (l ? PW3 : PW2) + m * MLP_H + n, MLP_H);
    } else {
        const int n = 32 * (job - 40);
        wgrad_tile<1>(a.dZ + 3 * MLP_H * a.ldb, MLP_OUT, H[3] + n * a.ldb, a.ldb, c0, c1, lane, part + PW4 + n, MLP_H);
    }
}

// Gradients from the partial sums: weights over the ns slices in ascending
// order (one thread each), biases over the nwg workgroups of the data
// gradients (one wave each: lane-strided sums, then a fixed tree).
constexpr int REDUCE_W_WG = (MLP_NPARAMS + 255) / 256;

__global__ void __launch_bounds__(256) mlp_reduce_kernel(const float *part, int ns, const float *part_b, int nwg,
                                                         float *grads) {
    if (blockIdx.x < REDUCE_W_WG) {
        const int i = blockIdx.x * 256 + threadIdx.x;
        const bool is_bias = (i >= PB1 && i < PW2) || (i >= PB2 && i < PW3) || (i >= PB3 && i < PW4) || i >= PB4;
        if (is_bias) return;
        float s = 0.f;
#pragma unroll 8
        for (int z = 0; z < ns; ++z) s += part[(long long)z * MLP_NPARAMS + i];
        grads[i] = s;
        return;
    }
    const int u = (blockIdx.x - REDUCE_W_WG) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (u >= NBIAS) return;
    float s = 0.f;
    for (int k = lane; k < nwg; k += 64) s += part_b[(long long)k * NBIAS + u];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) grads[u < MLP_H ? PB1 + u : u < 2 * MLP_H ? PB2 + u - MLP_H : u < 3 * MLP_H ? PB3 + u - 2 * MLP_H : PB4 + u - 3 * MLP_H] = s;
}

// The parameter's bfloat16 copies in the fragment orders of the forward pass
// (Wf) and of the data gradients (Wt); biases have none.
__device__ __forceinline__ void store_operands(int i, float p, bf16 *Wf, bf16 *Wt) {
    int l = 0, off = 0;
    if (i >= PW4) {
        l = 3;
        off = PW4;
    } else if (i >= PW3) {
        l = 2;
        off = PW3;
    } else if (i >= PW2) {
        l = 1;
        off = PW2;
    }
    const int din = l == 0 ? MLP_IN : MLP_H, dout = l == 3 ? MLP_OUT : MLP_H;
    const int e = i - off;
    if (e >= din * dout) return;  // a bias
    const int o = e / din, k = e - o * din;
    const bf16 v = (bf16)p;
    const int wf = l == 0 ? WF1 : l == 1 ? WF2 : l == 2 ? WF3 : WF4;
    Wf[wf + frag_at(o, k, din / 32)] = v;
    if (l > 0) {
        const int wt = l == 1 ? WT2 : l == 2 ? WT3 : WT4;
        Wt[wt + frag_at(k, o, l == 3 ? 1 : MLP_H / 32)] = v;
    }
}

// Outputs from a buffer of the network's to the caller's, de-standardised with
// norm (not null) as the forward kernel does it: for outputs that overlap the
// inputs, which other workgroups may still be reading.
__global__ void outputs_kernel(const float *src, const float *norm, float *out, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int o = (int)(i % MLP_OUT);
    out[i] = norm ? src[i] * norm[2 * MLP_IN + MLP_OUT + o] + norm[2 * MLP_IN + o] : src[i];
}

__global__ void pack_kernel(const float *p, bf16 *Wf, bf16 *Wt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < MLP_NPARAMS) store_operands(i, p[i], Wf, Wt);
}

// Adam (Kingma and Ba) on the flat fp32 parameters; bc1 = 1 - beta1^t, bc2 = 1 - beta2^t
__global__ void adam_kernel(float *p, const float *g, float *m1, float *m2, bf16 *Wf, bf16 *Wt, int n, float lr,
                            float b1, float b2, float eps, float bc1, float bc2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float m = b1 * m1[i] + (1.f - b1) * gi;
    const float v = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = m;
    m2[i] = v;
    const float q = p[i] - lr * (m / bc1) / (sqrtf(v / bc2) + eps);
    p[i] = q;
    store_operands(i, q, Wf, Wt);
}

}  // namespace

// Offsets of the flat parameter vector: W1, b1, W2, b2, W3, b3, W4, b4 (W row-major [out][in]).
const int kParamOff[8] = {0, 8192, 8320, 24704, 24832, 41216, 41344, 42112};

}  // namespace md

using md::bf16;
using md::kParamOff;

struct md_mlp {
    int max_batch = 0;
    int device = 0;
    float *params = nullptr, *grads = nullptr, *m1 = nullptr, *m2 = nullptr;
    int64_t t = 0;
    float *norm = nullptr;  // x_mean[64], x_inv_std[64], y_mean[6], y_std[6]
    bf16 *Wf = nullptr, *Wt = nullptr;  // weight operands, rewritten with every change of params
    // kept by the forward pass: inputs and activations [units][batch], the
    // pre-activations in fragment order, the standardised outputs
    bf16 *act = nullptr;
    float *Z = nullptr, *Y = nullptr;
    float *spare = nullptr;  // outputs of md_mlp_forward_noalloc that overlap its inputs
    bf16 *dZ = nullptr;  // operands of the weight gradients, [units][batch]
    float *part = nullptr, *part_b = nullptr;
    double *loss_part = nullptr;
    int last_B = 0, loss_parts = 0, fwd_B = 0;
    bool have_fwd = false, have_bwd = false;
    std::vector<void *> allocs;
    std::string err;
};

namespace {

// The network's device current for a scope, the caller's afterwards.
struct OnDevice {
    int caller = -1;
    explicit OnDevice(int device) {
        (void)hipGetDevice(&caller);
        if (caller != device) (void)hipSetDevice(device);
        else caller = -1;
    }
    ~OnDevice() {
        if (caller >= 0) (void)hipSetDevice(caller);
    }
};

md_status mlp_fail(md_mlp *m, md_status st, const std::string &msg) {
    m->err = msg;
    return st;
}

template <typename T>
hipError_t mlp_alloc(md_mlp *m, T **p, size_t n) {
    hipError_t e = hipMalloc((void **)p, sizeof(T) * (n > 0 ? n : 1));
    if (e == hipSuccess) {
        m->allocs.push_back(*p);
        e = hipMemset(*p, 0, sizeof(T) * (n > 0 ? n : 1));
    }
    return e;
}

}  // namespace

extern "C" {

md_status md_mlp_create(int max_batch, md_mlp **out) {
    if (!out || max_batch < 1 || max_batch > (1 << 24)) return MD_E_INVALID_ARG;
    *out = nullptr;
    md_mlp *m = new (std::nothrow) md_mlp();
    if (!m) return MD_E_OOM;
    m->max_batch = max_batch;
    (void)hipGetDevice(&m->device);
    // rows of the kept buffers: whole 32-sample chunks (md::padded)
    const size_t Bm = (size_t)md::padded(max_batch);
    hipError_t e = hipSuccess;
    auto A = [&](auto **p, size_t n) {
        if (e == hipSuccess) e = mlp_alloc(m, p, n);
    };
    A(&m->params, md::MLP_NPARAMS);
    A(&m->grads, md::MLP_NPARAMS);
    A(&m->m1, md::MLP_NPARAMS);
    A(&m->m2, md::MLP_NPARAMS);
    A(&m->norm, md::MLP_NORM);
    A(&m->Wf, md::WF_TOTAL);
    A(&m->Wt, md::WT_TOTAL);
    A(&m->act, Bm * md::ACT_ROWS);
    A(&m->Z, Bm * 3 * md::MLP_H);
    A(&m->Y, Bm * md::MLP_OUT);
    A(&m->spare, (size_t)MD_MLP_NOALLOC_MAX_BATCH * md::MLP_OUT);
    A(&m->dZ, Bm * md::DZ_ROWS);
    A(&m->part, (size_t)md::max_slices(max_batch) * md::MLP_NPARAMS);
    A(&m->part_b, (size_t)md::DGRAD_MAX_WG * md::NBIAS);
    A(&m->loss_part, md::DGRAD_MAX_WG);
    if (e != hipSuccess) {
        md_mlp_destroy(m);
        return MD_E_OOM;
    }
    // identity normalisation until set
    std::vector<float> nrm(md::MLP_NORM, 0.f);
    for (int i = 0; i < md::MLP_IN; ++i) nrm[md::MLP_IN + i] = 1.f;
    for (int i = 0; i < md::MLP_OUT; ++i) nrm[2 * md::MLP_IN + md::MLP_OUT + i] = 1.f;
    if (hipMemcpy(m->norm, nrm.data(), sizeof(float) * nrm.size(), hipMemcpyHostToDevice) != hipSuccess) {
        md_mlp_destroy(m);
        return MD_E_HIP;
    }
    *out = m;
    return MD_OK;
}

void md_mlp_destroy(md_mlp *m) {
    if (!m) return;
    (void)hipDeviceSynchronize();
    for (void *p : m->allocs) (void)hipFree(p);
    delete m;
}

const char *md_mlp_last_error(const md_mlp *m) { return m ? m->err.c_str() : "null md_mlp"; }

md_status md_mlp_set_params(md_mlp *m, const float *h_params) {
    if (!m || !h_params) return MD_E_INVALID_ARG;
    // copies find their device by the address, the packing kernel does not
    const OnDevice on(m->device);
    hipError_t e = hipMemcpy(m->params, h_params, sizeof(float) * md::MLP_NPARAMS, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(m->m1, 0, sizeof(float) * md::MLP_NPARAMS);
    if (e == hipSuccess) e = hipMemset(m->m2, 0, sizeof(float) * md::MLP_NPARAMS);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(md::pack_kernel, dim3((md::MLP_NPARAMS + 255) / 256), dim3(256), 0, nullptr, m->params,
                           m->Wf, m->Wt);
        e = hipGetLastError();
    }
    // the operands are in place for calls on any stream that follow
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return mlp_fail(m, MD_E_HIP, md::hip_msg("md_mlp_set_params", e));
    m->t = 0;
    return MD_OK;
}

md_status md_mlp_get_params(const md_mlp *m, float *h_params) {
    if (!m || !h_params) return MD_E_INVALID_ARG;
    (void)hipDeviceSynchronize();
    return hipMemcpy(h_params, m->params, sizeof(float) * md::MLP_NPARAMS, hipMemcpyDeviceToHost) == hipSuccess
               ? MD_OK
               : MD_E_HIP;
}

md_status md_mlp_set_norm(md_mlp *m, const float *h_norm) {
    if (!m || !h_norm) return MD_E_INVALID_ARG;
    for (int i = 0; i < md::MLP_IN; ++i)
        if (!(h_norm[md::MLP_IN + i] > 0.f)) return mlp_fail(m, MD_E_INVALID_ARG, "input scales must be > 0");
    for (int i = 0; i < md::MLP_OUT; ++i)
        if (!(h_norm[2 * md::MLP_IN + md::MLP_OUT + i] > 0.f))
            return mlp_fail(m, MD_E_INVALID_ARG, "output scales must be > 0");
    return hipMemcpy(m->norm, h_norm, sizeof(float) * md::MLP_NORM, hipMemcpyHostToDevice) == hipSuccess
               ? MD_OK
               : MD_E_HIP;
}

md_status md_mlp_get_norm(const md_mlp *m, float *h_norm) {
    if (!m || !h_norm) return MD_E_INVALID_ARG;
    return hipMemcpy(h_norm, m->norm, sizeof(float) * md::MLP_NORM, hipMemcpyDeviceToHost) == hipSuccess
               ? MD_OK
               : MD_E_HIP;
}

}  // extern "C"

namespace {

// The forward pass; keep: store what md_mlp_backward reads.  d_Y (nullable)
// receives the de-standardised outputs.
hipError_t mlp_forward_on(const md_mlp *m, const float *d_X, int B, bool keep, float *d_Y, hipStream_t st) {
    using namespace md;
    FwdArgs a;
    a.X = d_X;
    a.x16 = ((uintptr_t)d_X & 15) == 0;
    a.B = B;
    a.ldb = padded(B);
    a.tiles = keep ? (int)(a.ldb / 16) : (B + 15) / 16;
    a.norm = m->norm;
    a.W = m->Wf;
    a.P = m->params;
    a.act = m->act;
    a.Z = m->Z;
    a.Y = m->Y;
    const long long n = (long long)B * MLP_OUT;
    const uintptr_t x = (uintptr_t)d_X, y = (uintptr_t)d_Y;
    const bool overlap = d_Y && y < x + sizeof(float) * B * MLP_IN && x < y + sizeof(float) * n;
    a.out = !overlap ? d_Y : keep ? nullptr : m->spare;
    const int grid = std::min(a.tiles, FWD_MAX_WG);
    if (keep)
        hipLaunchKernelGGL(mlp_forward_kernel<true>, dim3(grid), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(mlp_forward_kernel<false>, dim3(grid), dim3(256), 0, st, a);
    if (overlap)
        hipLaunchKernelGGL(outputs_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, keep ? m->Y : m->spare,
                           keep ? m->norm : nullptr, d_Y, n);
    return hipGetLastError();
}

}  // namespace

extern "C" {

md_status md_mlp_forward(md_mlp *m, const float *d_X, int B, float *d_Y, void *stream) {
    using namespace md;
    if (!m || !d_X || B < 0) return MD_E_INVALID_ARG;
    if (B > m->max_batch) return mlp_fail(m, MD_E_INVALID_ARG, "batch exceeds max_batch");
    if (B == 0) return MD_OK;
    const hipError_t e = mlp_forward_on(m, d_X, B, true, d_Y, (hipStream_t)stream);
    if (e != hipSuccess) return mlp_fail(m, MD_E_HIP, hip_msg("md_mlp_forward", e));
    m->fwd_B = B;
    m->have_fwd = true;
    return MD_OK;
}

md_status md_mlp_forward_noalloc(md_mlp *m, const float *d_X, int B, float *d_Y, void *stream) {
    using namespace md;
    if (!m || !d_X || !d_Y || B < 0) {
        if (m) m->err = "md_mlp_forward_noalloc: null input or output, or B < 0";
        return MD_E_INVALID_ARG;
    }
    if (B > MD_MLP_NOALLOC_MAX_BATCH)
        return mlp_fail(m, MD_E_INVALID_ARG,
                        "md_mlp_forward_noalloc: batch " + std::to_string(B) + " exceeds its limit of " +
                            std::to_string(MD_MLP_NOALLOC_MAX_BATCH) + " samples");
    if (B == 0) return MD_OK;
    const hipError_t e = mlp_forward_on(m, d_X, B, false, d_Y, (hipStream_t)stream);
    if (e != hipSuccess) return mlp_fail(m, MD_E_HIP, hip_msg("md_mlp_forward_noalloc", e));
    return MD_OK;
}

md_status md_mlp_backward(md_mlp *m, const float *d_T, int B, void *stream) {
    using namespace md;
    if (!m || !d_T) return MD_E_INVALID_ARG;
    if (!m->have_fwd || m->fwd_B != B || B < 1) return mlp_fail(m, MD_E_INVALID_ARG, "backward needs the forward of the same batch");
    hipStream_t st = (hipStream_t)stream;
    DgradArgs d;
    d.Y = m->Y;
    d.T = d_T;
    d.B = B;
    d.ldb = padded(B);
    d.tiles = (int)(d.ldb / 16);
    d.norm = m->norm;
    d.W = m->Wt;
    d.Z = m->Z;
    d.dZ = m->dZ;
    d.part_b = m->part_b;
    d.loss_part = m->loss_part;
    const int nwg = std::min(d.tiles, DGRAD_MAX_WG);
    hipLaunchKernelGGL(mlp_dgrad_kernel, dim3(nwg), dim3(256), 0, st, d);
    hipError_t e = hipGetLastError();
    WgradArgs g;
    g.act = m->act;
    g.dZ = m->dZ;
    g.ldb = d.ldb;
    g.chunks = (int)(d.ldb / 32);
    g.slice = slice_chunks(g.chunks);
    g.part = m->part;
    const int ns = (g.chunks + g.slice - 1) / g.slice;
    if (e == hipSuccess) {
        hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(WGRAD_JOBS / 4, ns), dim3(256), 0, st, g);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(mlp_reduce_kernel, dim3(REDUCE_W_WG + (NBIAS + 3) / 4), dim3(256), 0, st, m->part, ns,
                           m->part_b, nwg, m->grads);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return mlp_fail(m, MD_E_HIP, hip_msg("md_mlp_backward", e));
    m->last_B = B;
    m->loss_parts = nwg;
    m->have_bwd = true;
    return MD_OK;
}

md_status md_mlp_get_grads(const md_mlp *m, float *h_grads) {
    if (!m || !h_grads) return MD_E_INVALID_ARG;
    (void)hipDeviceSynchronize();
    return hipMemcpy(h_grads, m->grads, sizeof(float) * md::MLP_NPARAMS, hipMemcpyDeviceToHost) == hipSuccess
               ? MD_OK
               : MD_E_HIP;
}

md_status md_mlp_loss(const md_mlp *m, double *out) {
    if (!m || !out) return MD_E_INVALID_ARG;
    if (!m->have_bwd) return MD_E_INVALID_ARG;
    (void)hipDeviceSynchronize();
    std::vector<double> h(m->loss_parts);
    if (hipMemcpy(h.data(), m->loss_part, sizeof(double) * h.size(), hipMemcpyDeviceToHost) != hipSuccess) return MD_E_HIP;
    double s = 0.0;
    for (double v : h) s += v;
    *out = s / ((double)m->last_B * md::MLP_OUT);
    return MD_OK;
}

md_status md_mlp_adam(md_mlp *m, float lr, float beta1, float beta2, float eps, void *stream) {
    if (!m || !(lr >= 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return MD_E_INVALID_ARG;
    if (!m->have_bwd) return mlp_fail(m, MD_E_INVALID_ARG, "adam needs gradients (call md_mlp_backward)");
    m->t += 1;
    const float bc1 = (float)(1.0 - std::pow((double)beta1, (double)m->t));
    const float bc2 = (float)(1.0 - std::pow((double)beta2, (double)m->t));
    hipLaunchKernelGGL(md::adam_kernel, dim3((md::MLP_NPARAMS + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       m->params, m->grads, m->m1, m->m2, m->Wf, m->Wt, md::MLP_NPARAMS, lr, beta1, beta2, eps, bc1, bc2);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? MD_OK : mlp_fail(m, MD_E_HIP, md::hip_msg("md_mlp_adam", e));
}

}  // extern "C"

namespace md {

const float *mlp_device_params(const md_mlp *m) { return m->params; }
const float *mlp_device_norm(const md_mlp *m) { return m->norm; }

}  // namespace md
