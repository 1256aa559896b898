// Training of one network (all widths up to 512) on gfx950 in three launches
// per minibatch.
//
// What bounds it: a minibatch of 4,096 rows is 4.6 GFLOP, a few microseconds of
// matrix work; launched product by product (24 kernels, the weight gradients
// on 2 to 32 blocks that each run through all 4,096 rows) it took 780 us.  So
//  * train_rows_kernel takes 16 rows per block through all four layers, the
//    loss and the three backward products; activations and errors stay in
//    LDS, the pre-activations in registers (the backward product of a layer
//    gives every lane the units and rows it had forward); weights come in
//    fragment order from L2.  16 rows, not 32, so that 4,096 rows fill 256 CUs;
//  * grad_kernel forms every weight and bias gradient in one launch, from
//    copies that the first kernel leaves unit by unit, so that both operands
//    are contiguous along the rows;
//  * adam_rows_kernel updates the parameters and writes the BF16 weights in the
//    three orders the other kernels read.
// Every product runs the layered GEMMs' MFMA sequence (16x16x32, the
// contraction in increasing steps): the trained weights have their bits.
// Measured (37-512-256-128-35, batch 4,096): 780 -> 57 us per minibatch (rows 28,
// gradients 18, update 6.5, the rest between launches; the rows kernel waits on
// weight fragments from L2 and on erf and exp of its GELU derivatives).

#include "surrogate_train.h"
#include "surrogate_math.h"

namespace chem {
namespace {

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kRows = 16;                       // rows per block
constexpr int kLd = kTrainMaxWidth + 8;         // LDS row of a layer's units (BF16), padded against conflicts
constexpr int kMaxJ = kTrainMaxWidth / 16 / kWaves;

// Element (n, k) of an [N][K] matrix in fragment order: its place in the 16 x 32
// operand of block n / 16 and step k / 32 (lane by lane, 8 values each).
__device__ __forceinline__ int64_t frag_at(int n, int k, int K)
{
    return ((int64_t)(n >> 4) * (K >> 5) + (k >> 5)) * 512 + ((n & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

// acc[j] += in (16 rows in LDS) x the weight fragments of column block
// wave + 8 j, over ksteps steps of 32.  Blocks past the layer repeat block 0
// (dropped by the caller), so that the loads have no branches around them.
template <int J, int D>
__device__ __forceinline__ void product_steps(const bf16_t *in, const bf16_t *__restrict__ Wf, int nblk, int ksteps,
                                              floatx4 (&acc)[kMaxJ])
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bf16_t *wf[J];
#pragma unroll
    for (int j = 0; j < J; j++) {
        const int jb = w + kWaves * j;
        wf[j] = Wf + (int64_t)(jb < nblk ? jb : 0) * ksteps * 512 + lane * 8;
        acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const bf16_t *arow = in + (lane & 15) * kLd + (lane >> 4) * 8;
    bf16x8 bq[D][J];   // fragments of the next D steps in flight
#pragma unroll
    for (int d = 0; d < D; d++)
#pragma unroll
        for (int j = 0; j < J; j++) __builtin_memcpy(&bq[d][j], wf[j] + d * 512, 16);
    for (int s0 = 0; s0 < ksteps; s0 += D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            const int ks = s0 + d;
            bf16x8 a;
            __builtin_memcpy(&a, arow + ks * 32, 16);
#pragma unroll
            for (int j = 0; j < J; j++) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bq[d][j], acc[j], 0, 0, 0);
            const int kn = ks + D < ksteps ? ks + D : ksteps - 1;
#pragma unroll
            for (int j = 0; j < J; j++) __builtin_memcpy(&bq[d][j], wf[j] + kn * 512, 16);
        }
    }
}

// K is a multiple of 64, nblk <= 8 kMaxJ
__device__ __forceinline__ void product(const bf16_t *in, const bf16_t *Wf, int nblk, int K, floatx4 (&acc)[kMaxJ])
{
    const int ksteps = K >> 5;
    if (nblk <= kWaves) {
        if (ksteps & 3) product_steps<1, 2>(in, Wf, nblk, ksteps, acc);
        else product_steps<1, 4>(in, Wf, nblk, ksteps, acc);
    } else if (nblk <= 2 * kWaves) {
        if (ksteps & 3) product_steps<2, 2>(in, Wf, nblk, ksteps, acc);
        else product_steps<2, 4>(in, Wf, nblk, ksteps, acc);
    } else {
        if (ksteps & 3) product_steps<4, 2>(in, Wf, nblk, ksteps, acc);
        else product_steps<4, 4>(in, Wf, nblk, ksteps, acc);
    }
}

// f(j, n) for this lane's columns n of a layer of nblk blocks
template <class F>
__device__ __forceinline__ void each_block(int nblk, F &&f)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int j = 0; j < kMaxJ; j++)
        if (w + kWaves * j < nblk) f(j, (w + kWaves * j) * 16 + (lane & 15));
}

// four rows of unit n: to LDS row by row (the next product's operand), and to
// the copy [unit][row] in fragment order (512 contiguous bytes per wave)
__device__ __forceinline__ void put(const bf16_t (&h)[4], int n, bf16_t *lds, bf16_t *__restrict__ T, int64_t ldT,
                                    int64_t r0)
{
    const int m = ((threadIdx.x & 63) >> 4) * 4;
    if (lds)
#pragma unroll
        for (int r = 0; r < 4; r++) lds[(m + r) * kLd + n] = h[r];
    uint2 pk;
    __builtin_memcpy(&pk, h, 8);
    *(uint2 *)(T + frag_at(n, (int)(r0 + m), (int)ldT)) = pk;
}

__global__ void __launch_bounds__(kThreads) train_rows_kernel(TrainArgs a)
{
    __shared__ __attribute__((aligned(16))) bf16_t buf[2][kRows * kLd];
    __shared__ double red[kWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t r0 = (int64_t)blockIdx.x * kRows;
    if (tid < kRows * 8) {
        // input rows, zero past the end
        const int r = tid >> 3, kc = (tid & 7) * 8;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (r0 + r < a.rows) {
            const int64_t src = a.order ? (int64_t)a.order[a.start + r0 + r] : a.start + r0 + r;
            v = *(const uint4 *)(a.X + src * 64 + kc);
        }
        *(uint4 *)&buf[0][r * kLd + kc] = v;
    }
    __syncthreads();
    if (tid < 128) {
        const int k = tid >> 1, half = (tid & 1) * 8;
        bf16_t x[8];
#pragma unroll
        for (int i = 0; i < 8; i++) x[i] = buf[0][(half + i) * kLd + k];
        uint4 pk;
        __builtin_memcpy(&pk, x, 16);
        *(uint4 *)(a.Xt + frag_at(k, (int)r0 + half, (int)a.ldT)) = pk;
    }
    floatx4 acc[kMaxJ];
    floatx4 u[3][kMaxJ];   // pre-activations of this lane's units
#pragma unroll
    for (int l = 0; l < 3; l++) {
        const int nblk = a.out_l[l] >> 4;
        product(buf[l & 1], a.W[l], nblk, a.in_l[l], acc);
        each_block(nblk, [&](int j, int n) __attribute__((always_inline)) {
            const float b = a.b[l][n];
            bf16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                u[l][j][r] = acc[j][r] + b;
                h[r] = act_bf16(gelu(u[l][j][r]));
            }
            put(h, n, buf[(l + 1) & 1], a.Ht[l], a.ldT, r0);
        });
        __syncthreads();
    }
    // output, loss and its derivative
    double s = 0.0;
    {
        const int nblk = a.out_l[3] >> 4;
        product(buf[1], a.W[3], nblk, a.in_l[3], acc);
        each_block(nblk, [&](int j, int n) __attribute__((always_inline)) {
            const float b = a.b[3][n];
            bf16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int64_t row = r0 + (lane >> 4) * 4 + r;
                float d = 0.0f;
                if (n < a.K && row < a.rows) {
                    const int64_t src = a.order ? (int64_t)a.order[a.start + row] : a.start + row;
                    d = acc[j][r] + b - a.Y[src * a.ldy + n];
                    s += (double)d * (double)d;
                }
                h[r] = to_bf16(a.scale * d);
            }
            put(h, n, buf[0], a.Dt[3], a.ldT, r0);
        });
        // the contraction of the next product is padded to a multiple of 64
        const int pad = ((a.out_l[3] + 63) & ~63) - a.out_l[3];
        for (int i = tid; i < kRows * pad; i += kThreads) buf[0][(i / pad) * kLd + a.out_l[3] + i % pad] = 0;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if (lane == 0) red[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < kWaves; i++) t += red[i];
        a.loss_part[blockIdx.x] = t;
    }
#pragma unroll
    for (int l = 2; l >= 0; l--) {
        // error of hidden layer l: (error of the next layer x its weights) gelu'(u)
        const int nblk = a.out_l[l] >> 4, Kd = (a.out_l[l + 1] + 63) & ~63;
        product(buf[l & 1], a.WT[l], nblk, Kd, acc);
        each_block(nblk, [&](int j, int n) __attribute__((always_inline)) {
            bf16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; r++) h[r] = act_bf16(acc[j][r] * gelu_grad(u[l][j][r]));
            put(h, n, l > 0 ? buf[(l + 1) & 1] : nullptr, a.Dt[l], a.ldT, r0);
        });
        if (l > 0) __syncthreads();
    }
}

// Weight gradients: one wave per 32 x 32 tile of a layer, through all rows in
// steps of 32 (the sum over the rows is one chain of products in row order, as
// the layer-by-layer GEMM forms it: a chain of 128 takes 2 us, and splitting
// it would round differently, which Adam's first steps, lr times the sign of
// the gradient, turn into other weights).  One-wave blocks, so that the 200
// tiles draw on 200 CUs' L1 rates; both operands come straight from L2 into
// registers, eight steps in flight.
// The blocks after the tiles sum the errors of 16 units each for their biases,
// by the scheme of the layered path: 64 row ranges, then the ranges in order.
__global__ void __launch_bounds__(64) grad_kernel(GradArgs a)
{
    const int lane = threadIdx.x;
    int t = blockIdx.x, l = 0;
    if (t >= a.all_tiles) {
        // lane: unit lane % 16 of a block of 16, every fourth range (the four
        // lanes of a unit read 256 contiguous bytes per group of 8 rows)
        __shared__ float part[16][65];
        t -= a.all_tiles;
        while (l < 3 && t >= a.out_l[l] >> 4) t -= a.out_l[l++] >> 4;
        const int unit = t * 16 + (lane & 15);
        const bf16_t *d = a.Dt[l];
        const int64_t per = (a.rows + 63) / 64;
        for (int c = lane >> 4; c < 64; c += 4) {
            const int64_t q0 = c * per, q1 = q0 + per < a.rows ? q0 + per : a.rows;
            float s = 0.0f;
            if (per % 8 == 0) {
#pragma unroll 8
                for (int64_t r = q0; r < q1; r += 8) {   // whole groups of 8; errors past the rows are 0
                    bf16_t x[8];
                    const uint4 v = *(const uint4 *)(d + frag_at(unit, (int)r, (int)a.ldT));
                    __builtin_memcpy(x, &v, 16);
#pragma unroll
                    for (int i = 0; i < 8; i++) s += r + i < q1 ? __uint_as_float((unsigned)x[i] << 16) : 0.0f;
                }
            } else {
                for (int64_t r = q0; r < q1; r++)
                    s += __uint_as_float((unsigned)d[frag_at(unit, (int)r, (int)a.ldT)] << 16);
            }
            part[lane & 15][c] = s;
        }
        __syncthreads();
        if (lane < 16) {
            float b = 0.0f;
#pragma unroll 16
            for (int c = 0; c < 64; c++) b += part[lane][c];
            a.g[a.off_b[l] + unit] = b;
        }
        return;
    }
    while (l < 3 && t >= a.tiles[l]) t -= a.tiles[l++];
    const int Nout = a.out_l[l], Kin = a.in_l[l], tn = Kin >> 5;
    const int m0 = (t / tn) * 32, n0 = (t % tn) * 32;
    const bf16_t *pa[2], *pb[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int m = m0 + i * 16;   // a block past the layer repeats its first one and is dropped
        pa[i] = a.Dt[l] + frag_at(m < Nout ? m : m0, 0, (int)a.ldT) + lane * 8;
        pb[i] = (l ? a.Ht[l - 1] : a.Xt) + frag_at(n0 + i * 16, 0, (int)a.ldT) + lane * 8;
    }
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr int D = 8;   // steps in flight
    const int64_t rows32 = (a.rows + 31) & ~int64_t(31);
    bf16x8 fa[D][2], fb[D][2];
    auto fetch = [&](int d, int64_t k) __attribute__((always_inline)) {
        const int64_t kk = k < rows32 ? k : rows32 - 32;   // past the end: fetched again, not used
#pragma unroll
        for (int i = 0; i < 2; i++) {
            __builtin_memcpy(&fa[d][i], pa[i] + kk * 16, 16);
            __builtin_memcpy(&fb[d][i], pb[i] + kk * 16, 16);
        }
    };
#pragma unroll
    for (int d = 0; d < D; d++) fetch(d, 32 * d);
    auto step = [&](int d) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[d][i], fb[d][j], acc[i][j], 0, 0, 0);
    };
    // whole groups without a branch, so that a step waits for its own loads only
    int64_t k = 0;
    for (; k + 32 * D <= rows32; k += 32 * D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            step(d);
            fetch(d, k + 32 * (d + D));
        }
    }
#pragma unroll
    for (int d = 0; d < D; d++)
        if (k + 32 * d < rows32) step(d);
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = m0 + i * 16 + (lane >> 4) * 4 + r;
            if (m < Nout)
#pragma unroll
                for (int j = 0; j < 2; j++)
                    a.g[a.off_W[l] + (int64_t)m * Kin + n0 + j * 16 + (lane & 15)] = acc[i][j][r];
        }
}

__device__ __forceinline__ void load8(const float *p, float (&x)[8])
{
    const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
    x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w, x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
}

__device__ __forceinline__ void store8(float *p, const float (&x)[8])
{
    *(float4 *)p = make_float4(x[0], x[1], x[2], x[3]);
    *(float4 *)(p + 4) = make_float4(x[4], x[5], x[6], x[7]);
}

// Eight adjacent parameters per thread (eight weights of one row, or biases):
// Adam unless `adam` is 0, and the BF16 weights row by row, in the forward and
// in the backward product's fragment order.
__global__ void __launch_bounds__(64) adam_rows_kernel(UpdateArgs a)
{
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 8;
    if (blockIdx.x == 0 && threadIdx.x < 64 && a.loss_part) {
        // the rows' squared errors, summed in a fixed order
        double s = 0.0;
        for (int b = threadIdx.x; b < a.loss_blocks; b += 64) s += a.loss_part[b];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
        if (threadIdx.x == 0) *a.loss += s;
    }
    if (!a.weights || i >= a.n_pad) return;
    float p[8];
    load8(a.o.p + i, p);
    if (a.adam) {
        float g[8], m[8], v[8];
        load8(a.o.g + i, g);
        load8(a.o.m + i, m);
        load8(a.o.v + i, v);
#pragma unroll
        for (int e = 0; e < 8; e++) {
            // these roundings whatever the surroundings: the weights of a run do not
            // depend on the path that computed its gradients
            m[e] = fmaf(a.o.omb1, g[e], a.o.beta1 * m[e]);
            v[e] = fmaf(g[e], a.o.omb2 * g[e], a.o.beta2 * v[e]);
            const float mh = m[e] / a.o.bc1, vh = v[e] / a.o.bc2;
            p[e] -= a.o.lr * mh / (sqrtf(vh) + a.o.eps);
        }
        store8(a.o.m + i, m);
        store8(a.o.v + i, v);
        store8(a.o.p + i, p);
    }
    bf16_t h[8];
#pragma unroll
    for (int e = 0; e < 8; e++) h[e] = to_bf16(p[e]);
    uint4 pk;
    __builtin_memcpy(&pk, h, 16);
    *(uint4 *)(a.wbf + i) = pk;
    int l = 0;
    while (l < 3 && i >= a.off_W[l + 1]) l++;
    const int64_t o = i - a.off_W[l];
    const int K = a.in_l[l];
    if (o >= (int64_t)a.out_l[l] * K) return;   // biases
    const int n = (int)(o / K), k = (int)(o % K);
    *(uint4 *)(a.wfrag + a.off_W[l] + frag_at(n, k, K)) = pk;
    if (l > 0 && a.wfragT) {
        const int Nt = (a.out_l[l] + 63) & ~63;
#pragma unroll
        for (int e = 0; e < 8; e++) a.wfragT[a.off_T[l] + frag_at(k + e, n, Nt)] = h[e];
    }
}

}  // namespace

bool train_fused_supported(const int in_l[4], const int out_l[4])
{
    if (in_l[0] != 64) return false;
    for (int l = 0; l < 3; l++)
        if (out_l[l] > kTrainMaxWidth || out_l[l] % 64 != 0) return false;
    return out_l[3] % 16 == 0 && out_l[3] <= 64;
}

hipError_t launch_train_rows(const TrainArgs &a, hipStream_t s)
{
    // whole steps of 32 rows for grad_kernel: the last block may hold no row
    const int64_t blocks = (a.rows + 31) / 32 * 2;
    hipLaunchKernelGGL(train_rows_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_grad(const GradArgs &a, hipStream_t s)
{
    const int units = (a.out_l[0] + a.out_l[1] + a.out_l[2] + a.out_l[3]) / 16;
    hipLaunchKernelGGL(grad_kernel, dim3((unsigned)(a.all_tiles + units)), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_update(const UpdateArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(adam_rows_kernel, dim3(blocks_for(a.n_pad, 64 * 8)), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace chem
