// Kernels of the learned sampling proposal: a 40 -> 512 x 4 -> 144 SiLU network with
// BF16 operands and FP32 accumulation on the gfx950 matrix cores.
//
// A training step is three launches: the pass over the network (forward, loss and backward of
// a block of rows in one workgroup, activations and errors on the chip), the weight gradients of
// all layers, and the parameter pass.  Every product is C = A B^T with both operands in the
// order in which the matrix instruction takes them:
//   forward     Z_l   = H_{l-1} W_l            A = H_{l-1} [B x fi],  B = W_l^T [fo x fi]
//   input grad  dA    = dZ_l W_l^T             A = dZ_l    [B x fo],  B = W_l   [fi x fo]
//   weight grad dW_l  = H_{l-1}^T dZ_l         A = H^T     [fi x B],  B = dZ^T  [fo x B]
// The weight gradient reduces over the batch and is split along it; the split partials
// and the per-row-block bias-gradient column sums are reduced in a fixed order, so a training
// step is deterministic.
#include <hip/hip_runtime.h>

#include "mlp_launch.h"

namespace mlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 ld8(const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }

constexpr int BK = kGemmBK;
constexpr int kPF = 2;       // k-tiles of global loads in flight

// 1 / (1 + exp(-z)).  exp(x) = 2^n 2^f with n + f = x log2(e) (the product in two parts, n its
// nearest whole number) and the hardware's 2^f; the quotient from the hardware's reciprocal and
// a Newton step; where exp(-z) is beyond float that gives NaN and the maximum 0.  Without the
// general division and the range checks of 1.f / (1.f + expf(-z)), two thirds of its
// instructions: a pass over 256 rows 19.4 us instead of 20.6, a training step's over 4096 rows
// 51 instead of 53.  Largest and rms relative error over [-87, 110] as that form's: 1.5e-7 and
// 3.8e-8; below -87.3 the result is not above 1.2e-38 and may be 0.
__device__ __forceinline__ float sigm(float z)
{
#pragma clang fp contract(off)
    const float x = __builtin_amdgcn_fmed3f(-z, -87.f, 89.f);
    const float t = x * 1.44269504f, n = rintf(t);
    const float f = (t - n) + fmaf(x, 1.92596300e-8f, fmaf(x, 1.44269504f, -t));
    const float d = 1.f + __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaxf(fmaf(fmaf(-d, r, 1.f), r, r), 0.f);
}
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float dsilu(float z)
{
    const float s = sigm(z);
    return s * (1.f + z * (1.f - s));
}

// The BF16 copies W^T and W are stored in the order in which the matrix instruction takes them:
// blocks of 16 rows (n) by 32 columns (k), k-blocks of a row panel consecutive, and in a block
// the 8 k-values of row l mod 16 and columns 8 (l / 16) .. +7 at place l.  A wave's fragment is
// 1 KiB in a row (read from rows of W^T it touched 16 lines for half a line each).
// frag_offset: element offset of row n, column k (a multiple of 8) of a matrix of K columns.
__device__ __forceinline__ size_t frag_offset(int n, int k, int K)
{
    return ((size_t)(n >> 4) * (K >> 5) + (k >> 5)) * 512 + ((n & 15) + 16 * ((k >> 3) & 3)) * 8;
}

// The activations and errors that the weight gradients reduce over the batch are in the same
// order in halves: a block holds column panel n / 16 of 16 batch rows r, and the panels of a
// group of 16 rows are consecutive, so what a row block writes of a layer is one run of 16 KiB.
// (With the rows along the panels instead, runs of 512 B at strides of the batch, a training
// step's pass over 4096 rows, then 59.5 us and now 51, took 61.8, the weight gradients the same.)
// batch_offset: element offset of column n, rows r (a multiple of 8) .. +7 of N columns.
__device__ __forceinline__ size_t batch_offset(int n, int r, int N)
{
    return ((size_t)(r >> 4) * (N >> 4) + (n >> 4)) * 256 + ((n & 15) + 16 * ((r >> 3) & 1)) * 8;
}

// ---------------------------------------------------------------------------------
// Weight gradients of all layers in one launch: dW_l[i][o] = sum over the batch of
// H_{l-1}[r][i] dZ_l[r][o], a 128 x 128 tile and one split of the batch for each workgroup of
// 4 waves (2 x 2, each 64 x 64).  Both operands are stored in fragment order along the batch,
// so a wave's 16 B loads, its LDS stores and its fragment reads each run over 1 KiB in a row,
// with the loads of the next kPF k-tiles in flight (in registers) while the current tile's
// products run and the next k-tile on its way to the other half of the LDS.  What bounds it is
// the way of the operands from memory, 34 MB for 4096 rows that other XCDs have just written:
// 64 x 64 tiles with twice the LDS traffic took the same time.  For 4096 rows 19 us, in launches
// for each layer 56 together; 4 splits instead of 8 save 2 us of a training step (15 MB fewer
// partials), but another order of the sums turns the first updates of parameters whose gradient
// is nearly zero.  dZ is the instruction's first operand, so a lane's four sums are consecutive
// columns of dW and leave as 16 bytes.  Where a matrix ends inside a tile (64 rows of the first
// layer, 192 columns of the last) the panels past its end repeat the last one and are not stored.
// ---------------------------------------------------------------------------------
constexpr int kGradTile = 128, kGradPanels = kGradTile / 16, kGradWave = kGradPanels / 2;
struct WgradArgs {
    GemmArgs g[kLayers];
    int first[kLayers + 1];  // first tile of each layer
    int splits;
};
__global__ __launch_bounds__(256, 2) void wgrad_kernel(WgradArgs w)
{
    __shared__ __align__(16) __bf16 sA[2][kGradTile * BK], sB[2][kGradTile * BK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int split = blockIdx.x % w.splits, tile = blockIdx.x / w.splits;
    int l = 0;
    while (l < kLayers - 1 && tile >= w.first[l + 1]) ++l;
    const GemmArgs& g = w.g[l];
    const int mp = g.M / 16, np = g.N / 16, mt = (mp + kGradPanels - 1) / kGradPanels;  // panels of 16, tiles
    const int mp0 = ((tile - w.first[l]) % mt) * kGradPanels, np0 = ((tile - w.first[l]) / mt) * kGradPanels;
    // 16 bytes of panel tid / 32 in each of the k-tile's 4 groups of 16 rows
    constexpr int C = BK / 16;
    const int pan = tid >> 5, at = split * g.K, pa = min(mp0 + pan, mp - 1), pb = min(np0 + pan, np - 1);
    u32x4 ra[kPF][C], rb[kPF][C];
    auto load = [&](int s, int k0) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int kg = (at + k0) / 16 + c;
            ra[s][c] = *reinterpret_cast<const u32x4*>(g.A + ((size_t)kg * mp + pa) * 256 + (tid & 31) * 8);
            rb[s][c] = *reinterpret_cast<const u32x4*>(g.B + ((size_t)kg * np + pb) * 256 + (tid & 31) * 8);
        }
    };
    auto store = [&](int s, int half) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int slot = ((pan * 2 + (c >> 1)) * 64 + (c & 1) * 32 + (tid & 31)) * 8;
            *reinterpret_cast<u32x4*>(sA[half] + slot) = ra[s][c];
            *reinterpret_cast<u32x4*>(sB[half] + slot) = rb[s][c];
        }
    };
    f32x4 acc[kGradWave][kGradWave];
#pragma unroll
    for (int i = 0; i < kGradWave; ++i)
#pragma unroll
        for (int j = 0; j < kGradWave; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kPF; ++s)
        if (s * BK < g.K) load(s, s * BK);
    store(0, 0);
    if (kPF * BK < g.K) load(0, kPF * BK);
    __syncthreads();
    const int wm = kGradWave * (wave >> 1), wn = kGradWave * (wave & 1);  // first panels of the wave
    for (int kt = 0; kt < g.K; kt += kPF * BK) {
#pragma unroll
        for (int s = 0; s < kPF; ++s) {
            // k-tile k0 is in half s mod 2 (kPF is even); the next goes into the other half, and
            // its registers take the k-tile kPF after it
            const int k0 = kt + s * BK, s1 = (s + 1) % kPF;
            if (k0 >= g.K) break;
            if (k0 + BK < g.K) store(s1, (s + 1) & 1);
            if (k0 + (kPF + 1) * BK < g.K) load(s1, k0 + (kPF + 1) * BK);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bf16x8 a[kGradWave], b[kGradWave];
#pragma unroll
                for (int i = 0; i < kGradWave; ++i) {
                    a[i] = ld8(sA[s & 1] + ((wm + i) * 2 + h) * 512 + lane * 8);
                    b[i] = ld8(sB[s & 1] + ((wn + i) * 2 + h) * 512 + lane * 8);
                }
#pragma unroll
                for (int i = 0; i < kGradWave; ++i)
#pragma unroll
                    for (int j = 0; j < kGradWave; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
            }
            __syncthreads();
        }
    }
    float* D = g.C + (size_t)split * g.c_split_stride;
#pragma unroll
    for (int i = 0; i < kGradWave; ++i)
#pragma unroll
        for (int j = 0; j < kGradWave; ++j)
            if (mp0 + wm + i < mp && np0 + wn + j < np)
                *reinterpret_cast<f32x4*>(D + (size_t)(16 * (mp0 + wm + i) + (lane & 15)) * g.ldc +
                                          16 * (np0 + wn + j) + (lane >> 4) * 4) = acc[i][j];
}

hipError_t launch_gemm(int epi, const GemmArgs& g, int splits, hipStream_t st)
{
    WgradArgs w{};
    int n = 0, tiles = 0;
    if (epi != EPI_SPLITK || splits < 1 || splits > kMaxSplits) return hipErrorInvalidValue;
    for (const GemmArgs* p = &g; p; p = p->next) {
        if (n == kLayers || !gemm_tile_m(p->M, p->N, splits) || p->K <= 0 || p->K % BK || p->lda != p->ldb ||
            p->lda < p->K * splits || p->lda % 32)
            return hipErrorInvalidValue;
        w.g[n] = *p;
        w.first[n++] = tiles;
        tiles += ((p->M + kGradTile - 1) / kGradTile) * ((p->N + kGradTile - 1) / kGradTile);
    }
    for (; n <= kLayers; ++n) w.first[n] = tiles;
    w.splits = splits;
    hipLaunchKernelGGL(wgrad_kernel, dim3(tiles * splits), dim3(256), 0, st, w);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// A pass over the network in one launch: a workgroup takes kNetRows rows through every layer,
// its activations in LDS, each of its 8 waves 64 of a hidden layer's 512 columns.  What bounds
// it is the stream of weights from L2, 1.75 MB for every workgroup whatever its rows (a training
// step takes 1.7 MB more): the waves read their fragments straight from memory (no other wave of
// the workgroup needs them), four 64-wide k-tiles ahead of the products (two: the same for 256
// rows, and 55 us against 51 for a training step's 4096).  16 rows, the matrix
// instruction's height, give the most workgroups: one row block's time is the pass's time up to
// 4096 rows (one a compute unit), where a launch for every layer paid its start and its drain.
// Launches per layer / here, us a pass: 1 row 29.1 / 18.3, 256 rows 29.4 / 19.4, 4096 rows 39.9
// / 21.5, 16384 rows 102 / 77; with three policies in turn, whose weights together exceed an
// XCD's L2, 256 rows 30.2 / 19.8.  A training step (three launches against sixteen): 64 rows
// 90 / 53, 512 rows 104 / 57, 4096 rows 150 / 75, 16384 rows 413 / 237.  The loss alone: 4096
// rows 52 / 24.
// ---------------------------------------------------------------------------------
constexpr int kNetThreads = 512, kNetLd = kHidden + 8, kOutLd = kOut + 4;

// the fragments of a wave's TN column tiles in flight: D k-tiles of 64
template <int TN, int D>
struct NetFrags {
    bf16x8 w[D][TN][2];
};

// k-tile t of the TN column tiles at b (W^T in fragment order, K columns, tiles `step` apart)
template <int K, int TN, int D>
__device__ __forceinline__ void net_load(const __bf16* b, int step, int t, NetFrags<TN, D>& f)
{
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) f.w[t % D][j][h] = ld8(b + (j * step * K * 16 + (2 * t + h) * 512) + (threadIdx.x & 63u) * 8);
}
template <int K, int TN, int D>
__device__ __forceinline__ void net_start(const __bf16* b, int step, NetFrags<TN, D>& f)
{
#pragma unroll
    for (int t = 0; t < D; ++t)
        if (t < K / 64) net_load<K, TN, D>(b, step, t, f);
}

// acc[j] = A (16 rows of LDS at sA, pitch kNetLd) x the column tiles, whose first fragments
// net_start has put in flight
template <int K, int TN, int D>
__device__ __forceinline__ void net_product(const __bf16* sA, const __bf16* b, int step, NetFrags<TN, D>& f, f32x4 acc[TN])
{
    constexpr int NT = K / 64;
    const int lane = threadIdx.x & 63;
    const __bf16* a = sA + (lane & 15) * kNetLd + (lane >> 4) * 8;
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bf16x8 av = ld8(a + 64 * t + 32 * h);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, f.w[t % D][j][h], acc[j], 0, 0, 0);
        }
        if (t + D < NT) net_load<K, TN, D>(b, step, t + D, f);
    }
}

// z = acc + b; silu(z) rounded to bf16 into the wave's columns of sH.  TRAIN: also to Ht in
// fragment order along the batch, and silu'(z) into dz, where the backward pass of this row
// block finds it.
template <bool TRAIN>
__device__ __forceinline__ void net_activate(const f32x4 acc[4], const float bv[4], __bf16* sH, int n0, __bf16* Ht,
                                             int r0, f32x4 dz[4])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + 16 * j + (lane & 15);
        bf16x4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float z = acc[j][r] + bv[j];
            h[r] = (__bf16)silu(z);
            sH[((lane >> 4) * 4 + r) * kNetLd + n] = h[r];
            if constexpr (TRAIN) {
                // computed here: left to itself the compiler keeps z and the sigmoid instead, two
                // registers for one
                float d = dsilu(z);
                asm volatile("" : "+v"(d));
                dz[j][r] = d;
            }
        }
        if constexpr (TRAIN) *reinterpret_cast<bf16x4*>(Ht + batch_offset(n, r0 + 8 * (lane >> 5), kHidden) + 4 * ((lane >> 4) & 1)) = h;
    }
}

// the output's TN column tiles j0, j0 + 8, whose first fragments are in flight, to the output
// rows or (SCORE) to the LDS rows sO
template <bool SCORE, int TN, int D>
__device__ __forceinline__ void net_output(const PrepArgs& p, const __bf16* sA, const __bf16* b, int j0, int r0,
                                           NetFrags<TN, D>& f, float* sO)
{
    const int lane = threadIdx.x & 63;
    f32x4 acc[TN];
    net_product<kHidden>(sA, b, 8, f, acc);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = 16 * (j0 + 8 * j) + (lane & 15);
        const float bv = p.net.bias[kLayers - 1][n];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = (lane >> 4) * 4 + r;
            if constexpr (SCORE) sO[row * kOutLd + n] = acc[j][r] + bv;
            else if (r0 + row < p.B) p.net.out[(size_t)(r0 + row) * kOut + n] = acc[j][r] + bv;
        }
    }
}

// Workgroups past the row blocks bring the weights into their XCD's L2 (workgroups go round the
// XCDs), part `part` of kNetWarm each: a few row blocks alone fetch them with a compute unit's
// misses in flight for each XCD, and a pass whose weights are not in L2 (several policies in
// turn, or after an update) waits for that: 256 rows, three policies in turn, 29.4 us without
// them, 19.8 with; a training step of 64 rows 63 and 53.  From
// kNetWarmBlocks row blocks on (16 an XCD) those have as much in flight themselves.  The values
// are not used.
constexpr int kNetWarm = 8, kXcds = 8, kNetWarmBlocks = 128;
__device__ __forceinline__ void net_warm(const __bf16* w, int elements, int part)
{
    const int bytes = elements * 2 / kNetWarm;
    const char* src = reinterpret_cast<const char*>(w) + (size_t)part * bytes;
#pragma unroll 8
    for (int i = threadIdx.x * 16; i < bytes; i += kNetThreads * 16) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(src + i);
        asm volatile("" ::"v"(v));
    }
}

// Gaussian NLL of the row block's output (LDS rows sO) against the standardised targets: the
// block's loss partial and, for a training step, dL/d(output): float over sO, bf16 rows with
// zero padding columns to sD, along the batch to dZt, and the block's column sums.
constexpr int kLossElems = (kNetRows * 72 + kNetThreads - 1) / kNetThreads;
struct NetTarget {
    float y[kLossElems];
};
__device__ __forceinline__ void net_target(const PrepArgs& p, int r0, NetTarget& t)
{
#pragma unroll
    for (int j = 0; j < kLossElems; ++j) {
        const int e = threadIdx.x + kNetThreads * j, rr = e / 72, d = e - rr * 72, r = r0 + rr;
        t.y[j] = 0.f;
        if (rr < kNetRows && r < p.B) {
            const int row = p.idx ? p.idx[r] : r;
            t.y[j] = (p.net.loss.Y[(size_t)row * 72 + d] - p.net.loss.omean[d]) / p.net.loss.ostd[d];
        }
    }
}
template <bool TRAIN>
__device__ __forceinline__ void net_loss(const PrepArgs& p, int r0, int block, const NetTarget& t, float* sO,
                                         __bf16* sD, float* red)
{
    const int tid = threadIdx.x;
    const float inv = 1.f / ((float)p.B * 72.f);
    float lsum = 0.f;
#pragma unroll
    for (int j = 0; j < kLossElems; ++j) {
        const int e = tid + kNetThreads * j, rr = e / 72, d = e - rr * 72;
        if (rr >= kNetRows) break;
        float dm = 0.f, dsv = 0.f;
        if (r0 + rr < p.B) {
            const float m = sO[rr * kOutLd + d], s = sO[rr * kOutLd + 72 + d];
            const float err = t.y[j] - m, w = expf(-2.f * s), q = err * err * w;
            lsum += 0.5f * q + s;
            dm = -err * w * inv;
            dsv = (1.f - q) * inv;
        }
        if constexpr (TRAIN) {
            sO[rr * kOutLd + d] = dm;
            sO[rr * kOutLd + 72 + d] = dsv;
            sD[rr * kNetLd + d] = (__bf16)dm;
            sD[rr * kNetLd + 72 + d] = (__bf16)dsv;
        }
    }
#pragma unroll
    for (int o = 32; o; o >>= 1) lsum += __shfl_xor(lsum, o);
    if (!(tid & 63)) red[tid >> 6] = lsum;
    if constexpr (TRAIN) {
        constexpr int kPad = kOutPad - kOut;
        for (int e = tid; e < kNetRows * kPad; e += kNetThreads)
            sD[(e / kPad) * kNetLd + kOut + e % kPad] = (__bf16)0.f;
    }
    __syncthreads();
    if (tid == 0) {
        float s = red[0];
        for (int k = 1; k < kNetThreads / 64; ++k) s += red[k];
        p.net.loss.lpart[block] = s;
    }
    if constexpr (TRAIN) {
        if (tid < 2 * kOutPad) {
            const int c = tid % kOutPad, h = 8 * (tid / kOutPad);
            bf16x8 v;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = sD[(h + u) * kNetLd + c];
            *reinterpret_cast<bf16x8*>(p.net.loss.dZt + batch_offset(c, r0 + h, kOutPad)) = v;
        }
        if (tid >= kNetThreads - kOutPad) {  // the waves that wrote none of it
            const int c = tid - (kNetThreads - kOutPad);
            float s = 0.f;
#pragma unroll
            for (int rr = 0; rr < kNetRows; ++rr) s += sO[rr * kOutLd + min(c, kOut - 1)];
            p.net.loss.dbpart[(size_t)block * kOutPad + c] = c < kOut ? s : 0.f;
        }
    }
}

// One step back: acc = dL/dh of the wave's columns, dz = acc silu'(z) to sD (unless it is the
// LAST step), along the batch to dZt, and the block's column sums
template <bool LAST>
__device__ __forceinline__ void net_back(const f32x4 acc[4], const f32x4 ds[4], __bf16* sD, int n0, __bf16* dZt,
                                         float* bpart, int r0)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + 16 * j + (lane & 15);
        bf16x4 h;
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float dz = acc[j][r] * ds[j][r];
            s += dz;
            h[r] = (__bf16)dz;
            if constexpr (!LAST) sD[((lane >> 4) * 4 + r) * kNetLd + n] = h[r];
        }
        *reinterpret_cast<bf16x4*>(dZt + batch_offset(n, r0 + 8 * (lane >> 5), kHidden) + 4 * ((lane >> 4) & 1)) = h;
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lane < 16) bpart[n] = s;
    }
}

// MODE NET_FORWARD: the output rows.  NET_LOSS: the loss partials.  NET_TRAIN: also the
// backward pass of the row block, its silu' of every layer in registers (64 of them a lane),
// leaving the operands of the weight gradients.
template <int MODE>
__global__ __launch_bounds__(kNetThreads, 2) void net_kernel(PrepArgs p)
{
    constexpr bool kTrain = MODE == NET_TRAIN, kScore = MODE != NET_FORWARD;
    __shared__ __align__(16) __bf16 sH[2][kNetRows * kNetLd];
    __shared__ float sO[kScore ? kNetRows * kOutLd : 1];
    __shared__ float red[kNetThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, r0 = blockIdx.x * kNetRows;
    // known to be the same for the wave: its weights are addressed from scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (r0 >= (kScore ? p.Bp : p.B)) {
        const int part = (blockIdx.x / kXcds) % kNetWarm;
#pragma unroll 1
        for (int l = 0; l < kLayers; ++l)
            net_warm(p.net.Wt[l], (l ? kHidden : kInPad) * (l < kLayers - 1 ? kHidden : kOut), part);
        if constexpr (kTrain)
#pragma unroll 1
            for (int l = kLayers - 1; l; --l) net_warm(p.net.Wn[l], kHidden * (l < kLayers - 1 ? kHidden : kOutPad), part);
        return;
    }
    const int n0 = wave * 64;
    NetFrags<4, 4> f;
    f32x4 acc[4];
    f32x4 ds[kLayers - 1][4];
    float bv[4];
    // each layer's first fragments and biases are requested before the wait for its input
    net_start<kInPad>(p.net.Wt[0] + (size_t)n0 * kInPad, 1, f);
#pragma unroll
    for (int j = 0; j < 4; ++j) bv[j] = p.net.bias[0][n0 + 16 * j + (lane & 15)];
    for (int e = tid; e < kNetRows * kInPad; e += kNetThreads) {
        const int rr = e / kInPad, c = e - rr * kInPad, r = r0 + rr;
        float v = 0.f;
        if (r < p.B && c < kIn) {
            const int row = p.idx ? p.idx[r] : r;
            v = (p.X[(size_t)row * kIn + c] - p.mean[c]) / p.std[c];
        }
        sH[0][rr * kNetLd + c] = (__bf16)v;
    }
    __syncthreads();
    if constexpr (kTrain) {
        if (tid < 2 * kInPad) {
            const int c = tid % kInPad, h = 8 * (tid / kInPad);
            bf16x8 v;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = sH[0][(h + u) * kNetLd + c];
            *reinterpret_cast<bf16x8*>(p.X0t + batch_offset(c, r0 + h, kInPad)) = v;
        }
    }
    net_product<kInPad>(sH[0], p.net.Wt[0] + (size_t)n0 * kInPad, 1, f, acc);
#pragma unroll(kTrain ? kLayers : 1)
    for (int l = 1; l < kLayers - 1; ++l) {
        const __bf16* b = p.net.Wt[l] + (size_t)n0 * kHidden;
        net_start<kHidden>(b, 1, f);
        net_activate<kTrain>(acc, bv, sH[l & 1], n0, p.net.Ht[l - 1], r0, ds[kTrain ? l - 1 : 0]);
#pragma unroll
        for (int j = 0; j < 4; ++j) bv[j] = p.net.bias[l][n0 + 16 * j + (lane & 15)];
        __syncthreads();
        net_product<kHidden>(sH[l & 1], b, 1, f, acc);
    }
    // the output's 9 column tiles: one a wave, the ninth by the first wave
    const __bf16* sL = sH[(kLayers - 1) & 1];
    const __bf16* b = p.net.Wt[kLayers - 1] + (size_t)wave * (kHidden * 16);
    NetFrags<2, 2> f2;
    NetFrags<1, 4> f1;
    if (wave == 0) net_start<kHidden>(b, 8, f2);
    else net_start<kHidden>(b, 8, f1);
    NetTarget y;
    if constexpr (kScore) net_target(p, r0, y);
    net_activate<kTrain>(acc, bv, sH[(kLayers - 1) & 1], n0, p.net.Ht[kLayers - 2], r0, ds[kLayers - 2]);
    __syncthreads();
    if (wave == 0) net_output<kScore>(p, sL, b, 0, r0, f2, sO);
    else net_output<kScore>(p, sL, b, wave, r0, f1, sO);
    if constexpr (kScore) {
        constexpr int kTop = (kLayers - 1) & 1;  // the output's input has been read by then
        const __bf16* w = p.net.Wn[kLayers - 1] + (size_t)n0 * kOutPad;
        if constexpr (kTrain) net_start<kOutPad>(w, 1, f);
        __syncthreads();
        net_loss<kTrain>(p, r0, blockIdx.x, y, sO, sH[kTop], red);
        if constexpr (kTrain) {
            net_product<kOutPad>(sH[kTop], w, 1, f, acc);
#pragma unroll
            for (int l = kLayers - 2; l > 0; --l) {  // layer l's dz from layer l + 1's product
                const __bf16* wl = p.net.Wn[l] + (size_t)n0 * kHidden;
                __bf16* sD = sH[l & 1];
                net_start<kHidden>(wl, 1, f);
                net_back<false>(acc, ds[l], sD, n0, p.net.dZt[l], p.net.bpart[l] + (size_t)blockIdx.x * kHidden, r0);
                __syncthreads();
                net_product<kHidden>(sD, wl, 1, f, acc);
            }
            net_back<true>(acc, ds[0], nullptr, n0, p.net.dZt[0], p.net.bpart[0] + (size_t)blockIdx.x * kHidden, r0);
        }
    }
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t st)
{
    const int rows = ((a.net.mode == NET_FORWARD ? a.B : a.Bp) + kNetRows - 1) / kNetRows;
    const dim3 grid(rows + (rows < kNetWarmBlocks ? kXcds * kNetWarm : 0));
    switch (a.net.mode) {
    case NET_FORWARD: hipLaunchKernelGGL(net_kernel<NET_FORWARD>, grid, dim3(kNetThreads), 0, st, a); break;
    case NET_LOSS: hipLaunchKernelGGL(net_kernel<NET_LOSS>, grid, dim3(kNetThreads), 0, st, a); break;
    case NET_TRAIN: hipLaunchKernelGGL(net_kernel<NET_TRAIN>, grid, dim3(kNetThreads), 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Parameter pass: the fixed-order gradient reduction, Adam, and the BF16 shadows, in one
// kernel with three modes over the same work split.  Every layer's fan-out is a multiple
// of 4 and its parameter offset too, so threads own groups of 4 consecutive columns and
// move them as 16-byte vectors.
//   Weight tiles, kTileI x kTileO of one layer's W (rows i, columns o): thread t owns
//   columns o0 + 4 (t mod 16) .. +3 of rows i0 + t/16 and i0 + t/16 + 16.  The split-K
//   partials, P, m, v and the row-major shadow W are accessed along o; the transposed
//   shadow W^T goes through an LDS tile and leaves as 16-byte pieces of its rows.
//   Bias blocks, 64 columns of one layer's b: 16 row groups sum contiguous slices of the
//   per-tile column partials, then the 16 sums are added in a fixed order.
// The reduction order is the same in every mode, so the fused step equals reduce + Adam
// bit for bit; the first bias block also sums the loss partials.
// ---------------------------------------------------------------------------------
constexpr int kTileI = 32, kTileO = 64;
enum { PASS_REDUCE = 0, PASS_ADAM = 1, PASS_REDUCE_ADAM = 2 };

__device__ __forceinline__ int weight_tiles(const LayerGeom& g, int l)
{
    return ((g.fi[l] + kTileI - 1) / kTileI) * ((g.fo[l] + kTileO - 1) / kTileO);
}

static int pass_blocks(const LayerGeom& g)
{
    int n = 0;
    for (int l = 0; l < kLayers; ++l)
        n += ((g.fi[l] + kTileI - 1) / kTileI) * ((g.fo[l] + kTileO - 1) / kTileO) + (g.fo[l] + 63) / 64;
    return n;
}

// Adam (Kingma and Ba) on 4 consecutive parameters from p (16-byte aligned):
// m <- b1 m + (1-b1) g, v <- b2 v + (1-b2) g^2, p <- p - lr (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps);
// returns the (new) weights
__device__ __forceinline__ f32x4 adam4(const AdamArgs& a, int p, f32x4 gr)
{
    f32x4 w = *reinterpret_cast<const f32x4*>(a.P + p);
    if (a.update) {
        f32x4 m = *reinterpret_cast<const f32x4*>(a.m + p), v = *reinterpret_cast<const f32x4*>(a.v + p);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            m[u] = a.b1 * m[u] + a.omb1 * gr[u];
            v[u] = a.b2 * v[u] + a.omb2 * gr[u] * gr[u];
            w[u] -= a.lr * (m[u] * a.inv_c1) / (sqrtf(v[u] * a.inv_c2) + a.eps);
        }
        *reinterpret_cast<f32x4*>(a.m + p) = m;
        *reinterpret_cast<f32x4*>(a.v + p) = v;
        *reinterpret_cast<f32x4*>(a.P + p) = w;
    }
    return w;
}

template <int MODE>
__global__ __launch_bounds__(256) void param_pass_kernel(ReduceArgs r, AdamArgs a)
{
    __shared__ __align__(16) __bf16 sT[kTileO][kTileI + 8];
    __shared__ __align__(16) float sS[16][64];
    const LayerGeom& g = (MODE == PASS_ADAM) ? a.g : r.g;
    const int t = threadIdx.x, oq = t & 15, rg = t >> 4;
    int rem = blockIdx.x, l = 0;
    while (l < kLayers && rem >= weight_tiles(g, l)) rem -= weight_tiles(g, l++);
    if (l < kLayers) {  // ---- weight tile
        const int fi = g.fi[l], fo = g.fo[l], fip = g.fip[l], fop = g.fop[l];
        const int nto = (fo + kTileO - 1) / kTileO;
        const int i0 = (rem / nto) * kTileI, o0 = (rem % nto) * kTileO, o = o0 + 4 * oq;
        const bool ocol = o < fo;  // all four columns (fo is a multiple of 4)
        f32x4 gr[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        if constexpr (MODE != PASS_ADAM) {
            // all partial loads issued together: rows and columns of the tile stay inside
            // the fip x fop planes, and planes past the last split re-read the last one
            const int S = r.S[l];
            const size_t stride = (size_t)fip * fop;
            f32x4 v[2][kMaxSplits];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float* wp = r.wpart[l] + (size_t)(i0 + rg + 16 * h) * fop + o;
#pragma unroll
                for (int k = 0; k < kMaxSplits; ++k)
                    v[h][k] = *reinterpret_cast<const f32x4*>(wp + (size_t)min(k, S - 1) * stride);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int k = 0; k < kMaxSplits; ++k)
                    if (k < S) gr[h] += v[h][k];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int il = rg + 16 * h, i = i0 + il;
            f32x4 w = f32x4{0.f, 0.f, 0.f, 0.f};
            if (ocol && i < fi) {
                const int p = g.off[l] + i * fo + o;
                if constexpr (MODE == PASS_REDUCE) {
                    *reinterpret_cast<f32x4*>(r.G + p) = gr[h];
                } else {
                    if constexpr (MODE == PASS_ADAM)
                        gr[h] = a.update ? *reinterpret_cast<const f32x4*>(a.G + p) : f32x4{0.f, 0.f, 0.f, 0.f};
                    w = adam4(a, p, gr[h]);
                }
            }
            if constexpr (MODE != PASS_REDUCE) {
#pragma unroll
                for (int u = 0; u < 4; ++u) sT[4 * oq + u][il] = (__bf16)w[u];
            }
        }
        if constexpr (MODE != PASS_REDUCE) {
            __syncthreads();
            const int row = t >> 2, c = t & 3;  // 64 rows of W^T, 4 pieces of 8 each
            *reinterpret_cast<bf16x8*>(a.Wt[l] + frag_offset(o0 + row, i0 + 8 * c, fip)) =
                *reinterpret_cast<const bf16x8*>(&sT[row][8 * c]);
            if (a.Wn[l]) {  // 32 rows of W, 8 pieces of 8 each: a wave's stores 1 KiB in a row
                const int i = (t & 15) + 16 * (t >> 7), k8 = 8 * ((t >> 4) & 7);
                bf16x8 v;
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = sT[k8 + u][i];
                *reinterpret_cast<bf16x8*>(a.Wn[l] + frag_offset(i0 + i, o0 + k8, fop)) = v;
            }
        }
        return;
    }
    // ---- bias block
    int lb = 0;
    while (lb < kLayers && rem >= (g.fo[lb] + 63) / 64) rem -= (g.fo[lb++] + 63) / 64;
    const int fi = g.fi[lb], fo = g.fo[lb], fop = g.fop[lb];
    const int o = rem * 64 + 4 * oq;
    const bool ocol = o < fo;
    if constexpr (MODE != PASS_ADAM) {
        const int T = r.T[lb], q = (T + 15) / 16, k0 = rg * q, k1 = min(T, k0 + q);
        f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
        if (ocol)
#pragma unroll 8
            for (int k = k0; k < k1; ++k) s += *reinterpret_cast<const f32x4*>(r.bpart[lb] + (size_t)k * fop + o);
        *reinterpret_cast<f32x4*>(&sS[rg][4 * oq]) = s;
        __syncthreads();
    }
    if (t < 16 && ocol) {
        const int p = g.off[lb] + fi * fo + o;
        f32x4 gr = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (MODE != PASS_ADAM) {
            gr = *reinterpret_cast<const f32x4*>(&sS[0][4 * oq]);
#pragma unroll
            for (int k = 1; k < 16; ++k) gr += *reinterpret_cast<const f32x4*>(&sS[k][4 * oq]);
        }
        if constexpr (MODE == PASS_REDUCE) {
            *reinterpret_cast<f32x4*>(r.G + p) = gr;
        } else {
            if constexpr (MODE == PASS_ADAM)
                gr = a.update ? *reinterpret_cast<const f32x4*>(a.G + p) : f32x4{0.f, 0.f, 0.f, 0.f};
            adam4(a, p, gr);
        }
    }
    if constexpr (MODE != PASS_ADAM) {
        if (lb == 0 && rem == 0 && r.loss) {  // loss: lane sums, then the lanes in order
            __syncthreads();
            float* sl = &sS[0][0];
            if (t < 64) {
                float s = 0.f;
                for (int k = t; k < r.nl; k += 64) s += r.lpart[k];
                sl[t] = s;
            }
            __syncthreads();
            if (t == 0) {
                float s = 0.f;
                for (int k = 0; k < 64; ++k) s += sl[k];
                r.loss[0] = s * r.lscale;
            }
        }
    }
}

template <int MODE>
static hipError_t launch_pass(const ReduceArgs& r, const AdamArgs& a, hipStream_t st)
{
    const LayerGeom& g = MODE == PASS_ADAM ? a.g : r.g;
    hipLaunchKernelGGL(param_pass_kernel<MODE>, dim3(pass_blocks(g)), dim3(256), 0, st, r, a);
    return hipGetLastError();
}

hipError_t launch_reduce(const ReduceArgs& r, hipStream_t st) { return launch_pass<PASS_REDUCE>(r, AdamArgs{}, st); }

hipError_t launch_reduce_adam(const ReduceArgs& r, const AdamArgs& a, hipStream_t st)
{
    return launch_pass<PASS_REDUCE_ADAM>(r, a, st);
}

hipError_t launch_adam(const AdamArgs& a, hipStream_t st) { return launch_pass<PASS_ADAM>(ReduceArgs{}, a, st); }

// ---------------------------------------------------------------------------------
__global__ void head_kernel(HeadArgs a)
{
    const int t = threadIdx.x;
    if (t >= 12 * a.nk) return;
    const int j = t / a.nk, i = t - j * a.nk;
    float m = 0.f, s = 0.f;
#pragma unroll
    for (int k = 0; k < kKnots; ++k) {
        const int d = j * kKnots + k;
        const float sd = a.ostd[d];
        m += a.R[i][k] * (a.out[d] * sd + a.omean[d]);
        s += a.R[i][k] * (a.out[72 + d] + logf(sd));
    }
    s = fminf(fmaxf(s, a.log_lo), a.log_hi);
    a.center[t] = m;
    a.sd[t] = expf(s);
}

hipError_t launch_head(const HeadArgs& a, hipStream_t st)
{
    hipLaunchKernelGGL(head_kernel, dim3(1), dim3(128), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void loss_sum_kernel(const float* __restrict__ lpart, int nl, float lscale,
                                                      float* __restrict__ loss)
{
    __shared__ float sl[64];
    const int t = threadIdx.x;
    float s = 0.f;
    for (int k = t; k < nl; k += 64) s += lpart[k];
    sl[t] = s;
    __syncthreads();
    if (t == 0) {
        float tot = 0.f;
        for (int k = 0; k < 64; ++k) tot += sl[k];
        loss[0] = tot * lscale;
    }
}

hipError_t launch_loss_sum(const float* lpart, int nl, float lscale, float* loss, hipStream_t st)
{
    hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(64), 0, st, lpart, nl, lscale, loss);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Training pairs of one closed-loop record per workgroup.  A row is usable while every
// value of it is finite and the base is above the fall height: the first row that is not
// ends the record (the smallest such index, found with an LDS minimum).  Rows before it
// give the features -- the state with the base x, y taken relative to the origin, then the
// command (v, 0, 0) -- and the targets, each joint's knots resampled to 6 with R.
__global__ __launch_bounds__(256) void pairs_kernel(PairsArgs a)
{
    __shared__ int first_bad;
    const int t = threadIdx.x, r = blockIdx.x;
    const int W = 37 + 12 * a.nk;
    const float* rec = a.rec + (size_t)r * a.steps * W;
    if (t == 0) first_bad = a.steps;
    __syncthreads();
    for (int k = t; k < a.steps; k += 256) {
        const float* row = rec + (size_t)k * W;
        bool ok = row[2] > a.fall_z;  // false for a NaN height too
        for (int c = 0; c < W; ++c) ok = ok && isfinite(row[c]);
        if (!ok) atomicMin(&first_bad, k);
    }
    __syncthreads();
    const int n = first_bad;
    if (t == 0) a.count[r] = n;
    const float ox = a.oc[3 * r], oy = a.oc[3 * r + 1], v = a.oc[3 * r + 2];
    float* feat = a.feat + (size_t)r * a.steps * 40;
    for (int e = t; e < n * 40; e += 256) {
        const int k = e / 40, c = e - k * 40;
        float x = 0.f;
        if (c < 37) x = rec[(size_t)k * W + c] - (c == 0 ? ox : c == 1 ? oy : 0.f);
        else if (c == 37) x = v;
        feat[e] = x;
    }
    float* tgt = a.tgt + (size_t)r * a.steps * 72;
    for (int e = t; e < n * 72; e += 256) {
        const int k = e / 72, d = e - k * 72, j = d / kKnots, i = d - j * kKnots;
        const float* kn = rec + (size_t)k * W + 37 + j * a.nk;
        float y = 0.f;
        for (int q = 0; q < a.nk; ++q) y += a.R[i][q] * kn[q];
        tgt[e] = y;
    }
}

hipError_t launch_pairs(const PairsArgs& a, hipStream_t st)
{
    if (a.n_rec < 1 || a.steps < 1 || a.nk < 2 || a.nk > 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL(pairs_kernel, dim3(a.n_rec), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace mlp
