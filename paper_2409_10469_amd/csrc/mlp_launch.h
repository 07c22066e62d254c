// Host-side launch interface of the proposal-network kernels (the pass over the network,
// weight gradients, gradient reduction, Adam, feature and head kernels).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlp {

constexpr int kLayers = 5;
constexpr int kIn = 40, kInPad = 64, kHidden = 512, kOut = 144, kOutPad = 192, kKnots = 6;
constexpr int kGemmBK = 64;  // reduction tile of the weight gradients; every K is a multiple of it
constexpr int kMaxSplits = 8;  // most batch splits of a weight-gradient product

// What a product's launch does with its sums.  The weight gradients are the one product left
// that is launched by itself; the others are steps of the pass over the network (launch_prep)
// and launch_gemm refuses them.
enum Epilogue { EPI_HIDDEN = 0, EPI_OUT = 1, EPI_DACT = 2, EPI_SPLITK = 3 };

// C[m][n] = sum_k A[m][k] B[n][k] over k in [z K, (z+1) K) for split z; A and B bf16 in
// groups of 16 columns in fragment order (batch_offset), lda = ldb columns, C + z * c_split_stride fp32 partials.  M, N, K
// multiples of 64.  The fields from bias on belong to the refused epilogues.
struct GemmArgs {
    const __bf16* A;
    const __bf16* B;
    int lda, ldb;
    int M, N, K;
    float* C;
    int ldc;
    long c_split_stride;
    const GemmArgs* next;  // a further product of the same launch, or null
    const float* bias;
    __bf16* H;
    int ldh;
    __bf16* Ht;
    int ldht;
    const float* Zp;
    int ldz;
    float* colpart;
    int m_store, n_store;
};
// the tile height of a product, or 0 on a shape error
inline int gemm_tile_m(int M, int N, int) { return M <= 0 || N <= 0 || M % 64 || N % 64 ? 0 : 64; }
// the products of the list g, g.next, ... (at most kLayers), all in `splits` splits
hipError_t launch_gemm(int epi, const GemmArgs& g, int splits, hipStream_t st);

// The Gaussian NLL of the output against standardised targets, a part of the pass over the
// network: rows idx[r] of Y (stride 72), and what it leaves (dZt only in a training step).
struct LossArgs {
    const float* out;  // not used: the output of the same pass
    const float* Y;
    const int* idx;
    int B, Bp;
    const float* omean;
    const float* ostd;
    __bf16* dZ;     // not used: stays on the chip
    __bf16* dZt;    // [192 x Bp]
    float* dbpart;  // [Bp / kNetRows][192]
    float* lpart;   // [Bp / kNetRows]
};

// A pass over the network: the raw features (rows idx[r] of X, stride 40) standardised and
// taken through every layer; then, by mode, the output rows (NET_FORWARD: B x 144), or the
// Gaussian NLL against the standardised rows of Y (NET_LOSS: a partial for each kNetRows of the
// Bp rows), or that and the backward pass up to the weight gradients (NET_TRAIN: X0, H of the
// hidden layers and dz of every layer in the order of launch_gemm's operands, and
// the column sums of dz of each kNetRows rows).
enum NetMode { NET_FORWARD = 0, NET_LOSS = 1, NET_TRAIN = 2 };
constexpr int kNetRows = 16;  // rows of a workgroup: the matrix instruction's height
struct NetArgs {
    int mode;
    const __bf16* Wt[kLayers];  // W^T [fop x fip] in fragment order
    const __bf16* Wn[kLayers];  // W [fip x fop] in fragment order (layers >= 1)
    const float* bias[kLayers];
    float* out;
    LossArgs loss;              // NET_LOSS, NET_TRAIN
    __bf16* Ht[kLayers - 1];    // [512 x Bp] of the hidden layers
    __bf16* dZt[kLayers - 1];   // [512 x Bp] of the hidden layers
    float* bpart[kLayers - 1];  // [Bp / kNetRows][512] of the hidden layers
};
struct PrepArgs {
    const float* X;
    const int* idx;
    int B, Bp;
    const float* mean;
    const float* std;
    __bf16* X0;   // not used: stays on the chip
    __bf16* X0t;  // [64 x Bp]
    NetArgs net;
};
hipError_t launch_prep(const PrepArgs& a, hipStream_t st);

struct LayerGeom {
    int off[kLayers + 1];  // flat parameter offsets (W then b per layer)
    int fi[kLayers], fo[kLayers], fip[kLayers], fop[kLayers];
};

// G = split-K and per-tile partial sums reduced in a fixed order; loss = sum(lpart) * scale
struct ReduceArgs {
    LayerGeom g;
    const float* wpart[kLayers];  // [S][fip][fop]
    const float* bpart[kLayers];  // [T][fop]
    int S[kLayers], T[kLayers];  // S <= kMaxSplits
    float* G;
    const float* lpart;
    int nl;
    float lscale;
    float* loss;
};
hipError_t launch_reduce(const ReduceArgs& a, hipStream_t st);

// Adam (update = 1) or shadow refresh only (update = 0); bf16 shadows W^T (fop x fip) and W
// (fip x fop, layers >= 1), both in fragment order, rewritten from the FP32 master weights
struct AdamArgs {
    LayerGeom g;
    float* P;
    float* m;
    float* v;
    const float* G;
    float lr, b1, b2, omb1, omb2, eps, inv_c1, inv_c2;  // omb = 1 - beta, rounded once from double
    __bf16* Wt[kLayers];
    __bf16* Wn[kLayers];
    int update;
};
hipError_t launch_adam(const AdamArgs& a, hipStream_t st);
// the reduction of launch_reduce and the update of launch_adam in one pass (G not stored)
hipError_t launch_reduce_adam(const ReduceArgs& r, const AdamArgs& a, hipStream_t st);

// network output (standardised) -> proposal centre and std for nk knots per joint
struct HeadArgs {
    const float* out;
    const float* omean;
    const float* ostd;
    int nk;
    float R[8][kKnots];  // resampling matrix, nk x 6
    float log_lo, log_hi;
    float* center;
    float* sd;
};
hipError_t launch_head(const HeadArgs& a, hipStream_t st);

// the mean loss from the loss kernel's partials, summed in the order of the parameter
// pass (lane t adds partials t, t + 64, ...; then the 64 lane sums in order), so it equals
// the loss a gradient or training step reports for the same rows
hipError_t launch_loss_sum(const float* lpart, int nl, float lscale, float* loss, hipStream_t st);

// closed-loop records -> training pairs (one workgroup per record)
struct PairsArgs {
    const float* rec;   // n_rec x steps x (37 + 12 nk): state, then the unshifted knots
    const float* oc;    // n_rec x 3: origin x, origin y, commanded forward velocity
    int n_rec, steps, nk;
    float fall_z;       // a row whose base height is not above this ends the record's pairs
    float R[kKnots][8]; // target knot i from record knot k, 6 x nk
    float* feat;        // n_rec x steps x 40
    float* tgt;         // n_rec x steps x 72
    int* count;         // n_rec: pairs of each record
};
hipError_t launch_pairs(const PairsArgs& a, hipStream_t st);

}  // namespace mlp
