// Range check of the proposal network's launches on the CPU: the policy runtime's host code,
// built against the stand-in HIP runtime (tests/hostcheck/hip), is driven through the C ABI
// over registered buffers, and the launchers here check what each kernel reads and writes, as
// the kernel derives it from its arguments:
//   * every range lies in a registered buffer;
//   * what a launch writes overlaps nothing else that it reads or writes;
//   * what it reads of the workspace's intermediate results (activations, errors, partial
//     sums, BF16 copies) was written by an earlier launch of the same call, or, for the copies,
//     of any call;
//   * what an earlier launch of the call left for a later one is not written in between.
// An argument names a buffer to be registered too small, or a launch to be left out of the
// record, so that the check can be seen to fail.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "hip/hip_runtime.h"
#include "mlp_launch.h"
#include "mppi_launch.h"
#include "mppi_policy.h"
#include "proposal_launch.h"

struct Range {
    const char *b, *e;
    std::string what;
};
static std::vector<Range> g_buffers, g_made, g_kept;  // registered; written in this call; BF16 copies
static std::vector<Range> g_in, g_out;                // of the launch at hand
static std::string g_plant;
static int g_bad = 0, g_launches = 0, g_products = 0;

static void bad(const char* how, const std::string& what)
{
    std::printf("  %s: %s\n", how, what.c_str());
    ++g_bad;
}
static bool inside(const std::vector<Range>& v, const char* b, const char* e)
{
    return std::any_of(v.begin(), v.end(), [&](const Range& r) { return b >= r.b && e <= r.e; });
}
// also called by the stand-in runtime's copies and fills
bool range_check(const void* p, size_t n, const char* what)
{
    const bool ok = p && inside(g_buffers, (const char*)p, (const char*)p + n);
    if (!ok) bad("OUT OF RANGE", what);
    return ok;
}
static void reads(const void* p, size_t n, const char* what)
{
    range_check(p, n, what);
    g_in.push_back({(const char*)p, (const char*)p + n, what});
}
static void writes(const void* p, size_t n, const char* what)
{
    range_check(p, n, what);
    g_out.push_back({(const char*)p, (const char*)p + n, what});
}
static void reads_made(const void* p, size_t n, const char* what)
{
    reads(p, n, what);
    if (!inside(g_made, (const char*)p, (const char*)p + n)) bad("NOT WRITTEN BEFORE", what);
}
static void reads_kept(const void* p, size_t n, const char* what)
{
    reads(p, n, what);
    if (!inside(g_kept, (const char*)p, (const char*)p + n)) bad("NOT WRITTEN BEFORE", what);
}
// the end of a launch; updates: a kernel whose threads write only what they themselves read
static hipError_t launched(const char* name, bool updates = false)
{
    const auto meet = [](const Range& a, const Range& b) { return a.b < b.e && b.b < a.e; };
    for (size_t i = 0; i < g_out.size(); ++i) {
        for (size_t j = 0; j < i; ++j)
            if (meet(g_out[i], g_out[j])) bad("TWO WRITES OVERLAP", g_out[i].what + " / " + g_out[j].what);
        for (const Range& r : g_in)
            if (meet(g_out[i], r) && !(updates && r.b == g_out[i].b && r.e == g_out[i].e))
                bad("WRITES WHAT IT READS", g_out[i].what + " / " + r.what);
        for (const Range& m : g_made)
            if (meet(g_out[i], m)) bad("OVERWRITES AN EARLIER LAUNCH", g_out[i].what + " / " + m.what);
    }
    if (g_plant != std::string("unwritten-") + name) g_made.insert(g_made.end(), g_out.begin(), g_out.end());
    g_in.clear();
    g_out.clear();
    ++g_launches;
    return hipSuccess;
}

namespace mlp {
static const int kFi[kLayers] = {kIn, kHidden, kHidden, kHidden, kHidden};
static const int kFo[kLayers] = {kHidden, kHidden, kHidden, kHidden, kOut};
static const int kFip[kLayers] = {kInPad, kHidden, kHidden, kHidden, kHidden};
static const int kFop[kLayers] = {kHidden, kHidden, kHidden, kHidden, kOutPad};

static void rows(const float* X, const int* idx, int B, int width, const char* what)
{
    if (idx) reads(idx, 4ull * B, "row indices");
    else reads(X, 4ull * B * width, what);
    for (int r = 0; idx && r < B; ++r) range_check(X + (size_t)idx[r] * width, 4ull * width, what);
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t)
{
    const NetArgs& n = a.net;
    const int blocks = a.Bp / kNetRows;
    if (a.B < 1 || a.Bp < a.B || a.Bp % 64 || n.mode < NET_FORWARD || n.mode > NET_TRAIN) bad("SHAPE", "network");
    rows(a.X, a.idx, a.B, kIn, "input rows");
    reads(a.mean, 4 * kIn, "input mean");
    reads(a.std, 4 * kIn, "input std");
    for (int l = 0; l < kLayers; ++l) {  // the last layer's 9 column tiles of 16
        reads_kept(n.Wt[l], 2ull * kFip[l] * kFo[l], "transposed weight copy");
        reads(n.bias[l], 4ull * kFo[l], "bias");
    }
    if (n.mode == NET_FORWARD) {
        writes(n.out, 4ull * a.B * kOut, "output rows");
        return launched("network");
    }
    rows(n.loss.Y, n.loss.idx, a.B, kOut / 2, "target rows");
    reads(n.loss.omean, 4 * kOut / 2, "output mean");
    reads(n.loss.ostd, 4 * kOut / 2, "output std");
    writes(n.loss.lpart, 4ull * blocks, "loss partials");
    if (n.loss.idx != a.idx || n.loss.B != a.B || n.loss.Bp != a.Bp) bad("SHAPE", "loss");
    if (n.mode == NET_LOSS) return launched("network");
    writes(a.X0t, 2ull * a.Bp * kInPad, "input, along the batch");
    for (int l = 0; l < kLayers; ++l) {
        if (l) reads_kept(n.Wn[l], 2ull * kFip[l] * kFop[l], "weight copy");
        if (l < kLayers - 1) {
            writes(n.Ht[l], 2ull * a.Bp * kHidden, "activations, along the batch");
            writes(n.dZt[l], 2ull * a.Bp * kHidden, "errors, along the batch");
            writes(n.bpart[l], 4ull * blocks * kHidden, "column sums");
        }
    }
    writes(n.loss.dZt, 2ull * a.Bp * kOutPad, "output errors, along the batch");
    writes(n.loss.dbpart, 4ull * blocks * kOutPad, "output column sums");
    return launched("network");
}

hipError_t launch_gemm(int epi, const GemmArgs& g, int splits, hipStream_t)
{
    if (epi != EPI_SPLITK || splits < 1 || splits > kMaxSplits) bad("SHAPE", "weight gradient");
    int n = 0;
    for (const GemmArgs* p = &g; p; p = p->next, ++n) {
        if (p->M % 64 || p->N % 64 || p->K < kGemmBK || p->K % kGemmBK || p->lda != p->ldb || p->lda != p->K * splits ||
            p->ldc < p->N || (splits > 1 && p->c_split_stride < (long)p->M * p->ldc))
            bad("SHAPE", "weight gradient");
        const size_t r = (size_t)p->K * splits;
        reads_made(p->A, 2 * r * p->M, "weight gradient A");
        reads_made(p->B, 2 * r * p->N, "weight gradient B");
        for (int z = 0; z < splits; ++z)
            writes(p->C + z * p->c_split_stride, 4ull * ((size_t)(p->M - 1) * p->ldc + p->N), "weight partials");
    }
    if (n != kLayers) bad("SHAPE", "weight gradients of every layer");
    g_products += n;
    return launched("gradients");
}

static void reduce_reads(const ReduceArgs& a)
{
    for (int l = 0; l < kLayers; ++l) {
        if (a.S[l] < 1 || a.S[l] > kMaxSplits || a.g.fip[l] != kFip[l] || a.g.fop[l] != kFop[l]) bad("SHAPE", "reduction");
        const size_t plane = (size_t)kFip[l] * kFop[l];
        for (int z = 0; z < a.S[l]; ++z) reads_made(a.wpart[l] + z * plane, 4 * plane, "weight partials");
        reads_made(a.bpart[l], 4ull * a.T[l] * kFop[l], "column sums");
    }
    if (a.loss) {
        reads_made(a.lpart, 4ull * a.nl, "loss partials");
        writes(a.loss, 4, "loss");
    }
}
static void adam_accesses(const AdamArgs& a, bool gradient)
{
    const size_t n = 4ull * a.g.off[kLayers];
    reads(a.P, n, "parameters");
    if (a.update) {
        reads(a.m, n, "first moments");
        reads(a.v, n, "second moments");
        if (gradient) reads(a.G, n, "gradient");
        writes(a.P, n, "parameters");
        writes(a.m, n, "first moments");
        writes(a.v, n, "second moments");
    }
    for (int l = 0; l < kLayers; ++l) {
        const size_t w = 2ull * kFip[l] * kFop[l];
        writes(a.Wt[l], w, "transposed weight copy");
        if (l) writes(a.Wn[l], w, "weight copy");
        if (g_plant != "unwritten-copies")
            for (const __bf16* p : {a.Wt[l], a.Wn[l]})
                if (p) g_kept.push_back({(const char*)p, (const char*)p + w, "copy"});
    }
}

hipError_t launch_reduce(const ReduceArgs& a, hipStream_t)
{
    reduce_reads(a);
    writes(a.G, 4ull * a.g.off[kLayers], "gradient");
    return launched("reduction");
}
hipError_t launch_adam(const AdamArgs& a, hipStream_t)
{
    adam_accesses(a, true);
    return launched("adam", true);
}
hipError_t launch_reduce_adam(const ReduceArgs& r, const AdamArgs& a, hipStream_t)
{
    reduce_reads(r);
    adam_accesses(a, false);
    return launched("adam", true);
}
hipError_t launch_loss_sum(const float* lpart, int nl, float, float* loss, hipStream_t)
{
    reads_made(lpart, 4ull * nl, "loss partials");
    writes(loss, 4, "loss");
    return launched("loss");
}
hipError_t launch_head(const HeadArgs& a, hipStream_t)
{
    reads(a.out, 4 * kOut, "head outputs");
    reads(a.omean, 4 * kOut / 2, "head mean");
    reads(a.ostd, 4 * kOut / 2, "head std");
    writes(a.center, 48ull * a.nk, "head centre");
    writes(a.sd, 48ull * a.nk, "head std out");
    return launched("head");
}
hipError_t launch_pairs(const PairsArgs&, hipStream_t) { return hipErrorInvalidValue; }  // not driven here
}  // namespace mlp

namespace prop {
hipError_t launch_features(const float* x, const float* co, float* f, hipStream_t)
{
    reads(x, 4 * 37, "features state");
    reads(co, 4 * 5, "features command");
    writes(f, 4 * 40, "features");
    return launched("features");
}
}  // namespace prop

void capture_begin() {}
void capture_replay() {}
namespace mppi_host {
mppi_status policy_infer(mppi_policy*, const float*, const float*, int, float, float*, float*, hipStream_t);
double spline_basis_at(int, double, int, double) { return 0.0; }
}  // namespace mppi_host

static std::vector<void*> g_mem;
static void* dev(size_t n, const char* name)
{
    void* p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    std::memset(p, 0, n);
    g_mem.push_back(p);
    // the workspace ends with padding to 256 bytes
    const size_t seen = g_plant != std::string("short-") + name ? n : n - (g_plant == "short-workspace" ? 256 : 4);
    g_buffers.push_back({(char*)p, (char*)p + seen, name});
    return p;
}
static float* devf(size_t n, const char* name) { return static_cast<float*>(dev(4 * n, name)); }

static void call(const char* what, mppi_status s)
{
    if (s < 0) bad("STATUS", std::string(what) + ": " + mppi_policy_last_error(nullptr));
    g_made.clear();
}
#define CALL(x) call(#x, (x))

int main(int argc, char** argv)
{
    if (argc > 1) g_plant = argv[1];
    const int max_batch = 1024, held = 1500, N = mppi_policy_n_params();
    mppi_policy* p = nullptr;
    CALL(mppi_policy_create(nullptr, 1, max_batch, &p));
    const size_t ws = mppi_policy_workspace_bytes(p);
    CALL(mppi_policy_bind(p, dev(ws, "workspace"), ws, nullptr));
    float *G = devf(N, "gradient"), *P = devf(N, "parameters"), *L = devf(1, "loss");
    float *Xi = devf((size_t)held * 40, "indexed-input"), *Yi = devf((size_t)held * 72, "indexed-target");
    for (int B : {1, 15, 16, 17, 37, 63, 64, 65, 100, 128, 192, 256, 448, 500, 512, 1000, 1024}) {
        float *X = devf((size_t)B * 40, "input"), *Y = devf((size_t)B * 72, "target"), *out = devf((size_t)B * 144, "output");
        int* idx = static_cast<int*>(dev(4ull * B, "indices"));
        for (int r = 0; r < B; ++r) idx[r] = r ? (r * 7919) % held : held - 1;
        CALL(mppi_policy_forward(p, X, B, out));
        // the output over the input: at its start, its middle, and its last row
        CALL(mppi_policy_forward(p, out, B, out));
        CALL(mppi_policy_forward(p, out + (size_t)B * 52, B, out));
        CALL(mppi_policy_forward(p, out + (size_t)B * 104, B, out));
        CALL(mppi_policy_grad(p, X, Y, nullptr, B, G, L));
        CALL(mppi_policy_grad(p, Xi, Yi, idx, B, nullptr, nullptr));
        CALL(mppi_policy_train_step(p, X, Y, nullptr, B, 1e-3f, L));
        CALL(mppi_policy_train_step(p, Xi, Yi, idx, B, 1e-3f, nullptr));
        CALL(mppi_policy_nll(p, X, Y, nullptr, B, L));
        CALL(mppi_policy_nll(p, Xi, Yi, idx, B, L));
    }
    CALL(mppi_policy_adam(p, G, 1e-3f));
    CALL(mppi_policy_get_params(p, P));
    CALL(mppi_policy_set_params(p, P));
    for (int nk = 2; nk <= 8; ++nk) {
        float *c = devf(12 * nk, "centre"), *s = devf(12 * nk, "std");
        CALL(mppi_host::policy_infer(p, devf(37, "state"), devf(5, "command"), nk, 0.25f, c, s, nullptr));
    }
    mppi_policy_destroy(p);
    for (void* m : g_mem) std::free(m);
    std::printf("launches: %d, weight-gradient products: %d\n", g_launches, g_products);
    std::printf("faults: %d\n", g_bad);
    return g_bad ? 1 : 0;
}
