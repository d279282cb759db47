// Runs every entry point of the library, compiled for the host against the HIP stand-in, on
// small shapes, under AddressSanitizer / UBSan.  Checks the outputs against the plain sum of
// eq. (1) of the paper and the coded packets of the different paths against each other.
// Usage: driver K r Q N T mode jobs [cus blocks_per_cu [geometry ...]]  (mode: 0 f32, 1 u32, 2 h32, 3 bf16, 4 f16)
// A geometry is pack,wavefronts,chunks,flags as in CCDC_Q_PIPELINE_LAUNCH: only the one-pass kernel runs then,
// as uploaded and with each geometry forced into the plan, against ccdc_combine + ccdc_encode and the plain sum.
// No chunks (0): the form for small inputs.
// "reduce a,b,c,d" says what CCDC_Q_REDUCE_LAUNCH does.  SHIM_REDUCE=waves and SHIM_NODE=pack,waves force the form of ccdc_reduce and of
// ccdc_node_decode_reduce (no wavefronts: their other kernels).
// SHIM_PLAN_ONLY=1: says what was chosen ("launch" and "reduce", a word and a value a line) and runs nothing; jobs 2 is the uncoded scheme.
// SHIM_ANY=1: no call is too small for packs at any element.  SHIM_ROUNDS=1: no chunks of node-local lists by round are too unequal.
// SHIM_PAST=1: no input is small enough to be read through the caches for its size.  "streamed C n" says that call C made
// n non-temporal loads, "workgroups node-decode n" how many the larger launch of ccdc_node_decode_reduce for all nodes has.
// Test infrastructure only.
#include <hip/hip_runtime.h>
#include <sanitizer/asan_interface.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "ccdc.h"
#include "plan.hpp"

#define CHECK(call)                                                                              \
    do {                                                                                         \
        const int rc_ = (call);                                                                  \
        if (rc_ != CCDC_OK) {                                                                    \
            std::fprintf(stderr, "%s -> %d (%s)\n", #call, rc_, ccdc_strerror(rc_));            \
            return 2;                                                                            \
        }                                                                                        \
    } while (0)

static int64_t query(const ccdc_plan_t *p, int what)
{
    int64_t v = -1;
    if (ccdc_plan_query(p, what, &v, sizeof v) != CCDC_OK) std::abort();
    return v;
}

static uint64_t mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

static float widen16(uint16_t b, bool bf)
{
    if (bf) return __uint_as_float((uint32_t)b << 16);
    _Float16 h;
    std::memcpy(&h, &b, 2);
    return (float)h;
}

// A shape whose work items fit 32 bits with four-element packs but not with one-element packs:
// ccdc_plan_bind accepts it; a call with pointers that are only 4-byte aligned falls back to
// one-element packs and must be refused with CCDC_ESIZE before anything is launched (the
// pointers given here point nowhere: a launch would be caught by the sanitizer).
static int limits()
{
    const int K = 4, r = 2, Q = 4, N = 6;
    const int64_t T = 200000000;
    ccdc_plan_t *p = nullptr;
    CHECK(ccdc_plan(K, r, Q, N, &p));
    CHECK(ccdc_plan_bind(p, T, CCDC_U32_XOR));
    CHECK(ccdc_plan_upload(p));
    const long before = shim::launches.load();
    void *a = reinterpret_cast<void *>(0x1004), *b = reinterpret_cast<void *>(0x2004), *c = reinterpret_cast<void *>(0x3004);
    int bad = 0;
    // combine and decode have one work item per pack of a W-long packet: 12 * 2e8 > 2^31 - 1
    // (the encoders have one per pack of a segment, r times fewer: those still fit)
    bad += ccdc_combine(p, a, b, nullptr) != CCDC_ESIZE;
    bad += ccdc_decode(p, a, b, c, nullptr) != CCDC_ESIZE;
    bad += shim::launches.load() != before;
    // a value length past what any pack width indexes is refused when the plan is bound
    bad += ccdc_plan_bind(p, (int64_t)1 << 38, CCDC_U32_XOR) != CCDC_ESIZE;
    ccdc_plan_destroy(p);

    // Launches that are only checked and counted.  Counts that would need tables of gigabytes are
    // written into the plan: no kernel runs.
    shim::dry_run = true;
    {   // packets of one element, padded segments of four: the packets' packs can be numbered, the segments' cannot
        CHECK(ccdc_plan(4, 3, 4, 4, &p));
        CHECK(ccdc_plan_bind(p, 1, CCDC_U32_XOR));
        CHECK(ccdc_plan_upload(p));
        const int64_t rounds = p->nround;
        p->nround = 150000000;
        const long at = shim::launches.load();
        bad += ccdc_decode(p, a, b, c, nullptr) != CCDC_OK || shim::launches.load() != at + 1;
        bad += ccdc_encode(p, b, a, nullptr) != CCDC_ESIZE;
        p->nround = rounds;
        ccdc_plan_destroy(p);
    }
    std::printf(bad ? "limits FAILED (%d)\n" : "limits ok\n", bad);
    return bad ? 1 : 0;
}

// The workspace that the plan's launches need now, exact.
static bool resize_workspace(ccdc_plan_t *p)
{
    (void)hipFree(p->d_workspace);
    p->d_workspace = nullptr;
    p->workspace_bytes = std::max(p->red_workspace_bytes, p->pipe_chunks > 1 ? (size_t)p->pipe_chunks * p->K * p->W * 4 : 0);
    return p->workspace_bytes == 0 || hipMalloc(&p->d_workspace, p->workspace_bytes) == hipSuccess;
}

// Forces the forms that SHIM_REDUCE and SHIM_NODE name.
static bool force_reductions(ccdc_plan_t *p)
{
    if (const char *text = std::getenv("SHIM_REDUCE")) {
        p->red_waves = std::atoi(text);
        if (p->red_waves < 0 || p->red_waves > (int)ccdc::kGroupMaxWaves) return false;
    }
    if (const char *text = std::getenv("SHIM_NODE")) {
        if (std::sscanf(text, "%d,%d", &p->node_vec, &p->node_waves) != 2) return false;
        const int pack = p->node_vec, waves = p->node_waves;
        if (waves != 0 && (!p->pipe_ok || (pack != 1 && pack != 2 && pack != 4) || p->W % pack != 0 || p->ell < pack || waves < 1 ||
                           waves > ccdc::kReceiveMaxWaves))
            return false;
    }
    return (!std::getenv("SHIM_REDUCE") && !std::getenv("SHIM_NODE")) || resize_workspace(p);
}

// Gives an uploaded plan another launch geometry for the one-pass kernel, with an exact-size workspace.
static bool force_geometry(ccdc_plan_t *p, const char *text)
{
    int pack, waves, chunks, flags;
    if (std::sscanf(text, "%d,%d,%d,%d", &pack, &waves, &chunks, &flags) != 4) return false;
    if (chunks == 0 && (p->W % pack != 0 || waves > ccdc::kReceiveMaxWaves)) return false;
    if ((pack != 1 && pack != 2 && pack != 4) || p->ell < pack || chunks < 0 || chunks > p->pipe_max_chunks || waves < 1 ||
        (chunks > 0 && (waves > ccdc::kPipeMaxWaves || p->K * p->r * ccdc::kPipeLanes * pack * 4 * waves > ccdc::kPipeGroupLds ||
                        p->K * p->r * ccdc::kPipeLanes * pack * 4 > ccdc::kPipeMaxLds)))
        return false;
    p->pipe_vec = pack;
    p->pipe_waves = waves;
    p->pipe_chunks = chunks;
    p->pipe_even = flags & 1;
    p->pipe_shallow = flags & 2;
    return resize_workspace(p);
}

// The workspace holds the partial sums that calls on the uploaded plan write, and no more.
static int workspace()
{
    // the last three: lists are split by no call, without and with chunks of rounds, and by both
    const int64_t shapes[][5] = {{7, 3, 7, 35, 100003}, {8, 2, 8, 28, 65536}, {10, 3, 10, 120, 4096}, {4, 1, 4, 4, 1 << 22},
                                 {15, 1, 15, 15, 680}, {12, 2, 12, 66, 5536}, {9, 5, 9, 1512, 64}};
    int bad = 0;
    shim::compute_units = 256;
    shim::blocks_per_cu = 16;
    for (const auto &s : shapes) {
        ccdc_plan_t *p = nullptr;
        CHECK(ccdc_plan((int)s[0], (int)s[1], (int)s[2], (int)s[3], &p));
        CHECK(ccdc_plan_bind(p, s[4], CCDC_F32_SUM));
        const int64_t most = query(p, CCDC_Q_WORKSPACE_BYTES);
        for (int again = 0; again < 2; again++) {
            CHECK(ccdc_plan_upload(p));
            int32_t sums[4];
            CHECK(ccdc_plan_query(p, CCDC_Q_REDUCE_LAUNCH, sums, sizeof sums));
            const int64_t phi = query(p, CCDC_Q_PHI_ELEMS) * 4;
            const int64_t red = sums[0] > 1 && (sums[1] == 0 || sums[3] == 0) ? sums[0] * phi : 0;
            const int64_t pipe = p->pipe_chunks > 1 ? p->pipe_chunks * phi : 0, got = query(p, CCDC_Q_WORKSPACE_BYTES);
            std::printf("K=%d r=%d T=%lld: %d chunks, split %d, %d and %d in one launch, workspace %lld\n", p->K, p->r, (long long)p->T,
                        p->pipe_chunks, sums[0], sums[1], sums[3], (long long)got);
            bad += got != std::max(red, pipe) || got > most;
        }
        ccdc_plan_destroy(p);
    }
    std::printf(bad ? "workspace FAILED (%d)\n" : "workspace ok\n", bad);
    return bad ? 1 : 0;
}

// The numberings of workgroups take every number below their count once; a span of 8 leaves them as they are, and with a longer
// one runs of neighbours stay on an XCD.
static int numberings()
{
    int bad = 0;
    for (uint32_t n = 1; n <= 1500; n++) {
        for (uint32_t span : {0u, 8u, 16u, 128u, 512u}) {
            std::vector<int> seen(n), xcd(n);
            for (uint32_t b = 0; b < n; b++) {
                const uint32_t w = ccdc::xcd_spans(b, n, span);
                if (w >= n || seen[w]++) return std::printf("numberings FAILED (%u of %u, %u)\n", b, n, span), 1;
                if ((span == 8 && w != b) || (span == 0 && w != ccdc::xcd_contiguous(b, n))) bad++;
                xcd[w] = b % 8;
            }
            const uint32_t run = span / 8;
            for (uint32_t i = 0; span && i + run <= n / span * span; i += run)
                for (uint32_t j = 0; j < run; j++) bad += xcd[i + j] != xcd[i];
        }
    }
    std::printf(bad ? "numberings FAILED (%d)\n" : "numberings ok\n", bad);
    return bad ? 1 : 0;
}

int main(int argc, char **argv)
{
    if (argc == 2 && std::strcmp(argv[1], "numberings") == 0) return numberings();
    if (argc == 2 && std::strcmp(argv[1], "workspace") == 0) return workspace();
    if (argc == 2 && std::strcmp(argv[1], "limits") == 0) return limits();
    if (argc < 8) return 64;
    const int K = atoi(argv[1]), r = atoi(argv[2]), Q = atoi(argv[3]), N = atoi(argv[4]);
    const int64_t T = atoll(argv[5]);
    const int mode = atoi(argv[6]), jobs = atoi(argv[7]);
    if (argc > 9) {
        shim::compute_units = atoi(argv[8]);
        shim::blocks_per_cu = atoi(argv[9]);
    }
    if (std::getenv("SHIM_PAST")) ccdc::kKeptBytes = ccdc::kKeptStageBytes = ccdc::kKeptNodeBytes = ccdc::kKeptOneNodeBytes =
                                       ccdc::kKeptPacketBytes = ccdc::kKeptSharedBytes = 0;
    if (std::getenv("SHIM_ANY")) ccdc::kAnyPacks = 1, ccdc::kAnyLanes = ccdc::kAnyListPacks = ccdc::kAnyListBytes = 0;
    if (std::getenv("SHIM_ROUNDS")) ccdc::kUnequalChunks = ccdc::kUnequalFileChunks = 1e9;
    const bool half = mode >= 3, real = mode != 1;
    const size_t eb = half ? 2 : 4;

    ccdc_plan_t *p = nullptr;
    const bool only = std::getenv("SHIM_PLAN_ONLY");
    if (jobs == 2 && !only) return 64;
    CHECK(jobs == 2 ? ccdc_plan_compression(K, r, Q, N, &p) : jobs ? ccdc_plan_jobs(K, r, Q, N, &p) : ccdc_plan(K, r, Q, N, &p));
    CHECK(ccdc_plan_bind(p, T, mode));
    CHECK(ccdc_plan_upload(p));
    if (!force_reductions(p)) {
        std::fprintf(stderr, "the form of a reduction does not fit the plan\n");
        return 3;
    }
    int32_t sums[4];
    CHECK(ccdc_plan_query(p, CCDC_Q_REDUCE_LAUNCH, sums, sizeof sums));
    std::printf("reduce %d,%d,%d,%d\n", sums[0], sums[1], sums[2], sums[3]);
    if (only) {
        int32_t launch[4] = {0, 0, 0, 0};
        (void)ccdc_plan_query(p, CCDC_Q_PIPELINE_LAUNCH, launch, sizeof launch);
        std::printf("launch %d,%d,%d,%d\n", launch[0], launch[1], launch[2], launch[3]);
        std::printf("by_round %d\n", p->node_list.empty() ? 0 : 1);
        std::printf("wide_lists %d\n", p->wide_lists ? 1 : 0);
        std::printf("any_element ");                         // with pointers that are aligned to their elements only
        using ccdc::Call;
        for (Call c : {Call::map, Call::combine, Call::encode, Call::decode, Call::reduce, Call::shuffle, Call::node_encode, Call::node_decode})
            std::printf("%d", ccdc::any_element(p, c) ? 1 : 0);
        std::printf("%d%d\n", ccdc::any_element(p, Call::node_encode, 0) ? 1 : 0, ccdc::any_element(p, Call::node_decode, 0) ? 1 : 0);
        ccdc_plan_destroy(p);
        return 0;
    }
    std::printf("lists by round %d\n", p->node_list.empty() ? 0 : 1);
    const int64_t nv = query(p, CCDC_Q_V_ELEMS), nvb = query(p, CCDC_Q_VBAR_ELEMS), nx = query(p, CCDC_Q_X_ELEMS),
                  nd = query(p, CCDC_Q_D_ELEMS), nphi = query(p, CCDC_Q_PHI_ELEMS), J = query(p, CCDC_Q_J);

    // exact-size heap blocks: any access outside them is reported by the sanitizer
    auto dev = [&](int64_t n) { return static_cast<unsigned char *>(std::malloc((size_t)n * eb)); };
    unsigned char *V = dev(nv), *Vbar = dev(nvb), *X = dev(nx), *D = dev(nd), *Phi = dev(nphi);
    unsigned char *X2 = dev(nx), *D2 = dev(nd), *Phi2 = dev(nphi), *X3 = dev(nx), *Phi3 = dev(nphi), *X4 = dev(nx),
                  *Phi4 = dev(nphi), *X5 = dev(nx), *Phi5 = dev(nphi);
    for (int64_t i = 0; i < nv; i++) {
        const uint64_t h = mix(0x9E3779B97F4A7C15ull * (uint64_t)(i + 1));
        if (half) {
            // small integers in the format: exact in every summation order
            const int v = (int)(h % 7) - 3;
            uint16_t b;
            if (mode == 3) {
                b = (uint16_t)(__float_as_uint((float)v) >> 16);
            } else {
                const _Float16 hh = (_Float16)(float)v;
                std::memcpy(&b, &hh, 2);
            }
            std::memcpy(V + i * 2, &b, 2);
        } else if (real) {
            const float v = (float)((int)(h % 2001) - 1000);        // integers: exact sums in fp32
            std::memcpy(V + i * 4, &v, 4);
        } else {
            const uint32_t v = (uint32_t)(h >> 32);
            std::memcpy(V + i * 4, &v, 4);
        }
    }
    // eq. (1): Phi[j][q][t] = sum over the N files of V[j][n][q][t]
    std::vector<double> want_r(real ? nphi : 0);
    std::vector<uint32_t> want_x(real ? 0 : nphi);
    for (int64_t j = 0; j < J; j++)
        for (int64_t n = 0; n < N; n++)
            for (int64_t q = 0; q < Q; q++)
                for (int64_t t = 0; t < T; t++) {
                    const int64_t src = ((j * N + n) * Q + q) * T + t, dst = (j * Q + q) * T + t;
                    if (half) {
                        uint16_t b;
                        std::memcpy(&b, V + src * 2, 2);
                        want_r[dst] += widen16(b, mode == 3);
                    } else if (real) {
                        float v;
                        std::memcpy(&v, V + src * 4, 4);
                        want_r[dst] += v;
                    } else {
                        uint32_t v;
                        std::memcpy(&v, V + src * 4, 4);
                        want_x[dst] ^= v;
                    }
                }
    int bad = 0;
    auto check_phi = [&](const unsigned char *got, const char *name) {
        for (int64_t i = 0; i < nphi; i++) {
            bool ok;
            if (half) {
                uint16_t b;
                std::memcpy(&b, got + i * 2, 2);
                const double g = widen16(b, mode == 3), w = want_r[i];
                ok = std::fabs(g - w) <= std::fabs(w) * (mode == 3 ? 1.0 / 256 : 1.0 / 2048) + 1e-9;
            } else if (real) {
                float g;
                std::memcpy(&g, got + i * 4, 4);
                ok = (double)g == want_r[i];
            } else {
                uint32_t g;
                std::memcpy(&g, got + i * 4, 4);
                ok = g == want_x[i];
            }
            if (!ok) {
                if (bad < 5) std::fprintf(stderr, "%s: output %lld differs from the plain sum\n", name, (long long)i);
                bad++;
            }
        }
    };
    auto same = [&](const unsigned char *a, const unsigned char *b, int64_t n, const char *name) {
        if (std::memcmp(a, b, (size_t)n * eb) != 0) {
            std::fprintf(stderr, "%s differs\n", name);
            bad++;
        }
    };

    auto streamed = [&](const char *name) { std::printf("streamed %s %ld\n", name, shim::streaming_loads.exchange(0)); };

    // SHIM_ONLY_PIPELINE=1: only the one-pass pipeline, checked against the plain sum (for shapes
    // at which the staged kernels, one emulated thread per work item, would take too long)
    if (std::getenv("SHIM_ONLY_PIPELINE")) {
        CHECK(ccdc_pipeline_fused(p, V, X3, Phi3, nullptr));
        check_phi(Phi3, "pipeline Phi");
        ccdc_plan_destroy(p);
        for (unsigned char *q : {V, Vbar, X, D, Phi, X2, D2, Phi2, X3, Phi3, X4, Phi4, X5, Phi5}) std::free(q);
        std::printf("K=%d r=%d Q=%d N=%d T=%lld mode=%d: pipeline only, %ld launches, %d mismatches\n", K, r, Q, N,
                    (long long)T, mode, shim::launches.load(), bad);
        std::fflush(stdout);
        return bad ? 1 : 0;
    }
    CHECK(ccdc_combine(p, V, Vbar, nullptr));
    streamed("combine");
    CHECK(ccdc_encode(p, Vbar, X, nullptr));
    const bool only_pipeline = argc > 10;
    if (!only_pipeline) {
        CHECK(ccdc_decode(p, X, Vbar, D, nullptr));
        shim::streaming_loads = 0;
        CHECK(ccdc_reduce(p, V, D, Phi, nullptr));
        streamed("reduce");
        check_phi(Phi, "staged Phi");
        same(D, Vbar, nd, "decoded packets vs pre-combined packets");

        CHECK(ccdc_shuffle_fused(p, V, X2, D2, nullptr));
        streamed("shuffle");
        CHECK(ccdc_reduce(p, V, D2, Phi2, nullptr));
        same(X2, X, nx, "fused X");
        same(D2, D, nd, "fused D");
        check_phi(Phi2, "fused Phi");
    }

    shim::streaming_loads = 0;
    const int rc = ccdc_pipeline_fused(p, V, X3, Phi3, nullptr);
    if (rc == CCDC_OK) streamed("pipeline");
    if (rc == CCDC_OK) {
        same(X3, X, nx, "pipeline X");
        check_phi(Phi3, "pipeline Phi");
        CHECK(ccdc_pipeline_fused_noalloc(p, V, X4, Phi4, nullptr));
        same(X4, X, nx, "no-alloc pipeline X");
        same(Phi4, Phi3, nphi, "no-alloc pipeline Phi");
    } else if (rc != CCDC_ESIZE) {
        std::fprintf(stderr, "ccdc_pipeline_fused -> %d\n", rc);
        return 2;
    }

    if (rc == CCDC_OK) {
        int32_t launch[4];
        CHECK(ccdc_plan_query(p, CCDC_Q_PIPELINE_LAUNCH, launch, sizeof launch));
        std::printf("launch %d,%d,%d,%d\n", launch[0], launch[1], launch[2], launch[3]);
    }
    for (int i = 10; i < argc; i++) {
        if (!force_geometry(p, argv[i])) {
            std::fprintf(stderr, "geometry %s does not fit the plan\n", argv[i]);
            return 3;
        }
        std::memset(X3, 0xA5, (size_t)nx * eb);
        std::memset(Phi3, 0xA5, (size_t)nphi * eb);
        shim::streaming_loads = 0;
        CHECK(ccdc_pipeline_fused(p, V, X3, Phi3, nullptr));
        streamed(argv[i]);
        same(X3, X, nx, argv[i]);
        check_phi(Phi3, argv[i]);
        CHECK(ccdc_pipeline_fused_noalloc(p, V, X4, Phi4, nullptr));
        same(X4, X, nx, argv[i]);
        same(Phi4, Phi3, nphi, argv[i]);
    }

    if (!only_pipeline) {
        shim::streaming_loads = 0;
        CHECK(ccdc_node_encode(p, -1, V, X5, nullptr));
        streamed("node-encode");
        shim::largest_launch = 0;
        CHECK(ccdc_node_decode_reduce(p, -1, V, X5, Phi5, nullptr));
        streamed("node-decode");
        std::printf("workgroups node-decode %ld\n", shim::largest_launch.load());
        same(X5, X, nx, "node-local X");
        check_phi(Phi5, "node-local Phi");
        // each node on its own: the same packets, and the outputs of the call for all of them.  Out of its reach (reported by the
        // sanitizer) are the files it does not store, the packets that it neither sends nor is sent, and other nodes' outputs.
        auto only = [&](unsigned char *buf, int64_t rows, int64_t row, auto mine) {      // rows of `row` elements
            for (int64_t i = 0; i < rows; i++)
                if (!mine(i)) __asan_poison_memory_region(buf + (size_t)(i * row) * eb, (size_t)row * eb);
        };
        auto all = [&](unsigned char *buf, int64_t n) { __asan_unpoison_memory_region(buf, (size_t)n * eb); };
        const int r1 = r + 1;
        auto stores = [&](int k) {
            return [&, k](int64_t file) {
                const int32_t *held = p->node_files.data() + k * p->files_per_node;
                return std::binary_search(held, held + p->files_per_node, (int32_t)file);
            };
        };
        auto sends = [&](int k) { return [&, k](int64_t i) { return p->round_member[i] == k; }; };
        auto is_sent = [&](int k) {
            return [&, k](int64_t i) {
                const int32_t *in = p->round_member.data() + i / r1 * r1;
                return in[i % r1] != k && std::find(in, in + r1, k) != in + r1;
            };
        };
        std::memset(X5, 0xA5, (size_t)nx * eb);
        for (int k = 0; k < K; k++) {
            only(V, J * N, Q * T, stores(k)), only(X5, p->nrows, p->ell, sends(k));
            CHECK(ccdc_node_encode(p, k, V, X5, nullptr));
            all(V, nv), all(X5, nx);
        }
        streamed("one-node-encode");
        same(X5, X, nx, "one node's X");
        std::memset(Phi4, 0xA5, (size_t)nphi * eb);
        for (int k = 0; k < K; k++) {
            only(V, J * N, Q * T, stores(k)), only(X5, p->nrows, p->ell, is_sent(k));
            only(Phi4, J * K, p->W, [&](int64_t o) { return o % K == k; });
            CHECK(ccdc_node_decode_reduce(p, k, V, X5, Phi4, nullptr));
            all(V, nv), all(X5, nx), all(Phi4, nphi);
        }
        streamed("one-node-decode");
        same(Phi4, Phi5, nphi, "one node's Phi");
    }

    // Map stand-in: out = theta - files (XOR in the field), separate buffer and in place
    if (!only_pipeline) {
        unsigned char *theta = dev(nphi), *out = dev(nv), *inpl = dev(nv);
        for (int64_t i = 0; i < nphi; i++) std::memcpy(theta + i * eb, V + ((i * 7) % nv) * eb, eb);   // any valid patterns
        std::memcpy(inpl, V, (size_t)nv * eb);
        shim::streaming_loads = 0;
        CHECK(ccdc_map(p, V, theta, out, nullptr));
        streamed("map");
        CHECK(ccdc_map(p, inpl, theta, inpl, nullptr));
        same(inpl, out, nv, "map in place");
        for (int64_t j = 0; j < J; j++)
            for (int64_t n = 0; n < N; n++)
                for (int64_t e = 0; e < (int64_t)Q * T; e++) {
                    const int64_t at = (j * N + n) * Q * T + e, th = j * Q * T + e;
                    bool ok;
                    if (half) {
                        uint16_t a, b, g;
                        std::memcpy(&a, theta + th * 2, 2);
                        std::memcpy(&b, V + at * 2, 2);
                        std::memcpy(&g, out + at * 2, 2);
                        ok = widen16(g, mode == 3) == widen16(a, mode == 3) - widen16(b, mode == 3);   // small integers: exact
                    } else if (real) {
                        float a, b, g;
                        std::memcpy(&a, theta + th * 4, 4);
                        std::memcpy(&b, V + at * 4, 4);
                        std::memcpy(&g, out + at * 4, 4);
                        ok = g == a - b;
                    } else {
                        uint32_t a, b, g;
                        std::memcpy(&a, theta + th * 4, 4);
                        std::memcpy(&b, V + at * 4, 4);
                        std::memcpy(&g, out + at * 4, 4);
                        ok = g == (a ^ b);
                    }
                    if (!ok && bad++ < 5) std::fprintf(stderr, "map: element %lld is wrong\n", (long long)at);
                }
        for (unsigned char *q : {theta, out, inpl}) std::free(q);
    }

    ccdc_plan_destroy(p);
    for (unsigned char *q : {V, Vbar, X, D, Phi, X2, D2, Phi2, X3, Phi3, X4, Phi4, X5, Phi5}) std::free(q);
    std::printf("K=%d r=%d Q=%d N=%d T=%lld mode=%d jobs=%d: %ld launches, pipeline %s, %d mismatches\n", K, r, Q, N,
                (long long)T, mode, jobs, shim::launches.load(), rc == CCDC_OK ? "ran" : "refused (size)", bad);
    return bad ? 1 : 0;
}
