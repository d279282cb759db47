// A stand-in for the Map phase (Sec. III): every file w_n of a job is mapped into the Q
// intermediate values v_{q,n} = g_q(w_n).  The paper leaves g_q free; the stand-in is the
// gradient step its motivation (distributed gradient descent, Sec. I) is about, for the
// quadratic model whose minimiser is the mean of the data: a file is a data vector of Q*T
// numbers, the job has a model theta of Q*T numbers, and
//     v_{q,n}[t] = d/dtheta (1/2 |theta - w_n|^2) at chunk q  =  theta[q][t] - w_n[q][t]
// (XOR in the field F_{2^T}).  Summed over the files by the shuffle path, the outputs are
// the chunks of the full gradient N*theta - sum_n w_n.  One streaming pass: a work item
// makes one pack of V from one pack of a file and one pack of theta (which every file of
// the job re-reads, so it stays in cache).
#include "common.hpp"

namespace {
using namespace ccdc;

// A workgroup covers kBlock consecutive packs (a tile) of ONE file (row), so that the file
// and job indices are wave-uniform and no work item divides.  Workgroups are ordered
// (group of at most kMapGroup tiles, file, tile in the group): the piece of theta a group covers
// (1 MiB) is used by every file before the next piece is touched, so it is fetched from
// HBM once and re-read from cache, while every file is still read in runs of up to 1 MiB.  Groups are
// of equal size, so that a small model leaves no workgroups without work: 2380 files of 14824 u32
// values (15 tiles; 256 a group before) with the pipeline after it 191 -> 108 us.  Each XCD walks a
// contiguous range of that order, so a piece of theta lives in one L2 and every XCD reads and writes long
// runs of its own: bound by memory, 28 files of 12.8 M f32 values (2.9 GB moved) 513 us with the tiles dealt to
// the XCDs in turn (480 with groups of 64), 461 this way (6.3 TB/s); 28 files of 25.6 M bf16 values 510, 463.  Four files a work
// item were 2 % faster on 28 files of 25.6 M bf16 values and up to 8 % slower elsewhere.
constexpr uint32_t kMapGroup = 256;
// A file's packs begin where V's lie on whole cache lines, whatever its length; the first and the last pack of a file may be
// parts of one, made element by element.  In one-element packs, which lengths that four does not divide took before, 5 files of
// 88 M bf16 values (1.8 GB moved) 1156 us, this way 298; 16 files of 7.9 M u32 values 380, 166.
template <class A, bool KEPT>
__global__ __launch_bounds__(kBlock) void k_map(const typename A::elem *files,      // may be V itself
                                                const typename A::elem *__restrict__ theta,
                                                typename A::elem *V, int64_t model, uint32_t tiles,
                                                uint32_t rows, uint32_t files_per_job, uint32_t group_tiles)
{
    using E = typename A::elem;
    constexpr int VEC = 16 / sizeof(E), LINE = 128 / sizeof(E);
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t per_group = rows * group_tiles;
    const uint32_t block = xcd_contiguous(blockIdx.x, gridDim.x);
    const uint32_t group = block / per_group, in_group = block - group * per_group;
    const uint32_t row = in_group / group_tiles, tile = group * group_tiles + (in_group - row * group_tiles);
    if (tile >= tiles) return;                        // the last group may be short
    const uint32_t job = row / files_per_job;
    const E *from = files + row * model, *with = theta + job * model;
    E *to = V + row * model;
    const int ahead = (int)(reinterpret_cast<uintptr_t>(to) / sizeof(E) % LINE);      // elements of the line before the file
    const int64_t e = ((int64_t)tile * kBlock + threadIdx.x) * VEC - ahead;
    if (e >= 0 && e + VEC <= model) {
        const P data = load_pack_any<KEPT, P, E>(from + e);
        const P at = load_pack_any<true, P, E>(with + e);
        store_stream_any<P, E>(to + e, O::gradient(at, data));
    } else {
#pragma unroll
        for (int i = 0; i < VEC; i++)
            if (e + i >= 0 && e + i < model) to[e + i] = A::gradient(with[e + i], from[e + i]);
    }
}

template <class A>
int run_map(const ccdc_plan_t *p, int vec, const void *files, const void *theta, void *V, hipStream_t st)
{
    using E = typename A::elem;
    constexpr uint64_t VEC = 16 / sizeof(E), LINE = 128 / sizeof(E);
    const uint64_t model = (uint64_t)p->Q * p->T, rows = (uint64_t)p->J * p->N;
    const uint64_t limit = cdiv(cdiv(model, vec), kBlock);            // launches of the packs that all of the call's rows align to
    if (!fits_launch(model / vec) || !fits_launch(rows * cdiv(limit, kMapGroup) * kMapGroup)) return CCDC_ESIZE;
    // packs of a file with what comes before it in its first line, which is never longer than VEC * kBlock
    const uint64_t phase = model % LINE == 0 && aligned(V, 128) ? 0 : LINE - 1;
    const uint64_t tiles = cdiv(cdiv(model + phase, VEC), kBlock), groups = (tiles + kMapGroup - 1) / kMapGroup;
    const uint64_t group_tiles = (tiles + groups - 1) / groups;      // equal groups: no workgroups without work
    if (!fits_launch(rows * groups * group_tiles)) return CCDC_ESIZE;
    const bool kept = moved_bytes(p, (double)p->J * p->Q * p->T) <= kKeptStageBytes;        // files and models: what it reads
    by_reads<false>(kept, [&](auto k) {
        k_map<A, decltype(k)::value><<<(uint32_t)(rows * groups * group_tiles), kBlock, 0, st>>>(
            (const E *)files, (const E *)theta, (E *)V, (int64_t)model, (uint32_t)tiles, (uint32_t)rows,
            (uint32_t)p->N, (uint32_t)group_tiles);
    });
    return launched();
}

}  // namespace

extern "C" int ccdc_map(const ccdc_plan_t *plan, const void *files, const void *theta, void *V, void *stream)
{
    int rc = ready(plan), vec = 1;
    if (rc != CCDC_OK) return rc;
    if ((rc = pick_vec(plan, &vec, files, theta, (const void *)V)) != CCDC_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    switch (plan->mode) {
    case CCDC_F32_SUM: return run_map<SumF32>(plan, vec, files, theta, V, st);
    case CCDC_F32_SUM_XOR: return run_map<HybF32>(plan, vec, files, theta, V, st);
    case CCDC_BF16_SUM_XOR: return run_map<HybBF16>(plan, vec, files, theta, V, st);
    case CCDC_F16_SUM_XOR: return run_map<HybF16>(plan, vec, files, theta, V, st);
    default: return run_map<XorU32>(plan, vec, files, theta, V, st);
    }
}
