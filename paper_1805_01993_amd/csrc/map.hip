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
// ANY (lengths or pointers that 16-byte packs do not divide): a file's packs begin where V's lie on whole cache lines; the first and
// the last may be parts of one, made element by element.  In the packs that the rows do align to, 5 files of 88 M bf16 values
// (1.8 GB moved) 1156 us, this way 298; 16 files of 7.9 M u32 values 380, 166.  Aligned rows keep whole packs from their own beginning: on lines
// they took 1.00 to 1.05 of the time, short ones up to 1.3 (13300 files of 336 bf16 values 8.0 -> 10.5 us).  So do, in narrow packs, calls that
// make under 64 thousand packs of 16 bytes, where a part of a pack is the longest wait (up to there 1.05 of the time, 1.26 at the worst, from
// there to 128 thousand 0.89, beyond 0.5), or under 128 thousand where rows align to 8 bytes (1.3 and 1.14, then 0.83).
template <class A, int VEC, bool KEPT, bool ANY>
__global__ __launch_bounds__(kBlock) void k_map(const typename A::elem *files,      // may be V itself
                                                const typename A::elem *__restrict__ theta,
                                                typename A::elem *V, int64_t model, uint32_t tiles,
                                                uint32_t rows, uint32_t files_per_job, uint32_t group_tiles)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t per_group = rows * group_tiles;
    const uint32_t block = xcd_contiguous(blockIdx.x, gridDim.x);
    const uint32_t group = block / per_group, in_group = block - group * per_group;
    const uint32_t row = in_group / group_tiles, tile = group * group_tiles + (in_group - row * group_tiles);
    if (tile >= tiles) return;                        // the last group may be short
    const uint32_t job = row / files_per_job;
    if constexpr (!ANY) {
        const uint32_t model_packs = (uint32_t)(model / VEC), e = tile * kBlock + threadIdx.x;
        if (e >= model_packs) return;
        const size_t at = (size_t)row * model_packs + e;
        const P data = load_pack<KEPT, P>(reinterpret_cast<const P *>(files) + at);
        const P with = reinterpret_cast<const P *>(theta)[(size_t)job * model_packs + e];
        store_stream(reinterpret_cast<P *>(V) + at, O::gradient(with, data));
    } else {
        constexpr int LINE = 128 / sizeof(E);
        const E *from = files + row * model, *with = theta + job * model;
        E *to = V + row * model;
        const int ahead = (int)(reinterpret_cast<uintptr_t>(to) / sizeof(E) % LINE);      // elements of the line before the file
        const int64_t e = ((int64_t)tile * kBlock + threadIdx.x) * VEC - ahead;
        if (e >= 0 && e + VEC <= model) {
            const P data = load_pack_any<KEPT, P, E>(from + e);
            const P at = load_pack_any<true, P, E>(with + e);
            store_stream_any<P, E>(to + e, O::gradient(at, data));
        } else if (e < model && e + VEC > 0) {
            P data, at;                               // all loads before the first store: files may be V, so they would wait for it
#pragma unroll
            for (int i = 0; i < VEC; i++) {
                const int64_t x = e + i < 0 ? 0 : e + i < model ? e + i : model - 1;
                data.v[i] = from[x];
                at.v[i] = with[x];
            }
            data = O::gradient(at, data);
#pragma unroll
            for (int i = 0; i < VEC; i++)
                if (e + i >= 0 && e + i < model) to[e + i] = data.v[i];
        }
    }
}

// rows_align: elements of the packs that all of the call's rows align to, which limit its launches whichever it takes
template <class A, int VEC, bool ANY>
int run_map(const ccdc_plan_t *p, int rows_align, const void *files, const void *theta, void *V, hipStream_t st)
{
    using E = typename A::elem;
    const uint64_t model = (uint64_t)p->Q * p->T, rows = (uint64_t)p->J * p->N;
    if (!fits_launch(model / rows_align)) return CCDC_ESIZE;
    if (!fits_launch(rows * cdiv(cdiv(model / rows_align, kBlock), kMapGroup) * kMapGroup)) return CCDC_ESIZE;
    // packs of a file with what comes before it in its first line, which is never longer than VEC * kBlock
    const uint64_t line = 128 / sizeof(E), phase = !ANY || (model % line == 0 && aligned(V, 128)) ? 0 : line - 1;
    const uint64_t tiles = cdiv(cdiv(model + phase, VEC), kBlock), groups = (tiles + kMapGroup - 1) / kMapGroup;
    const uint64_t group_tiles = (tiles + groups - 1) / groups;      // equal groups: no workgroups without work
    if (!fits_launch(rows * groups * group_tiles)) return CCDC_ESIZE;
    const bool kept = moved_bytes(p, (double)p->J * p->Q * p->T) <= kKeptStageBytes;        // files and models: what it reads
    by_reads<false>(kept, [&](auto k) {
        k_map<A, VEC, decltype(k)::value, ANY><<<(uint32_t)(rows * groups * group_tiles), kBlock, 0, st>>>(
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
    const int rows_align = vec, most = 16 / elem_bytes(plan->mode);
    const bool any = vec < most && (vec == 1 ? any_element(plan, Call::map) : makes_lanes(plan, (int64_t)plan->J * plan->N, (int64_t)plan->Q * plan->T, 4));
    hipStream_t st = (hipStream_t)stream;
    CCDC_DISPATCH(plan, vec, any, (run_map<A, VEC, ANY>(plan, rows_align, files, theta, V, st)));
}
