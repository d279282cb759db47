// ccdc_pipeline_fused and ccdc_node_decode_reduce for small inputs: one launch that needs no partial outputs in memory.
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace {
using namespace ccdc;

// A workgroup makes 64 packs of one segment of one node's output.  Its wavefronts share the rounds the node is in and
// the files it stores; their sums are added in LDS, in wavefront order.  For a round the wavefront reads the r packs
// of the coded packet that carries the node's segment, forms the coded pack, takes the r-1 packs the node can compute
// itself back out of it and adds what is left.  Each coded pack is so formed by its r receivers; the one that follows
// the sender in the round writes it to X.
//
// What bounds it: the chain kernel start, table entries, loads, sum, and then the instructions of the loads.  k_pipeline
// (pipeline.hip) reads every value once but keeps the outputs of all nodes in every wavefront, and where there are few
// columns it fills the chip by cutting the rounds into chunks, whose outputs a second kernel adds: that launch alone is
// 2.5 us of host time and as much on the device.  Here values are read by up to r nodes, r times as much through the
// L2s (an XCD works on neighbouring tiles, so memory is read once), and nothing is left to add.  Passes among others, this
// kernel against k_pipeline: 24 nodes, r = 1, T = 376 h32 (1.7 MB) 9.2 -> 6.1 us, 21 nodes, r = 1, T = 1112 u32 (3.9 MB) 8.1 ->
// 5.3, 7 nodes, r = 3, T = 212 f32 8.9 -> 6.1, 10 nodes, r = 2, two functions each, T = 340 f16 9.1 -> 6.1, 11 nodes, r = 2,
// T = 5536 u32 (19 MB) 10.2 -> 6.9; about 5.5 of these are the host's.  With many nodes and r >= 3 the rounds of a node are
// too many for one workgroup (17 nodes, r = 3, T = 134 u32: 11.2, 24.6 this way): see receive_prepare().
// Two stages of loads are in flight, and the list entries of the next.  One stage of 16 packs was 5 to 10 % faster
// below 4 MB and as much slower above; entries kept in the lanes and taken out with readlane cost more than scalar
// loads (1.05 of the time over 131 shapes).
constexpr int receive_steps(int regs, int r, bool multi)     // of a stage; regs: registers a pack takes
{
    const int rows = multi ? 6 : 10;                         // scalar registers: the rows of the packs
    const int packs = 20 / regs < rows ? 20 / regs : rows;
    return packs / r < 1 ? 1 : packs / r > 6 ? 6 : packs / r;
}
constexpr int receive_own(int regs) { return 16 / regs > 8 ? 8 : 16 / regs; }      // own files asked for together

// SHORT: the last segment is short or empty (W is a multiple of VEC all the same).
// CODED: the coded packs are read from X, which other nodes sent (ccdc_node_decode_reduce), not formed.
template <class A, int VEC, int R1, bool MULTI, bool SHORT, bool CODED>
__global__ __launch_bounds__(ccdc::kPipeLanes *ccdc::kReceiveMaxWaves) void k_receive(
    const typename A::elem *__restrict__ V, typename A::elem *__restrict__ X, typename A::elem *__restrict__ Phi,
    const int32_t *__restrict__ node_rows, const int64_t *__restrict__ src_off, const int64_t *__restrict__ own_rows,
    ReceiveArgs p)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    using Q = typename O::Q;
    constexpr int r = R1 - 1;
    constexpr uint32_t LANES = ccdc::kPipeLanes;
    constexpr int regs = (VEC * (int)sizeof(E) + 3) / 4;     // registers a pack takes
    constexpr int STEPS = receive_steps(regs, r, MULTI), OWN = receive_own(regs);
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t logical = xcd_contiguous(blockIdx.x, gridDim.x), outputs = (uint32_t)p.nodes * r;
    const uint32_t tile = logical / outputs, kr = logical - tile * outputs;
    const uint32_t node = (uint32_t)p.first_node + kr / r, rho = kr % r;
    const uint32_t lane = threadIdx.x % LANES, wave = wave_uniform(threadIdx.x / LANES), waves = blockDim.x / LANES;
    const uint32_t x = (tile * LANES + lane) * VEC, xb = x * (uint32_t)sizeof(E);
    Q acc = O::azero();

    // Pack x of segment seg of a row.  Past the packet's end the last pack stands in; it is not used.
    auto pack_at = [&](const E *row, uint32_t seg) {
        if constexpr (SHORT) {
            const uint32_t pos = seg * p.ell + x, last = p.W - VEC;
            return load_pack_any<true, P, E>(reinterpret_cast<const char *>(row) +
                                             lane_offset((pos < last ? pos : last) * (uint32_t)sizeof(E)));
        } else {
            return load_pack_any<true, P, E>(reinterpret_cast<const char *>(row + seg * p.ell) + lane_offset(xb));
        }
    };
    auto clip = [&](P v, uint32_t seg) {
        if constexpr (SHORT) v = O::select(seg * p.ell + x < p.W, v, O::zero());
        return v;
    };

    const uint32_t back = waves - 1 - wave;
    const uint32_t i0 = p.own * back / waves, i1 = p.own * (back + 1) / waves;
    const uint32_t j0 = p.rounds * wave / waves, j1 = p.rounds * (wave + 1) / waves;
    if (x < p.ell && (i1 > i0 || j1 > j0)) {
        const int64_t *own = own_rows + (size_t)node * p.own;
        const int32_t *mine = node_rows + (size_t)node * p.rounds;
        P first[OWN];
#pragma unroll
        for (int t = 0; t < OWN; t++) first[t] = pack_at(V + (own[i0 + t < p.own ? i0 + t : p.own - 1] >> 12), rho);

        // Rounds: a step is a round, or (MULTI) one file of it.  Two stages of steps are in flight, and the entries of the
        // list that the next one starts from.
        const uint32_t steps = MULTI ? (j1 - j0) * (uint32_t)p.m : j1 - j0;
        struct Stage {
            P w[STEPS][r];
            uint32_t packet[STEPS];
        };
        uint32_t next[STEPS], nf[STEPS], j = j0, f = 0, cf = 0;
        Q sum[r];
#pragma unroll
        for (int q = 0; q < r; q++) sum[q] = O::identity();
        auto ask = [&] {
#pragma unroll
            for (int t = 0; t < STEPS; t++) {
                next[t] = (uint32_t)mine[j < j1 ? j : j1 - 1];
                nf[t] = f;
                if constexpr (MULTI) {
                    if (++f == (uint32_t)p.m) { f = 0; j++; }
                } else {
                    j++;
                }
            }
        };
        auto load = [&](Stage &s) {
#pragma unroll
            for (int t = 0; t < STEPS; t++) {
                s.packet[t] = next[t];
                const uint32_t u = next[t] / R1, b = next[t] - u * R1, a = rho < b ? rho : rho + 1;
                const int64_t *src = src_off + (size_t)u * R1;
#pragma unroll
                for (int q = 0; q < r; q++) {
                    const uint32_t over = (uint32_t)q >= a ? 1 : 0;
                    const E *row = V + src[q + over];
                    if constexpr (MULTI) row += nf[t] * p.file_stride;
                    uint32_t seg = a - 1 + over;
                    if constexpr (CODED) {                   // in place of the pack to be decoded
                        const bool coded = q + over == b;
                        row = coded ? X + ((size_t)u * R1 + a) * p.ell : row;
                        seg = coded ? 0 : seg;
                    }
                    s.w[t][q] = pack_at(row, seg);
                }
            }
            ask();
        };
        auto use = [&](Stage &s, uint32_t left) {
#pragma unroll
            for (int t = 0; t < STEPS; t++) {
                if ((uint32_t)t >= left) break;
                P w[r];
                if constexpr (MULTI) {
#pragma unroll
                    for (int q = 0; q < r; q++) sum[q] = O::accum_file(sum[q], s.w[t][q]);
                    if (++cf < (uint32_t)p.m) continue;
                    cf = 0;
#pragma unroll
                    for (int q = 0; q < r; q++) {
                        w[q] = O::narrow(sum[q]);
                        sum[q] = O::identity();
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < r; q++) w[q] = s.w[t][q];
                }
                const uint32_t u = s.packet[t] / R1, b = s.packet[t] - u * R1, a = rho < b ? rho : rho + 1;
                const uint32_t me = b - (b > a ? 1 : 0);
                P coded = O::zero();
#pragma unroll
                for (int q = 0; q < r; q++) {
                    w[q] = clip(w[q], a - 1 + ((uint32_t)q >= a ? 1 : 0));
                    if constexpr (CODED) coded = O::select((uint32_t)q == me, s.w[t][q], coded);
                    else coded = O::code(coded, w[q]);
                }
                P d = coded;
#pragma unroll
                for (int k = 0; k < r; k++) {
                    if (me != (uint32_t)k) continue;
#pragma unroll
                    for (int q = 0; q < r; q++)
                        if (q != k) d = O::uncode(d, w[q]);
                }
                acc = O::accum(acc, d);
                if (!CODED && b == (a + 1 == R1 ? 0 : a + 1))
                    store_any<P, E>(reinterpret_cast<char *>(X + ((size_t)u * R1 + a) * p.ell) + lane_offset(xb), coded);
            }
        };
        if (steps > 0) {
            Stage even, odd;
            uint32_t left = steps;
            ask();
            load(even);
            for (;;) {
                if (left <= STEPS) {
                    use(even, left);
                    break;
                }
                load(odd);
                use(even, STEPS);
                left -= STEPS;
                if (left <= STEPS) {
                    use(odd, left);
                    break;
                }
                load(even);
                use(odd, STEPS);
                left -= STEPS;
            }
        }
#pragma unroll
        for (int t = 0; t < OWN; t++)
            if (i0 + t < i1) acc = O::accum(acc, first[t]);
        for (uint32_t i = i0 + OWN; i < i1; i += OWN) {
            P w[OWN];
#pragma unroll
            for (int t = 0; t < OWN; t++) w[t] = pack_at(V + (own[i + t < i1 ? i + t : i1 - 1] >> 12), rho);
#pragma unroll
            for (int t = 0; t < OWN; t++)
                if (i + t < i1) acc = O::accum(acc, w[t]);
        }
    }
    add_wavefronts<A, VEC>(smem, acc, waves, [&](uint32_t e, typename A::acc v) {
        const uint32_t at = tile * LANES * VEC + e, pos = rho * p.ell + at;
        if (at < p.ell && pos < p.W) Phi[(size_t)node * p.W + pos] = A::narrow(v);
    });
}

// For all nodes (node < 0) or one.  CODED: X is read.
template <class A, int VEC, int R1, bool MULTI, bool CODED>
int launch_receive(const ccdc_plan_t *p, int node, int waves, const void *V, const void *X, void *Phi, hipStream_t st)
{
    using E = typename A::elem;
    ReceiveArgs args;
    args.first_node = node < 0 ? 0 : node;
    args.nodes = node < 0 ? p->K : 1;
    args.m = p->m;
    args.W = (uint32_t)p->W;
    args.ell = (uint32_t)p->ell;
    args.rounds = (uint32_t)p->rows_per_node;
    args.own = (uint32_t)p->pipe_local_rows;
    args.file_stride = (int64_t)p->Q * p->T;
    const uint64_t groups = (uint64_t)args.nodes * p->r * cdiv((uint64_t)(p->ell / VEC), ccdc::kPipeLanes);
    if (!fits_launch(groups)) return CCDC_ESIZE;
    const int threads = ccdc::kPipeLanes * waves;
    const size_t lds = (size_t)threads * VEC * sizeof(typename A::acc);
    if (p->ell * p->r == p->W)
        k_receive<A, VEC, R1, MULTI, false, CODED><<<(uint32_t)groups, threads, lds, st>>>(
            (const E *)V, (E *)X, (E *)Phi, p->d_node_rows, p->d_src_off, p->d_loc_row, args);
    else
        k_receive<A, VEC, R1, MULTI, true, CODED><<<(uint32_t)groups, threads, lds, st>>>(
            (const E *)V, (E *)X, (E *)Phi, p->d_node_rows, p->d_src_off, p->d_loc_row, args);
    return launched();
}

template <class A, int VEC, int R1, bool CODED>
int run_files(const ccdc_plan_t *p, int node, int waves, const void *V, const void *X, void *Phi, hipStream_t st)
{
    return p->m > 1 ? launch_receive<A, VEC, R1, true, CODED>(p, node, waves, V, X, Phi, st)
                    : launch_receive<A, VEC, R1, false, CODED>(p, node, waves, V, X, Phi, st);
}

template <class A, int VEC, bool CODED>
int run_receive(const ccdc_plan_t *p, int node, int waves, const void *V, const void *X, void *Phi, hipStream_t st)
{
    switch (p->r) {
    case 1: return run_files<A, VEC, 2, CODED>(p, node, waves, V, X, Phi, st);
    case 2: return run_files<A, VEC, 3, CODED>(p, node, waves, V, X, Phi, st);
    case 3: return run_files<A, VEC, 4, CODED>(p, node, waves, V, X, Phi, st);
    case 4: return run_files<A, VEC, 5, CODED>(p, node, waves, V, X, Phi, st);
    default: return run_files<A, VEC, 6, CODED>(p, node, waves, V, X, Phi, st);
    }
}

}  // namespace

namespace ccdc {

template <class A, bool CODED>
int receive_run(const ccdc_plan_t *p, int node, int vec, int waves, const void *V, const void *X, void *Phi, hipStream_t st)
{
    if (vec == 4) return run_receive<A, 4, CODED>(p, node, waves, V, X, Phi, st);
    if (vec == 2) return run_receive<A, 2, CODED>(p, node, waves, V, X, Phi, st);
    return run_receive<A, 1, CODED>(p, node, waves, V, X, Phi, st);
}

// Compiled in five pieces, one for each algebra, the first with the entry.
#ifdef CCDC_RECEIVE_PART
#define CCDC_RECEIVE_FORM(A, CODED) \
    template int receive_run<A, CODED>(const ccdc_plan_t *, int, int, int, const void *, const void *, void *, hipStream_t)
#define CCDC_RECEIVE(A) CCDC_RECEIVE_FORM(A, false); CCDC_RECEIVE_FORM(A, true)
#define CCDC_ELSEWHERE(A) extern CCDC_RECEIVE_FORM(A, false); extern CCDC_RECEIVE_FORM(A, true)
#if CCDC_RECEIVE_PART == 0
CCDC_RECEIVE(SumF32);
CCDC_ELSEWHERE(XorU32);
CCDC_ELSEWHERE(HybF32);
CCDC_ELSEWHERE(HybBF16);
CCDC_ELSEWHERE(HybF16);
#elif CCDC_RECEIVE_PART == 1
CCDC_RECEIVE(XorU32);
#elif CCDC_RECEIVE_PART == 2
CCDC_RECEIVE(HybF32);
#elif CCDC_RECEIVE_PART == 3
CCDC_RECEIVE(HybBF16);
#else
CCDC_RECEIVE(HybF16);
#endif
#endif

#if !defined(CCDC_RECEIVE_PART) || CCDC_RECEIVE_PART == 0
// What a launch for `nodes` of the nodes is made of: generations of workgroups, the waits of a wavefront one after the other, and
// the loads that a compute unit issues.
struct Load {
    double gens, waits, issue;
    bool wide;                        // packs of 16 bytes
    double groups, group_loads;       // workgroups, and the loads of one
};
Load load_of(const ccdc_plan_t *p, int cus, int nodes, int vec, int waves)
{
    const int regs = (vec * elem_bytes(p->mode) + 3) / 4, r = p->r;
    const int64_t rounds = p->rows_per_node, own = p->pipe_local_rows;
    const double groups = (double)nodes * r * cdiv((uint64_t)(p->ell / vec), kPipeLanes), fill = std::min(1.0, groups / cus);
    const int64_t steps = (rounds + waves - 1) / waves * p->m, files = (own + waves - 1) / waves;
    const int at_once = receive_steps(regs, r, p->m > 1), own_at_once = receive_own(regs);
    const double group_loads = (double)(rounds * p->m * r + own);
    return {std::max(1.0, groups / (cus * std::max(1.0, 14.0 / waves))),
            (double)((steps + at_once - 1) / at_once + std::max<int64_t>(0, (files - 1) / own_at_once)),
            groups * group_loads / cus / fill, regs == 4, groups, group_loads};
}

int compute_units()
{
    int cus = 0, dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
        return cus;
    (void)hipGetLastError();
    return 0;
}

// The pack width and wavefronts of a workgroup of least estimated time: a start, for every generation of workgroups the waits
// of a wavefront and its own start, the loads a compute unit issues (of less than 16 bytes, of 16) and the bytes.
struct Shape {
    int vec, waves;
    double us;
};
struct Costs {
    double start, wait, load, load16, bytes_per_us;
};
Shape best_shape(const ccdc_plan_t *p, int cus, const Costs &c, double bytes)
{
    Shape best{1, 8, 1e30};
    for (int vec = 1; vec <= 4; vec *= 2) {
        if (p->W % vec != 0 || p->ell < vec) break;
        for (int waves : {2, 4, 8, 12, 16}) {
            const Load l = load_of(p, cus, p->K, vec, waves);
            const double us = c.start + l.gens * (c.wait * l.waits + 0.088 * waves) + l.issue * (l.wide ? c.load16 : c.load) +
                              bytes / c.bytes_per_us;
            if (us < best.us) best = {vec, waves, us};
        }
    }
    return best;
}

// Gives the plan this kernel where its estimated time (us) is below the one-pass kernel's, by one_pass_us, in both of two estimates, with a
// margin of a twentieth.  The first is fitted to passes of 475 shapes of the sizes below (K 4..24, r 1..5, every mode), each with the one-pass
// kernel's geometry and with 15 of this one's, and picks the pack and the wavefronts.  It knows no whole generations of workgroups: of 19140
// other plans that it favours 620 were over 3 % slower, by up to 67 %.  The second, fitted to those, counts them (16 wavefronts a
// compute unit) and the loads of the busiest unit (12 nodes, r = 2, two files, T = 1377 h32: 264 workgroups of 12 wavefronts, 12.9 us,
// 9.4 by k_pipeline); alone it let others in that are slower.  Many workgroups of two wavefronts with next to nothing to load are bound by
// their starts, which neither catches (4 nodes, r = 1, T = 50119 f32, 3136 of them, 6.6 us and 4.0).
// Of 10754 plans of 64 KB to 30 MB 5530 take this kernel, in 0.694 of the time, 80 of them over 3 % slower (worst 1.38: 9 nodes, r = 5,
// T = 124 u32 8.6 -> 11.9); by the first estimate alone 211 were.
// Above kReceiveBytes it gains little more on average (24 to 48 MB, r = 2: 0.94 with the best choice each time, r >= 3 0.98; but r = 1,
// where no value is read twice, 0.82, and 0.93 from 48 to 96 MB), though single plans just above that line would: 10 nodes, r = 3,
// T = 4096 u32 (24.4 MB) 11.4 us, by receiver 8.9.
void receive_prepare(ccdc_plan_t *p, double one_pass_us)
{
    const double bytes = moved_bytes(p, (double)p->nrows * p->ell + (double)p->Q * p->T);
    if (bytes > kKeptBytes || bytes > (p->r == 1 ? kReceiveBytesR1 : kReceiveBytes)) return;
    const int cus = compute_units();
    if (cus < 1) return;
    const Shape best = best_shape(p, cus, {4.1, 0.39, 0.0097, 0.0031, 11e6}, bytes);
    if (best.us >= 0.95 * (5.9 + (p->m > 1 ? 0.34 : 0.26) * one_pass_us + (p->pipe_chunks > 1 ? 1.1 : 0))) return;
    const Load l = load_of(p, cus, p->K, best.vec, best.waves);
    if (best.waves == 2 && l.groups >= 4 * cus && l.group_loads <= 9) return;
    const double gens = std::ceil(l.groups / (cus * (kReceiveMaxWaves / best.waves)));
    const double busiest = std::ceil(l.groups / cus) * l.group_loads;
    const double us = 3.06 + 0.305 * gens * l.waits + (l.wide ? 0.0118 : 0.0150) * busiest + bytes / 14.8e6;
    if (us >= 0.95 * (3.40 + (p->m > 1 ? 0.636 : 0.590) * one_pass_us)) return;
    p->pipe_vec = best.vec;
    p->pipe_waves = best.waves;
    p->pipe_chunks = 0;
}

// The same for ccdc_node_decode_reduce, against its other kernels: two launches where the row lists are split, a chain of rows
// each, and lanes without work where segments do not fill wavefronts.  A node's outputs are the same bits alone as with all
// nodes, so one form serves both calls, and it is this one only where it gains for both: the workgroups of one node are few, and where a
// node is in many rounds its other form spreads them over hundreds (12 nodes, r = 4, T = 1624 f32, 330 rounds: one node 9.2 us, by
// receiver 26.0; all nodes 20.6, 27.5).
// Both estimates are fitted to 16411 plans of 64 KB to 48 MB with either form forced, for one node and for all, and to 5800 more that
// kept the other.  Of 6314 other plans 2930 take this kernel: all nodes 0.565 of the time, one node 0.623; three are over 3 % slower
// for all nodes (worst 1.19: 7 nodes, r = 5, twelve files, T = 96 h32 13.8 -> 16.3), nine for one (1.18).  Chosen by all nodes
// alone, one node took up to 3.2 of its time, over 10 % more on one plan in ten; plans that are given up for that would have
// run all nodes in 0.76 of the time.  15 nodes, r = 1, T = 680 u32 9.7 -> 6.6 us, 9 nodes, r = 2, T = 8128 f16 13.1 -> 7.0, 6 nodes, r = 4, six files,
// T = 19264 f16 35.0 -> 10.2.  Above kReceiveNodeBytes, up to 500 MB, 0.86 of the time to 100 MB and 0.97 beyond, but some up to 1.46.
void receive_node_prepare(ccdc_plan_t *p)
{
    const int eb = elem_bytes(p->mode), r = p->r, cus = compute_units();
    const double bytes = moved_bytes(p, (double)p->nrows * p->ell + (double)p->Q * p->T), values = moved_bytes(p, 0);
    if (cus < 1 || bytes > kReceiveNodeBytes || values > (r == 1 ? kKeptStageBytes : (r - 1) * kKeptNodeBytes)) return;
    const int vec = eb == 4 ? (p->T % 4 == 0 ? 4 : 1) : p->T % 8 == 0 && p->ell % 8 == 0 ? 8 : p->T % 4 == 0 ? 4 : 1;
    const bool fills = fills_wavefronts((uint32_t)(p->ell / vec));
    // of the lists as they are cut for these packs (the estimates know no packs at any element, which take larger inputs on)
    const int split = (int)list_split(p->nout * ((p->W + (p->T % 4 == 0 ? 3 : 0)) / (p->T % 4 == 0 ? 4 : 1)), p->rows_per_node + p->pipe_local_rows);
    const double rounds = (double)p->rows_per_node, per_round = 1 + (r - 1.0) * p->m, own = (double)p->pipe_local_rows;
    const double longest = std::ceil((rounds + own) / split);                         // rows of a chunk
    const double chain = std::min(longest, rounds) * per_round / (fills ? 2 : 1) + std::max(0.0, longest - rounds) / 4;
    const Shape best = best_shape(p, cus, {4.05, 0.55, 0.0099, 0.0022, 19e6}, bytes);
    for (int nodes : {1, p->K}) {
        const Load l = load_of(p, cus, nodes, best.vec, best.waves);
        const double us = 3.44 + 0.277 * l.gens * l.waits + (l.wide ? 0.0109 : 0.0132) * l.issue + bytes * nodes / p->K / 30e6;
        const double rows = nodes * (rounds * per_round + own) * (double)p->W;               // elements that are read
        const double parts = split > 1 ? (double)split * nodes * r * (double)p->ell : 0;
        const double other = 3.08 + (split > 1 ? 3.31 : 0) + 1.53e-6 * parts + (fills ? 0 : 1.59e-6 * rows / vec) +
                             0.115e-6 * rows * eb + 0.194 * chain;
        if (us >= 0.85 * other) return;
    }
    p->node_vec = best.vec;
    p->node_waves = best.waves;
}

template <bool CODED>
int receive_any(const ccdc_plan_t *p, int node, int vec, int waves, const void *V, const void *X, void *Phi, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    switch (p->mode) {
    case CCDC_F32_SUM: return receive_run<SumF32, CODED>(p, node, vec, waves, V, X, Phi, st);
    case CCDC_F32_SUM_XOR: return receive_run<HybF32, CODED>(p, node, vec, waves, V, X, Phi, st);
    case CCDC_BF16_SUM_XOR: return receive_run<HybBF16, CODED>(p, node, vec, waves, V, X, Phi, st);
    case CCDC_F16_SUM_XOR: return receive_run<HybF16, CODED>(p, node, vec, waves, V, X, Phi, st);
    default: return receive_run<XorU32, CODED>(p, node, vec, waves, V, X, Phi, st);
    }
}

int receive_entry(const ccdc_plan_t *p, const void *V, void *X, void *Phi, void *stream)
{
    return receive_any<false>(p, -1, p->pipe_vec, p->pipe_waves, V, X, Phi, stream);
}

int receive_coded(const ccdc_plan_t *p, int node, const void *V, const void *X, void *Phi, void *stream)
{
    return receive_any<true>(p, node, p->node_vec, p->node_waves, V, X, Phi, stream);
}
#endif

}  // namespace ccdc
