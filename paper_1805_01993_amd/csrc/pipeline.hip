// One-pass pipeline kernel (combine + encode + decode + reduce) and its entry point.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"

namespace {
using namespace ccdc;

// ------------------------------------------------- whole path in one pass
// combine + encode + decode + reduce for a single-job plan.  A workgroup is up to
// eight wavefronts on one tile of columns (lane = in-segment pack x); each walks
// its share of the rounds and of the files that nodes store themselves.
// For a round it reads the r packs of each of the r+1 packets that sit at
// x (every needed element of V once), forms each sender's coded pack (written
// to X), decodes it for each receiver exactly as k_decode does, and adds the
// decoded pack to the receiver's running output.  Those running outputs (K nodes
// x r segments per lane) live in LDS, one private slot per lane of every wavefront:
// no atomics, one barrier at the end, and since only the owning lane touches a slot
// the summation order is program order.  (LDS float atomics were measured several
// times slower than this read-add-write of the round's slots.)
// The wavefronts' outputs are added in wavefront order; with more than one chunk
// the per-chunk outputs go to the workspace and k_reduce_final adds
// them in its fixed order.  Running outputs and chunk outputs are sums in the making
// (the algebra's acc type); they are narrowed to elements once, when Phi is written.
//
// What bounds it: bytes on large inputs (the 8-node gradient shape, 4.04 GB of
// traffic, runs at 5.4 TB/s); waiting on small ones and on large K*r, where LDS
// capacity, not registers, bounds how many wavefronts fit on a compute unit.  So
// the loads of the next PF steps are kept in flight in registers while a round is
// decoded.  A step is a round, or (MULTI: a batch has m > 1 files) one file of it:
// the packs of the m files are added up as they arrive.  Walking the files step
// by step in the same pipeline took the 8-node shape with 10 files a batch
// (h32, T = 25000) from 236 to 93 us; the kernel before read a round, waited, and
// went on.
// Packs are loaded and stored at element alignment, so any value length runs with
// wide packs (7 nodes, r = 3, f32, T = 100003: 38.4 us with one-element packs, 29.3 with four).
template <class A, int VEC, int R1, bool MULTI>
constexpr int prefetch_depth()
{
    constexpr int packs = R1 * (R1 - 1);
    constexpr int regs = packs * ((VEC * (int)sizeof(typename A::elem) + 3) / 4);
    constexpr int by_regs = (MULTI ? 80 : 120) / regs;       // registers a lane spends on rounds in flight
    constexpr int by_cnt = 56 / (packs + R1);                // the counter of outstanding loads and stores has 6 bits
    constexpr int most = R1 == 2 ? 6 : 4;
    constexpr int d = by_regs < by_cnt ? by_regs : by_cnt;
    return d < 1 ? 1 : (d > most ? most : d);
}

// With r = 1 and several files a batch, a packet long enough to make wavefronts of 16-byte packs for
// all of the chip runs faster with ONE step in flight: every wavefront then stays close to the same row
// of V, where deeper prefetch lets them drift apart and read from many rows at once.  Nine nodes, two
// functions each, four files a batch, T = 313700 f32 (1.0 GB): 220 us with six steps in flight, 205 with
// one; 11 nodes, two files, T = 892808 (1.3 GB): 278, 256; six nodes, two files, T = 2671248: 250, 208;
// two or three steps in flight are no better than six.  With shorter packets, or so many nodes that LDS
// holds fewer than eight wavefronts a compute unit, there is too little on the way with one step (23
// nodes, two functions, two files, T = 119076: 317 and 416 us).
template <class A, int VEC, int R1, bool MULTI>
constexpr bool can_be_shallow()
{
    return MULTI && R1 == 2 && VEC * sizeof(typename A::elem) == 16;
}
[[maybe_unused]] constexpr int64_t kLongPacket = 1200 * 1024;               // bytes: 1200 tiles of columns

// How a packet's last segment ends, at a given pack width.
enum Tail {
    kWhole = 0,                       // r segments of ell elements, whole packs everywhere
    kShort = 1,                       // the last segment is short or empty, but a pack is either in it or past its end
    kSplit = 2,                       // some pack would straddle the end of the packet
};

// Which (chunk, tile) pair a workgroup works on: the span of xcd_spans(), see order_of().
enum Order : uint32_t {
    kContiguous = 0,                  // each XCD on a contiguous range of pairs
    kInTurn = 8,                      // neighbouring tiles on different XCDs, as workgroups are handed out
    kRuns = 128,                      // the XCDs on runs of 16 neighbouring tiles in turn
};

}  // namespace

namespace ccdc {
struct PipeArgs {
    int K, m;
    uint32_t W, ell;                  // elements of a packet and of a segment
    uint32_t R, n_loc;
    uint32_t tiles, chunks, waves;
    bool even;                        // how the work is shared out, see walk()
    bool shallow;                     // one step in flight, see long_packets()
    uint32_t order;                   // of the workgroups: an Order
    uint32_t cols;                    // packs the wide columns cover (kSplit: the rest is the last tile's)
    int64_t file_stride, chunk_stride;
};
}  // namespace ccdc

namespace {

// One wavefront's share of the pass on one tile of columns: lane = VEC elements
// from in-segment position x on, rounds and own files of the wavefront's range.
template <class A, int VEC, int R1, bool MULTI, bool SHORT, bool KEPT>
__device__ __forceinline__ void walk(const typename A::elem *__restrict__ V, typename A::elem *__restrict__ X,
                                     typename A::elem *__restrict__ Phi, typename A::acc *__restrict__ part,
                                     const int64_t *__restrict__ rows, const int64_t *__restrict__ own,
                                     const PipeArgs &p, unsigned char *smem, uint32_t chunk, uint32_t wave,
                                     uint32_t lane, uint32_t x, bool active)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    using Q = typename O::Q;
    constexpr int r = R1 - 1;
    constexpr int LANES = ccdc::kPipeLanes;
    constexpr int PF = prefetch_depth<A, VEC, R1, MULTI>();
    constexpr int PFL = PF * R1;                     // own-file rows in flight (r packs each)
    const int K = p.K, slots = K * r;
    Q *all = reinterpret_cast<Q *>(smem) + lane;     // slot i of wavefront g, this lane: all[(g * slots + i) * LANES]
    Q *acc = all + (size_t)wave * slots * LANES;

    if (active) {
        bool valid[r];                // does segment rho reach position x (short / empty tail)
        uint32_t offb[r];             // byte offset of pack x of segment rho inside a packet
#pragma unroll
        for (int rho = 0; rho < r; rho++) {
            const uint32_t pos = rho * p.ell + x;
            valid[rho] = !SHORT || pos < p.W;
            offb[rho] = (valid[rho] ? pos : p.W - VEC) * (uint32_t)sizeof(E);
        }
        const uint32_t xb = x * (uint32_t)sizeof(E);
        auto pack_at = [](const E *row, uint32_t byte_off) -> P {
            return load_pack_any<KEPT, P, E>(reinterpret_cast<const char *>(row) + byte_off);
        };
        for (int i = 0; i < slots; i++) acc[i * LANES] = O::azero();

        struct Row {                  // a round's table entries (wave-uniform): (element offset << 12) | node
            int64_t e[R1];
        };
        struct Stage {
            P w[R1][r];               // w[b][rho]: pack x of segment rho of packet b (of one file of its batch)
            int slot[R1];             // first slot of the node packet b is for
        };
        auto fetch = [&](uint32_t u) {
            Row t;
#pragma unroll
            for (int b = 0; b < R1; b++) t.e[b] = rows[(size_t)u * R1 + b];
            return t;
        };
        auto issue = [&](const Row &t, int f, Stage &s) {
            uint32_t at[r];
#pragma unroll
            for (int rho = 0; rho < r; rho++) at[rho] = lane_offset(offb[rho]);
#pragma unroll
            for (int b = 0; b < R1; b++) {
                const E *row = V + (t.e[b] >> 12);
                if constexpr (MULTI) row += f * p.file_stride;
                s.slot[b] = (int)(t.e[b] & 4095) * r;
#pragma unroll
                for (int rho = 0; rho < r; rho++) s.w[b][rho] = pack_at(row, at[rho]);
            }
        };
        // Decode one round and add the r(r+1) decoded packs to their owners' outputs.
        // The slots of a round are distinct (receiver b, segment rank(a,b)), so they are
        // read ahead of the writes: all of them where registers allow (one LDS wait a round).
        auto finish = [&](uint32_t u, const P (&w)[R1][r], const int (&slot)[R1]) {
            constexpr int AHEAD = R1 * r * VEC <= 64 ? R1 : 2;       // senders whose slots are held at a time
            Q cur[AHEAD][R1];         // cur[a % AHEAD][b]: running output that sender a's pack for b goes to
            auto read = [&](int a) {
#pragma unroll
                for (int b = 0; b < R1; b++)
                    if (b != a) cur[a % AHEAD][b] = acc[(slot[b] + a - (a > b ? 1 : 0)) * LANES];
            };
#pragma unroll
            for (int a = 0; a + 1 < AHEAD; a++) read(a);
#pragma unroll
            for (int a = 0; a < R1; a++) {
                if (a + AHEAD - 1 < R1) read(a + AHEAD - 1);
                P coded = O::zero();
#pragma unroll
                for (int b = 0; b < R1; b++)
                    if (b != a) coded = O::code(coded, w[b][a - (a > b ? 1 : 0)]);
                store_stream_any<P, E>(reinterpret_cast<char *>(X + ((size_t)u * R1 + a) * p.ell) + lane_offset(xb), coded);
#pragma unroll
                for (int b = 0; b < R1; b++) {
                    if (b == a) continue;
                    P d = coded;
#pragma unroll
                    for (int b2 = 0; b2 < R1; b2++)
                        if (b2 != a && b2 != b) d = O::uncode(d, w[b2][a - (a > b2 ? 1 : 0)]);
                    // a slot past a short segment collects zeros and is never written out
                    acc[(slot[b] + a - (a > b ? 1 : 0)) * LANES] = O::accum(cur[a % AHEAD][b], d);
                }
            }
        };
        auto clip = [&](P v, int rho) -> P {
            if constexpr (SHORT) v = O::select(valid[rho], v, O::zero());
            return v;
        };

        // This wavefront's rounds [u0, u1) and own rows [i0, i1): the j-th of n equal shares of
        // each (even), or of the list of rounds (m files of r+1 rows each) followed by the own
        // rows, so that a wavefront with little to do mostly has one kind and one wait for it.
        const uint32_t j = chunk * p.waves + wave, n = p.chunks * p.waves;
        uint32_t u0, u1, i0, i1;
        if (p.even) {
            u0 = (uint32_t)((uint64_t)p.R * j / n);
            u1 = (uint32_t)((uint64_t)p.R * (j + 1) / n);
            i0 = (uint32_t)((uint64_t)p.n_loc * j / n);
            i1 = (uint32_t)((uint64_t)p.n_loc * (j + 1) / n);
        } else {
            const uint64_t per_round = (uint64_t)R1 * (uint32_t)p.m, in_rounds = per_round * p.R;
            const uint64_t total = in_rounds + p.n_loc;
            const uint64_t lo = total * j / n, hi = total * (j + 1) / n;
            u0 = lo < in_rounds ? (uint32_t)(lo / per_round) : p.R;
            u1 = hi < in_rounds ? (uint32_t)(hi / per_round) : p.R;
            i0 = lo < in_rounds ? 0 : (uint32_t)(lo - in_rounds);
            i1 = hi < in_rounds ? 0 : (uint32_t)(hi - in_rounds);
        }

        // Rounds: a step is one file of a round's batches (MULTI) or the whole round.
        // PF steps are in flight; the main loop has no condition on what to load.
        if (u1 > u0) {
            const uint32_t steps = MULTI ? (u1 - u0) * (uint32_t)p.m : u1 - u0;
            Stage st[PF];
            uint32_t iu = u0, cu = u0;               // round and file of the next step to load / to use
            int jf = 0, cf = 0;
            Q sum[MULTI ? R1 : 1][r];
            if constexpr (MULTI) {
#pragma unroll
                for (int b = 0; b < R1; b++)
#pragma unroll
                    for (int rho = 0; rho < r; rho++) sum[b][rho] = O::identity();
            }
            auto load = [&](const Row &t, Stage &s) {
                issue(t, jf, s);
                if constexpr (MULTI) {
                    if (++jf == p.m) { jf = 0; iu++; }
                } else {
                    iu++;
                }
            };
            auto use = [&](Stage &s) {
                if constexpr (MULTI) {
#pragma unroll
                    for (int b = 0; b < R1; b++)
#pragma unroll
                        for (int rho = 0; rho < r; rho++) sum[b][rho] = O::accum_file(sum[b][rho], s.w[b][rho]);
                    if (++cf == p.m) {
                        P w[R1][r];
#pragma unroll
                        for (int b = 0; b < R1; b++)
#pragma unroll
                            for (int rho = 0; rho < r; rho++) {
                                w[b][rho] = clip(O::narrow(sum[b][rho]), rho);
                                sum[b][rho] = O::identity();
                            }
                        finish(cu, w, s.slot);
                        cf = 0;
                        cu++;
                    }
                } else {
                    if constexpr (SHORT) {
#pragma unroll
                        for (int b = 0; b < R1; b++)
#pragma unroll
                            for (int rho = 0; rho < r; rho++) s.w[b][rho] = clip(s.w[b][rho], rho);
                    }
                    finish(cu, s.w, s.slot);
                    cu++;
                }
            };
            // The table row of a load is asked for a turn ahead, behind the loads of the turn before:
            // it arrives while those of the stage in hand are waited for.  (One row more than there
            // are rounds may be asked for; the table has it.)
            Row ahead;
            auto turn = [&](Stage &s) {
                use(s);
                load(ahead, s);
                ahead = fetch(iu);
            };
            // The compiler waits for a stage by counting the loads and stores issued after it,
            // and counts the least that any way into the code may have issued: the first turn
            // is taken out of the loop (no X store lies between its loads), and short ranges
            // fill the stages on a way of their own.
            uint32_t i = 0;
            bool shallow = false;
            if constexpr (can_be_shallow<A, VEC, R1, MULTI>()) shallow = p.shallow;
            if (shallow) {
                load(fetch(iu), st[0]);
                ahead = fetch(iu);
                for (; i + 1 < steps; i++) turn(st[0]);
                use(st[0]);
                i = steps;
            } else if (steps >= 3 * PF) {
#pragma unroll
                for (int s = 0; s < PF; s++) {
                    load(fetch(iu), st[s]);
                }
                ahead = fetch(iu);
#pragma unroll
                for (int s = 0; s < PF; s++) turn(st[s]);
                for (i = PF; i + 2 * PF <= steps; i += PF) {
#pragma unroll
                    for (int s = 0; s < PF; s++) turn(st[s]);
                }
            } else {
#pragma unroll
                for (int s = 0; s < PF; s++)
                    if ((uint32_t)s < steps) load(fetch(iu), st[s]);
            }
            for (; i < steps; i += PF) {
#pragma unroll
                for (int s = 0; s < PF; s++)
                    if (i + s < steps) {
                        use(st[s]);
                        if (i + s + PF < steps) load(fetch(iu), st[s]);
                    }
            }
        }

        // the files each node stores itself; table entries as above
        if (i1 > i0) {
            struct Own {
                P w[r];
                int slot;
            };
            auto load = [&](int64_t e, Own &s) {
                s.slot = (int)(e & 4095) * r;
                const E *row = V + (e >> 12);
#pragma unroll
                for (int rho = 0; rho < r; rho++) s.w[rho] = pack_at(row, lane_offset(offb[rho]));
            };
            auto use = [&](const Own &s) {
                Q cur[r];
#pragma unroll
                for (int rho = 0; rho < r; rho++) cur[rho] = acc[(s.slot + rho) * LANES];
#pragma unroll
                for (int rho = 0; rho < r; rho++) acc[(s.slot + rho) * LANES] = O::accum(cur[rho], clip(s.w[rho], rho));
            };
            Own ow[PFL];
            uint32_t i = i0;
            if (i1 - i0 >= 2 * PFL) {
#pragma unroll
                for (int s = 0; s < PFL; s++) load(own[i0 + s], ow[s]);
                for (; i + 2 * PFL <= i1; i += PFL) {
                    int64_t e[PFL];
#pragma unroll
                    for (int s = 0; s < PFL; s++) e[s] = own[i + s + PFL];
#pragma unroll
                    for (int s = 0; s < PFL; s++) {
                        use(ow[s]);
                        load(e[s], ow[s]);
                    }
                }
            } else {
#pragma unroll
                for (int s = 0; s < PFL; s++)
                    if (i0 + s < i1) load(own[i0 + s], ow[s]);
            }
            for (; i < i1; i += PFL) {
#pragma unroll
                for (int s = 0; s < PFL; s++)
                    if (i + s < i1) {
                        use(ow[s]);
                        if (i + s + PFL < i1) load(own[i + s + PFL], ow[s]);
                    }
            }
        }
    }

    // the outputs of the workgroup's wavefronts are added in wavefront order and written, the
    // only chunk's straight to Phi, else to the chunk's slice of the workspace
    if (p.waves > 1) __syncthreads();
    if (!active) return;
    typename A::acc *dst = part + (int64_t)chunk * p.chunk_stride;
    for (uint32_t i = wave; i < (uint32_t)slots; i += p.waves) {
        const uint32_t k = i / r, pos = (i - k * r) * p.ell + x;
        if (SHORT && pos >= p.W) continue;
        Q v = all[i * LANES];
        for (uint32_t g = 1; g < p.waves; g++) v = O::add(v, all[((size_t)g * slots + i) * LANES]);
        const int64_t at = (int64_t)k * p.W + pos;               // element index in [K][W]
        if (p.chunks == 1) store_any<P, E>(Phi + at, O::narrow(v));
        else store_any<Q, typename A::acc>(dst + at, v);
    }
}

template <class A, int VEC, int R1, bool MULTI, int TAIL, bool KEPT>
__global__ __launch_bounds__(ccdc::kPipeLanes *ccdc::kPipeMaxWaves) void k_pipeline(
    const typename A::elem *__restrict__ V, typename A::elem *__restrict__ X, typename A::elem *__restrict__ Phi,
    typename A::acc *__restrict__ part, const int64_t *__restrict__ rows, const int64_t *__restrict__ own, PipeArgs p)
{
    constexpr uint32_t LANES = ccdc::kPipeLanes;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t logical = xcd_spans(blockIdx.x, gridDim.x, p.order);
    const uint32_t tile = logical % p.tiles, chunk = logical / p.tiles;
    const uint32_t lane = threadIdx.x % LANES, wave = wave_uniform(threadIdx.x / LANES);
    if constexpr (TAIL == kSplit) {
        if (tile + 1 == p.tiles) {                   // what the wide columns leave: a few elements of every segment
            const uint32_t x = p.cols * VEC + lane;
            walk<A, 1, R1, MULTI, true, KEPT>(V, X, Phi, part, rows, own, p, smem, chunk, wave, lane, x, x < p.ell);
            return;
        }
    }
    const uint32_t c = tile * LANES + lane;
    walk<A, VEC, R1, MULTI, TAIL == kShort, KEPT>(V, X, Phi, part, rows, own, p, smem, chunk, wave, lane, c * VEC, c < p.cols);
}

}  // namespace

namespace ccdc {
// Every k_pipeline<A, VEC, R1, *, *, *> has this signature.
template <class A>
using PipeKernel = void (*)(const typename A::elem *, typename A::elem *, typename A::elem *, typename A::acc *,
                            const int64_t *, const int64_t *, PipeArgs);
}  // namespace ccdc

namespace {

template <int VEC>
Tail tail_kind(const ccdc_plan_t *p)
{
    if (p->ell * p->r == p->W) return kWhole;
    return p->W % VEC == 0 ? kShort : kSplit;       // ell is a multiple of 4 then
}

// Packs of a segment that the wide columns cover.  kSplit: those that every segment has whole; at
// most 4r + 2 elements are left (r*ell - W <= 4r - 1; when the last segment is empty ell itself is
// below 4r), which one wavefront of one-element packs covers.
template <int VEC>
uint32_t pipeline_cols(const ccdc_plan_t *p)
{
    if (tail_kind<VEC>(p) != kSplit) return (uint32_t)(p->ell / VEC);
    const int64_t last = p->W - (p->r - 1) * p->ell;
    return last > 0 ? (uint32_t)(last / VEC) : 0;
}

template <int VEC>
uint32_t pipeline_tiles(const ccdc_plan_t *p)
{
    return cdiv(pipeline_cols<VEC>(p), ccdc::kPipeLanes) + (tail_kind<VEC>(p) == kSplit ? 1 : 0);
}

// Whether rows of V or segments begin inside a sector (16-byte packs) or a cache line (narrower ones): two neighbouring
// tiles then both want what lies across their border.
template <class A, int VEC>
bool shares_lines(const ccdc_plan_t *p)
{
    constexpr int64_t eb = sizeof(typename A::elem), unit = VEC * eb >= 16 ? 32 : 128;
    return p->W * eb % unit != 0 || p->ell * eb % unit != 0;
}

// Whether the kernel reads V with ordinary loads (KEPT) or past the caches.  Ordinary ones where a pass is small
// (kKeptBytes), and where tiles share lines, which non-temporal loads fetch from memory for each: with packs of less than
// 16 bytes on inputs of any size, with wider ones, which cross the borders in fewer places, from kKeptWideBytes on.  Below
// that, wide packs share what they need in the L2 of an XCD that works on neighbouring tiles (order_of) and read past the
// caches up to 8 % faster; 63 shapes of 0.13 to 1.2 GB with one chunk take 0.94 of the time of such reads in the hardware's
// order, ordinary ones 0.96, 42 shapes with chunks 1.00 and 1.02 (six nodes, r = 5, T = 1841604 f32 in the hardware's order
// 64 us, so 60, kept 69; five nodes, r = 4, T = 3000004 75, 70, 79; six nodes, r = 3, ten files a batch, T = 125001 h32
// 117, 117, 123).  With r <= 2 and up to kKeptSharedBytes the cache still holds enough: 13 shapes of 128 to 200 MB past the
// caches 1.04 of the time of ordinary loads (18 nodes, r = 1, T = 51921 f32 29.1, 24.0; 24 nodes, r = 2, T = 3373 u32 46.0,
// 39.5), 15 shapes of 200 to 300 MB 0.98; with r >= 3 nothing was lost there.  Larger inputs are read faster through the caches, by 2 to 3 % on average and up to 8 (five nodes, r = 2,
// T = 6485985 f32, 1.8 GB, 428, 392, 367; eight nodes, r = 1, T = 5811425, 3.0 GB, 728, 734, 674); why is not known.
// Narrow packs, past the caches -> kept: 8 nodes, r = 2, T = 800008 bf16 134 -> 110 us; 16 nodes, r = 3, T = 6148 bf16
// 49.0 -> 45.0, T = 4096 f32 53.3 -> 50.9; 8 nodes, T = 800064 bf16, segments half a line off, 107.5 -> 103; in chunks with
// ten and more files a batch 0.90 to 1.07 of the time (12 nodes, r = 3, T = 2817 bf16 0.90, 8 nodes, r = 3, T = 20928 u32
// 1.07).  On whole lines ordinary loads are slower, T = 800000, f32 190 -> 199, bf16 98 -> 103.
template <class A, int VEC>
bool reads_kept(const ccdc_plan_t *p)
{
    const double bytes = moved_bytes(p, (double)p->nrows * p->ell + (double)p->Q * p->T);
    if (bytes <= kKeptBytes) return true;
    if (!shares_lines<A, VEC>(p)) return false;
    return VEC * sizeof(typename A::elem) < 16 || bytes >= kKeptWideBytes || (p->r <= 2 && bytes <= kKeptSharedBytes);
}

// The instantiation a plan runs.  Null for an r the kernel is not unrolled for, and where it would spill.
template <class A, int VEC, bool KEPT>
PipeKernel<A> kernel_of(const ccdc_plan_t *p)
{
    const Tail tail = tail_kind<VEC>(p);
    auto of = [&](auto r1) -> PipeKernel<A> {
        constexpr int R1 = decltype(r1)::value;
        // Narrow packs go past the caches where W and ell are whole lines.  r * ell exceeds W by less than 4r elements, that
        // is by less than a line, so then not at all: there are no other ends.
        constexpr bool ALL_ENDS = KEPT || VEC * sizeof(typename A::elem) >= 16;
        if (!ALL_ENDS && tail != kWhole) return nullptr;
        if (p->m > 1) {
            // Five segments of six packets, their sums and the file on the way do not fit the registers at four
            // elements a pack: those kernels spilled up to 112 of them.  Narrower packs were faster in 19 of 20
            // shapes measured (eight nodes, four files a batch, T = 60000 f32: 101 us at the best geometry of
            // four-element packs, 82 with two, 73 with one), the twentieth 4 % slower.
            if constexpr (VEC == 4 && R1 == 6) return nullptr;
            else if constexpr (VEC == 1 || !ALL_ENDS) return k_pipeline<A, VEC, R1, true, kShort, KEPT>;
            else return tail == kSplit ? k_pipeline<A, VEC, R1, true, kSplit, KEPT> : k_pipeline<A, VEC, R1, true, kShort, KEPT>;
        }
        if constexpr (VEC > 1 && ALL_ENDS) {
            if (tail == kSplit) return k_pipeline<A, VEC, R1, false, kSplit, KEPT>;
        }
        if constexpr (ALL_ENDS) {
            if (tail == kShort) return k_pipeline<A, VEC, R1, false, kShort, KEPT>;
        }
        return k_pipeline<A, VEC, R1, false, kWhole, KEPT>;
    };
    switch (p->r + 1) {
    case 2: return of(std::integral_constant<int, 2>());
    case 3: return of(std::integral_constant<int, 3>());
    case 4: return of(std::integral_constant<int, 4>());
    case 5: return of(std::integral_constant<int, 5>());
    case 6: return of(std::integral_constant<int, 6>());
    default: return nullptr;
    }
}

}  // namespace

namespace ccdc {

// The kernels that keep their reads, as kernel_of<A, VEC, true>; compiled in pieces of their own.
template <class A>
PipeKernel<A> pipeline_kernel_kept(const ccdc_plan_t *p, int vec)
{
    if (vec == 4) return kernel_of<A, 4, true>(p);
    if (vec == 2) return kernel_of<A, 2, true>(p);
    return kernel_of<A, 1, true>(p);
}

}  // namespace ccdc

#if !defined(CCDC_PIPELINE_PART) || CCDC_PIPELINE_PART < 5
namespace {

// When the rounds are cut into chunks, each XCD gets a contiguous range of (chunk, tile) pairs: the tiles of one
// chunk (adjacent pieces of the same rows, the same table entries) then run next to each other in time behind one
// L2.  The same with a single chunk where adjacent tiles share lines (8 nodes, r = 2, T = 800008 bf16 in the hardware's
// order 122 us, this way 112; f32 216, 212) or the input is small (0.93 of the time over 11 shapes that share lines, 0.995
// over 23 that do not).  With r = 1 and one file a batch some plans run a fifth slower that way,
// as if the XCDs' eight windows of each row got in each other's way (six nodes, T = 4746660 f32 in the hardware's order
// 334 us, contiguous ranges 410; seven nodes, T = 2080360 174, 203): there the XCDs take runs of 16 tiles in turn, all in
// the same window (308, 172; nine nodes, T = 3043714 477, 444, runs 449).  With r > 1 no such plan was found, and ranges
// are the better order (seven nodes, r = 3, T = 1815201 u32 536, 467, runs 536).  Else the hardware's order is kept: all
// XCDs then sweep the same window of every row together (2 to 3 % better).
template <class A, int VEC>
Order order_of(const ccdc_plan_t *p)
{
    if (p->pipe_chunks > 1) return kContiguous;
    if (!reads_kept<A, VEC>(p) && !shares_lines<A, VEC>(p)) return kInTurn;
    return p->r == 1 && p->m == 1 ? kRuns : kContiguous;
}

template <class A, int VEC>
PipeKernel<A> pipeline_kernel(const ccdc_plan_t *p)
{
    return reads_kept<A, VEC>(p) ? pipeline_kernel_kept<A>(p, VEC) : kernel_of<A, VEC, false>(p);
}

template <class A, int VEC, bool MULTI>
int pipeline_depth(int r)
{
    switch (r) {
    case 1: return prefetch_depth<A, VEC, 2, MULTI>();
    case 2: return prefetch_depth<A, VEC, 3, MULTI>();
    case 3: return prefetch_depth<A, VEC, 4, MULTI>();
    case 4: return prefetch_depth<A, VEC, 5, MULTI>();
    default: return prefetch_depth<A, VEC, 6, MULTI>();
    }
}

template <int VEC>
size_t pipeline_lds(const ccdc_plan_t *p)           // one wavefront's running outputs
{
    return (size_t)p->K * p->r * ccdc::kPipeLanes * VEC * sizeof(float);     // every algebra sums in 4 bytes
}

// Whether four-element packs of this plan run with one step in flight (see kLongPacket).
bool long_packets(const ccdc_plan_t *p)
{
    return p->r == 1 && p->m > 1 && elem_bytes(p->mode) == 4 && p->W * 4 >= kLongPacket &&
           8 * pipeline_lds<4>(p) <= (size_t)ccdc::kCuLds;
}

// The launch geometry of a plan: pack width, wavefronts of a workgroup (they share a tile of columns
// and add their outputs in LDS, so they cost no workspace traffic), chunks of rounds (they fill the
// chip where tiles are few, at the price of a second kernel and of writing and reading a copy of all
// outputs per chunk).  No single threshold on sizes separates the good from the bad: the candidates are
// ranked by an estimate of their time and the least is taken.  Its constants are fitted to measured
// passes of several hundred shapes (K 4..24, r 1..5, 64 KB..3.2 GB, every mode, 25 to 200 geometries
// each): they rank; as a time the estimate is up to twice the measured one.  Three sets of them, because
// what ranks the candidates differs between small inputs (waits, the second kernel, lanes in flight) and
// large ones (the loads a compute unit can issue, bytes, full generations).  With the first set alone 31
// of 143 shapes with one file a batch, r >= 3 and 200 MB or more ran 3 to 34 % slower than one wavefront a
// workgroup and at most N/8 chunks, the geometry before either set; with the second 12 do, by at most
// 10 %, and on average they take 0.97 of the time (11 nodes, r = 4, T = 138064 u32: 545 -> 478 us; 22 nodes,
// r = 4, T = 344 h32: 101 -> 77).  It also serves r = 5 with several files, where four-element packs are
// missing (0.94 of the time over 20 shapes), and r = 1 with several files and long packets (see kLongPacket).  Elsewhere it gave nothing: with r <= 2 1.00 of the time over
// 72 shapes, three of them 9 to 18 % slower; below 200 MB 1.00; with several files and r = 4 up to 20 % slower.
// The third set is for what the second leaves of r >= 3 where a compute unit's LDS holds fewer than 16 wavefronts even with
// one-element packs (four a SIMD: over 40 running outputs a lane); fitted with reads kept or not and with workgroups of up to
// 160 KB of LDS.  Against the first set's choice: 334 shapes below 200 MB 0.90 of the time, four of them over 3 % slower,
// the slowest 8 % (16 nodes, r = 4, T = 257 bf16, six files a batch 60 -> 34 us; 16 nodes, r = 3, T = 4096 f32 49 -> 46; 13
// nodes, r = 4, T = 688 h32 13.5 -> 14.0); 300 shapes with several files and 200 MB or more 0.92, five over 3 % slower, the
// slowest 10 %.  Where LDS holds 16 and more it gave 0.98 over 61 shapes, 11 of them over 3 % slower, up to 26 %; with r <= 2
// 0.98, some over 20 % slower.
struct Candidate {
    int vec, waves, chunks;
    bool even, shallow;
    double us;
};

constexpr double kLargeInput = 200e6;              // bytes a pass moves

template <class A, int VEC>
void consider(const ccdc_plan_t *p, Candidate *best)
{
    constexpr int elem = (int)sizeof(typename A::elem);
    PipeKernel<A> kernel = pipeline_kernel<A, VEC>(p);
    const size_t lds = pipeline_lds<VEC>(p);
    const bool narrowest = VEC == 1;
    if (!kernel || lds > (size_t)ccdc::kPipeMaxLds || (!narrowest && p->ell < VEC)) return;
    int limit = 0, cus = 0, dev = 0;                 // wavefronts a compute unit holds as far as registers go
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&limit, kernel, ccdc::kPipeLanes, 0) != hipSuccess || limit < 1 ||
        cus < 1) {
        (void)hipGetLastError();
        limit = cus = 1;
    }
    const double r1 = p->r + 1, R = (double)p->nround, m = p->m, own = (double)p->K * p->pipe_local_rows;
    const double rows = R * r1 * m + own;            // rows of r packs a tile reads
    const double tiles = pipeline_tiles<VEC>(p), bytes =
        ((double)p->N * p->Q * p->T + (double)p->nrows * p->ell + (double)p->Q * p->T) * elem;
    const bool longp = bytes >= kLargeInput && long_packets(p), shallow = can_be_shallow<A, VEC, 2, true>() && longp;
    const bool large = bytes >= kLargeInput && (p->m == 1 ? p->r >= 3 : p->r == 5 || longp);
    const int depth = p->m > 1 ? pipeline_depth<A, VEC, true>(p->r) : pipeline_depth<A, VEC, false>(p->r);
    const double used = (double)(p->ell / VEC) / (cdiv(p->ell / VEC, ccdc::kPipeLanes) * ccdc::kPipeLanes);    // share of lanes with work
    const double flight = (shallow ? 1 : depth) * r1 * p->r * ccdc::kPipeLanes * VEC * elem * used;                // bytes a wavefront has on the way
    constexpr int width = VEC * elem >= 16 ? 3 : VEC * elem == 8 ? 2 : VEC * elem == 4 ? 1 : 0;
    const bool deep = !large && p->r >= 3 && ccdc::kCuLds / pipeline_lds<1>(p) < 16;       // the third set of constants
    constexpr double peaks[4][4] = {                 // B/us
        {3.2e6, 4.2e6, 5.3e6, 6.5e6}, {4.2e6, 4.8e6, 6.2e6, 9.0e6},
        {3.6e6, 4.0e6, 5.65e6, 13.8e6}, {3.3e6, 5.85e6, 8.45e6, 23.7e6}};                // deep: past the caches, through them
    double peak = peaks[large ? 1 : !deep ? 0 : reads_kept<A, VEC>(p) ? 3 : 2][width];
    // Lanes without work cost the third set little while the last-level cache holds the input, and much beyond: a last tile that
    // is nearly empty then shares its lines with a neighbour that has long gone on (24 nodes, r = 3, eight files a batch, T =
    // 448 bf16 as two tiles of two-element packs, 64 and 12 lanes, 205 us, as three of one element 141; 22 nodes, r = 4, six
    // files, T = 576 f16 535, 306).  Over 241 shapes of 16 bits 0.92 -> 0.91 of the first set's time, 11 -> 5 of them over 3 %
    // slower, the slowest 53 -> 10 %; over 59 of 32 bits 0.95 -> 0.94, the slowest 12 -> 1 %.
    peak *= large ? used : std::pow(used, !deep ? 0.3 : bytes >= kLargeInput ? 3 : 0.25);
    if (p->T * elem % 8)                             // rows start anywhere: more lines an access
        peak *= 1 - (deep ? 0.2 : !large ? 0.4 : width == 0 ? 0.45 : 0.25) * std::min(1.0, 8.0 / (VEC * elem));
    // A workgroup may take most of a compute unit's LDS where the third set ranks, and with r = 2 on large inputs that have
    // fewer tiles than there are compute units: larger workgroups then save chunks.  Over 138 shapes 0.95 of the time with 64
    // KB, the slowest 9 % slower (18 nodes, two functions each, T = 45440 f16 150 -> 133 us); with a tile for every compute
    // unit they only gave some 0.96, others up to 1.16 (13 nodes, T = 502358 bf16 289 -> 336; eight nodes, T = 2068872 bf16
    // 280 -> 302).  Elsewhere 64 KB stay the limit: with r = 1 (22 nodes, T = 240608 bf16 89 -> 106), on small inputs (9
    // nodes, r = 2, T = 21340 f32 12.0 -> 16.1) and where the second set ranks (9 nodes, r = 5, T = 697096 bf16 322 -> 441).
    const bool few_tiles = p->r == 2 && bytes >= kLargeInput && tiles < cus;
    const size_t most_lds = deep || few_tiles ? ccdc::kPipeGroupLds : ccdc::kPipeMaxLds;
    const double issue = tiles * (rows * p->r + R * r1) * 0.012 / cus;       // us a compute unit takes to issue the loads and stores
    for (int waves = 1; waves <= ccdc::kPipeMaxWaves && waves * lds <= most_lds; waves++) {
        const size_t granule = large || deep ? ccdc::kLdsGranule : 1, group_lds = (waves * lds + granule - 1) / granule * granule;
        const int by_lds = (int)(ccdc::kCuLds / group_lds), by_regs = limit / waves;
        const int per_cu = std::max(1, std::min(by_lds, by_regs));
        const double room = (double)cus * per_cu * waves;                            // wavefronts in flight at most
        int64_t last = 0;
        for (int part = 8; part >= 0; part = part > 1 ? part / 2 : part - 1) {        // 1/8 .. 1 of what fills the chip, and 1 chunk
            int64_t chunks = part ? (int64_t)((double)cus * per_cu / (part * tiles)) : 1;
            chunks = std::max<int64_t>(1, std::min<int64_t>(chunks, p->pipe_max_chunks));
            if (chunks == last) continue;
            last = chunks;
            const double shares = (double)chunks * waves, per = R / shares;
            // equal shares of rounds and own rows: 2 % faster on large inputs, 3 % slower on small ones
            Candidate c{VEC, waves, (int)chunks, shares == 1 || per >= (large ? 2 : 32), shallow, 0};
            const double w = tiles * shares, fill = w / room, gens = std::max(1.0, fill);
            // rounds (and rounds' worth of own rows) the busiest wavefront walks
            const double steps = c.even ? std::ceil(per) * m + own / shares / r1 : std::ceil(rows / shares / (r1 * m)) * m;
            const double uneven = steps / (rows / r1 / shares), full = gens / std::ceil(gens);    // how full the generations are
            const double slots = gens * p->K * p->r * 4 * VEC, outputs = 2.0 * chunks * p->K * p->W * 4;
            const double latency = deep ? 0.7 : !large ? 0.8 : longp ? 0.1 : 0.2;      // us
            const double rate = std::pow(full, deep ? 1.8 : 0.5) / (latency / (std::min(w, room) * flight) + 1 / peak);
            if (large) {
                const double stream = bytes / rate * std::pow(uneven, 0.36);
                const double chain = 2.2 * gens * (steps / depth + 1);                // waits one after the other
                c.us = std::max({stream, chain, issue}) + 0.018 * slots;
                if (chunks > 1) c.us += 2 + outputs / 4.6e6;
            } else if (deep) {
                const double stream = bytes / rate * std::pow(uneven, 0.25);
                const double chain = 0.83 * gens * (steps / depth + 0.8);
                c.us = std::pow(std::pow(stream, 1.44) + std::pow(chain, 1.44), 1 / 1.44) + 0.053 * slots;
                c.us += 0.42 * (double)group_lds / 65536 * std::ceil(gens);           // slots to clear and add up, a group after the other
                if (chunks > 1) c.us += 3.8 + outputs / 1.34e6;
            } else {
                const double stream = bytes / rate * std::pow(uneven, 0.08);
                const double chain = 0.8 * gens * (steps / depth + 1);
                c.us = std::sqrt(stream * stream + chain * chain) + 0.007 * slots;
                if (chunks > 1) c.us += 4 + outputs / 1.8e6;
            }
            if (best->vec == 0 || c.us < best->us) *best = c;
        }
    }
}

// One launch of the pass with `chunks` round chunks; partial outputs of the
// chunks go to `part` (chunks * K * W sums) and k_reduce_final adds them.
template <class A, int VEC>
int run_pipeline(const ccdc_plan_t *p, const void *V, void *X, void *Phi, void *part, bool wide_final, hipStream_t st)
{
    using E = typename A::elem;
    using Acc = typename A::acc;
    PipeKernel<A> kernel = pipeline_kernel<A, VEC>(p);
    if (!kernel) return CCDC_ESIZE;
    const int chunks = p->pipe_chunks;
    const uint32_t tiles = pipeline_tiles<VEC>(p);
    if (!fits_launch((uint64_t)tiles * (uint64_t)chunks) || !fits_launch((uint64_t)p->K * (uint64_t)p->W)) return CCDC_ESIZE;
    PipeArgs args;
    args.K = p->K;
    args.m = p->m;
    args.W = (uint32_t)p->W;
    args.ell = (uint32_t)p->ell;
    args.R = (uint32_t)p->nround;
    args.n_loc = (uint32_t)(p->K * p->pipe_local_rows);
    args.tiles = tiles;
    args.chunks = (uint32_t)chunks;
    args.waves = (uint32_t)p->pipe_waves;
    args.even = p->pipe_even;
    args.shallow = p->pipe_shallow;
    args.order = order_of<A, VEC>(p);
    args.cols = pipeline_cols<VEC>(p);
    args.file_stride = (int64_t)p->Q * p->T;
    args.chunk_stride = (int64_t)p->K * p->W;
    kernel<<<tiles * (uint32_t)chunks, ccdc::kPipeLanes * p->pipe_waves, pipeline_lds<VEC>(p) * p->pipe_waves, st>>>(
        (const E *)V, (E *)X, (E *)Phi, (Acc *)part, p->d_pipe_row, p->d_loc_row, args);
    int rc = launched();
    if (rc != CCDC_OK || chunks == 1) return rc;
    const int64_t n = (int64_t)p->K * p->W;
    if (wide_final) {
        const int G = reduce_final_groups(n / 4, chunks);
        k_reduce_final<A, 4><<<cdiv(n / 4, kBlock / G), kBlock, 0, st>>>((const Acc *)part, (E *)Phi, chunks, n / 4,
                                                                          (uint32_t)(n / 4), G);
    } else {
        const int G = reduce_final_groups(n, chunks);
        k_reduce_final<A, 1><<<cdiv(n, kBlock / G), kBlock, 0, st>>>((const Acc *)part, (E *)Phi, chunks, n,
                                                                      (uint32_t)n, G);
    }
    return launched();
}

}  // namespace

namespace ccdc {

template <class A>
int pipeline_run(const ccdc_plan_t *p, const void *V, void *X, void *Phi, void *part, bool wide_final, hipStream_t st)
{
    if (p->pipe_vec == 4) return run_pipeline<A, 4>(p, V, X, Phi, part, wide_final, st);
    if (p->pipe_vec == 2) return run_pipeline<A, 2>(p, V, X, Phi, part, wide_final, st);
    return run_pipeline<A, 1>(p, V, X, Phi, part, wide_final, st);
}

template <class A>
double pipeline_geometry(ccdc_plan_t *p)
{
    Candidate best{0, 1, 1, true, false, 0};
    consider<A, 4>(p, &best);
    consider<A, 2>(p, &best);
    consider<A, 1>(p, &best);
    p->pipe_vec = best.vec;
    p->pipe_waves = best.waves;
    p->pipe_chunks = best.chunks;
    p->pipe_even = best.even;
    p->pipe_shallow = best.shallow;
    return best.us;
}

}  // namespace ccdc
#endif

// The kernel's instantiations take minutes to compile in one piece: with CCDC_PIPELINE_PART set, this
// file is one of ten pieces, two for each algebra: its kernels that read past the caches with the code that
// launches them (the first with the entry points), and those that keep their reads.
namespace ccdc {
#ifdef CCDC_PIPELINE_PART
#define CCDC_RUN(A)                                                                                              \
    template int pipeline_run<A>(const ccdc_plan_t *, const void *, void *, void *, void *, bool, hipStream_t); \
    template double pipeline_geometry<A>(ccdc_plan_t *)
#define CCDC_KEPT(A) template PipeKernel<A> pipeline_kernel_kept<A>(const ccdc_plan_t *, int)
#if CCDC_PIPELINE_PART % 5 == 0
using PieceAlgebra = SumF32;
#elif CCDC_PIPELINE_PART % 5 == 1
using PieceAlgebra = XorU32;
#elif CCDC_PIPELINE_PART % 5 == 2
using PieceAlgebra = HybF32;
#elif CCDC_PIPELINE_PART % 5 == 3
using PieceAlgebra = HybBF16;
#else
using PieceAlgebra = HybF16;
#endif
#if CCDC_PIPELINE_PART < 5
extern CCDC_KEPT(PieceAlgebra);
CCDC_RUN(PieceAlgebra);
#else
CCDC_KEPT(PieceAlgebra);
#endif
#if CCDC_PIPELINE_PART == 0
#define CCDC_ELSEWHERE(A)                                                                                               \
    extern template int pipeline_run<A>(const ccdc_plan_t *, const void *, void *, void *, void *, bool, hipStream_t); \
    extern template double pipeline_geometry<A>(ccdc_plan_t *)
CCDC_ELSEWHERE(XorU32);
CCDC_ELSEWHERE(HybF32);
CCDC_ELSEWHERE(HybBF16);
CCDC_ELSEWHERE(HybF16);
#endif
#endif
#if !defined(CCDC_PIPELINE_PART) || CCDC_PIPELINE_PART == 0

// ccdc_pipeline_fused: checks, pack width, dispatch on the algebra.  The partial
// outputs of round chunks go to the plan's workspace, or, when the caller brings
// a buffer (own_part, of own_part_bytes bytes), to that one; a launch whose
// chunks do not fit a brought buffer is refused.
int pipeline_entry(const ccdc_plan_t *plan, const void *V, void *X, void *Phi, void *stream, void *own_part,
                   size_t own_part_bytes)
{
    int rc = ready(plan), vec_any = 1;
    if (rc != CCDC_OK) return rc;
    if (plan->compression) return CCDC_ESTATE;       // nothing is coded in that scheme
    if (!plan->pipe_ok) return CCDC_ESIZE;
    if ((rc = pick_vec(plan, &vec_any, V, (const void *)X, (const void *)Phi)) != CCDC_OK) return rc;
    if (by_receiver(plan)) return receive_entry(plan, V, X, Phi, stream);
    const bool wide_final = vec_any >= 4;            // Phi can be written four elements at a time
    const int chunks = plan->pipe_chunks;
    void *part = plan->d_workspace;
    if (own_part) {
        if (chunks > 1 && (uint64_t)chunks * (uint64_t)plan->K * (uint64_t)plan->W * 4u > (uint64_t)own_part_bytes)
            return CCDC_ESIZE;
        part = own_part;
    }
    hipStream_t st = (hipStream_t)stream;
    WorkspaceOrder order(plan, st, !own_part && chunks > 1);
    switch (plan->mode) {
    case CCDC_F32_SUM: return pipeline_run<SumF32>(plan, V, X, Phi, part, wide_final, st);
    case CCDC_F32_SUM_XOR: return pipeline_run<HybF32>(plan, V, X, Phi, part, wide_final, st);
    case CCDC_BF16_SUM_XOR: return pipeline_run<HybBF16>(plan, V, X, Phi, part, wide_final, st);
    case CCDC_F16_SUM_XOR: return pipeline_run<HybF16>(plan, V, X, Phi, part, wide_final, st);
    default: return pipeline_run<XorU32>(plan, V, X, Phi, part, wide_final, st);
    }
}

void pipeline_prepare(ccdc_plan_t *p)
{
    p->pipe_chunks = p->pipe_waves = p->pipe_vec = 1;
    p->node_waves = 0;
    if (!p->pipe_ok) return;
    double us = 0;
    switch (p->mode) {
    case CCDC_F32_SUM: us = pipeline_geometry<SumF32>(p); break;
    case CCDC_F32_SUM_XOR: us = pipeline_geometry<HybF32>(p); break;
    case CCDC_BF16_SUM_XOR: us = pipeline_geometry<HybBF16>(p); break;
    case CCDC_F16_SUM_XOR: us = pipeline_geometry<HybF16>(p); break;
    default: us = pipeline_geometry<XorU32>(p); break;
    }
    receive_prepare(p, us);
    receive_node_prepare(p);
}

#endif

}  // namespace ccdc

#if !defined(CCDC_PIPELINE_PART) || CCDC_PIPELINE_PART == 0
extern "C" {

int ccdc_pipeline_fused(const ccdc_plan_t *plan, const void *V, void *X, void *Phi, void *stream)
{
    return ccdc::pipeline_entry(plan, V, X, Phi, stream, nullptr, 0);
}

}  // extern "C"
#endif
