// HIP kernels (gfx950) and the C entry points of libccdc.
//
// Everything here is a streaming, bandwidth-bound elementwise pass: every
// work item moves one pack (16 bytes when the value length allows it, else 8
// bytes or one element) per operand, consecutive lanes touch consecutive packs of the same
// row, and there is no reuse across work items, so no LDS tiling and no MFMA.
#include <algorithm>
#include <new>

#include "common.hpp"

namespace {
using namespace ccdc;

// On large inputs, packs of more than one element, the XCDs take runs of span / 8 neighbouring workgroups in turn, so that an L2
// sees whole stretches of the rows; small ones and packs that share lines keep the order in which workgroups are handed out.  Over 110
// passes of 60 MB to 4 GB by ccdc_combine with the calls after it, ccdc_shuffle_fused and ccdc_reduce, and the uncoded scheme, with these
// runs 0.981 of the time, of 300 MB and more 0.980, with the stores past the caches 0.970 (56 jobs on 8 nodes, r = 2, T = 150000 u32 731 -> 702 us; uncoded,
// 22 nodes, T = 39296 u32, the packets 301 -> 263, 23 nodes, T = 14300 f32 67 -> 58).  A call alone: ccdc_combine in runs of 8
// to 512 workgroups 0.988 to 0.966 of the time over 25 inputs, with one-element packs 1.01 to 1.03; ccdc_reduce in runs of 8 to 32 0.98 over
// 65; ccdc_shuffle_fused from a gigabyte on 0.984 over six, below it 0.99 to 1.02.
constexpr uint32_t kCombineSpan = 1024, kReduceSpan = 128, kShuffleSpan = 256;
constexpr double kShuffleRunsBytes = 1e9;
// From here on ccdc_combine's sums are stored past the caches: 24 inputs of over a gigabyte 0.965 of the time, ordinary
// stores 0.988.  Below it the next call still finds part of the packets (15 nodes, r = 4, four files, T = 376 f32, 248 MB, a pass
// of the four stages 53.1 -> 53.5; 23 nodes, r = 4, three files, T = 64 bf16 60.6 -> 61.9).
constexpr double kPastStoreBytes = 500e6;
template <bool LARGE>
__device__ __forceinline__ uint32_t in_runs(uint32_t span)
{
    return LARGE ? xcd_spans(blockIdx.x, gridDim.x, span) : blockIdx.x;
}

// ------------------------------------------------------------------ combine
// Sec. IV-B pre-combining.  One work item = one pack of one packet Vbar[u][b]:
// it adds the same pack of the files of the served batch (m of them, or
// row_files[row] when batches differ in size).
template <class A, int VEC, bool KEPT, bool TOGETHER, bool ANY>
__global__ __launch_bounds__(kBlock) void k_combine(const typename A::elem *__restrict__ V,
                                                    typename A::elem *__restrict__ Vbar,
                                                    const int64_t *__restrict__ src_off,
                                                    const int32_t *__restrict__ row_files, uint32_t Wv, uint32_t W, int m,
                                                    int64_t file_stride, uint32_t items, bool past)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    constexpr bool LARGE = !KEPT && VEC > 1;          // see in_runs()
    const uint32_t idx = in_runs<LARGE>(kCombineSpan) * kBlock + threadIdx.x;
    if (idx >= items) return;
    const uint32_t row = idx / Wv, e = column<ANY, VEC>(idx - row * Wv, W);
    const E *src = V + src_off[row] + e;
    E *to = Vbar + (size_t)row * W + e;
    const int files = row_files ? row_files[row] : m;
    const P first = load_at<KEPT, ANY, P, E>(src);
    if (files == 1) {                                 // not a sum: the packet is the file's values as they are
        store_at<false, ANY, P, E>(to, first);
        return;
    }
    const P sum = O::narrow(sum_files<O, KEPT, TOGETHER, ANY>(first, src, files, file_stride));
    if (LARGE && past) store_at<true, ANY, P, E>(to, sum);
    else store_at<false, ANY, P, E>(to, sum);
}

// Pre-combining for short packets and long batches (few packs per packet, many
// files to add): one wavefront per packet.  The 64 lanes are cut into SEG-lane
// segments, SEG = packs of the packet rounded up to a power of two; segment g
// adds files g, g+G, g+2G, ... (G = 64/SEG) of the batch, each lane one pack, and
// the G segment sums are then added across the wavefront by a butterfly of lane
// exchanges.  The order of additions is fixed by (m, SEG), not by timing; it
// differs from k_combine's file order, so the algebras whose packets are coded
// bit patterns (fixed_order) do not use it.
template <class A, int VEC, bool KEPT>
__global__ __launch_bounds__(64) void k_combine_wave(const typename A::elem *__restrict__ V,
                                                     typename A::elem *__restrict__ Vbar,
                                                     const int64_t *__restrict__ src_off, uint32_t Wv, int seg,
                                                     int m, int64_t file_stride, uint32_t rows)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t row = blockIdx.x;
    if (row >= rows) return;
    const int lane = threadIdx.x;
    const int e = lane % seg, g = lane / seg, G = 64 / seg;
    const E *src = V + src_off[row] + (int64_t)e * VEC;
    typename O::Q acc = O::azero();
    if ((uint32_t)e < Wv)
        for (int f = g; f < m; f += G) acc = O::accum(acc, load_pack<KEPT, P>(src + f * file_stride));
    // segmented butterfly: after the step with distance d, lane l holds the sum of
    // the segments whose index differs from its own only in the bits below d/seg
    for (int d = seg; d < 64; d <<= 1) {
        typename O::Q other;
#pragma unroll
        for (int i = 0; i < VEC; i++) {
            uint32_t bits;
            __builtin_memcpy(&bits, &acc.v[i], 4);
            bits = (uint32_t)__shfl_xor((int)bits, d, 64);
            __builtin_memcpy(&other.v[i], &bits, 4);
        }
        // lower segment first on both sides so that every lane adds in the same order
        acc = (lane & d) ? O::add(other, acc) : O::add(acc, other);
    }
    if (g == 0 && (uint32_t)e < Wv) reinterpret_cast<P *>(Vbar)[(size_t)row * Wv + e] = O::narrow(acc);
}

// ------------------------------------------------------------------- encode
// Sec. IV-B coded packet.  One work item = one pack of X[u][a]: the sum over
// the other members b of segment segment_rank(a,b) of Vbar[u][b] at the same
// in-segment position; positions past the end of a short segment add nothing.
template <class A, int VEC, bool ANY>
__global__ __launch_bounds__(kBlock) void k_encode(const typename A::elem *__restrict__ Vbar,
                                                   typename A::elem *__restrict__ X, int r1, uint32_t Lv,
                                                   uint32_t ell, uint32_t W, uint32_t items)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= items) return;
    const uint32_t ua = idx / Lv, x = column<ANY, VEC>(idx - ua * Lv, ell);
    const uint32_t u = ua / r1;
    const int a = (int)(ua - u * r1);
    const E *rows = Vbar + (size_t)u * r1 * W;
    P acc = O::zero();
    for (int b = 0; b < r1; b++) {
        if (b == a) continue;
        const uint32_t pos = segment_rank(a, b) * ell + x;
        if (pos < W) acc = O::code(acc, packet_pack<O, true, false, ANY>(rows + (size_t)b * W, pos, W, 1, 0));
    }
    store_at<false, ANY, P, E>(X + (ANY ? (size_t)ua * ell + x : (size_t)idx * VEC), acc);
}

// ------------------------------------------------------------------- decode
// Sec. IV-B decoding.  One work item = one pack of D[u][b].  The pack lies in
// segment rho of the packet meant for b, which was carried by the sender a
// whose label that segment has; from X[u][a] the receiver removes the packs
// of the other packets in it (b' not in {a,b}), all of which it stores.
template <class A, int VEC>
__global__ __launch_bounds__(kBlock) void k_decode(const typename A::elem *__restrict__ X,
                                                   const typename A::elem *__restrict__ Vbar,
                                                   typename A::elem *__restrict__ D, int r1, uint32_t Lv,
                                                   uint32_t Wv, uint32_t items)
{
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= items) return;
    const uint32_t ub = idx / Wv, e = idx - ub * Wv;
    const uint32_t u = ub / r1;
    const int b = (int)(ub - u * r1);
    const int rho = (int)(e / Lv);
    const uint32_t x = e - rho * Lv;
    const int a = rho < b ? rho : rho + 1;
    const P *rows = reinterpret_cast<const P *>(Vbar) + (size_t)u * r1 * Wv;
    P acc = reinterpret_cast<const P *>(X)[((size_t)u * r1 + a) * Lv + x];
    for (int b2 = 0; b2 < r1; b2++) {
        if (b2 == a || b2 == b) continue;
        const uint32_t pos = segment_rank(a, b2) * Lv + x;
        if (pos < Wv) acc = O::uncode(acc, rows[(size_t)b2 * Wv + pos]);
    }
    reinterpret_cast<P *>(D)[idx] = acc;
}

// The same, by sender: one work item = pack x of X[u][a] and the r decoded packs that come out of
// it, one for each receiver.  The r packs of Vbar it holds are read once and used for r-1 receivers
// each, where k_decode reads X r times and Vbar r-1 times (from cache) and is bound by that.  R1 = r+1
// at compile time (k_decode serves r > 5).  12 nodes, r = 3, T = 6000, f16: 15.3 -> 7.9 us, 55 MB.
template <class A, int VEC, int R1, bool ANY>
__global__ __launch_bounds__(kBlock) void k_decode_sender(const typename A::elem *__restrict__ X,
                                                          const typename A::elem *__restrict__ Vbar,
                                                          typename A::elem *__restrict__ D, uint32_t Lv, uint32_t ell,
                                                          uint32_t W, uint32_t items)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= items) return;
    const uint32_t ua = idx / Lv, x = column<ANY, VEC>(idx - ua * Lv, ell);
    const uint32_t u = ua / R1;
    const int a = (int)(ua - u * R1);
    const E *rows = Vbar + (size_t)u * R1 * W;
    E *out = D + (size_t)u * R1 * W;
    const P coded = load_at<true, ANY, P, E>(X + (ANY ? (size_t)ua * ell + x : (size_t)idx * VEC));
    P side[R1];
#pragma unroll
    for (int b = 0; b < R1; b++) {
        const uint32_t pos = segment_rank(a, b) * ell + x;
        side[b] = O::zero();
        if (b != a && pos < W) side[b] = packet_pack<O, true, false, ANY>(rows + (size_t)b * W, pos, W, 1, 0);
    }
#pragma unroll
    for (int b = 0; b < R1; b++) {
        if (b == a) continue;
        P d = coded;
#pragma unroll
        for (int b2 = 0; b2 < R1; b2++)
            if (b2 != b && b2 != a) d = O::uncode(d, side[b2]);
        store_in_row<O, false, ANY>(out + (size_t)b * W, segment_rank(a, b) * ell + x, W, d);
    }
}

// ----------------------------------------------- combine + encode + decode
// One work item = (round u, sender a, in-segment pack x).  It pre-combines the
// r packs sender a's packet is made of straight from V (each read once),
// writes the coded pack, and produces for each of the r receivers the decoded
// pack of its own packet by removing the other r-1 from the coded pack.
// R1 = r+1 at compile time keeps the r combined packs in registers; R1 = 0 is
// the any-r fallback that re-reads them (cache hits) instead.
// MULTI: several files a batch, where their packets are asked for together (a kernel of their own: their sums in the making take
// registers that the other would pay for with fewer wavefronts); elsewhere the one kernel looks at m.  What a small call reads of
// its arguments is in their first 64 bytes.
template <class A, int VEC, int R1, bool KEPT, bool MULTI, bool ANY>
__global__ __launch_bounds__(kBlock) void k_shuffle_fused(const typename A::elem *__restrict__ V,
                                                          typename A::elem *__restrict__ X,
                                                          typename A::elem *__restrict__ D,
                                                          const int64_t *__restrict__ src_off, uint32_t items, uint32_t Lv,
                                                          uint32_t ell, uint32_t W, int r1_rt, int m, int64_t file_stride,
                                                          uint32_t span)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const int r1 = R1 > 0 ? R1 : r1_rt;
    const uint32_t idx = in_runs<!KEPT && (VEC > 1)>(span) * kBlock + threadIdx.x;
    if (idx >= items) return;
    const uint32_t ua = idx / Lv, x = column<ANY, VEC>(idx - ua * Lv, ell);
    const uint32_t u = ua / r1;
    const int a = (int)(ua - u * r1);
    const int64_t *src = src_off + (size_t)u * r1;
    E *to = X + (ANY ? (size_t)ua * ell + x : (size_t)idx * VEC), *Drows = D + (size_t)u * r1 * W;

    auto combined = [&](int b) -> P {       // pack of Vbar[u][b] that sender a carries
        return packet_pack<O, KEPT, files_together<O, ANY>(), ANY>(V + src[b], segment_rank(a, b) * ell + x, W, m, file_stride);
    };

    if constexpr (R1 > 0 && packets_together<O, R1 - 1>()) {
        P v[R1 - 1];                                  // of the members other than a
        const E *at[R1 - 1];
        bool there[R1 - 1];
#pragma unroll
        for (int k = 0; k < R1 - 1; k++) {
            const int b = k + (k >= a ? 1 : 0);
            const uint32_t pos = segment_rank(a, b) * ell + x;
            there[k] = pos < W;
            at[k] = V + src[b] + (there[k] ? pos : 0);
        }
        sum_packets<O, KEPT>(v, at, there, MULTI ? m : 1, file_stride);
        P coded = O::zero();
#pragma unroll
        for (int k = 0; k < R1 - 1; k++) coded = O::code(coded, v[k]);
        store_at<true, ANY, P, E>(to, coded);
#pragma unroll
        for (int k = 0; k < R1 - 1; k++) {
            if (!there[k]) continue;
            const int b = k + (k >= a ? 1 : 0);
            P acc = coded;
#pragma unroll
            for (int k2 = 0; k2 < R1 - 1; k2++)
                if (k2 != k) acc = O::uncode(acc, v[k2]);
            store_stream(Drows + (size_t)b * W + segment_rank(a, b) * ell + x, acc);
        }
    } else if constexpr (R1 > 0) {
        P v[R1];
#pragma unroll
        for (int b = 0; b < R1; b++)
            if (b != a) v[b] = combined(b);
        P coded = O::zero();
#pragma unroll
        for (int b = 0; b < R1; b++)
            if (b != a) coded = O::code(coded, v[b]);
        store_at<true, ANY, P, E>(to, coded);
#pragma unroll
        for (int b = 0; b < R1; b++) {
            if (b == a) continue;
            P acc = coded;
#pragma unroll
            for (int b2 = 0; b2 < R1; b2++)
                if (b2 != a && b2 != b) acc = O::uncode(acc, v[b2]);
            store_in_row<O, !ANY, ANY>(Drows + (size_t)b * W, segment_rank(a, b) * ell + x, W, acc);
        }
    } else {
        P coded = O::zero();
        for (int b = 0; b < r1; b++)
            if (b != a) coded = O::code(coded, combined(b));
        store_at<true, ANY, P, E>(to, coded);
        for (int b = 0; b < r1; b++) {
            if (b == a) continue;
            P acc = coded;
            for (int b2 = 0; b2 < r1; b2++)
                if (b2 != a && b2 != b) acc = O::uncode(acc, combined(b2));
            // past the caches also at any element, where ordinary stores take 1.03 of the time (11 nodes, r = 9, T = 620003 f16 340 -> 361 us)
            store_in_row<O, true, ANY>(Drows + (size_t)b * W, segment_rank(a, b) * ell + x, W, acc);
        }
    }
}

// ------------------------------------------------------------------- reduce
// Sec. IV-B final reduction as a gather-sum of rows: output block o (one node's
// c functions of one job) is the sum of a list of W-long rows, some in V (files
// the node stores), some in D (packets it decoded).  The list is cut into
// `split` chunks; work item = (o, chunk, pack).  With split > 1 the chunk sums
// go, not yet narrowed, to the workspace and k_reduce_final adds them in its fixed order.
template <class A, int VEC, bool KEPT, bool ANY>
__global__ __launch_bounds__(kBlock) void k_reduce_rows(const typename A::elem *__restrict__ V,
                                                        const typename A::elem *__restrict__ D,
                                                        typename A::elem *__restrict__ out,
                                                        typename A::acc *__restrict__ part,
                                                        const int64_t *__restrict__ red_ptr,
                                                        const int64_t *__restrict__ red_row,
                                                        const int64_t *__restrict__ red_out, uint32_t Wv, uint32_t W,
                                                        uint32_t tiles, int split, int64_t chunk_stride)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    constexpr bool LARGE = !KEPT && VEC > 1;          // see in_runs()
    const uint32_t block = in_runs<LARGE>(kReduceSpan);
    const uint32_t tile = block % tiles;
    const uint32_t oc = block / tiles;
    const uint32_t o = oc / split;
    const int s = (int)(oc - o * split);
    const uint32_t pack = tile * kBlock + threadIdx.x;
    if (pack >= Wv) return;
    const uint32_t e = column<ANY, VEC>(pack, W);
    const int64_t first = red_ptr[o], n = red_ptr[o + 1] - first;
    const int64_t lo = first + n * s / split, hi = first + n * (s + 1) / split;
    typename O::Q acc = O::azero();
    int64_t i = lo;
    auto row_pack = [&](int64_t at) {
        const int64_t row = red_row[at];
        return load_at<KEPT, ANY, P, E>(((row & 1) ? D : V) + (row >> 1) + e);
    };
    // One-element packs are few bytes in flight: eight rows at a time.  16 lists of 22 rows and more 0.93 of the time with four (12
    // nodes, r = 5, T = 27763 bf16 153 -> 110 us); wide packs 0.99 to 1.08.
    if constexpr (VEC == 1) {
        for (; i + 8 <= hi; i += 8) {
            P v[8];
#pragma unroll
            for (int t = 0; t < 8; t++) v[t] = row_pack(i + t);
#pragma unroll
            for (int t = 0; t < 8; t++) acc = O::accum(acc, v[t]);
        }
    }
#pragma unroll 4
    for (; i < hi; i++) acc = O::accum(acc, row_pack(i));
    if (split > 1) store_at<false, ANY, typename O::Q, typename A::acc>(part + (int64_t)s * chunk_stride + red_out[o] + e, acc);
    else store_at<LARGE, ANY, P, E>(out + red_out[o] + e, O::narrow(acc));
}

// The same in one launch: the wavefronts of a workgroup share the row list of 64 packs of an output and add up in LDS.
// Bound by the launch and the chain list entry, load, sum; the second launch of the split form and the partial sums that
// it reads back were 2.5 to 5 us of its time.  Which plans: plan_groups() in plan.cpp.  14 nodes, r = 1, T = 952 u32 8.0 -> 5.6 us,
// 12 nodes, r = 3, two files, T = 6000 f16 (40 MB) 17.3 -> 11.1 to 12, uncoded, 13 nodes, T = 48768 f32 17.8 -> 11; with one stage
// of rows in flight 3 % slower over 282 plans.
template <class A, int VEC, bool KEPT, bool ANY>
__global__ __launch_bounds__(kGroupLanes *kGroupMaxWaves) void k_reduce_group(
    const typename A::elem *__restrict__ V, const typename A::elem *__restrict__ D, typename A::elem *__restrict__ out,
    const int64_t *__restrict__ red_ptr, const int64_t *__restrict__ red_row, const int64_t *__restrict__ red_out,
    uint32_t Wv, uint32_t W, uint32_t tiles)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    constexpr int AHEAD = 8;                              // rows asked for together, two such stages in flight
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t o = blockIdx.x / tiles, tile = blockIdx.x - o * tiles;
    const uint32_t lane = threadIdx.x % kGroupLanes, wave = wave_uniform(threadIdx.x / kGroupLanes), waves = blockDim.x / kGroupLanes;
    const uint32_t pack = tile * kGroupLanes + lane;
    const int64_t first = red_ptr[o], n = red_ptr[o + 1] - first;
    const int64_t lo = first + n * wave / waves, hi = first + n * (wave + 1) / waves;
    typename O::Q acc = O::azero();
    if (pack < Wv && hi > lo) {
        const uint32_t offset = column<ANY, VEC>(pack, W) * (uint32_t)sizeof(E);
        struct Stage {
            P v[AHEAD];
        };
        int64_t next = lo;
        // past the list's end the last row stands in and is not used: loads on a condition cost the overlap of the stages (6 % of
        // the time over 314 plans, up to 50 % on inputs of 40 to 140 MB)
        auto load = [&](Stage &s) {
#pragma unroll
            for (int t = 0; t < AHEAD; t++) {
                const int64_t row = red_row[next + t < hi ? next + t : hi - 1];
                const E *base = (row & 1) ? D : V;
                s.v[t] = load_at<KEPT, ANY, P, E>(reinterpret_cast<const char *>(base + (row >> 1)) + lane_offset(offset));
            }
            next += AHEAD;
        };
        auto use = [&](const Stage &s, int64_t left) {
#pragma unroll
            for (int t = 0; t < AHEAD; t++)
                if (t < left) acc = O::accum(acc, s.v[t]);
        };
        Stage even, odd;
        int64_t left = hi - lo;
        load(even);
        for (;;) {
            if (left <= AHEAD) {
                use(even, left);
                break;
            }
            load(odd);
            use(even, AHEAD);
            left -= AHEAD;
            if (left <= AHEAD) {
                use(odd, left);
                break;
            }
            load(even);
            use(odd, AHEAD);
            left -= AHEAD;
        }
    }
    add_wavefronts<A, VEC>(smem, acc, waves, [&](uint32_t i, typename A::acc v) {
        const uint32_t from = tile * kGroupLanes + i / VEC;
        if (from < Wv) out[red_out[o] + column<ANY, VEC>(from, W) + i % VEC] = A::narrow(v);
    });
}

void release_device(ccdc_plan_t *p)
{
    if (!p) return;
    if (p->uploaded || p->d_src_off || p->d_red_ptr || p->d_red_row || p->d_red_out || p->d_loc_row || p->d_pipe_row ||
        p->d_row_files || p->d_node_rows || p->d_node_list || p->d_workspace || p->ws_event) {
        int cur = -1;
        const bool sw = hipGetDevice(&cur) == hipSuccess && p->device >= 0 && cur != p->device &&
                        hipSetDevice(p->device) == hipSuccess;
        (void)hipFree(p->d_src_off);
        (void)hipFree(p->d_red_ptr);
        (void)hipFree(p->d_red_row);
        (void)hipFree(p->d_red_out);
        (void)hipFree(p->d_loc_row);
        (void)hipFree(p->d_pipe_row);
        (void)hipFree(p->d_row_files);
        (void)hipFree(p->d_node_rows);
        (void)hipFree(p->d_node_list);
        (void)hipFree(p->d_workspace);
        if (p->ws_event) (void)hipEventDestroy((hipEvent_t)p->ws_event);
        if (sw) (void)hipSetDevice(cur);
    }
    p->d_src_off = p->d_red_ptr = p->d_red_row = p->d_red_out = p->d_loc_row = nullptr;
    p->d_pipe_row = nullptr;
    p->d_row_files = nullptr;
    p->d_node_rows = nullptr;
    p->d_node_list = nullptr;
    p->d_workspace = nullptr;
    p->pipe_chunks = 0;
    p->ws_event = nullptr;
    p->ws_stream = nullptr;
    p->ws_used = false;
    p->uploaded = false;
    p->device = -1;
}

template <class T>
int to_device(const std::vector<T> &h, T **d)
{
    const size_t bytes = (h.empty() ? 1 : h.size()) * sizeof(T);
    if (hipMalloc((void **)d, bytes) != hipSuccess) {
        *d = nullptr;
        (void)hipGetLastError();
        return CCDC_ENOMEM;
    }
    if (!h.empty() && hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess)
        return CCDC_EHIP;
    return CCDC_OK;
}

// ---- typed launchers: A = algebra, VEC = pack width, ANY = packs at any element
template <class A, int VEC, bool ANY>
int run_combine(const ccdc_plan_t *p, const void *V, void *Vbar, hipStream_t st)
{
    using E = typename A::elem;
    const uint32_t Wv = cdiv(p->W, VEC), W = (uint32_t)p->W;
    const uint64_t items = (uint64_t)p->nrows * Wv;
    if (items == 0) return CCDC_OK;
    if (!fits_rows<VEC, ANY>(p->nrows, W)) return CCDC_ESIZE;
    const double packets = (double)p->nrows * p->W;
    const bool kept = moved_bytes(p, packets) <= kKeptStageBytes ||                      // V and Vbar
                      (VEC == 1 && packets * sizeof(E) <= kKeptPacketBytes);
    // short packets, long batches: a wavefront per packet with a cross-lane reduction
#ifndef CCDC_COMBINE_WAVE_MIN_FILES
#define CCDC_COMBINE_WAVE_MIN_FILES 8
#endif
    if constexpr (!A::fixed_order && !ANY) {
        if (Wv <= 16 && p->m >= CCDC_COMBINE_WAVE_MIN_FILES && !p->d_row_files) {
            int seg = 1;
            while ((uint32_t)seg < Wv) seg <<= 1;
            const uint32_t rows = (uint32_t)p->nrows;
            by_reads<false>(kept, [&](auto k) {
                k_combine_wave<A, VEC, decltype(k)::value><<<rows, 64, 0, st>>>(
                    (const E *)V, (E *)Vbar, p->d_src_off, Wv, seg, p->m, (int64_t)p->Q * p->T, rows);
            });
            return launched();
        }
    }
    const int files = p->compression ? p->batch_first[1] : p->m;        // of a batch, uncoded plans: of the largest
    const bool past = moved_bytes(p, packets) >= kPastStoreBytes;
    by_reads<false>(kept, [&](auto k) {
        by_files<Ops<A, VEC>, ANY>(files > 2, [&](auto together) {
            k_combine<A, VEC, decltype(k)::value, decltype(together)::value, ANY><<<cdiv(items, kBlock), kBlock, 0, st>>>(
                (const E *)V, (E *)Vbar, p->d_src_off, p->d_row_files, Wv, W, p->m, (int64_t)p->Q * p->T, (uint32_t)items, past);
        });
    });
    return launched();
}

template <class A, int VEC, bool ANY>
int run_encode(const ccdc_plan_t *p, const void *Vbar, void *X, hipStream_t st)
{
    using E = typename A::elem;
    const uint32_t Lv = cdiv(p->ell, VEC);
    const uint64_t items = (uint64_t)p->nround * (p->r + 1) * Lv;
    if (!fits_rows<VEC, ANY>((uint64_t)p->nround * (p->r + 1), p->ell)) return CCDC_ESIZE;
    k_encode<A, VEC, ANY><<<cdiv(items, kBlock), kBlock, 0, st>>>((const E *)Vbar, (E *)X, p->r + 1, Lv, (uint32_t)p->ell,
                                                                   (uint32_t)p->W, (uint32_t)items);
    return launched();
}

template <class A, int VEC, bool ANY>
int run_decode(const ccdc_plan_t *p, const void *X, const void *Vbar, void *D, hipStream_t st)
{
    using E = typename A::elem;
    const uint32_t Lv = cdiv(p->ell, VEC), ell = (uint32_t)p->ell, W = (uint32_t)p->W;
    if (!fits_rows<VEC, ANY>((uint64_t)p->nround * (p->r + 1), W)) return CCDC_ESIZE;
    // By sender where the packs of the padded segments can be numbered too (packets of fewer than four
    // elements have more of those than of their own); k_decode takes whatever the packets' packs allow.
    const uint64_t packs = (uint64_t)p->nround * (p->r + 1) * Lv;
    const uint32_t by_sender = (uint32_t)packs, blocks = cdiv(packs, kBlock);
    const E *x = (const E *)X, *v = (const E *)Vbar;
    switch (fits_launch(packs) ? p->r + 1 : 0) {
    case 2: k_decode_sender<A, VEC, 2, ANY><<<blocks, kBlock, 0, st>>>(x, v, (E *)D, Lv, ell, W, by_sender); break;
    case 3: k_decode_sender<A, VEC, 3, ANY><<<blocks, kBlock, 0, st>>>(x, v, (E *)D, Lv, ell, W, by_sender); break;
    case 4: k_decode_sender<A, VEC, 4, ANY><<<blocks, kBlock, 0, st>>>(x, v, (E *)D, Lv, ell, W, by_sender); break;
    case 5: k_decode_sender<A, VEC, 5, ANY><<<blocks, kBlock, 0, st>>>(x, v, (E *)D, Lv, ell, W, by_sender); break;
    case 6: k_decode_sender<A, VEC, 6, ANY><<<blocks, kBlock, 0, st>>>(x, v, (E *)D, Lv, ell, W, by_sender); break;
    default: {
        constexpr int PACK = ANY ? 1 : VEC;              // k_decode walks whole packets: their packs are not moved back
        const uint32_t Wv = (uint32_t)(p->W / PACK), Lw = (uint32_t)(p->ell / PACK);
        const uint64_t items = (uint64_t)p->nround * (p->r + 1) * Wv;
        k_decode<A, PACK><<<cdiv(items, kBlock), kBlock, 0, st>>>(x, v, (E *)D, p->r + 1, Lw, Wv, (uint32_t)items);
        break;
    }
    }
    return launched();
}

template <class A, int VEC, bool ANY, int R1>
void launch_shuffle(const ccdc_plan_t *p, const void *V, void *X, void *D, hipStream_t st)
{
    using E = typename A::elem;
    const uint32_t Lv = cdiv(p->ell, VEC);
    const uint64_t items = (uint64_t)p->nround * (p->r + 1) * Lv;
    const double bytes = moved_bytes(p, (double)p->nrows * (p->W + p->ell));                         // V, X and D
    const bool kept = bytes <= kKeptStageBytes;
    const uint32_t span = bytes >= kShuffleRunsBytes ? kShuffleSpan : kXcds;
    auto launch = [&](auto multi) {
        by_reads<VEC == 1>(kept, [&](auto k) {
            k_shuffle_fused<A, VEC, R1, decltype(k)::value, decltype(multi)::value, ANY><<<cdiv(items, kBlock), kBlock, 0, st>>>(
                (const E *)V, (E *)X, (E *)D, p->d_src_off, (uint32_t)items, Lv, (uint32_t)p->ell, (uint32_t)p->W, p->r + 1, p->m, (int64_t)p->Q * p->T, span);
        });
    };
    if constexpr (R1 > 0 && packets_together<Ops<A, VEC>, R1 - 1>()) {
        if (p->m == 1) return launch(std::false_type());
    }
    launch(std::true_type());
}

template <class A, int VEC, bool ANY>
int run_shuffle(const ccdc_plan_t *p, const void *V, void *X, void *D, hipStream_t st)
{
    if (!fits_rows<VEC, ANY>((uint64_t)p->nround * (p->r + 1), p->ell)) return CCDC_ESIZE;
    switch (p->r + 1) {
    case 2: launch_shuffle<A, VEC, ANY, 2>(p, V, X, D, st); break;
    case 3: launch_shuffle<A, VEC, ANY, 3>(p, V, X, D, st); break;
    case 4: launch_shuffle<A, VEC, ANY, 4>(p, V, X, D, st); break;
    case 5: launch_shuffle<A, VEC, ANY, 5>(p, V, X, D, st); break;
    case 6: launch_shuffle<A, VEC, ANY, 6>(p, V, X, D, st); break;
    case 7: launch_shuffle<A, VEC, ANY, 7>(p, V, X, D, st); break;
    case 8: launch_shuffle<A, VEC, ANY, 8>(p, V, X, D, st); break;
    default: launch_shuffle<A, VEC, ANY, 0>(p, V, X, D, st); break;
    }
    return launched();
}

// SHARED: rows begin anywhere in a cache line, see kKeptPacketBytes.
template <class A, int VEC, bool ANY, bool SHARED = VEC == 1>
void reduce_in_groups(const ccdc_plan_t *p, const void *V, const void *D, void *Phi, bool kept, hipStream_t st)
{
    using E = typename A::elem;
    // the widest packs that make enough workgroups, else those of four bytes
    if constexpr (VEC > 1 && VEC * sizeof(E) > 4) {
        if (p->nout * cdiv(cdiv(p->W, VEC), kGroupLanes) < kGroupsWanted)
            return reduce_in_groups<A, VEC / 2, ANY, SHARED>(p, V, D, Phi, kept, st);
    }
    const uint32_t Wv = cdiv(p->W, VEC), tiles = cdiv(Wv, kGroupLanes), threads = kGroupLanes * p->red_waves;
    by_reads<SHARED>(kept, [&](auto k) {
        k_reduce_group<A, VEC, decltype(k)::value, ANY><<<(uint32_t)p->nout * tiles, threads, threads * VEC * 4, st>>>(
            (const E *)V, (const E *)D, (E *)Phi, p->d_red_ptr, p->d_red_row, p->d_red_out, Wv, (uint32_t)p->W, tiles);
    });
}

template <class A, int VEC, bool ANY>
int run_reduce(const ccdc_plan_t *p, const void *V, const void *D, void *Phi, hipStream_t st)
{
    using E = typename A::elem;
    const uint32_t Wv = cdiv(p->W, VEC);
    const uint32_t tiles = cdiv(Wv, kBlock);
    const int split = p->red_split;
    const uint64_t blocks = (uint64_t)p->nout * split * tiles;
    const int64_t chunk_stride = (int64_t)p->J * p->Q * p->T;
    if (!fits_launch(ANY ? (uint64_t)p->nout * split * cdiv(p->W, kBlock) : blocks) || !fits_launch((uint64_t)chunk_stride / (ANY ? 1 : VEC))) return CCDC_ESIZE;
    using Acc = typename A::acc;
    const bool kept = moved_bytes(p, (double)p->nrows * p->W + (double)chunk_stride) <= kKeptStageBytes;        // V, D, Phi
    if (p->red_waves > 0) {
        reduce_in_groups<A, VEC, ANY>(p, V, D, Phi, kept, st);
        return launched();
    }
    WorkspaceOrder order(p, st, split > 1);
    by_reads<VEC == 1>(kept, [&](auto k) {
        k_reduce_rows<A, VEC, decltype(k)::value, ANY><<<(uint32_t)blocks, kBlock, 0, st>>>(
            (const E *)V, (const E *)D, (E *)Phi, (Acc *)p->d_workspace, p->d_red_ptr, p->d_red_row, p->d_red_out, Wv, (uint32_t)p->W,
            tiles, split, chunk_stride);
    });
    int rc = launched();
    if (rc != CCDC_OK || split == 1) return rc;
    return reduce_chunks<A, ANY ? 1 : VEC>(p, Phi, split, chunk_stride, st);
}

}  // namespace

// ------------------------------------------------------------ entry points
extern "C" {

int ccdc_plan(int K, int r, int Q, int N, ccdc_plan_t **out) { return ccdc::build_plan(K, r, Q, N, false, 1, out); }

int ccdc_plan_jobs(int K, int r, int Q, int N, ccdc_plan_t **out) { return ccdc::build_plan(K, r, Q, N, true, 1, out); }

int ccdc_plan_jobs_repeated(int K, int r, int Q, int N, int gamma, ccdc_plan_t **out)
{
    return ccdc::build_plan(K, r, Q, N, true, gamma, out);
}

int ccdc_plan_compression(int K, int r, int Q, int N, ccdc_plan_t **out)
{
    return ccdc::build_compression_plan(K, r, Q, N, out);
}

void ccdc_plan_destroy(ccdc_plan_t *plan)
{
    if (!plan) return;
    release_device(plan);
    delete plan;
}

int ccdc_plan_bind(ccdc_plan_t *plan, int64_t T, int mode)
{
    if (!plan) return CCDC_EINVAL;
    const int rc = ccdc::bind_plan(plan, T, mode);
    if (rc == CCDC_OK) release_device(plan);     // tables of an earlier binding are stale
    return rc;
}

int ccdc_plan_upload(ccdc_plan_t *plan)
{
    if (!plan) return CCDC_EINVAL;
    if (!plan->bound) return CCDC_ESTATE;
    release_device(plan);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return CCDC_EHIP;
    }
    plan->device = dev;
    ccdc::pipeline_prepare(plan);                 // launch geometry of the one-pass kernel on this device
    // partial sums of a split row list: where ccdc_reduce or ccdc_node_decode_reduce runs that form
    const bool split = plan->red_waves == 0 || (!plan->compression && plan->node_waves == 0);
    plan->workspace_bytes = split ? plan->red_workspace_bytes : 0;
    if (plan->pipe_chunks > 1)
        plan->workspace_bytes = std::max(plan->workspace_bytes, (size_t)plan->pipe_chunks * (size_t)plan->K * (size_t)plan->W * 4);
    int rc = to_device(plan->src_off, &plan->d_src_off);
    if (rc == CCDC_OK) rc = to_device(plan->red_ptr, &plan->d_red_ptr);
    if (rc == CCDC_OK) rc = to_device(plan->red_row, &plan->d_red_row);
    if (rc == CCDC_OK) rc = to_device(plan->red_out, &plan->d_red_out);
    if (rc == CCDC_OK) rc = to_device(plan->loc_row, &plan->d_loc_row);
    if (rc == CCDC_OK) rc = to_device(plan->pipe_row, &plan->d_pipe_row);
    if (rc == CCDC_OK && !plan->row_files.empty()) rc = to_device(plan->row_files, &plan->d_row_files);
    if (rc == CCDC_OK && !plan->node_rows.empty()) rc = to_device(plan->node_rows, &plan->d_node_rows);
    if (rc == CCDC_OK && !plan->node_list.empty()) rc = to_device(plan->node_list, &plan->d_node_list);
    if (rc == CCDC_OK && plan->workspace_bytes > 0 &&
        hipMalloc(&plan->d_workspace, plan->workspace_bytes) != hipSuccess) {
        plan->d_workspace = nullptr;
        (void)hipGetLastError();
        rc = CCDC_ENOMEM;
    }
    if (rc == CCDC_OK && plan->workspace_bytes > 0) {
        hipEvent_t ev = nullptr;
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            rc = CCDC_EHIP;
        }
        plan->ws_event = ev;
    }
    if (rc != CCDC_OK) {
        release_device(plan);
        return rc;
    }
    (void)ccdc::scratch_address(nullptr);         // set-up for ccdc_pipeline_fused_noalloc, which reports a failure itself
    plan->uploaded = true;
    return CCDC_OK;
}

int ccdc_plan_query(const ccdc_plan_t *p, int what, void *out, size_t out_bytes)
{
    if (!p || !out) return CCDC_EINVAL;
    auto scalar = [&](int64_t v) {
        if (out_bytes < sizeof(int64_t)) return (int)CCDC_EINVAL;
        *static_cast<int64_t *>(out) = v;
        return (int)CCDC_OK;
    };
    auto table = [&](const void *src, size_t bytes) {
        if (out_bytes < bytes) return (int)CCDC_EINVAL;
        if (bytes) __builtin_memcpy(out, src, bytes);
        return (int)CCDC_OK;
    };
    const int64_t r1 = p->r + 1;
    switch (what) {
    case CCDC_Q_K: return scalar(p->K);
    case CCDC_Q_R: return scalar(p->r);
    case CCDC_Q_Q: return scalar(p->Q);
    case CCDC_Q_N: return scalar(p->N);
    case CCDC_Q_J: return scalar(p->J);
    case CCDC_Q_C: return scalar(p->c);
    case CCDC_Q_M: return scalar(p->m);
    case CCDC_Q_NBATCH: return scalar(p->nbatch);
    case CCDC_Q_NROUND: return scalar(p->nround);
    case CCDC_Q_NROWS: return scalar(p->nrows);
    case CCDC_Q_SCHEME: return scalar(p->compression ? 2 : (p->paper_jobs ? 1 : 0));
    case CCDC_Q_BATCH_FIRST: return table(p->batch_first.data(), p->batch_first.size() * 4);
    case CCDC_Q_NODE_BATCH: return table(p->node_batch.data(), p->node_batch.size() * 4);
    case CCDC_Q_PACKET_RECV: return table(p->pkt_recv.data(), p->pkt_recv.size() * 4);
    case CCDC_Q_PACKET_BATCH: return table(p->pkt_batch.data(), p->pkt_batch.size() * 4);
    case CCDC_Q_PACKET_SEND: return table(p->pkt_send.data(), p->pkt_send.size() * 4);
    case CCDC_Q_ROWS_PER_NODE: return scalar(p->rows_per_node);
    case CCDC_Q_NODE_ROWS: return table(p->node_rows.data(), p->node_rows.size() * 4);
    case CCDC_Q_FILE_NODES:
        return p->compression ? (int)CCDC_ESTATE : table(p->file_nodes.data(), p->file_nodes.size() * 4);
    case CCDC_Q_FILES_PER_NODE: return p->compression ? (int)CCDC_ESTATE : scalar(p->files_per_node);
    case CCDC_Q_NODE_FILES:
        return p->compression ? (int)CCDC_ESTATE : table(p->node_files.data(), p->node_files.size() * 4);
    case CCDC_Q_BATCH_JOB: return table(p->batch_job.data(), p->batch_job.size() * 4);
    case CCDC_Q_BATCH_FILE0: return table(p->batch_file0.data(), p->batch_file0.size() * 4);
    case CCDC_Q_BATCH_LABEL: return table(p->batch_label.data(), p->batch_label.size() * 4);
    case CCDC_Q_ROUND_MEMBER: return table(p->round_member.data(), p->round_member.size() * 4);
    case CCDC_Q_ROUND_BATCH: return table(p->round_batch.data(), p->round_batch.size() * 4);
    case CCDC_Q_PIPELINE_LAUNCH: {
        if (!p->uploaded || !p->pipe_ok) return CCDC_ESTATE;
        const bool receiver = ccdc::by_receiver(p);
        const int32_t launch[4] = {p->pipe_vec, p->pipe_waves, receiver ? 1 : p->pipe_chunks,
                                   receiver ? 4 : (p->pipe_even ? 1 : 0) | (p->pipe_shallow ? 2 : 0)};
        return table(launch, sizeof launch);
    }
    case CCDC_Q_REDUCE_LAUNCH: {
        if (!p->uploaded) return CCDC_ESTATE;
        const int32_t launch[4] = {p->red_split, p->red_waves, p->node_waves > 0 ? p->node_vec : 0, p->node_waves};
        return table(launch, sizeof launch);
    }
    default: break;
    }
    if (!p->bound) {
        switch (what) {
        case CCDC_Q_T: case CCDC_Q_MODE: case CCDC_Q_W: case CCDC_Q_SEG_LEN: case CCDC_Q_SCHEDULED_ELEMS:
        case CCDC_Q_CLOSED_FORM_NUM: case CCDC_Q_CLOSED_FORM_DEN: case CCDC_Q_V_ELEMS: case CCDC_Q_VBAR_ELEMS:
        case CCDC_Q_X_ELEMS: case CCDC_Q_D_ELEMS: case CCDC_Q_PHI_ELEMS: case CCDC_Q_WORKSPACE_BYTES:
        case CCDC_Q_PACKET_LEN:
            return CCDC_ESTATE;
        default:
            return CCDC_EINVAL;
        }
    }
    switch (what) {
    case CCDC_Q_T: return scalar(p->T);
    case CCDC_Q_MODE: return scalar(p->mode);
    case CCDC_Q_W: return scalar(p->W);
    case CCDC_Q_SEG_LEN: return scalar(p->ell);
    case CCDC_Q_SCHEDULED_ELEMS: return scalar(p->scheduled);
    case CCDC_Q_CLOSED_FORM_NUM: return scalar(p->compression ? p->nrows * p->W : p->nround * r1 * p->W);
    case CCDC_Q_CLOSED_FORM_DEN: return scalar(p->compression ? 1 : p->r);
    case CCDC_Q_V_ELEMS: return scalar((int64_t)p->J * p->N * p->Q * p->T);
    case CCDC_Q_VBAR_ELEMS: return scalar(p->nrows * p->W);
    case CCDC_Q_X_ELEMS: return scalar(p->compression ? 0 : p->nrows * p->ell);
    case CCDC_Q_D_ELEMS: return scalar(p->nrows * p->W);
    case CCDC_Q_PHI_ELEMS: return scalar((int64_t)p->J * p->Q * p->T);
    case CCDC_Q_WORKSPACE_BYTES: return scalar((int64_t)p->workspace_bytes);
    case CCDC_Q_PACKET_LEN: return table(p->packet_len.data(), p->packet_len.size() * 8);
    default: return CCDC_EINVAL;
    }
}

const char *ccdc_strerror(int status)
{
    switch (status) {
    case CCDC_OK: return "ok";
    case CCDC_EINVAL: return "invalid argument";
    case CCDC_ENOMEM: return "out of memory";
    case CCDC_EHIP: return "HIP runtime error";
    case CCDC_ESIZE: return "size exceeds what the library indexes";
    case CCDC_ESTATE: return "plan is not bound/uploaded, or its device is not current";
    default: return "unknown status";
    }
}

int ccdc_combine(const ccdc_plan_t *plan, const void *V, void *Vbar, void *stream)
{
    int rc = ready(plan), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if ((rc = pick_wide(plan, Call::combine, -1, &vec, &any, V, (const void *)Vbar)) != CCDC_OK) return rc;
    // (packets of up to 16 packs are left as they are: in f32 and u32, batches of eight files and more have a wavefront each)
    if (!any && plan->W / vec > 16) narrow_files(plan, plan->compression ? plan->batch_first[1] : plan->m, plan->nrows, plan->W, &vec);
    hipStream_t st = (hipStream_t)stream;
    CCDC_DISPATCH(plan, vec, any, (run_combine<A, VEC, ANY>(plan, V, Vbar, st)));
}

int ccdc_encode(const ccdc_plan_t *plan, const void *Vbar, void *X, void *stream)
{
    int rc = ready(plan), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if (plan->compression) return CCDC_ESTATE;       // nothing is coded in that scheme
    if ((rc = pick_wide(plan, Call::encode, -1, &vec, &any, Vbar, (const void *)X)) != CCDC_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    CCDC_DISPATCH(plan, vec, any, (run_encode<A, VEC, ANY>(plan, Vbar, X, st)));
}

int ccdc_decode(const ccdc_plan_t *plan, const void *X, const void *Vbar, void *D, void *stream)
{
    int rc = ready(plan), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if (plan->compression) return CCDC_ESTATE;       // nothing is coded in that scheme
    if ((rc = pick_wide(plan, Call::decode, -1, &vec, &any, X, Vbar, (const void *)D)) != CCDC_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    CCDC_DISPATCH(plan, vec, any, (run_decode<A, VEC, ANY>(plan, X, Vbar, D, st)));
}

int ccdc_reduce(const ccdc_plan_t *plan, const void *V, const void *D, void *Phi, void *stream)
{
    int rc = ready(plan), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if ((rc = pick_wide(plan, Call::reduce, -1, &vec, &any, V, D, (const void *)Phi)) != CCDC_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    CCDC_DISPATCH(plan, vec, any, (run_reduce<A, VEC, ANY>(plan, V, D, Phi, st)));
}

int ccdc_shuffle_fused(const ccdc_plan_t *plan, const void *V, void *X, void *D, void *stream)
{
    int rc = ready(plan), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if (plan->compression) return CCDC_ESTATE;       // nothing is coded in that scheme
    if ((rc = pick_wide(plan, Call::shuffle, -1, &vec, &any, V, (const void *)X, (const void *)D)) != CCDC_OK) return rc;
    if (!any) narrow_files(plan, plan->m, plan->nrows, plan->ell, &vec);
    hipStream_t st = (hipStream_t)stream;
    CCDC_DISPATCH(plan, vec, any, (run_shuffle<A, VEC, ANY>(plan, V, X, D, st)));
}

}  // extern "C"
