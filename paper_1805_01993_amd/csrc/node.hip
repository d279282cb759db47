// What one node does in the shuffle (Sec. IV-B), from nothing but the files it
// stores and the coded packets it receives: the node-local form of the path.
// Run for every node it is the emulation in which no result is shared between
// nodes: each of the r nodes that store a batch pre-combines it for itself,
// as a real cluster would.
#include <type_traits>

#include "common.hpp"

namespace {
using namespace ccdc;

// What a call reads with ordinary loads, through the caches; the rest goes past them.
enum Reads {
    kPast = 0,                        // nothing
    kCoded = 1,                       // the coded packets
    kAll = 2,                         // and the files
};

// ------------------------------------------------------- a sender's packets
// Coded-packet equation of Sec. IV-B for the packets listed in `rows` (those one
// node sends; null = every packet).  One work item = one pack of X[u][a]: the
// sender pre-combines, for each other member b, the segment of b's packet that
// carries the sender's label; it stores all those batches.
template <class A, int VEC, int READS, bool TOGETHER, bool ANY>
__global__ __launch_bounds__(kBlock) void k_node_encode(const typename A::elem *__restrict__ V,
                                                        typename A::elem *__restrict__ X,
                                                        const int64_t *__restrict__ src_off,
                                                        const int32_t *__restrict__ rows, uint32_t items, uint32_t Lv,
                                                        uint32_t ell, uint32_t W, int r1, int m, int64_t file_stride)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= items) return;
    const uint32_t j = idx / Lv, x = column<ANY, VEC>(idx - j * Lv, ell);
    const uint32_t i = rows ? (uint32_t)rows[j] : j;
    const uint32_t u = i / r1;
    const int a = (int)(i - u * r1);
    const int64_t *src = src_off + (size_t)u * r1;
    P coded = O::zero();
    for (int b = 0; b < r1; b++) {
        if (b == a) continue;
        const uint32_t pos = segment_rank(a, b) * ell + x;
        if (pos < W) coded = O::code(coded, packet_pack<O, READS == kAll, TOGETHER, ANY>(V + src[b], pos, W, m, file_stride));
    }
    store_at<true, ANY, P, E>(X + (size_t)i * ell + x, coded);
}

// The element of its row that the pack at x of the segment which begins at `first` starts from.  A pack that reaches past the row's
// end is moved back to the last whole one (*x too), as in column(); a last segment has a pack.
template <bool ANY, int VEC>
__device__ __forceinline__ uint32_t in_segment(uint32_t first, uint32_t W, uint32_t *x)
{
    if (ANY && first + *x + VEC > W) *x = W - VEC - first;
    return first + *x;
}

// Chunk s of output block o's row list: an equal part of the rows [lo, hi), files the node stores before packets it receives; or, where
// the lists are cut by rounds, an equal part of the former (own_rows of them) and packets [first, last) of a list of their own.
struct Rows {
    int64_t lo, hi;
    uint32_t first, last;
};
__device__ __forceinline__ Rows chunk_of(const int64_t *__restrict__ red_ptr, const int32_t *__restrict__ list, uint32_t own_rows,
                                         uint32_t o, int s, int split)
{
    const int64_t start = red_ptr[o], n = list ? own_rows : red_ptr[o + 1] - start;
    const int64_t lo = start + n * s / split, hi = start + n * (s + 1) / split;
    if (!list) return {lo, hi, 0, 0};
    return {lo, hi, (uint32_t)list[o * split + s], (uint32_t)list[o * split + s + 1]};
}

// Lists are cut by rounds for r = 3, 4 and 5 only (bind_plan()); R1 = 0 is any r.
template <int R1>
constexpr bool kMayBeListed = R1 == 0 || R1 > 3;

// Calls walk(listed) with whether there is a list of packets as a compile-time constant: looked at in every row it parts the loads that are
// asked for together (a node alone, r = 1, 21 nodes, T = 13786 f32 3.9 -> 4.9 us).
template <bool MAY, class F>
__device__ __forceinline__ void by_list(const int32_t *list, F walk)
{
    if constexpr (MAY) {
        if (list) return walk(std::true_type());
    }
    walk(std::false_type());
}

// The number u*(r+1)+b of a received packet, the same for all lanes.  A row is its first element: element / W, exact in fp64, which leaves
// the result in a vector register and the tables that it indexes to vector loads if the compiler is not told.
template <bool LISTED>
__device__ __forceinline__ uint32_t packet_at(const int64_t *__restrict__ red_row, const int32_t *__restrict__ list_packets, int64_t at, double per_row)
{
    if constexpr (LISTED) return wave_uniform((uint32_t)list_packets[at]);
    else return wave_uniform((uint32_t)((double)(red_row[at] >> 1) * per_row + 0.5));
}

// --------------------------------------------- a receiver's decoding + output
// Decoding and final reduction of Sec. IV-B for the output blocks o_first,
// o_first + o_step, ... (one node's block in every job, or all blocks).  The
// row list of a block is ccdc_reduce's: the files the node stores, then the
// packets it receives.  A received packet is not read from a buffer: pack e of
// it lies in segment rho, carried by the sender whose label that segment has, and
// is recovered here as that sender's coded pack minus the packs of the other
// members' packets in it, which the receiver pre-combines from its own files.
// The list is cut into `split` chunks as in ccdc_reduce.
// What bounds it: each row is a chain of table entry, rows and data.  With r+1 at compile time (R1; 0 for r > 5 and batches of
// several files) four rows are asked for together, two for r >= 4.  Against one row after the other, all nodes, one file: 17 inputs of
// r = 3 0.80 of the time, 23 of r = 4 0.69, 15 of r = 5 0.65, r <= 2 0.98; a node alone the same.  21 nodes, r = 4, T = 138 f32 (9 packs a
// segment) 151 -> 71 us, 16 nodes, r = 4, T = 100 h32 24.9 -> 15.6, r = 5, T = 216 bf16 52 -> 27.  Four rows for every r: r = 4 0.95 of that,
// r = 5 1.04.
template <class A, int VEC, int R1, int READS, bool TOGETHER, bool ANY>
__global__ __launch_bounds__(kBlock) void k_node_decode_reduce(
    const typename A::elem *__restrict__ V, const typename A::elem *__restrict__ X, typename A::elem *__restrict__ out,
    typename A::acc *__restrict__ part, const int64_t *__restrict__ red_ptr, const int64_t *__restrict__ red_row, const int32_t *__restrict__ list,
    const int32_t *__restrict__ list_packets, uint32_t own_rows,
    const int64_t *__restrict__ red_out, const int64_t *__restrict__ src_off, int r1_rt, uint32_t Lv, uint32_t ell,
    uint32_t W, double per_row, int m, int64_t file_stride, uint32_t tiles, int split, int64_t chunk_stride, uint32_t o_first,
    uint32_t o_step)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const int r1 = R1 > 0 ? R1 : r1_rt;
    const uint32_t tile = blockIdx.x % tiles;
    const uint32_t oc = blockIdx.x / tiles;
    const uint32_t oi = oc / split;
    const int s = (int)(oc - oi * split);
    const uint32_t o = o_first + oi * o_step;
    const uint32_t pack = tile * kBlock + threadIdx.x, rho = pack / Lv;
    uint32_t x = column<ANY, VEC>(pack - rho * Lv, ell);
    if (rho >= (uint32_t)r1 - 1 || rho * ell + x >= W) return;
    const uint32_t e = in_segment<ANY, VEC>(rho * ell, W, &x);
    const Rows rows = chunk_of(red_ptr, kMayBeListed<R1> ? list : nullptr, own_rows, o, s, split);
    typename O::Q acc = O::azero();
    int64_t i = rows.lo, hi = rows.hi;
    auto own = [&](int64_t row) { return load_at<READS == kAll, ANY, P, E>(V + (row >> 1) + e); };
    if constexpr (R1 > 0) {
        constexpr int AHEAD = 4;
        for (; i + AHEAD <= hi; i += AHEAD) {                    // the files the node stores come first
            if (red_row[i + AHEAD - 1] & 1) break;
            P v[AHEAD];
#pragma unroll
            for (int t = 0; t < AHEAD; t++) v[t] = own(red_row[i + t]);
#pragma unroll
            for (int t = 0; t < AHEAD; t++) acc = O::accum(acc, v[t]);
        }
    }
    for (; i < hi && !(red_row[i] & 1); i++) acc = O::accum(acc, own(red_row[i]));
    // (one loop for both kinds of lists: two take a quarter to a half more registers here)
    const bool listed = kMayBeListed<R1> && list;
    if (listed) i = rows.first, hi = rows.last;
    auto packet = [&](int64_t at) {
        return listed ? packet_at<true>(red_row, list_packets, at, per_row) : packet_at<false>(red_row, list_packets, at, per_row);
    };
    if constexpr (R1 > 0) {
        constexpr int AHEAD = R1 <= 4 ? 4 : 2, r = R1 - 1;
        for (; i < hi; i += AHEAD) {
            P coded[AHEAD], side[AHEAD][r > 1 ? r - 1 : 1];      // side: of the members that are neither sender nor receiver
            int from[AHEAD];
            auto position = [&](int t, int q) { return (from[t] - (q < (int)rho ? 1 : 0)) * ell + x; };
#pragma unroll
            for (int t = 0; t < AHEAD; t++) {                    // past the list's end the last row stands in and is not used
                const uint32_t pk = packet(i + t < hi ? i + t : hi - 1), u = pk / R1;
                const int b = (int)(pk - u * R1);
                from[t] = (int)rho < b ? (int)rho : (int)rho + 1;
                coded[t] = load_at<READS != kPast, ANY, P, E>(X + ((size_t)u * R1 + from[t]) * ell + x);
                // Of the members other than the receiver, whose batches it stores, the sender is the rho-th.  Its own batch is not
                // one of them and is not read.
                int64_t stored[r];
#pragma unroll
                for (int j = 0; j < r; j++) stored[j] = src_off[(size_t)u * R1 + (j < b ? j : j + 1)];
#pragma unroll
                for (int q = 0; q < r - 1; q++) {
                    const uint32_t pos = position(t, q);
                    const int64_t src = q < (int)rho ? stored[q] : stored[q + 1];
                    side[t][q] = packet_pack<O, READS == kAll, false, ANY>(V + src, pos < W ? pos : 0, W, 1, 0);
                }
            }
#pragma unroll
            for (int t = 0; t < AHEAD; t++) {
                if (i + t >= hi) break;
                P d = coded[t];
#pragma unroll
                for (int q = 0; q < r - 1; q++) d = O::select(position(t, q) < W, O::uncode(d, side[t][q]), d);
                acc = O::accum(acc, d);
            }
        }
    } else {
        for (; i < hi; i++) {
            const uint32_t pk = packet(i), u = pk / r1;
            const int b = (int)(pk - u * r1);
            const int a = (int)rho < b ? (int)rho : (int)rho + 1;
            const int64_t *src = src_off + (size_t)u * r1;
            P d = load_at<READS != kPast, ANY, P, E>(X + ((size_t)u * r1 + a) * ell + x);
            for (int b2 = 0; b2 < r1; b2++) {
                if (b2 == a || b2 == b) continue;
                const uint32_t pos = segment_rank(a, b2) * ell + x;
                if (pos < W) d = O::uncode(d, packet_pack<O, READS == kAll, TOGETHER, ANY>(V + src[b2], pos, W, m, file_stride));
            }
            acc = O::accum(acc, d);
        }
    }
    if (split > 1) store_at<false, ANY, typename O::Q, typename A::acc>(part + (int64_t)s * chunk_stride + red_out[o] + e, acc);
    else store_at<false, ANY, P, E>(out + red_out[o] + e, O::narrow(acc));
}

// The same two, with a wavefront on 64 consecutive packs of ONE segment: sender, receiver, batch
// rows and segment are then the same for all lanes, so the index tables are read with scalar
// loads, nothing is divided per lane and the packs of several rows are asked for before the first
// is used.  The lane-packed kernels above spend more time on addresses and on waiting for one row
// after the other than on data.  A pass of both calls, lane-packed -> this: 16 nodes r = 3 T = 4096
// h32 107 -> 98 us (most of it cache traffic: every V pack is read by up to r nodes), 16 nodes r = 4
// T = 512 f32 113 -> 57, 12 nodes r = 3 T = 3000 bf16 with two files a batch 60 -> 38, 20 nodes r = 2
// T = 352 h32 64 -> 18 (there the chunk sums, added by one thread per output before, were most).
// The lane-packed kernels stay for segments that would leave over a quarter of the lanes idle.
constexpr int kWaves = kBlock / kWave;

// FILES: the files of a batch, one, several in turn or together.
enum Files { kOneFile, kInTurn, kTogether };

template <class A, int VEC, int R1, int FILES, int READS, bool ANY>
__global__ __launch_bounds__(kBlock) void k_node_encode_wave(const typename A::elem *__restrict__ V,
                                                             typename A::elem *__restrict__ X,
                                                             const int64_t *__restrict__ src_off,
                                                             const int32_t *__restrict__ rows, uint32_t Lv, uint32_t ell,
                                                             uint32_t W, int m, int64_t file_stride, uint32_t tiles,
                                                             uint32_t units)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    const uint32_t unit = blockIdx.x * kWaves + wave_uniform(threadIdx.x / kWave);
    if (unit >= units) return;
    const uint32_t j = unit / tiles, pack = (unit - j * tiles) * kWave + threadIdx.x % kWave;
    if (pack >= Lv) return;
    const uint32_t x = column<ANY, VEC>(pack, ell);
    const uint32_t i = rows ? (uint32_t)rows[j] : j;
    const uint32_t u = i / R1;
    const int a = (int)(i - u * R1);
    const int64_t *src = src_off + (size_t)u * R1;
    P part[R1 - 1];
    if constexpr (FILES == kTogether && packets_together<O, R1 - 1>()) {
        const E *at[R1 - 1];
        bool there[R1 - 1];
#pragma unroll
        for (int k = 0; k < R1 - 1; k++) {
            const int b = k + (k >= a ? 1 : 0);
            const uint32_t pos = segment_rank(a, b) * ell + x;
            there[k] = pos < W;
            at[k] = V + src[b] + (there[k] ? pos : 0);
        }
        sum_packets<O, READS == kAll>(part, at, there, m, file_stride);
    } else {
#pragma unroll
        for (int k = 0; k < R1 - 1; k++) {
            const int b = k + (k >= a ? 1 : 0);
            const uint32_t pos = segment_rank(a, b) * ell + x;
            part[k] = O::zero();
            if (ANY || pos < W) part[k] = packet_pack<O, READS == kAll, FILES == kTogether, ANY>(V + src[b], pos, W, FILES == kOneFile ? 1 : m, file_stride);
        }
    }
    P coded = O::zero();
#pragma unroll
    for (int k = 0; k < R1 - 1; k++) coded = O::code(coded, part[k]);
    store_at<true, ANY, P, E>(X + (size_t)i * ell + x, coded);
}

// How the units are numbered.
enum Numbering {
    kByOutput,                        // ((output block, chunk), segment, tile), as workgroups are handed out
    kByTile,                          // (tile, ((chunk, output block), segment)), an XCD on a contiguous range: neighbours_share()
    kByChunk,                         // (chunk, (output block, segment, tile)), an XCD on a contiguous range: lists_by_round()
};

template <class A, int VEC, int R1, int FILES, int READS, int NUMBERING, bool ANY>
__global__ __launch_bounds__(kBlock) void k_node_decode_reduce_wave(
    const typename A::elem *__restrict__ V, const typename A::elem *__restrict__ X, typename A::elem *__restrict__ out,
    typename A::acc *__restrict__ part, const int64_t *__restrict__ red_ptr, const int64_t *__restrict__ red_row, const int32_t *__restrict__ list,
    const int32_t *__restrict__ list_packets, uint32_t own_rows,
    const int64_t *__restrict__ red_out, const int64_t *__restrict__ src_off, uint32_t Lv, uint32_t ell, uint32_t W,
    double per_row, int m, int64_t file_stride, uint32_t tiles, int split, int64_t chunk_stride, uint32_t o_first,
    uint32_t o_step, uint32_t units)
{
    using E = typename A::elem;
    using O = Ops<A, VEC>;
    using P = typename O::P;
    constexpr int r = R1 - 1;
    constexpr int AHEAD = FILES != kOneFile ? 1 : (R1 <= 3 ? 4 : 2);     // received packets asked for together
    const uint32_t unit = (NUMBERING == kByOutput ? blockIdx.x : xcd_contiguous(blockIdx.x, gridDim.x)) * kWaves + wave_uniform(threadIdx.x / kWave);
    if (unit >= units) return;
    uint32_t tile, oi;
    int rho, s;
    if constexpr (NUMBERING == kByChunk) {
        const uint32_t per_chunk = units / split, in = unit % per_chunk, seg = in / tiles;
        s = (int)(unit / per_chunk);
        tile = in - seg * tiles;
        oi = seg / r;
        rho = (int)(seg - oi * r);
    } else if constexpr (NUMBERING == kByTile) {
        const uint32_t per_tile = units / tiles, blocks = per_tile / (r * split);
        tile = unit / per_tile;
        const uint32_t seg = unit - tile * per_tile, oc = seg / r;
        rho = (int)(seg - oc * r);
        s = (int)(oc / blocks);
        oi = oc - s * blocks;
    } else {
        const uint32_t seg = unit / tiles, oc = seg / r;
        rho = (int)(seg - oc * r);
        tile = unit - seg * tiles;
        oi = oc / split;
        s = (int)(oc - oi * split);
    }
    const uint32_t pack = tile * kWave + threadIdx.x % kWave;
    const uint32_t o = o_first + oi * o_step;
    uint32_t x = column<ANY, VEC>(pack, ell);
    if (pack >= Lv || rho * ell + x >= W) return;
    const uint32_t e = in_segment<ANY, VEC>(rho * ell, W, &x);
    const Rows rows = chunk_of(red_ptr, kMayBeListed<R1> ? list : nullptr, own_rows, o, s, split);
    typename O::Q acc = O::azero();
    int64_t i = rows.lo, hi = rows.hi;
    // the files the node stores come first in the list
    auto own = [&](int64_t row) { return load_at<READS == kAll, ANY, P, E>(V + (row >> 1) + e); };
    for (; i + 4 <= hi; i += 4) {
        const int64_t row[4] = {red_row[i], red_row[i + 1], red_row[i + 2], red_row[i + 3]};
        if (row[3] & 1) break;
        const P v[4] = {own(row[0]), own(row[1]), own(row[2]), own(row[3])};
#pragma unroll
        for (int t = 0; t < 4; t++) acc = O::accum(acc, v[t]);
    }
    for (; i < hi && !(red_row[i] & 1); i++) acc = O::accum(acc, own(red_row[i]));
    struct Packet {
        P coded, side[r > 1 ? r - 1 : 1];
    };
    auto load = [&](uint32_t pk, Packet &k) {
        const uint32_t u = pk / R1;
        const int b = (int)(pk - u * R1);
        const int a = rho < b ? rho : rho + 1;
        const int low = a < b ? a : b, high = a < b ? b : a;
        const int64_t *src = src_off + (size_t)u * R1;
        k.coded = load_at<READS != kPast, ANY, P, E>(X + ((size_t)u * R1 + a) * ell + x);
        auto position = [&](int q, int &b2) {                // of the q-th member that is neither a nor b
            b2 = q + (q >= low ? 1 : 0);
            b2 += b2 >= high ? 1 : 0;
            return segment_rank(a, b2) * ell + x;
        };
        if constexpr (FILES == kTogether && r > 2 && packets_together<O, r - 1>()) {
            const E *from[r - 1];
            bool there[r - 1];
#pragma unroll
            for (int q = 0; q < r - 1; q++) {
                int b2;
                const uint32_t pos = position(q, b2);
                there[q] = pos < W;
                from[q] = V + src[b2] + (there[q] ? pos : 0);
            }
            sum_packets<O, READS == kAll>(k.side, from, there, m, file_stride);
        } else {
#pragma unroll
            for (int q = 0; q < r - 1; q++) {
                int b2;
                const uint32_t pos = position(q, b2);
                k.side[q] = O::zero();
                if (ANY || pos < W) k.side[q] = packet_pack<O, READS == kAll, FILES == kTogether, ANY>(V + src[b2], pos, W, FILES == kOneFile ? 1 : m, file_stride);
            }
        }
    };
    auto use = [&](const Packet &k) {
        P d = k.coded;
#pragma unroll
        for (int q = 0; q < r - 1; q++) d = O::uncode(d, k.side[q]);
        acc = O::accum(acc, d);
    };
    auto received = [&](auto listed) {
        if constexpr (decltype(listed)::value) i = rows.first, hi = rows.last;
        for (; i + AHEAD <= hi; i += AHEAD) {
            Packet k[AHEAD];
#pragma unroll
            for (int t = 0; t < AHEAD; t++) load(packet_at<decltype(listed)::value>(red_row, list_packets, i + t, per_row), k[t]);
#pragma unroll
            for (int t = 0; t < AHEAD; t++) use(k[t]);
        }
        for (; i < hi; i++) {
            Packet k;
            load(packet_at<decltype(listed)::value>(red_row, list_packets, i, per_row), k);
            use(k);
        }
    };
    by_list<kMayBeListed<R1>>(list, received);
    if (split > 1) store_at<false, ANY, typename O::Q, typename A::acc>(part + (int64_t)s * chunk_stride + red_out[o] + e, acc);
    else store_at<false, ANY, P, E>(out + red_out[o] + e, O::narrow(acc));
}

// Adds the chunk sums of one node's output blocks, in k_reduce_final's order for the same G, so
// that a node's outputs do not depend on whether it was run alone.
template <class A, int VEC>
__global__ __launch_bounds__(kBlock) void k_node_final(const typename A::acc *__restrict__ part,
                                                       typename A::elem *__restrict__ Phi,
                                                       const int64_t *__restrict__ red_out, uint32_t Wv, int split,
                                                       int64_t chunk_stride, uint32_t o_first, uint32_t o_step,
                                                       uint32_t items, int G)
{
    using O = Ops<A, VEC>;
    using Q = typename O::Q;
    __shared__ Q sums[kBlock];
    const int per_block = kBlock / G;
    const int at = threadIdx.x % per_block, g = threadIdx.x / per_block;
    const uint32_t idx = blockIdx.x * per_block + at;
    const uint32_t oi = idx / Wv, e = idx - oi * Wv;
    const int64_t base = idx < items ? red_out[o_first + oi * o_step] : 0;
    Q acc = O::azero();
    if (idx < items) {
#pragma unroll 4
        for (int s = g; s < split; s += G)
            acc = O::add(acc, reinterpret_cast<const Q *>(part + (int64_t)s * chunk_stride + base)[e]);
    }
    sums[threadIdx.x] = acc;
    __syncthreads();
    if (g == 0 && idx < items) {
        for (int k = 1; k < G; k++) acc = O::add(acc, sums[k * per_block + at]);
        reinterpret_cast<typename O::P *>(Phi + base)[e] = O::narrow(acc);
    }
}

// Calls launch(r+1, files of a batch) with both as compile-time constants, r <= 5.
template <class O, bool ANY, class F>
void by_shape(const ccdc_plan_t *p, bool together, F launch)
{
    auto files = [&](auto r1) {
        if (p->m == 1) return launch(r1, std::integral_constant<int, kOneFile>());
        by_files<O, ANY>(together, [&](auto t) { launch(r1, std::integral_constant<int, decltype(t)::value ? kTogether : kInTurn>()); });
    };
    switch (p->r) {
    case 1: files(std::integral_constant<int, 2>()); break;
    case 2: files(std::integral_constant<int, 3>()); break;
    case 3: files(std::integral_constant<int, 4>()); break;
    case 4: files(std::integral_constant<int, 5>()); break;
    default: files(std::integral_constant<int, 6>()); break;
    }
}

// Whether V and X are read through the caches.  A call for one node reads each value once; one for all nodes reads a coded
// packet r times and a value that is side information r - 1 times, a job's nodes after each other.  All of it with
// ordinary loads up to a size of a job's values that grows with r - 1 (kKeptNodeBytes is the last-level cache's size), where
// both ways measure the same.  Beyond it V goes past the caches; the coded packets stay.  A pass of both calls in us,
// everything kept / V past the caches / everything past them:
//   r = 2, 8 nodes f32    179 MB of values 95 / 95 / 97, 358 MB 179 / 172 / 181, 717 MB 360 / 329 / 353, 2.9 GB 1455 / 1357 / 1390
//   r = 3, 10 nodes f32   115 MB 69 / 74 / 77, 461 MB 257 / 259 / 276, 922 MB 499 / 479 / 505, 1.8 GB 1044 / 956 / 1021
//   r = 5, 9 nodes f32    186 MB 90 / 120 / 116, 743 MB 347 / 361 / 379, 1.0 GB 533 / 531 / 567, 1.5 GB 812 / 747 / 798
//   15 jobs, r = 3, 6 nodes u32, 1.2 GB (77 MB a job) 463 / 495 / 528
// With r = 1 nothing is read twice: 12 nodes f32, 35 MB 35 / 38 / 39, 72 MB 51 / 50 / 49, 288 MB 154 / 154 / 150, 1.2 GB
// 576 / 571 / 547.  One-element packs and the lane-packed kernels share lines with their neighbours and gain nothing past the
// caches (8 nodes, r = 4, T = 1024001 f32 1343 / 1335 / 1455; 24 nodes, r = 4, T = 200 f32 248 / 300 / 300; the first, like the
// 24 nodes below, is read in packs at any element since, and one-element packs are segments of under 32 of those).
//   One node, its two calls for every node of the cluster in turn, everything kept / everything past: 6 nodes, r = 3, ten files
// a batch, h32: 96 MB 343 / 495, 480 MB 662 / 702; 8 nodes, r = 6, f32: 358 MB 329 / 375, 1.4 GB 665 / 619; 10 nodes, r = 3,
// f32, 1.8 GB 1130 / 994; 24 nodes, r = 4, T = 2047 f32 (2.1 GB, one-element packs) 17580 / 14570.
//   Decoding by rounds, where a value's readers run together, gains through the caches also far beyond that: 28 inputs of 1.0 to 2.0 GB
// 0.79 of the time that they take past them in equal cuts (kReadTogether times the limit: all that fit the device).
constexpr double kReadTogether = 64;
template <int VEC>
Reads node_reads(const ccdc_plan_t *p, int node, bool by_wavefront, bool by_round = false)
{
    const double values = moved_bytes(p, 0);
    if (node >= 0) return values <= kKeptOneNodeBytes ? kAll : kPast;
    if (!by_wavefront || VEC == 1) return kAll;
    if (p->r == 1) return values <= kKeptStageBytes ? kAll : kPast;
    return values / p->J <= (p->r - 1) * kKeptNodeBytes * (by_round ? kReadTogether : 1) ? kAll : kCoded;
}

// Calls launch(reads) with that as a compile-time constant.  CODED: whether kCoded is one of the answers there are.
template <bool CODED, class F>
void by_node_reads(Reads reads, F launch)
{
    if (reads == kAll) return launch(std::integral_constant<int, kAll>());
    if constexpr (CODED) {
        if (reads == kCoded) return launch(std::integral_constant<int, kCoded>());
    }
    launch(std::integral_constant<int, kPast>());
}

template <class A, int VEC, bool ANY>
int run_node_encode(const ccdc_plan_t *p, int node, const void *V, void *X, hipStream_t st)
{
    using E = typename A::elem;
    const uint32_t Lv = cdiv(p->ell, VEC), ell = (uint32_t)p->ell, W = (uint32_t)p->W;
    const int64_t rows = node < 0 ? p->nrows : p->rows_per_node;
    const uint64_t items = (uint64_t)rows * Lv;
    if (items == 0) return CCDC_OK;
    if (!fits_rows<VEC, ANY>(rows, ell)) return CCDC_ESIZE;
    const int32_t *list = node < 0 ? nullptr : p->d_node_rows + (size_t)node * p->rows_per_node;
    const uint32_t wave_tiles = cdiv(Lv, kWave);
    const uint64_t units = (uint64_t)rows * wave_tiles;
    if (p->r <= 5 && fills_wavefronts(Lv) && fits_launch(units + kWaves)) {
        auto launch = [&](auto r1, auto files) {
            constexpr int R1 = decltype(r1)::value;
            constexpr int FILES = decltype(files)::value;
            by_node_reads<false>(node_reads<VEC>(p, node, true), [&](auto reads) {
                k_node_encode_wave<A, VEC, R1, FILES, decltype(reads)::value, ANY><<<cdiv(units, kWaves), kBlock, 0, st>>>(
                    (const E *)V, (E *)X, p->d_src_off, list, Lv, ell, W, p->m, (int64_t)p->Q * p->T, wave_tiles,
                    (uint32_t)units);
            });
        };
        by_shape<Ops<A, VEC>, ANY>(p, true, launch);
        return launched();
    }
    by_node_reads<false>(node_reads<VEC>(p, node, false), [&](auto reads) {
        by_files<Ops<A, VEC>, ANY>(p->m > 2, [&](auto together) {
            k_node_encode<A, VEC, decltype(reads)::value, decltype(together)::value, ANY><<<cdiv(items, kBlock), kBlock, 0, st>>>(
                (const E *)V, (E *)X, p->d_src_off, list, (uint32_t)items, Lv, ell, W, p->r + 1, p->m, (int64_t)p->Q * p->T);
        });
    });
    return launched();
}

template <class A, int VEC, bool ANY>
int run_node_decode_reduce(const ccdc_plan_t *p, int node, const void *V, const void *X, void *Phi, hipStream_t st)
{
    using E = typename A::elem;
    using Acc = typename A::acc;
    const uint32_t Lv = cdiv(p->ell, VEC), ell = (uint32_t)p->ell, W = (uint32_t)p->W;
    // the packs of a row; one shorter than r whole segments has fewer than r * Lv (18 nodes, r = 3, two functions, T = 512 f32: 256, in
    // one tile 34.7 us, not 258, in two 41.6)
    const uint32_t tiles = cdiv((uint64_t)(W / ell) * Lv + cdiv(W % ell, VEC), kBlock);
    const int split = p->red_split;
    const bool by_round = p->d_node_list != nullptr;
    const int32_t *packets = by_round ? p->d_node_list + (size_t)p->nout * split + 1 : nullptr;
    const uint32_t own_rows = (uint32_t)(p->red_ptr[1] - p->red_ptr[0] - p->rows_per_node);      // of a node, one job
    const uint32_t count = node < 0 ? (uint32_t)p->nout : (uint32_t)p->J;
    const uint32_t o_first = node < 0 ? 0u : (uint32_t)node, o_step = node < 0 ? 1u : (uint32_t)p->K;
    const int64_t chunk_stride = (int64_t)p->J * p->Q * p->T;
    const uint64_t blocks = (uint64_t)count * split * tiles;
    if (!fits_launch(ANY ? (uint64_t)count * split * cdiv(W, kBlock) : blocks) || !fits_launch((uint64_t)chunk_stride / (ANY ? 1 : VEC))) return CCDC_ESIZE;
    WorkspaceOrder order(p, st, split > 1);
    const uint32_t wave_tiles = cdiv(Lv, kWave);
    const uint64_t units = (uint64_t)count * split * p->r * wave_tiles;
    if (p->r <= 5 && fills_wavefronts(Lv) && fits_launch(units + kWaves)) {
        auto launch = [&](auto r1, auto files) {
            constexpr int R1 = decltype(r1)::value;
            constexpr int FILES = decltype(files)::value;
            by_node_reads<(VEC > 1 && R1 > 2)>(node_reads<VEC>(p, node, true, by_round), [&](auto reads) {
                auto numbered = [&](auto numbering) {
                    k_node_decode_reduce_wave<A, VEC, R1, FILES, decltype(reads)::value, decltype(numbering)::value, ANY><<<cdiv(units, kWaves), kBlock, 0, st>>>(
                        (const E *)V, (const E *)X, (E *)Phi, (Acc *)p->d_workspace, p->d_red_ptr, p->d_red_row, p->d_node_list, packets, own_rows, p->d_red_out,
                        p->d_src_off, Lv, ell, W, 1.0 / (double)p->W, p->m, (int64_t)p->Q * p->T, wave_tiles, split, chunk_stride,
                        o_first, o_step, (uint32_t)units);
                };
                if constexpr (R1 > 3 && decltype(reads)::value == kAll) {
                    if (node < 0 && by_round) return numbered(std::integral_constant<int, kByChunk>());
                }
                if constexpr (VEC * sizeof(E) >= 16 && R1 > 2) {
                    if (node < 0 && neighbours_share(p, wave_tiles)) return numbered(std::integral_constant<int, kByTile>());
                }
                numbered(std::integral_constant<int, kByOutput>());
            });
        };
        by_shape<Ops<A, VEC>, ANY>(p, p->m > 2 || p->r > 2, launch);     // r = 2: one packet in the making, as in combine
    } else {
        by_node_reads<false>(node_reads<VEC>(p, node, false), [&](auto reads) {
            auto launch = [&](auto r1, auto together) {
                k_node_decode_reduce<A, VEC, decltype(r1)::value, decltype(reads)::value, decltype(together)::value, ANY><<<(uint32_t)blocks, kBlock, 0, st>>>(
                    (const E *)V, (const E *)X, (E *)Phi, (Acc *)p->d_workspace, p->d_red_ptr, p->d_red_row, p->d_node_list, packets, own_rows, p->d_red_out,
                    p->d_src_off, p->r + 1, Lv, ell, W, 1.0 / (double)p->W, p->m, (int64_t)p->Q * p->T, tiles, split, chunk_stride,
                    o_first, o_step);
            };
            if (p->m > 1 || p->r > 5)
                by_files<Ops<A, VEC>, ANY>(p->m > 2, [&](auto together) { launch(std::integral_constant<int, 0>(), together); });
            else if (p->r == 1) launch(std::integral_constant<int, 2>(), std::false_type());
            else if (p->r == 2) launch(std::integral_constant<int, 3>(), std::false_type());
            else if (p->r == 3) launch(std::integral_constant<int, 4>(), std::false_type());
            else if (p->r == 4) launch(std::integral_constant<int, 5>(), std::false_type());
            else launch(std::integral_constant<int, 6>(), std::false_type());
        });
    }
    int rc = launched();
    if (rc != CCDC_OK || split == 1) return rc;
    if (node < 0) return reduce_chunks<A, ANY ? 1 : VEC>(p, Phi, split, chunk_stride, st);    // every block: Phi from end to end, as in ccdc_reduce
    constexpr int PACK = ANY ? 1 : VEC;
    const uint32_t Wv = W / PACK;
    const uint64_t items = (uint64_t)count * Wv;
    const int G = reduce_final_groups(chunk_stride / PACK, split);
    k_node_final<A, PACK><<<cdiv(items, kBlock / G), kBlock, 0, st>>>((const Acc *)p->d_workspace, (E *)Phi, p->d_red_out, Wv, split,
                                                                       chunk_stride, o_first, o_step, (uint32_t)items, G);
    return launched();
}

}  // namespace

namespace ccdc {

// The calls for one algebra, at a pack width that pick_wide() gives.
template <class A>
int node_encode(const ccdc_plan_t *p, int vec, bool any, int node, const void *V, void *X, hipStream_t st)
{
    constexpr int MOST = 16 / sizeof(typename A::elem);
    if (any) return run_node_encode<A, MOST, true>(p, node, V, X, st);
    if (vec == MOST) return run_node_encode<A, MOST, false>(p, node, V, X, st);
    return vec == 4 ? run_node_encode<A, 4, false>(p, node, V, X, st) : run_node_encode<A, 1, false>(p, node, V, X, st);
}

template <class A>
int node_decode_reduce(const ccdc_plan_t *p, int vec, bool any, int node, const void *V, const void *X, void *Phi, hipStream_t st)
{
    constexpr int MOST = 16 / sizeof(typename A::elem);
    if (any) return run_node_decode_reduce<A, MOST, true>(p, node, V, X, Phi, st);
    if (vec == MOST) return run_node_decode_reduce<A, MOST, false>(p, node, V, X, Phi, st);
    return vec == 4 ? run_node_decode_reduce<A, 4, false>(p, node, V, X, Phi, st) : run_node_decode_reduce<A, 1, false>(p, node, V, X, Phi, st);
}

// Compiled in five pieces, one for each algebra, the first with the entry points.
#ifdef CCDC_NODE_PART
#define CCDC_NODE(A)                                                                                 \
    template int node_encode<A>(const ccdc_plan_t *, int, bool, int, const void *, void *, hipStream_t); \
    template int node_decode_reduce<A>(const ccdc_plan_t *, int, bool, int, const void *, const void *, void *, hipStream_t)
#define CCDC_ELSEWHERE(A)                                                                                   \
    extern template int node_encode<A>(const ccdc_plan_t *, int, bool, int, const void *, void *, hipStream_t); \
    extern template int node_decode_reduce<A>(const ccdc_plan_t *, int, bool, int, const void *, const void *, void *, hipStream_t)
#if CCDC_NODE_PART == 0
CCDC_NODE(SumF32);
CCDC_ELSEWHERE(XorU32);
CCDC_ELSEWHERE(HybF32);
CCDC_ELSEWHERE(HybBF16);
CCDC_ELSEWHERE(HybF16);
#elif CCDC_NODE_PART == 1
CCDC_NODE(XorU32);
#elif CCDC_NODE_PART == 2
CCDC_NODE(HybF32);
#elif CCDC_NODE_PART == 3
CCDC_NODE(HybBF16);
#else
CCDC_NODE(HybF16);
#endif
#endif

}  // namespace ccdc

#if !defined(CCDC_NODE_PART) || CCDC_NODE_PART == 0
namespace {

int node_ready(const ccdc_plan_t *plan, int node)
{
    const int rc = ready(plan);
    if (rc != CCDC_OK) return rc;
    if (plan->compression) return CCDC_ESTATE;       // nothing is coded in that scheme
    if (node < -1 || node >= plan->K) return CCDC_EINVAL;
    return CCDC_OK;
}

}  // namespace

extern "C" {

int ccdc_node_encode(const ccdc_plan_t *plan, int node, const void *V, void *X, void *stream)
{
    int rc = node_ready(plan, node), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if ((rc = pick_wide(plan, Call::node_encode, node, &vec, &any, V, (const void *)X)) != CCDC_OK) return rc;
    if (!any) narrow_files(plan, plan->m, node < 0 ? plan->nrows : plan->rows_per_node, plan->ell, &vec);
    hipStream_t st = (hipStream_t)stream;
    switch (plan->mode) {
    case CCDC_F32_SUM: return node_encode<SumF32>(plan, vec, any, node, V, X, st);
    case CCDC_F32_SUM_XOR: return node_encode<HybF32>(plan, vec, any, node, V, X, st);
    case CCDC_BF16_SUM_XOR: return node_encode<HybBF16>(plan, vec, any, node, V, X, st);
    case CCDC_F16_SUM_XOR: return node_encode<HybF16>(plan, vec, any, node, V, X, st);
    default: return node_encode<XorU32>(plan, vec, any, node, V, X, st);
    }
}

int ccdc_node_decode_reduce(const ccdc_plan_t *plan, int node, const void *V, const void *X, void *Phi, void *stream)
{
    int rc = node_ready(plan, node), vec = 1;
    bool any = false;
    if (rc != CCDC_OK) return rc;
    if ((rc = pick_wide(plan, Call::node_decode, node, &vec, &any, V, X, (const void *)Phi)) != CCDC_OK) return rc;
    if (plan->node_waves > 0) return receive_coded(plan, node, V, X, Phi, stream);
    hipStream_t st = (hipStream_t)stream;
    switch (plan->mode) {
    case CCDC_F32_SUM: return node_decode_reduce<SumF32>(plan, vec, any, node, V, X, Phi, st);
    case CCDC_F32_SUM_XOR: return node_decode_reduce<HybF32>(plan, vec, any, node, V, X, Phi, st);
    case CCDC_BF16_SUM_XOR: return node_decode_reduce<HybBF16>(plan, vec, any, node, V, X, Phi, st);
    case CCDC_F16_SUM_XOR: return node_decode_reduce<HybF16>(plan, vec, any, node, V, X, Phi, st);
    default: return node_decode_reduce<XorU32>(plan, vec, any, node, V, X, Phi, st);
    }
}

}  // extern "C"
#endif
