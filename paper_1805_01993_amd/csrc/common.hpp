// Shared by the kernel translation units: algebras, packs, launch helpers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ccdc.h"
#include "plan.hpp"

namespace ccdc {

// ----------------------------------------------------------------- algebras
// elem: what V, Vbar, X, D and Phi hold.  acc: what sums are carried in.
// widen / add / narrow: pre-combining and the final reduction (a sum is
// narrowed once, when it is stored as an elem).  next_file: add, for the files of a
// batch.  code / uncode: forming a coded
// packet and cancelling side information from it.  fixed_order: the bits of a
// pre-combined packet are part of the result (they are XOR-coded), so every
// kernel adds a batch's files in ascending order.
struct SumF32 {                       // real numbers throughout
    using elem = float;
    using acc = float;
    static constexpr bool fixed_order = false;
    static __device__ __forceinline__ elem zero() { return 0.0f; }
    static __device__ __forceinline__ acc azero() { return 0.0f; }
    static __device__ __forceinline__ acc identity() { return -0.0f; }
    static __device__ __forceinline__ acc widen(elem a) { return a; }
    static __device__ __forceinline__ elem narrow(acc a) { return a; }
    static __device__ __forceinline__ acc add(acc a, acc b) { return a + b; }
    static __device__ __forceinline__ acc next_file(acc a, acc b) { return a + b; }
    static __device__ __forceinline__ elem code(elem a, elem b) { return a + b; }
    static __device__ __forceinline__ elem uncode(elem a, elem b) { return a - b; }
    static __device__ __forceinline__ elem gradient(elem theta, elem data) { return theta - data; }
};
struct XorU32 {                       // the field F_{2^T} throughout
    using elem = uint32_t;
    using acc = uint32_t;
    static constexpr bool fixed_order = false;
    static __device__ __forceinline__ elem zero() { return 0u; }
    static __device__ __forceinline__ acc azero() { return 0u; }
    static __device__ __forceinline__ acc identity() { return 0u; }
    static __device__ __forceinline__ acc widen(elem a) { return a; }
    static __device__ __forceinline__ elem narrow(acc a) { return a; }
    static __device__ __forceinline__ acc add(acc a, acc b) { return a ^ b; }
    static __device__ __forceinline__ acc next_file(acc a, acc b) { return a ^ b; }
    static __device__ __forceinline__ elem code(elem a, elem b) { return a ^ b; }
    static __device__ __forceinline__ elem uncode(elem a, elem b) { return a ^ b; }
    static __device__ __forceinline__ elem gradient(elem theta, elem data) { return theta ^ data; }   // - is XOR in F_{2^T}
};
struct HybF32 {                       // numbers are summed, packets are XOR-coded bit patterns (Sec. II)
    using elem = float;
    using acc = float;
    static constexpr bool fixed_order = true;
    static __device__ __forceinline__ elem zero() { return 0.0f; }    // all-zero bits: also the XOR identity
    static __device__ __forceinline__ acc azero() { return 0.0f; }
    static __device__ __forceinline__ acc identity() { return -0.0f; }
    static __device__ __forceinline__ acc widen(elem a) { return a; }
    static __device__ __forceinline__ elem narrow(acc a) { return a; }
    static __device__ __forceinline__ acc add(acc a, acc b) { return a + b; }
    // Of two NaNs the addition hands on its first operand, and the compiler may exchange operands: a sum with two NaNs
    // of different patterns then differs from kernel to kernel, and a receiver that takes its own form of it out of a coded
    // packet is left with the difference of the two in place of another packet's number.  Here the sum so far comes first.
    static __device__ __forceinline__ acc next_file(acc a, acc b)
    {
#ifdef __HIP_DEVICE_COMPILE__
        acc sum;
        asm("v_add_f32 %0, %1, %2" : "=v"(sum) : "v"(a), "v"(b));
        return sum;
#else
        return a + b;
#endif
    }
    static __device__ __forceinline__ elem code(elem a, elem b)
    {
        return __uint_as_float(__float_as_uint(a) ^ __float_as_uint(b));
    }
    static __device__ __forceinline__ elem uncode(elem a, elem b) { return code(a, b); }
    static __device__ __forceinline__ elem gradient(elem theta, elem data) { return theta - data; }
};
// The same hybrid for 16-bit floating-point payloads: elements are bit patterns
// of bfloat16 (BF) or IEEE binary16 numbers, sums are carried in fp32 and
// rounded once, to nearest even, when stored.  A batch of one file is not a sum:
// its packet is the file's values as they are, pattern for pattern (every kernel
// copies in that case), so signalling or signed NaN patterns in the input pass
// through the coding untouched.
template <bool BF>
struct Hyb16 {
    using elem = uint16_t;
    using acc = float;
    static constexpr bool fixed_order = true;
    static __device__ __forceinline__ elem zero() { return 0; }
    static __device__ __forceinline__ acc azero() { return 0.0f; }
    static __device__ __forceinline__ acc identity() { return -0.0f; }
    static __device__ __forceinline__ acc widen(elem a)
    {
        if constexpr (BF) {
            return __uint_as_float((uint32_t)a << 16);
        } else {
            _Float16 h;
            __builtin_memcpy(&h, &a, 2);
            return (float)h;
        }
    }
    // A sum that is not a number is stored as the format's quiet NaN with a clear sign and
    // payload (0x7FC0 / 0x7E00), whatever NaN the additions produced.
    static __device__ __forceinline__ elem narrow(acc a)
    {
        if constexpr (BF) {
            if (a != a) return (elem)0x7FC0u;
#ifdef __HIP_DEVICE_COMPILE__
            // v_cvt_pk_bf16_f32 rounds to nearest even, subnormals and overflow to infinity included (all 2^32 patterns
            // compared with the integer form below).  The integer form's ten instructions an element kept the Map kernel
            // busy for half of its time: 28 files of 25.6 M bf16 values 532 us, as the 32-bit modes 505; with the
            // conversion 510.
            const __bf16 h = (__bf16)a;
            elem out;
            __builtin_memcpy(&out, &h, 2);
            return out;
#else
            // keep the upper 16 bits; round up when the dropped half is above the midpoint, or
            // on it with an odd kept part (the increment may carry into the exponent, up to infinity)
            const uint32_t b = __float_as_uint(a);
            const uint32_t kept = b >> 16, dropped = b & 0xFFFFu;
            return (elem)(kept + ((dropped > 0x8000u || (dropped == 0x8000u && (kept & 1u))) ? 1u : 0u));
#endif
        } else {
            if (a != a) return (elem)0x7E00u;
            const _Float16 h = (_Float16)a;              // the hardware conversion rounds to nearest even
            elem out;
            __builtin_memcpy(&out, &h, 2);
            return out;
        }
    }
    static __device__ __forceinline__ acc add(acc a, acc b) { return a + b; }
    static __device__ __forceinline__ acc next_file(acc a, acc b) { return a + b; }     // narrow() makes every NaN the same
    static __device__ __forceinline__ elem code(elem a, elem b) { return (elem)(a ^ b); }
    static __device__ __forceinline__ elem uncode(elem a, elem b) { return (elem)(a ^ b); }
    // the difference of the two values in fp32 (one rounding), rounded once more to the format
    static __device__ __forceinline__ elem gradient(elem theta, elem data) { return narrow(widen(theta) - widen(data)); }
};
using HybBF16 = Hyb16<true>;
using HybF16 = Hyb16<false>;

// VEC consecutive elements moved by one load/store.
template <class E, int VEC>
struct alignas(sizeof(E) * VEC) Pack {
    E v[VEC];
};

template <class A, int VEC>
struct Ops {
    using algebra = A;
    static constexpr int lanes = VEC;
    using P = Pack<typename A::elem, VEC>;       // as stored
    using Q = Pack<typename A::acc, VEC>;        // as summed
    static __device__ __forceinline__ P zero()
    {
        P z;
#pragma unroll
        for (int i = 0; i < VEC; i++) z.v[i] = A::zero();
        return z;
    }
    static __device__ __forceinline__ Q azero()
    {
        Q z;
#pragma unroll
        for (int i = 0; i < VEC; i++) z.v[i] = A::azero();
        return z;
    }
    static __device__ __forceinline__ Q identity()         // identity + a is a, pattern for pattern
    {
        Q z;
#pragma unroll
        for (int i = 0; i < VEC; i++) z.v[i] = A::identity();
        return z;
    }
    static __device__ __forceinline__ Q widen(P a)
    {
        Q q;
#pragma unroll
        for (int i = 0; i < VEC; i++) q.v[i] = A::widen(a.v[i]);
        return q;
    }
    static __device__ __forceinline__ P narrow(Q a)
    {
        P p;
#pragma unroll
        for (int i = 0; i < VEC; i++) p.v[i] = A::narrow(a.v[i]);
        return p;
    }
    static __device__ __forceinline__ Q add(Q a, Q b)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) a.v[i] = A::add(a.v[i], b.v[i]);
        return a;
    }
    static __device__ __forceinline__ Q accum(Q a, P b) { return add(a, widen(b)); }
    static __device__ __forceinline__ Q accum_file(Q a, P b)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) a.v[i] = A::next_file(a.v[i], A::widen(b.v[i]));
        return a;
    }
    static __device__ __forceinline__ P code(P a, P b)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) a.v[i] = A::code(a.v[i], b.v[i]);
        return a;
    }
    static __device__ __forceinline__ P uncode(P a, P b)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) a.v[i] = A::uncode(a.v[i], b.v[i]);
        return a;
    }
    static __device__ __forceinline__ P gradient(P theta, P data)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) theta.v[i] = A::gradient(theta.v[i], data.v[i]);
        return theta;
    }
    static __device__ __forceinline__ P select(bool c, P a, P b)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) a.v[i] = c ? a.v[i] : b.v[i];
        return a;
    }
};

// Streaming accesses: data that is read or written exactly once is marked
// non-temporal so that it does not displace anything worth keeping in cache.
#ifndef CCDC_STREAMING_HINTS
#define CCDC_STREAMING_HINTS 1
#endif
template <int BYTES>
struct Bits {                                       // 8 or 16 bytes: a vector of 32-bit words
    typedef uint32_t type __attribute__((ext_vector_type(BYTES / 4)));
};
template <>
struct Bits<4> {
    typedef uint32_t type;
};
template <>
struct Bits<2> {
    typedef uint16_t type;
};
template <class P>
__device__ __forceinline__ P load_stream(const void *p)
{
#if CCDC_STREAMING_HINTS
    using B = typename Bits<sizeof(P)>::type;
    const B b = __builtin_nontemporal_load(reinterpret_cast<const B *>(p));
    P out;
    __builtin_memcpy(&out, &b, sizeof(P));
    return out;
#else
    return *reinterpret_cast<const P *>(p);
#endif
}
template <class P>
__device__ __forceinline__ void store_stream(void *p, const P &v)
{
#if CCDC_STREAMING_HINTS
    using B = typename Bits<sizeof(P)>::type;
    B b;
    __builtin_memcpy(&b, &v, sizeof(P));
    __builtin_nontemporal_store(b, reinterpret_cast<B *>(p));
#else
    *reinterpret_cast<P *>(p) = v;
#endif
}

// The same for packs of E elements that are only aligned to E: global memory serves
// unaligned dwords and vectors of them in one instruction.
template <class P, class E>
struct AnyBits {
    typedef typename Bits<sizeof(P)>::type type __attribute__((aligned(sizeof(E))));
};
template <class P, class E>
__device__ __forceinline__ P load_stream_any(const void *p)
{
    using B = typename AnyBits<P, E>::type;
    const B b = __builtin_nontemporal_load(reinterpret_cast<const B *>(p));
    P out;
    __builtin_memcpy(&out, &b, sizeof(P));
    return out;
}
// Through the caches instead: KEPT loads are ordinary ones (see kKeptBytes).
template <bool KEPT, class P>
__device__ __forceinline__ P load_pack(const void *p)
{
    if constexpr (KEPT) return *reinterpret_cast<const P *>(p);
    else return load_stream<P>(p);
}
template <bool KEPT, class P, class E>
__device__ __forceinline__ P load_pack_any(const void *p)
{
    if constexpr (KEPT) {
        using B = typename AnyBits<P, E>::type;
        const B b = *reinterpret_cast<const B *>(p);
        P out;
        __builtin_memcpy(&out, &b, sizeof(P));
        return out;
    } else {
        return load_stream_any<P, E>(p);
    }
}

// ANY: aligned to its elements only.  (Told of whole packs the compiler keeps two 16-bit elements a register, else one.)
template <bool KEPT, bool ANY, class P, class E>
__device__ __forceinline__ P load_at(const void *p)
{
    if constexpr (ANY) return load_pack_any<KEPT, P, E>(p);
    else return load_pack<KEPT, P>(p);
}
template <class P, class E>
__device__ __forceinline__ void store_stream_any(void *p, const P &v)
{
    using B = typename AnyBits<P, E>::type;
    B b;
    __builtin_memcpy(&b, &v, sizeof(P));
    __builtin_nontemporal_store(b, reinterpret_cast<B *>(p));
}
template <class P, class E>
__device__ __forceinline__ void store_any(void *p, const P &v)
{
    using B = typename AnyBits<P, E>::type;
    B b;
    __builtin_memcpy(&b, &v, sizeof(P));
    *reinterpret_cast<B *>(p) = b;
}

template <bool STREAM, bool ANY, class P, class E>
__device__ __forceinline__ void store_at(void *p, const P &v)
{
    if constexpr (STREAM && ANY) store_stream_any<P, E>(p, v);
    else if constexpr (STREAM) store_stream(p, v);
    else if constexpr (ANY) store_any<P, E>(p, v);
    else *reinterpret_cast<P *>(p) = v;
}

// Packs of 16 bytes also where the value length or the pointers do not divide by them (ANY): rows then begin at any element, and
// one pack of a row may reach past its end.  Where whole rows are added, and along the columns of a segment, that pack is
// moved back to the last whole one, so two lanes make the same elements from the same numbers (column()); a pack
// of a packet's short last segment is made element by element (end_pack()).  One-element packs, which such calls were made of before,
// are as many instructions and addresses for an eighth or a quarter of the bytes.  916 calls alone of 100 plans of such lengths, 64 KB to 1.5
// GB, 0.80 of the time, from 10 MB on 0.68, five of them over 5 % slower: 18 nodes, r = 2, T = 56286 bf16 the four stages 931 -> 350 us, 70 jobs on 8 nodes,
// r = 3, four files, T = 105661 bf16 777 -> 477, 23 nodes, r = 2, T = 28754 f16 node-local 425 -> 185, 21 nodes, r = 3, T = 4282 f32 the stages 820 -> 529.
// With fewer packs than fill the chip the narrow ones stay, of which there are more lanes with less each to add (any_element(); uncoded, 19
// nodes, T = 4169 u32 12 and more files a packet 10.6 us, 28.7; 7 nodes, r = 5, eleven files, T = 5470 bf16 fused 5.3, 51).
template <bool ANY, int VEC>
__device__ __forceinline__ uint32_t column(uint32_t pack, uint32_t length)
{
    const uint32_t x = pack * VEC;
    return ANY && x + VEC > length ? length - VEC : x;
}

// The elements of a row (of the sums of `files` files' rows) from pos on, zeros past its end at W.
template <class O, class E>
__device__ __forceinline__ typename O::P end_pack(const E *row, uint32_t pos, uint32_t W, int files, int64_t file_stride)
{
    using A = typename O::algebra;
    typename O::P v = O::zero();
#pragma unroll
    for (int i = 0; i < O::lanes; i++) {
        if (pos + i >= W) continue;
        v.v[i] = row[pos + i];
        if (files > 1) {                                      // else not a sum: the value as it is
            typename A::acc sum = A::widen(v.v[i]);
            for (int f = 1; f < files; f++) sum = A::next_file(sum, A::widen(row[pos + i + f * file_stride]));
            v.v[i] = A::narrow(sum);
        }
    }
    return v;
}

// The pack from element pos on of the packet pre-combined from the batch whose first file's row this is; zeros past W.
template <class O, bool KEPT, bool TOGETHER, bool ANY, class E>
__device__ __forceinline__ typename O::P packet_pack(const E *row, uint32_t pos, uint32_t W, int files, int64_t file_stride);

// Writes the pack from element pos on of a row of W elements, as far as it lies in the row.
template <class O, bool STREAM, bool ANY, class E>
__device__ __forceinline__ void store_in_row(E *row, uint32_t pos, uint32_t W, const typename O::P &v)
{
    using P = typename O::P;
    if (ANY && pos + O::lanes > W) {
#pragma unroll
        for (int i = 0; i < O::lanes; i++)
            if (pos + i < W) row[pos + i] = v.v[i];
    } else if (pos < W) {
        store_at<STREAM, ANY, P, E>(row + pos, v);
    }
}

// Batches of several files.  Asked for one after the other, the files of a batch are as many waits; with packs of less than 16
// bytes, of which a wavefront has few bytes in flight, several files are asked for together.  Packs of 16 bytes stay with one
// at a time: past the caches that gives nothing (56 jobs on 8 nodes, r = 2, three files, T = 150000 u32 483 -> 491 us), and sums of
// eight elements take the registers of other wavefronts (12 nodes, r = 3, two files, T = 6000 f16, node-local decoding 33 -> 38).
// Two files alone stay too where they are a lane's only packs in flight: combine (6 nodes, r = 4, T = 634231 f32 129 -> 136,
// uncoded, 12 nodes, r = 1, T = 1278647 f32 548 -> 580) and the kernels of node.hip that pack lanes (17 nodes, r = 4, T = 99 h32 46 -> 56).  141 inputs of 20 MB to 2.5 GB: combine
// down to 0.60 of the time, the fused shuffle 0.42, node-local encoding 0.43, decoding 0.38 (9 nodes, r = 3, T = 36845 bf16, nine
// files, 0.61, 0.42, 0.45, 0.56).
template <class O, bool ANY = false>
constexpr bool files_together()
{
    return ANY || sizeof(typename O::P) < 16;
}

// Calls launch(together) with it as a compile-time constant.
template <class O, bool ANY = false, class F>
void by_files(bool together, F launch)
{
    if constexpr (files_together<O, ANY>()) {
        if (together) return launch(std::true_type());
    }
    launch(std::false_type());
}

// The sum of the same pack of `files` files, ascending: `first` is the first one's, at s.
template <class O, bool KEPT, bool TOGETHER, bool ANY, class E>
__device__ __forceinline__ typename O::Q sum_files(const typename O::P &first, const E *s, int files, int64_t file_stride)
{
    using P = typename O::P;
    typename O::Q acc = O::widen(first);
    int f = 1;
    if constexpr (TOGETHER) {
        for (; f + 4 <= files; f += 4) {
            P v[4];
#pragma unroll
            for (int t = 0; t < 4; t++) v[t] = load_at<KEPT, ANY, P, E>(s + (f + t) * file_stride);
#pragma unroll
            for (int t = 0; t < 4; t++) acc = O::accum_file(acc, v[t]);
        }
        if (f + 2 <= files) {
            const P v0 = load_at<KEPT, ANY, P, E>(s + f * file_stride), v1 = load_at<KEPT, ANY, P, E>(s + (f + 1) * file_stride);
            acc = O::accum_file(O::accum_file(acc, v0), v1);
            f += 2;
        }
    }
    for (; f < files; f++) acc = O::accum_file(acc, load_at<KEPT, ANY, P, E>(s + f * file_stride));
    return acc;
}

template <class O, bool KEPT, bool TOGETHER, bool ANY, class E>
__device__ __forceinline__ typename O::P packet_pack(const E *row, uint32_t pos, uint32_t W, int files, int64_t file_stride)
{
    using P = typename O::P;
    const uint32_t last = W - O::lanes;
    if (!ANY && pos >= W) return O::zero();
    const E *s = row + (ANY && pos > last ? last : pos);      // loads without a condition: they stay in flight together
    P v = load_at<KEPT, ANY, P, E>(s);
    if (files > 1) v = O::narrow(sum_files<O, KEPT, TOGETHER, ANY>(v, s, files, file_stride));      // a one-file batch is sent as it is
    if (ANY && pos > last) v = end_pack<O>(row, pos, W, files, file_stride);
    return v;
}

// Where the same file of N packets is asked for together: as far as the registers of their sums allow (beyond, wavefronts are
// lost: eight elements a pack, r = 4, 11 files 43 -> 56 us).
template <class O, int N>
constexpr bool packets_together()
{
    return files_together<O>() && N * sizeof(typename O::Q) / 4 <= 12;
}

// The same for the packs s[k] of N packets, narrowed, a file or two of all of them at a time; zeros where there is none (not
// valid[k]; s[k] can be read all the same).
template <class O, bool KEPT, int N, class E>
__device__ __forceinline__ void sum_packets(typename O::P (&v)[N], const E *const (&s)[N], const bool (&valid)[N], int files,
                                            int64_t file_stride)
{
    using P = typename O::P;
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = load_pack<KEPT, P>(s[k]);
    if (files > 1) {                                      // else not sums: the files' values as they are
        typename O::Q acc[N];
#pragma unroll
        for (int k = 0; k < N; k++) acc[k] = O::widen(v[k]);
        int f = 1;
        auto some = [&](auto count) {
            constexpr int C = decltype(count)::value;
            P w[C][N];
#pragma unroll
            for (int t = 0; t < C; t++)
#pragma unroll
                for (int k = 0; k < N; k++) w[t][k] = load_pack<KEPT, P>(s[k] + (f + t) * file_stride);
#pragma unroll
            for (int t = 0; t < C; t++)
#pragma unroll
                for (int k = 0; k < N; k++) acc[k] = O::accum_file(acc[k], w[t][k]);
            f += C;
        };
        if constexpr (N * sizeof(typename O::Q) / 4 <= 8) {
            while (f + 2 <= files) some(std::integral_constant<int, 2>());
        }
        while (f < files) some(std::integral_constant<int, 1>());
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = O::narrow(acc[k]);
    }
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = O::select(valid[k], v[k], O::zero());
}

// A value that is the same in all lanes of a wavefront, told to the compiler as such.
__device__ __forceinline__ uint32_t wave_uniform(uint32_t v)
{
#ifdef __HIP_DEVICE_COMPILE__
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
#else
    return v;
#endif
}

// A lane's 32-bit byte offset, made anew where it is used: the compiler then sees next to the
// access that it is 32 bits wide and adds it to the (uniform) row address in the access itself
// instead of in two registers a row.
__device__ __forceinline__ uint32_t lane_offset(uint32_t v)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(v));
#endif
    return v;
}

constexpr int kBlock = 256;
// Work items (and workgroups) of one launch are numbered in 32 bits.  ccdc_plan_bind checks the
// counts for the widest packs a shape allows; a call that has to fall back to narrower packs
// (pointers not aligned for the wide ones) has more items and checks again for itself.
constexpr uint64_t kMaxLaunchItems = 2147483647ull;
inline bool fits_launch(uint64_t items) { return items <= kMaxLaunchItems; }
// The same for `rows` rows of `length` elements in packs; packs at any element are limited as the one-element packs that their calls
// fall back to, whichever a call takes.
template <int VEC, bool ANY>
inline bool fits_rows(uint64_t rows, uint64_t length)
{
    return fits_launch(rows * ((length + VEC - 1) / VEC)) && (!ANY || fits_launch(rows * length));
}

// Which segment of packet b carries sender a's label: the rank of a among the members other than b.
__device__ __forceinline__ int segment_rank(int a, int b) { return a - (a > b ? 1 : 0); }

// Phi = sum over chunks of the per-chunk outputs part[split][chunk_packs].
// A workgroup owns kBlock/G consecutive packs; its G thread groups each add
// every G-th chunk (g, g+G, ...), then the G group sums are added in group
// order.  The order is fixed by (split, G), so results repeat run to run.
template <class A, int VEC>
__global__ __launch_bounds__(kBlock) void k_reduce_final(const typename A::acc *__restrict__ part,
                                                         typename A::elem *__restrict__ Phi, int split,
                                                         int64_t chunk_packs, uint32_t items, int G)
{
    using O = Ops<A, VEC>;
    using P = typename O::P;
    using Q = typename O::Q;
    __shared__ Q sums[kBlock];
    const int per_block = kBlock / G;                    // packs of this workgroup
    const int e = threadIdx.x % per_block, g = threadIdx.x / per_block;
    const uint32_t idx = blockIdx.x * per_block + e;
    Q acc = O::azero();
    if (idx < items) {
        const Q *src = reinterpret_cast<const Q *>(part) + idx;
#pragma unroll 4
        for (int s = g; s < split; s += G) acc = O::add(acc, src[(int64_t)s * chunk_packs]);
    }
    sums[threadIdx.x] = acc;
    __syncthreads();
    if (g == 0 && idx < items) {
        for (int k = 1; k < G; k++) acc = O::add(acc, sums[k * per_block + e]);
        reinterpret_cast<P *>(Phi)[idx] = O::narrow(acc);
    }
}

// Launch geometry of k_reduce_final: more thread groups when there are few packs.
inline int reduce_final_groups(int64_t items, int split)
{
    int G = 1;
    while (G < 16 && G * 2 <= split && items * G < (1 << 18)) G *= 2;
    return G;
}

// Sums of the wavefronts of one workgroup, every lane's acc: added in LDS (smem, 64 packs of sums a wavefront) in
// wavefront order; write(i, sum) gets element i of the 64 packs.
template <class A, int VEC, class F>
__device__ __forceinline__ void add_wavefronts(unsigned char *smem, const typename Ops<A, VEC>::Q &acc, uint32_t waves, F write)
{
    using Acc = typename A::acc;
    reinterpret_cast<typename Ops<A, VEC>::Q *>(smem)[threadIdx.x] = acc;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kGroupLanes * VEC; i += blockDim.x) {
        const Acc *parts = reinterpret_cast<const Acc *>(smem) + i;
        Acc v = parts[0];
        for (uint32_t g = 1; g < waves; g++) v = A::add(v, parts[g * kGroupLanes * VEC]);
        write(i, v);
    }
}

// ------------------------------------------------------------ host helpers
inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

inline int ready(const ccdc_plan_t *p)
{
    if (!p) return CCDC_EINVAL;
    if (!p->bound || !p->uploaded) return CCDC_ESTATE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return CCDC_EHIP;
    if (dev != p->device) return CCDC_ESTATE;
    return CCDC_OK;
}

// kKeptBytes, kKeptStageBytes: non-temporal loads pass the last-level cache (256 MB) by, ordinary ones leave the data
// there.  A call whose inputs and outputs take no more than this (ccdc_map: what it reads; V, as large again, is only written)
// therefore reads with ordinary loads: its inputs are then often still
// there from the call that made them.  Measured with three sets of buffers used in turn.  One-pass kernel, 8 nodes,
// r = 2, one file a batch, f32: 64 MB a pass 14.5 -> 12.6 us, 129 MB 24.1 -> 23.4, but 194 MB 43.1 -> 46.2 and 1 GB
// 190 -> 199.  The calls of single stages share the cache with what the other stages make: two functions a node,
// uncoded, 13 nodes, T = 780 u32 (17 MB of values) 23.5 -> 18.3 us, six nodes, T = 24256 u32 (50 MB a call) 33 -> 24,
// a step from files on 24 nodes (43 MB read) 47 -> 41, but the four stages at 87 MB a call (12 nodes, T = 6000 f16)
// 43.7 -> 46.4.

// Calls launch(kept) with that as a compile-time constant.  ALWAYS: only true is asked for.
template <bool ALWAYS, class F>
void by_reads(bool kept, F launch)
{
    if (ALWAYS || kept) launch(std::true_type());
    else if constexpr (!ALWAYS) launch(std::false_type());
}

// One-element packs mean rows that begin anywhere in a cache line, and neighbours that share lines.  ccdc_shuffle_fused and
// ccdc_reduce always keep the reads of those (a pass of both, past the caches -> kept: 56 jobs on 8 nodes, r = 2, T = 150001
// u32, 2.4 GB of values, 1162 -> 1140 us; 7 nodes, r = 2, T = 9001 f32 46.3 -> 43.8; reduce alone at most 1 % slower in a
// pass of the four stages), ccdc_combine while its packets take up to kKeptPacketBytes: beyond that, V in the caches pushes out
// the packets that the next call reads (the four stages, 9 nodes, r = 2, T = 150001 f32, 151 MB of packets, 311 -> 327; 10
// nodes, r = 3, T = 100001 bf16, 168 MB, 473 -> 490; but the uncoded scheme, 22 nodes, T = 85615 u32, 79 MB, 392 -> 383).
// For ccdc_map, which reads each line once, they are packs like others (62 MB and less 0.73 to 0.82 of the time, more
// 1.00 to 1.04).  The lengths in these figures were all read in one-element packs; since packs at any element the rules are left with segments
// of under 32 packs, with the fused shuffle of 32-bit values (r >= 3, or under 200 MB) and with what else any_element() says no to.

// Pack width (elements) for this call: 16 bytes when the value length, the
// segment length and every pointer allow it; for 2-byte elements else 8 bytes;
// else one element.
template <class... Ptr>
int pick_vec(const ccdc_plan_t *p, int *vec, Ptr... ptrs)
{
    const void *list[] = {ptrs...};
    const size_t eb = (size_t)elem_bytes(p->mode);
    bool a16 = true, a8 = true;
    for (const void *q : list) {
        if (!q) return CCDC_EINVAL;
        if (!aligned(q, eb)) return CCDC_EINVAL;
        a16 = a16 && aligned(q, 16);
        a8 = a8 && aligned(q, 8);
    }
    if (eb == 4) {
        *vec = (p->T % 4 == 0 && a16) ? 4 : 1;
    } else {
        if (p->T % 8 == 0 && p->ell % 8 == 0 && a16) *vec = 8;
        else if (p->T % 4 == 0 && a8) *vec = 4;
        else *vec = 1;
    }
    return CCDC_OK;
}

// The widest packs a call (of node `node`, -1 for all) can be made of: pick_vec()'s, or packs of 16 bytes at any element (*any), where
// those would be one-element packs and any_element() says so.
template <class... Ptr>
int pick_wide(const ccdc_plan_t *p, Call call, int node, int *vec, bool *any, Ptr... ptrs)
{
    const int rc = pick_vec(p, vec, ptrs...);
    *any = rc == CCDC_OK && *vec == 1 && any_element(p, call, node);
    if (*any) *vec = 16 / elem_bytes(p->mode);
    return rc;
}

// Batches of more than two files that make fewer than 128 thousand packs of 16 bytes (16 bits: 64) leave the chip short of lanes, each with the files of
// a packet to wait for one after the other: they take one-element packs, more lanes and files asked for together.  48 such calls of
// ccdc_combine, ccdc_shuffle_fused and ccdc_node_encode over 4 us 0.36 to 0.95 of the time (uncoded, 19 nodes, T = 4168 u32 28.7 -> 10.7 us; 7
// nodes, r = 5, eleven files, T = 5472 bf16 fused 23.3 -> 5.5); with up to 250 thousand packs 0.78 to 1.30, beyond 0.89 to 2.1.  In 16 bits, eight
// lanes for one, 64 to 128 thousand packs were 1.07, 0.84 (four of 11 over 5 % slower) and 1.06 of the time of the three (20 nodes, r = 3, two
// functions, nine files, T = 64 bf16 node-local sending 12.8 -> 19.5), half as many 0.90, 0.74 and 0.84.  (Not above what
// one-element packs can be numbered for, which is far beyond.)
inline void narrow_files(const ccdc_plan_t *p, int files, int64_t rows, int64_t length, int *vec)
{
    if (files > 2 && !makes_lanes(p, rows, length, elem_bytes(p->mode) == 2 ? 2 : 4)) *vec = 1;
}

inline int launched()
{
    return hipGetLastError() == hipSuccess ? CCDC_OK : CCDC_EHIP;
}

// The second kernel of a reduction of split lists: Phi from the chunk sums in the workspace.
template <class A, int VEC>
int reduce_chunks(const ccdc_plan_t *p, void *Phi, int split, int64_t chunk_stride, hipStream_t st)
{
    const uint64_t items = (uint64_t)chunk_stride / VEC;
    const int G = reduce_final_groups((int64_t)items, split);
    k_reduce_final<A, VEC><<<cdiv(items, kBlock / G), kBlock, 0, st>>>((const typename A::acc *)p->d_workspace, (typename A::elem *)Phi,
                                                                        split, chunk_stride / VEC, (uint32_t)items, G);
    return launched();
}

// The plan's workspace holds partial sums between the two kernels of one call.
// Calls that use it are put in order also when they come on different streams:
// the plan remembers the stream of the last such call, and a call that arrives
// on another stream first records the plan's event at the tail of that earlier
// stream and makes its own stream wait for it (so it waits for everything the
// earlier stream had been given, the earlier call included).  Calls that stay
// on one stream, the usual case, add no event and no wait.  Host threads take
// turns through the plan's mutex.  A stream under graph capture is left alone
// and forgotten (an event recorded outside a capture cannot be waited for
// inside one): whoever replays the graph keeps it apart from other users of
// the plan.  The earlier stream must still exist when the later call comes.
class WorkspaceOrder {
public:
    WorkspaceOrder(const ccdc_plan_t *p, hipStream_t st, bool uses_workspace)
        : p_(p), st_(st), on_(uses_workspace && p->ws_event != nullptr)
    {
        if (!on_) return;
        p_->ws_mutex.lock();
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st_, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
            (void)hipGetLastError();
            p_->ws_mutex.unlock();
            on_ = false;
            return;
        }
        if (p_->ws_used && p_->ws_stream != (void *)st_) {
            hipEvent_t ev = (hipEvent_t)p_->ws_event;
            hipStream_t earlier = (hipStream_t)p_->ws_stream;
            hipStreamCaptureStatus es = hipStreamCaptureStatusNone;       // nothing is recorded into someone's capture
            if (hipStreamIsCapturing(earlier, &es) != hipSuccess || es != hipStreamCaptureStatusNone ||
                hipEventRecord(ev, earlier) != hipSuccess || hipStreamWaitEvent(st_, ev, 0) != hipSuccess)
                (void)hipGetLastError();
        }
    }
    ~WorkspaceOrder()
    {
        if (!on_) return;
        p_->ws_used = true;
        p_->ws_stream = (void *)st_;
        p_->ws_mutex.unlock();
    }
    WorkspaceOrder(const WorkspaceOrder &) = delete;
    WorkspaceOrder &operator=(const WorkspaceOrder &) = delete;

private:
    const ccdc_plan_t *p_;
    hipStream_t st_;
    bool on_;
};

}  // namespace ccdc

// Dispatch on (payload mode, pack width): evaluates CALL with the algebra as type A, the pack width as constant VEC and
// whether packs may begin at any element as constant ANY, inside a function that has `using namespace ccdc`.
#define CCDC_DISPATCH_WIDTH(ALGEBRA, MOST, vec, any, CALL)                                    \
    do {                                                                                      \
        using A = ALGEBRA;                                                                    \
        if (any) { constexpr int VEC = MOST; constexpr bool ANY = true; return CALL; }        \
        constexpr bool ANY = false;                                                           \
        if ((vec) == MOST) { constexpr int VEC = MOST; return CALL; }                         \
        if ((vec) == 4) { constexpr int VEC = 4; return CALL; }                               \
        constexpr int VEC = 1;                                                                \
        return CALL;                                                                          \
    } while (0)
#define CCDC_DISPATCH(p, vec, any, CALL)                                                      \
    do {                                                                                      \
        switch ((p)->mode) {                                                                  \
        case CCDC_F32_SUM: CCDC_DISPATCH_WIDTH(SumF32, 4, vec, any, CALL);                    \
        case CCDC_F32_SUM_XOR: CCDC_DISPATCH_WIDTH(HybF32, 4, vec, any, CALL);                \
        case CCDC_BF16_SUM_XOR: CCDC_DISPATCH_WIDTH(HybBF16, 8, vec, any, CALL);              \
        case CCDC_F16_SUM_XOR: CCDC_DISPATCH_WIDTH(HybF16, 8, vec, any, CALL);                \
        default: CCDC_DISPATCH_WIDTH(XorU32, 4, vec, any, CALL);                              \
        }                                                                                     \
    } while (0)
