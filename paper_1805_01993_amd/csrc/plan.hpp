// Internal layout of a plan: host combinatorics, the bound segment schedule and
// the handles of the device tables.  Not part of the public interface.
#pragma once

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <vector>

#include "ccdc.h"

struct ccdc_plan_s {
    // problem (Sec. III): per job
    int K = 0, r = 0, Q = 0, N = 0;
    int J = 1;            // jobs
    int c = 0;            // Q / K functions per node
    int m = 0;            // files per batch
    bool paper_jobs = false;
    bool compression = false;           // uncoded comparison scheme (appendix): combine + reduce only
    int64_t nbatch = 0, nround = 0;
    int64_t nrows = 0;                  // packets: rows of Vbar and of D (nround*(r+1) for coded plans)

    // compression-only scheme: consecutive batches, node k stores batch k mod nbatch,
    // one uncoded packet per (receiver, batch it does not store)
    std::vector<int32_t> batch_first;   // [nbatch+1]
    std::vector<int32_t> node_batch;    // [K]
    std::vector<int32_t> pkt_recv, pkt_batch, pkt_send;   // [nrows]
    std::vector<int32_t> row_files;     // [nrows] files added into each packet (batches differ in size)

    // placement (Sec. IV-A) and rounds (Sec. IV-B)
    std::vector<int32_t> batch_job;     // [nbatch]
    std::vector<int32_t> batch_file0;   // [nbatch]
    std::vector<int32_t> batch_label;   // [nbatch][r]
    std::vector<int32_t> round_member;  // [nround][r+1]
    std::vector<int32_t> round_batch;   // [nround][r+1]
    std::vector<int32_t> node_rows;     // [K][rows_per_node] packets (u*(r+1)+a) that node k sends, ascending
    int64_t rows_per_node = 0;          // nrows / K: every node is in the same number of rounds
    std::vector<int32_t> file_nodes;    // [J*N][r] nodes storing file job*N+n, ascending (Sec. IV-A)
    std::vector<int32_t> node_files;    // [K][files_per_node] the sets M_k, ascending
    int64_t files_per_node = 0;         // r*J*N/K

    // fixed by ccdc_plan_bind
    bool bound = false;
    int64_t T = 0, W = 0, ell = 0;
    int mode = 0;
    std::vector<int64_t> packet_len;    // [r+1]
    int64_t scheduled = 0;              // elements on the wire

    // tables the kernels read (host copies)
    std::vector<int64_t> src_off;       // [nround][r+1] element offset in V of the served
                                        //   batch's first file, at the target's functions
    std::vector<int64_t> red_ptr;       // [nout+1] row-list bounds of each (job, node) output
    std::vector<int64_t> red_row;       // rows: (element offset << 1) | (1 = in D, 0 = in V)
    std::vector<int64_t> red_out;       // [nout] element offset of the output block in Phi
    int64_t nout = 0;                   // J * K output blocks of W elements
    std::vector<int32_t> node_list;     // the packets of ccdc_node_decode_reduce's lists where those are cut by rounds (else
                                        //   empty): [nout*red_split+1] bounds of the chunks, then packets u*(r+1)+b
    bool wide_lists = false;            // lists are summed in 16-byte packs at any element where rows do not divide by them
    int red_split = 1;                  // the row list of an output is summed in this many chunks
    int red_waves = 0;                  // > 0: ccdc_reduce sums it in one workgroup of that many wavefronts instead
    size_t red_workspace_bytes = 0;     // partial sums of the split reductions
    size_t workspace_bytes = 0;         // what those and the one-pass kernel's chunks need; exact once uploaded

    // whole path in one pass (single-job plans): the partial outputs of all K
    // nodes are accumulated in LDS, one private slot per (node, segment, lane)
    bool pipe_ok = false;               // shape supported by ccdc_pipeline_fused
    int pipe_max_chunks = 1;            // upper bound on round chunks
    int64_t pipe_local_rows = 0;        // rows of V every node adds from its own files
    std::vector<int64_t> loc_row;       // [K][pipe_local_rows] (element offset in V << 12) | node
    std::vector<int64_t> pipe_row;      // [nround][r+1] (src_off << 12) | member

    // device side, set by ccdc_plan_upload
    bool uploaded = false;
    int device = -1;
    int64_t *d_src_off = nullptr, *d_red_ptr = nullptr, *d_red_row = nullptr, *d_red_out = nullptr;
    int64_t *d_loc_row = nullptr, *d_pipe_row = nullptr;
    int32_t *d_node_list = nullptr;     // node_list empty: null
    int32_t *d_row_files = nullptr;     // null when every packet adds m files
    int32_t *d_node_rows = nullptr;
    void *d_workspace = nullptr;

    // launch geometry of the one-pass kernel on this device, fixed at upload time: elements of a
    // pack, wavefronts of a workgroup (they share a tile of columns) and chunks of rounds (0: by receiver, receive.hip)
    int pipe_vec = 1, pipe_waves = 1, pipe_chunks = 0;
    bool pipe_even = true;              // every wavefront takes a share of the rounds and one of the own rows
    bool pipe_shallow = false;          // one step of the rounds in flight (r = 1, several files a batch)

    // ccdc_node_decode_reduce by receiver: elements of a pack and wavefronts of a workgroup, 0 for its other kernels
    int node_vec = 1, node_waves = 0;

    // Order of the calls that use the workspace, across streams: the last such call
    // recorded ws_event (a hipEvent_t made by ccdc_plan_upload) on ws_stream.
    mutable std::mutex ws_mutex;
    mutable void *ws_event = nullptr;
    mutable void *ws_stream = nullptr;
    mutable bool ws_used = false;
};

namespace ccdc {

// Host-side construction; both return a ccdc_status.
int build_plan(int K, int r, int Q, int N, bool paper_jobs, int gamma, ccdc_plan_t **out);
int build_compression_plan(int K, int r, int Q, int N, ccdc_plan_t **out);
int bind_plan(ccdc_plan_t *p, int64_t T, int mode);

// Limits of the one-pass pipeline kernel.
constexpr int kPipeLanes = 64;                 // columns of a tile: one wavefront wide
constexpr int kPipeMaxWaves = 8;               // wavefronts of a workgroup
constexpr int kPipeMaxLds = 64 * 1024;         // bytes of LDS one wavefront may take
constexpr int kPipeGroupLds = 160 * 1024;      // bytes of LDS one workgroup may take: all that gfx950 has
constexpr int kCuLds = 160 * 1024;             // bytes of LDS of a compute unit
constexpr int kLdsGranule = 1280;              // bytes it is given out in
constexpr int kPipeMaxR1 = 6;                  // r+1 the kernel is unrolled for
constexpr int kReceiveMaxWaves = 16;           // wavefronts of a workgroup of the form for small inputs (receive.hip)
constexpr double kReceiveBytes = 24e6, kReceiveBytesR1 = 48e6;       // a pass of that form moves at most (r = 1: the second)
constexpr double kReceiveNodeBytes = 48e6;     // inputs and outputs of a node-local decoding of that form

// Reductions in one launch: 64 packs of an output a workgroup.
constexpr uint32_t kGroupLanes = 64;
constexpr uint32_t kGroupMaxWaves = 16;
constexpr int64_t kGroupsWanted = 128;         // a workgroup for every second compute unit

// Bytes up to which a call reads with ordinary loads (the rules that use them, with both sides measured, are in
// common.hpp, node.hip and pipeline.hip).  The CPU build of the kernels makes variables of them, to run either side on small inputs.
#ifdef CCDC_VARIABLE_READ_LIMITS
#define CCDC_READ_LIMIT inline double
#else
#define CCDC_READ_LIMIT constexpr double
#endif
CCDC_READ_LIMIT kKeptBytes = 128e6, kKeptStageBytes = 64e6, kKeptNodeBytes = 256e6, kKeptOneNodeBytes = 640e6;
CCDC_READ_LIMIT kKeptPacketBytes = 100e6, kKeptSharedBytes = 200e6;
CCDC_READ_LIMIT kKeptWideBytes = 1.4e9;        // from these on

// Packs of a segment from which on they may begin at any element, and the 16-byte packs that a call must make for it
// (any_element() and wide_lists() in plan.cpp).
CCDC_READ_LIMIT kAnyPacks = 32, kAnyLanes = 32e3, kAnyListPacks = 1 << 18, kAnyListBytes = 200e6;
CCDC_READ_LIMIT kUnequalChunks = 1.4, kUnequalFileChunks = 2;      // lists_by_round() in plan.cpp

// One-pass pipeline (pipeline.hip): fixes the launch geometry (pipe_vec .. pipe_shallow) for the current device.
void pipeline_prepare(ccdc_plan_t *p);
// Body of ccdc_pipeline_fused.  own_part = null: partial outputs of round chunks go
// to the plan's workspace; else to the caller's buffer of own_part_bytes bytes
// (CCDC_ESIZE when they do not fit).
int pipeline_entry(const ccdc_plan_t *plan, const void *V, void *X, void *Phi, void *stream, void *own_part,
                   size_t own_part_bytes);

// The form of the pass for small inputs, by receiver (receive.hip): a plan with pipe_chunks = 0 takes it.
struct ReceiveArgs {
    int first_node, nodes, m;
    uint32_t W, ell;                  // elements of a packet and of a segment
    uint32_t rounds, own;             // rounds a node is in, files it stores
    int64_t file_stride;
};
inline bool by_receiver(const ccdc_plan_t *p) { return p->pipe_chunks == 0; }
void receive_prepare(ccdc_plan_t *p, double one_pass_us);
void receive_node_prepare(ccdc_plan_t *p);
int receive_entry(const ccdc_plan_t *p, const void *V, void *X, void *Phi, void *stream);
int receive_coded(const ccdc_plan_t *p, int node, const void *V, const void *X, void *Phi, void *stream);

// Device address of the fixed scratch array of ccdc_pipeline_fused_noalloc on the
// current device (noalloc.hip); out may be null to only look it up ahead of time.
int scratch_address(void **out);

// Workgroups are handed to the 8 XCDs round-robin.  This numbers them so that each XCD gets a contiguous
// range of the work, behind its own L2.
constexpr uint32_t kXcds = 8;
constexpr uint32_t xcd_contiguous(uint32_t block, uint32_t blocks)
{
    const uint32_t q = blocks / kXcds, rem = blocks % kXcds, xcd = block % kXcds, j = block / kXcds;
    return (xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q) + j;
}

// The same within every `span` workgroups (a power of two, 0: all of them): the XCDs take runs of span / 8 neighbours in turn,
// and all of them stay in the same part of the work.  With a span of 8 that is the order in which workgroups are handed out.
constexpr uint32_t xcd_spans(uint32_t block, uint32_t blocks, uint32_t span)
{
    const uint32_t first = block & (0u - span), left = blocks - first;
    return first + xcd_contiguous(block - first, span - 1 < left - 1 ? span : left);
}

inline int elem_bytes(int mode) { return (mode == CCDC_BF16_SUM_XOR || mode == CCDC_F16_SUM_XOR) ? 2 : 4; }

// Whether calls whose value length or pointers only allow one-element packs are made of 16-byte packs at any element.
inline bool wide_anyway(int r, int64_t W, int64_t ell, int elem)
{
    const int64_t pack = 16 / elem;
    return ell >= pack && (double)ell >= kAnyPacks * (double)pack && (ell == W || W - (r - 1) * ell >= pack);      // and the last segment has a pack
}

// The chunks that row lists of min_rows rows or more are cut into, `items` packs of outputs in all.
inline int64_t list_split(int64_t items, int64_t min_rows)
{
    if (items >= (1 << 18)) return 1;
    const int64_t most = min_rows < 1 ? 1 : min_rows < 256 ? min_rows : 256, wanted = ((1 << 19) + items - 1) / items;
    return wanted < most ? wanted : most;
}

inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

constexpr int kWave = 64;
// Segments fill the wavefronts of a tile row to at least 3/4.
inline bool fills_wavefronts(uint32_t Lv)
{
    const uint64_t lanes = (uint64_t)cdiv(Lv, kWave) * kWave;
    return (uint64_t)Lv * 4 >= lanes * 3;
}

// Whether k_node_decode_reduce_wave numbers its units by tile, an XCD on a contiguous range of them, so that the nodes that read
// the same packs run next to each other behind one L2; else the tiles of one output are neighbours, on all XCDs.  For all nodes
// of one job and packs of 16 bytes, where a tile has 14 outputs (a node's segment) or more to share its packs: with fewer it is
// slower (r = 2, 4 nodes 1.04 of the time, 5 nodes 1.03, 6 nodes 0.99; 4 nodes, r = 3 0.99, 5 nodes 0.90).  The fewer readers a pack has
// and the more files are summed for one, the less is shared, so r = 2 and batches of several files ask for more tiles.  Over 3303 inputs
// of 48 MB to 2.9 GB and 16 tiles or more: 2110 are numbered by tile and take 0.886 of the time (one file and r >= 3 0.848, r = 2 0.967, several files
// 0.910; 12 nodes, r = 2, two functions each, T = 155840 u32 271 -> 249 us), 32 over 3 % more (8 nodes, r = 4, T = 72064 f16 28.6 -> 35.0, else up to 1.09);
// the other 1193 would take 1.001 of it, 245 over 3 % more.
// With fewer than 16 tiles the rows of one are more than an L2 holds (22 nodes, r = 3, seven files, T = 1352 f32, two tiles, 448 us, 786);
// narrower packs 0.99, up to 1.05; with r = 1 nothing is read twice, 1.04.  Chosen in the kernel both ways cost short wavefronts up to 15 %.
inline bool neighbours_share(const ccdc_plan_t *p, uint32_t tiles)
{
    if (p->J > 1 || p->K * p->r < 14 || (p->r == 2 && p->m > 1)) return false;
    return tiles >= (p->m > 1 ? 200u : p->r == 2 ? 64u : 16u);
}

// Whether segments in packs of 16 bytes fill their wavefronts, or in one-element packs do not either: a node-local call whose
// packs would leave lanes idle where one-element packs do not keeps those (14 nodes, r = 4, three files, T = 1193 f32, 75 packs a segment,
// decoding 102 us, in lane-packed wide packs 121).
inline bool wide_fills(int64_t ell, int elem)
{
    return fills_wavefronts(cdiv(ell, 16 / elem)) || !fills_wavefronts((uint32_t)ell);
}

// The bytes a call that reads V moves, with `elements` of other inputs and outputs.
inline double moved_bytes(const ccdc_plan_t *p, double elements)
{
    return ((double)p->J * p->N * p->Q * (double)p->T + elements) * elem_bytes(p->mode);
}

// Whether `rows` rows of `length` elements make `times` kAnyLanes packs of 16 bytes.
inline bool makes_lanes(const ccdc_plan_t *p, int64_t rows, int64_t length, double times)
{
    return (double)rows * (double)length * elem_bytes(p->mode) >= 16 * times * kAnyLanes;
}

// Whether a call (of node `node`, -1 for all) whose value length or pointers only allow one-element packs is made of 16-byte packs at any
// element.
enum class Call { map, combine, encode, decode, reduce, shuffle, node_encode, node_decode };
bool any_element(const ccdc_plan_t *p, Call call, int node = -1);

// Elements of the packs of a node-local decoding with aligned pointers.  any: lists may be summed in packs at any element.
inline int node_pack(bool any, int elem, int64_t T, int64_t ell)
{
    if (T % 4 != 0) return any && wide_fills(ell, elem) ? 16 / elem : 1;
    return elem == 2 && T % 8 == 0 && ell % 8 == 0 ? 8 : 4;
}

// Rank of sender a's label among the members other than b.
inline int label_rank(int a, int b) { return a - (a > b ? 1 : 0); }

}  // namespace ccdc
