// Host side of the plan: file placement (Sec. IV-A), round schedule (Sec. IV-B),
// segment split and the index tables the kernels consume.  Subsets are handled
// through their lexicographic rank (combinatorial number system), no subset
// table is ever materialised.
#include "plan.hpp"

#include <algorithm>
#include <limits>
#include <new>

namespace ccdc {
namespace {

constexpr int64_t kMaxTable = 2147483647LL;          // int32 indexable
constexpr int64_t kMaxElems = 1LL << 40;             // per buffer
constexpr int64_t kMaxItems = 2147483647LL;          // work items of one launch

// Pascal's triangle with saturation, C[n][k] for 0 <= k <= n <= nmax.
struct Binom {
    int nmax;
    std::vector<int64_t> tab;
    explicit Binom(int n) : nmax(n), tab((size_t)(n + 1) * (n + 1), 0) {
        const int64_t cap = std::numeric_limits<int64_t>::max() / 2;
        for (int i = 0; i <= n; i++) {
            at(i, 0) = 1;
            for (int k = 1; k <= i; k++) at(i, k) = std::min(cap, at(i - 1, k - 1) + (k <= i - 1 ? at(i - 1, k) : 0));
        }
    }
    int64_t &at(int n, int k) { return tab[(size_t)n * (nmax + 1) + k]; }
    int64_t operator()(int n, int k) const {
        if (n < 0 || k < 0 || k > n) return 0;
        return tab[(size_t)n * (nmax + 1) + k];
    }
};

// Number of k-subsets of {0..n-1} that precede the ascending subset s in
// lexicographic order.
int64_t lex_rank(const Binom &C, int n, int k, const int *s)
{
    int64_t rank = 0;
    int lo = 0;
    for (int i = 0; i < k; i++) {
        // subsets that agree on s[0..i-1] and have a smaller element at position i
        for (int v = lo; v < s[i]; v++) rank += C(n - 1 - v, k - 1 - i);
        lo = s[i] + 1;
    }
    return rank;
}

// Inverse of lex_rank.
void lex_unrank(const Binom &C, int n, int k, int64_t rank, int *s)
{
    int v = 0;
    for (int i = 0; i < k; i++) {
        while (C(n - 1 - v, k - 1 - i) <= rank) {
            rank -= C(n - 1 - v, k - 1 - i);
            v++;
        }
        s[i] = v++;
    }
}

}  // namespace

int build_plan(int K, int r, int Q, int N, bool paper_jobs, int gamma, ccdc_plan_t **out)
{
    if (!out) return CCDC_EINVAL;
    *out = nullptr;
    if (gamma < 1 || (gamma > 1 && !paper_jobs)) return CCDC_EINVAL;
    // Sec. III network model (K | Q, K <= N) and Theorem 1 (mu*K in 1..K-1)
    if (K < 2 || r < 1 || r > K - 1 || Q < 1 || N < 1 || Q % K != 0 || K > N) return CCDC_EINVAL;
    if (K > 4096) return CCDC_ESIZE;

    const Binom C(K);
    const int r1 = r + 1;
    const int64_t nlabel = C(K, r), G = C(K, r1);
    if (nlabel > kMaxTable || G > kMaxTable) return CCDC_ESIZE;
    const int64_t per_job = paper_jobs ? r1 : nlabel;
    if (N % per_job != 0) return CCDC_EINVAL;                 // Sec. IV-A: even batches
    const int64_t nround = paper_jobs ? G * (K - r) : G;
    const int64_t nbatch = paper_jobs ? G * r1 : nlabel;
    if (nround * r1 > kMaxTable / gamma || nbatch * r > kMaxTable / gamma || G > kMaxTable / gamma) return CCDC_ESIZE;

    ccdc_plan_t *p = new (std::nothrow) ccdc_plan_t;
    if (!p) return CCDC_ENOMEM;
    try {
        p->K = K; p->r = r; p->Q = Q; p->N = N;
        p->c = Q / K;
        p->m = (int)(N / per_job);
        p->paper_jobs = paper_jobs;
        p->J = paper_jobs ? (int)G : 1;
        p->nbatch = nbatch;
        p->nround = nround;
        p->nrows = nround * r1;
        p->batch_job.resize((size_t)nbatch);
        p->batch_file0.resize((size_t)nbatch);
        p->batch_label.resize((size_t)nbatch * r);
        p->round_member.resize((size_t)nround * r1);
        p->round_batch.resize((size_t)nround * r1);

        std::vector<int> S(r1 + 1), P(r1 + 1);
        if (!paper_jobs) {
            // One job over the whole cluster: batch p <-> p-th r-subset.
            for (int64_t b = 0; b < nbatch; b++) {
                lex_unrank(C, K, r, b, P.data());
                p->batch_job[b] = 0;
                p->batch_file0[b] = (int32_t)(b * p->m);
                std::copy(P.begin(), P.begin() + r, p->batch_label.begin() + b * r);
            }
            // Round u <-> u-th (r+1)-subset; member b is served the batch whose
            // label is the subset without s_b.
            for (int64_t u = 0; u < nround; u++) {
                lex_unrank(C, K, r1, u, S.data());
                for (int b = 0; b < r1; b++) {
                    p->round_member[u * r1 + b] = S[b];
                    int w = 0;
                    for (int i = 0; i < r1; i++)
                        if (i != b) P[w++] = S[i];
                    p->round_batch[u * r1 + b] = (int32_t)lex_rank(C, K, r, P.data());
                }
            }
        } else {
            // Job j lives on the j-th (r+1)-subset K_j.  Its r+1 batches are its
            // r-subsets in lexicographic order: local batch q drops position r-q.
            for (int64_t j = 0; j < G; j++) {
                lex_unrank(C, K, r1, j, S.data());
                for (int q = 0; q < r1; q++) {
                    const int64_t bt = j * r1 + q;
                    p->batch_job[bt] = (int32_t)j;
                    p->batch_file0[bt] = q * p->m;
                    int w = 0;
                    for (int i = 0; i < r1; i++)
                        if (i != r - q) p->batch_label[bt * r + w++] = S[i];
                }
            }
            int64_t u = 0;
            for (int64_t j = 0; j < G; j++) {
                lex_unrank(C, K, r1, j, S.data());
                // stage 1: job j inside K_j
                for (int b = 0; b < r1; b++) {
                    p->round_member[u * r1 + b] = S[b];
                    p->round_batch[u * r1 + b] = (int32_t)(j * r1 + (r - b));
                }
                u++;
                // stage 2: one round per outside node i.  Member s_b is served the
                // batch labelled K_j \ {s_b} of the job living on K_j \ {s_b} + {i}.
                int next_member = 0;
                for (int i = 0; i < K; i++) {
                    if (next_member < r1 && S[next_member] == i) { next_member++; continue; }
                    for (int b = 0; b < r1; b++) {
                        int w = 0, pos = -1;
                        for (int t = 0; t < r1; t++) {
                            if (t == b) continue;
                            if (pos < 0 && S[t] > i) { pos = w; P[w++] = i; }
                            P[w++] = S[t];
                        }
                        if (pos < 0) { pos = w; P[w++] = i; }
                        const int64_t jb = lex_rank(C, K, r1, P.data());
                        p->round_member[u * r1 + b] = S[b];
                        p->round_batch[u * r1 + b] = (int32_t)(jb * r1 + (r - pos));
                    }
                    u++;
                }
            }
        }
        // J = gamma * C(K, r+1) jobs (Sec. IV): the same placement and the same rounds
        // again for every further block of C(K, r+1) jobs
        if (gamma > 1) {
            const int64_t nb1 = p->nbatch, nr1 = p->nround;
            const int J1 = p->J;
            p->J = J1 * gamma;
            p->nbatch = nb1 * gamma;
            p->nround = nr1 * gamma;
            p->nrows = p->nround * r1;
            p->batch_job.resize((size_t)p->nbatch);
            p->batch_file0.resize((size_t)p->nbatch);
            p->batch_label.resize((size_t)p->nbatch * r);
            p->round_member.resize((size_t)p->nround * r1);
            p->round_batch.resize((size_t)p->nround * r1);
            for (int g = 1; g < gamma; g++) {
                for (int64_t b = 0; b < nb1; b++) {
                    p->batch_job[g * nb1 + b] = p->batch_job[b] + g * J1;
                    p->batch_file0[g * nb1 + b] = p->batch_file0[b];
                    for (int s = 0; s < r; s++) p->batch_label[(g * nb1 + b) * r + s] = p->batch_label[b * r + s];
                }
                for (int64_t i = 0; i < nr1 * r1; i++) {
                    p->round_member[g * nr1 * r1 + i] = p->round_member[i];
                    p->round_batch[g * nr1 * r1 + i] = p->round_batch[i] + (int32_t)(g * nb1);
                }
            }
        }
        // packets each node sends: by symmetry nrows / K of them (C(K-1,r) rounds, times K-r for the J-job schedule)
        p->rows_per_node = p->nrows / K;
        p->node_rows.assign((size_t)p->nrows, 0);
        std::vector<int64_t> fill((size_t)K, 0);
        for (int64_t i = 0; i < p->nrows; i++) {
            const int k = p->round_member[i];
            if (fill[k] < p->rows_per_node) p->node_rows[(size_t)k * p->rows_per_node + fill[k]] = (int32_t)i;
            fill[k]++;
        }
        for (int k = 0; k < K; k++)
            if (fill[k] != p->rows_per_node) {
                delete p;
                return CCDC_EINVAL;
            }
        // placement seen from the files and from the nodes (Sec. IV-A): file -> the label of its
        // batch; node -> every file of every batch whose label holds it
        const int64_t nfiles = (int64_t)p->J * N;
        if (nfiles * r > kMaxTable) {
            delete p;
            return CCDC_ESIZE;
        }
        p->file_nodes.assign((size_t)nfiles * r, -1);
        std::vector<std::vector<int32_t>> held((size_t)K);
        for (int64_t bt = 0; bt < p->nbatch; bt++)
            for (int f = 0; f < p->m; f++) {
                const int64_t file = (int64_t)p->batch_job[bt] * N + p->batch_file0[bt] + f;
                for (int s = 0; s < r; s++) {
                    p->file_nodes[(size_t)file * r + s] = p->batch_label[bt * r + s];
                    held[p->batch_label[bt * r + s]].push_back((int32_t)file);
                }
            }
        p->files_per_node = nfiles * r / K;
        p->node_files.clear();
        for (int k = 0; k < K; k++) {
            if ((int64_t)held[k].size() != p->files_per_node) {     // symmetric placement: |M_k| = mu*J*N
                delete p;
                return CCDC_EINVAL;
            }
            std::sort(held[k].begin(), held[k].end());
            p->node_files.insert(p->node_files.end(), held[k].begin(), held[k].end());
        }
    } catch (const std::bad_alloc &) {
        delete p;
        return CCDC_ENOMEM;
    }
    *out = p;
    return CCDC_OK;
}

// Compression-only comparison scheme (appendix of the paper): no coding.  With
// mu = r/K (taken as 1/2 when larger) the files are cut into nb = ceil(1/mu)
// consecutive batches of mu*N files (the last takes the rest), node k stores
// batch k mod nb, and for every node k and batch t it does not store, the next
// node after k (cyclically) that stores B_t pre-combines and sends one packet.
int build_compression_plan(int K, int r, int Q, int N, ccdc_plan_t **out)
{
    if (!out) return CCDC_EINVAL;
    *out = nullptr;
    if (K < 2 || r < 1 || r > K - 1 || Q < 1 || N < 1 || Q % K != 0 || K > N) return CCDC_EINVAL;
    if (K > 4096) return CCDC_ESIZE;
    int64_t num = r, den = K;
    if (2 * r > K) { num = 1; den = 2; }                   // more than half the files does not help here
    if (((int64_t)N * num) % den != 0) return CCDC_EINVAL;  // mu*N files per batch
    const int64_t per = (int64_t)N * num / den;
    const int nb = (int)((den + num - 1) / num);
    ccdc_plan_t *p = new (std::nothrow) ccdc_plan_t;
    if (!p) return CCDC_ENOMEM;
    try {
        p->K = K; p->r = r; p->Q = Q; p->N = N;
        p->c = Q / K;
        p->m = (int)per;
        p->compression = true;
        p->J = 1;
        p->nbatch = nb;
        p->nround = K;                                     // one group of packets per receiver
        p->nrows = (int64_t)K * (nb - 1);
        p->batch_first.resize((size_t)nb + 1);
        for (int t = 0; t < nb; t++) p->batch_first[t] = (int32_t)(t * per);
        p->batch_first[nb] = N;
        p->batch_job.assign((size_t)nb, 0);
        p->batch_file0.assign(p->batch_first.begin(), p->batch_first.end() - 1);
        p->node_batch.resize((size_t)K);
        for (int k = 0; k < K; k++) p->node_batch[k] = k % nb;
        for (int k = 0; k < K; k++)
            for (int t = 0; t < nb; t++) {
                if (t == p->node_batch[k]) continue;
                int sender = -1;
                for (int d = 1; d < K && sender < 0; d++)
                    if (p->node_batch[(k + d) % K] == t) sender = (k + d) % K;
                p->pkt_recv.push_back(k);
                p->pkt_batch.push_back(t);
                p->pkt_send.push_back(sender);
                p->row_files.push_back(p->batch_first[t + 1] - p->batch_first[t]);
            }
    } catch (const std::bad_alloc &) {
        delete p;
        return CCDC_ENOMEM;
    }
    *out = p;
    return CCDC_OK;
}

namespace {

// Whether lists are summed in packs of 16 bytes where rows do not divide by them: where those fill the chip without cutting the lists, where
// the second launch that cut ones take is little of the time, and where one-element packs need it too and the call is not short.
// values: bytes of V.  Where nothing is cancelled (uncoded, r = 1) a batch is read as the one packet it was combined into, and calls are as
// long as their lists (24 nodes, r = 2, 288 files, T = 14345 u32 uncoded, 397 MB of values, 48 MB of lists, 11.3 us, as a long call 18.4; four
// such plans 1.29 of the time).
bool wide_lists(int r, bool coded, int64_t nout, int64_t rows, int64_t W, int elem, double values)
{
    const double bytes = coded && r > 1 ? values : (double)rows * (double)W * elem;
    return (double)(nout * ((W + 3) / 4)) >= kAnyListPacks || bytes >= kAnyListBytes ||
           (nout * W < (1 << 18) && bytes >= (elem == 2 ? 0.16 : 0.64) * kAnyListBytes);
}

// Wavefronts of a workgroup that sums a whole row list (ccdc_reduce in one launch), 0 where the list is better split over
// workgroups and added by a second kernel.  Only for plans whose outputs are too few to fill the chip with whole lists
// (split > 1).  Measured over 282 such plans of 64 KB to 400 MB (every scheme and mode): the one launch takes 0.657 of the
// split form's time (up to 4 MB 0.68, 4 to 48 MB 0.59, above 0.84), with the best pack and count of wavefronts each time
// 0.645.  A wavefront for two rows is the best share (four 0.659), in all at most 3072, with the workgroups counted in packs of up to four
// elements: by the packs of eight that 16-bit rows are summed in, 462 of 2998 such plans get more wavefronts and take 1.035 of the time.  (A call with
// pointers that are not aligned for wide packs has more workgroups of the same count.)
// Lists of over 640 rows are left to the split: 16 nodes, r = 4, T = 728 f32 (1820 rows) 24 us, in one launch 28 to 45; 14
// nodes, r = 5, T = 1227 f16 (2002) 26, 39; so are inputs past the last-level cache, and one-element packs of 16 bits with over 64
// rows a wavefront, 1.04 of the time over 31 plans (of 2998 16-bit plans 24 were over 3 % slower, 18 of them these).  Rows in packs at any element
// count as wide ones: 14 nodes, r = 3, T = 6735 f16 in one-element packs 24.0 split, 29.8 in one launch; at any element 24.1 and 21.3.
int plan_groups(int64_t nout, int64_t rows, int64_t W, int vec, int elem, int64_t split, double bytes)
{
    if (split <= 1 || rows > 640 * nout || bytes > 256e6) return 0;
    const bool narrow = elem == 2 && vec == 1;
    int64_t tiles = 0;
    for (; vec > 0; vec /= 2) {
        tiles = (W / vec + kGroupLanes - 1) / kGroupLanes;
        if (nout * tiles >= kGroupsWanted) break;
    }
    const int64_t wanted = std::max<int64_t>(2, std::min<int64_t>(kGroupMaxWaves, rows / (2 * nout)));
    const int64_t waves = std::max<int64_t>(2, std::min<int64_t>(wanted, 3072 / (nout * tiles)));
    return narrow && rows > 64 * nout * waves ? 0 : (int)waves;
}

// The chunk of the row lists that each round's packets go to: of a few, the next in turn among them, the one that is shortest where the
// round's members have most, so that a node's packets are spread evenly whatever the order of the rounds.  (In turn alone the longest
// chunk of 16 nodes, r = 3, 32 chunks has 1.69 times the mean, of 24 nodes, r = 4, 25 chunks 1.46; the best of two 1.34 and 1.02, of four
// 1.20 and 1.01.)  count: [node][chunk] of packets, zeros at first.
template <int R1>
void spread_rounds(const int32_t *member, int64_t rounds, int split, int choices, int32_t *count, uint8_t *chunk)
{
    const int step = (split + choices - 1) / choices;
    for (int64_t u = 0, turn = 0; u < rounds; u++, turn = turn + 1 == split ? 0 : turn + 1) {
        const int32_t *in = member + u * R1;
        int best = (int)turn;
        int64_t least = std::numeric_limits<int64_t>::max();
        for (int c = 0, s = (int)turn; c < choices; c++) {
            int32_t most = 0;
            int64_t sum = 0;
            for (int b = 0; b < R1; b++) {
                const int32_t n = count[in[b] * (int64_t)split + s];
                most = std::max(most, n);
                sum += n;
            }
            const int64_t cost = ((int64_t)most << 32) + sum;
            if (cost < least) least = cost, best = s;
            s += step;
            if (s >= split) s -= split;
        }
        for (int b = 0; b < R1; b++) count[in[b] * (int64_t)split + best]++;
        chunk[u] = (uint8_t)best;
    }
}

// The row lists of ccdc_node_decode_reduce and the chunks they are cut into.  A coded packet is read by its r receivers and a value
// that is side information by r - 1, so lists are best cut by rounds: chunk s of every list then has the packets of the
// same rounds (not of neighbouring ones, which would be all of the first nodes'),
// and units that are numbered by chunk (node.hip) read them together, behind one L2.  The price is chunks of unequal length, and
// a chunk is a chain of waits, on an XCD with the same chunk of other lists: no such lists where the longest has over kUnequalChunks
// times the mean to load (kUnequalFileChunks with several files a batch).
void lists_by_round(const ccdc_plan_t *p, int64_t local_rows, int64_t split, std::vector<int32_t> *lists)
{
    const int r1 = p->r + 1;
    const int64_t loads = 1 + (int64_t)(p->r - 1) * p->m;    // of a received packet: the coded one and the files of r - 1 batches
    const int64_t chunks = p->K * split;
    std::vector<int32_t> at((size_t)chunks + 1, 0);
    std::vector<uint8_t> chunk((size_t)p->nround);           // split <= 256
    const int choices = p->nround > 8192 ? 2 : 4;            // many rounds are spread well enough by two, in half the time
    auto spread = p->r == 3 ? spread_rounds<4> : p->r == 4 ? spread_rounds<5> : spread_rounds<6>;
    spread(p->round_member.data(), p->nround, (int)split, choices, at.data() + 1, chunk.data());
    int64_t longest = 0;                                     // with the chunk's part of the files the node stores
    for (int64_t i = 0; i < chunks; i++) {
        const int64_t s = i % split;
        longest = std::max(longest, loads * at[i + 1] + local_rows * (s + 1) / split - local_rows * s / split);
    }
    if ((double)longest * (double)split > (p->m > 1 ? kUnequalFileChunks : kUnequalChunks) * (double)(local_rows + loads * p->rows_per_node)) return;
    for (int64_t i = 0; i < chunks; i++) at[i + 1] += at[i];
    lists->resize(at.size() + (size_t)at.back());
    std::copy(at.begin(), at.end(), lists->begin());
    int32_t *list = lists->data() + at.size();
    for (int k = 0; k < p->K; k++) {                         // a list after the other: its chunks' ends stay in the first cache
        int32_t *end = at.data() + k * split;
        const int32_t *packet = p->node_rows.data() + k * p->rows_per_node;
        for (int64_t j = 0; j < p->rows_per_node; j++) list[end[chunk[(uint32_t)packet[j] / (uint32_t)r1]]++] = packet[j];
    }
}

// ccdc_plan_bind for the compression-only scheme: the packet is sent whole (no
// segments), so ell = W, and every packet is both what is transmitted and what
// the receiver adds.
int bind_compression(ccdc_plan_t *p, int64_t T, int mode)
{
    if (mode != CCDC_F32_SUM && mode != CCDC_U32_XOR) return CCDC_EINVAL;   // nothing is coded: no hybrid of it
    if (T > kMaxElems / p->c) return CCDC_ESIZE;
    const int64_t W = (int64_t)p->c * T;
    const int vec = (T % 4 == 0) ? 4 : 1;
    if ((double)p->N * p->Q * (double)T > (double)kMaxElems || (double)p->nrows * (double)W > (double)kMaxElems)
        return CCDC_ESIZE;
    if ((double)std::max<int64_t>(p->nrows, p->K) * (double)((W + vec - 1) / vec) > (double)kMaxItems) return CCDC_ESIZE;
    try {
        std::vector<int64_t> src((size_t)p->nrows);
        for (int64_t i = 0; i < p->nrows; i++)
            src[i] = ((int64_t)p->batch_first[p->pkt_batch[i]] * p->Q + (int64_t)p->pkt_recv[i] * p->c) * T;
        // reduce lists: own batch from V, then the received packets in order
        const int64_t nout = p->K;
        std::vector<int64_t> ptr((size_t)nout + 1, 0), rows, outs((size_t)nout);
        int64_t min_rows = std::numeric_limits<int64_t>::max();
        for (int k = 0; k < p->K; k++) {
            const int j = p->node_batch[k];
            for (int n = p->batch_first[j]; n < p->batch_first[j + 1]; n++)
                rows.push_back((((int64_t)n * p->Q + (int64_t)k * p->c) * T) << 1);
            for (int64_t i = 0; i < p->nrows; i++)
                if (p->pkt_recv[i] == k) rows.push_back(((i * W) << 1) | 1);
            ptr[k + 1] = (int64_t)rows.size();
            outs[k] = (int64_t)k * W;
            min_rows = std::min(min_rows, ptr[k + 1] - ptr[k]);
        }
        const bool any = wide_anyway(p->r, W, W, 4) && wide_lists(p->r, false, nout, (int64_t)rows.size(), W, 4, (double)p->N * p->Q * (double)T * 4);
        const int pack = any ? 4 : vec;                      // elements of a call's packs
        const int64_t items = nout * ((W + pack - 1) / pack);
        const int64_t split = list_split(items, min_rows);
        p->T = T; p->W = W; p->ell = W; p->mode = mode;
        p->packet_len.assign(1, W);
        p->scheduled = p->nrows * W;
        p->src_off.swap(src);
        p->red_ptr.swap(ptr);
        p->red_row.swap(rows);
        p->red_out.swap(outs);
        p->nout = nout;
        p->wide_lists = any;
        p->red_split = (int)split;
        p->red_waves = plan_groups(nout, (int64_t)p->red_row.size(), W, pack, 4, split, ((double)p->N * p->Q * (double)T) * 4);
        p->workspace_bytes = p->red_workspace_bytes = split > 1 && p->red_waves == 0 ? (size_t)split * (size_t)p->Q * (size_t)T * 4 : 0;
        p->pipe_ok = false;
        p->loc_row.clear();
        p->pipe_row.clear();
        p->bound = true;
    } catch (const std::bad_alloc &) {
        return CCDC_ENOMEM;
    }
    return CCDC_OK;
}

}  // namespace

int bind_plan(ccdc_plan_t *p, int64_t T, int mode)
{
    if (!p || T < 1 || mode < CCDC_F32_SUM || mode > CCDC_F16_SUM_XOR) return CCDC_EINVAL;
    if (p->compression) return bind_compression(p, T, mode);
    const int r = p->r, r1 = r + 1;
    if (T > kMaxElems / p->c) return CCDC_ESIZE;
    const int64_t W = (int64_t)p->c * T;

    // Split of a packet into r segments (Sec. IV-B): exact when 4r | W, else
    // ceil(W/r) rounded up to a multiple of 4 elements with a short/empty tail.
    int64_t ell;
    if (W % (4 * (int64_t)r) == 0) {
        ell = W / r;
    } else {
        ell = (W + r - 1) / r;
        ell = (ell + 3) / 4 * 4;
    }

    // size limits of buffers and of one launch
    const double v_elems = (double)p->J * p->N * p->Q * (double)T;
    const double rows = (double)p->nround * r1;
    if (v_elems > (double)kMaxElems || rows * (double)W > (double)kMaxElems) return CCDC_ESIZE;
    const int vec = (T % 4 == 0) ? 4 : 1;
    if (rows * (double)((W + vec - 1) / vec) > (double)kMaxItems) return CCDC_ESIZE;

    try {
        // true length of what sender a transmits: the longest segment it carries
        std::vector<int64_t> plen(r1, 0);
        int64_t per_round = 0;
        for (int a = 0; a < r1; a++) {
            for (int b = 0; b < r1; b++) {
                if (b == a) continue;
                const int64_t lo = label_rank(a, b) * ell;
                const int64_t cnt = lo >= W ? 0 : std::min(ell, W - lo);
                plen[a] = std::max(plen[a], cnt);
            }
            per_round += plen[a];
        }

        // where each round's r+1 packets are combined from
        std::vector<int64_t> src((size_t)p->nround * r1);
        for (int64_t i = 0; i < p->nround * r1; i++) {
            const int32_t bt = p->round_batch[i];
            const int64_t file = (int64_t)p->batch_job[bt] * p->N + p->batch_file0[bt];
            src[i] = (file * p->Q + (int64_t)p->round_member[i] * p->c) * T;
        }

        // Row lists of the final reduction: for output block (job, node) first the
        // files the node stores itself (batch order), then what it decoded (round order).
        const int64_t nout = (int64_t)p->J * p->K;
        std::vector<int64_t> cnt((size_t)nout + 1, 0);
        for (int64_t bt = 0; bt < p->nbatch; bt++)
            for (int s = 0; s < r; s++)
                cnt[(int64_t)p->batch_job[bt] * p->K + p->batch_label[bt * r + s] + 1] += p->m;
        if (p->J == 1)                                           // every node is in as many rounds
            for (int64_t o = 0; o < nout; o++) cnt[o + 1] += p->rows_per_node;
        else
            for (int64_t i = 0; i < p->nround * r1; i++)
                cnt[(int64_t)p->batch_job[p->round_batch[i]] * p->K + p->round_member[i] + 1] += 1;
        for (int64_t o = 0; o < nout; o++) cnt[o + 1] += cnt[o];
        std::vector<int64_t> rows_tab((size_t)cnt[nout]);
        std::vector<int64_t> fill(cnt.begin(), cnt.end() - 1);
        for (int64_t bt = 0; bt < p->nbatch; bt++)
            for (int s = 0; s < r; s++) {
                const int k = p->batch_label[bt * r + s];
                const int64_t o = (int64_t)p->batch_job[bt] * p->K + k;
                for (int f = 0; f < p->m; f++) {
                    const int64_t file = (int64_t)p->batch_job[bt] * p->N + p->batch_file0[bt] + f;
                    rows_tab[fill[o]++] = ((file * p->Q + (int64_t)k * p->c) * T) << 1;
                }
            }
        if (p->J == 1) {                                         // a list after the other
            for (int64_t o = 0; o < nout; o++)
                for (int64_t j = 0; j < p->rows_per_node; j++)
                    rows_tab[fill[o] + j] = ((p->node_rows[o * p->rows_per_node + j] * W) << 1) | 1;
        } else {
            for (int64_t i = 0; i < p->nround * r1; i++) {
                const int64_t o = (int64_t)p->batch_job[p->round_batch[i]] * p->K + p->round_member[i];
                rows_tab[fill[o]++] = ((i * W) << 1) | 1;
            }
        }
        std::vector<int64_t> outs((size_t)nout);
        int64_t min_rows = std::numeric_limits<int64_t>::max();
        for (int64_t o = 0; o < nout; o++) {
            outs[o] = ((o / p->K) * p->Q + (o % p->K) * (int64_t)p->c) * T;
            min_rows = std::min(min_rows, cnt[o + 1] - cnt[o]);
        }

        // Few, long outputs (small T, many rounds) would leave the chip idle: cut
        // each row list into red_split chunks summed by different workgroups and
        // added up, in a fixed order, by a second pass.
        const int elem = elem_bytes(mode);
        const bool any = wide_anyway(r, W, ell, elem) && wide_lists(r, true, nout, cnt[nout], W, elem, v_elems * elem);
        const int64_t pack = any ? 4 : vec, items = nout * ((W + pack - 1) / pack);
        const int64_t split = list_split(items, min_rows);
        if (items * split > kMaxItems) return CCDC_ESIZE;

        // One-pass pipeline: single job, unrolled r, accumulators of K nodes x r
        // segments per lane must fit in LDS.  Pack width, wavefronts and chunks are
        // chosen at upload, when the device is known.
        bool pipe_ok = !p->paper_jobs && r1 <= kPipeMaxR1 && W < (1LL << 29) &&   // 32-bit byte offsets in a packet
                       (int64_t)p->K * r * 4 * kPipeLanes <= kPipeMaxLds;
        int64_t pipe_cap = 1, local_rows = 0;
        std::vector<int64_t> loc, pipe;
        if (pipe_ok) {
            // The chunks' outputs are kept under 64 MiB: what ccdc_pipeline_fused_noalloc's array
            // holds, and no workgroups are short of work at outputs large enough to feel it.
            const double kw = (double)p->K * (double)W;
            pipe_cap = std::max<int64_t>(1, std::min<int64_t>({(int64_t)1024, p->nround, (int64_t)((64 << 20) / (4 * kw))}));
            // rows of V each node adds from its own files: the V entries of its
            // reduce list (the same count for every node of a single job)
            for (int64_t i = cnt[0]; i < cnt[1]; i++) local_rows += !(rows_tab[i] & 1);
            loc.resize((size_t)p->K * local_rows);
            for (int k = 0; k < p->K; k++) {
                int64_t w = 0;
                for (int64_t i = cnt[k]; i < cnt[k + 1]; i++)
                    if (!(rows_tab[i] & 1)) {
                        // entry = (element offset << 12) | node; K <= 4096, offsets < 2^40
                        if (w < local_rows) loc[(size_t)k * local_rows + w] = ((rows_tab[i] >> 1) << 12) | k;
                        w++;
                    }
                if (w != local_rows) pipe_ok = false;
            }
            pipe.resize(src.size() + r1, 0);         // and one row that is read but not used
            for (size_t i = 0; i < src.size(); i++) pipe[i] = (src[i] << 12) | p->round_member[i];
        }

        std::vector<int32_t> node_list;
        const int node_vec = node_pack(any, elem, T, ell);
        // Lists by round: where a value has two readers or more besides its owner's output (r >= 3; r = 2 0.94 to 1.08 of the
        // time), with a wavefront on one segment and units that are not shared by tile already.  One file a batch: a chunk may have
        // up to 1.4 times the mean to load (kUnequalChunks): 105 such plans of 1 MB to 1.3 GB 0.75 of the time of equal cuts for all nodes and
        // 0.74 for a node alone (16 nodes, r = 3, T = 4096 h32 61 -> 48 and 15.4 -> 14.8 us), one of them over 5 % slower, a node alone, which
        // shares nothing with others; 16 with up to 1.7 times 0.92 and 0.94, four; 42 beyond 1.01 and 1.01.  Several files: equal cuts
        // have the files that a node stores in the first chunks and all packets, of many loads, in the last, so up to twice the mean 29 plans
        // 0.62 and 0.39, one of them slower (7 nodes, r = 5, eleven files, T = 142976 u32 255 -> 283); 18 beyond 1.01.  In few chunks
        // one-element packs gain only while the values' readers can find them in the last-level cache (21 nodes, r = 3, T = 4711
        // f32, 1.3 GB, six chunks, 281 -> 295).
        const bool wide = node_vec > 1;
        const bool by_round = split > 1 && p->J == 1 && r >= 3 && r <= 5 && fills_wavefronts((uint32_t)(ell / node_vec)) &&
                              (wide || split >= 8 || v_elems * elem <= (r - 1) * kKeptNodeBytes) &&
                              !(node_vec * elem == 16 && neighbours_share(p, cdiv((uint64_t)(ell / node_vec), kPipeLanes)));
        if (by_round) lists_by_round(p, cnt[1] - p->rows_per_node, split, &node_list);

        p->T = T; p->W = W; p->ell = ell; p->mode = mode;
        p->node_list.swap(node_list);
        p->pipe_ok = pipe_ok;
        p->pipe_max_chunks = (int)pipe_cap;
        p->pipe_local_rows = pipe_ok ? local_rows : 0;
        p->loc_row.swap(loc);
        p->pipe_row.swap(pipe);
        p->packet_len.swap(plen);
        p->scheduled = per_round * p->nround;
        p->src_off.swap(src);
        p->red_ptr.swap(cnt);
        p->red_row.swap(rows_tab);
        p->red_out.swap(outs);
        p->nout = nout;
        p->wide_lists = any;
        p->red_split = (int)split;
        p->red_waves = plan_groups(nout, (int64_t)p->red_row.size(), W, (int)pack, elem, split, v_elems * elem);
        p->red_workspace_bytes = split > 1 ? (size_t)split * (size_t)p->J * p->Q * (size_t)T * 4 : 0;
        p->workspace_bytes = p->red_workspace_bytes;         // until upload has fixed the chunks: the most it can be
        if (pipe_ok && pipe_cap > 1)
            p->workspace_bytes = std::max(p->workspace_bytes, (size_t)pipe_cap * (size_t)p->K * (size_t)W * 4);
        p->bound = true;
    } catch (const std::bad_alloc &) {
        return CCDC_ENOMEM;
    }
    return CCDC_OK;
}

// The lines are where the one-element packs stop being faster; packs and times as there were with the calls alone, over draws of 64 KB to 3 GB.
bool any_element(const ccdc_plan_t *p, Call call, int node)
{
    const int elem = elem_bytes(p->mode);
    const bool half = elem == 2;
    if (call == Call::map)                           // see k_map
        return makes_lanes(p, (int64_t)p->J * p->N, (int64_t)p->Q * p->T, 2);
    if (!wide_anyway(p->r, p->W, p->ell, elem)) return false;
    switch (call) {
    case Call::combine: return makes_lanes(p, p->nrows, p->W, p->m == 1 ? 1 : 4);
    // 64 to 128 thousand packs 0.84 (16 bits) and 0.97 of the time over 35 inputs, half as many 1.05 and 1.01 over 26
    case Call::encode: return makes_lanes(p, p->nrows, p->ell, 2);
    // 16 bits: 128 to 256 thousand packs 0.91 of the time (51 inputs), half as many 1.03, a quarter 1.26; 32 bits: 256 to 512 thousand
    // 0.95 (46 inputs), half as many 1.03, a quarter 1.13 (the ends of packets are made element by element)
    case Call::decode: return makes_lanes(p, p->nrows, p->ell, half ? 4 : 8);
    case Call::reduce: return p->wide_lists;
    // By the packs of the segments.  In 16 bits, one file a batch, from 512 thousand on (36 inputs 0.76 of the time, two over 5 % slower; 256
    // to 512 thousand 27 inputs 0.98, nine, 128 to 256 31 inputs 1.12); several files are asked for together in one-element packs, those of
    // all packets, so only from 256 thousand on with r = 1 (24 inputs 0.51), a million with r = 2 (18 inputs 0.65; half of it 1.07), two
    // million with r >= 3 (7 inputs 0.74; half of it 1.07, less 1.23).  32 bits gain with r <= 2 on large inputs (10 jobs on 5 nodes, r = 2,
    // T = 400097 u32 95 -> 79 us; from two million packs on 11 inputs 0.96, below 1.05), else one-element packs are faster (4 nodes, r = 3, T =
    // 4015094 f32 25.0 and 27.4, 6 nodes, r = 5, T = 1690898 u32 73 and 79).
    case Call::shuffle:
        if (!half && (p->r > 2 || moved_bytes(p, 0) < kAnyListBytes)) return false;
        return makes_lanes(p, p->nrows, p->ell, !half ? 64 : p->m == 1 ? 16 : p->r == 1 ? 8 : p->r == 2 ? 32 : 64);
    // One file a batch, or one packet in the making: 16 bits from 64 thousand on (up to 256 thousand 39 inputs 0.86 of the time, three over
    // 5 % slower; several files for a node alone 1.13, from 128 thousand on 0.61), 32 bits from 256 thousand (29 inputs 0.85; fewer, 47
    // inputs, 0.94, but seven up to 1.27).  With several files and 2 <= r <= 5 one-element packs ask for the files of all packets
    // together: 16 bits from half a million on (54 inputs 0.81; half of it 1.02, a quarter 1.30), 32 bits from four million (6 inputs 0.93;
    // fewer, 92 inputs, 1.06).  A node alone from a quarter of a million on (10 and 13 inputs 0.74 and 0.88; half of it 1.08 and 1.04).
    case Call::node_encode: {
        double lanes = node >= 0 ? 8 : half ? 16 : 128;
        if (p->m == 1 || p->r == 1 || p->r > 5) lanes = !half ? 8 : p->m == 1 ? 2 : 4;
        return wide_fills(p->ell, elem) && makes_lanes(p, node < 0 ? p->nrows : p->rows_per_node, p->ell, lanes);
    }
    // One node of a plan whose lists are not cut has a K-th of the lanes: from 64 thousand packs of its own on (32 bits, several files: 128)
    // 31 inputs 0.77 of the time, none slower, 26 of fewer 1.14, up to 1.98.  (The width of packs does not change the order of sums.)
    default:
        if (node >= 0 && p->red_split == 1 && !makes_lanes(p, p->J, p->W, !half && p->m > 1 ? 4 : 2)) return false;
        return p->wide_lists && wide_fills(p->ell, elem);
    }
}

}  // namespace ccdc
