// Host side of the flmoe C ABI: argument checks, workspace partition, launches.
// Every shuffle call only enqueues kernels on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "../../include/flmoe.h"
#include "common.h"
#include "kernels_layout.h"
#include "kernels_shuffle.h"

using namespace flmoe;

// Scratch of fl_moe_layout_static, part of the device image: every GPU the library
// is loaded on holds its own copy at its own address.  In host code this name is
// only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[FL_STATIC_SCRATCH_BYTES];

namespace {

enum KernelId {
    KID_ROUTE_LAYOUT = 0, KID_DISPATCH_PACK, KID_DISPATCH_UNPACK, KID_COMBINE_PACK, KID_COMBINE_REDUCE,
    KID_DISPATCH_PACK_E4M3, KID_COMBINE_PARTIAL_PACK, KID_GATE_DISPATCH, KID_GATE_COMBINE,
    KID_ANNOUNCE_DISPATCH, KID_ANNOUNCE_COMBINE
};
const char *kKernelNames[FL_KERNEL_COUNT] = {
    "route_layout_kernel", "dispatch_pack_kernel", "dispatch_unpack_kernel", "combine_pack_kernel",
    "combine_reduce_kernel", "dispatch_pack_e4m3_kernel", "combine_partial_pack_kernel",
    "arrival_gate_kernel(dispatch)", "arrival_gate_kernel(combine)", "announce_kernel(dispatch)",
    "announce_kernel(combine)"};

constexpr int kEventPool = 512;
constexpr long long kMaxRowBlocks = 1 << 18;      // per launch of a row kernel; rows beyond are looped over
constexpr long long kDefaultSpin = 1 << 20;       // polls about 2 us apart: gives up after about 2 s

constexpr size_t kBigPage = 2u << 20;
constexpr int kComputeUnits = 256;                // of the part, where a context has not asked the device
constexpr int kCachedReplyMiB = 1024;             // see replies_cached
constexpr int kLaunchMiB = 860;
constexpr int kSelfAnnounceBlocks = 4096;         // see announces_itself
constexpr int kWavesPerUnit = 32;                 // wave slots of a compute unit
size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// From row to row of a receive buffer: rows start on 128-byte lines where that takes at most a sixteenth more room.
// Stores that begin inside lines cost more than loads that do.  us of a step of 32 ranks, rows packed and rows on lines
// (slices as before): 14 352-byte rows, 128 tokens 538 and 507; 10 000 bytes 368 and 345; 2064 bytes 117.3 and 111.9;
// 2032 bytes, 1024 tokens 647 and 623.  Where padding takes more room the lines themselves cost: 1552 bytes (112 of
// padding) 500 and 513, 272 bytes 177 and 196.
int row_stride(long long row_bytes) {
    const long long lines = (long long)align_up((size_t)row_bytes, 128);
    return (int)((lines - row_bytes) * 16 <= row_bytes ? lines : row_bytes);
}

// Waves of a receive launch that may wait inside the kernel (waits_itself): a hardware queue runs one such launch at a
// time, so if every queue but one holds one (4 queues unless the environment says otherwise) they take less than
// half of the machine's wave slots, and a sender's workgroup, the layout step's sixteen waves included, still finds room.
int self_wait_waves(int cu_count) {
    const char *set = getenv("GPU_MAX_HW_QUEUES");
    const int queues = std::max(set ? atoi(set) : 0, 4);
    return cu_count * kWavesPerUnit / 2 / queues;
}

// Walks the workspace; with base == nullptr it only measures.
struct Carver {
    char *base; size_t cur = 0;
    explicit Carver(void *b) : base((char *)b) {}
    template <class T> T *take(size_t count) {
        cur = align_up(cur, 256);
        T *p = base ? (T *)(base + cur) : nullptr;
        cur += count * sizeof(T);
        return p;
    }
};

int resolve(const fl_moe_config *c, Dims *D) {
    if (!c) return FL_ERR_INVALID_ARG;
    if (c->n_ranks < 1 || c->n_ranks > FL_MAX_RANKS) return FL_ERR_INVALID_ARG;
    if (c->n_experts < c->n_ranks || c->n_experts > FL_MAX_EXPERTS ||
        c->n_experts % c->n_ranks != 0) return FL_ERR_INVALID_ARG;
    const int El = c->n_experts / c->n_ranks;
    if (El > FL_MAX_EXPERTS_PER_RANK) return FL_ERR_INVALID_ARG;
    if (c->top_k < 1 || c->top_k > FL_MAX_TOPK || c->top_k > c->n_experts) return FL_ERR_INVALID_ARG;
    if (c->max_tokens < 1 || c->max_tokens >= (1 << 24)) return FL_ERR_INVALID_ARG;
    if (c->hidden < 8 || c->hidden > (1 << 20)) return FL_ERR_INVALID_ARG;
    if ((c->hidden * 2) % 16 != 0) return FL_ERR_ALIGNMENT;
    if (c->dispatch_dtype != FL_DTYPE_BF16 && c->dispatch_dtype != FL_DTYPE_E4M3_BLOCK128)
        return FL_ERR_INVALID_ARG;
    if (c->dispatch_dtype == FL_DTYPE_E4M3_BLOCK128 && c->hidden % 128 != 0) return FL_ERR_ALIGNMENT;
    if (c->expert_align < 1 || c->expert_align > (1 << 16)) return FL_ERR_INVALID_ARG;
    if (c->flags & ~(FL_FLAG_ZERO_PAD | FL_FLAG_STREAM_ORDERED | FL_FLAG_PEER_PUSH | FL_FLAG_PARTIAL_SUMS |
                     FL_FLAG_PROGRESSIVE_RECV))
        return FL_ERR_INVALID_ARG;
    if ((c->flags & FL_FLAG_PROGRESSIVE_RECV) && (c->flags & FL_FLAG_STREAM_ORDERED)) return FL_ERR_INVALID_ARG;
    if (c->recv_capacity_rows < 0 || c->expert_capacity_rows < 0 || c->spin_limit < 0)
        return FL_ERR_INVALID_ARG;
    if (c->max_private_rows < 0 || c->reserved != 0) return FL_ERR_INVALID_ARG;

    D->N = c->n_ranks; D->E = c->n_experts; D->El = El; D->T = c->max_tokens; D->K = c->top_k;
    D->H = c->hidden; D->dtype = c->dispatch_dtype; D->align = c->expert_align; D->flags = c->flags;
    D->route_len = route_record_words(D->E, D->N, D->T);
    D->KM = (D->K + 3) / 4 * 4;
    D->MW = (c->flags & FL_FLAG_PARTIAL_SUMS) ? 2 * D->KM : D->KM;
    const long long NT = (long long)D->N * D->T;
    const long long minKEl = D->K < El ? D->K : El;
    const long long worst_recv = NT;
    const long long worst_expert = NT * minKEl + (long long)(El - 1) * (D->align - 1);
    D->recv_cap = c->recv_capacity_rows ? c->recv_capacity_rows : worst_recv;
    D->expert_cap = c->expert_capacity_rows ? c->expert_capacity_rows : worst_expert;
    if (D->recv_cap > worst_recv) D->recv_cap = worst_recv;
    if (D->expert_cap > worst_expert) D->expert_cap = worst_expert;
    D->P = c->max_private_rows < D->T ? c->max_private_rows : D->T;   // a source sends at most T rows
    D->recv_rows = (long long)D->N * D->P + D->recv_cap;
    if (D->recv_rows >= (1ll << 31) || D->expert_cap >= (1ll << 31)) return FL_ERR_INVALID_ARG;
    D->send_cap = (long long)D->T * (D->K < D->N ? D->K : D->N);
    D->Bx = 2ll * D->H;
    D->Bc = 2ll * D->H;
    if (D->dtype == FL_DTYPE_BF16) {
        D->Bw = D->Bx; D->Be = D->Bx; D->scales_per_row = 0;
    } else {
        D->scales_per_row = D->H / 128;
        D->Be = D->H;
        // wire rows start on 128-byte lines: measured 5-10 % faster pack and unpack than 16-byte packing
        D->Bw = (long long)align_up((size_t)(D->H + 4ll * D->scales_per_row), 128);
    }
    // bufA receives the combine replies, bufB the dispatched rows.
    D->Sw = row_stride(D->Bw);
    D->Sc = row_stride(D->Bc);
    const size_t need_a = (size_t)D->T * D->K * D->Sc, need_b = (size_t)D->recv_rows * D->Sw;
    // Large payload buffers start on 2 MB boundaries of the workspace, rank by rank (the
    // page size the driver maps big allocations with): measured 3 % faster unpack at the
    // decode shape than 256-byte packing.  Small ones stay packed.
    D->bufA_rank_bytes = (long long)align_up(need_a, need_a >= kBigPage ? kBigPage : 256);
    D->bufB_rank_bytes = (long long)align_up(need_b, need_b >= kBigPage ? kBigPage : 256);
    // arrival counters count 16-byte units in 32 bits with a wrap-safe comparison
    if ((long long)D->T * (D->Bc / 16) >= (1ll << 31)) return FL_ERR_INVALID_ARG;
    D->spin_limit = c->spin_limit ? c->spin_limit : kDefaultSpin;
    // Largest LDS tile of the counting kernel that stays under 60 KB.
    int tt = 32;
    while (tt < 1024 && route_count_lds_bytes(D->E, D->N, D->K, tt * 2) <= 60 * 1024) tt *= 2;
    const int need = (D->T + 31) / 32 * 32;
    D->TT = need < tt ? need : tt;
    D->tune_rows = 0;
    D->tune_reduce = 0;
    D->tune_slices = 0;
    D->tune_cached_mb = kCachedReplyMiB;
    D->tune_grid_pct = -1;
    D->tune_self = kSelfAnnounceBlocks;
    D->tune_wait = self_wait_waves(kComputeUnits);
    D->tune_cap8 = 3;
    D->tune_order = 0;
    D->tune_parts = 0;
    {   // a token reaches a given rank unless its K distinct experts, drawn uniformly, all live elsewhere
        double miss = 1.0;
        for (int k = 0; k < D->K; ++k) miss *= std::max(0.0, (double)(D->E - El - k) / (D->E - k));
        D->typ_recv_rows = (long long)(NT * (1.0 - miss)) + 1;
        D->typ_pair_rows = (long long)D->T * D->K;
    }
    return FL_OK;
}

// Returns the number of bytes of the small-table prefix (cleared at create).
size_t carve(const Dims &D, void *base, Tables *W, size_t *total) {
    Carver c(base);
    const size_t N = D.N, E = D.E, El = D.El, T = D.T, K = D.K;
    W->status = c.take<int>(64);
    W->epoch_route = c.take<unsigned>(N);
    W->arrive_route = c.take<unsigned>(N * N);
    W->arrive_disp = c.take<unsigned>(N * N);
    W->arrive_comb = c.take<unsigned>(N * N);
    W->expect_disp = c.take<unsigned>(N * N);
    W->expect_comb = c.take<unsigned>(N * N);
    W->done_disp = c.take<unsigned>(done_words(D.N));
    W->done_comb = c.take<unsigned>(done_words(D.N));
    W->plan_ok = c.take<int>(N);
    W->gate_disp = c.take<int>(N);
    W->gate_comb = c.take<int>(N);
    W->routes = c.take<unsigned long long>(N * N * D.route_len);
    W->C = c.take<int>(N * E);
    W->M = c.take<int>(N * N);
    W->send_off = c.take<int>(N * (N + 1));
    W->comb_off = c.take<int>(N * (N + 1));
    W->G = c.take<int>(N * El);
    W->expert_off = c.take<int>(N * (El + 1));
    W->recv_off = c.take<int>(N * (N + 1));
    W->recv_shared_off = c.take<int>(N * N);
    W->dst_off = c.take<int>(N * N);
    W->comb_dst_off = c.take<int>(N * N);
    W->ret_off = c.take<int>(N * N);
    W->base_x = c.take<int>(N * El * N);
    W->cs_base = c.take<int>(N * N * El);
    W->cs_off = c.take<int>(N * (N + 1));
    const size_t small = align_up(c.cur, 256);
    W->send_to = c.take<int>(N * T * K);
    W->pair_meta = c.take<unsigned>(N * T * K);
    W->comb_pos = c.take<int>(N * T * K);
    W->recv_meta = c.take<unsigned>(N * (size_t)D.recv_rows * D.MW);
    if ((size_t)D.bufA_rank_bytes >= kBigPage) c.cur = align_up(c.cur, kBigPage);
    W->bufA = c.take<char>(N * (size_t)D.bufA_rank_bytes);
    if ((size_t)D.bufB_rank_bytes >= kBigPage) c.cur = align_up(c.cur, kBigPage);
    W->bufB = c.take<char>(N * (size_t)D.bufB_rank_bytes);
    *total = align_up(c.cur, 256);
    return small;
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// Blocks that share one token in the pack kernel (each takes a slice of the row).
int pack_slices(long long row_bytes, int tune_slices) {
    if (tune_slices > 0) return tune_slices;
    const long long nvec = row_bytes / 16;
    // measured: rows up to 8 KB are fastest with two vectors per thread (4 KB rows: one block,
    // 30 -> 25 us; 7 KB rows of e4m3 codes: two blocks, 61 -> 54 us), longer rows with one
    if (nvec <= 4 * kPackThreads) return (int)((nvec + 2 * kPackThreads - 1) / (2 * kPackThreads));
    // about one vector per thread; a slice more for the last few vectors costs (14 352-byte rows: 7 slices 483, 8 499 us a step)
    long long s = (nvec + kPackThreads / 2) / kPackThreads;
    return (int)(s < 1 ? 1 : s > 16 ? 16 : s);
}

// Grids are sized from capacities (the rows really in use are only known on the
// device), so a generous capacity would launch mostly idle blocks; beyond this
// many blocks per launch the kernels loop instead.
unsigned capped_grid(long long blocks_needed, int rank_count, long long max_blocks,
                     int multiple_of = 1) {
    long long limit = max_blocks / rank_count;
    if (limit < 1) limit = 1;
    long long g = blocks_needed < limit ? blocks_needed : limit;
    g = (g + multiple_of - 1) / multiple_of * multiple_of;
    return (unsigned)(g < 1 ? 1 : g);
}

// Rows a row-kernel's grid is sized for: what uniform routing would bring and six times its
// standard deviation (at most the square root of the mean), never more than the capacity; the
// kernels loop when a rank holds more.  Idle blocks are not free: at twice the mean the unpack
// of a 512-token step takes 651 us, at 1.25 times 624, its combine pack 649 and 637; with few
// rows (4 tokens per rank, 29 rows) 1.25 times is too tight: 12.0 -> 13.2 us.
long long grid_rows(const Dims &D, long long capacity, long long typical) {
    if (D.tune_grid_pct == 0) return capacity;
    const long long want = D.tune_grid_pct > 0 ? typical * D.tune_grid_pct / 100 + 1
                                               : typical + (long long)(6.0 * std::sqrt((double)typical)) + 1;
    return want < capacity ? want : capacity;
}

// Whether the unpack or a reply kernel moves its rows by workgroups that plan a chunk of rows and copy it as one
// run of vectors (true), or by a wave per row or share of a row (false).  Waves of their own have the shorter chain
// of loads, but a short row leaves most lanes idle, and once there are more rows than waves fit on the machine at
// once (five workgroups of four per compute unit) the rate at which waves start and end bounds the kernel, some
// 0.6 ns per row however short.  16 ranks, top 8, us of unpack / combine pack, waves against chunks:
//   128-byte rows: 16 tokens per rank 7.3 / 6.9 against 8.1 / 7.2, 32: 7.9 / 7.3 and 8.5 / 7.1, 64: 10.3 / 9.4 and
//     8.4 / 6.9, 256: 23 / 21 and 9.4 / 8.3, 4096: 262 / 264 and 28 / 32
//   1 KB rows: 64 tokens 11.2 / 12.7 and 10.9 / 10.7, 1024: 72 / 82 and 48 / 45
//   2 KB rows: 32 tokens 8.6 / 10.6 and 10.4 / 10.3, 1024: 86 / 101 and 77 / 84
//   3 KB rows: 1024 tokens 116 / 124 and 125 / 125, longer ones up to 7 % in favour of waves
// The partial-sum pack reads several rows per row written, so its lanes have more to do: 1.5 KB rows, 1024 tokens
// 76 and 65, 2 KB rows, 256 tokens 27.7 and 29.7.
constexpr long long kChunkRowBytes = 2048, kChunkPartialRowBytes = 1536;
constexpr long long kRowWavesPerUnit = 5 * kCopyThreads / kWave;
bool by_chunks(const Dims &D, int cu_count, long long row_bytes, long long max_row_bytes, long long rows) {
    return (D.flags & FL_FLAG_PROGRESSIVE_RECV) || (row_bytes <= max_row_bytes && rows > kRowWavesPerUnit * cu_count);
}
bool unpack_by_chunks(const Dims &D, int cu_count, int rank_count) {
    return by_chunks(D, cu_count, D.Be, kChunkRowBytes, std::min(D.typ_recv_rows, D.recv_rows) * rank_count);
}
bool replies_by_chunks(const Dims &D, int cu_count, int rank_count) {
    const bool partial = D.flags & FL_FLAG_PARTIAL_SUMS;
    const long long rows = partial ? std::min(D.typ_recv_rows, D.recv_rows) : std::min(D.typ_pair_rows, D.expert_cap);
    return by_chunks(D, cu_count, D.Bc, partial ? kChunkPartialRowBytes : kChunkRowBytes, rows * rank_count);
}

long long recv_grid_rows(const Dims &D) {        // received rows: unpack, partial-sum pack
    return grid_rows(D, std::min(D.recv_rows, (long long)D.N * D.T), D.typ_recv_rows);
}
long long reply_grid_rows(const Dims &D) {       // rows a rank sends back: one per pair, or one per received row
    return D.flags & FL_FLAG_PARTIAL_SUMS ? recv_grid_rows(D) : grid_rows(D, D.expert_cap, D.typ_pair_rows);
}

// Workgroups per sender of the dispatch pack kernel; ready: the caller quantised the rows itself.
int quant_threads(const Dims &D) { return D.scales_per_row > 256 / kQuantLanes ? 512 : 256; }
int dispatch_slices(const Dims &D, bool ready) {
    const int per_block = quant_threads(D) / kQuantLanes;            // quantisation blocks per workgroup
    if (D.dtype == FL_DTYPE_E4M3_BLOCK128 && !ready) return (D.scales_per_row + per_block - 1) / per_block;
    return pack_slices(ready ? D.Be : D.Bx, D.tune_slices);
}
long long dispatch_workgroups(const Dims &D, bool ready) { return (long long)D.T * dispatch_slices(D, ready); }

// Waves that share a row of `vecs` 16-byte vectors in the unpack and the combine pack kernel: up
// to four vectors per lane.
int waves_per_row(long long vecs) {
    const long long w = (vecs + 4 * kWave - 1) / (4 * kWave);
    return (int)(w > 16 ? 16 : w);
}

// Whether a combine_send call over `rank_count` ranks writes its replies through (st_payload) or streams them.  All
// ranks' replies are written before the first reduce, whatever number of calls they come in, so the bytes of the
// whole group decide; calls for part of the ranks gain nothing earlier already.  us of a step, rows of 14 KB,
// streaming against written through:
//   one call: 0.44 GiB of replies 487 and 452, 0.9 GiB 975 and 941, 1.3 GiB 1413 and 1443, 3.5 GiB 3772 and 3835
//   rank by rank: 0.9 GiB 1679 and 1679, 1.75 GiB 2630 and 2686
// (1.75 GiB in one call 1990 and 1911; allocations at other addresses move steps of this size by 4 %.)
// Partial sums write fewer rows but read as many; counted by pairs as well.
bool replies_cached(const Dims &D, int rank_count) {
    const long long limit = (long long)D.tune_cached_mb << 20;
    return (long long)D.N * D.T * D.K * D.Bc <= (rank_count < D.N ? limit / 2 : limit);
}

// How the reduce kernel writes its output: written through, but with one or two rows per sum and a group's output larger than
// this with the streaming hint, and not written through where rows begin or end inside lines (all sides at the kernel).
constexpr long long kStreamedOutputBytes = 40ll << 20;
OutputStores output_stores(const Dims &D, const void *out) {
    if (D.K > 2 || (long long)D.N * D.T * D.Bc <= kStreamedOutputBytes) return kOutThrough;
    return D.Bc % 128 == 0 && ((uintptr_t)out & 127) == 0 ? kOutThroughHint : kOutHint;
}

// Whether the send kernels of a call, of `workgroups` per sender, announce their transfers themselves
// (announce_when_last) rather than having a kernel launched behind them: up to a number of workgroups that was measured.
// A workgroup that waits for its stores holds its place meanwhile, which costs more than a launch once a call has several
// times as many as fit on the machine (4096 of the dispatch pack's two waves, 2048 of the combine packs' four, 1024 or 2048
// of the quantising pack's eight or four).  us of a step, with announce kernels and without: 2 ranks x 16 tokens of 512
// bytes (16 workgroups) 34.0 and 28.6; 8 ranks, 64 tokens of 8 KB, rank by rank (324 a call) 277 and 215; 32 ranks, 14 KB
// rows, both calls, by the combine pack's workgroups: 4 tokens (2176) 45.6 and 44.6, 8 (3616) 57.0 and 56.3, 16 (7168)
// 81.3 and 82.6, 32 (14 336) 131.5 and 133.8, 128 (57 344) 452 and 468; the dispatch pack alone: 4 tokens (896) 46.6 and
// 46.1, 8 (1792) 57.7 and 56.7, 16 (3584) 81.5 and 80.9.  The quantising pack gains up to 512 workgroups (73.2 and 72.4)
// and does not care on either side of the line: 2048 196.3 and 196.6, 4096 356.8 and 357.1, 8192 719.3 and 721.1 (noise 0.4).
bool announces_itself(const Dims &D, long long workgroups, int rank_count) {
    return !(D.flags & (FL_FLAG_PROGRESSIVE_RECV | FL_FLAG_STREAM_ORDERED)) && workgroups * rank_count <= D.tune_self;
}

// The form of a combine_send call over `rank_count` ranks, one for all its launches (a group of its ranks has fewer
// rows, so it takes waves where the call does).  A call announces itself only if it writes through, so a small one for part
// of the ranks does both whatever the group's replies come to: us of a step rank by rank, 32 ranks, rows of 14 KB, streamed
// and announced by a kernel against written through and announcing itself: 160 tokens 1306 and 1261, 256: 1680 and 1633, 448:
// 2388 and 2363.  One call of that few workgroups but more replies than replies_cached allows (rows of megabytes) gains
// nothing by it (4 ranks x 40 tokens of 2 MB 1512 and 1520).
ReplyForm reply_form(const Dims &D, int cu_count, int rank_count) {
    const bool cached = replies_cached(D, rank_count);
    const long long workgroups = (reply_grid_rows(D) * waves_per_row(D.Bc / 16) * kWave + kCopyThreads - 1) / kCopyThreads;
    if ((cached || rank_count < D.N) && announces_itself(D, workgroups, rank_count) && !replies_by_chunks(D, cu_count, rank_count))
        return kRepliesThroughAnnounced;
    return cached ? kRepliesThrough : kRepliesStreamed;
}

// The whole rank range of a call, and where in it the current launch group sits: the
// gate kernel of a receive call runs once, before the first group, for all its ranks,
// and the announce kernel of a send call once, behind the last group (a receiver needs
// every sender's rows anyway, so announcing group by group would let nobody start earlier).
struct CallSpan {
    int rank_begin, rank_count;
    bool first, last;
};

// Whether a receive launch of `waves` waits for the arrival counters itself instead of having a gate kernel in front:
// if the waves that wait leave the senders room whatever else waits (self_wait_waves: 1024 on a whole MI355X).  us of a
// step with gate kernels and without: 2 ranks x 16 tokens of 512 bytes 28.2 and 24.5, 8 x 4 tokens of 4 KB 32.7 and 28.5,
// 8 ranks one by one: 8 tokens of 14 KB 225 and 165, 64 tokens of 8 KB 225 and 200.
bool waits_itself(const Dims &D, long long waves, const CallSpan &call, int rank_count) {
    return !(D.flags & (FL_FLAG_PROGRESSIVE_RECV | FL_FLAG_STREAM_ORDERED)) && rank_count == call.rank_count &&
           waves * rank_count <= D.tune_wait;
}

// Workgroups per rank of a dispatch_recv launch whose waves work alone, `share` of them to a row.
unsigned unpack_workgroups(const Dims &D, int rank_count, int *share) {
    const int G = waves_per_row(D.Be / 16 + (D.scales_per_row % 4 == 0 ? D.scales_per_row / 4 : 0));
    const int wpb = kCopyThreads / kWave;
    unsigned gx = capped_grid((recv_grid_rows(D) * G + wpb - 1) / wpb, rank_count, kMaxRowBlocks, G);
    if (gx < (unsigned)D.El) gx = (unsigned)((D.El + G - 1) / G * G);    // the first El-1 blocks also clear padding rows
    *share = G;
    return gx;
}
bool unpack_waits(const Dims &D, int cu_count, const CallSpan &call, int rank_count) {
    int share;
    return !unpack_by_chunks(D, cu_count, rank_count) &&
           waits_itself(D, (long long)unpack_workgroups(D, rank_count, &share) * (kCopyThreads / kWave), call, rank_count);
}

// A combine_reduce launch: `parts` workgroups of `threads` share a token, each taking a slice of the row; `groups` such sets
// per rank walk the tokens.
struct ReduceShape {
    int parts, threads;
    unsigned groups;
    long long waves() const { return (long long)groups * parts * (threads / kWave); }
};
ReduceShape reduce_shape(const Dims &D, int cu_count, int rank_count) {
    const bool progressive = D.flags & FL_FLAG_PROGRESSIVE_RECV;
    const int nvec = (int)(D.Bc / 16);
    // measured: long rows are summed fastest by many small workgroups, one payload wave each
    // (7168-wide rows: 14 workgroups of 2 waves 86 us, 2 of 7 waves 90 us, 1 of 14 waves 92 us);
    // rows of 4 KB and less gain nothing; capped polling grids keep one workgroup per token
    int parts = D.tune_parts > 0 ? D.tune_parts : (nvec >= 512 && !progressive ? (nvec + kWave - 1) / kWave : 1);
    if (parts > nvec) parts = nvec;
    const int per = whole_lines((nvec + parts - 1) / parts);
    int nt = (per + kWave - 1) / kWave * kWave;
    if (nt > kReduceMaxThreads) nt = kReduceMaxThreads;
    if (nt < 2 * kWave) nt = 2 * kWave;      // wave 0 waits, wave 1 fetches positions and weights
    // progressive (polling) receivers take at most three eighths of the machine's wave slots
    const unsigned gx = progressive ? capped_grid(D.T, rank_count, (long long)cu_count * 256 * D.tune_cap8 / nt / parts)
                                    : (unsigned)D.T;
    return {parts, nt, gx};
}

int rows_per_block(long long row_bytes, int tune_rows) {
    long long rb = tune_rows > 0 ? tune_rows : 16384 / row_bytes;
    if (rb < 1) rb = 1;
    if (rb > kMaxRowsPerBlock) rb = kMaxRowsPerBlock;
    return (int)rb;
}

}  // namespace

struct fl_moe_ctx {
    fl_moe_config cfg;
    Dims D;
    Tables W;
    size_t workspace_bytes;
    const int32_t *indices = nullptr;
    const int32_t *num_tokens = nullptr;
    unsigned recv_launches = 0;   // names a receive launch that waits itself (launch_ticket)
    int cu_count = kComputeUnits;
    int launch_mb = kLaunchMiB;   // payload a launch should move per direction, see ranks_per_launch
    // profiling
    int profile = 0;
    hipEvent_t ev_start[kEventPool], ev_stop[kEventPool];
    int ev_kernel[kEventPool];
    int ev_used = 0;
    double total_ms[FL_KERNEL_COUNT];
    int64_t launches[FL_KERNEL_COUNT];
};

namespace {

struct LaunchTimer {
    fl_moe_ctx *ctx; hipStream_t st; int slot = -1;
    LaunchTimer(fl_moe_ctx *c, int kid, hipStream_t s) : ctx(c), st(s) {
        if (c->profile && c->ev_used < kEventPool) {
            slot = c->ev_used++;
            c->ev_kernel[slot] = kid;
            (void)hipEventRecord(c->ev_start[slot], st);
        }
    }
    ~LaunchTimer() { if (slot >= 0) (void)hipEventRecord(ctx->ev_stop[slot], st); }
};

int check_ranks(const fl_moe_ctx *ctx, int rb, int rc) {
    if (!ctx) return FL_ERR_INVALID_ARG;
    if (rb < 0 || rc < 1 || rb + rc > ctx->D.N) return FL_ERR_INVALID_ARG;
    return FL_OK;
}

int launch_status() { return hipGetLastError() == hipSuccess ? FL_OK : FL_ERR_HIP; }

// Counting blocks per source: one per tile of tokens, as long as they and the planning blocks fit on the
// machine together (two 1024-thread blocks on each compute unit); beyond that a block walks several
// tiles, and there are only as many blocks as the tiles so dealt out need: every block counts all of the
// source's tokens, also one that would own no tile.
int layout_parts(const Dims &D, int cu_count, int rank_count) {
    const int tiles = (D.T + D.TT - 1) / D.TT;
    const int most = std::min(tiles, std::max(1, 2 * cu_count / rank_count - 1));
    const int per_block = (tiles + most - 1) / most;
    return (tiles + per_block - 1) / per_block;
}

void launch_layout(const Dims &D, const Tables &W, int cu_count, int rb, int rc, const int32_t *indices,
                   const int32_t *num_tokens, hipStream_t st) {
    const int parts = layout_parts(D, cu_count, rc);
    const size_t lds = std::max(route_count_lds_bytes(D.E, D.N, D.K, D.TT), route_plan_lds_bytes(D.E, D.N, D.El));
    auto kernel = route_wide(D.T) ? route_layout_kernel<true> : route_layout_kernel<false>;
    kernel<<<dim3(rc * (parts + 1)), dim3(kRouteThreads), lds, st>>>(D, W, rb, rc, parts, indices, num_tokens);
}

// Ranks one launch of a payload kernel serves.  A launch that walks many GB runs
// measurably slower than the same work cut into launches of somewhat under a GB
// (a plain copy: 6.1 TB/s in 1 GiB launches, 5.7 TB/s as one 12 GiB launch; the
// 4096-token step: 8 % faster in 2-rank launches), while cutting a launch that is
// small already only adds launch tails.  So a call whose ranks move more than three
// times the target is cut into rank groups of about the target size.  Not in
// progressive mode: its receive kernels run on capped grids and its copies write
// through, and there the cut measured 3 % slower.
int ranks_per_launch(const Dims &D, int launch_mb, int rc) {
    if (launch_mb <= 0 || (D.flags & FL_FLAG_PROGRESSIVE_RECV)) return rc;
    const long long row = D.Bw > D.Bc ? D.Bw : D.Bc;
    const long long per_rank = (long long)D.T * D.K * row;
    const long long target = (long long)launch_mb << 20;
    if (per_rank * rc <= 3 * target) return rc;
    long long launches = (per_rank * rc + target - 1) / target;
    if (launches > rc) launches = rc;
    return (int)((rc + launches - 1) / launches);
}

// Runs f(rank_begin, rank_count, span) over the rank groups of one call.
template <class F>
int for_rank_groups(const fl_moe_ctx *ctx, int rb, int rc, F f) {
    int e = check_ranks(ctx, rb, rc);
    if (e != FL_OK) return e;
    const int g = ranks_per_launch(ctx->D, ctx->launch_mb, rc);
    for (int r = rb; r < rb + rc; r += g) {
        const int n = rb + rc - r < g ? rb + rc - r : g;
        e = f(r, n, CallSpan{rb, rc, r == rb, r + n == rb + rc});
        if (e != FL_OK) return e;
    }
    return FL_OK;
}

// ---------------------------------------------------------------- static scratch
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];          // device address of `scratch` on each GPU, looked up once

// Address of the current device's copy of `scratch`.
int static_scratch(void **ptr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return FL_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FL_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return FL_OK;
}

// Whether fl_moe_layout_static takes a configuration: when what fl_moe_layout keeps beside the caller-visible tables
// (counters, route records of E + 2N + 1 words, offsets, per-pair tables) would fit the array.  The call itself
// needs less, a record per counting block (static_parts).
bool fits_static(const Dims &D) {
    const size_t N = D.N, El = D.El, pairs = (size_t)D.T * D.K * N;
    size_t sum = 0;
    for (size_t words : {N, N * N, N * N, N * N, N * N * (D.E + 2 * N + 1), N * N, N * N, N * N, N * N, N * El * N, N * N * El,
                         N * (N + 1), pairs, pairs})
        sum = align_up(sum, 256) + words * sizeof(int);
    return align_up(sum, 256) <= FL_STATIC_SCRATCH_BYTES;
}

// Tile size and blocks per source of fl_moe_layout_static: about kStaticBlocks over all sources, each with an
// equal run of tiles.  At most 128 records of at most 1088 words: 0.6 MB of the array.
int static_parts(Dims *D) {
    const int want = std::min(kStaticMaxParts, std::max(1, kStaticBlocks / D->N));
    const int per_part = ((D->T + want - 1) / want + 31) / 32 * 32;
    D->TT = std::min(D->TT, per_part);
    const int tiles = (D->T + D->TT - 1) / D->TT, per = (tiles + want - 1) / want;
    return (tiles + per - 1) / per;
}

}  // namespace

extern "C" {

int fl_moe_query_sizes(const fl_moe_config *cfg, fl_moe_sizes *out) {
    if (!out) return FL_ERR_INVALID_ARG;
    Dims D;
    int rc = resolve(cfg, &D);
    if (rc != FL_OK) return rc;
    Tables W;
    size_t total;
    carve(D, nullptr, &W, &total);
    out->workspace_bytes = total;
    out->recv_capacity_rows = D.recv_cap;
    out->expert_capacity_rows = D.expert_cap;
    out->send_capacity_rows = D.send_cap;
    out->x_row_bytes = D.Bx;
    out->wire_row_bytes = D.Bw;
    out->expert_x_row_bytes = D.Be;
    out->scales_per_row = D.scales_per_row;
    out->combine_row_bytes = D.Bc;
    out->private_rows = D.P;
    out->recv_buffer_rows = D.recv_rows;
    return FL_OK;
}

int fl_moe_create(const fl_moe_config *cfg, void *workspace, size_t workspace_bytes,
                  fl_moe_ctx **out) {
    if (!out || !workspace) return FL_ERR_INVALID_ARG;
    if (((uintptr_t)workspace & 255) != 0) return FL_ERR_ALIGNMENT;
    Dims D;
    int rc = resolve(cfg, &D);
    if (rc != FL_OK) return rc;
    Tables W;
    size_t total;
    carve(D, nullptr, &W, &total);
    if (workspace_bytes < total) return FL_ERR_WORKSPACE;
    fl_moe_ctx *ctx = new (std::nothrow) fl_moe_ctx();
    if (!ctx) return FL_ERR_INVALID_ARG;
    ctx->cfg = *cfg;
    ctx->D = D;
    const size_t small = carve(D, workspace, &ctx->W, &total);
    ctx->workspace_bytes = total;
    if (hipMemset(workspace, 0, small) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        delete ctx;
        return FL_ERR_HIP;
    }
    {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            cus > 0)
            ctx->cu_count = cus;
        ctx->D.tune_wait = self_wait_waves(ctx->cu_count);
    }
    for (int i = 0; i < kEventPool; ++i) {      // created when profiling is first enabled
        ctx->ev_start[i] = nullptr;
        ctx->ev_stop[i] = nullptr;
    }
    memset(ctx->total_ms, 0, sizeof(ctx->total_ms));
    memset(ctx->launches, 0, sizeof(ctx->launches));
    *out = ctx;
    return FL_OK;
}

int fl_moe_destroy(fl_moe_ctx *ctx) {
    if (!ctx) return FL_ERR_INVALID_ARG;
    for (int i = 0; i < kEventPool; ++i) {
        if (ctx->ev_start[i]) (void)hipEventDestroy(ctx->ev_start[i]);
        if (ctx->ev_stop[i]) (void)hipEventDestroy(ctx->ev_stop[i]);
    }
    delete ctx;
    return FL_OK;
}

int fl_moe_layout(fl_moe_ctx *ctx, int rb, int rc, const int32_t *indices,
                  const int32_t *num_tokens, fl_moe_layout_view *view, void *stream) {
    int e = check_ranks(ctx, rb, rc);
    if (e != FL_OK) return e;
    if (!indices || !num_tokens) return FL_ERR_INVALID_ARG;
    if (((uintptr_t)indices & 3) || ((uintptr_t)num_tokens & 3)) return FL_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const Dims &D = ctx->D;
    ctx->indices = indices;
    ctx->num_tokens = num_tokens;
    {
        LaunchTimer t(ctx, KID_ROUTE_LAYOUT, st);
        launch_layout(D, ctx->W, ctx->cu_count, rb, rc, indices, num_tokens, st);
    }
    if (view) {
        const Tables &W = ctx->W;
        view->counts = W.C; view->dedup_counts = W.M; view->tokens_per_expert = W.G;
        view->send_off = W.send_off; view->recv_off = W.recv_off; view->expert_off = W.expert_off;
        view->comb_off = W.comb_off; view->comb_pos = W.comb_pos; view->plan_ok = W.plan_ok;
    }
    return launch_status();
}

int fl_moe_layout_static(const fl_moe_config *cfg, const int32_t *indices, const int32_t *num_tokens,
                         const fl_moe_layout_out *out, void *stream) {
    if (!cfg || !indices || !num_tokens || !out) return FL_ERR_INVALID_ARG;
    int32_t *const outs[] = {out->counts, out->dedup_counts, out->tokens_per_expert, out->send_off,
                             out->recv_off, out->expert_off, out->comb_off, out->comb_pos,
                             out->plan_ok, out->status};
    for (int32_t *p : outs) {
        if (!p) return FL_ERR_INVALID_ARG;
        if ((uintptr_t)p & 3) return FL_ERR_ALIGNMENT;
    }
    if (((uintptr_t)indices & 3) || ((uintptr_t)num_tokens & 3)) return FL_ERR_ALIGNMENT;
    Dims D;
    int e = resolve(cfg, &D);
    if (e != FL_OK) return e;
    if (!fits_static(D)) return FL_ERR_STATIC_LIMIT;
    void *ptr = nullptr;
    e = static_scratch(&ptr);
    if (e != FL_OK) return e;
    const int parts = static_parts(&D);
    int *records = (int *)ptr, *invalid = records + (size_t)D.N * parts * static_record_words(D.E, D.N, D.T);
    const StaticOut tables{out->counts, out->dedup_counts, out->tokens_per_expert, out->send_off, out->recv_off,
                           out->expert_off, out->comb_off, out->comb_pos, out->plan_ok, out->status};
    hipStream_t st = (hipStream_t)stream;
    static_count_kernel<<<dim3(D.N * parts), dim3(kStaticCountThreads),
                          (size_t)2 * static_record_words(D.E, D.N, D.T) * sizeof(int), st>>>(
        D, parts, indices, num_tokens, records, invalid);
    auto kernel = route_wide(D.T) ? static_tables_kernel<true> : static_tables_kernel<false>;
    kernel<<<dim3(D.N * parts + 1), dim3(kRouteThreads), static_tables_lds_bytes(D.E, D.N, D.K, D.TT), st>>>(
        D, tables, parts, indices, num_tokens, records, invalid);
    return launch_status();
}

static int dispatch_send_range(fl_moe_ctx *ctx, int rb, int rc, CallSpan call, const void *x, const float *weights,
                               const float *ready_scales, void *stream) {
    int e = check_ranks(ctx, rb, rc);
    if (e != FL_OK) return e;
    if (!x || !ctx->indices) return FL_ERR_INVALID_ARG;
    // the weights travel with the tokens exactly when the expert ranks need them
    if (((ctx->D.flags & FL_FLAG_PARTIAL_SUMS) != 0) != (weights != nullptr)) return FL_ERR_INVALID_ARG;
    if (!aligned16(x) || ((uintptr_t)weights & 3) || ((uintptr_t)ready_scales & 3)) return FL_ERR_ALIGNMENT;
    if (ready_scales && ctx->D.dtype != FL_DTYPE_E4M3_BLOCK128) return FL_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const Dims &D = ctx->D;
    const Tables &W = ctx->W;
    // fenced: every block reports what it delivered (progressive receivers).  Otherwise the send kernel's
    // first block advances the counters (stream-ordered callers), its last one does (small calls), or a kernel
    // of its own behind the payload kernels in this (the sender's) stream.
    const bool fenced = D.flags & FL_FLAG_PROGRESSIVE_RECV;
    const char *xp = (const char *)x;
    const int slices = dispatch_slices(D, ready_scales != nullptr);
    const bool self = announces_itself(D, dispatch_workgroups(D, ready_scales != nullptr), call.rank_count);
    if (D.dtype == FL_DTYPE_E4M3_BLOCK128 && !ready_scales) {
        LaunchTimer t(ctx, KID_DISPATCH_PACK_E4M3, st);
        auto go = [&](auto threads) {
            constexpr int QT = decltype(threads)::value;
            auto kernel = fenced ? dispatch_pack_e4m3_kernel<true, QT> : dispatch_pack_e4m3_kernel<false, QT>;
            kernel<<<dim3((unsigned)D.T * slices, rc), dim3(QT), 0, st>>>(D, W, rb, xp, ctx->num_tokens, slices, weights,
                                                                          self ? W.done_disp : nullptr);
        };
        if (quant_threads(D) == 512) go(std::integral_constant<int, 512>{});
        else go(std::integral_constant<int, 256>{});
    } else {
        LaunchTimer t(ctx, KID_DISPATCH_PACK, st);
        // bf16 rows, or e4m3 codes the caller quantised itself (their scales go along)
        const long long src_row = ready_scales ? D.Be : D.Bx;
        auto kernel = fenced ? dispatch_pack_kernel<true> : dispatch_pack_kernel<false>;
        kernel<<<dim3((unsigned)D.T * slices, rc), dim3(kPackThreads), 0, st>>>(
            D, W, rb, xp, ctx->num_tokens, slices, weights, src_row, ready_scales, self ? W.done_disp : nullptr);
    }
    if (!self && !fenced && !(D.flags & FL_FLAG_STREAM_ORDERED) && call.last) {   // once, behind every payload kernel of the call
        LaunchTimer t(ctx, KID_ANNOUNCE_DISPATCH, st);
        announce_kernel<<<dim3(call.rank_count), dim3(kWave), 0, st>>>(D, W, call.rank_begin, W.send_off,
                                                                        W.arrive_disp, (unsigned)(D.Bw / 16));
    }
    return launch_status();
}

static int dispatch_send_impl(fl_moe_ctx *ctx, int rb, int rc, const void *x, const float *weights,
                              const float *ready_scales, void *stream) {
    return for_rank_groups(ctx, rb, rc, [&](int r, int n, CallSpan call) {
        return dispatch_send_range(ctx, r, n, call, x, weights, ready_scales, stream);
    });
}

int fl_moe_dispatch_send(fl_moe_ctx *ctx, int rb, int rc, const void *x, void *stream) {
    return dispatch_send_impl(ctx, rb, rc, x, nullptr, nullptr, stream);
}

int fl_moe_dispatch_send_weighted(fl_moe_ctx *ctx, int rb, int rc, const void *x, const float *weights,
                                  void *stream) {
    if (!weights) return FL_ERR_INVALID_ARG;
    return dispatch_send_impl(ctx, rb, rc, x, weights, nullptr, stream);
}

int fl_moe_dispatch_send_e4m3(fl_moe_ctx *ctx, int rb, int rc, const void *codes, const float *scales,
                              const float *weights, void *stream) {
    if (!scales) return FL_ERR_INVALID_ARG;
    return dispatch_send_impl(ctx, rb, rc, codes, weights, scales, stream);
}

static int dispatch_recv_range(fl_moe_ctx *ctx, int rb, int rc, CallSpan call, void *expert_x, float *expert_scales,
                               int32_t *tokens_per_expert, void *stream) {
    int e = check_ranks(ctx, rb, rc);
    if (e != FL_OK) return e;
    const Dims &D = ctx->D;
    if (!expert_x || !tokens_per_expert) return FL_ERR_INVALID_ARG;
    if ((D.scales_per_row != 0) != (expert_scales != nullptr)) return FL_ERR_INVALID_ARG;
    if (!aligned16(expert_x) || !aligned16(expert_scales) || ((uintptr_t)tokens_per_expert & 3))
        return FL_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const bool gated = !(D.flags & FL_FLAG_STREAM_ORDERED);
    const bool progressive = D.flags & FL_FLAG_PROGRESSIVE_RECV;
    const bool chunks = unpack_by_chunks(D, ctx->cu_count, rc);
    const bool waits = unpack_waits(D, ctx->cu_count, call, rc);
    // Default: a gate kernel of one wave per rank polls the rank's arrival counters, and the
    // unpack kernel runs behind it in the stream on a full grid.  Stream-ordered callers need
    // no gate, and small launches wait themselves.
    const int *gate = nullptr;
    if (gated && !progressive && !waits) {
        if (call.first) {
            LaunchTimer t(ctx, KID_GATE_DISPATCH, st);
            arrival_gate_kernel<<<dim3(call.rank_count), dim3(kWave), 0, st>>>(
                D, ctx->W, call.rank_begin, ctx->W.arrive_disp, ctx->W.expect_disp, ctx->W.gate_disp);
        }
        gate = ctx->W.gate_disp;
    }
    char *ex = (char *)expert_x;
    LaunchTimer t(ctx, KID_DISPATCH_UNPACK, st);
    if (chunks) {
        // Progressive: the unpack kernel polls itself and starts on each
        // source's rows as they land; it may be running while senders still need somewhere to
        // run, so it takes at most three eighths of the resident-block slots (measured best), and
        // to keep the memory system busy with that few waves a block moves 32 KB per turn.
        int rbk = rows_per_block(D.Bw, D.tune_rows);
        if (progressive && D.tune_rows == 0) {
            long long n = (32768 + D.Bw - 1) / D.Bw;
            rbk = (int)(n > kMaxRowsPerBlock ? kMaxRowsPerBlock : n);
        }
        unsigned gx = capped_grid((recv_grid_rows(D) + rbk - 1) / rbk, rc,
                                  progressive ? (long long)ctx->cu_count * D.tune_cap8 : kMaxRowBlocks);
        if (gx < (unsigned)D.El) gx = D.El;      // the first El-1 blocks also clear padding rows
        auto kernel = progressive ? D.P ? dispatch_unpack_chunk_kernel<true, true> : dispatch_unpack_chunk_kernel<false, true>
                                  : D.P ? dispatch_unpack_chunk_kernel<true, false> : dispatch_unpack_chunk_kernel<false, false>;
        kernel<<<dim3(gx, rc), dim3(kCopyThreads), 0, st>>>(D, ctx->W, rb, ex, expert_scales, tokens_per_expert, rbk, gate);
    } else {
        int G;
        const unsigned gx = unpack_workgroups(D, rc, &G);
        auto kernel = waits ? D.P ? dispatch_unpack_kernel<true, true> : dispatch_unpack_kernel<false, true>
                            : D.P ? dispatch_unpack_kernel<true, false> : dispatch_unpack_kernel<false, false>;
        // a launch that waits holds as little as it can
        kernel<<<dim3(gx, rc), dim3(kCopyThreads), waits ? 0 : kRowWavesLdsBytes, st>>>(D, ctx->W, rb, ex, expert_scales,
                                                                                      tokens_per_expert, G, ++ctx->recv_launches, gate);
    }
    return launch_status();
}

int fl_moe_dispatch_recv(fl_moe_ctx *ctx, int rb, int rc, void *expert_x, float *expert_scales,
                         int32_t *tokens_per_expert, void *stream) {
    return for_rank_groups(ctx, rb, rc, [&](int r, int n, CallSpan call) {
        return dispatch_recv_range(ctx, r, n, call, expert_x, expert_scales, tokens_per_expert, stream);
    });
}

static int combine_send_range(fl_moe_ctx *ctx, int rb, int rc, CallSpan call, const void *expert_y, ReplyForm form,
                              void *stream) {
    int e = check_ranks(ctx, rb, rc);
    if (e != FL_OK) return e;
    if (!expert_y) return FL_ERR_INVALID_ARG;
    if (!aligned16(expert_y)) return FL_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const Dims &D = ctx->D;
    const Tables &W = ctx->W;
    const int rbk = rows_per_block(D.Bc, D.tune_rows);
    const bool fenced = D.flags & FL_FLAG_PROGRESSIVE_RECV;      // as in dispatch_send_range
    const bool partial = D.flags & FL_FLAG_PARTIAL_SUMS;
    const bool self = form == kRepliesThroughAnnounced;
    const long long reply_grid = reply_grid_rows(D);
    const unsigned gx = capped_grid((reply_grid + rbk - 1) / rbk, rc, kMaxRowBlocks);
    {
        const dim3 grid(gx, rc), block(kCopyThreads);
        const char *yp = (const char *)expert_y;
        LaunchTimer t(ctx, partial ? KID_COMBINE_PARTIAL_PACK : KID_COMBINE_PACK, st);
        if (replies_by_chunks(D, ctx->cu_count, rc)) {
            auto kernel = fenced   ? partial ? combine_partial_pack_chunk_kernel<true, true> : combine_pack_chunk_kernel<true, true>
                          : form == kRepliesStreamed
                              ? partial ? combine_partial_pack_chunk_kernel<false, false> : combine_pack_chunk_kernel<false, false>
                              : partial ? combine_partial_pack_chunk_kernel<false, true> : combine_pack_chunk_kernel<false, true>;
            kernel<<<grid, block, 0, st>>>(D, W, rb, yp, rbk);
        } else {
            const int G = waves_per_row(D.Bc / 16), wpb = kCopyThreads / kWave;
            const unsigned gw = capped_grid((reply_grid * G + wpb - 1) / wpb, rc, kMaxRowBlocks, G);
            auto kernel = form == kRepliesStreamed
                              ? partial ? combine_partial_pack_kernel<kRepliesStreamed> : combine_pack_kernel<kRepliesStreamed>
                          : form == kRepliesThrough
                              ? partial ? combine_partial_pack_kernel<kRepliesThrough> : combine_pack_kernel<kRepliesThrough>
                              : partial ? combine_partial_pack_kernel<kRepliesThroughAnnounced>
                                        : combine_pack_kernel<kRepliesThroughAnnounced>;
            // No need to hold workgroups back where partial sums read several rows per row written (see the kernel) or
            // in a small call, whose workgroups wait for their stores (4 tokens per rank, step 44.2 -> 43.1 us).
            kernel<<<dim3(gw, rc), block, partial || self ? 0 : kRowWavesLdsBytes, st>>>(D, W, rb, yp, G);
        }
    }
    if (!self && !fenced && !(D.flags & FL_FLAG_STREAM_ORDERED) && call.last) {
        LaunchTimer t(ctx, KID_ANNOUNCE_COMBINE, st);
        announce_kernel<<<dim3(call.rank_count), dim3(kWave), 0, st>>>(
            D, W, call.rank_begin, partial ? W.recv_off : W.cs_off, W.arrive_comb, (unsigned)(D.Bc / 16));
    }
    return launch_status();
}

int fl_moe_combine_send(fl_moe_ctx *ctx, int rb, int rc, const void *expert_y, void *stream) {
    if (!ctx) return FL_ERR_INVALID_ARG;
    const ReplyForm form = reply_form(ctx->D, ctx->cu_count, rc);
    return for_rank_groups(ctx, rb, rc, [&](int r, int n, CallSpan call) {
        return combine_send_range(ctx, r, n, call, expert_y, form, stream);
    });
}

static int combine_reduce_range(fl_moe_ctx *ctx, int rb, int rc, CallSpan call, const float *weights, void *out,
                                void *stream) {
    int e = check_ranks(ctx, rb, rc);
    if (e != FL_OK) return e;
    if (!weights || !out || !ctx->indices) return FL_ERR_INVALID_ARG;
    if (!aligned16(out) || ((uintptr_t)weights & 3)) return FL_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const Dims &D = ctx->D;
    const bool gated = !(D.flags & FL_FLAG_STREAM_ORDERED), partial = D.flags & FL_FLAG_PARTIAL_SUMS;
    const bool progressive = D.flags & FL_FLAG_PROGRESSIVE_RECV;
    const ReduceShape shape = reduce_shape(D, ctx->cu_count, rc);
    const dim3 grid(shape.groups * shape.parts, rc);
    char *o = (char *)out;
    const bool waits = waits_itself(D, shape.waves(), call, rc);
    const int *gate = nullptr;
    if (gated && !progressive && !waits) {         // as in dispatch_recv: a gate kernel, then the full grid
        if (call.first) {
            LaunchTimer t(ctx, KID_GATE_COMBINE, st);
            arrival_gate_kernel<<<dim3(call.rank_count), dim3(kWave), 0, st>>>(
                D, ctx->W, call.rank_begin, ctx->W.arrive_comb, ctx->W.expect_comb, ctx->W.gate_comb);
        }
        gate = ctx->W.gate_comb;
    }
    LaunchTimer t(ctx, KID_COMBINE_REDUCE, st);
    const unsigned launch = ++ctx->recv_launches;
    auto go = [&](auto form, auto shares) {
        constexpr int W = decltype(form)::value;
        constexpr bool P = decltype(shares)::value;
        const OutputStores stores = output_stores(D, out);
        auto kernel = stores == kOutThrough       ? combine_reduce_kernel<W, P, kOutThrough>
                      : stores == kOutThroughHint ? combine_reduce_kernel<W, P, kOutThroughHint>
                                                  : combine_reduce_kernel<W, P, kOutHint>;
        kernel<<<grid, dim3(shape.threads), 0, st>>>(D, ctx->W, rb, weights, o, ctx->num_tokens, gate, shape.parts, launch);
    };
    auto with = [&](auto form) {
        if (partial) go(form, std::true_type{});
        else go(form, std::false_type{});
    };
    if (progressive) with(std::integral_constant<int, kProgressive>{});
    else if (waits) with(std::integral_constant<int, kWaitsItself>{});
    else with(std::integral_constant<int, kBehindGate>{});
    return launch_status();
}

int fl_moe_combine_reduce(fl_moe_ctx *ctx, int rb, int rc, const float *weights, void *out,
                          void *stream) {
    return for_rank_groups(ctx, rb, rc, [&](int r, int n, CallSpan call) {
        return combine_reduce_range(ctx, r, n, call, weights, out, stream);
    });
}

int fl_moe_status(fl_moe_ctx *ctx, int32_t *host_out, void *stream) {
    if (!ctx || !host_out) return FL_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (hipMemcpyAsync(host_out, ctx->W.status, sizeof(int32_t), hipMemcpyDeviceToHost, st) !=
        hipSuccess) return FL_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return FL_ERR_HIP;
    if (*host_out != 0) {
        if (hipMemsetAsync(ctx->W.status, 0, sizeof(int32_t), st) != hipSuccess) return FL_ERR_HIP;
        if (hipStreamSynchronize(st) != hipSuccess) return FL_ERR_HIP;
    }
    return FL_OK;
}

int fl_moe_reset(fl_moe_ctx *ctx, void *stream) {
    if (!ctx) return FL_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    // status word and every counter: the contiguous head of the workspace up to plan_ok
    const size_t bytes = (size_t)((char *)ctx->W.plan_ok - (char *)ctx->W.status);
    if (hipMemsetAsync(ctx->W.status, 0, bytes, st) != hipSuccess) return FL_ERR_HIP;
    // and the route records, whose words name steps that are now to come
    const size_t records = (size_t)ctx->D.N * ctx->D.N * ctx->D.route_len * sizeof(*ctx->W.routes);
    if (hipMemsetAsync(ctx->W.routes, 0, records, st) != hipSuccess) return FL_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return FL_ERR_HIP;
    return FL_OK;
}

int fl_moe_required_capacities(fl_moe_ctx *ctx, int64_t *recv_capacity_rows, int64_t *expert_capacity_rows,
                               void *stream) {
    if (!ctx || !recv_capacity_rows || !expert_capacity_rows) return FL_ERR_INVALID_ARG;
    const Dims &D = ctx->D;
    const size_t nC = (size_t)D.N * D.E, nM = (size_t)D.N * D.N;
    int *host = new (std::nothrow) int[nC + nM];
    if (!host) return FL_ERR_HIP;
    int *C = host, *M = host + nC;          // the sources' own tables: valid whether or not the plan was
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e == hipSuccess) e = hipMemcpy(C, ctx->W.C, nC * sizeof(int), hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(M, ctx->W.M, nM * sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) { delete[] host; return FL_ERR_HIP; }
    long long need_recv = 1, need_expert = 1;   // 0 would read as "worst case" in a configuration
    for (int d = 0; d < D.N; ++d) {
        long long recv = 0, rows = 0;
        for (int s = 0; s < D.N; ++s) recv += std::max(M[(size_t)s * D.N + d] - D.P, 0);
        for (int j = 0; j < D.El; ++j) {
            long long g = 0;
            for (int s = 0; s < D.N; ++s) g += C[(size_t)s * D.E + (size_t)d * D.El + j];
            rows += (j + 1 < D.El) ? (g + D.align - 1) / D.align * D.align : g;   // as the planning block pads
        }
        need_recv = std::max(need_recv, recv);
        need_expert = std::max(need_expert, rows);
    }
    delete[] host;
    *recv_capacity_rows = need_recv;
    *expert_capacity_rows = need_expert;
    return FL_OK;
}

const char *fl_moe_strerror(int code) {
    switch (code) {
        case FL_OK: return "ok";
        case FL_ERR_INVALID_ARG: return "invalid argument";
        case FL_ERR_ALIGNMENT: return "pointer or size not aligned as required";
        case FL_ERR_WORKSPACE: return "workspace too small";
        case FL_ERR_HIP: return "HIP runtime error";
        case FL_ERR_STATIC_LIMIT:
            return "configuration needs more scratch than the library's static array (FL_STATIC_SCRATCH_BYTES)";
        default: return "unknown error";
    }
}

int fl_moe_debug_views(fl_moe_ctx *ctx, fl_moe_debug_view *out) {
    if (!ctx || !out) return FL_ERR_INVALID_ARG;
    const Tables &W = ctx->W;
    out->buf_a = W.bufA; out->buf_b = W.bufB;
    out->buf_a_rank_bytes = ctx->D.bufA_rank_bytes; out->buf_b_rank_bytes = ctx->D.bufB_rank_bytes;
    out->arrive_route = W.arrive_route; out->arrive_disp = W.arrive_disp;
    out->arrive_comb = W.arrive_comb;
    out->epoch_route = W.epoch_route; out->expect_disp = W.expect_disp; out->expect_comb = W.expect_comb;
    out->status = W.status;
    return FL_OK;
}

int fl_moe_debug_row_strides(const fl_moe_config *cfg, int64_t *dispatch_bytes, int64_t *combine_bytes) {
    if (!dispatch_bytes || !combine_bytes) return FL_ERR_INVALID_ARG;
    Dims D;
    int e = resolve(cfg, &D);
    if (e != FL_OK) return e;
    *dispatch_bytes = D.Sw;
    *combine_bytes = D.Sc;
    return FL_OK;
}

int fl_moe_debug_tune(fl_moe_ctx *ctx, int knob, int value) {
    if (!ctx || value < -1) return FL_ERR_INVALID_ARG;
    const bool dflt = value == -1;             // -1 = back to the default
    switch (knob) {
        case 0: if (value > kMaxRowsPerBlock) return FL_ERR_INVALID_ARG; ctx->D.tune_rows = dflt ? 0 : value; break;
        case 1: if (value > 8) return FL_ERR_INVALID_ARG; ctx->D.tune_reduce = dflt ? 0 : value; break;
        case 2: break;                         // shaped a copy kernel that is no longer launched: accepted, no effect
        case 3: if (value > 16) return FL_ERR_INVALID_ARG; ctx->D.tune_slices = dflt ? 0 : value; break;
        case 4: ctx->D.tune_cached_mb = dflt ? kCachedReplyMiB : value; break;
        case 5: if (value > 1000) return FL_ERR_INVALID_ARG; ctx->D.tune_grid_pct = value; break;
        case 6: ctx->launch_mb = dflt ? kLaunchMiB : value; break;
        case 7: if (value > 8 || value == 0) return FL_ERR_INVALID_ARG; ctx->D.tune_cap8 = dflt ? 3 : value; break;
        case 8: if (value > 2) return FL_ERR_INVALID_ARG; ctx->D.tune_order = dflt ? 0 : value; break;
        case 9: if (value > 64) return FL_ERR_INVALID_ARG; ctx->D.tune_parts = dflt ? 0 : value; break;
        case 11: ctx->D.tune_wait = dflt ? self_wait_waves(ctx->cu_count) : value; break;
        case 10: ctx->D.tune_self = dflt ? kSelfAnnounceBlocks : value; break;
        default: return FL_ERR_INVALID_ARG;
    }
    return FL_OK;
}

int fl_moe_debug_launch_groups(const fl_moe_config *cfg, int rank_count, int launch_mb, int *ranks_per_group) {
    if (!ranks_per_group || launch_mb < -1) return FL_ERR_INVALID_ARG;
    Dims D;
    int e = resolve(cfg, &D);
    if (e != FL_OK) return e;
    if (rank_count < 1 || rank_count > D.N) return FL_ERR_INVALID_ARG;
    *ranks_per_group = ranks_per_launch(D, launch_mb < 0 ? kLaunchMiB : launch_mb, rank_count);
    return FL_OK;
}

int fl_moe_debug_launch_plan(const fl_moe_config *cfg, int rank_count, fl_moe_launch_plan *out) {
    if (!out) return FL_ERR_INVALID_ARG;
    Dims D;
    int e = resolve(cfg, &D);
    if (e != FL_OK) return e;
    if (rank_count < 1 || rank_count > D.N) return FL_ERR_INVALID_ARG;
    out->unpack_by_chunks = unpack_by_chunks(D, kComputeUnits, rank_count);
    out->replies_by_chunks = replies_by_chunks(D, kComputeUnits, rank_count);
    out->replies_cached = replies_cached(D, rank_count);
    out->layout_blocks = layout_parts(D, kComputeUnits, rank_count);
    out->layout_tiles = (D.T + D.TT - 1) / D.TT;
    out->recv_grid_rows = recv_grid_rows(D);
    out->reply_grid_rows = reply_grid_rows(D);
    return FL_OK;
}

int fl_moe_debug_ordering_plan(const fl_moe_config *cfg, int rank_count, int cached_mb, fl_moe_ordering_plan *out) {
    if (!out || cached_mb < -1) return FL_ERR_INVALID_ARG;
    Dims D;
    int e = resolve(cfg, &D);
    if (e != FL_OK) return e;
    if (rank_count < 1 || rank_count > D.N) return FL_ERR_INVALID_ARG;
    if (cached_mb >= 0) D.tune_cached_mb = cached_mb;
    const bool own = D.flags & (FL_FLAG_PROGRESSIVE_RECV | FL_FLAG_STREAM_ORDERED);    // modes without announce kernels
    const ReplyForm form = reply_form(D, kComputeUnits, rank_count);
    out->dispatch_announce_kernel = !own && !announces_itself(D, dispatch_workgroups(D, false), rank_count);
    out->replies_written_through = (D.flags & FL_FLAG_PROGRESSIVE_RECV) || form != kRepliesStreamed;
    out->combine_announce_kernel = !own && form != kRepliesThroughAnnounced;
    const CallSpan call{0, rank_count, true, true};
    const int group = ranks_per_launch(D, kLaunchMiB, rank_count);
    out->dispatch_gate_kernel = !own && !unpack_waits(D, kComputeUnits, call, group);
    out->combine_gate_kernel = !own && !waits_itself(D, reduce_shape(D, kComputeUnits, group).waves(), call, group);
    return FL_OK;
}

// launch shapes of the three plain kernels: the fastest measured for each (see the kernels)
constexpr int kPlainCopyThreads = 64, kPlainCopyVecs = 4;
constexpr int kPlainFillThreads = 256, kPlainFillVecs = 1;
constexpr int kPlainReadThreads = 1024, kPlainReadVecs = 1;

int fl_moe_debug_copy(void *dst, const void *src, size_t bytes, void *stream) {
    if (!dst || !src || bytes == 0 || bytes % 16 != 0) return FL_ERR_INVALID_ARG;
    if (!aligned16(dst) || !aligned16(src)) return FL_ERR_ALIGNMENT;
    const size_t nvec = bytes / 16, per = (size_t)kPlainCopyThreads * kPlainCopyVecs;
    const size_t blocks = (nvec + per - 1) / per;
    if (blocks >= (1ull << 31)) return FL_ERR_INVALID_ARG;
    plain_copy_kernel<kPlainCopyThreads, kPlainCopyVecs>
        <<<dim3((unsigned)blocks), dim3(kPlainCopyThreads), 0, (hipStream_t)stream>>>((v4u *)dst, (const v4u *)src, nvec);
    return launch_status();
}

int fl_moe_debug_fill(void *dst, size_t bytes, void *stream) {
    if (!dst || bytes == 0 || bytes % 16 != 0) return FL_ERR_INVALID_ARG;
    if (!aligned16(dst)) return FL_ERR_ALIGNMENT;
    const size_t nvec = bytes / 16, per = (size_t)kPlainFillThreads * kPlainFillVecs;
    const size_t blocks = (nvec + per - 1) / per;
    if (blocks >= (1ull << 31)) return FL_ERR_INVALID_ARG;
    plain_fill_kernel<kPlainFillThreads, kPlainFillVecs>
        <<<dim3((unsigned)blocks), dim3(kPlainFillThreads), 0, (hipStream_t)stream>>>((v4u *)dst, nvec, 0x3C3C3C3Cu);
    return launch_status();
}

int fl_moe_debug_read(const void *src, size_t bytes, void *sink, void *stream) {
    if (!src || !sink || bytes == 0 || bytes % 16 != 0) return FL_ERR_INVALID_ARG;
    if (!aligned16(src) || ((uintptr_t)sink & 3)) return FL_ERR_ALIGNMENT;
    const size_t nvec = bytes / 16, per = (size_t)kPlainReadThreads * kPlainReadVecs;
    const size_t blocks = (nvec + per - 1) / per;
    if (blocks >= (1ull << 31)) return FL_ERR_INVALID_ARG;
    plain_read_kernel<kPlainReadThreads, kPlainReadVecs>
        <<<dim3((unsigned)blocks), dim3(kPlainReadThreads), 0, (hipStream_t)stream>>>((const v4u *)src, nvec,
                                                                                       (unsigned *)sink);
    return launch_status();
}

int fl_moe_profile_enable(fl_moe_ctx *ctx, int on) {
    if (!ctx) return FL_ERR_INVALID_ARG;
    if (on && !ctx->ev_start[kEventPool - 1]) {     // first use: the event pool
        for (int i = 0; i < kEventPool; ++i) {
            if (!ctx->ev_start[i] && hipEventCreate(&ctx->ev_start[i]) != hipSuccess) return FL_ERR_HIP;
            if (!ctx->ev_stop[i] && hipEventCreate(&ctx->ev_stop[i]) != hipSuccess) return FL_ERR_HIP;
        }
    }
    ctx->profile = on ? 1 : 0;
    ctx->ev_used = 0;
    return FL_OK;
}

int fl_moe_profile_collect(fl_moe_ctx *ctx, void *stream) {
    if (!ctx) return FL_ERR_INVALID_ARG;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return FL_ERR_HIP;
    for (int i = 0; i < ctx->ev_used; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, ctx->ev_start[i], ctx->ev_stop[i]) != hipSuccess)
            return FL_ERR_HIP;
        ctx->total_ms[ctx->ev_kernel[i]] += ms;
        ctx->launches[ctx->ev_kernel[i]] += 1;
    }
    ctx->ev_used = 0;
    return FL_OK;
}

int fl_moe_profile_read(fl_moe_ctx *ctx, double *total_ms, int64_t *launches) {
    if (!ctx || !total_ms || !launches) return FL_ERR_INVALID_ARG;
    for (int i = 0; i < FL_KERNEL_COUNT; ++i) {
        total_ms[i] = ctx->total_ms[i];
        launches[i] = ctx->launches[i];
    }
    return FL_OK;
}

#ifndef FLMOE_BUILD_ID
#define FLMOE_BUILD_ID "unknown"
#endif
const char *fl_moe_build_id(void) { return FLMOE_BUILD_ID; }

const char *fl_moe_kernel_name(int kernel_id) {
    if (kernel_id < 0 || kernel_id >= FL_KERNEL_COUNT) return "";
    return kKernelNames[kernel_id];
}

}  // extern "C"
