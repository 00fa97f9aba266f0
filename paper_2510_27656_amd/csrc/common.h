// Shared device-side definitions of the flmoe kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/flmoe.h"

namespace flmoe {

constexpr int kWave = 64;

// Shapes and strides of one context; passed to every kernel by value.
struct Dims {
    int N, E, El, T, K, H;
    int dtype, align, flags;
    int TT;               // tokens per LDS tile of the counting blocks (multiple of 32)
    int route_len;        // 8-byte words of one route record (route_record_words)
    int scales_per_row;   // 0 or H/128
    long long recv_cap, expert_cap, send_cap;   // rows per rank
    int P;                // private rows per (source, destination) at the head of a receive buffer
    long long recv_rows;  // physical rows of a dispatch receive buffer: N*P private + recv_cap shared
    long long Bx, Bw, Be, Bc;                   // row bytes: input, wire, expert_x, combine
    int Sw, Sc;           // bytes from row to row of a dispatch, a combine receive buffer (row_stride)
    long long bufA_rank_bytes, bufB_rank_bytes;
    long long spin_limit;
    int KM;               // sidecar entries per row: K rounded up to a multiple of 4
    int MW;               // words per sidecar row: KM, or 2*KM when the routing weights travel too
    int tune_rows;        // rows per block of the kernels that take chunks of rows (0 = by row size)
    int tune_reduce;      // loads in flight per thread in the reduce kernel (0 = all K)
    int tune_slices;      // blocks per token in the pack kernel (0 = by row size)
    int tune_cached_mb;   // combine replies are written through up to this many MiB of the group, then streamed (replies_cached)
    int tune_grid_pct;    // row-kernel grids cover this percentage of the rows uniform routing would bring
                          // (0 = the whole capacity, -1 = the mean and six standard deviations); kernels
                          // loop over whatever is beyond
    long long typ_recv_rows, typ_pair_rows;   // per rank, under uniform routing: received rows, pairs
    int tune_parts;       // workgroups per token in the reduce kernel (0 = by row size)
    int tune_order;       // test switch: order in which the send kernels take their rows
    int tune_self;        // send calls of up to this many workgroups announce their transfers themselves (announces_itself)
    int tune_wait;        // receive launches of up to this many waves wait for the counters themselves (waits_itself)
    int tune_cap8;        // progressive receivers: eighths of the machine's block slots their grids may take
};

// Row of a dispatch receive buffer that holds the i-th row source s sent to this
// rank: the first P rows of every source have fixed private slots at the head of
// the buffer (known without any exchange), later rows are packed into the shared
// range behind them in source order (section MoE Dispatch/Combine, figure
// "Dispatch into private and contiguous buffers").
__host__ __device__ inline int recv_buffer_row(int N, int P, int s, int i, int shared_start) {
    return i < P ? s * P + i : N * P + shared_start + (i - P);
}

// Device pointers into the caller's workspace.
struct Tables {
    int *status;
    unsigned *epoch_route;                                    // [N] layout calls of each rank
    unsigned *arrive_route;                                   // [N dst][N src] step of the last route record received
    // Payload counters, monotone: a completed transfer adds its payload in 16-byte units
    // plus one (default: by the announce kernel behind the payload kernels, or their last
    // workgroup; stream-ordered callers: by the send kernel's first block; progressive mode: the
    // units by every copying block); expect_* is advanced by the receiver's own planning block from the
    // counts it was sent, so a receiver waits for arrive >= expect per source.
    unsigned *arrive_disp, *arrive_comb;                      // [N dst][N src]
    unsigned *expect_disp, *expect_comb;                      // [N dst][N src]
    unsigned *done_disp, *done_comb;  // [N][kDoneWords] workgroups of a sender's kernel that have ended (announce_when_last);
                                      // behind them verdicts of receive launches that wait themselves (done_words)
    unsigned long long *routes;   // [N receiver][N source][route_len], in words that carry their step's number
    // written by the source side of the layout step
    int *C;               // [N][E]
    int *M;               // [N][N]
    int *send_off;        // [N][N+1]
    int *comb_off;        // [N][N+1]
    int *send_to;         // [N][T][K]  for the first slot of each destination: (destination << 24) | number of this
                          //            copy among those the source sends there, in token order; else ~destination
    unsigned *pair_meta;  // [N][T][K]  (local expert << 24) | rank of the token among the source's tokens of that expert
    int *comb_pos;        // [N][T][K]
    // written by the receiving side of the layout step
    int *G;               // [N][El]
    int *expert_off;      // [N][El+1]
    int *recv_off;        // [N][N+1]         received rows of lower sources (the order unpack walks)
    int *recv_shared_off; // [N dst][N src]   shared-range rows of lower sources: sum of max(M - P, 0)
    int *dst_off;         // [N src][N dst]   the same number as seen by the sender: where src's rows
                          //                  beyond its private slots start in dst's shared range
    int *comb_dst_off;    // [N d][N s]       row in s's combine receive buffer where d's reply starts
    int *ret_off;         // [N d][N s]       partial sums: row in s's buffer where d's shares start,
                          //                  = rows s sent to lower ranks (send_off[s][d])
    int *base_x;          // [N][El][N]       first expert-major row of (local expert, source)
    int *cs_base;         // [N][N][El]       first combine-send row of (source, local expert)
    int *cs_off;          // [N][N+1]         first combine-send row of each source
    int *plan_ok;         // [N]
    int *gate_disp;       // [N] default mode: 1 once the gate kernel saw every source's dispatch payload complete
    int *gate_comb;       // [N] the same for the combine replies
    unsigned *recv_meta;  // [N][recv_rows][MW]
    char *bufA;           // [N][bufA_rank_bytes]  combine receive buffer
    char *bufB;           // [N][bufB_rank_bytes]  dispatch receive buffer
};

constexpr unsigned kNoEntry = 0xFFFFFFFFu;
constexpr int kDoneParts = 16;                           // partial counts, then their count, ...
constexpr int kDoneLine = 32;                            // ... each on a 128-byte line of its own
constexpr int kDoneWords = (kDoneParts + 1) * kDoneLine;

// ---------------------------------------------------------------- atomics
// FENCED names the progressive mode, in which senders and receivers overlap in time
// inside their kernels: every sending block reports the units it delivered and the
// receive kernels poll.  On gfx950 each XCD has its own L2, so a payload only
// becomes visible to a receiver on another XCD once it has left the sender's L2.
// An agent-scope release fence would write back the whole L2 (measured: 5x to 25x
// slower copy kernel, depending on how many waves fence).  Instead the sender
// writes the payload with device-scope stores (sc1: written through to memory),
// waits until its own stores are acknowledged, and only then updates the counter;
// the receiver polls the counter with device-scope loads and, once it has arrived,
// invalidates its caches (agent-scope acquire) before touching the payload.
// FENCED = false covers the other two modes.  Default: the announce kernel behind the payload
// kernels orders payload and counters, or, in small calls that write through, the last workgroup to have
// seen its stores acknowledged (announce_when_last); the receive kernels start behind a gate kernel, or,
// in small launches, wait as in progressive mode, with one verdict per rank (wave_wait_together).
// FL_FLAG_STREAM_ORDERED: the caller's stream order does; nothing waits for the payload
// stores inside the kernels then, and the in-kernel counter accesses are relaxed atomics.
__device__ inline unsigned ld_relaxed(const unsigned *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The result is never used, so the hardware atomic does not return a value and
// the wave does not wait for it.
__device__ inline void add_counter(unsigned *p, unsigned v) {
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// After a wave's last payload store and before the add that vouches for it: waits until every
// store of this wave (including the device-scope ones issued from inline assembly, which
// the compiler does not count) has been acknowledged.
__device__ inline void stores_done() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
template <bool FENCED>
__device__ inline void acquire_payload() {
    if (FENCED) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}
__device__ inline void st_word(int *p, int v) {        // small table entries pushed to a peer: written through, as rows are
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void latch_status(int *status, int bit) {
    __hip_atomic_fetch_or(status, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether a counter has reached its expectation; both wrap, so the difference is taken in unsigned words
// (a signed one may be compiled into a plain comparison, which fails while they pass 2^31).
__device__ inline bool arrived(unsigned have, unsigned want) { return (int)(have - want) >= 0; }

// Bounded wait of one wavefront: lane i (< n) polls ctr[i] until it has reached
// its expectation (wrap-safe comparison; `expect` is either one value for all or,
// with expect_arr, one per counter).  Returns true when all n counters arrived,
// false when the poll budget ran out.  Every lane of the wave must call it.
// Polls are 64 * 64 clocks apart (with the load about 1.8 us): a wait may last as long as a copy kernel and must not
// crowd out the senders it waits for.
__device__ inline bool wave_wait_counters(const unsigned *ctr, const unsigned *expect_arr,
                                          unsigned expect, int n, long long spin_limit) {
    const int lane = threadIdx.x & (kWave - 1);
    for (int base = 0; base < n; base += kWave) {
        const int i = base + lane;
        long long spins = 0;
        if (expect_arr && i < n) expect = expect_arr[i];
        for (;;) {
            bool ok = true;
            if (i < n) ok = arrived(ld_relaxed(ctr + i), expect);
            if (__all(ok)) break;
            if (++spins > spin_limit) return false;
            __builtin_amdgcn_s_sleep(64);
        }
    }
    return true;
}

// The same wait by many waves of one launch which must all come to one verdict, so that a delivery at the very end of
// the wait does not leave part of a rank's output written: every wave may go ahead, or none.
// One wave of the launch decides.  When its polls are used up it writes `closing` into *word, waits until the store is in
// memory, looks once more, and writes what it found.  Every other wave reads the word after it has seen the counters
// arrive.  If it reads no `closing`, its look at the counters came before the deciding wave's last one, which
// therefore sees them arrived as well: it may go ahead.  Otherwise it waits for what the deciding wave finds.
// So a launch whose senders come in time writes nothing here, and a wave's verdict costs one more load, which need
// not have returned before the wave's first store (verdict_read, verdict_allows).
// ticket: names this launch in the word, so that nothing has to be cleared on the way.  A graph that holds the receive call
// but not the layout repeats the ticket, so a verdict to give up is cleared by the last wave that leaves on it (verdict_left).
typedef unsigned long long verdict_word;
constexpr unsigned kVerdictClosing = 1, kVerdictCame = 2, kVerdictGaveUp = 3;
__device__ inline verdict_word launch_ticket(unsigned step, unsigned launch) {
    return (verdict_word)step << 32 | (verdict_word)(launch & 0x3FFFFFFFu) << 2;
}
// of rank r; done: done_disp, done_comb.  (Two more pointers in Tables took the kernels' arguments past 768 bytes and
// 0.1 us a launch: 8 ranks one by one 196.2 -> 199.3 us a step.)
// Behind the verdicts, as many words of verdict_left.
__host__ __device__ inline size_t done_words(int N) { return (size_t)N * kDoneWords + 4 * (size_t)N; }
__device__ inline verdict_word *verdict_of(unsigned *done, int N, int r) {
    return (verdict_word *)(done + (size_t)N * kDoneWords) + r;
}
__device__ inline verdict_word verdict_read(const verdict_word *word) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");      // after the counters
    return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// w: the word as read after the counters had arrived.  Whether the wave may go ahead; the deciding wave is between its
// two stores where this has to wait (bounded all the same).
__device__ inline bool verdict_allows(const verdict_word *word, verdict_word ticket, verdict_word w) {
    for (int polls = 0; w == (ticket | kVerdictClosing) && polls < 65536; ++polls) {
        __builtin_amdgcn_s_sleep(16);
        w = verdict_read(word);
    }
    return w != (ticket | kVerdictClosing) && w != (ticket | kVerdictGaveUp);
}
// Counts `waves` of the `all` waves of a rank's launch that leave without having stored; each is counted once, after it
// has read the word for the last time, and the last one clears the word.  One lane calls it, only after a wait that gave up.
__device__ inline void verdict_left(verdict_word *word, int N, verdict_word ticket, unsigned waves, unsigned all) {
    constexpr verdict_word kCount = (1u << 20) - 1;
    verdict_word *left = word + N;
    const verdict_word mine = ticket << 18 & ~kCount;           // the launch's number and the low bits of the step's
    verdict_word old = __hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
    do next = ((old & ~kCount) == mine ? old : mine) + waves;
    while (!__hip_atomic_compare_exchange_strong(left, &old, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if ((next & kCount) != all) return;
    __hip_atomic_store(left, (verdict_word)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(word, (verdict_word)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The wait of a wave whose first look at the counters (have, lane = counter) did not find them all arrived.
// A wave that finds no verdict in four times the polls gives up by itself: only if the deciding wave, in the rank's first
// workgroup, never ran.  The first 64 polls are a quarter as far apart and are not counted: a small receive launch is
// mostly there a few microseconds before its senders are done.  n <= 64; whole wave.
__device__ inline bool wave_wait_together(const unsigned *ctr, unsigned have, unsigned want, int n, long long spin_limit,
                                          verdict_word *word, verdict_word ticket, bool decides, int *status) {
    const int lane = threadIdx.x & (kWave - 1);
    auto came = [&]() { return __all(lane >= n || arrived(have, want)) != 0; };
    auto look = [&]() { if (lane < n) have = ld_relaxed(ctr + lane); };
    auto write = [&](unsigned verdict) {
        if (lane == 0) __hip_atomic_store(word, ticket | verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stores_done();
    };
    long long spins = 0;
    for (int quick = 64; !came();) {
        if (spins > spin_limit) {
            if (decides) {
                write(kVerdictClosing);
                look();
                const bool late = came();
                write(late ? kVerdictCame : kVerdictGaveUp);
                if (!late && lane == 0) latch_status(status, FL_STATUS_TIMEOUT);
                return late;
            }
            const verdict_word w = verdict_read(word);
            if (w == (ticket | kVerdictCame)) return true;
            if (w == (ticket | kVerdictGaveUp)) return false;
            if ((spins - 1024) >> 2 > spin_limit) {
                if (lane == 0) latch_status(status, FL_STATUS_TIMEOUT);
                return false;
            }
        }
        if (quick > 0) {
            --quick;
            __builtin_amdgcn_s_sleep(16);
        } else {
            ++spins;
            __builtin_amdgcn_s_sleep(64);
        }
        look();
    }
    return decides || verdict_allows(word, ticket, verdict_read(word));
}

// ---------------------------------------------------------------- scans / search
// Inclusive scan over the wave, all 64 lanes active: within rows of 16 lanes by shifts, then the
// last lane of each row (of each half) carried into the next.  Six data-parallel adds; through
// LDS permutes the same scan takes some ten times as long.
__device__ inline int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);    // row_shr:1, lanes without a source add 0
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);    // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);    // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);    // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);    // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);    // row_bcast:31 into rows 2 and 3
    return v;
}

// Exclusive scan over the block (one value per thread, blockDim <= 1024); only the first
// `waves` waves hold values other than zero.  tmp: LDS int[17].  *total receives the block
// sum.  Contains two barriers.
__device__ inline int block_excl_scan(int v, int *tmp, int *total, int waves) {
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int inc = wid < waves ? wave_incl_scan(v) : 0;
    __syncthreads();
    if (lane == kWave - 1) tmp[wid] = inc;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < waves; ++w) {          // the same words for every thread
        if (w == wid) before = all;
        all += tmp[w];
    }
    *total = all;
    return inc - v + before;
}

// Largest i in [0, n) with off[i] <= x; needs off[0] <= x.  With equal
// neighbours (empty segments) this is the segment that really contains x.
__device__ inline int seg_of(const int *off, int n, int x) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// seg_of for a short table in global memory: all entries are fetched at once (one
// round trip instead of one per halving step); *start receives off[result].
__device__ inline int seg_of_short(const int *off, int n, int x, int *start) {
    if (n > 16) {
        const int j = seg_of(off, n, x);
        *start = off[j];
        return j;
    }
    int c[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = i < n ? off[i] : 0x7fffffff;
    int j = 0, cj = c[0];
#pragma unroll
    for (int i = 1; i < 16; ++i)
        if (c[i] <= x) { j = i; cj = c[i]; }
    *start = cj;
    return j;
}

// ---------------------------------------------------------------- row copies
// 16-byte streaming accesses.  The payload of every copy kernel is touched once
// per kernel, so loads, and the unpack kernel's stores, carry the non-temporal hint; on this part a
// plain copy with these hints and four independent loads per thread in flight
// measured fastest (more loads in flight per CU than that overruns the L2).
typedef unsigned v4u __attribute__((ext_vector_type(4)));
__device__ inline v4u ld_stream(const v4u *p) { return __builtin_nontemporal_load(p); }
__device__ inline void st_stream(v4u *p, v4u v) { __builtin_nontemporal_store(v, p); }
// 16-byte load at device scope from a row whose address is the same in the whole wave: what another XCD has written
// through is seen whatever the caches here hold, as by the counters' own loads (with the streaming hint it takes as
// long as ld_stream).
__device__ inline v4u ld_coherent(const char *row, int vec) {
    constexpr int kDeviceScopeStreaming = 0x12;             // sc1, nt
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)row, 0, 0x7FFFFFFF, 0x00020000);
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, vec * 16, 0, kDeviceScopeStreaming);
}
// 16-byte store at device scope: written through the XCD's L2 to memory, where every XCD sees it once it
// has been acknowledged.  No dirty line is left for the end of the kernel, which otherwise waits until the
// L2s have written theirs back (32 ranks x 4 tokens: 3.9 us from the pack kernel's last store to the next
// kernel's first instruction, 1.5 behind a kernel without dirty lines).
// The hardware reads the data of a 128-bit store a little after it has issued: a vector instruction may overwrite those
// registers two wait states later at the earliest.  The compiler sees to that behind its own stores, not behind inline
// assembly, hence the s_nop.  (Buffer stores, which take the same cache bits as a builtin, need one base for the whole wave;
// here every lane may store into another rank's buffer.)
__device__ inline void st_through(v4u *p, v4u v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// The same with the streaming hint, for whole lines: what the unpack kernel hands the caller.  Neither dirty lines at
// the end of the kernel nor lines kept for nobody.  us of a step, streaming stores -> this: 128 tokens of 14 KB 451.4 -> 448.4,
// 32: 132.7 -> 131.8; 2048 tokens and 45 ready-made e4m3 tokens: no difference beyond noise (1 %); rows that end inside
// lines lose (6672 bytes, 301 tokens 96.6 -> 101.3) and keep the streaming stores.
__device__ inline void st_through_stream(v4u *p, v4u v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");      // as in st_through
}
// Payload store into a peer's receive buffer: written through (THROUGH), so that the last-level cache may
// hold the rows until the receive kernel reads them, or a streaming store.  us of a DeepSeek-V3 step with
// ordinary stores in the send kernels -> written through: 4 tokens per rank 47.2 -> 46.2, 32: 136.8 -> 135.8,
// 128: 465 -> 455, e4m3 128: 368 -> 362, 256: 990 -> 964; replies streamed instead: 128 487, 256 975 (larger
// calls: replies_cached).  Dispatch rows never lose written through.  All of top 8.  Of the kernels that write what the
// caller reads, the reduce kernel writes through as well (128: 455 -> 452, 32: 135.8 -> 134.0, 16 ranks x 256 tokens of
// 4 KB 123.4 -> 120.3, e4m3 512: 1523 -> 1478), with the streaming hint where one or two rows make up a sum (see there);
// the unpack kernel writes whole lines through with the hint and streams other rows (written through without the hint,
// 128: 505, e4m3 393; ordinary stores 490: the write-backs land on the kernel after).
template <bool THROUGH>
__device__ inline void st_payload(v4u *p, v4u v) {
    if (THROUGH) st_through(p, v);
    else st_stream(p, v);
}

// Vectors rounded up to whole 128-byte lines: slices of a row that starts on a line do so as well (rows of 14 352
// bytes, 128 tokens per rank: pack kernel 103 -> 86 us with slices of 113 vectors -> 136, reduce 85 -> 81).
__host__ __device__ inline int whole_lines(int vecs) { return (vecs + 7) / 8 * 8; }

// A block copies `nrows` rows of `nvec` vectors each; vector v of the chunk lies
// in row v / nvec.  src_of(row) / dst_of(row) return the row's byte address.
// All loads of a batch are issued before its stores.
template <int NT, bool THROUGH, class SrcFn, class DstFn>
__device__ inline void copy_rows_flat(int nrows, int nvec, int tid, SrcFn src_of, DstFn dst_of) {
    if (nrows == 1) {                          // one row per block: addresses are uniform
        const v4u *s = (const v4u *)src_of(0);
        v4u *d = (v4u *)dst_of(0);
        for (int b = tid; b < nvec; b += 4 * NT) {
            v4u r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b + i * NT < nvec) r[i] = ld_stream(s + b + i * NT);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b + i * NT < nvec) st_payload<THROUGH>(d + b + i * NT, r[i]);
        }
        return;
    }
    const int total = nrows * nvec;
    for (int b = tid; b < total; b += 4 * NT) {
        v4u r[4];
        int row[4], col[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = b + i * NT;
            if (v < total) {
                row[i] = v / nvec;
                col[i] = v - row[i] * nvec;
                r[i] = ld_stream((const v4u *)src_of(row[i]) + col[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = b + i * NT;
            if (v < total) st_payload<THROUGH>((v4u *)dst_of(row[i]) + col[i], r[i]);
        }
    }
}

// ---------------------------------------------------------------- bf16
__device__ inline float bf16_lo(unsigned u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(unsigned u) { return __uint_as_float(u & 0xffff0000u); }
__device__ inline unsigned f32_to_bf16_bits(float f) {
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;   // NaN stays a quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);                                  // ties to even
    return u >> 16;
}
__device__ inline unsigned pack_bf16x2(float lo, float hi) {
    return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

}  // namespace flmoe
