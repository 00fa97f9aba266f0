// Layout step: counting, deterministic ranks, route exchange, offset tables.
//
// Paper, section MoE Dispatch/Combine: the dispatch kernel first counts the
// tokens sent to each expert in shared memory (Dispatch); all peers exchange
// these per-expert counts to determine a unique range in each contiguous receive
// buffer (Architecture).  The paper computes the ranges on a host proxy; here
// both halves run on the device.
//
// Bound by latency: a few KB per rank go through one chain of load, count, exchange, scan.
// So every link is one round of independent loads or one pass of all the block's
// threads.  32 ranks, 256 experts, top 8, from the first block's first instruction to the last
// one's last, message counters behind the route records -> words that carry their step: 4 tokens
// per rank 9.9 -> 8.4 us (ids there 1.6, counts 2.3, records pushed 2.9, received 5.3, sums 6.7),
// 128: 10.9 -> 9.2; 2 ranks x 16 tokens 7.2 -> 5.8.  2048 tokens 22 (a third of it the count of
// all tokens in every counting block).
#pragma once
#include "common.h"

namespace flmoe {

constexpr int kRouteThreads = 1024;
constexpr int kRoutePreload = 4;             // pair ids a thread fetches while the bit matrices are being cleared

// Words per row of the LDS bit matrices: the words in use, padded to an odd
// number so that rows do not all start in the same bank.
__host__ __device__ inline int route_row_stride(int TT) { return (TT / 32) | 1; }

__host__ __device__ inline size_t route_count_lds_bytes(int E, int N, int K, int TT) {
    size_t rows = (size_t)E + N;
    return rows * route_row_stride(TT) * 2 * sizeof(unsigned) + rows * 5 * sizeof(int) + 32 * sizeof(int) +
           (size_t)TT * K * sizeof(unsigned short);
}

// Route record, one per (receiver, source), of 8-byte words that each say which step they belong to: the source's E
// expert counts and N per-rank counts, three 16-bit counts a word (one of 32 bits where T does not fit), behind a
// head, which is known last: the first row of the receiver's reply in the source's combine receive buffer.
// A word is stored whole, so a receiver that finds this step's tag in it has the word's counts: the exchange costs
// one store and one load, where a message counter behind the record cost the sender an acknowledgement and an add
// and the receiver a poll, an invalidation of its caches and another load.
// The tag: bit 15 marks a word as written, bit 14 says whether the source's ids were valid, below are the lowest
// bits of the step's number.  Every step writes every word, so what a receiver may find is the step before, this
// one, or, when calls that contain nothing but the layout step run ahead on another stream, the next.
typedef unsigned long long route_word;
__host__ __device__ inline bool route_wide(int T) { return T > 65535; }
__host__ __device__ inline int route_per_word(bool wide) { return wide ? 1 : 3; }
__host__ __device__ inline int route_record_words(int E, int N, int T) {
    const int per = route_per_word(route_wide(T));
    return 1 + (E + N + per - 1) / per;
}
__device__ inline unsigned route_tag(unsigned step) { return 0x8000u | (step & 0x3FFFu); }
constexpr unsigned kRouteValid = 0x4000u;
__device__ inline bool route_ready(route_word w, unsigned tag) {
    const unsigned have = (unsigned)(w >> 48);
    return (have & 0x8000u) && ((have - tag) & 0x3FFFu) <= 1u;
}
__device__ inline route_word ld_route(const route_word *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_route(route_word *p, route_word v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// e / El for 0 <= e < 1024 and El <= 256 by a multiplication: m = ceil(2^20 / El),
// exact because e * (El - 1) < 2^20.
__device__ inline unsigned div_magic(int El) { return ((1u << 20) + El - 1) / (unsigned)El; }
__device__ inline int div_by(unsigned e, unsigned m) { return (int)((e * m) >> 20); }

// Counts the tokens [t0, t1) of one source, one per thread and turn: hit(t, row) for every expert that token t
// lists and, once each, for every rank (row E + rank) with one of its experts.  A token counts once per expert and
// once per rank, as in the bit matrices below; ids outside the range or repeated raise *bad.  KT >= K: with a loop of
// the largest top-k there is, comparing ids took most of the time (2048 tokens x top 8: 10 us of the layout kernel).
template <int KT, class HitFn>
__device__ __forceinline__ void count_tokens(const int *__restrict__ ids, int t0, int t1, int threads, int E, int K,
                                             unsigned by_el, int *bad, HitFn hit) {
    bool wrong = false;
    for (int t = t0 + (int)threadIdx.x; t < t1; t += threads) {
        int id[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) id[k] = k < K ? ids[(size_t)t * K + k] : -1;
        unsigned long long ranks = 0;                      // N <= 64
#pragma unroll
        for (int k = 0; k < KT; ++k)
            if (k < K) {
                bool again = (unsigned)id[k] >= (unsigned)E;
#pragma unroll
                for (int k2 = 0; k2 < k; ++k2) again |= id[k2] == id[k];
                wrong |= again;
                if (again) continue;
                hit(t, id[k]);
                const int d = div_by(id[k], by_el);
                if (!(ranks >> d & 1)) hit(t, E + d);
                ranks |= 1ull << d;
            }
    }
    if (wrong) *bad = 1;
}

// Block `part` of the `parts` blocks of source rank s.
//
// For every tile of TT tokens a block keeps two LDS bit matrices: row e of the
// first has bit t set when token t lists expert e, row d of the second when any
// of token t's experts lives on rank d (OR-ing makes the per-destination
// de-duplication free and the result independent of thread order).  The rank of
// token t among the tokens that hit the same row, in token order, is then
//     rows_before_tile + popcount prefix of the row's words + popcount of the
//     bits below t in its word
// which is the stable counting-sort position the canonical (source rank, token
// index) order needs, with no ticket atomics.
//
// One tile (T <= TT): its popcounts are the counts.  Several: the tiles are shared out
// over the blocks, and every block first counts all of the source's tokens with LDS
// adds (and, apart, those before its own first tile), one token per thread: counting
// them again in every block costs less than the blocks would wait for each other's parts
// unless there are many tokens, and keeps a counting block from ever waiting.  One scan over
// the E + N totals gives the offsets.  The last pass writes every pair's final positions.
//
// Outputs for rank s: by part 0, C[s][.], M[s][.], send_off[s][.], comb_off[s][.] and the
// route record, which is pushed into every peer's routes[peer][s]; by every part, send_to /
// pair_meta / comb_pos of the pairs of its tiles.
template <bool WIDE>
__device__ __forceinline__ void route_count_block(const Dims &D, const Tables &W, int s, int part, int parts,
                                                  const int *__restrict__ indices,
                                                  const int *__restrict__ num_tokens, unsigned *lds) {
    const int tid = threadIdx.x;
    const int E = D.E, N = D.N, El = D.El, K = D.K;
    const int rows = E + N;
    const int Wn = D.TT / 32;                              // words in use per row
    const int Wd = route_row_stride(D.TT);                 // row stride in words
    const unsigned by_el = div_magic(El);
    const unsigned by_k = 0xFFFFFFFFu / (unsigned)K + 1u;  // p / K for p < 2^16 by the high half of a product (K > 1)
    unsigned *bits = lds;                                  // [rows][Wd]
    unsigned *pre = bits + (size_t)rows * Wd;              // [rows][Wd] popcount prefix inside the tile
    int *count = (int *)(pre + (size_t)rows * Wd);         // [rows] hits over all tiles (C | M)
    int *start = count + rows;                             // [rows] exclusive scan of count
    int *base = start + rows;                              // [rows] hits in the tiles before the current one
    int *hits = base + rows;                               // [rows] hits of the current tile
    int *scan_tmp = hits + rows;                           // [17]
    unsigned short *ids = (unsigned short *)(scan_tmp + 20);   // [TT * K] expert ids of the tile
    __shared__ int bad;

    const int *idx_s = indices + (size_t)s * D.T * K;
    const int tiles = (D.T + D.TT - 1) / D.TT;             // of the capacity; the tokens in use may fill fewer
    const int per = (tiles + parts - 1) / parts;
    const int tile0 = part * per;
    int Ts = num_tokens[s];                                // on its way while the counters are cleared
    // its planning block counts the step once this one's record is there
    const unsigned tag = part == 0 ? route_tag(W.epoch_route[s] + 1u) : 0u;
    for (int r = tid; r < rows; r += kRouteThreads) { count[r] = 0; base[r] = 0; }
    if (tid == 0) bad = (Ts < 0 || Ts > D.T) ? 1 : 0;
    Ts = max(0, min(Ts, D.T));
    // the first ids are on their way while the bit matrices are cleared; never those of absent tokens,
    // which need not exist
    int early[kRoutePreload];
#pragma unroll
    for (int i = 0; i < kRoutePreload; ++i) {
        const int p = tid + i * kRouteThreads;
        early[i] = p < min(D.TT, Ts - tile0 * D.TT) * K ? idx_s[(size_t)tile0 * D.TT * K + p] : 0;
    }
    for (int i = tid; i < rows * Wd; i += kRouteThreads) bits[i] = 0;
    const int used = (Ts + D.TT - 1) / D.TT;
    __syncthreads();

    // bits (already cleared), ids, in-tile popcount prefixes and row totals of one tile
    auto fill_tile = [&](int t0, int nt, int *totals) {
        auto take = [&](int p, int e) {
            const bool ok = e >= 0 && e < E;
            ids[p] = (unsigned short)(ok ? e : 0xFFFF);
            if (!ok) { bad = 1; return; }
            const int tl = K > 1 ? (int)__umulhi((unsigned)p, by_k) : p;
            const unsigned bit = 1u << (tl & 31);
            const unsigned old = atomicOr(&bits[(size_t)e * Wd + (tl >> 5)], bit);
            if (old & bit) bad = 1;                        // same expert twice in one token
            atomicOr(&bits[(size_t)(E + div_by(e, by_el)) * Wd + (tl >> 5)], bit);
        };
#pragma unroll
        for (int i = 0; i < kRoutePreload; ++i) {
            const int p = tid + i * kRouteThreads;
            if (p < nt * K) take(p, t0 == tile0 * D.TT ? early[i] : idx_s[(size_t)t0 * K + p]);
        }
        for (int p = tid + kRoutePreload * kRouteThreads; p < nt * K; p += kRouteThreads)
            take(p, idx_s[(size_t)t0 * K + p]);
        __syncthreads();
        for (int r = tid; r < rows; r += kRouteThreads) {
            int run = 0;
            for (int w0 = 0; w0 < Wn; w0 += 4) {
                unsigned b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) b[i] = w0 + i < Wn ? bits[(size_t)r * Wd + w0 + i] : 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (w0 + i < Wn) pre[(size_t)r * Wd + w0 + i] = run;
                    run += __popc(b[i]);
                }
            }
            totals[r] = run;
        }
        __syncthreads();
    };

    if (tiles == 1) {
        fill_tile(0, Ts, count);
    } else {                                               // one token per thread and turn
        // the LDS adds are what this pass takes its time for: where both counts fit, one word holds the
        // total in its lower and the hits before this block's tiles in its upper half
        const int mine = min(tile0 * D.TT, Ts);
        auto hit = [&](int t, int row) {
            atomicAdd(&count[row], !WIDE && t < mine ? 0x10001 : 1);
            if (WIDE && t < mine) atomicAdd(&base[row], 1);
        };
        if (K <= 8) count_tokens<8>(idx_s, 0, Ts, kRouteThreads, E, K, by_el, &bad, hit);
        else count_tokens<FL_MAX_TOPK>(idx_s, 0, Ts, kRouteThreads, E, K, by_el, &bad, hit);
        __syncthreads();
        if (!WIDE) {
            for (int r = tid; r < rows; r += kRouteThreads) {
                const unsigned c = (unsigned)count[r];
                count[r] = (int)(c & 0xFFFFu);
                base[r] = (int)(c >> 16);
            }
            __syncthreads();
        }
    }

    // The counts go out as soon as they are known (every index was seen, so `bad` is final as well); the record's head
    // follows the scan.  The peers' planning overlaps with what is left to do here, the pair tables that
    // only this rank's later kernels read.
    route_word *to = W.routes + (size_t)s * D.route_len;   // in peer p's table: + p * N * route_len
    const size_t peer_step = (size_t)N * D.route_len;
    const route_word stamp = (route_word)(tag | (bad ? 0u : kRouteValid)) << 48;
    if (part == 0) {
        constexpr int kPer = WIDE ? 1 : 3;
        const int words = D.route_len - 1;
        for (int f = tid & (kWave - 1); f < words; f += kWave) {
            route_word v = stamp;                          // beyond the last count: whatever follows, never looked at
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                v |= WIDE ? (route_word)(unsigned)count[f] : (route_word)((unsigned)count[f * kPer + i] & 0xFFFFu) << (16 * i);
            for (int peer = tid / kWave; peer < N; peer += kRouteThreads / kWave) st_route(to + peer * peer_step + 1 + f, v);
        }
    }
    // one exclusive scan over the E + N totals (two slots per thread)
    {
        const int a = 2 * tid < rows ? count[2 * tid] : 0;
        const int b = 2 * tid + 1 < rows ? count[2 * tid + 1] : 0;
        int total;
        const int ex = block_excl_scan(a + b, scan_tmp, &total, (rows + 2 * kWave - 1) / (2 * kWave));
        if (2 * tid < rows) start[2 * tid] = ex;
        if (2 * tid + 1 < rows) start[2 * tid + 1] = ex + a;
    }
    __syncthreads();
    // start[e] = first combine-receive row of expert e; start[E + d] = pairs + send_off[d]
    const int pairs_total = start[E];
    if (part == 0) {
        if (tid < N) st_route(to + tid * peer_step, stamp | (unsigned)start[tid * El]);
        if (bad && tid == 0) latch_status(W.status, FL_STATUS_BAD_INDEX);
        if (tid < E) W.C[(size_t)s * E + tid] = count[tid];
        if (tid < N) {
            W.M[(size_t)s * N + tid] = count[E + tid];
            W.send_off[(size_t)s * (N + 1) + tid] = start[E + tid] - pairs_total;
            W.comb_off[(size_t)s * (N + 1) + tid] = start[tid * El];
        }
        if (tid == 0) {
            W.send_off[(size_t)s * (N + 1) + N] = start[E + N - 1] + count[E + N - 1] - pairs_total;
            W.comb_off[(size_t)s * (N + 1) + N] = pairs_total;
        }
    }

    // final position of every pair of this block's tiles
    for (int tile = tile0; tile < min(tile0 + per, used); ++tile) {
        const int t0 = tile * D.TT, nt = min(D.TT, Ts - t0);
        if (tiles > 1) {
            if (tile > tile0) {                            // behind the tile before
                __syncthreads();
                for (int r = tid; r < rows; r += kRouteThreads) base[r] += hits[r];
                for (int i = tid; i < rows * Wd; i += kRouteThreads) bits[i] = 0;
                __syncthreads();
            }
            fill_tile(t0, nt, hits);
        }
        for (int p = tid; p < nt * K; p += kRouteThreads) {
            const int tl = K > 1 ? (int)__umulhi((unsigned)p, by_k) : p, k = p - tl * K;
            const int e = ids[p];
            if (e == 0xFFFF) continue;
            const int d = div_by(e, by_el);
            const unsigned below = (1u << (tl & 31)) - 1u;
            const int w = tl >> 5;
            const int re = e, rd = E + d;
            const int rank_e =
                base[re] + pre[(size_t)re * Wd + w] + __popc(bits[(size_t)re * Wd + w] & below);
            const int rank_d =
                base[rd] + pre[(size_t)rd * Wd + w] + __popc(bits[(size_t)rd * Wd + w] & below);
            bool first = true;                             // first slot of this token bound for rank d?
            for (int k2 = 1; k2 <= k; ++k2) {
                const unsigned e2 = ids[p - k2];
                if (e2 != 0xFFFFu && div_by(e2, by_el) == d) first = false;
            }
            const size_t o = ((size_t)s * D.T + t0) * K + p;
            W.comb_pos[o] = start[re] + rank_e;
            W.pair_meta[o] = ((unsigned)(e - d * El) << 24) | (unsigned)rank_e;
            W.send_to[o] = first ? d << 24 | rank_d : ~d;
        }
    }
}

__host__ __device__ inline size_t route_plan_lds_bytes(int E, int N, int El) {
    return ((size_t)3 * E /*all ranks' totals, own columns, own row*/ + (size_t)N * (N + 1) /*M*/ + El + 1 + (size_t)N) * sizeof(int);
}

// One block per rank r: takes the route records of all sources as they arrive (bounded),
// then derives every table rank r needs for the step: one phase of sums and scans, a wave
// each, and one that uses them.  All ranks see the same records, so all reach
// the same verdict on validity and capacity: a bad step is skipped by everyone
// without further communication.
template <bool WIDE>
__device__ __forceinline__ void route_plan_block(const Dims &D, const Tables &W, int r, unsigned *lds) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    constexpr int kWaves = kRouteThreads / kWave;
    const int E = D.E, N = D.N, El = D.El, RL = D.route_len;
    int *G_all = (int *)lds;              // [E]      tokens per expert over all sources
    int *Cown = G_all + E;                // [El][N]  counts of rank r's experts per source
    int *Crow = Cown + E;                 // [E]      rank r's own counts
    const int MS = N + 1;                 // row stride: a column's entries on different LDS banks
    int *Mall = Crow + E;                 // [N][MS]  de-duplicated counts, [source][destination]
    int *eoff = Mall + N * MS;            // [El+1]   expert offsets of rank r
    int *csoff = eoff + El + 1;           // [N]      first combine-send row of each source
    __shared__ int late, invalid, over;
    const route_word *rt = W.routes + (size_t)r * N * RL;
    // Rank r has planned epoch_route[r] steps so far (only this block touches the word, and only
    // once its own source's record of the step is there or given up).
    const unsigned expect = W.epoch_route[r] + 1u, tag = route_tag(expect);
    if (tid == 0) { late = 0; invalid = 0; over = 0; }
    for (int e = tid; e < E; e += kRouteThreads) G_all[e] = 0;
    __syncthreads();
    {
        // A thread takes one word of every `parts`-th source's record, four at a time.
        constexpr int kPer = WIDE ? 1 : 3;                 // counts per word
        const int words = RL - 1, cols = min(words, kRouteThreads), parts = kRouteThreads / cols;
        const int part = tid / cols;
        long long spins = 0;
        bool ok = true;
        unsigned valid = kRouteValid;
        for (int f = tid - part * cols; f < words && part < parts && ok; f += cols) {
            int acc[kPer];
#pragma unroll
            for (int i = 0; i < kPer; ++i) acc[i] = 0;
            for (int s0 = part; s0 < N && ok; s0 += 4 * parts) {
                route_word q[4];
                for (;;) {
                    bool here = true;
#pragma unroll
                    for (int u = 0; u < 4; ++u) q[u] = ld_route(rt + (size_t)min(s0 + u * parts, N - 1) * RL + 1 + f);
#pragma unroll
                    for (int u = 0; u < 4; ++u) here &= route_ready(q[u], tag);
                    if (here) break;
                    if (++spins > D.spin_limit) { ok = false; break; }
                    __builtin_amdgcn_s_sleep(2);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int s = s0 + u * parts;
                    if (s >= N) continue;
                    valid &= (unsigned)(q[u] >> 48);
#pragma unroll
                    for (int i = 0; i < kPer; ++i) {
                        const int c = WIDE ? (int)(unsigned)q[u] : (int)(q[u] >> (16 * i) & 0xFFFFu), at = f * kPer + i;
                        if (at < E) {
                            acc[i] += c;
                            if (s == r) Crow[at] = c;
                            if ((unsigned)(at - r * El) < (unsigned)El) Cown[(at - r * El) * N + s] = c;
                        } else if (at < E + N) Mall[s * MS + at - E] = c;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                if (f * kPer + i < E) atomicAdd(&G_all[f * kPer + i], acc[i]);
        }
        if (!ok) late = 1;
        else if (!(valid & kRouteValid)) invalid = 1;
    }
    __syncthreads();
    if (tid == 0) W.epoch_route[r] = expect;
    if (late) {
        if (tid == 0) { W.plan_ok[r] = 0; latch_status(W.status, FL_STATUS_TIMEOUT); }
        return;
    }
    if (invalid) {
        if (tid == 0) W.plan_ok[r] = 0;       // the offending source latched BAD_INDEX
        return;
    }

    // wave = destination d, lane = source: the shared-range rows of lower sources
    const bool partial = D.flags & FL_FLAG_PARTIAL_SUMS;
    for (int d = wid; d < N; d += kWaves) {
        const int m = lane < N ? Mall[lane * MS + d] : 0;
        const int beyond = max(m - D.P, 0);   // rows past the source's private slots
        int inc = wave_incl_scan(beyond);
        if (lane == r) W.dst_off[(size_t)r * N + d] = inc - beyond;
        if (lane == N - 1 && inc > D.recv_cap) over = 1;   // what d's shared range must hold
        if (d == r) {
            if (lane < N) W.recv_shared_off[(size_t)r * N + lane] = inc - beyond;
            inc = wave_incl_scan(m);
            if (lane < N) W.recv_off[(size_t)r * (N + 1) + lane] = inc - m;
            if (lane == N - 1) W.recv_off[(size_t)r * (N + 1) + N] = inc;
        }
    }
    if (partial)                              // wave = source, lane = rank: rows the source sent to ranks below r
        for (int s = wid; s < N; s += kWaves) {
            const int m = lane < N ? Mall[s * MS + lane] : 0;
            const int inc = wave_incl_scan(m);
            if (lane == r) W.ret_off[(size_t)r * N + s] = inc - m;
        }
    // sums over the experts of a rank, lane = rank (the last rank's again in lanes beyond)
    const int of = min(lane, N - 1);
    auto over_experts = [&](auto sum, auto term) {
        for (int j0 = 0; j0 < El; j0 += 8) {
            unsigned v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (unsigned)term(min(j0 + i, El - 1));
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += j0 + i < El ? v[i] : 0u;
        }
        return sum;
    };
    const unsigned al = (unsigned)D.align;
    auto room = [&](int j, int g) { return j + 1 < El && al > 1 ? ((unsigned)g + al - 1) / al * al : (unsigned)g; };
    unsigned exp_units = 0;       // last wave: lane = source; the one before: lane = peer answering in combine
    if (wid == kWaves - 1) {
        // what source s will have added once its transfer to this rank is complete: the
        // payload in 16-byte units, plus one for the transfer itself (an empty one still counts)
        if (lane < N) exp_units = (unsigned)Mall[lane * MS + r] * (unsigned)(D.Bw / 16) + 1u;
        const int n = lane < N ? (int)over_experts(0u, [&](int j) { return Cown[j * N + of]; }) : 0;
        const int inc = wave_incl_scan(n);
        if (lane < N) { csoff[lane] = inc - n; W.cs_off[(size_t)r * (N + 1) + lane] = inc - n; }
        if (lane == N - 1) W.cs_off[(size_t)r * (N + 1) + N] = inc;
    } else if (wid == kWaves - 2) {
        // with partial sums one share per row r sent to the peer, else one reply per pair
        const unsigned pairs = over_experts(0u, [&](int j) { return Crow[of * El + j]; });
        if (lane < N) exp_units = (partial ? (unsigned)Mall[r * MS + lane] : pairs) * (unsigned)(D.Bc / 16) + 1u;
    } else if (wid == kWaves - 4) {        // rows of every rank's expert layout, padding included
        if (over_experts(0ull, [&](int j) { return room(j, G_all[of * El + j]); }) > (unsigned long long)D.expert_cap) over = 1;
    } else if (wid == kWaves - 5) {        // the sources' heads, there by now or soon
        route_word head = 0;
        long long spins = 0;
        while (lane < N && !route_ready(head = ld_route(rt + (size_t)lane * RL), tag)) {
            if (++spins > D.spin_limit) { late = 1; break; }
            __builtin_amdgcn_s_sleep(2);
        }
        if (lane < N) { W.comb_dst_off[(size_t)r * N + lane] = (int)(unsigned)head; W.arrive_route[(size_t)r * N + lane] = expect; }
    } else if (wid == kWaves - 3) {        // offsets of rank r's experts, 64 at a time
        unsigned carry = 0;
        for (int j0 = 0; j0 < El; j0 += kWave) {
            const int j = j0 + lane;
            const unsigned g = j < El ? (unsigned)G_all[r * El + j] : 0u, rows = j < El ? room(j, (int)g) : 0u;
            const unsigned inc = (unsigned)wave_incl_scan((int)rows);
            if (j < El) {
                eoff[j] = (int)(carry + inc - rows);
                if (j == El - 1) eoff[El] = (int)(carry + inc);
                W.G[(size_t)r * El + j] = (int)g;
            }
            carry += (unsigned)__shfl((int)inc, kWave - 1);
        }
    }
    __syncthreads();
    if (late || over) {
        if (tid == 0) { W.plan_ok[r] = 0; latch_status(W.status, late ? FL_STATUS_TIMEOUT : FL_STATUS_CAPACITY); }
        return;
    }
    for (int j = tid; j <= El; j += kRouteThreads) W.expert_off[(size_t)r * (El + 1) + j] = eoff[j];
    // base_x[j][s] = expert_off[j] + rows of lower sources in expert j (a wave per expert, lane = source);
    // cs_base[s][j] = cs_off[s] + rows of lower experts for source s (a wave per source, lane = expert)
    for (int job = wid; job < El + N; job += kWaves) {
        if (job < El) {
            const int c = lane < N ? Cown[job * N + lane] : 0;
            const int inc = wave_incl_scan(c);
            if (lane < N) W.base_x[((size_t)r * El + job) * N + lane] = eoff[job] + inc - c;
        } else {
            const int s = job - El;
            int carry = csoff[s];
            for (int j0 = 0; j0 < El; j0 += kWave) {
                const int c = j0 + lane < El ? Cown[(j0 + lane) * N + s] : 0;
                const int inc = wave_incl_scan(c);
                if (j0 + lane < El) W.cs_base[((size_t)r * N + s) * El + j0 + lane] = carry + inc - c;
                carry += __shfl(inc, kWave - 1);
            }
        }
    }
    if (wid == kWaves - 1 && lane < N) W.expect_disp[(size_t)r * N + lane] += exp_units;
    if (wid == kWaves - 2 && lane < N) W.expect_comb[(size_t)r * N + lane] += exp_units;
    if (tid == 0) W.plan_ok[r] = 1;
}

// One launch for both halves of the layout step: the first rank_count * parts blocks
// count (the first rank_count of them, part 0 of every source, push the route records),
// the last rank_count plan for their rank from the records of all sources, which they poll
// (bounded) while the counting blocks run: workgroups are dispatched in index order, so every
// counting block has its place before a poller takes one, and a poller never keeps a counter
// from starting.  Records cross compute dies inside one kernel, in words stored and loaded at device scope.
template <bool WIDE>
__global__ __launch_bounds__(kRouteThreads) void route_layout_kernel(
    Dims D, Tables W, int rank_begin, int rank_count, int parts, const int *__restrict__ indices,
    const int *__restrict__ num_tokens) {
    extern __shared__ __align__(16) unsigned lds[];
    const int b = blockIdx.x;
    if (b < rank_count * parts)
        route_count_block<WIDE>(D, W, rank_begin + b % rank_count, b / rank_count, parts, indices, num_tokens, lds);
    else
        route_plan_block<WIDE>(D, W, rank_begin + b - rank_count * parts, lds);
}

// ------------------------------------------------------------------ the layout step without a context
// Two kernels instead of one: the boundary between them does what the message counters and the wait do above, so
// nothing has to be cleared before a call or trusted from the call before.  Bound by latency like the kernel above:
// a chain of load, count, scan, store.  The first counts every tile of tokens once, a block each; the second
// scans (every block of a source for itself, from its parts' counts) and writes the pairs' positions, one block more
// derives the receivers' tables for all ranks.  The call, against a kernel that cleared counters and the single
// kernel behind it (32 ranks x 256 experts, top 8): 16 tokens per rank 12.7 -> 9.5 us (what two launches take the
// host), 512: 14.8 -> 10.4, 2048: 23.2 -> 12.8; 8 ranks x 128 experts, 3000 tokens 31.4 -> 9.6.
constexpr int kStaticCountThreads = 256;
// Counting blocks a call aims at, over all sources: with more, the tables take longer to read than the tiles to
// count (2048 tokens, 64 / 128 / 256 / 512 blocks: 18.0 / 12.8 / 13.4 / 16.9 us).
constexpr int kStaticBlocks = 128;
constexpr int kStaticMaxParts = 64;

struct StaticOut {                           // the caller's tables
    int *C, *M, *G, *send_off, *recv_off, *expert_off, *comb_off, *comb_pos, *plan_ok, *status;
};

// Counts of one block: E + N numbers, 16 bits each unless a count may need more; whole 16-byte vectors.
__host__ __device__ inline int static_record_words(int E, int N, int T) {
    return ((route_wide(T) ? E + N : (E + N + 1) / 2) + 3) / 4 * 4;
}

__host__ __device__ inline size_t static_tables_lds_bytes(int E, int N, int K, int TT) {
    const size_t rows = (size_t)E + N;
    const size_t block = ((size_t)E * route_row_stride(TT) * 2 + 3 * rows + E + 20) * sizeof(int) + (size_t)TT * K * 2;
    const size_t plan = ((size_t)E + (size_t)N * N + N) * sizeof(int);
    return block > plan ? block : plan;
}

// Block (source s, part): its tiles' tokens; *record and the part's verdict on its ids.
__global__ __launch_bounds__(kStaticCountThreads) void static_count_kernel(
    Dims D, int parts, const int *__restrict__ indices, const int *__restrict__ num_tokens, int *__restrict__ records,
    int *__restrict__ invalid) {
    extern __shared__ __align__(16) unsigned lds[];
    __shared__ int bad;
    const int s = blockIdx.x / parts, part = blockIdx.x - s * parts, tid = threadIdx.x;
    const int words = static_record_words(D.E, D.N, D.T);
    int *count = (int *)lds;                               // [2 * words], of which E + N count
    const int given = num_tokens[s];
    for (int r = tid; r < 2 * words; r += kStaticCountThreads) count[r] = 0;
    if (tid == 0) bad = given < 0 || given > D.T;
    const int Ts = max(0, min(given, D.T));
    const int tiles = (D.T + D.TT - 1) / D.TT, per = (tiles + parts - 1) / parts;
    const int t0 = min(part * per * D.TT, Ts), t1 = min((part + 1) * per * D.TT, Ts);
    __syncthreads();
    auto hit = [&](int, int row) { atomicAdd(&count[row], 1); };
    const int *ids = indices + (size_t)s * D.T * D.K;
    if (D.K <= 8) count_tokens<8>(ids, t0, t1, kStaticCountThreads, D.E, D.K, div_magic(D.El), &bad, hit);
    else count_tokens<FL_MAX_TOPK>(ids, t0, t1, kStaticCountThreads, D.E, D.K, div_magic(D.El), &bad, hit);
    __syncthreads();
    int *record = records + (size_t)blockIdx.x * words;
    for (int w = tid; w < words; w += kStaticCountThreads)
        record[w] = route_wide(D.T) ? count[w] : (int)((unsigned)count[2 * w] | (unsigned)count[2 * w + 1] << 16);
    if (tid == 0) invalid[blockIdx.x] = bad;
}

// Blocks [0, N * parts): the tables of their source (part 0) and the positions of their tiles' pairs; the last
// block: what the receivers know, for every rank.
template <bool WIDE>
__device__ __forceinline__ void static_positions_block(const Dims &D, const StaticOut &out, int s, int part, int parts,
                                                       const int *__restrict__ indices, const int *__restrict__ num_tokens,
                                                       const int *__restrict__ records, unsigned *lds) {
    const int tid = threadIdx.x, E = D.E, N = D.N, El = D.El, K = D.K, rows = E + N;
    const int words = static_record_words(E, N, D.T);
    const int Wn = D.TT / 32, Wd = route_row_stride(D.TT);
    unsigned *bits = lds;                                  // [E][Wd]
    unsigned *pre = bits + (size_t)E * Wd;                 // [E][Wd] popcount prefix inside the tile
    int *count = (int *)(pre + (size_t)E * Wd);            // [rows] over all parts
    int *start = count + rows;                             // [rows] exclusive scan of count
    int *base = start + rows;                              // [rows] hits before the current tile
    int *hits = base + rows;                               // [E] of the current tile
    int *scan_tmp = hits + E;                              // [17]
    unsigned short *ids = (unsigned short *)(scan_tmp + 20);   // [TT * K]
    const int *idx_s = indices + (size_t)s * D.T * K;
    const unsigned by_k = 0xFFFFFFFFu / (unsigned)K + 1u;      // p / K for p < 2^16 by the high half of a product (K > 1)
    const int tiles = (D.T + D.TT - 1) / D.TT, per = (tiles + parts - 1) / parts, tile0 = part * per;
    const int Ts = max(0, min(num_tokens[s], D.T));
    int early[kRoutePreload];                              // as in route_count_block
#pragma unroll
    for (int i = 0; i < kRoutePreload; ++i) {
        const int p = tid + i * kRouteThreads;
        early[i] = p < min(D.TT, Ts - tile0 * D.TT) * K ? idx_s[(size_t)tile0 * D.TT * K + p] : -1;
    }
    for (int r = tid; r < rows; r += kRouteThreads) {
        int all = 0, before = 0;
        for (int p0 = 0; p0 < parts; p0 += 8) {
            int c[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int *rec = records + (size_t)(s * parts + min(p0 + i, parts - 1)) * words;
                c[i] = WIDE ? rec[r] : (int)((const unsigned short *)rec)[r];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (p0 + i < parts) { all += c[i]; before += p0 + i < part ? c[i] : 0; }
        }
        count[r] = all;
        base[r] = before;
    }
    for (int i = tid; i < E * Wd; i += kRouteThreads) bits[i] = 0;
    __syncthreads();
    {
        const int a = 2 * tid < rows ? count[2 * tid] : 0, b = 2 * tid + 1 < rows ? count[2 * tid + 1] : 0;
        int total;
        const int ex = block_excl_scan(a + b, scan_tmp, &total, (rows + 2 * kWave - 1) / (2 * kWave));
        if (2 * tid < rows) start[2 * tid] = ex;
        if (2 * tid + 1 < rows) start[2 * tid + 1] = ex + a;
    }
    const int used = (Ts + D.TT - 1) / D.TT;
    for (int tile = tile0; tile < min(tile0 + per, used); ++tile) {
        const int t0 = tile * D.TT, nt = min(D.TT, Ts - t0);
        if (tile > tile0) {
            __syncthreads();
            for (int r = tid; r < E; r += kRouteThreads) base[r] += hits[r];
            for (int i = tid; i < E * Wd; i += kRouteThreads) bits[i] = 0;
            __syncthreads();
        }
        auto take = [&](int p, int e) {
            const bool ok = e >= 0 && e < E;
            ids[p] = (unsigned short)(ok ? e : 0xFFFF);
            const int tl = K > 1 ? (int)__umulhi((unsigned)p, by_k) : p;
            if (ok) atomicOr(&bits[(size_t)e * Wd + (tl >> 5)], 1u << (tl & 31));
        };
#pragma unroll
        for (int i = 0; i < kRoutePreload; ++i) {
            const int p = tid + i * kRouteThreads;
            if (p < nt * K) take(p, tile == tile0 ? early[i] : idx_s[(size_t)t0 * K + p]);
        }
        for (int p = tid + kRoutePreload * kRouteThreads; p < nt * K; p += kRouteThreads)
            take(p, idx_s[(size_t)t0 * K + p]);
        __syncthreads();
        for (int r = tid; r < E; r += kRouteThreads) {
            int run = 0;
            for (int w = 0; w < Wn; ++w) {
                pre[(size_t)r * Wd + w] = run;
                run += __popc(bits[(size_t)r * Wd + w]);
            }
            hits[r] = run;
        }
        __syncthreads();
        for (int p = tid; p < nt * K; p += kRouteThreads) {
            const int e = ids[p];
            if (e == 0xFFFF) continue;
            const int tl = K > 1 ? (int)__umulhi((unsigned)p, by_k) : p, w = tl >> 5;
            out.comb_pos[((size_t)s * D.T + t0) * K + p] =
                start[e] + base[e] + (int)pre[(size_t)e * Wd + w] +
                __popc(bits[(size_t)e * Wd + w] & ((1u << (tl & 31)) - 1u));
        }
    }
    if (part == 0) {
        __syncthreads();                                   // start, also when the source has no tile in use
        const int pairs = start[E];
        for (int e = tid; e < E; e += kRouteThreads) out.C[(size_t)s * E + e] = count[e];
        if (tid < N) {
            out.M[(size_t)s * N + tid] = count[E + tid];
            out.send_off[(size_t)s * (N + 1) + tid] = start[E + tid] - pairs;
            out.comb_off[(size_t)s * (N + 1) + tid] = start[tid * El];
        }
        if (tid == 0) {
            out.send_off[(size_t)s * (N + 1) + N] = start[E + N - 1] + count[E + N - 1] - pairs;
            out.comb_off[(size_t)s * (N + 1) + N] = pairs;
        }
    }
}

template <bool WIDE>
__device__ __forceinline__ void static_plan_block(const Dims &D, const StaticOut &out, int parts,
                                                  const int *__restrict__ records, const int *__restrict__ invalid,
                                                  unsigned *lds) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    constexpr int kWaves = kRouteThreads / kWave;
    const int E = D.E, N = D.N, El = D.El, words = static_record_words(E, N, D.T), recs = N * parts;
    int *G = (int *)lds;                                   // [E]
    int *M = G + E;                                        // [N][N]
    __shared__ int wrong, over;
    auto entry = [&](int rec, int f) -> int {
        return WIDE ? records[(size_t)rec * words + f] : (int)((const unsigned short *)(records + (size_t)rec * words))[f];
    };
    for (int e = tid; e < E; e += kRouteThreads) G[e] = 0;
    if (tid == 0) { wrong = 0; over = 0; }
    int bad = 0;
    for (int i = tid; i < recs; i += kRouteThreads) bad |= invalid[i];
    for (int i = tid; i < N * N; i += kRouteThreads) {     // (source, rank): over the source's parts
        const int s = i / N, d = i - s * N;
        int m = 0;
        for (int p0 = 0; p0 < parts; p0 += 8) {
            int c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = entry(s * parts + min(p0 + u, parts - 1), E + d);
#pragma unroll
            for (int u = 0; u < 8; ++u) m += p0 + u < parts ? c[u] : 0;
        }
        M[i] = m;
    }
    __syncthreads();
    {   // experts: the threads of one 16-byte column share the records out
        constexpr int kPer = WIDE ? 4 : 8;                 // counts per vector; the last one may reach into the rank counts
        const int vecs = (E + kPer - 1) / kPer, groups = kRouteThreads / vecs, v = tid % vecs, first = tid / vecs;
        int acc[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) acc[i] = 0;
        if (first < groups && first < recs) {
            for (int r0 = first; r0 < recs; r0 += 8 * groups) {
                v4u q[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    q[u] = ((const v4u *)(records + (size_t)min(r0 + u * groups, recs - 1) * words))[v];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (r0 + u * groups >= recs) continue;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        if (WIDE) acc[w % kPer] += (int)q[u][w];
                        else { acc[2 * w % kPer] += (int)(q[u][w] & 0xFFFFu); acc[(2 * w + 1) % kPer] += (int)(q[u][w] >> 16); }
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                if (v * kPer + i < E) atomicAdd(&G[v * kPer + i], acc[i]);
        }
    }
    if (bad) wrong = 1;
    __syncthreads();
    if (wrong) {
        if (tid < N) out.plan_ok[tid] = 0;
        if (tid == 0) *out.status = FL_STATUS_BAD_INDEX;
        return;
    }
    const unsigned al = (unsigned)D.align;
    for (int d = wid; d < N; d += kWaves) {                // a wave per rank
        const int m = lane < N ? M[lane * N + d] : 0;
        const int inc = wave_incl_scan(m), beyond = wave_incl_scan(max(m - D.P, 0));
        if (lane < N) out.recv_off[(size_t)d * (N + 1) + lane] = inc - m;
        if (lane == N - 1) {
            out.recv_off[(size_t)d * (N + 1) + N] = inc;
            if (beyond > D.recv_cap) over = 1;
        }
        unsigned long long rows = 0;                       // of its expert layout, padding included
        for (int j0 = 0; j0 < El; j0 += kWave) {
            const int j = j0 + lane;
            const unsigned g = j < El ? (unsigned)G[d * El + j] : 0u;
            if (j < El) out.G[(size_t)d * El + j] = (int)g;
            const unsigned room = j + 1 < El && al > 1 ? (g + al - 1) / al * al : g;
            rows += (unsigned)__shfl(wave_incl_scan((int)room), kWave - 1);
        }
        if (lane == 0 && rows > (unsigned long long)D.expert_cap) over = 1;
    }
    __syncthreads();
    if (!over)
        for (int d = wid; d < N; d += kWaves) {
            unsigned carry = 0;
            for (int j0 = 0; j0 < El; j0 += kWave) {
                const int j = j0 + lane;
                const unsigned g = j < El ? (unsigned)G[d * El + j] : 0u;
                const unsigned room = j + 1 < El && al > 1 ? (g + al - 1) / al * al : g;
                const unsigned inc = (unsigned)wave_incl_scan((int)room);
                if (j < El) out.expert_off[(size_t)d * (El + 1) + j] = (int)(carry + inc - room);
                if (j == El - 1) out.expert_off[(size_t)d * (El + 1) + El] = (int)(carry + inc);
                carry += (unsigned)__shfl((int)inc, kWave - 1);
            }
        }
    if (tid < N) out.plan_ok[tid] = over ? 0 : 1;
    if (tid == 0) *out.status = over ? FL_STATUS_CAPACITY : 0;
}

template <bool WIDE>
__global__ __launch_bounds__(kRouteThreads) void static_tables_kernel(
    Dims D, StaticOut out, int parts, const int *__restrict__ indices, const int *__restrict__ num_tokens,
    const int *__restrict__ records, const int *__restrict__ invalid) {
    extern __shared__ __align__(16) unsigned lds[];
    const int b = blockIdx.x - 1;                          // the longest chain starts first
    if (b < 0) static_plan_block<WIDE>(D, out, parts, records, invalid, lds);
    else static_positions_block<WIDE>(D, out, b / parts, b % parts, parts, indices, num_tokens, records, lds);
}

}  // namespace flmoe
