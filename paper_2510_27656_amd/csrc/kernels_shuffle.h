// The memory-bound half of the shuffle: send, unpack, send back, reduce.
//
// Paper, section MoE Dispatch/Combine.  Dispatch: one copy of every token per
// destination rank goes to a range of that rank's receive buffer which the exchanged
// counts reserved; the receiver waits for all transfers and re-orders tokens into the
// grouped-GEMM layout.  Combine: one scatter per peer re-using the routing information,
// then a locally computed weighted sum.  Every kernel moves whole rows with 16-byte
// accesses; nothing here is a contraction, so there is no MFMA.
//
// The fabric is the send kernels' own stores.  The paper packs rows into a send buffer,
// because a NIC wants one contiguous source per peer, and pushes from the send kernel
// itself where the peer's memory can be stored to (section Dispatch, within a node).
// Here every receive buffer can, so there is no send buffer: staging the rows cost a write,
// a read and a kernel in each direction (DeepSeek-V3 decode step, 128 tokens per rank:
// 761 us with the staging copy, 516 without; 4 tokens per rank: 71 and 57).
#pragma once
#include "common.h"

namespace flmoe {

constexpr int kCopyThreads = 256;
constexpr int kPackThreads = 128;
constexpr int kMaxRowsPerBlock = 64;

// What a completed (sender, receiver) transfer adds to the receiver's counter: its
// payload in 16-byte units plus one for the transfer itself, so that an EMPTY transfer
// is announced too (section TransferEngine: an immediate is delivered even for a
// zero-size write) and a receiver that has seen all its counters complete knows that
// every peer's send call has got as far as announcing - which is what makes the re-use
// of the receive buffers safe without a separate barrier.
//
// Stream-ordered mode: one add per (sender, receiver) announces the whole
// transfer, like the single immediate a NIC delivers after a WRITE (section
// TransferEngine, ImmCounter).  It is issued once per sender inside the send kernel:
// receivers are ordered after that kernel by the stream, so they find counters and
// payload complete together, and no extra launch is spent.
// off = the sender's row of the segment table ([N + 1] row offsets by receiver);
// threads first, first + step, ... each take one receiver.  only_the_ones: the
// payload units are reported by the waves that deliver them (progressive mode).
__device__ inline void announce_transfers(const int *off, unsigned *arrive, unsigned units_per_row,
                                          int sender, int N, int first, int step, bool only_the_ones = false) {
    for (int p = first; p < N; p += step) {
        const int rows = off[p + 1] - off[p];
        add_counter(arrive + (size_t)p * N + sender, only_the_ones ? 1u : (unsigned)rows * units_per_row + 1u);
    }
}

// Default mode, small steps: the last workgroup of a sender's payload kernel announces its whole transfers, so that
// no kernel has to be launched for it.  Every workgroup waits until what it stored has been acknowledged (payload and
// sidecars are written through, so it is in memory then, where every XCD sees it) and counts itself; the one that
// completes the count adds to the receivers' counters.  Adds to one word take 12 ns each, so a
// workgroup counts on one of kDoneParts words, whose last one counts on the word for all; who completes a word clears
// it for the next call.  done: the sender's words; number: this workgroup's, of `workgroups`; rows: lane p < N of the
// first wave holds those for receiver p.  Where the line to an announce kernel lies: announces_itself in flmoe.hip.
__device__ inline void announce_when_last(unsigned *done, unsigned number, unsigned workgroups, unsigned *arrive, int rows,
                                          unsigned units_per_row, int sender, int N, int lane, bool first_wave) {
    stores_done();
    __syncthreads();
    if (!first_wave) return;
    auto completes = [&](unsigned *word, unsigned all) {
        unsigned before = 0;
        if (lane == 0) before = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane(before) + 1 != all) return false;
        if (lane == 0) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    };
    const unsigned part = number % kDoneParts;
    if (!completes(done + part * kDoneLine, (workgroups - part + kDoneParts - 1) / kDoneParts)) return;
    if (!completes(done + kDoneParts * kDoneLine, min(workgroups, (unsigned)kDoneParts))) return;
    if (lane < N) add_counter(arrive + (size_t)lane * N + sender, (unsigned)rows * units_per_row + 1u);
}

// Test switch (knob 8): the order in which a send kernel takes its `n` units of work.  Nothing may
// depend on it: 0 = ascending, 1 = descending, 2 = starting in the middle and wrapping round.
__device__ inline int in_order(int order, int i, int n) {
    if (order == 1) return n - 1 - i;
    if (order == 2) return i + n / 2 < n ? i + n / 2 : i + n / 2 - n;
    return i;
}

// Where the copies of token (s, t) go.  Lane k < K of a block's first wave fetches the k-th expert's
// entries, lane d < N rank d's offset, all in the kernel's first round of loads (the tables hold
// something for every t < T; it is used only once the step and the token are known to be valid).
// One round instead of three in a row: e4m3 pack of 128 tokens per rank 57.5 -> 52.7 us (its one
// workgroup per row had nothing else to do meanwhile), bf16 4 / 8 tokens 10.0 / 11.4 -> 9.4 / 10.8,
// the same from 32 tokens on.  The caller's expert ids are not read again: those of absent tokens
// need not exist, so fetching them would have to wait for the token count.
struct CopyPlan {
    int to, dst_off;
    unsigned meta, weight;
    __device__ inline void load(const Dims &D, const Tables &W, int s, size_t pair0, int lane,
                                const float *__restrict__ weights /* null: they do not travel */) {
        to = -1; meta = 0; dst_off = 0; weight = 0;
        if (lane < D.K) {
            to = W.send_to[pair0 + lane];
            meta = W.pair_meta[pair0 + lane];
            if (weights) weight = __float_as_uint(weights[pair0 + lane]);
        }
        if (lane < D.N) dst_off = W.dst_off[(size_t)s * D.N + lane];
    }
    // destination rank of this lane's expert, and the row in its receive buffer when the token's copy
    // for that rank belongs to this lane (the first of its experts there), else -1; whole wave
    __device__ inline int target(const Dims &D, int s, int *dst) const {
        const int d = to >= 0 ? to >> 24 : ~to;
        *dst = d;
        const int shared = __shfl(dst_off, d);
        return to >= 0 ? recv_buffer_row(D.N, D.P, s, to & 0xFFFFFF, shared) : -1;
    }
    // Sidecars of the token's copies, behind the payload stores: K words that name, for every expert of the token on the
    // copy's rank, the local expert and the token's rank among the source's tokens of that expert (and as many weights of
    // those experts, for the expert rank's partial sum), then kNoEntry.  A lane per word, which finds its entry by looking
    // through the experts' lanes; whole first wave.  row, dst: what target() gave this lane.  A lane per copy that
    // read the others' entries from LDS and stored its words one by one, in front of the payload, made
    // the workgroup of a token's first slice the slowest: us of a step, 32 ranks x 4 tokens of 14 KB 45.3 -> 44.3,
    // 128: 454.6 -> 450.2, 16 ranks x 1024 tokens of 512 bytes 122 -> 110.
    __device__ inline void write_sidecars(const Dims &D, const Tables &W, int row, int dst, int lane) const {
        const int per_copy = (65536 + D.KM - 1) / D.KM;    // i / KM for i < K * KM <= 256 by a product: KM = 4, 8, 12, 16
        for (int i0 = 0; i0 < D.K * D.KM; i0 += kWave) {
            const int i = i0 + lane, copy = (i * per_copy) >> 16, m = i - copy * D.KM;
            const int to_row = __shfl(row, copy & (kWave - 1)), d = __shfl(dst, copy & (kWave - 1));
            unsigned entry = kNoEntry, w = 0;
            int seen = 0;
            for (int k = 0; k < D.K; ++k) {
                const bool here = __builtin_amdgcn_readlane(dst, k) == d;
                if (here && seen == m) {
                    entry = (unsigned)__builtin_amdgcn_readlane(meta, k);
                    w = (unsigned)__builtin_amdgcn_readlane(weight, k);
                }
                seen += here;
            }
            if (copy < D.K && to_row >= 0) {
                unsigned *to_meta = W.recv_meta + ((size_t)d * D.recv_rows + to_row) * D.MW + m;
                st_word((int *)to_meta, (int)entry);
                if (D.MW > D.KM && entry != kNoEntry) st_word((int *)to_meta + D.KM, (int)w);
            }
        }
    }
};

// ------------------------------------------------------------------ dispatch: pack
// `slices` blocks per token (s, t), each taking a slice of the row (so a thread
// usually has a single vector): the slice is read once and stored once per
// distinct destination rank d, into the row of d's receive buffer that follows from
// (rank of t among s's tokens bound for d).  Each copy carries a sidecar of K words
// naming, for every expert of the token that lives on d, the local expert and the
// token's rank among s's tokens of that expert; the receiver turns that into an
// expert-major row.
//
// FENCED (progressive mode): device-scope stores, and the block adds the 16-byte
// units it wrote to arrive[destination][source] itself once they are acknowledged;
// stream-ordered, the sender's first block announces the whole transfers; otherwise its
// last one does (done given) or the announce kernel.
template <bool FENCED>
__global__ __launch_bounds__(kPackThreads) void dispatch_pack_kernel(
    Dims D, Tables W, int rank_begin, const char *__restrict__ x, const int *__restrict__ num_tokens, int slices,
    const float *__restrict__ weights /* [N][T][K], only when the sidecar carries them */,
    long long src_row_bytes /* bytes of one row of x: 2*H, or H for ready-made e4m3 codes */,
    const float *__restrict__ src_scales /* [N][T][H/128] with ready-made codes, else null */,
    unsigned *done /* announce_when_last; null: announced elsewhere */) {
    const int s = rank_begin + blockIdx.y, slice = blockIdx.x % slices;
    const int t = in_order(D.tune_order, blockIdx.x / slices, D.T);
    const int tid = threadIdx.x;
    const int K = D.K;
    // The slice's payload depends on nothing but (s, t), and neither do the routing tables'
    // entries: everything the block needs is fetched in one round (x has T rows per rank, so
    // the loads are in bounds for absent tokens too).
    const int nvec = (int)(src_row_bytes / 16);
    const int per = whole_lines((nvec + slices - 1) / slices); // vectors of this slice: [v0, v1)
    const int v0 = min(slice * per, nvec), v1 = min(v0 + per, nvec);
    const v4u *src = (const v4u *)(x + ((size_t)s * D.T + t) * src_row_bytes);
    v4u r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (v0 + tid + i * kPackThreads < v1) r[i] = ld_stream(src + v0 + tid + i * kPackThreads);
    const size_t pair0 = ((size_t)s * D.T + t) * K;
    CopyPlan plan;
    if (tid < kWave) plan.load(D, W, s, pair0, tid, D.MW > D.KM ? weights : nullptr);
    const int plan_ok = W.plan_ok[s], tokens = num_tokens[s];
    const int sent = done && tid < D.N ? W.M[(size_t)s * D.N + tid] : 0;
    // the sender's first block announces the transfers (a sender without tokens still announces
    // its empty ones), unless an announce kernel will
    if ((FENCED || (D.flags & FL_FLAG_STREAM_ORDERED)) && blockIdx.x == 0 && plan_ok)
        announce_transfers(W.send_off + (size_t)s * (D.N + 1), W.arrive_disp, (unsigned)(D.Bw / 16), s, D.N,
                           tid, kPackThreads, FENCED);
    if (!plan_ok) return;
    const unsigned workgroups = (unsigned)(tokens * slices);   // of this sender that have a token
    if (t >= tokens) {
        if (done && tokens == 0 && blockIdx.x == 0)            // none has: one announces the empty transfers
            announce_when_last(done + s * kDoneWords, 0u, 1u, W.arrive_disp, sent, (unsigned)(D.Bw / 16), s, D.N, tid & (kWave - 1),
                               tid < kWave);
        return;
    }
    __shared__ int s_row[FL_MAX_TOPK];
    __shared__ int s_dst[FL_MAX_TOPK];
    int target = -1, my_d = 0;                 // of this lane's copy: row in rank my_d's receive buffer
    if (tid < kWave) {
        target = plan.target(D, s, &my_d);
        if (tid < K) { s_row[tid] = target; s_dst[tid] = my_d; }
    }
    __syncthreads();
    for (int b = v0 + tid; b < v1; b += 4 * kPackThreads) {
        if (b != v0 + tid) {                   // later batches (rows beyond 8 KB per slice)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b + i * kPackThreads < v1) r[i] = ld_stream(src + b + i * kPackThreads);
        }
        for (int k = 0; k < K; ++k) {
            const int row = s_row[k];          // uniform: one copy per distinct destination
            if (row < 0) continue;
            char *base = W.bufB + (size_t)s_dst[k] * D.bufB_rank_bytes;
            v4u *dst = (v4u *)(base + (size_t)row * D.Sw);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b + i * kPackThreads < v1)
                    st_payload<true>(dst + b + i * kPackThreads, r[i]);
        }
    }
    if (slice == 0 && tid < kWave) plan.write_sidecars(D, W, target, my_d, tid);
    // Ready-made e4m3 codes (section Kernel Microbenchmarks: the dispatched token is 7168
    // fp8 values and 56 fp32 scaling factors): the scales follow the codes in the wire row.
    const bool with_scales = src_scales != nullptr && slice == 0;
    if (with_scales) {
        const float *sc = src_scales + ((size_t)s * D.T + t) * D.scales_per_row;
        if (D.scales_per_row % 4 == 0) {       // whole 16-byte vectors (rows of scales stay aligned)
            for (int v = tid; v < D.scales_per_row / 4; v += kPackThreads) {
                const v4u val = ld_stream((const v4u *)sc + v);
                for (int k = 0; k < K; ++k) {
                    const int row = s_row[k];
                    if (row < 0) continue;
                    char *base = W.bufB + (size_t)s_dst[k] * D.bufB_rank_bytes;
                    st_payload<true>((v4u *)(base + (size_t)row * D.Sw + D.Be) + v, val);
                }
            }
        } else {
            for (int v = tid; v < D.scales_per_row; v += kPackThreads) {
                const int val = __float_as_int(sc[v]);
                for (int k = 0; k < K; ++k) {
                    const int row = s_row[k];
                    if (row < 0) continue;
                    char *base = W.bufB + (size_t)s_dst[k] * D.bufB_rank_bytes;
                    st_word((int *)(base + (size_t)row * D.Sw + D.Be) + v, val);
                }
            }
        }
    }
    if (FENCED) {                      // what this block delivered, per destination
        stores_done();
        __syncthreads();
        const unsigned units = (unsigned)(v1 - v0) + (with_scales ? (unsigned)((D.Bw - D.Be) / 16) : 0u);
        if (tid < K && target >= 0 && units > 0)
            add_counter(W.arrive_disp + (size_t)my_d * D.N + s, units);
    } else if (done) {
        announce_when_last(done + s * kDoneWords, (unsigned)(t * slices + slice), workgroups, W.arrive_disp, sent,
                           (unsigned)(D.Bw / 16), s, D.N, tid & (kWave - 1), tid < kWave);
    }
}

// ------------------------------------------------------------------ dispatch: pack with e4m3 quantisation
// Payload of section Kernel Microbenchmarks: H e4m3 bytes followed by H/128 fp32
// scales per token.  Rule per 128-element block: amax = max |x|, scale =
// amax / 448 (1 when amax is 0), q = e4m3(x / scale) rounded to nearest even and
// saturated at +-448; both divisions are IEEE fp32 divisions.
//
// OCP E4M3, finite-only: 1 sign, 4 exponent bits (bias 7), 3 mantissa bits,
// subnormals m * 2^-9, largest finite 448, no infinities.
//
// Four quotients to four e4m3 bytes with the part's own converter (OCP E4M3 on
// gfx950, round to nearest even, subnormals included; checked against the oracle's
// arithmetic encoder on every finite bf16 input under several block maxima).  A quotient can exceed 448
// by one fp32 step (both divisions round), so magnitudes are held at 448 first.
// The block maximum skips NaN elements (an ordered comparison, as in the rule's plain reading).
__device__ inline float e4m3_hold(float v) {
    return fabsf(v) >= 448.0f ? copysignf(448.0f, v) : v;
}
__device__ inline unsigned e4m3_pack4(float a, float b, float c, float d) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_hold(a), e4m3_hold(b), 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_hold(c), e4m3_hold(d), w, true);
    return (unsigned)w;
}
// Non-finite inputs (Inf or NaN, exponent bits all ones): the quotient is NaN either
// way (NaN / scale; Inf / Inf, because an Inf makes the block's scale infinite) and the
// code is the NaN code 0x7f with the sign of the INPUT element, which IEEE leaves
// open for Inf / Inf and the converter for NaN.  lo16 / hi16: the two bf16 inputs of
// a packed word; byte positions 2 * i and 2 * i + 1 of the four-code word.
__device__ inline bool bf16x2_nonfinite(unsigned w) {
    return ((w & 0x7f80u) == 0x7f80u) || ((w & 0x7f800000u) == 0x7f800000u);
}
__device__ inline unsigned e4m3_fix_nonfinite(unsigned codes, unsigned w0, unsigned w1) {
    const unsigned in[4] = {w0 & 0xffffu, w0 >> 16, w1 & 0xffffu, w1 >> 16};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if ((in[i] & 0x7f80u) == 0x7f80u)
            codes = (codes & ~(0xffu << (8 * i))) | ((((in[i] >> 8) & 0x80u) | 0x7fu) << (8 * i));
    return codes;
}

constexpr int kQuantLanes = 8;     // lanes per 128-element block: 16 bf16 values each

// One workgroup of QT threads takes QT / 8 consecutive quantisation blocks of one
// token (QT = 512 covers a 7168-element row whole, 4 us of 64 faster than two
// workgroups of 256; more blocks per lane group measured no gain); every lane loads
// 32 bytes, takes part in an 8-lane max, and stores 16 bytes of e4m3 per destination
// copy; the scales go out as 16-byte vectors from LDS.
template <bool FENCED, int QT>   // FENCED as in dispatch_pack_kernel
__global__ __launch_bounds__(QT) void dispatch_pack_e4m3_kernel(
    Dims D, Tables W, int rank_begin, const char *__restrict__ x, const int *__restrict__ num_tokens, int slices,
    const float *__restrict__ weights /* [N][T][K], only when the sidecar carries them */,
    unsigned *done /* as in dispatch_pack_kernel */) {
    constexpr int kQuantThreads = QT;
    const int s = rank_begin + blockIdx.y, slice = blockIdx.x % slices;
    const int t = in_order(D.tune_order, blockIdx.x / slices, D.T);
    const int tid = threadIdx.x;
    const int K = D.K;
    // as in dispatch_pack_kernel, the payload loads go first
    const int nblk = D.scales_per_row;                          // 128-element blocks in the row
    const int blk = slice * (kQuantThreads / kQuantLanes) + tid / kQuantLanes;
    const int sub = tid % kQuantLanes;
    const bool live = blk < nblk;
    v4u in0 = {0u, 0u, 0u, 0u}, in1 = {0u, 0u, 0u, 0u};
    if (live) {
        const v4u *src = (const v4u *)(x + ((size_t)s * D.T + t) * D.Bx) + (size_t)blk * 16 + sub * 2;
        in0 = ld_stream(src);
        in1 = ld_stream(src + 1);
    }
    const size_t pair0 = ((size_t)s * D.T + t) * K;
    CopyPlan plan;
    if (tid < kWave) plan.load(D, W, s, pair0, tid, D.MW > D.KM ? weights : nullptr);
    const int plan_ok = W.plan_ok[s], tokens = num_tokens[s];
    const int sent = done && tid < D.N ? W.M[(size_t)s * D.N + tid] : 0;
    if ((FENCED || (D.flags & FL_FLAG_STREAM_ORDERED)) && blockIdx.x == 0 && plan_ok)   // as in dispatch_pack_kernel
        announce_transfers(W.send_off + (size_t)s * (D.N + 1), W.arrive_disp, (unsigned)(D.Bw / 16), s, D.N,
                           tid, kQuantThreads, FENCED);
    if (!plan_ok) return;
    const unsigned workgroups = (unsigned)(tokens * slices);   // of this sender that have a token
    if (t >= tokens) {
        if (done && tokens == 0 && blockIdx.x == 0)            // none has: one announces the empty transfers
            announce_when_last(done + s * kDoneWords, 0u, 1u, W.arrive_disp, sent, (unsigned)(D.Bw / 16), s, D.N, tid & (kWave - 1),
                               tid < kWave);
        return;
    }
    __shared__ int s_row[FL_MAX_TOPK];
    __shared__ int s_dst[FL_MAX_TOPK];
    int target = -1, my_d = 0;
    if (tid < kWave) {
        target = plan.target(D, s, &my_d);
        if (tid < K) { s_row[tid] = target; s_dst[tid] = my_d; }
    }
    __syncthreads();
    float f[16];
    const unsigned w[8] = {in0.x, in0.y, in0.z, in0.w, in1.x, in1.y, in1.z, in1.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) { f[2 * i] = bf16_lo(w[i]); f[2 * i + 1] = bf16_hi(w[i]); }
    float amax = 0.f;              // a NaN element (quiet or signalling) fails the comparison and is skipped
#pragma unroll
    for (int i = 0; i < 16; ++i) { const float a = fabsf(f[i]); amax = a > amax ? a : amax; }
#pragma unroll
    for (int o = 1; o < kQuantLanes; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
    const float scale = amax == 0.f ? 1.0f : __fdiv_rn(amax, 448.0f);
    unsigned q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        q[i] = e4m3_pack4(__fdiv_rn(f[4 * i], scale), __fdiv_rn(f[4 * i + 1], scale),
                          __fdiv_rn(f[4 * i + 2], scale), __fdiv_rn(f[4 * i + 3], scale));
    bool odd_values = false;       // rare: keep the common path free of the per-byte fix-up
#pragma unroll
    for (int i = 0; i < 8; ++i) odd_values |= bf16x2_nonfinite(w[i]);
    if (odd_values) {
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = e4m3_fix_nonfinite(q[i], w[2 * i], w[2 * i + 1]);
    }
    const v4u out = {q[0], q[1], q[2], q[3]};
    // the block's scales are gathered in LDS and stored as 16-byte vectors when the
    // row's scale count allows it (scattered 4-byte stores are partial-line writes)
    __shared__ __align__(16) float s_scale[kQuantThreads / kQuantLanes];
    const bool scale_vectors = nblk % 4 == 0;
    if (scale_vectors) {
        if (live && sub == 0) s_scale[tid / kQuantLanes] = scale;
        __syncthreads();
    }
    const int blk0 = slice * (kQuantThreads / kQuantLanes);
    const int nsv = (min(nblk - blk0, kQuantThreads / kQuantLanes)) / 4;   // scale vectors of this block
    for (int k = 0; k < K; ++k) {
        const int row = s_row[k];
        if (row < 0) continue;
        char *dst = W.bufB + (size_t)s_dst[k] * D.bufB_rank_bytes + (size_t)row * D.Sw;
        if (live) st_payload<true>((v4u *)dst + (size_t)blk * kQuantLanes + sub, out);
        if (scale_vectors) {
            if (tid < nsv)
                st_payload<true>((v4u *)(dst + D.Be) + blk0 / 4 + tid,
                                                 ((const v4u *)s_scale)[tid]);
        } else if (live && sub == 0) {
            st_word((int *)(dst + D.Be) + blk, __float_as_int(scale));
        }
    }
    if (slice == 0 && tid < kWave) plan.write_sidecars(D, W, target, my_d, tid);
    if (FENCED) {
        // Units of the row this block wrote: 8 per quantisation block of codes, and the
        // 16-byte units its scales fall into (blocks start on multiples of 32 scales, so
        // no unit is shared between blocks; the row's last unit may be part padding).
        const int n_live = min(nblk - blk0, kQuantThreads / kQuantLanes);
        stores_done();
        __syncthreads();
        // the padding that brings a wire row to a whole number of 128-byte lines is nobody's
        // to write; the first block claims it so that a row's units add up to Bw / 16
        const int pad_units = (int)(D.Bw / 16) - (nblk * 8 + (nblk + 3) / 4);
        if (tid < K && target >= 0 && n_live > 0)
            add_counter(W.arrive_disp + (size_t)my_d * D.N + s,
                        (unsigned)(n_live * 8 + (n_live + 3) / 4 + (slice == 0 ? pad_units : 0)));
    } else if (done) {
        announce_when_last(done + s * kDoneWords, (unsigned)(t * slices + slice), workgroups, W.arrive_disp, sent,
                           (unsigned)(D.Bw / 16), s, D.N, tid & (kWave - 1), tid < kWave);
    }
}

// ------------------------------------------------------------------ announce
// Counter-ordered mode (the default), sending side: enqueued behind the payload
// kernels of a send call in the sender's own stream, so it starts once they have
// ended and everything they stored has left for memory; one wave per sender then
// adds each whole (sender, receiver) transfer to the receiver's arrival counter
// with release semantics - the single immediate a NIC delivers after a completed
// WRITE (section TransferEngine, ImmCounter).  off: [N][N+1] row offsets of the
// senders' segment tables.
__global__ __launch_bounds__(kWave) void announce_kernel(Dims D, Tables W, int rank_begin, const int *off,
                                                         unsigned *arrive, unsigned units_per_row) {
    const int s = rank_begin + blockIdx.x, N = D.N;
    const int p = threadIdx.x;
    const int plan_ok = W.plan_ok[s];               // one round of loads: the verdict and the segment table
    const int lo = p < N ? off[(size_t)s * (N + 1) + p] : 0, hi = p < N ? off[(size_t)s * (N + 1) + p + 1] : 0;
    if (!plan_ok) return;                           // step skipped: nothing was sent
    if (p < N) {       // payload units plus one per transfer, empty transfers included (announce_transfers)
        const int rows = hi - lo;
        (void)__hip_atomic_fetch_add(arrive + (size_t)p * N + s, (unsigned)rows * units_per_row + 1u,
                                     __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ------------------------------------------------------------------ arrival gate
// Default mode, receiving side: one wave per rank polls the rank's arrival
// counters (bounded) until every source has delivered what the exchanged counts
// promised.  That is how the paper's receive half begins as well (section
// Dispatch: it first waits until all transfers are complete, the proxy raising a
// flag once the ImmCounter has reached its expectation).  The receive kernel
// proper follows in the same stream: it starts after this kernel has ended, with
// clean caches, so what it reads is what the counters vouched for: when they were added to, the
// senders' payload kernels had ended and their stores were written back (announce kernel), or all
// their stores had been written through and acknowledged (announce_when_last).
// Waiting costs one wave per rank instead of a grid of pollers, so senders that
// run at the same time keep the machine.
__global__ __launch_bounds__(kWave) void arrival_gate_kernel(Dims D, Tables W, int rank_begin,
                                                             const unsigned *arrive, const unsigned *expect,
                                                             int *gate) {
    const int r = rank_begin + blockIdx.x, N = D.N, lane = threadIdx.x;
    // one round of loads: the verdict, what to expect, and the first look at the counters
    const int plan_ok = W.plan_ok[r];
    const unsigned want = lane < N ? expect[(size_t)r * N + lane] : 0u;
    unsigned have = lane < N ? ld_relaxed(arrive + (size_t)r * N + lane) : 0u;
    if (!plan_ok) return;                           // step skipped: the receive kernel leaves on plan_ok too
    bool ok = true;
    for (long long spins = 0; !__all(arrived(have, want)); ++spins) {      // bounded
        if (spins >= D.spin_limit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(64);
        if (lane < N) have = ld_relaxed(arrive + (size_t)r * N + lane);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");     // pairs with the senders' release adds
    if (threadIdx.x == 0) {
        gate[r] = ok ? 1 : 0;
        if (!ok) latch_status(W.status, FL_STATUS_TIMEOUT);
    }
}

// ------------------------------------------------------------------ dispatch: unpack
// Receiver half at rank d: every received row is written once per local expert that
// wants it, at
//   base_x[d][local expert][source] + rank carried in the sidecar,
// which is the (expert, source rank, token) order of the grouped layout.
//
// What both unpack kernels do beside the rows: block 0 hands the counts to the caller,
// the first blocks clear the padding between the experts when asked to.
__device__ inline void unpack_extras(const Dims &D, const Tables &W, int d, int tid, char *xd, float *expert_scales,
                                     int *tokens_per_expert) {
    const int El = D.El;
    if (blockIdx.x == 0)
        for (int j = tid; j < El; j += kCopyThreads)
            tokens_per_expert[(size_t)d * El + j] = W.G[(size_t)d * El + j];
    if ((D.flags & FL_FLAG_ZERO_PAD) && (int)blockIdx.x < El - 1) {
        const int j = blockIdx.x;
        const long long lo = W.expert_off[(size_t)d * (El + 1) + j] + W.G[(size_t)d * El + j];
        const long long hi = W.expert_off[(size_t)d * (El + 1) + j + 1];
        const long long nv = (hi - lo) * (D.Be / 16);
        uint4 *p = (uint4 *)(xd + lo * D.Be);
        for (long long v = tid; v < nv; v += kCopyThreads) p[v] = make_uint4(0, 0, 0, 0);
        if (expert_scales) {
            float *sp = expert_scales + ((size_t)d * D.expert_cap + lo) * D.scales_per_row;
            for (long long v = tid; v < (hi - lo) * D.scales_per_row; v += kCopyThreads) sp[v] = 0.f;
        }
    }
}

// Rows that have landed before the kernel starts (behind a gate kernel, or in the caller's
// stream order), unless they are many and short.  Bound by memory traffic in large steps and by the chain of dependent loads
// in small ones, so a wave works alone, without LDS or barriers: offsets and verdicts in one
// round, by a ballot over the offsets the row's source, then the wave's share of the row
// together with the sidecar, then, lane k for the k-th copy, its place, then the stores.
// (Loading the payload in the first round as well, before the number of rows is known, fetches
// rows nobody has: 151 -> 205 us.)  Large steps want fewer loads in flight than a
// compute unit can hold waves for: kRowWavesLdsBytes keeps five workgroups on each instead of
// eight (128 tokens, 14 KB rows: 160 us at eight, 156 at six, 147 at five and four; small
// steps and shorter rows measure the same).  Against a block that planned its rows in LDS
// first: 4 tokens 12.0 -> 9.7 us, 128: 151 -> 147, e4m3 75 -> 72, 6.7 KB rows 31 -> 29.
constexpr int kRowWavesLdsBytes = 32 << 10;
//
// WAIT (small launches in the default mode): no gate kernel ran; every wave waits (bounded) until all of the rank's
// sources have delivered, and reads rows and sidecars at device scope, because the launch may have been running when
// they landed; all waves of a rank reach one verdict (wave_wait_together).  Which launches: waits_itself in flmoe.hip.
template <bool PRIVATE, bool WAIT>   // PRIVATE: the receive buffer has private slots (P > 0): a row's place depends on its source
__global__ __launch_bounds__(kCopyThreads, 8) void dispatch_unpack_kernel(
    Dims D, Tables W, int rank_begin, char *__restrict__ expert_x,
    float *__restrict__ expert_scales, int *__restrict__ tokens_per_expert, int waves_per_row,
    unsigned launch /* WAIT: number of this launch */,
    const int *__restrict__ gate /* [N] or null: a gate kernel's verdict, 0 = its wait gave up */) {
    const int d = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, El = D.El, K = D.K;
    const int lane = tid & (kWave - 1);
    const int wave = blockIdx.x * (kCopyThreads / kWave) + __builtin_amdgcn_readfirstlane(tid / kWave);
    const int G = waves_per_row, sub = wave % G;
    const int row_step = (int)(gridDim.x * (kCopyThreads / kWave)) / G;     // the grid is a multiple of G blocks
    const char *recv = W.bufB + (size_t)d * D.bufB_rank_bytes;
    const int nvec = (int)(D.Be / 16);
    // e4m3: when the scales of a row are a whole number of 16-byte vectors they are moved by
    // the same loop (the vectors after the code bytes go to expert_scales)
    const bool scales_as_vectors = D.scales_per_row > 0 && D.scales_per_row % 4 == 0;
    const int rowvec = nvec + (scales_as_vectors ? D.scales_per_row / 4 : 0);
    const bool whole = D.Be % 128 == 0 && ((uintptr_t)expert_x & 127) == 0;    // expert rows are whole lines
    const int v0 = sub * kWave, step = G * kWave;          // the wave's first vectors of the row, distance to the next
    constexpr int U = 4;
    v4u val[U];
    unsigned m = kNoEntry;
    auto load_batch = [&](int phys, int b) {
        const char *src = recv + (size_t)phys * D.Sw;
#pragma unroll
        for (int i = 0; i < U; ++i)
            if (b + i * step < rowvec) val[i] = WAIT ? ld_coherent(src, b + i * step) : ld_stream((const v4u *)src + b + i * step);
    };
    auto load_meta = [&](int phys) {
        const unsigned *meta = W.recv_meta + ((size_t)d * D.recv_rows + phys) * D.MW + lane;
        m = lane < K ? WAIT ? ld_relaxed(meta) : *meta : kNoEntry;
    };
    // first round of loads, all independent
    int r = wave / G;
    const int plan_ok = W.plan_ok[d], gate_ok = gate ? gate[d] : 1;
    const int total = W.recv_off[(size_t)d * (N + 1) + N];
    const int off = lane < N ? W.recv_off[(size_t)d * (N + 1) + lane] : 0x7fffffff;
    const int shared_off = PRIVATE && lane < N ? W.recv_shared_off[(size_t)d * N + lane] : 0;
    const unsigned step_no = WAIT ? W.epoch_route[d] : 0u;
    unsigned want = 0, have = 0;
    if (!gate && lane < N) {
        want = W.expect_disp[(size_t)d * N + lane];
        have = ld_relaxed(W.arrive_disp + (size_t)d * N + lane);
    }
    if (!plan_ok || !gate_ok) return;               // step skipped, or the arrival wait timed out (already latched)
    // The counters are read by relaxed loads: the fence in verdict_read also keeps the compiler from moving the rows' loads in
    // front of them (no cache needs to be invalidated, the rows are read at device scope).
    const verdict_word ticket = WAIT ? launch_ticket(step_no, launch) : 0;
    verdict_word verdict = 0;
    bool go = !WAIT;                                // whether this wave may store
    auto leave = [&]() {                            // it may not
        if (lane == 0) verdict_left(verdict_of(W.done_disp, N, d), N, ticket, 1u, gridDim.x * (kCopyThreads / kWave));
    };
    if (WAIT) {
        if (__all(lane >= N || arrived(have, want))) {
            verdict = verdict_read(verdict_of(W.done_disp, N, d));         // on its way while the first row is loaded
        } else {
            if (!wave_wait_together(W.arrive_disp + (size_t)d * N, have, want, N, D.spin_limit, verdict_of(W.done_disp, N, d), ticket,
                                    wave == 0, W.status)) {
                leave();
                return;
            }
            go = true;
        }
    }
    auto may_store = [&]() {
        if (!WAIT || go) return true;
        asm volatile("" : "+v"(verdict));           // looked at here and not where it is read
        go = verdict_allows(verdict_of(W.done_disp, N, d), ticket, verdict);
        return go;
    };
    char *xd = expert_x + (size_t)d * D.expert_cap * D.Be;
    if (!WAIT) unpack_extras(D, W, d, tid, xd, expert_scales, tokens_per_expert);
    for (; r < total; r += row_step) {              // capacities are upper bounds: the grid may be smaller than the rows
        const int s = __popcll(__ballot(off <= r)) - 1;
        const int in_source = r - __builtin_amdgcn_readlane(off, s);
        const int phys = PRIVATE ? recv_buffer_row(N, D.P, s, in_source, __builtin_amdgcn_readlane(shared_off, s)) : r;
        if (!WAIT && !gate) {                       // stream order has made it so; checked, bounded
            const unsigned expected = (unsigned)__builtin_amdgcn_readlane(want, s);
            bool landed = arrived((unsigned)__builtin_amdgcn_readlane(have, s), expected);
            if (!landed) {
                for (long long spins = 0; !landed && spins < D.spin_limit; ++spins) {
                    __builtin_amdgcn_s_sleep(64);
                    landed = arrived(ld_relaxed(W.arrive_disp + (size_t)d * N + s), expected);
                }
                if (!landed) {
                    if (lane == 0) latch_status(W.status, FL_STATUS_TIMEOUT);
                    return;
                }
            }
        }
        load_batch(phys, v0 + lane);
        load_meta(phys);
        if (!may_store()) { leave(); return; }
        // copies of this row: entries come first in the sidecar
        const int n = __popcll(__ballot(m != kNoEntry));
        int place = 0;
        if (m != kNoEntry) place = W.base_x[((size_t)d * El + (m >> 24)) * N + s] + (int)(m & 0xFFFFFFu);
        // the whole wave stays in these loops, lanes beyond the row idle: a copy's place may stand in any lane
        for (int b0 = v0; b0 < rowvec; b0 += U * step) {
            const int b = b0 + lane;
            if (b0 != v0) load_batch(phys, b);
            for (int k = 0; k < n; ++k) {
                const size_t dr = (size_t)__builtin_amdgcn_readlane(place, k);
                v4u *dst = (v4u *)(xd + dr * D.Be);
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    const int v = b + i * step;
                    if (v < nvec) { if (whole) st_through_stream(dst + v, val[i]); else st_stream(dst + v, val[i]); }
                    else if (v < rowvec)
                        st_stream((v4u *)(expert_scales + ((size_t)d * D.expert_cap + dr) * D.scales_per_row) + (v - nvec),
                                  val[i]);
                }
            }
        }
        if (D.scales_per_row && !scales_as_vectors && sub == 0) {   // odd scale counts: element by element
            const float *ssrc = (const float *)(recv + (size_t)phys * D.Sw + D.Be);
            for (int b = 0; b < D.scales_per_row; b += kWave) {
                const int v = b + lane;
                const float sc = v >= D.scales_per_row ? 0.f
                                 : WAIT ? __uint_as_float(ld_relaxed((const unsigned *)ssrc + v)) : ssrc[v];
                for (int k = 0; k < n; ++k) {
                    const size_t dr = (size_t)__builtin_amdgcn_readlane(place, k);
                    if (v < D.scales_per_row) expert_scales[((size_t)d * D.expert_cap + dr) * D.scales_per_row + v] = sc;
                }
            }
        }
    }
    if (WAIT) {
        if (may_store()) unpack_extras(D, W, d, tid, xd, expert_scales, tokens_per_expert);
        else leave();
    }
}

// Short rows, and every row in progressive mode: a block takes a chunk of received rows at a time,
// plans their copies in LDS and moves the chunk as one run of vectors, so that no lane idles however
// short a row is; the wave kernel above is bound by the rate at which waves start then (rule and
// both sides' times: by_chunks in flmoe.hip).
//
// POLL (progressive mode): the block waits (bounded) for the arrival counters of the sources its
// rows came from.  The kernel may have been started before any payload
// exists, on a grid that is a fraction of the machine, so a block walks many
// chunks.  It keeps the set of sources it has seen complete: a chunk whose
// sources are all in the set costs no poll; otherwise one wave polls the
// counters of ALL sources at once (one load per lane), waits until the chunk's
// own sources are complete, and invalidates the caches once, because it is about
// to rely on arrivals it had not seen before.  That is the whole visibility
// rule: payload and sidecar of a source are read only after its counter was
// seen complete and the caches were invalidated after that observation (a line
// fetched earlier, for a neighbouring row, may hold this source's bytes from
// before they landed; a line fetched later cannot).  The chunk's first payload
// loads are issued before its sidecars are decoded, so a chunk costs one memory
// round trip, not four.
template <bool PRIVATE, bool POLL>   // PRIVATE: the receive buffer has private slots (P > 0)
__global__ __launch_bounds__(kCopyThreads) void dispatch_unpack_chunk_kernel(
    Dims D, Tables W, int rank_begin, char *__restrict__ expert_x,
    float *__restrict__ expert_scales, int *__restrict__ tokens_per_expert, int rows_per_block,
    const int *__restrict__ gate /* as in dispatch_unpack_kernel */) {
    const int d = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, El = D.El, K = D.K;
    __shared__ int off[FL_MAX_RANKS + 1];
    __shared__ int dst_rows[kMaxRowsPerBlock][FL_MAX_TOPK];
    __shared__ int dst_cnt[kMaxRowsPerBlock];
    __shared__ int src_phys[kMaxRowsPerBlock];      // with private slots: buffer row of each received row
    __shared__ int timed_out;
    __shared__ unsigned long long seen_pub;         // wave 0 publishes the set of complete sources
    // first round of loads, all independent: the verdicts, the rows in use, the source offsets
    const int plan_ok = W.plan_ok[d], gate_ok = gate ? gate[d] : 1;
    const int total = W.recv_off[(size_t)d * (N + 1) + N];
    const int off_mine = tid <= N ? W.recv_off[(size_t)d * (N + 1) + tid] : 0;
    if (!plan_ok || !gate_ok) return;
    char *xd = expert_x + (size_t)d * D.expert_cap * D.Be;
    unpack_extras(D, W, d, tid, xd, expert_scales, tokens_per_expert);
    // grids are sized from capacities: blocks beyond the rows in use leave at once
    if ((int)blockIdx.x * rows_per_block >= total) return;
    if (tid <= N) off[tid] = off_mine;
    if (tid == 0) timed_out = 0;
    __syncthreads();
    const char *recv = W.bufB + (size_t)d * D.bufB_rank_bytes;
    const int nvec = (int)(D.Be / 16);
    const bool scales_as_vectors = D.scales_per_row > 0 && D.scales_per_row % 4 == 0;
    const int rowvec = nvec + (scales_as_vectors ? D.scales_per_row / 4 : 0);
    unsigned long long seen = 0;                    // POLL: sources seen complete (same in every thread)
    unsigned my_expect = 0;                         // POLL, wave 0: lane i holds what source i must deliver
    if (POLL && tid < N) my_expect = W.expect_disp[(size_t)d * N + tid];
    // capacities are upper bounds, so the grid may be smaller than the rows in use
    for (int r0 = blockIdx.x * rows_per_block; r0 < total; r0 += gridDim.x * rows_per_block) {
        const int r1 = min(r0 + rows_per_block, total);
        const int s0 = seg_of(off, N, r0), s1 = seg_of(off, N, r1 - 1);
        if (POLL && tid < kWave) {
            const unsigned long long range = ((s1 - s0 == 63) ? ~0ull : ((1ull << (s1 - s0 + 1)) - 1)) << s0;
            if (range & ~seen) {                // uniform: every thread holds the same `seen`
                long long spins = 0;
                for (;;) {
                    bool ok = false;
                    if (tid < N) ok = arrived(ld_relaxed(W.arrive_disp + (size_t)d * N + tid), my_expect);
                    seen |= __ballot(ok);
                    if (!(range & ~seen)) break;
                    if (++spins > D.spin_limit) {
                        if (tid == 0) { timed_out = 1; latch_status(W.status, FL_STATUS_TIMEOUT); }
                        break;
                    }
                    __builtin_amdgcn_s_sleep(64);
                }
                acquire_payload<true>();      // arrivals not relied on before: drop what the caches hold
            }
            if (tid == 0) seen_pub = seen;
        } else if (!POLL && !gate && tid < kWave) {    // stream order has made it so; checked, bounded
            if (!wave_wait_counters(W.arrive_disp + (size_t)d * N + s0, W.expect_disp + (size_t)d * N + s0, 0u,
                                    s1 - s0 + 1, D.spin_limit)) {
                if (tid == 0) { timed_out = 1; latch_status(W.status, FL_STATUS_TIMEOUT); }
            }
        }
        __syncthreads();
        if (timed_out) return;
        if (POLL) seen = seen_pub;
        // e4m3: when the scales of a row are a whole number of 16-byte vectors they are
        // moved by the same loop (the vectors after the code bytes go to expert_scales)
        const int chunk = (r1 - r0) * rowvec;
        // U loads per thread in flight: a full grid keeps the memory system busy with 4; the
        // capped grid of polling receivers has fewer waves per compute unit and needs 8
        constexpr int U = POLL ? 8 : 4;
        auto load_batch = [&](int b, v4u *val, int *row, int *col) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int v = b + i * kCopyThreads;
                if (v < chunk) {
                    row[i] = v / rowvec;
                    col[i] = v - row[i] * rowvec;
                    const int pr = PRIVATE ? src_phys[row[i]] : r0 + row[i];
                    val[i] = ld_stream((const v4u *)(recv + (size_t)pr * D.Sw) + col[i]);
                }
            }
        };
        auto plan_rows = [&]() {
            if (tid < r1 - r0) {               // plan of one received row: its expert-major rows
                const int r = r0 + tid;
                const int s = seg_of(off, N, r);
                int phys = r;
                if (PRIVATE) {
                    phys = recv_buffer_row(N, D.P, s, r - off[s], W.recv_shared_off[(size_t)d * N + s]);
                    src_phys[tid] = phys;
                }
                // entry k + 1 is fetched before entry k is looked at, so that it travels together
                // with the base row of entry k (most rows have one entry: two round trips, not three)
                const unsigned *meta = W.recv_meta + ((size_t)d * D.recv_rows + phys) * D.MW;
                int n = 0;
                unsigned m = meta[0];
                for (int k = 0; k < K; ++k) {
                    const unsigned m_next = k + 1 < K ? meta[k + 1] : kNoEntry;
                    if (m == kNoEntry) break;
                    const int j = (int)(m >> 24), i = (int)(m & 0xFFFFFFu);
                    dst_rows[tid][n++] = W.base_x[((size_t)d * El + j) * N + s] + i;
                    m = m_next;
                }
                dst_cnt[tid] = n;
            }
        };
        auto store_batch = [&](int b, const v4u *val, const int *row, const int *col) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int v = b + i * kCopyThreads;
                if (v < chunk) {
                    const int n = dst_cnt[row[i]];
                    for (int j = 0; j < n; ++j) {
                        const size_t dr = (size_t)dst_rows[row[i]][j];
                        if (col[i] < nvec)
                            st_stream((v4u *)(xd + dr * D.Be) + col[i], val[i]);
                        else
                            st_stream((v4u *)(expert_scales + ((size_t)d * D.expert_cap + dr) *
                                                                  D.scales_per_row) + (col[i] - nvec), val[i]);
                    }
                }
            }
        };
        if (POLL && !PRIVATE) {
            // the first batch's loads go out before the sidecars are decoded: a chunk then
            // costs one memory round trip instead of three in a row (polling receivers run with few
            // waves per compute unit; on a full grid the registers it takes cost more than it gains)
            v4u val[U];
            int row[U], col[U];
            load_batch(tid, val, row, col);
            plan_rows();
            __syncthreads();
            store_batch(tid, val, row, col);
            for (int b = tid + U * kCopyThreads; b < chunk; b += U * kCopyThreads) {
                load_batch(b, val, row, col);
                store_batch(b, val, row, col);
            }
        } else {
            plan_rows();
            __syncthreads();
            for (int b = tid; b < chunk; b += U * kCopyThreads) {
                v4u val[U];
                int row[U], col[U];
                load_batch(b, val, row, col);
                store_batch(b, val, row, col);
            }
        }
        if (D.scales_per_row && !scales_as_vectors) {   // odd scale counts: element by element
            for (int v = tid; v < (r1 - r0) * D.scales_per_row; v += kCopyThreads) {
                const int row = v / D.scales_per_row, col = v - row * D.scales_per_row;
                const int pr = PRIVATE ? src_phys[row] : r0 + row;
                const float val = ((const float *)(recv + (size_t)pr * D.Sw + D.Be))[col];
                for (int i = 0; i < dst_cnt[row]; ++i)
                    expert_scales[((size_t)d * D.expert_cap + dst_rows[row][i]) * D.scales_per_row + col] = val;
            }
        }
        __syncthreads();                       // the row plan in LDS is rewritten by the next chunk
    }
}

// How a combine_send call stores its replies and who announces them: one choice (reply_form in flmoe.hip), because
// a workgroup's acknowledged stores are in memory only when they are written through.  Streamed replies may still be
// dirty in an L2 until their kernel ends, so only the announce kernel behind it can vouch for them.
enum ReplyForm {
    kRepliesStreamed,            // announced behind the kernel
    kRepliesThrough,             // written through (st_payload), announced behind the kernel
    kRepliesThroughAnnounced     // written through, and the sender's last workgroup announces them (announce_when_last)
};

// ------------------------------------------------------------------ combine: pack
// Rank d sends every source s the rows of its experts that belong to s (contiguous
// per expert in the grouped layout) as one contiguous reply, into s's combine receive
// buffer: reply row q of source s and local expert j comes from expert-major row
// base_x[d][j][s] + (q - cs_base[d][s][j]).
//
// A wave works alone on its share of a row, as in the unpack kernel: the row's source by a
// ballot over the reply offsets, its expert by one over the source's per-expert offsets
// (fetched together with the expert rows they stand for), then the copy: three dependent
// rounds of loads and no barrier, against five and two when a workgroup planned its rows in LDS.
// Bound by memory traffic from 32 tokens on (6.5 TB/s at 128 tokens, the plain copy's rate),
// by the chain below.  Before -> now: 4 tokens 11.6 -> 11.0 us, 8: 15.9 -> 15.0, 32: 40.7 -> 39.5,
// 128: 144.5 -> 144, 512: 649 -> 631 (672 with eight workgroups per unit).
template <int FORM>   // ReplyForm
__global__ __launch_bounds__(kCopyThreads, 8) void combine_pack_kernel(
    Dims D, Tables W, int rank_begin, const char *__restrict__ expert_y, int waves_per_row) {
    const int d = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, El = D.El;
    const int lane = tid & (kWave - 1);
    const int wave = blockIdx.x * (kCopyThreads / kWave) + __builtin_amdgcn_readfirstlane(tid / kWave);
    const int G = waves_per_row, sub = wave % G;
    const int row_step = (int)(gridDim.x * (kCopyThreads / kWave)) / G;     // the grid is a multiple of G blocks
    const int nvec = (int)(D.Bc / 16), v0 = sub * kWave + lane, step = G * kWave;
    // one round of loads
    const int plan_ok = W.plan_ok[d];
    const int total = W.cs_off[(size_t)d * (N + 1) + N];
    const int off = lane < N ? W.cs_off[(size_t)d * (N + 1) + lane] : 0x7fffffff;
    const int reply = lane < N ? W.comb_dst_off[(size_t)d * N + lane] : 0;
    if (!plan_ok) return;
    // stream-ordered: the rank's first block announces the replies (a rank without rows its empty ones)
    if ((D.flags & FL_FLAG_STREAM_ORDERED) && blockIdx.x == 0)
        announce_transfers(W.cs_off + (size_t)d * (N + 1), W.arrive_comb, (unsigned)nvec, d, N, tid, kCopyThreads);
    const char *yd = expert_y + (size_t)d * D.expert_cap * D.Bc;
    for (int i = wave / G; i < total; i += row_step) {      // capacities are upper bounds: the grid may be smaller
        const int q = in_order(D.tune_order, i, total);
        const int s = __popcll(__ballot(off <= q)) - 1;
        int src_row = 0;                                    // of the last expert whose rows for s start at or before q
        for (int j0 = 0; j0 < El; j0 += kWave) {
            const bool in = j0 + lane < El;
            const int first = in ? W.cs_base[((size_t)d * N + s) * El + j0 + lane] : 0x7fffffff;
            const int base = in ? W.base_x[((size_t)d * El + j0 + lane) * N + s] : 0;
            const int j = __popcll(__ballot(first <= q)) - 1;
            if (j >= 0) src_row = __builtin_amdgcn_readlane(base, j) + q - __builtin_amdgcn_readlane(first, j);
            if (j < kWave - 1) break;
        }
        const v4u *src = (const v4u *)(yd + (size_t)src_row * D.Bc);
        v4u *dst = (v4u *)(W.bufA + (size_t)s * D.bufA_rank_bytes +
                           (size_t)(__builtin_amdgcn_readlane(reply, s) + q - __builtin_amdgcn_readlane(off, s)) * D.Sc);
        for (int b = v0; b < nvec; b += 4 * step) {
            v4u val[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (b + u * step < nvec) val[u] = ld_stream(src + b + u * step);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (b + u * step < nvec) st_payload<FORM != kRepliesStreamed>(dst + b + u * step, val[u]);
        }
    }
    if (FORM == kRepliesThroughAnnounced) {
        const int *rows = W.cs_off + (size_t)d * (N + 1) + lane;
        announce_when_last(W.done_comb + d * kDoneWords, blockIdx.x, gridDim.x, W.arrive_comb, lane < N ? rows[1] - rows[0] : 0,
                           (unsigned)nvec, d, N, lane, wave % (kCopyThreads / kWave) == 0);
    }
}

// Short rows, and every row in progressive mode: a workgroup per chunk of rows, as in the unpack kernels.
// FENCED (progressive mode): written through, and the workgroup adds each row's units
// to arrive[source][this rank] itself, once per row rather than once per wave.
template <bool FENCED, bool THROUGH>
__global__ __launch_bounds__(kCopyThreads) void combine_pack_chunk_kernel(
    Dims D, Tables W, int rank_begin, const char *__restrict__ expert_y, int rows_per_block) {
    const int d = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, El = D.El;
    __shared__ int off[FL_MAX_RANKS + 1];
    __shared__ int src_row[kMaxRowsPerBlock];
    __shared__ int2 push_to[kMaxRowsPerBlock];     // (source rank, row of its combine receive buffer)
    if (!W.plan_ok[d]) return;
    const int nvec = (int)(D.Bc / 16);
    // the rank's first block announces the replies (a rank without rows its empty ones), unless an
    // announce kernel will
    if ((FENCED || (D.flags & FL_FLAG_STREAM_ORDERED)) && blockIdx.x == 0)
        announce_transfers(W.cs_off + (size_t)d * (N + 1), W.arrive_comb, (unsigned)nvec, d, N, tid, kCopyThreads,
                           FENCED);
    // grids are sized from capacities: blocks beyond the rows in use leave at once
    const int total = W.cs_off[(size_t)d * (N + 1) + N];
    if ((int)blockIdx.x * rows_per_block >= total) return;
    if (tid <= N) off[tid] = W.cs_off[(size_t)d * (N + 1) + tid];
    __syncthreads();
    const char *yd = expert_y + (size_t)d * D.expert_cap * D.Bc;
    // capacities are upper bounds, so the grid may be smaller than the rows in use
    const int chunks = (total + rows_per_block - 1) / rows_per_block;
    for (int c = blockIdx.x; c < chunks; c += gridDim.x) {
        const int q0 = in_order(D.tune_order, c, chunks) * rows_per_block, q1 = min(q0 + rows_per_block, total);
        if (tid < q1 - q0) {
            const int q = q0 + tid;
            const int s = seg_of(off, N, q);
            int first;                         // first reply row of (source s, local expert j)
            const int j = seg_of_short(W.cs_base + ((size_t)d * N + s) * El, El, q, &first);
            src_row[tid] = W.base_x[((size_t)d * El + j) * N + s] + (q - first);
            push_to[tid] = make_int2(s, W.comb_dst_off[(size_t)d * N + s] + (q - off[s]));
        }
        __syncthreads();
        copy_rows_flat<kCopyThreads, THROUGH>(
            q1 - q0, nvec, tid,
            [&](int r) { return yd + (size_t)src_row[r] * D.Bc; },
            [&](int r) {
                return W.bufA + (size_t)push_to[r].x * D.bufA_rank_bytes + (size_t)push_to[r].y * D.Sc;
            });
        if (FENCED) {
            stores_done();
            __syncthreads();
            if (tid < q1 - q0) add_counter(W.arrive_comb + (size_t)push_to[tid].x * N + d, (unsigned)nvec);
        }
        __syncthreads();                       // the row plan is rewritten by the next chunk
    }
}

// acc[0..7] += wk * (the eight bf16 values of y), fused
__device__ inline void fma8(float *acc, float wk, v4u y) {
    acc[0] = fmaf(wk, bf16_lo(y.x), acc[0]); acc[1] = fmaf(wk, bf16_hi(y.x), acc[1]);
    acc[2] = fmaf(wk, bf16_lo(y.y), acc[2]); acc[3] = fmaf(wk, bf16_hi(y.y), acc[3]);
    acc[4] = fmaf(wk, bf16_lo(y.z), acc[4]); acc[5] = fmaf(wk, bf16_hi(y.z), acc[5]);
    acc[6] = fmaf(wk, bf16_lo(y.w), acc[6]); acc[7] = fmaf(wk, bf16_hi(y.w), acc[7]);
}

// ------------------------------------------------------------------ combine: pack with sender-side partial sums
// Section Comparison with DeepEP: tokens can be pre-accumulated on the sending
// side, which moves fewer rows at the price of a bf16 rounding between the two
// stages.  Rank d answers every row it received with ONE row: the fp32 fused
// multiply-add chain, in the order of the row's sidecar (ascending k), of
// weight * expert output over the token's experts on d, rounded to bf16.  The
// share of received row number i from source s goes back to row
// ret_off[d][s] + i of s's combine receive buffer, the position of the token copy among
// all copies s sent, so s finds it through its own send_to table.
//
// A wave works alone on its share of a row, as in the unpack and combine pack kernels: the
// row's source by a ballot, lane k for the sidecar's k-th entry, its expert row and its weight,
// then the sum.  Bound by reads (P rows read, D written); workgroups are not held back here: the
// same five per unit as the plain copy takes measured 30 us where all eight take 26 (6.7 KB rows).
// Against a workgroup that planned its rows in LDS: 301 tokens x 8 ranks, 6.7 KB rows 30.6 -> 26.1 us;
// 14 KB rows, 32 ranks: 8 tokens 20.4 -> 16.1, 128: 147 -> 136, 512: 641 -> 627.  The launch bound keeps
// it at 72 registers; one more and only six workgroups fit a unit: 2 KB rows, step 277 -> 286 us.  So nothing that announcing
// needs is held over the row loop, and calls that do not announce themselves carry none of it: with both in every variant
// three registers were spilled; us of a step without: 8 tokens of 14 KB 58.6 -> 57.7, 301 of 6.7 KB 92.5 -> 91.7, 128: 445 -> 442.
//
// A sidecar is what a sender stored, and behind an arrival wait that gave up (the caller's calls are all
// enqueued by then) it holds whatever was there before: the expert row it names is kept inside expert_y.
__device__ inline int sidecar_expert_row(const Dims &D, const Tables &W, int d, int s, unsigned entry) {
    const unsigned j = min(entry >> 24, (unsigned)D.El - 1u);
    const unsigned row = (unsigned)W.base_x[((size_t)d * D.El + j) * D.N + s] + (entry & 0xFFFFFFu);
    return (int)min(row, (unsigned)D.expert_cap - 1u);
}

template <int FORM>   // ReplyForm
__global__ __launch_bounds__(kCopyThreads, 7) void combine_partial_pack_kernel(
    Dims D, Tables W, int rank_begin, const char *__restrict__ expert_y, int waves_per_row) {
    const int d = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, K = D.K;
    const int lane = tid & (kWave - 1);
    const int wave = blockIdx.x * (kCopyThreads / kWave) + __builtin_amdgcn_readfirstlane(tid / kWave);
    const int G = waves_per_row, sub = wave % G;
    const int row_step = (int)(gridDim.x * (kCopyThreads / kWave)) / G;     // the grid is a multiple of G blocks
    const int nvec = (int)(D.Bc / 16), v0 = sub * kWave, step = G * kWave;
    // one round of loads
    const int plan_ok = W.plan_ok[d];
    const int total = W.recv_off[(size_t)d * (N + 1) + N];
    const int off = lane < N ? W.recv_off[(size_t)d * (N + 1) + lane] : 0x7fffffff;
    const int ret = lane < N ? W.ret_off[(size_t)d * N + lane] : 0;
    const int shared_off = D.P && lane < N ? W.recv_shared_off[(size_t)d * N + lane] : 0;
    if (!plan_ok) return;
    if ((D.flags & FL_FLAG_STREAM_ORDERED) && blockIdx.x == 0)   // as in combine_pack_kernel
        announce_transfers(W.recv_off + (size_t)d * (N + 1), W.arrive_comb, (unsigned)nvec, d, N, tid, kCopyThreads);
    const char *yd = expert_y + (size_t)d * D.expert_cap * D.Bc;
    for (int c = wave / G; c < total; c += row_step) {
        const int r = in_order(D.tune_order, c, total);
        const int s = __popcll(__ballot(off <= r)) - 1;
        const int i = r - __builtin_amdgcn_readlane(off, s);
        const int phys = D.P ? recv_buffer_row(N, D.P, s, i, __builtin_amdgcn_readlane(shared_off, s)) : r;
        const unsigned *meta = W.recv_meta + ((size_t)d * D.recv_rows + phys) * D.MW;
        const unsigned m = lane < K ? meta[lane] : kNoEntry;
        const unsigned weight = lane < K ? meta[D.KM + lane] : 0u;
        const int n = __popcll(__ballot(m != kNoEntry));       // entries come first in the sidecar
        int place = 0;
        if (m != kNoEntry) place = sidecar_expert_row(D, W, d, s, m);
        char *dst = W.bufA + (size_t)s * D.bufA_rank_bytes + (size_t)(__builtin_amdgcn_readlane(ret, s) + i) * D.Sc;
        constexpr int U = 4;
        // the whole wave, as in the unpack kernel; lanes beyond the row sum its last vector and store nothing
        for (int b0 = v0; b0 < nvec; b0 += U * step) {
            const int b = b0 + lane;
            float acc[U][8];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[u][e] = 0.f;
            for (int k = 0; k < n; ++k) {
                const v4u *src = (const v4u *)(yd + (size_t)__builtin_amdgcn_readlane(place, k) * D.Bc);
                const float wk = __uint_as_float(__builtin_amdgcn_readlane(weight, k));
                v4u y[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (b0 + u * step < nvec) y[u] = ld_stream(src + min(b + u * step, nvec - 1));
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (b0 + u * step < nvec) fma8(acc[u], wk, y[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (b + u * step < nvec) {
                    v4u o;
                    o.x = pack_bf16x2(acc[u][0], acc[u][1]); o.y = pack_bf16x2(acc[u][2], acc[u][3]);
                    o.z = pack_bf16x2(acc[u][4], acc[u][5]); o.w = pack_bf16x2(acc[u][6], acc[u][7]);
                    st_payload<FORM != kRepliesStreamed>((v4u *)dst + b + u * step, o);
                }
        }
    }
    if (FORM == kRepliesThroughAnnounced) {        // the offsets again, not held over the loop
        const int *rows = W.recv_off + (size_t)d * (N + 1) + lane;
        announce_when_last(W.done_comb + d * kDoneWords, blockIdx.x, gridDim.x, W.arrive_comb, lane < N ? rows[1] - rows[0] : 0,
                           (unsigned)nvec, d, N, lane, wave % (kCopyThreads / kWave) == 0);
    }
}

// Short rows, and every row in progressive mode: a workgroup per chunk of rows; FENCED, THROUGH as in
// combine_pack_chunk_kernel.
template <bool FENCED, bool THROUGH>
__global__ __launch_bounds__(kCopyThreads) void combine_partial_pack_chunk_kernel(
    Dims D, Tables W, int rank_begin, const char *__restrict__ expert_y, int rows_per_block) {
    const int d = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, K = D.K;
    __shared__ int off[FL_MAX_RANKS + 1];
    __shared__ int src_rows[kMaxRowsPerBlock][FL_MAX_TOPK];
    __shared__ float src_w[kMaxRowsPerBlock][FL_MAX_TOPK];
    __shared__ int src_cnt[kMaxRowsPerBlock];
    __shared__ int2 share_to[kMaxRowsPerBlock];
    if (!W.plan_ok[d]) return;
    const int nvec = (int)(D.Bc / 16);
    if ((FENCED || (D.flags & FL_FLAG_STREAM_ORDERED)) && blockIdx.x == 0)
        announce_transfers(W.recv_off + (size_t)d * (N + 1), W.arrive_comb, (unsigned)nvec, d, N, tid, kCopyThreads,
                           FENCED);
    const int total = W.recv_off[(size_t)d * (N + 1) + N];
    if ((int)blockIdx.x * rows_per_block >= total) return;
    if (tid <= N) off[tid] = W.recv_off[(size_t)d * (N + 1) + tid];
    __syncthreads();
    const char *yd = expert_y + (size_t)d * D.expert_cap * D.Bc;
    const int chunks = (total + rows_per_block - 1) / rows_per_block;
    for (int c = blockIdx.x; c < chunks; c += gridDim.x) {
        const int r0 = in_order(D.tune_order, c, chunks) * rows_per_block, r1 = min(r0 + rows_per_block, total);
        if (tid < r1 - r0) {
            const int r = r0 + tid;
            const int s = seg_of(off, N, r);
            const int i = r - off[s];
            const int phys = D.P ? recv_buffer_row(N, D.P, s, i, W.recv_shared_off[(size_t)d * N + s]) : r;
            const unsigned *meta = W.recv_meta + ((size_t)d * D.recv_rows + phys) * D.MW;
            int n = 0;
            src_rows[tid][0] = 0;              // read below whatever the sidecar says
            src_w[tid][0] = 0.f;
            for (int k = 0; k < K; ++k) {
                const unsigned m = meta[k];
                if (m == kNoEntry) break;
                src_rows[tid][n] = sidecar_expert_row(D, W, d, s, m);
                src_w[tid][n] = __uint_as_float(meta[D.KM + k]);
                ++n;
            }
            src_cnt[tid] = n;
            share_to[tid] = make_int2(s, W.ret_off[(size_t)d * N + s] + i);
        }
        __syncthreads();
        const int chunk = (r1 - r0) * nvec;
        for (int b = tid; b < chunk; b += 4 * kCopyThreads) {
            v4u y0[4];
            int row[4], col[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {          // the first expert row of four items in flight
                const int v = b + u * kCopyThreads;
                if (v < chunk) {
                    row[u] = v / nvec;
                    col[u] = v - row[u] * nvec;
                    y0[u] = ld_stream((const v4u *)(yd + (size_t)src_rows[row[u]][0] * D.Bc) + col[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int v = b + u * kCopyThreads;
                if (v >= chunk) continue;
                float acc[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = 0.f;
                fma8(acc, src_w[row[u]][0], y0[u]);
                const int n = src_cnt[row[u]];
                for (int k = 1; k < n; ++k)
                    fma8(acc, src_w[row[u]][k],
                         ld_stream((const v4u *)(yd + (size_t)src_rows[row[u]][k] * D.Bc) + col[u]));
                v4u o;
                o.x = pack_bf16x2(acc[0], acc[1]); o.y = pack_bf16x2(acc[2], acc[3]);
                o.z = pack_bf16x2(acc[4], acc[5]); o.w = pack_bf16x2(acc[6], acc[7]);
                char *dst = W.bufA + (size_t)share_to[row[u]].x * D.bufA_rank_bytes + (size_t)share_to[row[u]].y * D.Sc;
                st_payload<THROUGH>((v4u *)dst + col[u], o);
            }
        }
        if (FENCED) {
            stores_done();
            __syncthreads();
            if (tid < r1 - r0) add_counter(W.arrive_comb + (size_t)share_to[tid].x * N + d, (unsigned)nvec);
        }
        __syncthreads();                       // the row plan is rewritten by the next chunk
    }
}

// ------------------------------------------------------------------ combine: reduce
// One block per token (s, t):
//   out[s][t] = bf16( sum_k w[k] * float(row comb_pos[s][t][k]) ), fp32 fused
// multiply-add, k ascending, one final rounding.

// With one or two rows per sum the output is a third of the traffic or more: where it is large it is written through with
// the streaming hint, so that lines nobody reads again do not push out rows that are.  us of a step of 32 ranks, 14 KB rows,
// without the hint and with it: top 1: 48 tokens (22 MB of output) 66.0 and 66.5, 80: 88.5 and 88.5, 112: 112.3 and 111.8, 144:
// 137.6 and 133.6, 256: 226 and 217 (ordinary streaming stores 218), 1024: 851 and 833; top 2: 80 tokens 112.5 and 112.3, 112: 147.5
// and 145.3, 208: 259 and 245, 1024: 1238 and 1226; 16 ranks, 4 KB rows, 33 MB top 2 95.6 and 96.7, 84 MB 212 and 196.
// Rows that begin or end inside lines lose by writing through in parts: streaming stores there.  us of a step written through,
// with the hint as well, with the hint alone: 16 ranks x 1000 tokens of 6672 bytes top 1 181, 188.5, 180.4, top 2 273.5, 273.6,
// 264.5; 32 ranks x 512 of 14 352 top 1 437, 432, 425, top 2 652, 635, 635; 32 x 2032 of 2352 top 1 251.6, 255, 250.1 (256 tokens,
// 19 MB: 63.2, 64.4, 64.0).  Whole lines, 16 x 1024 of 4 KB top 2 163.6, 164.4, 165.1.
// More rows per sum gain nothing (top 3, 256 tokens 416 and 418; top 8, 128: 449 and 451).
// (A choice inside the kernel cost what it gained.  Rule: output_stores in flmoe.hip.)
enum OutputStores { kOutThrough, kOutThroughHint, kOutHint };      // OUT: output_stores in flmoe.hip
template <int OUT>
__device__ inline void st_output(v4u *p, v4u v) {
    if (OUT == kOutThrough) st_through(p, v);
    else if (OUT == kOutThroughHint) st_through_stream(p, v);
    else st_stream(p, v);
}

// KT = number of row loads issued together (then consumed in k order); the sum
// itself always runs k = 0..K-1.
template <int KT, int OUT, class MayFn>
__device__ inline void reduce_row(const char *__restrict__ recv, const int *pos, const float *w,
                                  int K, long long stride, int v0, int nvec, v4u *__restrict__ out, int tid, MayFn may_store) {
    for (int v = v0 + tid; v < nvec; v += (int)blockDim.x) {
        float acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        int k0 = 0;
        for (; k0 + KT <= K; k0 += KT) {
            v4u y[KT];
#pragma unroll
            for (int k = 0; k < KT; ++k)
                y[k] = ld_stream((const v4u *)(recv + (size_t)pos[k0 + k] * stride) + v);
#pragma unroll
            for (int k = 0; k < KT; ++k) fma8(acc, w[k0 + k], y[k]);
        }
        for (; k0 < K; ++k0)
            fma8(acc, w[k0], ld_stream((const v4u *)(recv + (size_t)pos[k0] * stride) + v));
        v4u o;
        o.x = pack_bf16x2(acc[0], acc[1]); o.y = pack_bf16x2(acc[2], acc[3]);
        o.z = pack_bf16x2(acc[4], acc[5]); o.w = pack_bf16x2(acc[6], acc[7]);
        if (!may_store()) return;
        st_output<OUT>(out + v, o);
    }
}

// The same sum for a row count only known on the device (partial sums: one row per
// distinct expert rank of the token): batches of up to 8 loads, predicated.
template <int OUT, class MayFn>
__device__ inline void reduce_row_counted(const char *__restrict__ recv, const int *pos,
                                          const float *w, int n, long long stride, int v0, int nvec,
                                          v4u *__restrict__ out, int tid, MayFn may_store) {
    for (int v = v0 + tid; v < nvec; v += (int)blockDim.x) {
        float acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        for (int k0 = 0; k0 < n; k0 += 8) {
            v4u y[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k0 + k < n) y[k] = ld_stream((const v4u *)(recv + (size_t)pos[k0 + k] * stride) + v);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k0 + k < n) fma8(acc, w[k0 + k], y[k]);
        }
        v4u o;
        o.x = pack_bf16x2(acc[0], acc[1]); o.y = pack_bf16x2(acc[2], acc[3]);
        o.z = pack_bf16x2(acc[4], acc[5]); o.w = pack_bf16x2(acc[6], acc[7]);
        if (!may_store()) return;
        st_output<OUT>(out + v, o);
    }
}

// The block has min(1024, vectors per row rounded up to a wave) threads, so a
// 7168-wide row is one vector per thread and all K loads of a thread are in
// flight at once.
constexpr int kReduceMaxThreads = 1024;
//
// WAITS: kBehindGate when the rows have landed before the kernel starts (or in the caller's stream order: checked, bounded).
// The other two wait for the counters themselves and invalidate the caches before they read the rows: kProgressive,
// every workgroup for itself; kWaitsItself, small launches of the default mode (waits_itself in flmoe.hip), all waves of a rank
// with one verdict.  What the verdict needs costs registers (65, one workgroup of 14 waves per unit instead of two), so the
// progressive form carries none of it: 32 ranks x 128 tokens of 14 KB on two streams 647 us a step with it, 616 without.
enum ReduceWaits { kBehindGate, kProgressive, kWaitsItself };
//
// PARTIAL (sender-side partial sums): the token's rows are the shares of its
// distinct expert ranks, found through send_to[s][t][k] for every k that is the first
// of its rank; they are added in that order in fp32 (a fused multiply-add with
// weight 1 is an exact add), the weights having been applied on the expert ranks.
template <int WAITS, bool PARTIAL, int OUT>
__global__ __launch_bounds__(kReduceMaxThreads, 7) void combine_reduce_kernel(
    Dims D, Tables W, int rank_begin, const float *__restrict__ weights, char *__restrict__ out,
    const int *__restrict__ num_tokens, const int *__restrict__ gate /* as in dispatch_unpack_kernel */,
    int parts /* workgroups that share one token, each taking a slice of the row */,
    unsigned launch /* number of this launch where it waits in the default mode */) {
    const int s = rank_begin + blockIdx.y, tid = threadIdx.x, N = D.N, K = D.K;
    const int t0 = blockIdx.x / parts, part = blockIdx.x - t0 * parts, t_step = gridDim.x / parts;
    // two sets of positions and weights: while the block sums one token, wave 1 already
    // fetches the next one's (a block only walks several tokens when the grid is smaller
    // than the token count, as it is for the polling receivers of progressive mode)
    __shared__ int pos[2][FL_MAX_TOPK];
    __shared__ float w[2][FL_MAX_TOPK];
    __shared__ int n_shares[2];
    __shared__ int timed_out;
    // every load the block needs before its rows go out in ONE round: the verdicts, the token
    // count and (wave 1) the first token's positions and weights, which exist for every t < T
    const int plan_ok = W.plan_ok[s], gate_ok = gate ? gate[s] : 1, Ts = num_tokens[s];
    constexpr bool alone = WAITS == kWaitsItself;             // in place of a gate kernel
    const unsigned *ctr = W.arrive_comb + (size_t)s * N;
    verdict_word *word = verdict_of(W.done_comb, N, s);
    verdict_word ticket = 0;
    unsigned have = 0, want = 0;
    const int lane = tid & (kWave - 1);
    if (alone) {
        ticket = launch_ticket(W.epoch_route[s], launch);
        if (tid < N) { want = W.expect_comb[(size_t)s * N + tid]; have = ld_relaxed(ctr + tid); }
    }
    const bool fetcher = tid >= kWave && tid < 2 * kWave;     // wave 1
    const int k = tid - kWave;
    int pf_pos = -1;
    float pf_w = 1.0f;
    const int sent = PARTIAL && fetcher && k < N ? W.send_off[(size_t)s * (N + 1) + k] : 0;   // lane d: copies for lower ranks
    // token t's row positions (and weights): the load, then, once it has landed, the LDS copy
    auto fetch = [&](int t) {
        if (k >= K) { pf_pos = -1; return; }
        const size_t pair = ((size_t)s * D.T + t) * K + k;
        if (PARTIAL) pf_pos = W.send_to[pair];                // share rows: first k of each expert rank
        else { pf_pos = W.comb_pos[pair]; pf_w = weights[pair]; }
    };
    auto publish = [&](int buf) {
        if (PARTIAL) {                                        // compacted in k order, weight 1: an exact add
            const unsigned long long have = __ballot(pf_pos >= 0);
            const int first = __shfl(sent, pf_pos >= 0 ? pf_pos >> 24 : 0);
            if (pf_pos >= 0) {
                const int at = __popcll(have & ((1ull << k) - 1));
                pos[buf][at] = first + (pf_pos & 0xFFFFFF);
                w[buf][at] = 1.0f;
            }
            if (k == 0) n_shares[buf] = __popcll(have);
        } else if (k < K) {
            pos[buf][k] = pf_pos;
            w[buf][k] = pf_w;
        }
    };
    if (fetcher) fetch(t0);
    // in the default mode a rank without tokens waits for its (empty) replies all the same
    if (!plan_ok || !gate_ok || (t0 >= Ts && !(alone && blockIdx.x == 0))) return;
    if (tid == 0) timed_out = 0;               // wave 0 itself is the only one that may raise it
    if (fetcher) publish(0);
    // behind a gate kernel the counters were already seen complete, for every source of this rank
    if (!gate && tid < kWave) {
        if (alone) {                           // one verdict for all of the rank's workgroups
            if (!__all(lane >= N || arrived(have, want)) &&
                !wave_wait_together(ctr, have, want, N, D.spin_limit, word, ticket, blockIdx.x == 0, W.status) && tid == 0)
                timed_out = 1;
        } else if (!wave_wait_counters(ctr, W.expect_comb + (size_t)s * N, 0u, N, D.spin_limit)) {
            if (tid == 0) { timed_out = 1; latch_status(W.status, FL_STATUS_TIMEOUT); }
        }
        acquire_payload<WAITS != kBehindGate>();
    }
    __syncthreads();
    auto leave = [&](unsigned waves) {         // of the rank's workgroups that have a token, or of its first one
        const unsigned groups = max(1u, min(gridDim.x, (unsigned)(Ts * parts)));
        verdict_left(word, N, ticket, waves, groups * (blockDim.x / kWave));
    };
    if (timed_out) {
        if (alone && tid == 0) leave(blockDim.x / kWave);
        return;
    }
    verdict_word verdict = alone ? verdict_read(word) : 0;   // on its way while the rows are
    bool go = !alone;
    auto may_store = [&]() {
        if (!alone || go) return true;
        asm volatile("" : "+v"(verdict));      // looked at here and not where it is read
        go = verdict_allows(word, ticket, verdict);
        return go;
    };
    const char *recv = W.bufA + (size_t)s * D.bufA_rank_bytes;
    const int nvec_row = (int)(D.Bc / 16);
    const int per = whole_lines((nvec_row + parts - 1) / parts);   // this block's slice: [v0, nvec)
    const int v0 = part * per, nvec = min(v0 + per, nvec_row);
    const int kt = D.tune_reduce ? D.tune_reduce : K;
    // one token per block unless the grid was made smaller than the token count
    int cur = 0;
    for (int t = t0; t < Ts; t += t_step) {
        const int next = t + t_step;
        if (fetcher && next < Ts) fetch(next);                // in flight while the rows are summed
        v4u *o = (v4u *)(out + ((size_t)s * D.T + t) * D.Bc);
        if (PARTIAL) reduce_row_counted<OUT>(recv, pos[cur], w[cur], n_shares[cur], D.Sc, v0, nvec, o, tid, may_store);
        else if (kt >= 8) reduce_row<8, OUT>(recv, pos[cur], w[cur], K, D.Sc, v0, nvec, o, tid, may_store);
        else if (kt >= 4) reduce_row<4, OUT>(recv, pos[cur], w[cur], K, D.Sc, v0, nvec, o, tid, may_store);
        else if (kt >= 2) reduce_row<2, OUT>(recv, pos[cur], w[cur], K, D.Sc, v0, nvec, o, tid, may_store);
        else reduce_row<1, OUT>(recv, pos[cur], w[cur], K, D.Sc, v0, nvec, o, tid, may_store);
        if (next >= Ts) break;
        if (fetcher) publish(cur ^ 1);
        __syncthreads();                       // the other set is complete; this one may be rewritten
        cur ^= 1;
    }
    if (alone && !may_store() && lane == 0) leave(1u);
}

// ------------------------------------------------------------------ diagnostic copy
// Plain linear copy, fill and read: the machine's ceilings for a stream of 16-byte
// accesses, each in the launch shape that measured fastest for it on this part (1 GiB,
// non-temporal accesses).  Workgroups that move little and end at once do best:
//   copy  64 threads x 4 vectors (4 KB per workgroup) 6 450 GB/s of read + write traffic;
//         256 x 1: 6 340; 256 x 4 (16 KB): 5 930; 1024 x 4 (64 KB): 5 290
//   fill  256 x 1 (4 KB) 6 790 GB/s; 128 x 2: 6 490; 64 x 4: 6 320; 256 x 4 (16 KB): 6 000;
//         256 x 16 (64 KB): 4 940
//   read  flat at 7 000 - 7 100 GB/s from 2 KB to 32 KB per workgroup, 1024 x 1: 7 200 - 7 500
// THREADS threads take U vectors each, all loads before the stores.
template <int THREADS, int U>
__global__ __launch_bounds__(THREADS) void plain_copy_kernel(v4u *__restrict__ dst, const v4u *__restrict__ src,
                                                             size_t nvec) {
    const size_t base = (size_t)blockIdx.x * THREADS * U + threadIdx.x;
    v4u r[U];
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (base + (size_t)i * THREADS < nvec) r[i] = ld_stream(src + base + (size_t)i * THREADS);
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (base + (size_t)i * THREADS < nvec) st_stream(dst + base + (size_t)i * THREADS, r[i]);
}

// Write-only and read-only companions: the two one-directional ceilings, against which
// kernels that mostly write (dispatch pack) or mostly read (combine reduce) are judged.
template <int THREADS, int U>
__global__ __launch_bounds__(THREADS) void plain_fill_kernel(v4u *__restrict__ dst, size_t nvec, unsigned value) {
    const size_t base = (size_t)blockIdx.x * THREADS * U + threadIdx.x;
    const v4u v = {value, value, value, value};
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (base + (size_t)i * THREADS < nvec) st_stream(dst + base + (size_t)i * THREADS, v);
}

template <int THREADS, int U>
__global__ __launch_bounds__(THREADS) void plain_read_kernel(const v4u *__restrict__ src, size_t nvec,
                                                             unsigned *__restrict__ sink) {
    const size_t base = (size_t)blockIdx.x * THREADS * U + threadIdx.x;
    v4u r[U] = {};
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (base + (size_t)i * THREADS < nvec) r[i] = ld_stream(src + base + (size_t)i * THREADS);
    unsigned x = 0;
#pragma unroll
    for (int i = 0; i < U; ++i) x ^= r[i].x ^ r[i].y ^ r[i].z ^ r[i].w;
    if (x == 0x9E3779B9u) *sink = x;      // keeps the loads alive; practically never taken
}

}  // namespace flmoe
