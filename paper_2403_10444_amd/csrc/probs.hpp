// Verification with the distributions themselves as inputs (the ps / qs arrays of App. A): target rows
// hold p_i(x), draft rows q_i(x), used as given - no temperature, no normalisation sweep.  The weight
// w_i of Alg. 2 needs only the two gathered probabilities of each earlier drafted token, so every
// element is read from HBM exactly once and no workgroup waits for another on the way to its sums:
//
//   1. probs_residual_kernel  one workgroup per (sequence, position, chunk of kChunk tokens): the position's weight from
//                             the ratios r_1 .. r_i of the drafted tokens and the recursion w_i = min(w_{i-1} r_i, 1) (in
//                             double, in the log domain), by its first wave under the workgroup's loads; then the
//                             chunk's share of S_i = sum_x max(w_i p_i(x) - q_i(x), 0)
//                             (numerator of the block acceptance formula; for greedy block verification,
//                             Alg. 4, also the rejected mass sum_x max(q_i - w_i p_i, 0)); at the
//                             sequence's last position the chunk's share of sum_x p(x)
//   2. probs_finish           one workgroup per sequence: S_i, h_i, the accept tests of Alg. 1 / 2 / 4,
//                             then the inverse-CDF draw of Y (pick the chunk from the partial sums,
//                             re-read that one chunk)
// (Most calls over up to 2048 tokens have a kernel that keeps whole sequences in registers, packed.hpp; the others: packed_launch.)
// Calls whose workgroups all run at once have one launch: a sequence's last workgroup goes on with step 2.  Larger ones have a launch for it
// (probs_finish_kernel): there the waiting workgroups, and the registers of step 2 in all of them, cost more than the second launch
// (probs_at_once).  (In some calls the weights come from a kernel in front, probs_weights_kernel, one wave per sequence.)
// What bounds it: the bytes, then the second launch.  B = 64, gamma = 8, V = 128256, bf16: 42.2 us (6.6 TB/s) for the first
// kernel, 6.2 for the second, which took 10.7 while its threads read the chunk in stretches of 64 bytes each (uncoalesced)
// and scanned all of it, and 6.8 while a wave summed one position at a time and the chunk was picked behind a barrier of its own; now each wave reads a quarter of
// the chunk, and the one that holds the token draws from its registers.
#pragma once

#include "fused.hpp"

namespace sv {

// Target rows of at most half a chunk: up to how many each workgroup forms its position's weight (beyond: a kernel in front).  Each workgroup / in front, us, over 2049 ... 4096
// tokens: bf16 309 sequences of 6 over 2086 17.1 / 18.2, 1031 of 3 over 3418 27.5 / 27.5, 876 of 5 over 2263 27.9 / 27.5, 1989 of 3 over 2828 42.0 / 39.7; float32 221 of 9 over 2547
// 19.8 / 20.7, 824 of 4 over 3321 33.9 / 34.5, 561 of 8 over 2444 29.0 / 28.5, 1182 of 6 over 3163 51.4 / 50.2; own draft lengths 185 of 10 over 3158 15.1 / 16.4, 705 of 6 over 2353
// 22.6 / 23.3, 1007 of 8 over 2252 28.1 / 28.0 (1642 calls of 1000 to 11000 rows: the line is 0.7 % over the faster of the two on average, one at 2000 2.3 %).  Shorter rows come here
// from 6000 rows on only, where the kernel in front is the better one: float32 1064 of 10 over 1747 53.4 / 44.3, bf16 1105 of 8 over 1513 36.1 / 33.1.
constexpr int kProbsFormMax = 5000;
// Workgroups that run at once, or nearly, and what they read of the target rows: up to there forming the weights in every workgroup
// costs no more than a launch in front (Alg. 1; every workgroup / in front, gamma = 8: V = 128256: bf16 864 workgroups 13.2 / 14.2 us, 1152
// 14.4 / 14.3, 1440 15.3 / 14.9; float32 432 14.1 / 15.6, 576 15.1 / 14.7, 1152 20.1 / 16.6; V = 8192: bf16 1098 15.1 / 15.3, 1494 16.4 / 15.4; float32
// 693 17.0 / 16.9, 1098 21.3 / 18.2; gamma = 16, V = 500, float32: 816 12.3 / 14.7)
constexpr unsigned kProbsAtOnce = 1280;
constexpr size_t kProbsAtOnceBytes = 20u << 20;
// Calls of up to this many workgroups have one launch (`resident`: how many of that launch's run at once).  Two / one, us: bf16: B = 10, gamma = 4, V = 16000
// 10.9 / 9.5; B = 1, gamma = 8, V = 50257 11.4 / 10.3; B = 4, gamma = 4, V = 256000 (640 workgroups) 12.9 / 11.4; B = 25, gamma = 1, V = 128256 (800) 11.9 / 12.0;
// float32: B = 34, gamma = 4, V = 16000 16.0 / 14.1; B = 21, gamma = 4, V = 128256 (1680) 25.4 / 23.7.  Beyond: B = 64, gamma = 1, V = 128256,
// float32 (2048) 24.1 / 30.6, bf16, gamma = 16, B = 11, V = 128256 (2992) 23.9 / 22.9, gamma = 8, B = 64, V = 128256 (9216) 47.3 / 49.2.
// Unaligned bf16 rows, whose loads straddle lines, with long drafts less far: V = 109165, gamma = 14, 1050 workgroups 19.2 / 17.2, 1260 20.2 / 19.8, 1470
// 21.0 / 21.5; V = 30001, gamma = 8, 1296 21.1 / 20.4, 1512 21.6 / 22.4, 2016 24.7 / 24.8 (aligned, V = 109168, 1470 18.3 / 17.6; unaligned float32 26.9 / 26.1).
inline long long probs_at_once(long long resident, int gamma, bool f32, bool aligned)
{
    if (gamma < 4) return resident;
    return gamma >= 8 && !f32 && !aligned ? resident + resident / 4 : 2 * resident;
}
constexpr unsigned kProbsSixPerUnit = 26000;   // bytes of LDS of which a compute unit holds six, not seven
constexpr int kProbsKeepMax = 8192;      // chunk sums of one sequence that the workgroup that finishes it keeps in LDS (32 KB)

struct ProbWeight {
    double w;            // w_i (1 for token verification, whose residual is p - q)
    double one_minus_w;
    double h_token;      // min(r_i, 1), r_i the ratio of drafted token i judged with rows i-1; 1 at i = 0
    float w_hi, w_lo;    // w_i split into two floats
    int needed;          // whether the sums over rows i can matter (see probs_weights_kernel); where not, none are formed
};

// kVec consecutive probabilities of a row from the vector as loaded (load_raw); elements at or beyond V count as 0
template <typename T, bool ALIGNED>
__device__ __forceinline__ void unpack_probs(const uint4 &raw, int V, int idx, float *out)
{
    unpack_raw<T, ALIGNED>(raw, V, idx, out);
#pragma unroll
    for (int e = 0; e < ElemTraits<T>::kVec; ++e) out[e] = fmaxf(out[e], 0.f);
}

// w p - q with w = w_hi + w_lo (a double split into two floats): the products are exact inside the
// fused multiply-adds, so a small residual keeps its relative accuracy
__device__ __forceinline__ float prob_residual(float p, float q, float w_hi, float w_lo)
{
    return __builtin_fmaf(w_lo, p, __builtin_fmaf(w_hi, p, -q));
}

// A vector's part of a chunk's share of S_i (`last`: a sequence's last target row, q == 0) and, for Alg. 4, of the rejected mass.
template <bool GREEDY, int N>
__device__ __forceinline__ void add_residuals(const float (&xp)[N], const float (&xq)[N], bool last, float w_hi, float w_lo, float &acc, float &rej)
{
    if (last) {
#pragma unroll
        for (int e = 0; e < N; ++e) acc += xp[e];
        return;
    }
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const float d = prob_residual(xp[e], xq[e], w_hi, w_lo);
        acc += fmaxf(d, 0.f);
        if constexpr (GREEDY) rej += fmaxf(-d, 0.f);
    }
}

__device__ __forceinline__ int clamped_draft_len(const int32_t *draft_lens, int b, int gamma)
{
    if (!draft_lens) return gamma;
    const int g = draft_lens[b];
    return g < 1 ? 1 : g > gamma ? gamma : g;
}

template <int N> struct Lanes { static constexpr int value = N; };

// doubles of LDS in front of the kept sums: S_i and the rejected masses, the constants
__host__ __device__ inline int probs_finish_doubles(int gamma) { return (2 + (int)(sizeof(ProbWeight) / sizeof(double))) * (gamma + 1); }

constexpr ProbWeight kFirstWeight = {1.0, 0.0, 1.0, 1.f, 0.f, 1};      // position 0: w_0 = 1; tau = 0 draws from the residual of rows 0

// log2 r_i of a drafted token's two probabilities, and the powers below, by the series of double's full length: what is kept of a weight is 48 bits (prob_residual), of which the
// short ones that logits use would leave 41.  Error of the logarithm 1.8e-15 (most of it the last place of the result), of a power 1.2e-16 of it; the library's, which they are as
// exact as (logarithms of p and q apart: 3.1e-15), take a tenth of a microsecond more on the chain.  Kept finite downwards (a token outside the target's support: r = 0); infinite where only the draft rules the token out.
__device__ __forceinline__ double log2_ratio(float p, float q)
{
    const bool is_ratio = p > 0.f && p < INFINITY && q > 0.f && q < INFINITY;
    const double l = log2_precise<true, true>(is_ratio ? (double)p / (double)q : 1.0);
    return is_ratio ? fmax(l, kLog2RatioFloor) : p > 0.f && q >= 0.f && q < INFINITY ? (double)INFINITY : kLog2RatioFloor;
}

// Lane j of a segment of SEG = 16 or 64 lanes gets log2 w_{j+1} of w_i = min(w_{i-1} r_i, 1), w_0 = 1, from log2 r_{j+1}.  A stretch of positions takes w to min(a w, c): two
// neighbouring ones to min(a' a w, min(a c', c)), logarithms here.  As against a difference of prefix sums, what a large ratio added is gone where the min is taken, so that a
// weight behind it is as exact as any (a ratio of infinity leaves no infinity: it is c = 1).  Lanes without a source get the zeros of a stretch that does nothing to a weight of at most 1.
template <int CTRL, int ROW_MASK = 0xf> __device__ __forceinline__ void join_stretches(double &a, double &c)
{
    const double a_before = dpp_shift_double<CTRL, ROW_MASK>(a), c_before = dpp_shift_double<CTRL, ROW_MASK>(c);
    c = fmin(c_before + a, c);
    a += a_before;
}
template <int SEG> __device__ __forceinline__ double clamped_weights(double log2r)
{
    double a = log2r, c = 0.0;
    join_stretches<0x111>(a, c);
    join_stretches<0x112>(a, c);
    join_stretches<0x114>(a, c);
    join_stretches<0x118>(a, c);
    if constexpr (SEG == kWave) {
        join_stretches<0x142, 0xa>(a, c);
        join_stretches<0x143, 0xc>(a, c);
    }
    return fmin(a, c);
}

// w_0 = 1, w_i = min(w_{i-1} r_i, 1) (Alg. 2; Alg. 4 omits the min), r_i = p_{i-1}(X_i) / q_{i-1}(X_i), for positions
// 1 .. n of a sequence of draft length gb, by one wave: lane j comes with drafted token j + 1 (and its uniform), gathers its
// two probabilities, and gets position j + 1's constants by a scan over the log2 r (products of ratios neither overflow nor lose
// 1 - w_i next to 1).  `for_tests`: whether one_minus_w and h_token are wanted, which only the workgroup that finishes the sequence reads.
// What bounds it: one wave's chain of operations in double, which every workgroup of a position waits for: one logarithm of the ratio instead of two, a scan
// over the lanes instead of a loop over the positions, and one power: calls that do not fill the device for long are 5 to 10 % faster (us a call, before / now, with
// the changes of the finish: bf16: 204 of 10 over 8718 30.3 / 27.8, 117 ragged of 13 over 11200 18.8 / 17.3, 400 of 8 over 50257 118 / 111.7; float32: 143 ragged of 15
// over 16146 42.4 / 39.6, 6 of 15 over 18438 14.0 / 12.5; with short series 27.7, 17.1, 111.5, 39.6, 12.5).
template <typename T>
__device__ __forceinline__ ProbWeight form_weights(const T *target_seq, const T *draft_seq, size_t tstride, size_t dstride, int tok, float eta,
                                                   int n, int gb, int algo, bool every_sum, bool for_tests)
{
    const int lane = threadIdx.x & 63, i = lane + 1;
    double log2r = 0.0;
    if (lane < n) log2r = log2_ratio(logit_as_float(target_seq + (size_t)lane * tstride + tok), logit_as_float(draft_seq + (size_t)lane * dstride + tok));
    const double log2w = algo == kBlock ? clamped_weights<kWave>(log2r) : algo == kGreedy ? wave_scan(log2r) : 0.0;
    ProbWeight pw;
    pw.w = log2w < 2000.0 ? exp2_precise<true, true>(log2w) : (double)INFINITY;
    pw.w_hi = (float)pw.w;
    pw.w_lo = (float)(pw.w - (double)pw.w_hi);
    pw.one_minus_w = 0.0;
    pw.h_token = 1.0;
    if (algo == kToken) pw.h_token = exp2_precise<true, true>(fmin(log2r, 0.0));
    else if (for_tests && algo == kBlock) pw.one_minus_w = one_minus_exp2<true, true>(log2w);
    // Which sums can matter (exact, whatever the rows sum to).  Alg. 1 stops at the first failed test, so only a
    // position that every earlier test let through can become tau; the last target row is summed (and drawn
    // from) only if tau = gamma: every test passed (Alg. 1), or the last one did (Alg. 2 / 4: eta < w_gamma).
    // The tests are evaluated with the expressions the finishing kernel uses, on the same stored values.
    const unsigned long long failed = __ballot(i <= n && !((double)eta < pw.h_token));
    const bool prefix_pass = (failed & ((2ull << lane) - 1ull)) == 0;     // tests 1 .. i
    if (every_sum) pw.needed = 1;
    else if (algo == kToken) pw.needed = prefix_pass ? 1 : 0;
    else pw.needed = (i < gb || (double)eta < fmin(pw.w, 1.0)) ? 1 : 0;
    return pw;
}

// One wave per sequence: the constants of all its positions.
template <typename T>
__global__ __launch_bounds__(64) void probs_weights_kernel(
    const T *__restrict__ target, const T *__restrict__ draft, size_t tstride, size_t dstride,
    const int32_t *__restrict__ tokens, const int32_t *__restrict__ draft_lens, int gamma, int algo,
    ProbWeight *__restrict__ weights, const float *__restrict__ uniforms, int every_sum)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    const int gb = clamped_draft_len(draft_lens, b, gamma);
    const int tok = lane < gb ? tokens[(size_t)b * gamma + lane] : 0;
    const float eta = lane < gb ? uniforms[(size_t)b * (gamma + 1) + lane] : 1.f;
    const ProbWeight pw = form_weights(target + (size_t)b * (gamma + 1) * tstride, draft + (size_t)b * gamma * dstride, tstride, dstride,
                                       tok, eta, gb, gb, algo, every_sum != 0, true);
    ProbWeight *wb = weights + (size_t)b * (gamma + 1);
    if (lane == 0) wb[0] = kFirstWeight;
    if (lane < gb) wb[lane + 1] = pw;
}

struct ProbsParams {
    const void *target, *draft;
    size_t tstride, dstride;
    const int32_t *tokens, *draft_lens;
    const float *uniforms;
    int gamma, V, nchunks, algo, every_sum, keep;      // keep: whether a sequence's chunk sums fit the launch's LDS
    int spin_limit;
    u64 call;                     // calls of one launch: this call's number (see ShareWords)
    // a chunk's shares of S_i and of the rejected mass (Alg. 4).  Calls of more launches: `part`, [B, gamma + 1, nchunks], both in one word.
    // Calls of one: `part`, [B, gamma, nchunks, 2], of the row pairs, `part_last` and `check_last`, [B, nchunks], of a sequence's last target row
    u64 *part, *part_last;
    unsigned *check_last;
    ProbWeight *weights;          // [B, gamma + 1], calls of more launches than one
    int32_t *accept_len, *next_token;
    float *debug_out;
};

// ------------------------------------------------------------------ calls of one launch: how the shares reach the workgroup that finishes a sequence
// That is its last one, which waits for the words of the others (all of them started before it); where a wait runs out (another kernel holds the
// compute units for seconds) it forms the missing shares itself, in the same order.  The memory is not prepared: it holds whatever
// other kernels, other calls or other tensors left there.  So a chunk's shares count where 64 bits beside them are this call's number, which
// no call before it had: two words of 32 bits of it and one share each, every half of the number combined with the OTHER word's share.  A pair
// of one old word and a new one is then taken only where the old word's share is the new one; a pair of two old words where all 64 bits meet by chance.
// (The last target row's chunks have one share: a word, and a check of 32 bits.)  Counted arrivals instead of a wait, found by a count per
// sequence, were slower: read-modify-writes of one line by workgroups all over the device take 40 ns each, one after the other.
__device__ __forceinline__ void leave_shares(u64 *words, u64 call, float acc, float rej)
{
    const unsigned a = __float_as_uint(acc), r = __float_as_uint(rej);
    st_u64(words, (u64)((unsigned)(call >> 32) ^ r) << 32 | a);
    st_u64(words + 1, (u64)((unsigned)call ^ a) << 32 | r);
}
constexpr float kMissingShare = -1.f;                     // (shares are sums of what is not negative)
__device__ __forceinline__ float2 await_shares(const u64 *words, u64 call, int limit, bool &gave_up)
{
    for (int spins = 0;;) {
        const u64 v = ld_u64(words), w = ld_u64(words + 1);
        const unsigned a = (unsigned)v, r = (unsigned)w;
        if (((unsigned)(v >> 32) ^ r) == (unsigned)(call >> 32) && ((unsigned)(w >> 32) ^ a) == (unsigned)call) return make_float2(__uint_as_float(a), __uint_as_float(r));
        if (++spins > limit) { gave_up = true; return make_float2(kMissingShare, 0.f); }
        __builtin_amdgcn_s_sleep(1);
    }
}
__device__ __forceinline__ void leave_last_share(u64 *word, unsigned *check, u64 call, float acc)
{
    st_u64(word, (call >> 32) << 32 | __float_as_uint(acc));
    st_u32(check, (unsigned)call ^ __float_as_uint(acc));
}
__device__ __forceinline__ float await_last_share(const u64 *word, const unsigned *check, u64 call, int limit, bool &gave_up)
{
    for (int spins = 0;;) {
        const u64 v = ld_u64(word);
        const unsigned c = ld_u32(check);
        if (v >> 32 == call >> 32 && (c ^ (unsigned)v) == (unsigned)call) return __uint_as_float((unsigned)v);
        if (++spins > limit) { gave_up = true; return kMissingShare; }
        __builtin_amdgcn_s_sleep(1);
    }
}

template <typename T, bool ALIGNED, bool GREEDY, bool ONE>
__device__ __forceinline__ void probs_finish(const ProbsParams &P, int b, int gb, const ProbWeight &mine);

// A position's share: one workgroup per (sequence, position, chunk).  FORM: the workgroup forms its position's weight itself, under its
// loads.  (Without: it comes from probs_weights_kernel.)  ONE: the last workgroup of a sequence goes on with probs_finish; else a
// sequence's chunk-0 workgroups leave the weights for the kernel that finishes it.
template <typename T, bool ALIGNED, bool GREEDY, bool FORM, bool ONE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ONE ? 4 : 1))) void probs_residual_kernel(const ProbsParams P)
{
    constexpr int kVec = ElemTraits<T>::kVec;
    constexpr int kU = kChunk / (kThreads * kVec);
    __shared__ float lds[kWaves];
    __shared__ ProbWeight formed;
    const int gamma = P.gamma, V = P.V, nchunks = P.nchunks, algo = P.algo, every_sum = P.every_sum;
    const size_t tstride = P.tstride, dstride = P.dstride;
    const int pr = blockIdx.x / nchunks, c = blockIdx.x - pr * nchunks, tid = threadIdx.x;
    const int b = pr / (gamma + 1), i = pr - b * (gamma + 1);
    const int gb = clamped_draft_len(P.draft_lens, b, gamma);
    if (i > gb) return;                                          // a position this sequence does not use
    const T *target_seq = static_cast<const T *>(P.target) + (size_t)b * (gamma + 1) * tstride;
    const T *draft_seq = static_cast<const T *>(P.draft) + (size_t)b * gamma * dstride;
    const T *prow = target_seq + (size_t)i * tstride;
    const bool last = i == gb;                                   // no draft row: q == 0
    const T *qrow = draft_seq + (size_t)(last ? 0 : i) * dstride;
    ProbWeight mine;                                             // ONE, the last target row, first wave: lane j, position j + 1's

    uint4 rp[kU], rq[kU];
    const int in_row = V - c * kChunk;                           // (short rows: vectors beyond the row are left out, for the whole workgroup)
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (u * kThreads * kVec >= in_row) continue;
            const int idx = c * kChunk + (u * kThreads + tid) * kVec;
            rp[u] = load_raw<T, ALIGNED, true>(prow, V, idx);
            if (!last) rq[u] = load_raw<T, ALIGNED, true>(qrow, V, idx);
        }
    };
    bool wanted = true;                                          // (else: sums that cannot matter, for the whole workgroup)
    if constexpr (FORM) {
        // (the drafted tokens are asked for in front of the rows, so that their probabilities follow under the rows' loads;
        // a last target row, which is needed only where the last test passes, waits for its weight)
        const bool at_once = !last || every_sum;
        const bool forms = tid < kWave && i > 0;
        int tok = 0;
        float eta = 1.f;
        if (forms && tid < i) { tok = P.tokens[(size_t)b * gamma + tid]; eta = P.uniforms[(size_t)b * (gamma + 1) + tid]; }
        if (at_once) load();
        if (forms) {
            const ProbWeight pw = form_weights(target_seq, draft_seq, tstride, dstride, tok, eta, i, gb, algo, every_sum != 0, ONE ? last && c == nchunks - 1 : c == 0);
            if (tid == i - 1) { formed = pw; if (!ONE && c == 0) P.weights[pr] = pw; }
            if constexpr (ONE) mine = pw;
        } else if (tid == 0) {
            formed = kFirstWeight;
            if (!ONE && c == 0) P.weights[pr] = kFirstWeight;
        }
        __syncthreads();
        wanted = formed.needed != 0;
        if (wanted && !at_once) load();
    } else {
        wanted = P.weights[pr].needed != 0;
        if (wanted) load();
    }
    if (wanted) {
        const float w_hi = FORM ? formed.w_hi : P.weights[pr].w_hi, w_lo = FORM ? formed.w_lo : P.weights[pr].w_lo;
        float acc = 0.f, rej = 0.f;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (u * kThreads * kVec >= in_row) continue;
            const int idx = c * kChunk + (u * kThreads + tid) * kVec;
            float xp[kVec], xq[kVec];
            unpack_probs<T, ALIGNED>(rp[u], V, idx, xp);
            // (one question per vector: float32, 34 sequences of 4 over 16000 tokens 14.0 -> 13.9 us)
            if (last) {
                add_residuals<GREEDY>(xp, xp, true, w_hi, w_lo, acc, rej);
            } else {
                unpack_probs<T, ALIGNED>(rq[u], V, idx, xq);
                add_residuals<GREEDY>(xp, xq, false, w_hi, w_lo, acc, rej);
            }
        }
        acc = block_sum(acc, lds);
        if constexpr (GREEDY) rej = block_sum(rej, lds);
        if (tid == 0) {
            const size_t last_word = (size_t)b * nchunks + c;
            if constexpr (!ONE) P.part[(size_t)pr * nchunks + c] = pack_stat(acc, rej);
            else if (last) leave_last_share(P.part_last + last_word, P.check_last + last_word, P.call, acc);
            else leave_shares(P.part + 2 * (((size_t)b * gamma + i) * nchunks + c), P.call, acc, rej);
        }
    }
    if constexpr (ONE) {
        if (last && c == nchunks - 1) probs_finish<T, ALIGNED, GREEDY, true>(P, b, gb, mine);
    }
}
// One workgroup per sequence, after probs_residual_kernel.  Four waves per SIMD, so that 1024 sequences are finished at once instead of 768 (aligned float32, 1000
// sequences of 12 over 10728 tokens, Alg. 1: 59.3 -> 56.7 us the whole call); unaligned float32 rows would spill (this kernel, sequences of 12 over 10727, three
// waves / four: 1000 19.5 / 18.8 us, 500 11.9 / 12.9).
template <typename T, bool ALIGNED, bool GREEDY>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ElemTraits<T>::kVec == 8 || ALIGNED ? 4 : 3))) void probs_finish_kernel(const ProbsParams P)
{
    const int b = blockIdx.x, tid = threadIdx.x, gb = clamped_draft_len(P.draft_lens, b, P.gamma);
    ProbWeight pw = kFirstWeight;
    if (tid < gb) pw = P.weights[(size_t)b * (P.gamma + 1) + tid + 1];
    probs_finish<T, ALIGNED, GREEDY, false>(P, b, gb, pw);
}

// The weights of a wave's kWaveChunk consecutive tokens of a row pair from `start` on, in its registers: element
// v * kVec + e of a lane is token start + (v * 64 + lane) * kVec + e (every load instruction covers 1 KB).
template <typename T, bool ALIGNED>
__device__ __forceinline__ void prob_wave_weights(const T *prow, const T *qrow, int V, int start, bool residual,
                                                  float w_hi, float w_lo, float (&wgt)[kPerThread])
{
    constexpr int kVec = ElemTraits<T>::kVec, kNV = kPerThread / kVec;
    const int first = start + (int)(threadIdx.x & 63) * kVec;
    uint4 rp[kNV], rq[kNV];
    if (!ALIGNED && V < kVec) {
        // (asked once instead of at each of the loads: unaligned float32 rows, 1000 sequences of 12 over 10727 tokens, this kernel 23.7 -> 19.4 us)
        const uint4 p = load_short_row(prow, V), q = load_short_row(qrow, V);
#pragma unroll
        for (int v = 0; v < kNV; ++v) { rp[v] = p; rq[v] = q; }
    } else {
#pragma unroll
        for (int v = 0; v < kNV; ++v) {
            rp[v] = load_raw<T, ALIGNED, false>(prow, V, first + v * kWave * kVec);
            if (residual) rq[v] = load_raw<T, ALIGNED, false>(qrow, V, first + v * kWave * kVec);
        }
    }
#pragma unroll
    for (int v = 0; v < kNV; ++v) {
        float xp[kVec], xq[kVec];
        unpack_probs<T, ALIGNED>(rp[v], V, first + v * kWave * kVec, xp);
        if (residual) unpack_probs<T, ALIGNED>(rq[v], V, first + v * kWave * kVec, xq);
#pragma unroll
        for (int e = 0; e < kVec; ++e) wgt[v * kVec + e] = residual ? fmaxf(prob_residual(xp[e], xq[e], w_hi, w_lo), 0.f) : xp[e];
    }
}

// S_i, h_i, the accept tests and the draw of Y of a sequence, by one workgroup (`mine`: first wave, lane j: position j + 1's constants).
template <typename T, bool ALIGNED, bool GREEDY, bool ONE>
__device__ __forceinline__ void probs_finish(const ProbsParams &P, int b, int gb, const ProbWeight &mine)
{
    extern __shared__ double smd[];                     // [gamma+1] S_i, [gamma+1] rejected mass, the constants, then the kept partial sums
    __shared__ double wave_tot[kWaves];
    __shared__ int s_tau, s_chunk, s_mode, s_gave_up;
    __shared__ double s_t, s_total;
    const int gamma = P.gamma, V = P.V, nchunks = P.nchunks, algo = P.algo;
    const size_t tstride = P.tstride, dstride = P.dstride;
    const T *const target = static_cast<const T *>(P.target), *const draft = static_cast<const T *>(P.draft);
    int32_t *const accept_len = P.accept_len, *const next_token = P.next_token;
    float *const debug_out = P.debug_out;
    double *S = smd, *R = smd + (gamma + 1);
    ProbWeight *const wb = reinterpret_cast<ProbWeight *>(smd + 2 * (gamma + 1));          // the sequence's constants, read once
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u64 *const pb = P.part + (size_t)b * (ONE ? 2 * gamma : gamma + 1) * nchunks;
    const float *eta = P.uniforms + (size_t)b * (gamma + 1);
    // the chunk sums stay in LDS for the draw when they fit (the host sizes the dynamic LDS to match: one float per
    // sum, a second one per chunk for Alg. 4's rejected mass)
    const bool keep = ONE || P.keep != 0;               // (calls of one launch have no more sums than that)
    float *kept = reinterpret_cast<float *>(smd + probs_finish_doubles(gamma));
    float *kept_rej = kept + (gamma + 1) * nchunks;

    float eta_i = 0.f, u = 0.f;
    ProbWeight pw = mine;
    auto constants = [&]() {
        if (wave != 0) return;
        if (lane + 1 <= gb) { eta_i = eta[lane]; wb[lane + 1] = pw; }
        if (lane == 0) { wb[0] = kFirstWeight; s_gave_up = 0; }
        u = eta[gb];
    };
    // every chunk sum (ONE: of the positions that have any; else all are read, stale ones of the others among them, which are
    // never used: one trip to memory for the sums and the constants)
    bool gave_up = false;
    const int n_words = (gb + 1) * nchunks;
    if (ONE) { constants(); __syncthreads(); }
    if (keep) {
        for (int w = tid; w < n_words; w += kThreads) {
            const int i = w / nchunks;
            float2 v = make_float2(0.f, 0.f);
            if constexpr (!ONE) {
                const u64 word = pb[w];
                v = make_float2(stat_shift(word), stat_sum(word));
            } else if (wb[i].needed) {
                const size_t last_word = (size_t)b * nchunks + (w - i * nchunks);
                if (i == gb) v.x = await_last_share(P.part_last + last_word, P.check_last + last_word, P.call, P.spin_limit, gave_up);
                else v = await_shares(pb + 2 * w, P.call, P.spin_limit, gave_up);
            }
            kept[w] = v.x;
            if constexpr (GREEDY) kept_rej[w] = v.y;
        }
    }
    if (!ONE) constants();
    if (ONE && gave_up) s_gave_up = 1;
    __syncthreads();
    if (ONE && __builtin_expect(s_gave_up != 0, 0)) {
        constexpr int kVec = ElemTraits<T>::kVec;
        __shared__ float sums[kWaves];
        for (int w = 0; w < n_words; ++w) {
            if (kept[w] != kMissingShare) continue;              // (the same for the whole workgroup)
            const int i = w / nchunks, start = (w - i * nchunks) * kChunk;
            const T *const prow = target + ((size_t)b * (gamma + 1) + i) * tstride, *const qrow = draft + ((size_t)b * gamma + (i < gb ? i : 0)) * dstride;
            float acc = 0.f, rej = 0.f;
#pragma unroll 1
            for (int at = 0; at < kChunk && start + at < V; at += kThreads * kVec) {
                const int idx = start + at + tid * kVec;
                float xp[kVec], xq[kVec];
                unpack_probs<T, ALIGNED>(load_raw<T, ALIGNED, true>(prow, V, idx), V, idx, xp);
                unpack_probs<T, ALIGNED>(load_raw<T, ALIGNED, true>(qrow, V, idx), V, idx, xq);
                add_residuals<GREEDY>(xp, xq, i == gb, wb[i].w_hi, wb[i].w_lo, acc, rej);
            }
            acc = block_sum(acc, sums);
            if constexpr (GREEDY) rej = block_sum(rej, sums);
            if (tid == 0) { kept[w] = acc; if constexpr (GREEDY) kept_rej[w] = rej; }
        }
        __syncthreads();
    }

    // S_i = sum over the chunks, lanes stride over them: sixteen lanes for a position where that is all of its chunks (four positions to a wave: the same
    // sums in the same order), else a wave.  (Rows whose sums were not formed: S stays 0, their tests are decided without it and they cannot become tau)
    auto form_sums = [&](auto segment) {
        constexpr int G = decltype(segment)::value;
        const int e = lane & (G - 1);
        for (int i = tid / G; i <= gb; i += kThreads / G) {
            double acc = 0.0, rej = 0.0;
            if (wb[i].needed) for (int c = e; c < nchunks; c += G) {
                if (keep) {
                    acc += (double)kept[i * nchunks + c];
                    if (GREEDY) rej += (double)kept_rej[i * nchunks + c];
                } else {
                    const u64 v = pb[(size_t)i * nchunks + c];
                    acc += (double)stat_shift(v); rej += (double)stat_sum(v);
                }
            }
            acc = group_sum<G>(acc);
            if (GREEDY) rej = group_sum<G>(rej);
            if (e == 0) { S[i] = acc; R[i] = rej; }
        }
    };
    if (nchunks <= 16) form_sums(Lanes<16>{});
    else form_sums(Lanes<kWave>{});
    __syncthreads();

    if (wave == 0) {
        // accept tests eta_i < h_i: lane l judges position l + 1 (positions 1 .. gb <= 64)
        const int i = lane + 1;
        bool pass = false;
        if (i <= gb) {
            double h;
            if (algo == kToken) h = pw.h_token;                                         // min(r_i, 1)
            else if (i == gb) h = fmin(pw.w, 1.0);                                      // h_gamma = w_gamma
            else if (algo == kGreedy) h = R[i] > 0.0 ? fmin(S[i] / R[i], 1.0) : 1.0;    // p_remain / p_rej
            else h = pw.w >= 1.0 ? 1.0 : S[i] / (S[i] + pw.one_minus_w);                // block acceptance formula
            pass = (double)eta_i < h;
            if (debug_out) {
                float *d = debug_out + ((size_t)b * (gamma + 1) + i) * 3;
                // q == 0 at the last position: the residual mass there is w times the row's own sum
                d[0] = (float)pw.w; d[1] = (float)(i == gb ? (algo == kBlock ? pw.w : pw.w * S[gb]) : S[i]); d[2] = (float)h;
            }
        }
        const unsigned long long passed = __ballot(pass);                               // bit l: position l + 1
        // token verification stops at the first failure; block / greedy keep the last passing sub-block
        const int tau = algo == kToken ? (~passed ? __ffsll((long long)~passed) - 1 : 64)
                                       : (passed ? 64 - __clzll((long long)passed) : 0);
        // weights of the draw: the residual of row tau, or p_tau when everything was accepted (its chunk
        // sums are then the partial sums of the last position) or when no residual mass is left at all
        const int mode = tau == gb ? 1 : S[tau] > 0.0 ? 0 : 2;
        if (lane == 0) {
            if (debug_out) {
                float *d = debug_out + (size_t)b * (gamma + 1) * 3;
                d[0] = 1.f; d[1] = (float)S[0]; d[2] = 1.f;
            }
            accept_len[b] = tau;
            s_tau = tau;
            s_mode = mode;
        }
        if (mode != 2) {
            // pick the chunk of row tau that holds t = u * (total weight): 64 chunk sums at a time, scanned in order
            const double total = mode == 1 ? S[gb] : S[tau];
            const double t = (double)u * total;
            const u64 *pp = pb + (size_t)tau * nchunks;
            int chunk = -1, last_nonzero = 0;
            double carry = 0.0, t_in = INFINITY;
            for (int c0 = 0; c0 < nchunks && chunk < 0; c0 += 64) {
                const int c = c0 + lane;
                const double v = c < nchunks ? (double)(keep ? kept[tau * nchunks + c] : stat_shift(pp[c])) : 0.0;
                const double inc = wave_scan(v) + carry;
                const unsigned long long nz = __ballot(v > 0.0), hit = __ballot(c < nchunks && inc > t);
                if (nz) last_nonzero = c0 + 63 - __clzll((long long)nz);
                if (hit) {
                    const int first = __ffsll((long long)hit) - 1;
                    chunk = c0 + first;
                    t_in = t - read_lane_double(inc - v, first);
                }
                carry = read_lane_double(inc, 63);
            }
            if (lane == 0) {
                s_chunk = chunk < 0 ? last_nonzero : chunk;      // rounding pushed t past the end: the last chunk with weight
                s_t = t_in;
            }
        }
    }
    __syncthreads();
    const int tau = s_tau, mode = s_mode;
    const bool residual = mode == 0;
    const T *prow = target + ((size_t)b * (gamma + 1) + tau) * tstride;
    const T *qrow = draft + ((size_t)b * gamma + (tau < gb ? tau : 0)) * dstride;
    float w_hi = 1.f, w_lo = 0.f;
    if (residual) { w_hi = wb[tau].w_hi; w_lo = wb[tau].w_lo; }
    float wgt[kPerThread];

    // the workgroup's chunk c, a quarter per wave: the sum of the waves before the thread's own, the chunk's
    auto sum_chunk = [&](int c, double &before, double &total) {
        prob_wave_weights<T, ALIGNED>(prow, qrow, V, c * kChunk + wave * kWaveChunk, residual, w_hi, w_lo, wgt);
        double sum = 0.0;
#pragma unroll
        for (int e = 0; e < kPerThread; ++e) sum += (double)wgt[e];
        sum = group_sum<kWave>(sum);
        __syncthreads();
        if (lane == 0) wave_tot[wave] = sum;
        __syncthreads();
        before = total = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { if (w < wave) before += wave_tot[w]; total += wave_tot[w]; }
    };

    if (mode == 2) {
        // chunk sums of p_tau were never formed for this row: form the row total here (rare: rounding ate a residual)
        double row_total = 0.0;
        for (int c = 0; c < nchunks; ++c) {
            double before, total;
            sum_chunk(c, before, total);
            row_total += total;
        }
        if (tid == 0) s_total = (double)u * row_total;
        __syncthreads();
    }

    // walk: the chosen chunk, or (mode 2) every chunk in turn until the one whose running sum passes t.
    // Inside that chunk the token lies with the first wave whose running sum exceeds t, which then draws it from its
    // registers; where rounding left t at or beyond the chunk's own total, with the last wave that has weight, and
    // there it is the last token with weight (token 0 of the chunk if nothing has any).
    int c = mode == 2 ? 0 : s_chunk;
    double t_in = mode == 2 ? s_total : s_t;
    double before, total;
    for (int last_c = -1;;) {
        sum_chunk(c, before, total);
        if (mode != 2 || t_in < total) break;
        if (total > 0.0) last_c = c;
        if (c + 1 >= nchunks) {
            // rounding left t beyond the row's total: the last token with weight
            if (last_c >= 0 && last_c != c) { c = last_c; sum_chunk(c, before, total); }
            t_in = INFINITY;
            break;
        }
        t_in -= total;
        ++c;
    }
    int holder = -1, last_weight = 0;
    {
        double running = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (wave_tot[w] > 0.0) last_weight = w;
            running += wave_tot[w];
            if (holder < 0 && running > t_in) holder = w;
        }
    }
    if (wave != (holder < 0 ? last_weight : holder)) return;
    const double t = holder < 0 ? INFINITY : t_in - before;
    const int offset = draw_in_group<kWave, kPerThread / ElemTraits<T>::kVec, ElemTraits<T>::kVec>(
        [&](int j) { return wgt[j]; }, kPerThread / ElemTraits<T>::kVec, [&](double) { return t; });
    if (lane == 0) next_token[b] = c * kChunk + wave * kWaveChunk + offset;
}

}  // namespace sv
