// Calls whose workgroups all run at once, or nearly (rows of at most 32 workgroups).
//
// Such a call is over when its chain of dependent steps is: words that travel between workgroups through device memory (0.7 - 0.9 us a trip
// while all of them poll) and, between them, the arithmetic of single waves (3 ns per dependent instruction, 9 per step of a scan
// in double).  In the kernel for calls of few resident sets (resident.hpp) the chain has four trips: the row's words, the ratio that
// the row's leader makes of them, the shares of S_i, the drawn token.  Here the second is gone: every workgroup reads the
// words of its own row AND of all earlier ones - its four waves share the rows, a wave takes several side by side in segments of
// its lanes - and forms all their ratios itself, with the same arithmetic on the same words, so that all of them agree.  The price is
// more to read for every workgroup (about 1 KB where its logits are 32 KB) and more registers (four waves per SIMD), which is why
// most bf16 calls of more than one resident set stay with the other kernel (runs_together).  What else is different: the words exist in
// three copies, every wave forms the row constants for itself, the running sums that a draw needs are ready before it is known
// where the token lies, positions that another one rules out are left out on the ratios alone, and the last target row's
// leader asks only for the positions that can matter.
// Measured, the other kernel / this one: bf16, B = 1, gamma = 8, V = 128256 10.9 / 9.3 us; B = 24, gamma = 4, V = 50257 14.6 / 12.7;
// float32, B = 8, gamma = 8, V = 32000 11.5 / 9.9; 115 calls of at most one resident set: 1.08 times as fast on average.  What is left at B = 1: words at 3.3 us
// after the first workgroup's start (loads 1.7, sweeps 0.7, start and skew 0.9), ratios and weights 5.1, second sweep 5.7, shares 7.0, place 7.4, token and outputs 9.
#pragma once

#include "resident.hpp"

namespace sv {

// ------------------------------------------------------------------ segments of a wave
// A wave works on several rows at once, four lanes for each or sixteen (reductions over a segment: group_max, group_sum).
// Inclusive scans over the first n lanes (the others hold 0; up to 16 they lie in one DPP row: four steps instead of six).
__device__ __forceinline__ double scan_of(double v, int n)
{
    v += dpp_shift_double<0x111>(v);
    v += dpp_shift_double<0x112>(v);
    v += dpp_shift_double<0x114>(v);
    v += dpp_shift_double<0x118>(v);
    if (n > 16) {
        v += dpp_shift_double<0x142, 0xa>(v);
        v += dpp_shift_double<0x143, 0xc>(v);
    }
    return v;
}
__device__ __forceinline__ double scan_max0_of(double v, int n)
{
    v = fmax(v, 0.0);
    v = fmax(v, dpp_shift_double<0x111>(v));
    v = fmax(v, dpp_shift_double<0x112>(v));
    v = fmax(v, dpp_shift_double<0x114>(v));
    v = fmax(v, dpp_shift_double<0x118>(v));
    if (n > 16) {
        v = fmax(v, dpp_shift_double<0x142, 0xa>(v));
        v = fmax(v, dpp_shift_double<0x143, 0xc>(v));
    }
    return v;
}

// ------------------------------------------------------------------ the words of a row, several times over
// Every workgroup of a sequence reads the words of its row and of all earlier ones, and a line that many workgroups poll takes
// a write only slowly (eight words of one line written while 128 workgroups poll it: the last one sees them after 1.1 us, 0.6
// with four copies of the line, 0.57 with sixteen).  So a row's words exist kWordCopies times and a workgroup polls the
// copy of its column: copy 0 where the large kernel has its words, copies 1 and 2 in the area of the words per wave chunk,
// which this kernel has no other use for.  (The shares of S_i likewise, side by side in the area of the shares per wave chunk.)
constexpr int kWordCopies = 3;
static_assert((kWordCopies - 1) * 2 <= kWaves && kWordCopies <= kWaves, "two more copies of the pairs fit the words per wave chunk, the shares' copies theirs");
// copy `copy` of the pairs (target word, draft word) of row `drow`
__device__ __forceinline__ u64 *row_pairs(const Words &W, size_t drow, int nwg, int copy)
{
    return copy == 0 ? W.pgrp + 2 * drow * nwg : W.pstat + (drow * 2 + (copy - 1)) * 2 * nwg;
}

// The rows of a sequence are dealt out over a workgroup's lanes in segments, one row each; a kernel's FORM is made for rows of so
// many workgroups: 0: at most 4, segments of 4 lanes; 1: at most 16, segments of 16; 2: at most 32, segments of 16, lane e takes the
// words of the workgroups e and e + 16.
template <int FORM> constexpr int kSegment = FORM == 0 ? 4 : 16;
template <int FORM> constexpr int kWaveRows = kWave / kSegment<FORM>;

// What the waves work out of the words of these rows, for the whole workgroup.
struct RowsOut {
    double lr[SV_MAX_GAMMA];       // log2 r_{j+1} of the rows 0 .. n - 1
    double L[2];                   // L_p, L_q of row `own`
    int gave_up[kWaves];
};

// The logit of row `row`'s drafted token `tok`: the target row's in even lanes, the draft row's in odd ones.
template <typename T>
__device__ __forceinline__ uint32_t token_logit(const FusedParams &P, size_t seq_d, size_t seq_u, int row, int tok)
{
    const bool q = (threadIdx.x & 1) != 0;
    const T *const p = static_cast<const T *>(q ? P.draft : P.target);
    return logit_bits(p + ((q ? seq_d : seq_u) + row) * (q ? P.dstride : P.tstride) + tok);
}

// Rows 0 .. n - 1, by the workgroup's four waves: waits for their words, forms the normalisers and the ratios log2 r_{j+1} = log2
// p_j(X_{j+1}) - log2 q_j(X_{j+1}) (see the large kernel for the correction by k_eps), all rows of a wave side by side.
// `pairs`: the words of row 0 of the sequence in the copy that this workgroup polls, the next row's `pair_stride` further on.
// `bits`: token_logit in the first two lanes of the segments of the first pass (later passes fetch theirs here).
template <typename T, int FORM>
__device__ __forceinline__ void rows_normalisers(const FusedParams &P, size_t seq_d, size_t seq_u, const u64 *pairs, int pair_stride, int n, int own, int nwg,
                                                 int wave, uint32_t bits, RowsOut &out, bool &gave_up)
{
    constexpr bool kTwo = FORM == 2;
    const int lane = threadIdx.x & 63, e = lane & (kSegment<FORM> - 1), e2 = e + kSegment<FORM>;
    for (int r0 = wave * kWaveRows<FORM>; r0 < n; r0 += kWaves * kWaveRows<FORM>) {
        const int row = r0 + lane / kSegment<FORM>;
        const bool used = row < n;
        // (lanes without a word of their own look at one that is waited for anyway)
        const u64 *const words = pairs + (unsigned)((used ? row : r0) * pair_stride);
        const u64 *const word = words + 2 * (e < nwg ? e : 0), *const word2 = words + 2 * (e2 < nwg ? e2 : 0);
        u64 p = ld_u64(word), q = ld_u64(word + 1), p2 = 1, q2 = 1;
        if constexpr (kTwo) { p2 = ld_u64(word2); q2 = ld_u64(word2 + 1); }
        for (int spins = 0; __any(p == 0 || q == 0 || p2 == 0 || q2 == 0);) {
            if (++spins > P.spin_limit) { gave_up = true; break; }
            __builtin_amdgcn_s_sleep(1);
            p = ld_u64(word); q = ld_u64(word + 1);
            if constexpr (kTwo) { p2 = ld_u64(word2); q2 = ld_u64(word2 + 1); }
        }
        // the lane's words against the segment's largest, through exact powers of two
        float mp = e < nwg ? stat_shift(p) : -INFINITY, mq = e < nwg ? stat_shift(q) : -INFINITY, Mp = mp, Mq = mq;
        if constexpr (kTwo) { Mp = e2 < nwg ? fmaxf(mp, stat_shift(p2)) : mp; Mq = e2 < nwg ? fmaxf(mq, stat_shift(q2)) : mq; }
        Mp = group_max<kSegment<FORM>>(Mp); Mq = group_max<kSegment<FORM>>(Mq);
        auto mass = [](bool is, u64 w, float M) {
            const float m = stat_shift(w);
            const double z = ldexp((double)stat_sum(w), (int)(shift_of(m) - shift_of(M)));
            return is && m > -INFINITY ? z : 0.0;
        };
        double zp = mass(e < nwg, p, Mp);
        double zq = mass(e < nwg, q, Mq);
        if constexpr (kTwo) { zp += mass(e2 < nwg, p2, Mp); zq += mass(e2 < nwg, q2, Mq); }
        zp = group_sum<kSegment<FORM>>(zp);
        zq = group_sum<kSegment<FORM>>(zq);
        // even lanes go on with the target row, odd ones with the draft row
        const bool odd = (lane & 1) != 0;
        const float M = odd ? Mq : Mp;
        const double L = (double)shift_of(M) + log2_precise<true>(odd ? zq : zp);
        const double l = (double)logit_bits_as_float<T>(bits) * P.kd - (L + P.k_eps * (double)M);
        const double lr = fmax(l - dpp_shift_double<0xB1>(l), kLog2RatioFloor);        // (even lanes)
        if (used && e == 0) out.lr[row] = lr;
        if (used && e < 2 && row == own) out.L[e] = L;
        // (fetched at the end of a pass: at its beginning a wait for the first pass's logits would stand in front of the words)
        const int later = row + kWaves * kWaveRows<FORM>;
        if (later < n && e < 2) bits = token_logit<T>(P, seq_d, seq_u, later, P.tokens[seq_d + later]);
    }
    if (lane == 0) out.gave_up[wave] = gave_up ? 1 : 0;
}

// log2 w_{j+1} in lane j from the ratios in lanes 0 .. n - 1 (0 beyond); `passed` (Alg. 1): bit j, whether the test of X_{j+1} passes.  See weights_from_ratios.
__device__ __forceinline__ double weights_from_logs(int algo, double lr, u64 passed, int n)
{
    if (algo == kToken) return (~passed & ((2ull << (threadIdx.x & 63)) - 1ull)) == 0 ? 0.0 : kLog2RatioFloor;
    const double sum = scan_of(lr, n);
    return algo == kBlock ? sum - scan_max0_of(sum, n) : sum;
}

// ------------------------------------------------------------------ the draw inside one wave's unit
// A unit is 64 * LANE logits (vocabulary order inside it: vector, lane, element).  What can be prepared before it is known
// where the token lies: the weights' sums per (vector, lane) meet in `sums` (64 * NV floats in LDS that only this wave
// uses), every lane takes NV consecutive ones, and a scan over the wave gives the running sums.
template <int NV>
struct UnitSums {
    float ent[NV], mine;
    double inc;
    __device__ __forceinline__ void load(const float *sums)
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int lane = threadIdx.x & 63;
        mine = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j) { ent[j] = sums[lane * NV + j]; mine += ent[j]; }
        inc = wave_scan((double)mine);
    }
    // The entry whose running sum exceeds t first (else the last one with any weight); `t_e`: what is left of t inside it.
    __device__ __forceinline__ int locate(double t, double &t_e) const
    {
        const int lane = threadIdx.x & 63;
        const u64 hit = __ballot(inc > t), nz = __ballot(mine > 0.f);
        const int hl = hit ? __ffsll((long long)hit) - 1 : nz ? 63 - __clzll((long long)nz) : 0;
        // (every lane goes through its own entries; the one that counts is read)
        double r = inc - (double)mine, before = 0.0;
        int last_j = 0, found = -1;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            if (found < 0 && hit && r + (double)ent[j] > t) { found = j; before = r; }
            if (ent[j] > 0.f) last_j = j;
            r += (double)ent[j];
        }
        t_e = read_lane_double(found >= 0 ? t - before : INFINITY, hl);
        return __builtin_amdgcn_readlane(hl * NV + (found < 0 ? last_j : found), hl);
    }
};
// Which of the calls that resident_sets() admits this kernel takes (`workgroups` of them; `resident`: how many of this kernel's the device keeps
// resident).  Other kernel / this one, us.  float32: every call but those of long drafts over the widest rows (gamma = 16, V = 200000, 850
// workgroups 18.1 / 20.0; gamma = 8: 1125 18.9 / 19.2, 576 13.6 / 12.9); elsewhere V = 128256, gamma = 8, 1152 19.2 / 18.1, V = 64000, gamma = 8, 1872 27.3 /
// 25.5, V = 16000, gamma = 16, 2584 33.6 / 31.2, V = 5000, gamma = 8, 1899 23.6 / 22.5.  bf16: up to one resident set (of 1024): gamma = 8, V = 16000, 702 12.4 / 10.8,
// V = 30001, 684 13.4 / 11.6; drafts of four and more up to an eighth beyond, where only last target rows are late: gamma = 4, V = 30001, 1100
// 15.6 / 13.8, gamma = 8, V = 100277, 1053 15.6 / 14.4 (gamma = 2, V = 5000, 1101 12.7 / 13.1).  Beyond, the other kernel runs a fifth more workgroups at once:
// gamma = 8, V = 64000, 1368 15.5 / 16.3, V = 100277, 1404 17.2 / 18.1; further on neither is ahead by much (gamma = 8, V = 64000, 1872 18.6 / 17.4, gamma = 16, V =
// 100277, 2652 29.2 / 31.0), and with every S_i reported this one is behind.  Long float32 drafts of wider rows that nearly fill the device or more (everybody reads
// the words of thirteen rows and more) are the other kernel's too: gamma = 13, V = 89412, 924 workgroups 16.3 / 17.2, V = 130372, 896 15.5 / 16.1, gamma = 15, V =
// 96256, 960 16.1 / 16.5, 1152 18.3 / 18.8; gamma = 16, V = 56644, 714 14.5 / 13.2, V = 130372, 816 14.8 / 14.5, gamma = 12, V = 66000, 936 16.5 / 15.9.
inline bool runs_together(long long workgroups, long long resident, int groups, int gamma, bool f32)
{
    if (groups > 16 && (gamma > 8 || (gamma > 4 && workgroups > resident))) return false;
    if (f32 && groups > 4 && gamma > 12 && 5 * workgroups > 4 * resident) return false;
    return f32 || workgroups <= (gamma >= 4 ? resident + resident / 8 : resident);
}

// Grid (x, y, z) = (workgroup of the row, sequence, slot): slot i is row pair i, slot gamma the sequence's last target
// row; x runs fastest in the start order, so a row's workgroups start together and a position's before the next one's.
// A workgroup waits for workgroups of its own row and of earlier positions only (the last target row: of all), so the earliest
// unfinished row can always run, whatever else the device is busy with.
template <typename T, bool ALIGNED, int FORM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void together_verify_kernel(const FusedParams P_args)
{
    constexpr int LANE = kLaneSmall, kUnitLogits = kWave * LANE, kVec = ElemTraits<T>::kVec, kNV = LANE / kVec;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = blockIdx.x, b = blockIdx.y, slot = blockIdx.z, nwg = gridDim.x;
    const int gamma = P_args.gamma, V = P_args.V, nu = P_args.nu;
    const float k = P_args.k;
    long long *stamps = nullptr;
#ifdef SV_PROFILE
    if (P_args.prof) stamps = P_args.prof + (((size_t)b * (gamma + 1) + slot) * nwg + c) * 16;      // one record per workgroup
#endif
    SV_STAMP(0);
    int gb = gamma;
    if (P_args.draft_lens) { gb = load_uniform(P_args.draft_lens + b); gb = gb < 1 ? 1 : gb > gamma ? gamma : gb; }
    const bool last_row = slot == gamma;
    const bool unused = !last_row && slot >= gb;
    const int i = last_row ? gb : slot;
    const size_t seq_d = (size_t)b * gamma, seq_u = (size_t)b * (gamma + 1);
    const size_t drow = seq_d + (last_row ? 0 : i);
    const T *rowA = static_cast<const T *>(P_args.target) + (seq_u + i) * P_args.tstride;
    const T *rowB = static_cast<const T *>(P_args.draft) + drow * P_args.dstride;
    const int unit_first = (c * kWaves + wave) * kUnitLogits;
    // the rows whose ratios this workgroup needs: its own and all earlier ones
    const int n_rows = last_row ? gb : i + 1;
    const int first_row = wave * kWaveRows<FORM> + lane / kSegment<FORM>;                        // the lane's row in the first pass
    const bool wants_token = first_row < n_rows && (lane & (kSegment<FORM> - 1)) < 2;

    // the rows' loads first: they depend on the arguments only; behind them the drafted tokens of the wave's rows and the uniforms
    RawSlice<T, ALIGNED, LANE> rawA, rawB;
    uint32_t tok_bits = 0;
    int tok = 0;
    float eta = 0.f;                                              // lane j: eta_{j+1}
    if (!unused) {
        issue_loads<T, ALIGNED, LANE>(rowA, unit_first, V, rawA);
        if (!last_row) issue_loads<T, ALIGNED, LANE>(rowB, unit_first, V, rawB);
        asm volatile("" ::: "memory");
        if constexpr (FORM == 0) {
            if (wants_token) tok = P_args.tokens[seq_d + first_row];
        } else {
            // (four rows: their tokens through the scalar path, which does not queue behind the rows)
            const int r0 = wave * kWaveRows<FORM>, top = n_rows - 1;
            const int t0 = load_uniform(P_args.tokens + seq_d + min(r0, top)), t1 = load_uniform(P_args.tokens + seq_d + min(r0 + 1, top));
            const int t2 = load_uniform(P_args.tokens + seq_d + min(r0 + 2, top)), t3 = load_uniform(P_args.tokens + seq_d + min(r0 + 3, top));
            const int s = lane / kSegment<FORM>;
            tok = s < 2 ? (s == 0 ? t0 : t1) : s == 2 ? t2 : t3;
            if (wants_token) tok_bits = token_logit<T>(P_args, seq_d, seq_u, first_row, tok);
        }
        if (lane < gb) eta = P_args.uniforms[seq_u + lane];
    }
    asm volatile("" ::: "memory");
    const int magic_word = load_uniform(P_args.header + kHdrMagic);
    const unsigned par = (unsigned)load_uniform(P_args.gen + b) & 1u;
    if (magic_word != P_args.magic) {
        if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
            for (int s = threadIdx.x; s < P_args.B; s += kThreads) { P_args.accept_len[s] = -1; P_args.next_token[s] = -1; }
        return;
    }
    // every slot's words are cleared, in the copy that this call does not use, by the last wave of the slot's last
    // workgroup, once it has nothing to wait for any more (an unused position's in both copies: the other one may hold an
    // earlier, longer call's words)
    const bool row_end = c == nwg - 1, leader = wave == 0 && row_end, clears = wave == kWaves - 1 && row_end;
    if (unused) {
        if (clears) { clear_row_words(P_args, P_args.words, b, slot, true); clear_row_words(P_args, words_of(P_args, 1), b, slot, true); }
        return;
    }
    // (the addresses in the copy that this call uses are formed where they are used: the kernel is short of scalar registers)
#define SV_WORDS words_of(P, launder(par))
    const float u = load_uniform(P_args.uniforms + seq_u + gb);
    const bool token_algo = P_args.algo == kToken;
    const int copy = c % kWordCopies;

    __shared__ u64 wave_words[2][kWaves];
    __shared__ float wave_part[kWaves];
    __shared__ double draw_t;
    __shared__ int draw_role, draw_wave, draw_passes;
    __shared__ float draw_sums[kWaves][kWave * kNV];               // per wave: its unit's weights summed per (vector, lane)
    __shared__ RowsOut rows;
    bool gave_up = false;

    // ---- first sweep (as in the large kernel): exponentials stay in xa / xb
    float xa[LANE], xb[LANE];
    float shiftA, shiftB = 0.f;
    unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawA, xa);
    const u64 stA = first_sweep_row(xa, k, shiftA);
    if (!last_row) unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawB, xb);
    // (the drafted tokens' logits, asked for now: the tokens have come in with the rows, and the logits will have before the words)
    if constexpr (FORM == 0) { if (wants_token) tok_bits = token_logit<T>(P_args, seq_d, seq_u, first_row, tok); }
    if (!last_row) {
        const u64 stB = first_sweep_row(xb, k, shiftB);
        if (lane == 0) wave_words[1][wave] = stB;
    }
    if (lane == 0) wave_words[0][wave] = stA;
    __syncthreads();
    SV_STAMP(1);
    u64 own_plast = 0;
    if (wave == 0) {
        const Words W = words_of(P_args, par);
        // the workgroup's two words, into every copy (lanes 8 c, 8 c + 4: target, draft word of copy c); a last target row has one
        const u64 w = quad_word(wave_words[(lane >> 2) & 1][lane & 3]);
        if (last_row) {
            own_plast = read_lane_u64(w, 0);
            if (lane == 0) st_u64(W.plast + (size_t)b * nu + c, w);
        } else if ((lane & 3) == 0 && lane < 8 * kWordCopies) {
            const unsigned entry = 2 * c + ((lane >> 2) & 1);
            u64 *const first = row_pairs(W, drow, nwg, 0), *const others = row_pairs(W, drow, nwg, 1);
            st_u64(lane < 8 ? first + entry : others + ((lane >> 3) - 1) * 2 * nwg + entry, w);
        }
    }
    // ---- the normalisers and ratios of the own row and all earlier ones
    // (the arguments once more: fewer scalar registers spilled on the way here, B = 8, gamma = 8, V = 32000, float32 10.4 -> 9.9 us; form 1 spills
    // few as it is and would wait for them)
    const FusedParams P = FORM == 1 ? P_args : reread_params();
    rows_normalisers<T, FORM>(P, seq_d, seq_u, row_pairs(SV_WORDS, seq_d, nwg, copy), (copy == 0 ? 2 : 4) * nwg, n_rows, last_row ? -1 : i, nwg, wave, tok_bits, rows, gave_up);
    SV_STAMP(7);
    __syncthreads();
    if (clears) {
        clear_row_words(P, words_of(P, par ^ 1u), b, slot, true);
        // (one writer: every workgroup reads this line at its start, and 1600 writes to it cost 48 us)
        if (last_row && b == 0 && lane == 0) __hip_atomic_store(SV_GLOBAL(int, P.header + kHdrRowWords), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    gave_up = (rows.gave_up[0] | rows.gave_up[1] | rows.gave_up[2] | rows.gave_up[3]) != 0;
    if (gave_up) report_gave_up(P);
    // ---- (every wave for itself) what the ratios say: the weights, which positions can become tau, which surely pass
    const double lr = lane < n_rows ? rows.lr[lane] : 0.0;
    const u64 passed = token_algo ? __ballot(lane < n_rows && (double)eta < exp2_precise<true>(fmin(lr, 0.0))) : 0;       // Alg. 1: bit j, the test of X_{j+1}
    const double lw = weights_from_logs(P.algo, lr, passed, n_rows);                                                      // lane j: log2 w_{j+1}
    SV_STAMP(9);

    // =================================================================== the sequence's last target row
    if (last_row) {
        // Y comes from it where every token is accepted, which its workgroups see from the ratios; the leader writes
        // tau and Y (Y from the word of position tau, or from the word that the workgroup holding it publishes)
        const Words W = SV_WORDS;
        u64 *const y_word = W.lw + seq_d + gb - 1;                    // (a word this kernel has no other use for)
        const u64 *const pl_word = W.plast + (size_t)b * nu + (lane < nwg ? lane : 0);
        bool all_accepted;
        double w_last = 1.0;
        if (token_algo) {
            all_accepted = (passed & (gb < 64 ? (1ull << gb) - 1ull : ~0ull)) == (gb < 64 ? (1ull << gb) - 1ull : ~0ull);
        } else {
            const double lw_g = read_lane_double(lw, gb - 1);
            const float eta_g = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(eta), gb - 1));
            w_last = exp2_precise<true>(P.algo == kGreedy ? fmin(lw_g, 100.0) : lw_g);
            all_accepted = (double)eta_g < fmin(w_last, 1.0);                      // eta_gamma < h_gamma = w_gamma
        }
        u64 pl = 0;                                                   // the row's words (lane e: workgroup e's)
        if (all_accepted && !gave_up) {
            if (wave == 0) {
                // the row's words, all of them: where u * (the row's sum) falls
                pl = wait_word(pl_word, lane == c ? own_plast : ld_u64(pl_word), lane < nwg, P.spin_limit, gave_up);
                const float m = lane < nwg ? stat_shift(pl) : -INFINITY;
                const float M = wave_max(m);
                const double z = m > -INFINITY ? ldexp((double)stat_sum(pl), (int)(shift_of(m) - shift_of(M))) : 0.0;
                const double inc = scan_of(z, nwg);
                double t_in;
                int role = 0;
                const int e = locate_entry(z, inc, late_double(u) * read_lane_double(inc, nwg - 1), t_in);
                if (e == c && !gave_up) {
                    // ... and in which of the workgroup's four units
                    const u64 ww = wave_words[0][lane & 3];
                    const float mw = lane < kWaves ? stat_shift(ww) : -INFINITY;
                    const double zw = mw > -INFINITY ? ldexp((double)stat_sum(ww), (int)(shift_of(mw) - shift_of(M))) : 0.0;
                    double t_w;
                    const int wv = locate_entry(zw, scan_of(zw, kWaves), t_in, t_w);
                    // (into the units of that wave's exponentials, which are relative to its own shift)
                    const float m_wv = stat_shift(read_lane_u64(ww, wv));
                    if (lane == 0) { draw_wave = wv; draw_t = ldexp(t_w, (int)(shift_of(M) - shift_of(m_wv))); }
                    role = 1;
                }
                if (gave_up) { report_gave_up(P); if (lane == 0) st_u64(y_word, kPoison64); }
                if (lane == 0) draw_role = role;
            }
            __syncthreads();
            if (draw_role == 1 && wave == draw_wave) {
                const int off = draw_in_unit<kVec, LANE>([&](int j) { return xa[j]; }, draw_t, draw_sums[wave]);
                if (lane == 0) st_u64(y_word, pack_rowres(true, min(unit_first + off, V - 1)));
            }
        }
        if (!leader) return;

        // ---- the leader: tau and Y
        if (pl == 0) pl = lane == c ? own_plast : ld_u64(pl_word);
        int tau, y;
        if (all_accepted) {
            tau = gb;
            y = rowres_token(wait_word(y_word, P.spin_limit, gave_up));
        } else if (token_algo) {
            // tau is the length of the leading run of passed tests; its position's word holds the token
            tau = __ffsll((long long)~passed) - 1;
            y = rowres_token(wait_word(W.rowres + seq_d + tau, P.spin_limit, gave_up));
        } else {
            // tau is the last position whose test passes, else 0.  A test whose w is 1 passes: only the positions from the
            // last such one on count, and of these only those that can become tau have a word (bit j of the masks: position j).
            const u64 in_draft = gb < 64 ? (1ull << gb) - 1ull : ~0ull;
            const u64 sure = __ballot(lane < gb && lw >= 0.0) << 1 & in_draft;
            const u64 can = (__ballot(lane < gb && (double)__builtin_amdgcn_logf(eta) < lw + 1.0e-3) << 1 | 1ull) & in_draft;
            const int from = sure ? 63 - __clzll((long long)sure) : 0;
            const u64 counts = can & ~(sure >> 1) & ~((1ull << from) - 1ull);
            const bool mine = (counts >> lane & 1ull) != 0;
            const u64 res = wait_word(W.rowres + seq_d + (lane < gb ? lane : 0), mine ? ld_u64(W.rowres + seq_d + lane) : 0, mine, P.spin_limit, gave_up);
            const u64 tests = __ballot(mine && rowres_passes(res)) & ~1ull;
            tau = tests ? 63 - __clzll((long long)tests) : from;
            y = rowres_token(read_lane_u64(res, tau));
        }
        if (lane == 0) {
            P.accept_len[b] = gave_up ? -1 : tau;
            P.next_token[b] = gave_up ? -1 : max(y, 0);
        }
        if (P.debug_out && lane == 0) {
            float *d = P.debug_out + (seq_u + gb) * 3;       // S_gamma = w_gamma: q_gamma == 0
            d[0] = (float)w_last; d[1] = (float)w_last;
            d[2] = token_algo ? (float)exp2_precise<true>(fmin(read_lane_double(lr, gb - 1), 0.0)) : (float)fmin(w_last, 1.0);
        }
        // the call count flips once every workgroup of the sequence has read it: the row pairs' have where their words are
        // there (this workgroup has them all), the last target row's where theirs are
        bool late = false;
        wait_word(pl_word, pl, lane < nwg, P.spin_limit, late);
        if (gave_up || late) report_gave_up(P);
        if (lane == 0) {
            if (late) { P.accept_len[b] = -1; P.next_token[b] = -1; }
            __hip_atomic_store(P.gen + b, (int)(par ^ 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        SV_STAMP(6);
        return;
    }

    // =================================================================== a row pair
    double log2w = i > 0 ? read_lane_double(lw, i - 1) : 0.0;
    const float eta_i = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(eta), i > 0 ? i - 1 : 0));
    const bool next_passes = (passed >> i & 1ull) != 0;              // Alg. 1: the test of X_{i+1}
    const bool candidate = can_become_tau(P.algo, i, log2w, eta_i);
    // Whether S_i matters: the position can become tau (position 0 always can), and the next test does not pass whatever its
    // uniform is (Alg. 1: tau is the position whose next test fails).  The leader of the last target row, which has the same ratios,
    // does not ask for the others; their word says that their test fails all the same (rows whose arithmetic makes NaNs may
    // look different to the two).
    const bool counts = candidate && !(token_algo ? next_passes : read_lane_double(lw, i) >= 0.0);
    if (!counts && !P.debug_out && !gave_up) {
        if (leader && lane == 0) st_u64(SV_WORDS.rowres + drow, pack_rowres(false, -1));
        return;
    }
    if (token_algo) log2w = 0.0;                                // the residual of token verification is p - q
    if (P.algo == kGreedy) log2w = fmin(log2w, 100.0);          // keeps w p finite in float
    // ---- the second sweep's row constants (see the large kernel); the three powers side by side in three lanes
    const double Lq = rows.L[1], A = rows.L[0] - log2w, Ai = rint(A), Qi = rint(Lq);
    double fq, frho, frho_inv;
    {
        const double dq = Qi - Lq, d = (Ai - A) - dq;
        const double x = exp2_precise<true>(lane == 0 ? dq : lane == 1 ? d : -d);
        fq = read_lane_double(x, 0); frho = read_lane_double(x, 1); frho_inv = read_lane_double(x, 2);
    }
    SV_STAMP(2);

    // ---- second sweep, from registers (as in the large kernel): terms in [0, 1] in units of the larger row factor
    const int ea = unit_exponent(shiftA, Ai), eq = unit_exponent(shiftB, Qi);
    const double rho = ldexp(frho, ea - eq);
    const bool q_units = rho <= 1.0;
    const float factor = q_units ? (float)rho : -(float)ldexp(frho_inv, eq - ea);
    const float scale = q_units ? (float)ldexp(fq, eq) : (float)ldexp(fq * frho, ea);
    {
        // (the sums per vector stay behind in LDS: the draw, if it falls into this unit, starts from them)
        float acc = 0.f;
        auto sums = [&](auto term) {
#pragma unroll
            for (int v = 0; v < kNV; ++v) {
                float sv_ = 0.f;
#pragma unroll
                for (int e = 0; e < kVec; ++e) sv_ += term(v * kVec + e);
                draw_sums[wave][v * kWave + lane] = sv_;
                acc += sv_;
            }
        };
        if (q_units) sums([&](int j) { return __builtin_amdgcn_fmed3f(__builtin_fmaf(xa[j], factor, -xb[j]), 0.f, 1.f); });
        else sums([&](int j) { return __builtin_amdgcn_fmed3f(__builtin_fmaf(xb[j], factor, xa[j]), 0.f, 1.f); });
        acc = wave_sum(acc * scale);
        if (lane == 0) wave_part[wave] = acc;
    }
    __syncthreads();
    SV_STAMP(4);
    // ---- the workgroup's share of S_i goes out, into every copy
    const unsigned *sp_word = nullptr;
    unsigned own_part = 0, sp = 0;
    if (wave == 0) {
        const Words W = SV_WORDS;
        sp_word = W.spart + drow * nu + copy * nwg + (lane < nwg ? lane : 0);
        own_part = gave_up ? kPoison32 : pack_partial((wave_part[0] + wave_part[1]) + (wave_part[2] + wave_part[3]));
        if (lane < kWordCopies) st_u32(W.spart + drow * nu + lane * nwg + c, own_part);
        sp = lane == c ? own_part : ld_u32(sp_word);
    }
    // ---- while the shares travel: each wave's running sums over its unit, what the accept test needs of w_i
    UnitSums<kNV> unit;
    unit.load(draw_sums[wave]);
    if (wave == 0) {
        const Words W = SV_WORDS;
        const bool has_test = !token_algo && i > 0;
        const double one_minus_w = has_test ? one_minus_exp2<true>(fmin(log2w, 0.0)) : 0.0;
        sp = wait_word32(sp_word, sp, lane < nwg, P.spin_limit, gave_up);
        SV_STAMP(5);
        double z = lane < nwg ? (double)unpack_partial(sp) : 0.0;
        double inc = scan_of(z, nwg);
        const double S_i = read_lane_double(inc, nwg - 1);
        // ---- the position's accept test (Alg. 2 / 4); Alg. 1: the test of X_{i+1} came with the ratio
        // (Alg. 2 / 4, position i >= 1: eta_i < h_i = S_i / (S_i + 1 - w_i), 1 where w_i >= 1 - see AcceptTest; judged
        // without the division)
        const bool test_passes = has_test && candidate && (log2w >= 0.0 || late_double(eta_i) * (S_i + one_minus_w) < S_i);
        // the token that follows if this position becomes tau is drawn where it can
        const bool want = !gave_up && counts && (token_algo || i == 0 || test_passes);
        int role = 0;
        if (want) {
            // where u * S_i falls; a residual without any mass is drawn from p_i instead (weights: the exponentials)
            const bool from_p = !(S_i > 0.0);
            float Mp = 0.f;
            if (from_p) {
                const u64 grp = ld_u64(row_pairs(W, drow, nwg, copy) + 2 * (lane < nwg ? lane : 0));
                const float m = lane < nwg ? stat_shift(grp) : -INFINITY;
                Mp = wave_max(m);
                z = m > -INFINITY ? ldexp((double)stat_sum(grp), (int)(shift_of(m) - shift_of(Mp))) : 0.0;
                inc = scan_of(z, nwg);
            }
            double t_in;
            const int e = locate_entry(z, inc, late_double(u) * read_lane_double(inc, nwg - 1), t_in);
            if (e == c) {
                role = 1;
                if (from_p) {
                    const u64 ww = wave_words[0][lane & 3];
                    const float mw = lane < kWaves ? stat_shift(ww) : -INFINITY;
                    const double zw = mw > -INFINITY ? ldexp((double)stat_sum(ww), (int)(shift_of(mw) - shift_of(Mp))) : 0.0;
                    double t_w;
                    const int wv = locate_entry(zw, scan_of(zw, kWaves), t_in, t_w);
                    t_in = ldexp(t_w, (int)(shift_of(Mp) - shift_of(stat_shift(read_lane_u64(ww, wv)))));
                    if (lane == 0) draw_wave = wv;
                    role = 2;
                }
                if (lane == 0) { draw_t = t_in; draw_passes = token_algo ? 0 : test_passes ? 1 : 0; }
            }
        } else if (leader && lane == 0) {
            st_u64(W.rowres + drow, gave_up ? kPoison64 : pack_rowres(false, -1));
        }
        if (gave_up) report_gave_up(P);
        if (lane == 0) draw_role = role;
        SV_STAMP(10);
        if (P.debug_out && leader && lane == 0) {
            float *d = P.debug_out + (seq_u + i) * 3;            // (w_i, S_i, h_i); Alg. 1 has no w, its h_i = min(r_i, 1)
            double h_i = has_test && log2w < 0.0 ? S_i / (S_i + one_minus_w) : 1.0;
            if (token_algo && i > 0) h_i = exp2_precise<true>(fmin(rows.lr[i - 1], 0.0));
            d[0] = has_test ? (float)exp2_precise<true>(log2w) : 1.f; d[1] = (float)S_i; d[2] = (float)h_i;
        }
    }
    __syncthreads();
    SV_STAMP(11);
    const int role = draw_role;
    if (role == 0) return;
    // ---- the wave that holds the token draws it from its registers and publishes the position's word
    const double t = draw_t;
    int off;
    if (role == 2) {
        if (wave != draw_wave) return;
        off = draw_in_unit<kVec, LANE>([&](int j) { return xa[j]; }, t, draw_sums[wave]);
    } else {
        // the first wave whose running sum exceeds t; where rounding leaves none, the last one with any mass
        int holder = -1, last_wave = 0;
        double running = 0.0, front = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const double part = (double)wave_part[w];
            if (holder < 0 && running + part > t) { holder = w; front = running; }
            if (part > 0.0) last_wave = w;
            running += part;
        }
        if (wave != (holder < 0 ? last_wave : holder)) return;
        double t_e;
        const int entry = unit.locate(holder < 0 ? INFINITY : (t - front) / (double)scale, t_e);
        // (the terms once more: kept from the sweep, they would cost the kernel its registers)
        float f = factor;
        asm volatile("" : "+v"(f));
        off = entry * kVec + walk_entry<kVec, LANE>([&](int j) {
            return q_units ? __builtin_amdgcn_fmed3f(__builtin_fmaf(xa[j], f, -xb[j]), 0.f, 1.f)
                           : __builtin_amdgcn_fmed3f(__builtin_fmaf(xb[j], f, xa[j]), 0.f, 1.f); }, entry, t_e);
    }
    // (a row of which the arithmetic makes NaNs still ends inside the vocabulary)
    if (lane == 0) st_u64(SV_WORDS.rowres + drow, pack_rowres(draw_passes != 0, max(0, min(unit_first + off, V - 1))));
    SV_STAMP(15);
#undef SV_WORDS
}

}  // namespace sv
