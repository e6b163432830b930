// Sequences of short rows, as many to a workgroup as fill its waves: a row pair in the registers of 1, 4, 16, 32 or 64 lanes, as
// small_verify_kernel (tiny.hpp) has it, and what exists once per position - normalisers, ratios, weights, row factors, tests, all in
// double, about 900 instructions - side by side for up to four sequences, each in sixteen lanes of a wave.
// What bounds it: for few sequences the chain of steps (4.9 us a call on the device at best, of which the launch and one trip to memory
// are four), for many the vector instructions: a wave per row pair, or per sequence of a few tokens, spends most of them on reductions over
// lanes and on scalars in double with most lanes idle.  8192 sequences of 10 over 2 tokens, float32: 11.8 -> 5.9 us; 8192 of 4 over 60 17.9 ->
// 13.8; 3541 of 11 over 192, bf16 41.8 -> 21.2 (which lanes and how many sequences: packed_launch, with both sides' times).
// Probabilities (PROBS) take this kernel up to 2048 tokens (but for the calls that packed_launch names), in one launch and on no scratch memory: 2207 of 10 over 256, float32 55.7 -> 15;
// 6000 of 10 over 2 163 -> 5.8; 64 of 10 over 2 13.1 -> 4.9.
#pragma once

#include "tiny.hpp"
#include "probs.hpp"

namespace sv {

// Inclusive scans over segments of SEG = 16 or 64 lanes.
template <int SEG> __device__ __forceinline__ double segment_scan(double v) { return group_scan<SEG>(v); }
template <int SEG> __device__ __forceinline__ double segment_scan_max0(double v)
{
    if constexpr (SEG == kWave) return wave_scan_max0(v);
    v = fmax(v, 0.0);
    v = fmax(v, dpp_shift_double<0x111>(v));
    v = fmax(v, dpp_shift_double<0x112>(v));
    v = fmax(v, dpp_shift_double<0x114>(v));
    v = fmax(v, dpp_shift_double<0x118>(v));
    return v;
}

// A workgroup holds P.group_seqs sequences.  SEG: lanes that a sequence's positions take where they are worked on one per lane.  PROBS: the rows are
// probabilities, used as given (see probs.hpp); a row has no normaliser then, and a workspace's control words are not looked at.
// Uses of FusedParams: see tiny_verify_kernel; group_seqs, inv_slots (of gamma + 1).
template <typename T, bool PROBS, int G, int LANE, int SEG>
__global__ __launch_bounds__(G == 1 ? 2 * kWave : kTinyThreads)
void packed_verify_kernel(const FusedParams P)
{
    constexpr bool kFma = LANE == 8;                // (see series_step)
    constexpr int kMost = G == 1 ? 2 * kWave : kTinyThreads, kGroups = kMost / G, kSeqs = kMost / SEG;
    constexpr int kVec = ElemTraits<T>::kVec, kNV = LANE / kVec;
    // per row pair, as its group leaves them: the sums of both rows' exponentials, their largest scaled logits, the drafted token's two
    // logits; what the second sweep takes as the positions' lanes form it (PROBS: w in two floats); the sum of the residual terms (Alg. 4 on
    // probabilities: and the rejected mass, in sum_q)
    __shared__ struct {
        double sum_p[kGroups], sum_q[kGroups], mass[kGroups];
        float max_p[kGroups], max_q[kGroups], tok_p[kGroups], tok_q[kGroups], factor[kGroups], w_lo[PROBS ? kGroups : 1];
        int tau[kSeqs], residual[kSeqs];            // residual: whether the draw is from the residual of row tau
    } own;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = lane & (G - 1);
    const int first = (int)blockIdx.x * P.group_seqs;
    const int gamma = P.gamma, V = P.V, algo = P.algo, n_seqs = min(P.group_seqs, P.B - first);
    const float k = P.k;
    const bool token_algo = algo == kToken, greedy_algo = algo == kGreedy;
    auto draft_len = [&](int b) {
        if (!P.draft_lens) return gamma;
        const int g = P.draft_lens[b];
        return g < 1 ? 1 : g > gamma ? gamma : g;
    };
    // the group's row: row pair i of sequence s, its last target row (i == gb), or nothing (the groups beyond)
    const int g = tid / G, s = (int)__umulhi((unsigned)g, P.inv_slots), i = g - s * (gamma + 1);
    const int b = first + min(s, n_seqs - 1), gb = draft_len(b);
    const bool has_a = s < n_seqs && i <= gb, pair = s < n_seqs && i < gb;
    const size_t seq_d = (size_t)b * gamma, seq_u = (size_t)b * (gamma + 1);
    const T *const rowA = static_cast<const T *>(P.target) + (seq_u + (has_a ? i : gb)) * P.tstride;
    const T *const rowB = static_cast<const T *>(P.draft) + (seq_d + (pair ? i : 0)) * P.dstride;
    const int nv = (V - 1) / (G * kVec) + 1;                                  // vectors of a lane that reach into the row
    // the position that a lane works on between the sweeps: position j of sequence sj (`here`: there is one)
    const bool scalar_wave = wave * kWave < n_seqs * SEG;
    const int sj = min(tid / SEG, n_seqs - 1), j = tid & (SEG - 1), bj = first + sj, gbj = draft_len(bj);
    const bool here = tid < n_seqs * SEG && j < gbj;
    const int at = sj * (gamma + 1) + (here ? j : 0);                         // its group
    const size_t seq_uj = (size_t)bj * (gamma + 1);

    // ---- everything that depends on the arguments only, asked for at once
    const int tok = pair ? P.tokens[seq_d + i] : 0;
    uint4 rawA[kNV], rawB[kNV];
#pragma unroll
    for (int v = 0; v < kNV; ++v)
        if (v < nv) {
            rawA[v] = rawB[v] = make_uint4(0, 0, 0, 0);
            if (has_a) rawA[v] = load_raw<T, false, true>(rowA, V, (v * G + l) * kVec);
            if (pair) rawB[v] = load_raw<T, false, true>(rowB, V, (v * G + l) * kVec);
        }
    float eta = 0.f, eta_next = 0.f;                                          // eta_j, eta_{j+1}
    if (scalar_wave) {
        eta = P.uniforms[seq_uj + (here && j > 0 ? j - 1 : 0)];
        eta_next = P.uniforms[seq_uj + (here ? j : 0)];
    }
    const float u = P.uniforms[seq_u + gb];
    if constexpr (!PROBS) {
        const int magic_word = load_uniform(P.header + kHdrMagic);
        if (magic_word != P.magic) {
            // the workspace was not initialised for this shape: this kernel needs none of it, but the contract is one
            if (s < n_seqs && i == 0 && l == 0) { P.accept_len[b] = -1; P.next_token[b] = -1; }
            return;
        }
    }
    const float ya = logit_as_float(rowA + tok), yb = logit_as_float(rowB + tok);

    // ---- first sweep: exponentials against an integer shift per row, their sums in double (PROBS: the rows as they are)
    float xa[LANE], xb[LANE];
    auto sweep = [&](uint4 (&raw)[kNV], bool there, float (&x)[LANE], float &M) {
        float m = -INFINITY;
#pragma unroll
        for (int v = 0; v < kNV; ++v)
            if (v < nv) {
                // (only a row's last vectors reach beyond it)
                if (v + 1 < nv) unpack_vec<T>(raw[v], x + v * kVec);
                else unpack_raw<T, false>(raw[v], V, (v * G + l) * kVec, x + v * kVec);
#pragma unroll
                for (int e = 0; e < kVec; ++e) {
                    if constexpr (PROBS) x[v * kVec + e] = fmaxf(x[v * kVec + e], 0.f);
                    else m = fmaxf(m, x[v * kVec + e]);
                }
            }
        if constexpr (PROBS) return 0.0;
        M = group_max<G>(m * k);
        const float shift = shift_of(M);
        double acc = 0.0;
#pragma unroll
        for (int v = 0; v < kNV; ++v)
            if (v < nv) {
#pragma unroll
                for (int e = 0; e < kVec; ++e) {
                    float &y = x[v * kVec + e];
                    y = there ? fast_exp2(__builtin_fmaf(y, k, -shift)) : 0.f;
                    acc += (double)y;
                }
            }
        return group_sum<G>(acc);
    };
    {
        float Mp = 0.f, Mq = 0.f;
        const double zp = sweep(rawA, has_a, xa, Mp), zq = sweep(rawB, pair, xb, Mq);
        if (pair && l == 0) {
            own.tok_p[g] = ya; own.tok_q[g] = yb;
            if constexpr (!PROBS) { own.sum_p[g] = zp; own.sum_q[g] = zq; own.max_p[g] = Mp; own.max_q[g] = Mq; }
        }
    }
    __syncthreads();

    // ---- one position per lane: L_p, L_q, log2 r_{j+1}, log2 w_j, the second sweep's factor
    const u64 in_segment = SEG == kWave ? ~0ull : (1ull << (SEG & 63)) - 1ull;
    const int segment = lane & ~(SEG - 1);                   // its first lane
    auto ballot = [&](bool p) { return __ballot(p) >> segment & in_segment; };
    // (of probabilities by the series' full length: see log2_ratio; Alg. 4's w is infinite from a token on that only the draft rules out, as in the kernels for wider rows)
    auto power = [&](double x) { return PROBS && !(x < 2000.0) ? (double)INFINITY : exp2_precise<PROBS || kFma, PROBS>(x); };
    u64 tests_passed = 0;                                    // Alg. 1: bit j, the test of X_{j+1}
    double lr = 0.0, lw = 0.0, lw_next = 0.0, scale = 1.0;   // log2 r_{j+1}, log2 w_j, log2 w_{j+1}, the unit of the residual terms
    if (scalar_wave) {
        double log2_zp = 0.0, log2_zq = 0.0;
        if constexpr (PROBS) {
            lr = log2_ratio(own.tok_p[at], own.tok_q[at]);
        } else {
            const float Mp = own.max_p[at], Mq = own.max_q[at], sp = shift_of(Mp), sq = shift_of(Mq);
            log2_zp = log2_precise<kFma>(own.sum_p[at]); log2_zq = log2_precise<kFma>(own.sum_q[at]);
            // (see the large kernel for the correction by k_eps)
            const double lp = (double)own.tok_p[at] * P.kd - ((double)sp + log2_zp + P.k_eps * (double)Mp);
            const double lq = (double)own.tok_q[at] * P.kd - ((double)sq + log2_zq + P.k_eps * (double)Mq);
            lr = fmax(lp - lq, kLog2RatioFloor);
        }
        if (token_algo) tests_passed = ballot(here && (double)eta_next < power(fmin(lr, 0.0)));
        if constexpr (PROBS) {
            lw_next = algo == kBlock ? clamped_weights<SEG>(here ? lr : 0.0) : segment_scan<SEG>(here ? lr : 0.0);
        } else {
            const double sum = segment_scan<SEG>(here ? lr : 0.0);
            lw_next = algo == kBlock ? sum - segment_scan_max0<SEG>(sum) : sum;
        }
        lw = __shfl_up(lw_next, 1, kWave);
        // (the residual of token verification is p - q; Alg. 4 on logits: w stays finite)
        if (j == 0 || token_algo) lw = 0.0;
        if constexpr (PROBS) {
            const double w = power(lw);
            const float hi = (float)w;
            if (here) { own.factor[at] = hi; own.w_lo[at] = (float)(w - (double)hi); }
        } else {
            if (greedy_algo) { lw = fmin(lw, 100.0); lw_next = fmin(lw_next, 100.0); }
            const TinyCoef c = tiny_coef<kFma>(lw - log2_zp, -log2_zq);
            scale = c.scale;
            if (here) own.factor[at] = c.q_units ? c.f : -c.f;
        }
    }
    __syncthreads();

    // ---- S_i = sum_x max(w_i p_i(x) - q_i(x), 0), in units of the larger row factor (PROBS: as it is; of the last target row, its sum)
    const float f = pair ? own.factor[g] : 0.f, f_lo = PROBS && pair ? own.w_lo[PROBS ? g : 0] : 0.f;
    const bool q_units = !(f < 0.f);
    auto term = [&](int n) {
        if constexpr (PROBS) return fmaxf(prob_residual(xa[n], xb[n], f, f_lo), 0.f);
        else return q_units ? __builtin_amdgcn_fmed3f(__builtin_fmaf(xa[n], f, -xb[n]), 0.f, 1.f)
                            : __builtin_amdgcn_fmed3f(__builtin_fmaf(xb[n], f, xa[n]), 0.f, 1.f);
    };
    {
        double acc = 0.0, rej = 0.0;
        if constexpr (PROBS) {
            // (a vector's terms in float, of vectors in double: no chain of more than eight, as in the kernels for wider rows)
#pragma unroll
            for (int v = 0; v < kNV; ++v)
                if (v < nv) {
                    float mine = 0.f, against = 0.f;
#pragma unroll
                    for (int e = 0; e < kVec; ++e) {
                        const int n = v * kVec + e;
                        const float d = prob_residual(xa[n], xb[n], f, f_lo);
                        mine += pair ? fmaxf(d, 0.f) : xa[n];
                        against += fmaxf(-d, 0.f);
                    }
                    acc += (double)mine; rej += (double)against;
                }
        } else {
#pragma unroll
            for (int v = 0; v < kNV; ++v)
                if (v < nv) {
#pragma unroll
                    for (int e = 0; e < kVec; ++e) acc += (double)term(v * kVec + e);
                }
        }
        acc = group_sum<G>(acc);
        if (PROBS && greedy_algo) rej = group_sum<G>(rej);
        if ((PROBS ? has_a : pair) && l == 0) {
            own.mass[g] = acc;
            if (PROBS && greedy_algo) own.sum_q[g] = rej;
        }
    }
    __syncthreads();

    // ---- one position per lane again: the accept tests, tau
    if (scalar_wave) {
        const double S = (here ? own.mass[at] : 0.0) * scale;
        // Alg. 2 / 4, lane j judges position j >= 1: eta_j < h_j = S_j / (S_j + 1 - w_j), 1 where w_j >= 1 (see AcceptTest),
        // without the division; the last position, by lane gb - 1: eta_gb < w_gb.  Alg. 1: the tests came with the ratios.  (Alg. 4 on
        // probabilities, whose rows need not sum to one: S_j over the rejected mass)
        const double one_minus_w = one_minus_exp2<PROBS || kFma, PROBS>(fmin(lw, 0.0));
        const double R = PROBS && greedy_algo ? own.sum_q[at] : S + one_minus_w;
        const bool sure = PROBS && greedy_algo ? !(R > 0.0) : lw >= 0.0;                // h_j = 1
        const u64 tests = token_algo ? tests_passed : ballot(here && j > 0 && (sure || (double)eta * R < S));
        int tau;
        if (token_algo) {
            tau = min(__ffsll((long long)~tests) - 1, gbj);                              // leading run of passes
            if (tau < 0) tau = gbj;
        } else {
            const bool last = here && j == gbj - 1 && (lw_next >= 0.0 || (double)eta_next < power(lw_next));
            tau = ballot(last) ? gbj : tests ? 63 - __clzll((long long)tests) : 0;       // last passing sub-block
        }
        if (P.debug_out && here) {
            const double next_h = power(fmin(token_algo ? lr : lw_next, 0.0));
            const double h = j == 0 || sure ? 1.0 : fmin(S / R, 1.0);
            float *d = P.debug_out + (seq_uj + j) * 3;
            d[0] = (float)power(lw); d[1] = (float)S;
            if (!token_algo || j == 0) d[2] = (float)h;
            // (Alg. 1 has no w; its h_i = min(r_i, 1).  q_gamma == 0: S_gamma = w_gamma, times what the last target row sums to)
            if (token_algo) d[5] = (float)next_h;
            if (j == gbj - 1) {
                const double w_last = token_algo ? 1.0 : power(lw_next);
                d[3] = (float)w_last; d[4] = (float)(PROBS && algo != kBlock ? w_last * own.mass[at + 1] : w_last);
                d[5] = (float)next_h;
            }
        }
        if (tid < n_seqs * SEG) {
            if (j == 0) own.tau[sj] = tau;
            if (j == (tau < gbj ? tau : 0)) own.residual[sj] = tau < gbj && S > 0.0;     // (a residual without mass: Y comes from p_tau)
        }
    }
    __syncthreads();
    // ---- Y, by the groups that hold row tau of their sequences
    const int tau = own.tau[min(s, n_seqs - 1)];
    const bool draws = s < n_seqs && i == tau;
    if (!__any(draws)) return;
    const bool residual = own.residual[min(s, n_seqs - 1)] != 0;
    const int y = draw_in_group<G, kNV, kVec>([&](int n) { return residual ? term(n) : xa[n]; }, nv, [&](double total) { return (double)u * total; });
    if (draws && l == 0) { P.accept_len[b] = tau; P.next_token[b] = y; }
}

}  // namespace sv
