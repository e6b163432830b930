// Calls of few resident sets (rows of at most 32 workgroups); at the end, rows that one workgroup holds, in calls of any size beyond what
// runs at once.  Most calls whose workgroups all run at once, and most float32 ones, go to the kernel in together.hpp, which has one trip less
// and holds more registers; those here have the others.
//
// Such a call is as long as its chain of dependent trips through device memory.  The large kernel (fused.hpp) hands a
// row pair's results to ONE wave, the row's leader: it collects the row's partial sums of S_i, judges the position's
// accept test and, for the draw of the token that follows if tau = i, reads the chunk that holds the token a second
// time; the leader of the sequence's last row pair then collects one word per position.  That is the cheapest way for
// a call whose rows follow each other in waves over the device, and two trips too many for a call that is over
// when its one wave of workgroups is.  Here every workgroup of a row pair keeps its exponentials in registers until the
// row's S_i is known, and EVERY workgroup's first wave reads all partial sums of the row: all of them form the same S_i
// from the same words in the same order, judge the same test and find the same place for u * S_i - and the workgroup
// that holds that place draws the token from its registers and publishes the position's word itself.  The last
// target row works the same way (its workgroups know from the ratios alone whether every token is accepted); the first
// wave of its last workgroup writes tau and Y and hands the words over to the next call.  Words, copies, call count:
// the large kernel's (so calls of either may follow each other on one workspace); the arithmetic of the sweeps too.
#pragma once

#include "fused.hpp"

namespace sv {

constexpr int kResidentMaxGroups = 32;        // workgroups per row: one poll of a wave covers the words of both rows
// Up to how many times the workgroups that the device keeps resident the library takes this kernel by itself.  Its
// workgroups hold their registers until the row's S_i is there, which costs nothing while everything runs at once and
// more and more as workgroups queue for the compute units; the large kernel has its row leaders read the logits once more
// instead.  Measured, this kernel / the large one (before the calls of one set, and most float32 ones, had the kernel of together.hpp, which is faster
// there: the line is the same for both):
//   bf16, V = 128256: gamma = 2: 1.3 sets 18 / 22 us, 2.4 sets 27 / 26; gamma = 8: 1.2 sets 19 / 21, 2.4 sets 27 / 29,
//   3.9 sets 40 / 37; gamma = 16: 2.3 sets 28 / 29, 3.8 sets 38 / 35
//   bf16, V = 32000: gamma = 2: 2.4 sets 26 / 26; gamma = 8: 2.4 sets 28 / 31, 4.0 sets 40 / 40; gamma = 16: 4.0 sets 39 / 42
//   float32 (a quarter fewer workgroups resident), V = 128256: gamma = 4: 1.2 sets 21 / 23, 2.3 sets 32 / 30; gamma = 16:
//   2.4 sets 33 / 33; V = 32000: gamma = 8: 1.3 sets 23 / 25, 2.4 sets 34 / 34
//   with draft lengths of the sequences' own (half of the workgroups have nothing to do): bf16, V = 32000, gamma = 8: 2.4 sets
//   22 / 26, 4.0 sets 28 / 28; V = 100277, gamma = 6: 3.4 sets 27.8 / 29.0
// The line is the same with and without the report of every S_i, so that the report changes no decision (it favours the
// large kernel: gamma = 8, V = 128256: 2.4 sets 32 / 30).
inline double resident_sets(int gamma, int groups, bool f32, bool own_lengths, bool aligned)
{
    const double narrow = groups < 16 ? 1.0 + (16 - groups) / 40.0 : 1.0;
    const double sets = (f32 ? 1.8 : 2.5) * (own_lengths ? 1.25 : 1.0), few_positions = 1.0 + 0.5 * gamma;
    double line = (sets < few_positions ? sets : few_positions) * narrow;
    // What that line misses for rows of a few workgroups, where the large kernel has less to gain, above all where rows are not
    // 16-byte aligned: float32, gamma = 8, 2.9 sets, V = 30001 35.2 / 36.8; aligned float32: gamma = 8, V = 32000, 2.7 sets 35.0 / 33.9, 2.6 sets 33.2 / 34.9,
    // gamma = 4 33.2 / 32.6; own lengths, gamma = 8, 3.0 sets 26.4 / 27.5.
    // Rows of one and of two workgroups have the kernel of one workgroup per row (below, rows_verify_kernel) beyond this line, and up to 12288 logits before it too: there
    // it only decides whether that kernel may hand w_i on in a chain, which matters to neither side (1884 calls from where the chain would begin, up to the line: 0.3 % over the faster of
    // the two on average).  Rows of 12289 ... 16384 logits, the kernels for few resident sets / that one: float32, 162 of 8 over 12808 (2.8 sets) 29.9 / 30.9, 220 of 8 over 14016
    // (3.9) 41.0 / 40.7, not aligned 122 of 12 over 14613 (3.1) 37.2 / 39.2, own lengths 150 of 12 over 15200 (3.8) 29.2 / 29.5; bf16 189 of 6 over 14064 (2.1) 23.5 / 24.5, 188 of 8 over
    // 13776 (2.6) 27.7 / 26.8, not aligned 184 of 8 over 15349 (2.6) 29.8 / 30.1, 363 of 6 over 13717 (4.0) 42.2 / 41.5, own lengths 263 of 6 over 14096 (2.9) 23.4 / 24.1, 205 of 12 over
    // 13392 (4.2) 25.4 / 23.9.  Over 3800 such calls of 0.9 to 4.5 sets the line is 0.7 % over the faster of the two on average; worst, by 4 to 6 %, float32 of own lengths and not aligned
    // from 3 to 4 sets.
    if (groups == 1 || (!aligned && groups <= (f32 ? 4 : 2))) line = line > 3.0 ? line : 3.0;
    else if (f32 && groups <= 4 && gamma >= 6) { const double to = own_lengths ? 3.0 : groups == 2 ? 2.8 : 2.6; line = line > to ? line : to; }
    // ... and where it goes beyond three sets though the large kernel is the faster one there: bf16, V = 24000, 3.2 sets, gamma = 4 32.2 / 29.3, gamma = 6
    // 32.7 / 30.8; own lengths, V = 65536, 3.6 sets, gamma = 4 27.3 / 25.9, gamma = 8 25.3 / 23.8
    if (own_lengths ? groups >= 5 : groups >= 3 && gamma < 8) line = line < 3.0 ? line : 3.0;
    return line;
}
constexpr double kResidentSetsForced = 3.0;   // at least this where the testing hook asks for this kernel or that of together.hpp

// (largest scaled logit, sum) of four words, one per lane of a quad: every lane of the quad gets the combination
// (fixed order, the sums through exact powers of two).
__device__ __forceinline__ u64 quad_word(u64 w)
{
    const float m = stat_shift(w);
    float M = fmaxf(m, __int_as_float(dpp_shift<0xB1>(__float_as_int(m))));            // quad_perm:[1,0,3,2]
    M = fmaxf(M, __int_as_float(dpp_shift<0x4E>(__float_as_int(M))));                   // quad_perm:[2,3,0,1]
    double z = m > -INFINITY ? ldexp((double)stat_sum(w), (int)(shift_of(m) - shift_of(M))) : 0.0;
    z += dpp_shift_double<0xB1>(z);
    z += dpp_shift_double<0x4E>(z);
    return pack_stat(M, (float)z);
}

// A wave-uniform float as a double, converted where it is used: left to itself the compiler converts the uniforms at
// the top of the kernel and keeps the doubles in vector registers through both sweeps.
__device__ __forceinline__ double late_double(float v)
{
    asm volatile("" : "+s"(v));
    return (double)v;
}

// The draw inside one wave's unit of 64 * LANE logits (vocabulary order inside the unit: vector, lane, element), in two
// steps.  First, by any wave: `sums` holds the unit's weights summed per (vector, lane), in that order (64 * NV floats
// in LDS); every lane takes NV consecutive ones, one scan over the wave finds the lane and that lane the entry whose
// running sum exceeds t first (else the last entry with any weight).  Returns the entry, `t_e`: what is left of t
// inside it.
template <int NV>
__device__ __forceinline__ int locate_in_sums(const float *sums, double t, double &t_e)
{
    const int lane = threadIdx.x & 63;
    float ent[NV], mine = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) { ent[j] = sums[lane * NV + j]; mine += ent[j]; }
    const double inc = wave_scan((double)mine);
    const u64 hit = __ballot(inc > t), nz = __ballot(mine > 0.f);
    const int hl = hit ? __ffsll((long long)hit) - 1 : nz ? 63 - __clzll((long long)nz) : 0;
    int entry = 0;
    double left = INFINITY;
    if (lane == hl) {
        double r = inc - (double)mine, before = 0.0;
        int last_j = 0, found = -1;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            if (found < 0 && hit && r + (double)ent[j] > t) { found = j; before = r; }
            if (ent[j] > 0.f) last_j = j;
            r += (double)ent[j];
        }
        entry = hl * NV + (found < 0 ? last_j : found);
        if (found >= 0) left = t - before;
    }
    t_e = read_lane_double(left, hl);
    return __builtin_amdgcn_readlane(entry, hl);
}
// Then, by the wave that holds the unit's weights in registers (weight(j), j the register index): the element of that
// entry - KVEC weights of one lane - whose running sum exceeds t_e first, else the last one with any weight.
template <int KVEC, int LANE, typename F>
__device__ __forceinline__ int walk_entry(F weight, int entry, double t_e)
{
    constexpr int kNV = LANE / KVEC;
    const int dv = entry / kWave, dl = entry % kWave;        // the entry's vector and lane
    int cand = 0;
    if ((int)(threadIdx.x & 63) == dl) {
        float wgt[KVEC];
#pragma unroll
        for (int v = 0; v < kNV; ++v)
            if (v == dv) {
#pragma unroll
                for (int e = 0; e < KVEC; ++e) wgt[e] = weight(v * KVEC + e);
            }
        double r = 0.0;
        int last_e = 0, found = -1;
#pragma unroll
        for (int e = 0; e < KVEC; ++e) {
            r += (double)wgt[e];
            if (wgt[e] > 0.f) last_e = e;
            if (found < 0 && r > t_e) found = e;
        }
        cand = found < 0 ? last_e : found;
    }
    return __builtin_amdgcn_readlane(cand, dl);
}
// Both steps by the wave that holds the weights (`sums`: 64 * LANE / KVEC floats that only this wave uses meanwhile).
// Returns the token's offset inside the unit.
template <int KVEC, int LANE, typename F>
__device__ __forceinline__ int draw_in_unit(F weight, double t, float *sums)
{
    constexpr int kNV = LANE / KVEC;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < kNV; ++v) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < KVEC; ++e) s += weight(v * KVEC + e);
        sums[v * kWave + lane] = s;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double t_e;
    const int entry = locate_in_sums<kNV>(sums, t, t_e);
    return entry * KVEC + walk_entry<KVEC, LANE>(weight, entry, t_e);
}

// Grid (x, y, z) = (workgroup of the row, sequence, slot): slot i is row pair i, slot gamma the sequence's last target
// row; x runs fastest in the start order, so a row's workgroups start together and a position's before the next one's.
// (bf16 rows: held to the registers of five waves per SIMD, as the large kernel is - in calls of more than one resident
// set a fifth of the workgroups more run at a time: B = 20 of the shape above 28.3 -> 25.5 us)
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ElemTraits<T>::kVec == 8 ? SV_WAVES_SMALL : 4)))
void resident_verify_kernel(const FusedParams P)
{
    constexpr int LANE = kLaneSmall, kUnitLogits = kWave * LANE, kVec = ElemTraits<T>::kVec;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = blockIdx.x, b = blockIdx.y, slot = blockIdx.z, nwg = gridDim.x;
    const int gamma = P.gamma, V = P.V, nu = P.nu;
    const float k = P.k;
    long long *stamps = nullptr;
#ifdef SV_PROFILE
    if (P.prof) stamps = P.prof + (((size_t)b * (gamma + 1) + slot) * nwg + c) * 16;      // one record per workgroup
#endif
    SV_STAMP(0);
    int gb = gamma;
    if (P.draft_lens) { gb = load_uniform(P.draft_lens + b); gb = gb < 1 ? 1 : gb > gamma ? gamma : gb; }
    const bool last_row = slot == gamma;
    const bool unused = !last_row && slot >= gb;
    const int i = last_row ? gb : slot;
    const size_t seq_d = (size_t)b * gamma, seq_u = (size_t)b * (gamma + 1);
    const size_t drow = seq_d + (last_row ? 0 : i);
    const T *rowA = static_cast<const T *>(P.target) + (seq_u + i) * P.tstride;
    const T *rowB = static_cast<const T *>(P.draft) + drow * P.dstride;
    const int unit_first = (c * kWaves + wave) * kUnitLogits;

    // the rows' loads first: they depend on the arguments only
    RawSlice<T, ALIGNED, LANE> rawA, rawB;
    if (!unused) {
        issue_loads<T, ALIGNED, LANE>(rowA, unit_first, V, rawA);
        if (!last_row) issue_loads<T, ALIGNED, LANE>(rowB, unit_first, V, rawB);
    }
    asm volatile("" ::: "memory");
    const int magic_word = load_uniform(P.header + kHdrMagic);
    const unsigned par = (unsigned)load_uniform(P.gen + b) & 1u;
    if (magic_word != P.magic) {
        if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
            for (int s = threadIdx.x; s < P.B; s += kThreads) { P.accept_len[s] = -1; P.next_token[s] = -1; }
        return;
    }
    // every slot's words are cleared, in the copy that this call does not use, by the first wave of the slot's last
    // workgroup (an unused position's in both copies: the other one may hold an earlier, longer call's words)
    const bool leader = wave == 0 && c == nwg - 1;
    if (unused) {
        if (leader) { const bool rw = row_words_used<kLaneSmall>(P.header); clear_row_words(P, P.words, b, slot, rw); clear_row_words(P, words_of(P, 1), b, slot, rw); }
        return;
    }
    if (leader) clear_row_words(P, words_of(P, par ^ 1u), b, slot, slot != P.gamma && row_words_used<kLaneSmall>(P.header));
    const Words W = words_of(P, par);
    const bool token_algo = P.algo == kToken;

    __shared__ u64 wave_words[2][kWaves];
    __shared__ float wave_part[kWaves];
    __shared__ double row_values[8];
    __shared__ int row_flag[4];
    __shared__ float draw_sums[kWaves][kWave * (LANE / kVec)];      // per wave: its unit's weights summed per (vector, lane)
    __shared__ float wave_scale[kWaves];
    // what the first wave keeps across the second sweep lives here meanwhile (its registers are the whole workgroup's):
    // the row's words as its lanes hold them, the words of log2 r_{i+1} and log2 r_i, log2 w_i, the row's largest
    // scaled target logit, whether the position can become tau
    __shared__ u64 kept_grp[kWave], kept_words[4];
    __shared__ float kept_Mp;
    __shared__ int draw_entry;
    bool gave_up = false;

    // =================================================================== the sequence's last target row
    if (last_row) {
        // Y comes from it where every token is accepted, which its workgroups see from the ratios; the leader writes
        // tau and Y (Y from the word of position tau, or from the word that the workgroup holding it publishes)
        u64 *const y_word = W.lw + seq_d + gb - 1;                    // (a word this kernel has no other use for)
        u64 rw = 0, res_first = 0;
        float eta_g = 0.f, u = 0.f;
        if (wave == 0) {
            eta_g = load_uniform(P.uniforms + seq_u + gb - 1);
            u = load_uniform(P.uniforms + seq_u + gb);
            rw = ld_u64(W.ratio + seq_d + (lane < gb ? lane : 0));
            if (leader) res_first = ld_u64(W.rowres + seq_d + (lane < gb ? lane : 0));
        }
        float xa[LANE], shiftA;
        unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawA, xa);
        const u64 stA = first_sweep_row(xa, k, shiftA);
        if (lane == 0) wave_words[0][wave] = stA;
        __syncthreads();
        bool all_accepted = false;
        double w_last = 1.0;
        u64 pl = 0;                                                   // the row's words (lane e: workgroup e's)
        const u64 *const pl_word = W.plast + (size_t)b * nu + (lane < nwg ? lane : 0);
        if (wave == 0) {
            const u64 own_plast = quad_word(wave_words[0][lane & 3]);
            if (lane == 0) st_u64(W.plast + (size_t)b * nu + c, own_plast);
            rw = wait_word(W.ratio + seq_d + (lane < gb ? lane : 0), rw, lane < gb, P.spin_limit, gave_up);
            // (by now the row's other workgroups have published theirs: a look that the waits below pick up)
            pl = lane == c ? own_plast : ld_u64(pl_word);
            if (token_algo) {
                const u64 failed = __ballot(lane < gb && !ratio_passes(rw));
                all_accepted = failed == 0;
            } else {
                const double lw_g = read_lane_double(weights_from_ratios(P.algo, rw, gb), gb - 1);
                w_last = exp2_precise(P.algo == kGreedy ? fmin(lw_g, 100.0) : lw_g);
                all_accepted = (double)eta_g < fmin(w_last, 1.0);                      // eta_gamma < h_gamma = w_gamma
            }
            int role = 0;
            if (all_accepted && !gave_up) {
                // the row's words, all of them: where u * (the row's sum) falls
                const u64 pw = pl = wait_word(pl_word, pl, lane < nwg, P.spin_limit, gave_up);
                const float m = lane < nwg ? stat_shift(pw) : -INFINITY;
                const float M = wave_max(m);
                const double z = m > -INFINITY ? ldexp((double)stat_sum(pw), (int)(shift_of(m) - shift_of(M))) : 0.0;
                const double inc = wave_scan(z);
                double t_in;
                const int e = locate_entry(z, inc, late_double(u) * read_lane_double(inc, kWave - 1), t_in);
                if (e == c && !gave_up) {
                    // ... and in which of the workgroup's four units
                    const u64 ww = wave_words[0][lane & 3];
                    const float mw = lane < kWaves ? stat_shift(ww) : -INFINITY;
                    const double zw = mw > -INFINITY ? ldexp((double)stat_sum(ww), (int)(shift_of(mw) - shift_of(M))) : 0.0;
                    double t_w;
                    const int wv = locate_entry(zw, wave_scan(zw), t_in, t_w);
                    // (into the units of that wave's exponentials, which are relative to its own shift)
                    const float m_wv = stat_shift(read_lane_u64(ww, wv));
                    if (lane == 0) { row_flag[1] = wv; row_values[0] = ldexp(t_w, (int)(shift_of(M) - shift_of(m_wv))); }
                    role = 1;
                }
            }
            if (gave_up) { report_gave_up(P); if (lane == 0) st_u64(y_word, kPoison64); }
            if (lane == 0) row_flag[0] = role;
        }
        __syncthreads();
        if (row_flag[0] == 1 && wave == row_flag[1]) {
            const int off = draw_in_unit<kVec, LANE>([&](int j) { return xa[j]; }, row_values[0], draw_sums[wave]);
            if (lane == 0) st_u64(y_word, pack_rowres(true, min(unit_first + off, V - 1)));
        }
        if (!leader) return;

        // ---- the leader: tau and Y
        int tau, y;
        if (all_accepted) {
            tau = gb;
            y = rowres_token(wait_word(y_word, P.spin_limit, gave_up));
        } else if (token_algo) {
            // tau is the length of the leading run of passed tests; its position's word holds the token
            const u64 failed = __ballot(lane < gb && !ratio_passes(rw));
            tau = __ffsll((long long)failed) - 1;
            y = rowres_token(wait_word(W.rowres + seq_d + tau, read_lane_u64(res_first, tau), true, P.spin_limit, gave_up));
        } else {
            // one word per position: bit l, whether the test of position l passes (none at position 0); tau is the
            // last position whose test passes, else 0
            const u64 res = wait_word(W.rowres + seq_d + (lane < gb ? lane : 0), res_first, lane < gb, P.spin_limit, gave_up);
            const u64 tests = __ballot(lane < gb && rowres_passes(res)) & ~1ull;
            tau = tests ? 63 - __clzll((long long)tests) : 0;
            y = rowres_token(read_lane_u64(res, tau));
        }
        if (P.debug_out && lane == 0) {
            float *d = P.debug_out + (seq_u + gb) * 3;       // S_gamma = w_gamma: q_gamma == 0
            d[0] = (float)w_last; d[1] = (float)w_last;
            d[2] = token_algo ? (float)exp2_precise(fmin(unpack_ratio(read_lane_u64(rw, gb - 1)), 0.0)) : (float)fmin(w_last, 1.0);
        }
        // every workgroup of the sequence has read the call count once the last target row's words are there (the row
        // pairs' workgroups published words that the ratios, which this wave has, were made of)
        wait_word(pl_word, pl, lane < nwg, P.spin_limit, gave_up);
        if (gave_up) report_gave_up(P);
        if (lane == 0) {
            P.accept_len[b] = gave_up ? -1 : tau;
            P.next_token[b] = gave_up ? -1 : max(y, 0);          // (rows of which the arithmetic makes NaNs: the two rules above need not agree there)
            __hip_atomic_store(P.gen + b, (int)(par ^ 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        SV_STAMP(6);
        return;
    }

    // =================================================================== a row pair
    const int n_prev = i;                                     // ratios that w_i is made of
    u64 wt = 0;                                               // first wave, lane j: the word of log2 r_{j+1}
    float eta_i = 0.f, eta_next = 0.f, u = 0.f;
    int tok = 0;
    if (wave == 0) {
        eta_i = load_uniform(P.uniforms + seq_u + (n_prev > 0 ? n_prev - 1 : 0));
        eta_next = load_uniform(P.uniforms + seq_u + n_prev);
        u = load_uniform(P.uniforms + seq_u + gb);
        tok = load_uniform(P.tokens + drow);
        wt = ld_u64(W.ratio + seq_d + (lane <= n_prev ? lane : 0));
    }
    // ---- first sweep (as in the large kernel): exponentials stay in xa / xb
    float xa[LANE], xb[LANE];
    float shiftA, shiftB;
    unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawA, xa);
    const u64 stA = first_sweep_row(xa, k, shiftA);
    unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawB, xb);
    uint32_t ya_bits = 0, yb_bits = 0;
    if (leader) { ya_bits = logit_bits(rowA + tok); yb_bits = logit_bits(rowB + tok); }
    const u64 stB = first_sweep_row(xb, k, shiftB);
    if (lane == 0) { wave_words[0][wave] = stA; wave_words[1][wave] = stB; }
    __syncthreads();
    SV_STAMP(1);

    if (wave == 0) {
        u64 grp = 0;                // the row's words (lanes 0..: the target row's, lanes 32..: the draft row's)
        float Mp = 0.f;
        double log2w = 0.0;
        u64 own_word = 0, prev_word = 0;
        bool candidate = true;
        publish_group_words(wave_words, W.pgrp + 2 * (drow * nwg + c), W.qgrp + 2 * (drow * nwg + c));
        // ---- L_p, L_q from the words of all workgroups of the row
        const int e = lane & 31;
        const bool need = e < nwg;
        const u64 *word = (lane < 32 ? W.pgrp : W.qgrp) + 2 * (drow * nwg + (need ? e : nwg - 1));
        grp = wait_word(word, ld_u64(word), need, P.spin_limit, gave_up);
        StatAcc acc;
        if (need) acc.add(grp);
        float Mq;
        halves_max(acc.m, Mp, Mq);
        double zp, zq;
        halves_sum_f64(acc.relative_to(lane < 32 ? Mp : Mq), zp, zq);
        // (the two side by side in the wave's halves)
        const double L = (double)shift_of(lane < 32 ? Mp : Mq) + log2_precise(lane < 32 ? zp : zq);
        const double Lp = read_lane_double(L, 0), Lq = read_lane_double(L, 32);
        SV_STAMP(7);
        if (leader) {
            // log2 r_{i+1} = log2 p_i(X_{i+1}) - log2 q_i(X_{i+1}) (see the large kernel for the correction by k_eps)
            const double ya = (double)logit_bits_as_float<T>(ya_bits), yb = (double)logit_bits_as_float<T>(yb_bits);
            const double lp = ya * P.kd - (Lp + P.k_eps * (double)Mp), lq = yb * P.kd - (Lq + P.k_eps * (double)Mq);
            const double lr = fmax(lp - lq, kLog2RatioFloor);
            own_word = pack_ratio(lr, token_algo && (double)eta_next < exp2_precise(fmin(lr, 0.0)));
            if (gave_up) report_gave_up(P);
            if (lane == 0) st_u64(W.ratio + drow, gave_up ? kPoison64 : own_word);
        }
        SV_STAMP(8);
        // ---- the ratios of the earlier positions, and this row's own (the leader has it already)
        wt = wait_word(W.ratio + seq_d + (lane <= n_prev ? lane : 0), wt, lane < n_prev || (lane == n_prev && !leader), P.spin_limit, gave_up);
        if (!leader) own_word = read_lane_u64(wt, n_prev);
        // (the scan's lane j depends on the lanes before it only: lane n_prev - 1 is this position's log2 w_i, lane n_prev the next one's)
        const bool looks_on = ElemTraits<T>::kVec == 8 && P.prune && !P.debug_out;
        double lw_next = -1.0;
        if (n_prev > 0 || looks_on) {
            const double lw = weights_from_ratios(P.algo, looks_on && lane == n_prev ? own_word : wt, looks_on ? n_prev + 1 : n_prev);
            if (looks_on) lw_next = read_lane_double(lw, n_prev);
            if (n_prev > 0) {
                log2w = read_lane_double(lw, n_prev - 1);
                prev_word = read_lane_u64(wt, n_prev - 1);
            }
        }
        SV_STAMP(9);
        candidate = can_become_tau(P.algo, i, log2w, eta_i);
        // S_i is formed where the position can become tau (position 0 always can) or the caller wants every S_i.  In calls of more row pairs than run at once also only where the
        // next test does not pass whatever S_{i+1} is (Alg. 2 / 4: w_{i+1} >= 1; Alg. 1: that test is judged with the ratio).  Before / now, us, bf16: 59 ragged of 16 over
        // 22739, Alg. 4, 29.7 / 28.2; 12 of 8 over 128256, Alg. 1, 17.2 / 16.7; 30 of 8 over 50257 22.0 / 21.5.  In calls of one set it frees nobody's place, and the scan that
        // position 0 needs for it is on the chain (2 ragged of 14 over 228689 13.0 / 13.2); nor in
        // float32 calls, which are of less than two sets (8 of 16 over 128256, Alg. 1, 26.6 / 26.6; 7 of 16 over 70848 14.6 / 14.9).
        const bool beyond = looks_on && (token_algo ? ratio_passes(own_word) : lw_next >= 0.0);
        const bool needed = (candidate && !beyond) || P.debug_out != nullptr || gave_up;
        if (token_algo) log2w = 0.0;                                // the residual of token verification is p - q
        if (P.algo == kGreedy) log2w = fmin(log2w, 100.0);          // keeps w p finite in float
        if (needed) {
            // the second sweep's row constants (see the large kernel)
            const double A = Lp - log2w, Ai = rint(A), Qi = rint(Lq);
            // (three powers side by side in three lanes: fq, frho and its inverse.  This, the two logarithms above and the one branch of the
            // sweep below, against one after the other and a select per term: 108 sequences of 2 drafted tokens and 30 001 entries bf16 15.7 ->
            // 15.2 us, 18 of 8 and 128 256 ragged 18.6 -> 17.9)
            const double dq = Qi - Lq, d = (Ai - A) - dq;
            const double x = exp2_precise(lane == 0 ? dq : lane == 1 ? d : -d);
            if (lane < 3) row_values[5 + lane] = x;
            if (lane == 0) { row_values[3] = Ai; row_values[4] = Qi; }
        } else if (leader && lane == 0) {
            // nothing more to say about tau than this (Alg. 2 / 4: the test fails; Alg. 1: how the test of X_{i+1} went)
            st_u64(W.rowres + drow, pack_rowres(token_algo && ratio_passes(own_word), -1));
        }
        if (gave_up) report_gave_up(P);
        if (needed) {
            kept_grp[lane] = grp;
            if (lane == 0) {
                kept_words[0] = own_word; kept_words[1] = prev_word; kept_words[2] = (u64)__double_as_longlong(log2w);
                kept_words[3] = candidate ? 1 : 0;
                kept_Mp = Mp;
                draw_entry = 0;       // (never left to chance: with NaN sums the two looks at from_p below need not agree)
            }
        }
        if (lane == 0) row_flag[0] = needed ? 1 : 0;
        SV_STAMP(2);
    }
    __syncthreads();
    if (!row_flag[0]) return;

    // ---- second sweep, from registers (as in the large kernel): terms in [0, 1] in units of the larger row factor
    const int ea = unit_exponent(shiftA, row_values[3]), eq = unit_exponent(shiftB, row_values[4]);
    const double rho = ldexp(row_values[6], ea - eq);
    const bool q_units = rho <= 1.0;
    const float factor = q_units ? (float)rho : -(float)ldexp(row_values[7], eq - ea);
    const float scale = q_units ? (float)ldexp(row_values[5], eq) : (float)ldexp(row_values[5] * row_values[6], ea);
    {
        // (the sums per vector stay behind in LDS: the draw, if it falls into this unit, starts from them.  One branch for the whole sweep, two
        // instructions per term)
        constexpr int kNV = LANE / kVec;
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
        if (lane == 0) { wave_part[wave] = acc; wave_scale[wave] = scale; }
    }
    __syncthreads();
    SV_STAMP(4);

    if (wave == 0) {
        // ---- the workgroup's share of S_i goes out; all shares of the row come in
        const float mine = (wave_part[0] + wave_part[1]) + (wave_part[2] + wave_part[3]);
        const unsigned own_part = gave_up ? kPoison32 : pack_partial(mine);
        if (lane == 0) st_u32(W.spart + drow * nu + c, own_part);
        const u64 own_word = kept_words[0], prev_word = kept_words[1];
        const double log2w = __longlong_as_double((long long)kept_words[2]);
        const bool candidate = kept_words[3] != 0;
        // (while the shares travel: what the accept test needs of w_i)
        const bool has_test = !token_algo && i > 0;
        const double one_minus_w = has_test ? one_minus_exp2(fmin(log2w, 0.0)) : 0.0;
        const unsigned sp = wait_word32(W.spart + drow * nu + (lane < nwg ? lane : 0), lane == c ? own_part : 0u, lane < nwg, P.spin_limit, gave_up);
        SV_STAMP(5);
        double z = lane < nwg ? (double)unpack_partial(sp) : 0.0;
        double inc = wave_scan(z);
        const double S_i = read_lane_double(inc, kWave - 1);
        // ---- the position's accept test (Alg. 2 / 4); Alg. 1: the test of X_{i+1} came with the ratio
        // (Alg. 2 / 4, position i >= 1: eta_i < h_i = S_i / (S_i + 1 - w_i), 1 where w_i >= 1 - see AcceptTest; judged
        // without the division)
        const bool test_passes = has_test && candidate && (log2w >= 0.0 || late_double(eta_i) * (S_i + one_minus_w) < S_i);
        const bool next_passes = ratio_passes(own_word);
        const bool own_passes = token_algo ? next_passes : test_passes;
        // the token that follows if this position becomes tau is drawn where it can
        const bool want = !gave_up && (token_algo ? candidate && !next_passes : i == 0 || own_passes);
        if (P.debug_out && leader && lane == 0) {
            float *d = P.debug_out + (seq_u + i) * 3;            // (w_i, S_i, h_i); Alg. 1 has no w, its h_i = min(r_i, 1)
            double h_i = has_test && log2w < 0.0 ? S_i / (S_i + one_minus_w) : 1.0;
            if (token_algo && i > 0) h_i = exp2_precise(fmin(unpack_ratio(prev_word), 0.0));
            d[0] = has_test ? (float)exp2_precise(log2w) : 1.f; d[1] = (float)S_i; d[2] = (float)h_i;
        }
        int role = 0;
        if (want) {
            // where u * S_i falls; a residual without any mass is drawn from p_i instead (weights: the exponentials)
            const bool from_p = !(S_i > 0.0);
            const float Mp = kept_Mp;
            const u64 grp = kept_grp[lane];
            if (from_p) {
                const float m = lane < nwg ? stat_shift(grp) : -INFINITY;
                z = m > -INFINITY ? ldexp((double)stat_sum(grp), (int)(shift_of(m) - shift_of(Mp))) : 0.0;
                inc = wave_scan(z);
            }
            double t_in;
            const int e = locate_entry(z, inc, late_double(u) * read_lane_double(inc, kWave - 1), t_in);
            if (e == c) {
                // ... in which of the workgroup's four units, and what is left of t in that unit's own units
                double t_w;
                int wv;
                if (from_p) {
                    const u64 ww = wave_words[0][lane & 3];
                    const float mw = lane < kWaves ? stat_shift(ww) : -INFINITY;
                    const double zw = mw > -INFINITY ? ldexp((double)stat_sum(ww), (int)(shift_of(mw) - shift_of(Mp))) : 0.0;
                    wv = locate_entry(zw, wave_scan(zw), t_in, t_w);
                    t_w = ldexp(t_w, (int)(shift_of(Mp) - shift_of(stat_shift(read_lane_u64(ww, wv)))));
                } else {
                    double before = 0.0;
                    int last_w = 0;
                    wv = -1; t_w = INFINITY;
#pragma unroll
                    for (int w = 0; w < kWaves; ++w) {
                        const double zw = (double)wave_part[w];
                        if (wv < 0 && before + zw > t_in) { wv = w; t_w = t_in - before; }
                        if (zw > 0.0) last_w = w;
                        before += zw;
                    }
                    if (wv < 0) wv = last_w;
                    // ... and at which (vector, lane) of that unit: its sums per vector are in LDS, in the terms' own
                    // units (the shares were scaled, the terms are not)
                    double t_e;
                    const int entry = locate_in_sums<LANE / kVec>(draw_sums[wv], t_w / (double)wave_scale[wv], t_e);
                    if (lane == 0) draw_entry = entry;
                    t_w = t_e;
                }
                if (lane == 0) { row_flag[1] = wv; row_flag[2] = from_p ? 1 : 0; row_flag[3] = own_passes ? 1 : 0; row_values[0] = t_w; }
                role = 1;
            }
        } else if (leader && lane == 0) {
            st_u64(W.rowres + drow, gave_up ? kPoison64 : pack_rowres(own_passes, -1));
        }
        if (gave_up) report_gave_up(P);
        if (lane == 0) row_flag[0] = role;
        SV_STAMP(10);
    }
    __syncthreads();
    SV_STAMP(11);
    if (row_flag[0] != 1 || wave != row_flag[1]) return;
    // ---- the wave that holds the token draws it from its registers and publishes the position's word
    int off;
    if (row_flag[2]) {
        off = draw_in_unit<kVec, LANE>([&](int j) { return xa[j]; }, row_values[0], draw_sums[wave]);
    } else {
        const int entry = __builtin_amdgcn_readfirstlane(draw_entry);      // (the same for the whole wave, and known to be)
        // (the terms once more: kept from the sweep, they would cost the kernel its registers)
        float f = factor;
        asm volatile("" : "+v"(f));
        off = entry * kVec + walk_entry<kVec, LANE>([&](int j) {
            return q_units ? __builtin_amdgcn_fmed3f(__builtin_fmaf(xa[j], f, -xb[j]), 0.f, 1.f)
                           : __builtin_amdgcn_fmed3f(__builtin_fmaf(xb[j], f, xa[j]), 0.f, 1.f); }, entry, row_values[0]);
    }
    // (a row of which the arithmetic makes NaNs still ends inside the vocabulary)
    if (lane == 0) st_u64(W.rowres + drow, pack_rowres(row_flag[3] != 0, min(unit_first + off, V - 1)));
    SV_STAMP(15);
}

// ------------------------------------------------------------------ rows that one workgroup holds
// The same for rows of at most 20480 logits, one workgroup per row (pair), WAVES waves each with as many neighbouring logits: a row's
// normalisers, its S_i and the place of its token never leave the workgroup (LDS and three barriers), and two kinds of words are left, the
// ratio (or the chain's log2 w, see the large kernel) on the way from position to position and what each position contributes to tau and Y.
// Calls of more workgroups than run at once take it (and some of fewer: rows_alone), also those that the large kernel would have.
// What bounds such calls is not their bytes but how many rows are under way: a row that begins a second workgroup of 8192 logits pays for its
// slot and its words whatever it holds (512 sequences of 4, bf16: V = 8192 22.9 us, V = 8200 31.3), and every row for the steps of single waves
// between its sweeps.  So the workgroup's width follows the row's: two waves (up to 4096 logits), four or eight (beyond 16384), 24 ... 64 logits per lane and
// row, and as many waves per SIMD as that leaves registers for.  Waves of 32 logits and as many as the row needs were slower where they do not divide over the
// four SIMDs (five: 1000 sequences of 8 over 9072 73.8 us, four of 40 58.5).  In 64 logits per lane only three waves per SIMD are left: rows beyond 12288 come
// here where they are many only (138 sequences of 7 over 15381 25.5 us, the other form 23.4; 300 38.5 / 40.1; 920 of 3 over 14912 41.0 / 45.6); eight waves
// of 40 again everywhere (120 of 8 over 17000 26.2 / 20.7 us, 600 83.4 / 70.0), of 48 nowhere (200 of 4 over 24000 25.1 / 25.1).
// The other kernels / this one, us, bf16 unless said: 1200 sequences of 4 over 3000 38.4 / 19.1, 800 of 8 over 5000 45.5 / 30.7, 2000 of 4 over 8192 64.3 / 50.4, 131 of
// 8 over 9072 19.1 / 14.5, 1000 of them 89.6 / 58.5; 744 of 5 over 11289 61.3 / 43.2; float32: 800 of 8 over 2500 53.4 / 28.7, 400 of 8 over 9072 58.8 / 42.9; with
// every S_i 600 of 8 over 9072 67.3 / 42.1.  Error against 64 bits over 360 such calls, rms: 9.2e-7 / 5.6e-7.
constexpr int kRowsMaxRow = 2 * kThreads * 40;
constexpr int kRowsMaxRowFew = kThreads * 48;   // in calls of few resident sets rows beyond, up to 16384 logits, do not come here
// Calls of few resident sets that take it (`workgroups` of 8192 logits, `resident` of together.hpp's at once; `together`: whether that kernel has
// the call else), from how many sixteenths of a resident set on (the kernel else / this one, us; the report of every S_i, which favours this one, decides nothing):
//   up to 4096 logits four, bf16: 39 of 8 over 2100 10.4 / 9.4, 102 12.2 / 10.1; float32 68 of 8 over 4000 11.2 / 10.6, 853 of 2 over 2049 26.5 / 14.3; beyond 3072, drafts of up to eleven, six
//   (bf16 53 of 6 over 3075, close models 11.2 / 11.6, 44 of 5 over 3678, others 10.2 / 9.9, float32 62 of 4 over 4073, close ones 11.5 / 12.2: 0.25 to 0.4 sets of close models 4 % slower);
//   up to 6144 drafts of twelve and more too (54 of 12 over 4529, bf16 12.5 / 10.2, 31 of 14 over 4480 10.0 / 9.1), others from nearly a set on: float32 230 of 3 over 5000 13.5 /
//   12.7, 153 11.8 / 11.8; up to 8192 from a set on (327 of 4 over 8001 25.5 / 21.6, 184 16.4 / 16.3), drafts of
//   twelve and more of Alg. 1, whose tests ask for no S_i, from four too (75 of 12 over 6900 12.0 / 11.5; Alg. 2 and 4 are faster here with poor drafts only, and slower by as much again with
//   good ones: bf16 33 of 13 over 6484, poor 11.3 / 11.0, 21 of 15 over 6345, good 11.8 / 12.9, 59 of 13 over 7680 11.3 / 12.4, float32 22 of 12 over 6562, good 12.6 / 13.7, 54 of 16 over
//   7168 14.6 / 15.7), own lengths from where that kernel's calls end (bf16 62 of 16 over 6853, good 13.6 / 14.3, 101 of 10 over 7896, poor 11.9 / 11.9), in float32 from 1.75 (94 of 12 over 7018 14.5 /
//   15.8, 127 of 9 over 8064 13.9 / 15.1, 138 of 12 over 7488 17.1 / 17.1, 304 of 6 over 6882 21.0 / 18.4; up to 6144 like the others: 139 of 7 over 4736 12.2 / 11.7, 312 of 6 over
//   4864 18.1 / 14.9, 341 of 8 over 5000 22.4 / 17.5);
//   beyond, where two workgroups become one, later: up to 10240 float32 62 of 8 over 9000 14.8 / 13.9, 34 11.3 / 11.9, own lengths, float32, from 1.6 (42 of 14 over 9721 14.3 / 15.2,
//   136 of 5 over 9369 15.9 / 16.6, 59 of 14 over 9938 16.6 / 16.6, 49 of 19 over 9668 16.2 / 15.5; bf16 ones gain from the first);
//   up to 12288, 48 logits per lane, from one and a half sets on (bf16 34 of 16 over 10688 12.5 / 13.4, 43 of 13 over 11072 12.3 / 13.8, 86 of 8 over 12004 18.1 / 14.9; float32
//   102 of 5 over 11000 15.5 / 16.5, 136 20.3 / 18.9; Alg. 1 58 of 12 over 11456, bf16 13.7 / 12.0, 107 of 5 over 10912 13.7 / 13.3), where sequences bring their own draft lengths, half of whose workgroups have
//   nothing to do, from two (bf16 74 of 9 over 11712 11.9 / 13.1, 76 of 8 over 11503 14.2 / 15.4, 72 of 14 over 10944 16.5 / 12.8; float32 97 of 8 over 11328 15.1 / 16.2, 149 of 6 over
//   10888 18.4 / 17.1); up to 17920 float32 60 of 8 over 18000 (1.6 sets) 19.5 / 18.8;
//   beyond, where the eighth wave has logits too, bf16 from about one and a half on (35 of 10 over 18785 15.2 / 17.4, 31 of 13 over 20031 16.1 / 17.2, 34 of 14 over 19136 17.0 / 14.5), own
//   lengths from two and a quarter (73 of 8 over 19633 15.2 / 18.0, 55 of 10 over 19116 13.3 / 15.1, 69 over 20096 20.6 / 17.2), not in float32 (79 of 6 over 19712, ragged 14.4 / 17.6, 54 of
//   12 over 20142 25.5 / 27.6, 59 of 14 over 19779 31.1 / 33.4); Alg. 1 with drafts of eight and more again sooner (28 of 16 over 19108 14.6 / 12.1, 32 of 12 over 19456 13.1 / 11.8; float32 55
//   of 14 over 18368 28.0 / 25.8; own lengths, bf16 43 of 16 over 18048 14.6 / 12.2, 39 of 9 over 19456 11.4 / 12.1).
inline bool rows_alone(long long workgroups, long long resident, int gamma, int V, bool f32, bool own_lengths, bool together, bool token_algo)
{
    if (V > kRowsMaxRow || (V > kRowsMaxRowFew && V <= kThreads * 64)) return false;
    int sixteenths = 0;
    if (V <= kThreads * 40) {
        if (!together) return true;
        if (V <= kThreads * 16) sixteenths = V > kThreads * 12 && gamma < 12 ? 6 : 4;
        else if (V <= kThreads * 24) sixteenths = gamma >= 12 ? 4 : 14;
        else if (V <= kThreads * 32) sixteenths = own_lengths ? (f32 ? 28 : 18) : gamma >= 12 && token_algo ? 4 : 16;
        else sixteenths = f32 && own_lengths ? 26 : 18;
    } else if (V <= kThreads * 48) {
        sixteenths = own_lengths ? 32 : token_algo ? 20 : 24;
    } else if (V <= 7 * kWave * 40) {
        sixteenths = together ? 24 : 0;
    } else if (token_algo && gamma >= 8) {
        sixteenths = own_lengths ? 34 : 20;
    } else {
        if (f32) return false;
        sixteenths = own_lengths ? 36 : 23;
    }
    return 16 * workgroups > sixteenths * resident;
}
// waves per SIMD of a form: by what it has to keep in registers, 2 LANE floats per lane and some thirty more
template <int LANE> constexpr int kRowsWavesPerSimd = LANE == 24 ? 6 : LANE == 32 ? 5 : LANE <= 48 ? 4 : 3;

// Clears a sequence's words in one copy (one wave), as the layout of the other kernels has them: whoever used that copy, the next call finds it clean.
__device__ __forceinline__ void clear_sequence_words(const FusedParams &P, const Words &W, int b, bool row_words)
{
    const int lane = threadIdx.x & 63, G = P.gamma, nu = P.nu, nwg = nu / kWaves;
    const size_t drow = (size_t)b * G;
    for (int e = lane; e < G; e += kWave) { st_u64(W.ratio + drow + e, 0); st_u64(W.lw + drow + e, 0); st_u64(W.rowres + drow + e, 0); }
    for (int e = lane; e < 2 * G * nwg; e += kWave) st_u64(W.pgrp + 2 * drow * nwg + e, 0);
    for (int e = lane; e < G * nu; e += kWave) { st_u32(W.spart + drow * nu + e, 0); if (row_words) st_u64(W.pstat + drow * nu + e, 0); }
    for (int e = lane; e < nu; e += kWave) st_u64(W.plast + (size_t)b * nu + e, 0);
    for (int e = lane; e < nwg; e += kWave) st_u64(W.lseen + (size_t)b * nwg + e, 0);
}

// A wave's part of its row's mass, relative to the largest scaled logit M of the row: lanes 0 .. 3 the target row's, 4 .. 7 the draft row's.
template <int WAVES> constexpr int kRowsSegment = WAVES > 4 ? 16 : 4;
template <int WAVES>
__device__ __forceinline__ double rows_mass(const u64 (&wave_words)[2][WAVES], float &M)
{
    constexpr int SEG = kRowsSegment<WAVES>;
    const int lane = threadIdx.x & 63;
    const u64 w = (lane & (SEG - 1)) < WAVES ? wave_words[lane / SEG & 1][lane & (WAVES - 1)] : kEmptyUnit;
    const float m = stat_shift(w);
    M = group_max<SEG>(m);
    return m > -INFINITY ? ldexp((double)stat_sum(w), (int)(shift_of(m) - shift_of(M))) : 0.0;
}

// Grid (x, y) = (sequence in group, group * (gamma + 1) + slot): position-major inside groups of sequences, as the large kernel's.  A workgroup
// waits for earlier positions of its sequence only (the last target row: for all).
template <typename T, bool ALIGNED, int WAVES, int LANE, bool CHAIN>
__global__ __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(kRowsWavesPerSimd<LANE>)))
void rows_verify_kernel(const FusedParams P)
{
    constexpr int kVec = ElemTraits<T>::kVec, kNV = LANE / kVec;
    constexpr int kSums = LANE > 32 ? LANE / 8 : 4;               // (partial sums of no more than eight terms, as in the other kernels)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gamma = P.gamma, V = P.V;
    const float k = P.k;
    int grp = 0, slot = blockIdx.y;
    if (P.B > P.group_seqs) { grp = (int)__umulhi(blockIdx.y, P.inv_slots); slot = blockIdx.y - grp * (gamma + 1); }
    const int b = grp * P.group_seqs + blockIdx.x;
    if (b >= P.B) return;
    int gb = gamma;
    if (P.draft_lens) { gb = load_uniform(P.draft_lens + b); gb = gb < 1 ? 1 : gb > gamma ? gamma : gb; }
    const bool last_row = slot == gamma;
    if (!last_row && slot >= gb) return;                          // (a position that the sequence does not use)
    const int i = last_row ? gb : slot;
    const size_t seq_d = (size_t)b * gamma, seq_u = (size_t)b * (gamma + 1);
    const size_t drow = seq_d + (last_row ? 0 : i);
    const T *rowA = static_cast<const T *>(P.target) + (seq_u + i) * P.tstride;
    const T *rowB = static_cast<const T *>(P.draft) + drow * P.dstride;
    const int unit_first = wave * kWave * LANE;
    const bool idle = unit_first >= V;                            // (none of the row's logits are this wave's)
    // the rows' loads first: they depend on the arguments only (a last target row waits until it is known to be needed)
    RawSlice<T, ALIGNED, LANE> rawA, rawB;
    if (!last_row && !idle) {
        issue_loads<T, ALIGNED, LANE>(rowA, unit_first, V, rawA);
        issue_loads<T, ALIGNED, LANE>(rowB, unit_first, V, rawB);
    }
    asm volatile("" ::: "memory");
    const int magic_word = load_uniform(P.header + kHdrMagic);
    const unsigned par = (unsigned)load_uniform(P.gen + b) & 1u;
    if (magic_word != P.magic) {
        if (blockIdx.x == 0 && blockIdx.y == 0)
            for (int s = threadIdx.x; s < P.B; s += WAVES * kWave) { P.accept_len[s] = -1; P.next_token[s] = -1; }
        return;
    }
#define SV_WORDS words_of(P, launder(par))
    const bool token_algo = P.algo == kToken;

    __shared__ u64 wave_words[2][WAVES];
    __shared__ float wave_part[WAVES], wave_scale[WAVES];
    __shared__ double row_values[8];
    __shared__ int row_flag[4];
    __shared__ float draw_sums[WAVES][kWave * kNV];      // per wave: its unit's weights summed per (vector, lane)
    __shared__ u64 kept_words[4];                                 // what the first wave keeps across the second sweep
    bool gave_up = false;

    // where t = u * (the row's sum of exponentials) falls: the unit, and what is left of t in that unit's own terms
    auto place_in_row = [&](float u, double &t_w) {
        float M;
        const double z = rows_mass(wave_words, M);
        const double zp = lane < WAVES ? z : 0.0, inc = wave_scan(zp);
        const int wv = locate_entry(zp, inc, late_double(u) * read_lane_double(inc, kWave - 1), t_w);
        const float Mp = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(M), 0));
        t_w = ldexp(t_w, (int)(shift_of(Mp) - shift_of(stat_shift(wave_words[0][wv]))));
        return wv;
    };

    // =================================================================== the sequence's last target row
    if (last_row) {
        // Y comes from it where every token is accepted, which its first wave sees from the weights alone: only then is it read.  That
        // wave writes tau and Y and hands the words over to the next call.
        double w_last = 1.0;
        u64 rw = 0, res = 0;
        float u = 0.f;
        if (wave == 0) {
            const Words W = SV_WORDS;
            const u64 *const word = CHAIN ? W.lw + seq_d + gb - 1 : W.ratio + seq_d + (lane < gb ? lane : 0);
            rw = ld_u64(word);
            res = ld_u64(W.rowres + seq_d + (lane < gb ? lane : 0));
            const float eta_g = load_uniform(P.uniforms + seq_u + gb - 1);
            u = load_uniform(P.uniforms + seq_u + gb);
            rw = wait_word(word, rw, CHAIN || lane < gb, P.spin_limit, gave_up);
            const double lw_g = CHAIN ? unpack_ratio(read_lane_u64(rw, 0)) : read_lane_double(weights_from_ratios(P.algo, rw, gb), gb - 1);
            if (!token_algo) w_last = exp2_precise(P.algo == kGreedy ? fmin(lw_g, 100.0) : lw_g);
            const bool all = token_algo ? lw_g > 0.5 * kLog2RatioFloor : (double)eta_g < fmin(w_last, 1.0);      // eta_gamma < h_gamma = w_gamma
            if (lane == 0) row_flag[0] = all && !gave_up ? 1 : 0;
        }
        __syncthreads();
        const bool all_accepted = row_flag[0] != 0;
        if (wave == WAVES - 1) clear_sequence_words(P, words_of(P, par ^ 1u), b, load_uniform(P.header + kHdrRowWords) != 0);
        int y = -1;
        if (all_accepted) {
            float xa[LANE], shiftA;
            u64 stA = kEmptyUnit;
            if (!idle) {
                issue_loads<T, ALIGNED, LANE>(rowA, unit_first, V, rawA);
                unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawA, xa);
                stA = first_sweep_row<LANE, kSums>(xa, k, shiftA);
            }
            if (lane == 0) wave_words[0][wave] = stA;
            __syncthreads();
            if (wave == 0) {
                double t_w;
                const int wv = place_in_row(u, t_w);
                if (lane == 0) { row_flag[1] = wv; row_values[0] = t_w; }
            }
            __syncthreads();
            if (wave == row_flag[1]) {
                const int off = draw_in_unit<kVec, LANE>([&](int j) { return xa[j]; }, row_values[0], draw_sums[wave]);
                if (lane == 0) row_flag[2] = min(unit_first + off, V - 1);
            }
            __syncthreads();
            y = row_flag[2];
        }
        if (wave != 0) return;
        const Words W = SV_WORDS;
        // one word per position: bit l, whether the test of position l passes (none at position 0; Alg. 1: that of X_{l+1})
        res = wait_word(W.rowres + seq_d + (lane < gb ? lane : 0), res, lane < gb, P.spin_limit, gave_up);
        const u64 flags = __ballot(lane < gb && rowres_passes(res));
        int tau;
        if (all_accepted) tau = gb;
        else if (token_algo) { tau = __ffsll((long long)~flags) - 1; if (tau < 0 || tau >= gb) tau = gb - 1; }      // leading run of passes
        else tau = (flags & ~1ull) ? 63 - __clzll((long long)(flags & ~1ull)) : 0;                                      // last position whose test passes
        if (!all_accepted) y = max(rowres_token(read_lane_u64(res, tau)), 0);
        if (gave_up) report_gave_up(P);
        if (lane == 0) {
            P.accept_len[b] = gave_up ? -1 : tau;
            P.next_token[b] = gave_up ? -1 : y;
            if (P.debug_out) {
                float *d = P.debug_out + (seq_u + gb) * 3;       // S_gamma = w_gamma: q_gamma == 0
                d[0] = (float)w_last; d[1] = (float)w_last;
                // (Alg. 1's h_gamma is the last position's to write: it has the ratio)
                if (!token_algo) d[2] = (float)fmin(w_last, 1.0);
            }
            // (every workgroup that read the call count has published its position's word since)
            __hip_atomic_store(P.gen + b, (int)(par ^ 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }

    // =================================================================== a row pair
    u64 wt = 0;                                                   // first wave: the chain's word of log2 w_i; else lane j: the word of log2 r_{j+1}
    float eta_i = 0.f, eta_next = 0.f;
    int tok = 0;
    if (wave == 0) {
        eta_i = load_uniform(P.uniforms + seq_u + (i > 0 ? i - 1 : 0));
        eta_next = load_uniform(P.uniforms + seq_u + i);
        tok = load_uniform(P.tokens + drow);
    }
    // ---- first sweep (as in the large kernel): exponentials stay in xa / xb
    float xa[LANE], xb[LANE];
    float shiftA = kNoWeight, shiftB = kNoWeight;
    u64 stA = kEmptyUnit, stB = kEmptyUnit;
    if (!idle) {
        unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawA, xa);
        stA = first_sweep_row<LANE, kSums>(xa, k, shiftA);
        unpack_slice<T, ALIGNED, LANE>(unit_first, V, rawB, xb);
    }
    uint32_t ya_bits = 0, yb_bits = 0;
    if (wave == 0) { ya_bits = logit_bits(rowA + tok); yb_bits = logit_bits(rowB + tok); }
    if (!idle) stB = first_sweep_row<LANE, kSums>(xb, k, shiftB);
    if (lane == 0) { wave_words[0][wave] = stA; wave_words[1][wave] = stB; }
    __syncthreads();

    if (wave == 0) {
        const Words W = SV_WORDS;
        const u64 *const w_word = CHAIN ? W.lw + seq_d + (i > 0 ? i - 1 : 0) : W.ratio + seq_d + (lane < i ? lane : 0);
        wt = ld_u64(w_word);
        // ---- L_p, L_q, log2 r_{i+1} = log2 p_i(X_{i+1}) - log2 q_i(X_{i+1}) (see the large kernel for the correction by k_eps)
        float M;
        constexpr int SEG = kRowsSegment<WAVES>;
        const double z = group_sum<SEG>(rows_mass(wave_words, M));
        const double L = (double)shift_of(M) + log2_precise(z);
        const double Lp = read_lane_double(L, 0), Lq = read_lane_double(L, SEG);
        const double y = (double)logit_bits_as_float<T>(lane < SEG ? ya_bits : yb_bits);
        const double l = y * P.kd - (L + P.k_eps * (double)M);
        const double lr = fmax(read_lane_double(l, 0) - read_lane_double(l, SEG), kLog2RatioFloor);
        const u64 own_word = pack_ratio(lr, token_algo && (double)eta_next < exp2_precise(fmin(lr, 0.0)));
        const bool next_passes = ratio_passes(own_word);
        if (!CHAIN && lane == 0) st_u64(W.ratio + drow, own_word);
        // ---- log2 w_i, log2 w_{i+1}
        double log2w = 0.0, lw_next;
        if (i > 0) wt = wait_word(w_word, wt, CHAIN || lane < i, P.spin_limit, gave_up);
        if (CHAIN) {
            if (i > 0) log2w = unpack_ratio(read_lane_u64(wt, 0));
            lw_next = unpack_ratio(pack_ratio(next_weight(P.algo, log2w, unpack_ratio(own_word), next_passes), false));
            if (lane == 0) st_u64(W.lw + drow, gave_up ? kPoison64 : pack_ratio(lw_next, false));
        } else {
            // (one scan for both: lane i - 1 does not depend on lane i)
            const double lw = weights_from_ratios(P.algo, lane == i ? own_word : wt, i + 1);
            if (i > 0) log2w = read_lane_double(lw, i - 1);
            lw_next = read_lane_double(lw, i);
        }
        // Whether S_i matters: the position can become tau (position 0 always can), and the next test does not pass whatever its uniform is
        // (Alg. 1: tau is the position whose next test fails)
        const bool candidate = can_become_tau(P.algo, i, log2w, eta_i);
        const bool counts = candidate && !(token_algo ? next_passes : lw_next >= 0.0);
        const bool needed = counts || P.debug_out != nullptr || gave_up;
        if (token_algo) log2w = 0.0;                                // the residual of token verification is p - q
        if (P.algo == kGreedy) log2w = fmin(log2w, 100.0);          // keeps w p finite in float
        if (needed) {
            // the second sweep's row constants (see the large kernel), the three powers side by side in three lanes
            const double A = Lp - log2w, Ai = rint(A), Qi = rint(Lq);
            const double dq = Qi - Lq, d = (Ai - A) - dq;
            const double x = exp2_precise(lane == 0 ? dq : lane == 1 ? d : -d);
            if (lane < 3) row_values[5 + lane] = x;
            if (lane == 0) {
                row_values[3] = Ai; row_values[4] = Qi;
                kept_words[0] = own_word; kept_words[1] = (u64)__double_as_longlong(log2w); kept_words[2] = (candidate ? 1 : 0) | (counts ? 2 : 0);
            }
        } else if (lane == 0) {
            // nothing more to say about tau than this (Alg. 2 / 4: the test fails, or does not count; Alg. 1: how the test of X_{i+1} went)
            st_u64(W.rowres + drow, pack_rowres(token_algo && next_passes, -1));
        }
        if (gave_up) report_gave_up(P);
        if (lane == 0) row_flag[0] = needed ? 1 : 0;
    }
    __syncthreads();
    if (!row_flag[0]) return;

    // ---- second sweep, from registers (as in the large kernel): terms in [0, 1] in units of the larger row factor
    const int ea = unit_exponent(shiftA, row_values[3]), eq = unit_exponent(shiftB, row_values[4]);
    const double rho = ldexp(row_values[6], ea - eq);
    const bool q_units = rho <= 1.0;
    const float factor = q_units ? (float)rho : -(float)ldexp(row_values[7], eq - ea);
    const float scale = q_units ? (float)ldexp(row_values[5], eq) : (float)ldexp(row_values[5] * row_values[6], ea);
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
        if (idle) acc = 0.f;
        else if (q_units) sums([&](int j) { return __builtin_amdgcn_fmed3f(__builtin_fmaf(xa[j], factor, -xb[j]), 0.f, 1.f); });
        else sums([&](int j) { return __builtin_amdgcn_fmed3f(__builtin_fmaf(xb[j], factor, xa[j]), 0.f, 1.f); });
        if (!idle) acc = wave_sum(acc * scale);
        if (lane == 0) { wave_part[wave] = acc; wave_scale[wave] = scale; }
    }
    __syncthreads();

    if (wave == 0) {
        const Words W = SV_WORDS;
        const u64 own_word = kept_words[0];
        const double log2w = __longlong_as_double((long long)kept_words[1]);
        const bool candidate = (kept_words[2] & 1) != 0, counts = (kept_words[2] & 2) != 0;
        const bool has_test = !token_algo && i > 0;
        const double one_minus_w = has_test ? one_minus_exp2(fmin(log2w, 0.0)) : 0.0;
        const double z = lane < WAVES ? (double)wave_part[lane] : 0.0, inc = wave_scan(z);
        const double S_i = read_lane_double(inc, kWave - 1);
        // ---- the position's accept test (Alg. 2 / 4: eta_i < h_i = S_i / (S_i + 1 - w_i), 1 where w_i >= 1, judged without the division);
        // Alg. 1: the test of X_{i+1} came with the ratio
        const bool test_passes = has_test && candidate && (log2w >= 0.0 || late_double(eta_i) * (S_i + one_minus_w) < S_i);
        const bool next_passes = ratio_passes(own_word), own_passes = token_algo ? next_passes : test_passes;
        const bool want = !gave_up && counts && (token_algo || i == 0 || test_passes);
        if (P.debug_out && lane == 0) {
            float *d = P.debug_out + (seq_u + i) * 3;            // (w_i, S_i, h_i); Alg. 1 has no w, its h_{i+1} = min(r_{i+1}, 1)
            d[0] = has_test ? (float)exp2_precise(log2w) : 1.f; d[1] = (float)S_i;
            if (!token_algo || i == 0) d[2] = has_test && log2w < 0.0 ? (float)(S_i / (S_i + one_minus_w)) : 1.f;
            if (token_algo) d[5] = (float)exp2_precise(fmin(unpack_ratio(own_word), 0.0));
        }
        int role = 0;
        if (want) {
            // where u * S_i falls: the unit, and the (vector, lane) of it whose sums are in LDS, in the terms' own units (the shares were
            // scaled, the terms are not); a residual without any mass is drawn from p_i instead (weights: the exponentials)
            const float u = load_uniform(P.uniforms + seq_u + gb);
            double t_w;
            int wv;
            if (!(S_i > 0.0)) {
                wv = place_in_row(u, t_w);
                role = 2;
            } else {
                double t_in;
                wv = locate_entry(z, inc, late_double(u) * S_i, t_in);
                const int entry = locate_in_sums<kNV>(draw_sums[wv], t_in / (double)wave_scale[wv], t_w);
                if (lane == 0) row_flag[3] = entry;
                role = 1;
            }
            if (lane == 0) { row_flag[1] = wv; row_flag[2] = own_passes ? 1 : 0; row_values[0] = t_w; }
        } else if (lane == 0) {
            st_u64(W.rowres + drow, gave_up ? kPoison64 : pack_rowres(own_passes, -1));
        }
        if (lane == 0) row_flag[0] = role;
    }
    __syncthreads();
    const int role = row_flag[0];
    if (role == 0 || wave != row_flag[1]) return;
    // ---- the wave that holds the token draws it from its registers and publishes the position's word
    int off;
    if (role == 2) {
        off = draw_in_unit<kVec, LANE>([&](int j) { return xa[j]; }, row_values[0], draw_sums[wave]);
    } else {
        const int entry = __builtin_amdgcn_readfirstlane(row_flag[3]);
        // (the terms once more: kept from the sweep, they would cost the kernel its registers)
        float f = factor;
        asm volatile("" : "+v"(f));
        off = entry * kVec + walk_entry<kVec, LANE>([&](int j) {
            return q_units ? __builtin_amdgcn_fmed3f(__builtin_fmaf(xa[j], f, -xb[j]), 0.f, 1.f)
                           : __builtin_amdgcn_fmed3f(__builtin_fmaf(xb[j], f, xa[j]), 0.f, 1.f); }, entry, row_values[0]);
    }
    // (a row of which the arithmetic makes NaNs still ends inside the vocabulary)
    if (lane == 0) st_u64(SV_WORDS.rowres + drow, pack_rowres(row_flag[2] != 0, max(0, min(unit_first + off, V - 1))));
#undef SV_WORDS
}

}  // namespace sv
