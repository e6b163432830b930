// The drafting step of the outer loop of speculative decoding (Alg. 3, "sample X_1 .. X_gamma from M_s")
// for a model whose conditional distributions are handed over as rows of logits: one token per row
// from softmax(logits / T), Y = min{x : C_x > u * C_total} with C the running sum in vocabulary order
// (the same convention as the draw of the correction token).
//
// One read of the row.  A row is cut into units of 64 * 32 contiguous logits, a wave takes a stretch of neighbouring
// units: it loads the next unit (sixteen-byte loads, 1 KB per instruction) while it turns the one before into
// exponentials against an integer shift of the unit's own, and keeps each unit's (largest scaled logit, sum) in one of
// its lanes.  The waves' totals meet in LDS once; every wave then knows which wave's stretch holds u * C_total, and that
// wave finds the unit from its lanes, reads that one unit again and walks it.  Sums are formed in double throughout
// (exponentials are float), recombined through exact powers of two.
//
// What bounds it: the bytes where there are rows for the whole device (2048 rows of 128256 bf16 logits: 91 us, 5.8 TB/s;
// float32 161 us, 6.5 TB/s); with fewer rows the vector instructions of the one compute unit a row has (64 such rows: 13.6
// us, about 8 of them in the sweep).  The kernel before this one gave each thread a contiguous stretch (uncoalesced) and
// read the row three times: 255 us for the 64 rows, 7497 for the 2048.
#pragma once

#include "fused.hpp"

namespace sv {

constexpr int kSampleUnit = kWave * kLaneSmall;          // logits per unit
// Rows of at most this many logits go to one thread each (81920 rows of 2: 7.4 us, launch included, against 88 with a
// wave per row), up to 512 to sixteen lanes (65536 rows of 100: 9.4 against 71), up to a unit to a wave (65536 rows of
// 1000: 40 against 244).
constexpr int kSampleSerial = 32;
// Sixteen waves per row are a row's shortest time (64 rows of 128256 bf16 logits: 13.6 us against 15.4 with eight waves);
// four let the draws of some rows run under the sweeps of others once every compute unit has several rows (512 rows 32.1 us with
// sixteen, 31.8 with four; 4096 rows of 32000: 49 with four).  Rows of up to four units have no work for more than four.
constexpr int kSampleManyRows = 512;
// With scratch memory the units of a row go to any compute unit, for a second launch (about 2 us): worth it for rows wide
// enough to keep one compute unit busy for longer than that, until the rows fill the device by themselves.  One workgroup
// per row / two launches, bf16: V = 32000: 64 rows 6.3 / 7.1 us; V = 50257: 8 rows 8.2 / 7.0, 64 9.0 / 8.0, 128 9.5 / 9.1, 256 10.1 / 11.1;
// V = 128256: 1 row 12.7 / 6.8, 64 13.4 / 8.8, 256 17.0 / 15.9; V = 256000: 64 22.1 / 11.0, 512 50.4 / 46.2; float32 alike.
constexpr int kSampleMinSplit = 24;                          // units of a row: from more than this on
constexpr int kSampleSplitUnits = 8 * kWave;                 // ... to this many (V <= 1 Mi)
constexpr int kSampleSplitRows = 4;                          // rows: up to this many per unit

// (largest scaled logit, sum of the exponentials relative to its integer shift) of a stretch of the row.
struct SampleEntry {
    float m;
    double z;
    // another stretch's added, through exact powers of two
    __device__ __forceinline__ void add(const SampleEntry &other)
    {
        if (!(other.m > -INFINITY)) return;
        const float top = fmaxf(m, other.m);
        z = (m > -INFINITY ? ldexp(z, (int)(shift_of(m) - shift_of(top))) : 0.0) + ldexp(other.z, (int)(shift_of(other.m) - shift_of(top)));
        m = top;
    }
    __device__ __forceinline__ double relative_to(float M) const { return m > -INFINITY ? ldexp(z, (int)(shift_of(m) - shift_of(M))) : 0.0; }
};

// Entries of the calls on the null stream that bring no scratch memory: the null stream exists once per device, is never
// destroyed nor captured, and what runs on it runs in turn, so that one array is enough for all of them and every GPU that the
// library runs on has its own (a call's two launches must follow each other there: the host holds a lock over them).
constexpr int kSampleOwnEntries = 1 << 18;                   // 4 MiB
__device__ SampleEntry g_null_stream_entries[kSampleOwnEntries];
// Calls on it of up to this many workgroups have one launch: their entries are words that announce themselves, three each (entry_word).
// Two launches / one, us: 1 row of 128256 bf16 logits 7.8 / 5.3, 8 rows 8.3 / 5.7, 64 rows (1024 workgroups) 8.1 / 7.3,
// float32 10.0 / 9.2; 64 rows of 202267, float32 (1600) 13.1 / 12.9; beyond, the workgroups that wait are in the way of others: 64 rows of 256000,
// float32 (2048) 14.8 / 15.4, 200 rows of 128256 bf16 (3200) 13.2 / 15.4.
constexpr int kSampleOneLaunch = 1536;
constexpr int kSampleOneUnits = 4 * kWave;                   // ... of rows of up to this many units (V = 1000003: 2 rows 7.4 / 7.7 us)
// A word is the call's number, never 0, above 32 bits of the entry (its largest logit; the two halves of its sum), and counts for the call
// of that number only: what the waves of a call whose wait ran out left behind (below) is nobody's.  Otherwise zero between calls.
constexpr int kEntryWords = 3;
__device__ u64 g_null_stream_words[kEntryWords * kSampleOneLaunch * kWaves];
__device__ __forceinline__ u64 entry_word(const SampleEntry &e, int n, unsigned call)
{
    const u64 z = (u64)__double_as_longlong(e.z);
    return (u64)call << 32 | (n == 0 ? __float_as_uint(e.m) : (unsigned)(n == 1 ? z : z >> 32));
}
__device__ __forceinline__ SampleEntry unpack_entry(u64 m, u64 lo, u64 hi)
{
    return {__uint_as_float((unsigned)m), __longlong_as_double((long long)(hi << 32 | (lo & 0xffffffffull)))};
}

// One unit of a row as loaded -> its entry (every lane gets it).  `left`: logits of the row from the unit's start on.
template <typename T>
__device__ __forceinline__ SampleEntry sweep_unit(RawSlice<T, false, kLaneSmall> &raw, int left, float k)
{
    constexpr int LANE = kLaneSmall;
    float x[LANE];
    unpack_slice<T, false, LANE>(0, left, raw, x);
    float m = x[0];
#pragma unroll
    for (int j = 1; j < LANE; ++j) m = fmaxf(m, x[j]);
    SampleEntry e;
    e.m = wave_max(m * k);
    const float shift = shift_of(e.m);
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < LANE; ++j) acc[j & 1] += (double)fast_exp2(__builtin_fmaf(x[j], k, -shift));
    double z0, z1;
    halves_sum_f64(acc[0] + acc[1], z0, z1);
    e.z = z0 + z1;
    return e;
}

// The same entry, vector by vector from a second look at the unit: slow, and in few registers (`unit`: the unit's start).
template <typename T>
__device__ __forceinline__ SampleEntry sweep_unit_slowly(const T *unit, int left, float k)
{
    constexpr int LANE = kLaneSmall, kVec = ElemTraits<T>::kVec;
    const int lane = threadIdx.x & 63;
    SampleEntry e = {-INFINITY, 0.0};
    double acc[2] = {0.0, 0.0};
    float x[kVec], m = -INFINITY, shift = 0.f;
#pragma unroll 1
    for (int step = 0; step < 2 * (LANE / kVec); ++step) {
        const int at = ((step & (LANE / kVec - 1)) * kWave + lane) * kVec;
        const uint4 raw = load_raw<T, false, true>(unit, left, at);
        unpack_raw<T, false>(raw, left, at, x);
        if (step < LANE / kVec) {
#pragma unroll
            for (int j = 0; j < kVec; ++j) m = fmaxf(m, x[j]);
            if (step == LANE / kVec - 1) { e.m = wave_max(m * k); shift = shift_of(e.m); }
        } else {
#pragma unroll
            for (int j = 0; j < kVec; ++j) acc[j & 1] += (double)fast_exp2(__builtin_fmaf(x[j], k, -shift));
        }
    }
    double z0, z1;
    halves_sum_f64(acc[0] + acc[1], z0, z1);
    e.z = z0 + z1;
    return e;
}

// The token, by one wave: units `from` to `end` of the row again, in vocabulary order (vector, lane, element), weights
// relative to `shift`, the first whose running sum exceeds t (else the last with weight, token 0 if there is none).
template <typename T>
__device__ __forceinline__ int walk_units(const T *row, int V, float k, float shift, double t, int from, int end)
{
    constexpr int LANE = kLaneSmall, kVec = ElemTraits<T>::kVec, kNV = LANE / kVec;
    const int lane = threadIdx.x & 63;
    int y = -1, last_positive = -1;
    for (int unit = from; unit < end && y < 0; ++unit) {
        const int at = unit * kSampleUnit, left = V - at;
        RawSlice<T, false, LANE> raw;
        issue_loads<T, false, LANE>(row + at, 0, left, raw);
        float x[LANE];
        unpack_slice<T, false, LANE>(0, left, raw, x);
#pragma unroll
        for (int v = 0; v < kNV; ++v) {
            if (y >= 0) continue;
            double mine = 0.0;
#pragma unroll
            for (int e = 0; e < kVec; ++e) {
                float &wgt = x[v * kVec + e];
                wgt = fast_exp2(__builtin_fmaf(wgt, k, -shift));
                mine += (double)wgt;
                if (wgt > 0.f) last_positive = at + (v * kWave + lane) * kVec + e;
            }
            const double inc = wave_scan(mine);
            const u64 here = __ballot(inc > t);
            if (here) {
                const int l = __ffsll((long long)here) - 1;
                double run = inc - mine;
                int e_hit = -1, e_last = 0;
#pragma unroll
                for (int e = 0; e < kVec; ++e) {
                    const float wgt = x[v * kVec + e];
                    run += (double)wgt;
                    if (wgt > 0.f) e_last = e;
                    if (e_hit < 0 && run > t) e_hit = e;
                }
                // (scan and walk may round differently: then the lane's last token with weight)
                y = at + (v * kWave + l) * kVec + __builtin_amdgcn_readlane(e_hit < 0 ? e_last : e_hit, l);
            }
            t -= read_lane_double(inc, kWave - 1);
        }
    }
    if (y < 0) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) last_positive = max(last_positive, __shfl_xor(last_positive, off, kWave));
        y = last_positive < 0 ? 0 : last_positive;
    }
    return y;
}

// Rows of more than one unit: one workgroup of WPR waves per row.
template <typename T, int WPR>
__global__ __launch_bounds__(WPR * kWave)
void sample_rows_kernel(const T *logits, int V, float k, const float *uniforms, int32_t *tokens)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t r = blockIdx.x;
    const T *const row = logits + r * (size_t)V;
    const float u = load_uniform(uniforms + r);

    // the wave's entries (at most one per lane): `span` units each, neighbours
    const int units = (V - 1) / kSampleUnit + 1;
    const int span = (units - 1) / (WPR * kWave) + 1;
    const int entries = (units - 1) / span + 1;
    const int per = (entries - 1) / WPR + 1;
    const int first_unit = min((long long)w * per * span, (long long)units), end_unit = min((long long)(w + 1) * per * span, (long long)units);

    SampleEntry own = {-INFINITY, 0.0};                      // lane j: the wave's entry j
    {
        // (a unit is addressed from its own start: offsets stay small whatever V is)
        auto issue = [&](int unit, RawSlice<T, false, kLaneSmall> &raw) {
            const int at = unit * kSampleUnit;
            issue_loads<T, false, kLaneSmall>(row + at, 0, V - at, raw);
        };
        RawSlice<T, false, kLaneSmall> raw, next;
        if (first_unit < end_unit) issue(first_unit, raw);
        int entry = 0, in_entry = 0;
        for (int unit = first_unit; unit < end_unit; ++unit) {
            if (unit + 1 < end_unit) issue(unit + 1, next);
            const SampleEntry e = sweep_unit<T>(raw, V - unit * kSampleUnit, k);
            if (lane == entry) own.add(e);
            if (++in_entry == span) { in_entry = 0; ++entry; }
            raw = next;
        }
    }

    // ---- the waves' totals, relative to the integer shift of the wave's largest
    const float Mw = wave_max(own.m);
    const double z_lane = own.relative_to(Mw);
    const double inc_lane = wave_scan(z_lane);
    __shared__ float wave_m[WPR];
    __shared__ double wave_z[WPR];
    if (lane == 0) { wave_m[w] = Mw; wave_z[w] = read_lane_double(inc_lane, kWave - 1); }
    __syncthreads();
    const SampleEntry of_wave = {lane < WPR ? wave_m[lane] : -INFINITY, wave_z[lane & (WPR - 1)]};
    const float M = wave_max(of_wave.m);
    const double z = of_wave.relative_to(M);
    const double inc = wave_scan(z);
    double t;                                                // what is left of u * C_total where the wave's stretch begins
    if (locate_entry(z, inc, (double)u * read_lane_double(inc, kWave - 1), t) != w) return;
    // ---- the entry of the wave's stretch, then the token
    const int entry = locate_entry(z_lane, inc_lane, ldexp(t, (int)(shift_of(M) - shift_of(Mw))), t);
    const float shift = shift_of(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(own.m), entry)));
    const int from = first_unit + entry * span;
    const int y = walk_units(row, V, k, shift, ldexp(t, (int)(shift_of(Mw) - shift)), from, min(from + span, end_unit));
    if (lane == 0) tokens[r] = y;
}

// For rows too few to fill the device: every wave sweeps one unit and leaves its entry; one wave per row then scans them (up
// to kSampleSplitUnits units, a stretch of neighbours per lane), finds the unit and walks it: in a launch of its own, from `entries` [rows, units]
// (NULL: the null stream's); or (ONE, calls on the null stream) as the first wave of the row's last workgroup, which waits for the words
// of the others and clears them.  Where that wait runs out (another kernel holds the compute units for seconds), it forms the missing entries itself.
template <typename T, int PER>
__device__ __forceinline__ int draw_from_entries(const T *row, int V, int units, int per, float k, float u, const SampleEntry (&mine)[PER])
{
    const int lane = threadIdx.x & 63;
    SampleEntry own = {-INFINITY, 0.0};
#pragma unroll
    for (int j = 0; j < PER; ++j) if (j < per) own.add(mine[j]);
    const float M = wave_max(own.m);
    const double z = own.relative_to(M), inc = wave_scan(z);
    double t;
    const int holder = locate_entry(z, inc, (double)u * read_lane_double(inc, kWave - 1), t);
    // the unit among the holder's neighbours: the first whose running sum exceeds t, else its last with weight
    int unit = 0;
    double left = INFINITY, running = 0.0;
    float m_unit = -INFINITY;
    bool found = false;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (j < per) {
            const double zj = mine[j].relative_to(M);
            if (!found && zj > 0.0) {
                unit = lane * per + j;
                m_unit = mine[j].m;
                if (running + zj > t) { found = true; left = t - running; }
            }
            running += zj;
        }
    unit = __builtin_amdgcn_readlane(unit, holder);
    const float shift = shift_of(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(m_unit), holder)));
    left = ldexp(read_lane_double(left, holder), (int)(shift_of(M) - shift));
    return walk_units(row, V, k, shift, left, unit, unit + 1);
}

template <typename T, bool ONE>
__global__ __launch_bounds__(kThreads)
void sample_units_kernel(const T *logits, int V, int units, float k, const float *uniforms, int32_t *tokens, SampleEntry *entries, unsigned call, int spin_limit)
{
    constexpr int kPer = kSampleOneUnits / kWave;
    const int lane = threadIdx.x & 63, unit = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kWaves + (threadIdx.x >> 6)));
    const size_t r = blockIdx.y;
    if (unit >= units) return;
    const T *const row = logits + r * (size_t)V;
    const int at = unit * kSampleUnit;
    RawSlice<T, false, kLaneSmall> raw;
    issue_loads<T, false, kLaneSmall>(row + at, 0, V - at, raw);
    const SampleEntry e = sweep_unit<T>(raw, V - at, k);
    if constexpr (!ONE) {
        if (lane == 0) (entries ? entries : g_null_stream_entries)[r * units + unit] = e;
    } else {
        u64 *const words = g_null_stream_words + kEntryWords * r * units;
        if (lane < kEntryWords) st_u64(words + kEntryWords * unit + lane, entry_word(e, lane, call));
        if (blockIdx.x != gridDim.x - 1 || threadIdx.x >= kWave) return;
        const float u = load_uniform(uniforms + r);
        const int per = (units - 1) / kWave + 1;
        // (lanes without an entry of their own look at the last one, which is waited for anyway)
        u64 m[kPer], lo[kPer], hi[kPer];
        for (int spins = 0;; ++spins) {
            int missing = 0;                                 // bit j: the lane's entry j
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                m[j] = lo[j] = hi[j] = 0;
                if (j < per) {
                    const u64 *const word = words + kEntryWords * min(lane * per + j, units - 1);
                    m[j] = ld_u64(word); lo[j] = ld_u64(word + 1); hi[j] = ld_u64(word + 2);
                }
            }
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (j < per && ((unsigned)(m[j] >> 32) != call || (unsigned)(lo[j] >> 32) != call || (unsigned)(hi[j] >> 32) != call)) missing |= 1 << j;
            if (!__any(missing != 0)) break;
            __builtin_amdgcn_s_sleep(6);                 // (looks in quick succession hold up the writes to the lines they look at: 8 rows of 128256 logits 6.1 us with 1, 5.7 with 6)
            if (spins < spin_limit) continue;
            // (the words that a late wave will write, the same; nothing of it is prepared in front of the wait)
            for (int n = 0; n < units; ++n) {
                asm volatile("" : "+s"(n));
                if ((__builtin_amdgcn_readlane(missing, n / per) >> n % per & 1) == 0) continue;
                const SampleEntry again = sweep_unit_slowly<T>(row + n * kSampleUnit, V - n * kSampleUnit, k);
                if (lane < kEntryWords) st_u64(words + kEntryWords * n + lane, entry_word(again, lane, call));
            }
        }
        SampleEntry mine[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) mine[j] = j < per && lane * per + j < units ? unpack_entry(m[j], lo[j], hi[j]) : SampleEntry{-INFINITY, 0.0};
        for (int n = lane; n < kEntryWords * units; n += kWave) st_u64(words + n, 0);
        const int y = draw_from_entries(row, V, units, per, k, u, mine);
        if (lane == 0) tokens[r] = y;
    }
}
template <typename T>
__global__ __launch_bounds__(kWave)
void sample_finish_kernel(const T *logits, int V, int units, float k, const float *uniforms, const SampleEntry *entries, int32_t *tokens)
{
    constexpr int kPer = kSampleSplitUnits / kWave;
    const int lane = threadIdx.x;
    const size_t r = blockIdx.x;
    const float u = load_uniform(uniforms + r);
    const int per = (units - 1) / kWave + 1;
    if (!entries) entries = g_null_stream_entries;
    SampleEntry mine[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        mine[j] = {-INFINITY, 0.0};
        if (j < per && lane * per + j < units) mine[j] = entries[r * units + lane * per + j];
    }
    const int y = draw_from_entries(logits + r * (size_t)V, V, units, per, k, u, mine);
    if (lane == 0) tokens[r] = y;
}

// Rows of at most G * 32 logits: G lanes per row, the whole row in their registers, nothing read twice.
template <typename T, int G>
__global__ __launch_bounds__(kThreads)
void sample_small_rows_kernel(const T *logits, int rows, int V, float k, const float *uniforms, int32_t *tokens)
{
    constexpr int kVec = ElemTraits<T>::kVec, kNV = kLaneSmall / kVec;
    const int lane = threadIdx.x & 63, l = lane & (G - 1);
    const long long at = ((long long)blockIdx.x * kThreads + threadIdx.x) / G;
    const bool mine = at < rows;                                              // (lanes beyond the last row work on it too and write nothing)
    const size_t r = mine ? (size_t)at : (size_t)rows - 1;
    const T *const row = logits + r * (size_t)V;
    const int nv = (V - 1) / (G * kVec) + 1;                                  // vectors of a lane that reach into the row
    uint4 raw[kNV];
#pragma unroll
    for (int v = 0; v < kNV; ++v)
        if (v < nv) raw[v] = load_raw<T, false, true>(row, V, (v * G + l) * kVec);
    const float u = uniforms[r];
    float x[kNV * kVec], m = -INFINITY;
#pragma unroll
    for (int v = 0; v < kNV; ++v)
        if (v < nv) {
            if (v + 1 < nv) unpack_vec<T>(raw[v], x + v * kVec);              // (only a row's last vectors reach beyond it)
            else unpack_raw<T, false>(raw[v], V, (v * G + l) * kVec, x + v * kVec);
#pragma unroll
            for (int e = 0; e < kVec; ++e) m = fmaxf(m, x[v * kVec + e]);
        }
    const float shift = shift_of(group_max<G>(m * k));
#pragma unroll
    for (int v = 0; v < kNV; ++v)
        if (v < nv) {
#pragma unroll
            for (int e = 0; e < kVec; ++e) x[v * kVec + e] = fast_exp2(__builtin_fmaf(x[v * kVec + e], k, -shift));
        }
    const int y = draw_in_group<G, kNV, kVec>([&](int j) { return x[j]; }, nv, [&](double total) { return (double)u * total; });
    if (l == 0 && mine) tokens[r] = y;
}

// Rows of a handful of logits (the toy models of Sec. 2): one thread per row; the row's three readings after the first
// come from the cache.
template <typename T>
__global__ __launch_bounds__(kThreads)
void sample_short_rows_kernel(const T *logits, int rows, int V, float k, const float *uniforms, int32_t *tokens)
{
    const long long r = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (r >= rows) return;
    const T *row = logits + (size_t)r * (size_t)V;
    float m = -INFINITY;
    for (int x = 0; x < V; ++x) m = fmaxf(m, logit_as_float(row + x));
    const float shift = shift_of(m * k);
    double total = 0.0;
    for (int x = 0; x < V; ++x) total += (double)fast_exp2(__builtin_fmaf(logit_as_float(row + x), k, -shift));
    const double target = (double)uniforms[r] * total;
    double c = 0.0;
    int y = -1, last_positive = 0;
    for (int x = 0; x < V && y < 0; ++x) {
        const float e = fast_exp2(__builtin_fmaf(logit_as_float(row + x), k, -shift));
        c += (double)e;
        if (e > 0.f) last_positive = x;
        if (c > target) y = x;
    }
    tokens[r] = y < 0 ? last_positive : y;
}

}  // namespace sv
