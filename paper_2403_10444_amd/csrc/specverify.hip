// Draft verification for speculative decoding on gfx950: the C ABI of include/specverify.h.
//
// Host side only: argument checks, workspace layout and kernel launches.  The kernels are in
// fused.hpp (one launch, every logit read from HBM once; the default), resident.hpp and together.hpp (calls of few
// resident sets, of one), tiny.hpp (one workgroup per sequence), packed.hpp (several sequences to a workgroup) and staged.hpp (four launches, no limit
// on the vocabulary size); probs.hpp holds the kernels for inputs that are probabilities already,
// sample.hpp those of the drafting step.

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <atomic>
#include <chrono>
#include <mutex>

#include "../../include/specverify.h"
#include "common.hpp"
#include "fused.hpp"
#include "probs.hpp"
#include "sample.hpp"
#include "staged.hpp"
#include "tiny.hpp"
#include "packed.hpp"
#include "resident.hpp"
#include "together.hpp"

namespace {

using namespace sv;

constexpr int kDefaultSpinLimit = 1 << 20;

// Threads of one launch along x.  HIP refuses none beyond 2^32 - 1 but runs their number modulo 2^32, so a call of more is cut into
// launches of whole sequences or rows (2^24 + 3 rows of 2049 logits to draw from, 256 threads each: three rows were drawn).
constexpr unsigned long long kMaxLaunchThreads = 0xffffffffull;

std::atomic<int> g_path{0};                       // 0 auto, 1 staged, 2 fused, 5 one workgroup per sequence, 7 the kernels for calls of few resident sets, 8 / 9 that of together.hpp / of resident.hpp (testing hook; 3 / 4 / 6: fused with small / large units / small ones without the chain)
std::atomic<int> g_spin_limit{kDefaultSpinLimit};
std::atomic<int> g_last_kernel{0};                  // the kernels of the last verification call that was launched (SV_KERNEL_*)
std::atomic<int> g_last_chain{-1};                  // whether the last call on the fused kernel had the chain
std::atomic<int> g_last_together{-1};               // whether the last call of few resident sets had the kernel of together.hpp
std::atomic<int> g_last_form{0};                    // which form of its kernel the last verification call had (SV_FORM_*)
std::atomic<int> g_lane{0};                        // 0 auto, 32 or 64: logits per lane of the fused kernel's units (testing hook)
std::atomic<int> g_chain{-1};                      // -1 auto, 0 / 1: whether the fused kernel's leaders hand w_i on in a chain (testing hook)
#ifdef SV_PROFILE
std::atomic<long long *> g_prof{nullptr};          // device buffer for per-workgroup timestamps (tuning builds only)
#endif

struct Layout {
    size_t total;
    // fused path
    bool fused_ok;
    int nu;                       // wave chunks per row = 4 * workgroups per row
    size_t fused_grid;            // workgroups of the fused kernel
    size_t control_words;         // header, call counts and both copies of the words that cross waves: in ints, at offset 0
    size_t off_gen, copy_bytes;   // the call counts; bytes from one copy of the words to the other
    size_t off_ratio, off_lw, off_rowres, off_pstat, off_plast, off_pgrp, off_qgrp, off_spart, off_lseen;     // copy 0
    // staged path
    int nchunks;                  // chunks of kChunk logits per row
    size_t rows_total;
    size_t off_stats, off_coef, off_sspart;
};

bool make_layout(int32_t B, int32_t gamma, int32_t V, Layout &L)
{
    if (B < 1 || gamma < 1 || V < 1 || gamma > SV_MAX_GAMMA) return false;
    L.nchunks = (V + kChunk - 1) / kChunk;
    L.rows_total = (size_t)B * (2 * (size_t)gamma + 1);
    if (L.rows_total * (size_t)L.nchunks > 0x7fffffffull) return false;     // 1-D grids of 32-bit size
    const size_t rows_t = (size_t)B * (gamma + 1), rows_d = (size_t)B * gamma;

    // a workgroup is four waves, each with one wave chunk of a row
    L.nu = (V + kWaves * kWave * kLaneSmall - 1) / (kWaves * kWave * kLaneSmall) * kWaves;
    L.fused_grid = rows_t * (size_t)(L.nu / kWaves);
    L.fused_ok = L.nu <= kMaxUnitsPerRow && L.fused_grid <= 0x7fffffffull;
    size_t off = kHdrWords * sizeof(int);
    L.off_gen = off;    off = align_up(off + (size_t)B * sizeof(int), 256);
    const size_t copy0 = off;
    L.off_ratio = off;  off += rows_d * sizeof(u64);
    L.off_lw = off;     off += rows_d * sizeof(u64);
    L.off_rowres = off; off += rows_d * sizeof(u64);
    L.off_pstat = off;  off += rows_d * L.nu * sizeof(u64);
    L.off_plast = off;  off += (size_t)B * L.nu * sizeof(u64);
    off = align_up(off, 16);
    L.off_pgrp = off;   off += rows_d * (L.nu / kWaves) * 2 * sizeof(u64);     // (target word, draft word) pairs
    L.off_qgrp = L.off_pgrp + sizeof(u64);
    L.off_spart = off;  off += rows_d * L.nu * sizeof(unsigned);
    off = align_up(off, 8);
    L.off_lseen = off;  off += (size_t)B * (L.nu / kWaves) * sizeof(u64);
    L.copy_bytes = align_up(off - copy0, 256);
    off = copy0 + 2 * L.copy_bytes;
    L.control_words = off / sizeof(int);
    off = align_up(off, 256);
    // the staged path's scratch follows, so that it never touches the control words
    L.off_stats = off;  off = align_up(off + L.rows_total * L.nchunks * sizeof(float2), 256);
    L.off_coef = off;   off = align_up(off + rows_t * sizeof(SeqCoef), 256);
    L.off_sspart = off; off = align_up(off + rows_d * L.nchunks * sizeof(float), 256);
    L.total = off;
    return true;
}

template <typename T> constexpr int dtype_bytes() { return ElemTraits<T>::kVec == 4 ? 4 : 2; }

// Workgroups of a kernel that the current device keeps resident at once (cached per kernel).
template <typename K>
int resident_workgroups(K kernel, std::atomic<int> &cache, int threads = kThreads)
{
    if (cache.load() > 0) return cache.load();
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) return 0;
    cache.store(cus * per_cu);
    return cus * per_cu;
}

void report_form(int form, int lanes, int logits) { g_last_form.store(form * 1000000 + lanes * 1000 + logits); }

template <typename T, bool ALIGNED>
sv_status_t launch_staged(int algo, const void *target_v, const void *draft_v, const int32_t *tokens, const int32_t *draft_lens,
                          size_t tstride, size_t dstride, const float *uniforms, int B, int gamma, int V, float k, double kd, const Layout &L,
                          char *ws, int32_t *accept_len, int32_t *next_token, float *debug_out,
                          hipStream_t stream)
{
    const T *target = static_cast<const T *>(target_v);
    const T *draft = static_cast<const T *>(draft_v);
    float2 *stats = reinterpret_cast<float2 *>(ws + L.off_stats);
    SeqCoef *coef = reinterpret_cast<SeqCoef *>(ws + L.off_coef);
    float *spart = reinterpret_cast<float *>(ws + L.off_sspart);
    const int n_target_rows = B * (gamma + 1);

    row_stats_kernel<T, ALIGNED><<<(unsigned)((size_t)B * (2 * gamma + 1) * L.nchunks), kThreads, 0, stream>>>(
        target, draft, tstride, dstride, B, gamma, V, k, L.nchunks, stats);
    const size_t sm2 = 2 * (gamma + 1) * sizeof(double) + 2 * (gamma + 1) * sizeof(float);
    prefix_weights_kernel<T><<<B, 64, sm2, stream>>>(target, draft, tstride, dstride, tokens, gamma, V, k, kd, kd / (double)k - 1.0, L.nchunks,
                                                    n_target_rows, algo, stats, coef, draft_lens, uniforms, debug_out ? 1 : 0);
    const unsigned pair_blocks = (unsigned)((size_t)B * gamma * L.nchunks);
    residual_kernel<T, ALIGNED><<<pair_blocks, kThreads, 0, stream>>>(
        target, draft, tstride, dstride, gamma, V, k, L.nchunks, coef, spart);
    const size_t sm4 = (gamma + 1) * sizeof(double);
    finalize_kernel<T, ALIGNED><<<B, kThreads, sm4, stream>>>(
        target, draft, tstride, dstride, uniforms, gamma, V, k, L.nchunks, algo, stats, coef, spart,
        accept_len, next_token, debug_out, draft_lens);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

// A number of 64 bits for a call with probabilities: no other call of this process has it, and which ones come is anyone's guess (a count
// from a start that depends on the time and on where the process lies, through a bijection), so that what an unprepared workspace holds is not
// taken for this call's (see probs.hpp).
u64 probs_call_number()
{
    auto mixed = [](u64 x) {                             // (splitmix64's finishing steps)
        x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
        x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
        return x ^ (x >> 31);
    };
    static std::atomic<u64> next{mixed((u64)std::chrono::steady_clock::now().time_since_epoch().count()) ^ (u64)reinterpret_cast<uintptr_t>(&next)};
    u64 n;
    do n = mixed(next.fetch_add(1)); while (n == 0);     // (what zeros say is no call's)
    return n;
}

// Whether calls on the stream are being recorded (the null stream's never are).
bool being_captured(hipStream_t stream)
{
    if (!stream) return false;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();                             // (what is wrong with the stream the launches will say)
    return true;
}

// The kernel that holds several short sequences, or one, in the registers of a workgroup, and its launch (none: the rows or their groups are
// too many).  Lanes per row pair and sequences per workgroup by the row's length, the rows in the call and the draft's length, us a call on the
// device (dense calls, another one / the one taken):
//   up to 8 tokens a lane per row pair, four sequences per wave: 8192 of 10 over 2, float32: four lanes each, one sequence per wave 11.8 / 5.9 (not float32 rows a line
//   apart in long drafts, of which every lane of a wave reads another line: 3914 of 50 over 5, 69 apart 16.3 / 22.3, 1952 of 60 over 6 9.5 / 10.4, dense 4756 of 53 over 4 13.2 / 7.2);
//   up to 32 four lanes: 8192 of 10 over 30, bf16, one sequence per workgroup / four 14.0 / 10.5, 64 of them the same;
//   up to 128 sixteen: four sequences where drafts are short: 8192 of 4 over 60 17.9 / 13.8; bf16 2385 of 7 over 82 9.3 / 8.8 (own lengths up to five drafted tokens, beyond in smaller calls
//   only: float32 7744 of 5 over 59 15.7 / 15.1, 7197 of 6 over 52 15.5 / 16.4; bf16 4834 of 7 over 77 13.7 / 14.1);
//   one sequence gets no more from this kernel than from small_verify_kernel, which has 56 registers instead of 68 (eight waves per SIMD, not seven; that one / this one:
//   bf16, 5430 of 16 over 101 25.4 / 29.7, 4308 of 15 over 128 15.5 / 16.9, 7465 of 8 over 64 21.1 / 22.1, 3289 of 63 over 27 13.4 / 14.8; float32, 6711 of 12 over 78 24.0 /
//   26.5, 7613 of 15 over 116 28.7 / 30.5, 7620 of 7 over 67 18.6 / 18.8);
//   up to 256 32, in calls of many rows sixteen with twice the logits each: 512 of 8 over 192, bf16, a wave per row pair / 32 lanes / 16
//   8.5 / 7.0 / 7.6, 8192 of them 73.3 / 45.3 / 38.6; float32, 1024 of 12 over 256 16.8 / 12.5 / 11.5; 2048 of 6 over 250 17.3 / 11.7 / 11.8, 10.8 with four sequences; drafts of 24 and
//   more, of whose workgroups a compute unit holds one, in calls of more sequences than units sixteen too (32 / 16: bf16 393 of 26 over 162 11.0 / 8.9, float32 264 of 26 over 255
//   12.6 / 10.5; small_verify_kernel's sixteen of 32 9.2, 11.2);
//   up to 512 a wave per row pair (small_verify_kernel; probabilities: here), or 32 lanes: bf16 rows in bulk (that one / this one: 2048 of 14 over 500 32.7 / 26.1,
//   7206 of 5 over 461 41.0 / 35.0, 2859 over 320 18.8 / 17.3; of 4 7946 over 284 40.2 / 38.7, 4339 over 512 21.0 / 22.4, of own lengths 5875 over 356 28.4 / 29.3, 16384 over 410 71.7 / 71.4; of 2 3375 over 512 12.4 / 15.0; float32 2048 of 10 over
//   400 28.5 / 30.7), and drafts that a workgroup's sixteen waves do not hold, else sixteen lanes of 32 (small_verify_kernel): up to drafts of 23 (two
//   workgroups to a compute unit: 772 of 21 over 512, bf16 21.2 / 17.5, 864 of 20 over 448, float32 22.9 / 20.4, 2966 of 16 over 512 63.7 / 57.5; not bf16 rows of three vectors of sixteen lanes, in
//   bulk: 1820 of 16 over 384 30.5 / 32.1, 2057 over 347 36.9 / 38.4, 1160 over 320 22.8 / 22.2), of 31 while each workgroup has its compute unit alone (144 of 26 over 512, float32
//   10.9 / 9.5; 452 over 259 12.3 / 15.1; bf16 3090 of 27 over 384 52.6 / 77.3); from 32 on both are the same.
// Probabilities, against the kernels for wider rows: 6000 of 10 over 2 163 / 5.8; 6000 of 10 over 256, float32 132.6 / 32.1; 1000 of 12 over 768, bf16 30.4 / 17.7 (a
// wave per row pair 21.8; 200 of 12 7.3 either way); over 1025 ... 2048 tokens with longer drafts only while the workgroups are few: 512 of 10 over 2000, bf16 20.7 /
// 16.6, 1000 28.8 / 30.5, 2048 50.4 / 58.0; 2048 of 4 35.1 / 32.4; and not few sequences of long drafts over more than 1536, whose rows those spread over the device (float32 1 of 13 over
// 1875 9.5 / 11.2, 25 of 10 over 1740 9.4 / 10.0, 53 of 13 over 1600 10.9 / 10.8; bf16 29 of 14 over 2031 9.7 / 10.5, 6 of 10 over 1689 8.8 / 8.8, 59 of 14 over 2013 10.6 / 10.5).
// Alg. 1 without the report, long drafts: the kernels for wider rows do not read what lies behind the first failed test, which from this many bytes of target rows on saves
// more than this kernel does (this one / those, drafts of 8 and more over 1025 ... 2048 tokens, of 16 over 513 ... 1024: float32 372 of 15 over 1864 26.9 / 22.4, 882 of 18 over 953 37.7 /
// 32.3, 1503 of 27 over 814 75.3 / 52.4, 197 of 27 over 995 (20 MiB) 14.4 / 16.8, 412 of 12 over 1105 (22 MiB) 18.4 / 20.2; bf16 1383 of 19 over 810 41.0 / 38.3, 633 of 8 over 1620 20.2 / 19.5; poor drafts
// more, up to 2.2 times), over 257 ... 512 with drafts of 32 and more from four times as many (float32 2172 of 53 over 367 108 / 94, 1467 of 52 over 266 (79 MiB) 60.9 / 61.0).
constexpr size_t kPackedEarlyBytes = 32u << 20;
constexpr int kComputeUnits = 256;
struct PackedLaunch {
    void (*kernel)(const FusedParams);
    unsigned blocks, threads;
    int seqs, lanes, logits;             // sequences of a workgroup; lanes of a row pair, logits of a row per lane
};
// (SEG: the only one of the two that calls of this form have; 0: by the draft's length)
template <typename T, bool PROBS, int G, int LANE, int SEG = 0>
PackedLaunch packed_launch_of(int B, int gamma, int seqs)
{
    const bool seg16 = SEG ? SEG == 16 : gamma <= 16;
    void (*const kernel)(const FusedParams) = seg16 ? packed_verify_kernel<T, PROBS, G, LANE, SEG ? SEG : 16> : packed_verify_kernel<T, PROBS, G, LANE, SEG ? SEG : kWave>;
    const int seg = seg16 ? 16 : kWave, one = (gamma + 1) * G > seg ? (gamma + 1) * G : seg;      // lanes of one sequence
    const int threads = (seqs * one + kWave - 1) / kWave * kWave;
    if (threads > (G == 1 ? 2 * kWave : kTinyThreads)) return {};
    return {kernel, (unsigned)((B - 1) / seqs + 1), (unsigned)threads, seqs, G, LANE};
}
// (`stops_early`: Alg. 1 on probabilities without the report)
template <typename T, bool PROBS>
PackedLaunch packed_launch(int B, int gamma, int V, size_t tstride, bool own_lengths, bool stops_early)
{
    const long long rows = (long long)B * (gamma + 1);
    const bool bf16 = ElemTraits<T>::kVec == 8;
    if (!PROBS && !bf16 && V <= 8 && gamma > 16 && tstride >= 32) return {};
    if (V <= 8) return packed_launch_of<T, PROBS, 1, 8>(B, gamma, gamma < 16 ? 4 : gamma == 16 ? 3 : 1);
    if (V <= 4 * 8) {
        if (!PROBS && gamma > 16) return {};
        return packed_launch_of<T, PROBS, 4, 8, PROBS ? 0 : 16>(B, gamma, gamma <= 16 && B >= 512 ? 4 : 1);
    }
    if (V <= 16 * 8) {
        const bool several = gamma == 7 ? B >= (PROBS ? 1024 : 2048) && (PROBS || bf16) : gamma < 7 && B >= 1024;
        // (own lengths: the waves of the sequences' last positions wait for nothing, so that long drafts gain less from sharing a workgroup)
        const bool apart = !PROBS && own_lengths && gamma >= 6 && B >= (bf16 ? 4096 : 2048);
        if constexpr (PROBS) return gamma < 64 ? packed_launch_of<T, PROBS, 16, 8>(B, gamma, several ? 4 : 1) : packed_launch_of<T, PROBS, 4, 32, kWave>(B, gamma, 1);
        else return several && !apart ? packed_launch_of<T, PROBS, 16, 8, 16>(B, gamma, 4) : PackedLaunch{};
    }
    if (V <= 16 * 16) {
        if (rows > 12288 || gamma >= 32 || (!PROBS && gamma >= 24 && B > kComputeUnits)) return packed_launch_of<T, PROBS, 16, 16>(B, gamma, gamma < 8 ? 4 : 1);
        return packed_launch_of<T, PROBS, 32, 8>(B, gamma, 1);
    }
    if constexpr (PROBS) {
        const size_t bytes = (size_t)rows * V * sizeof(T);
        if (stops_early && ((V > 32 * 16 && gamma >= (V > 32 * 32 ? 8 : 16) && bytes > kPackedEarlyBytes) || (V > 16 * 16 && gamma >= 32 && bytes > 4 * kPackedEarlyBytes))) return {};
    }
    if (V <= 32 * 16) {
        if constexpr (PROBS) {
            if (gamma >= 32) return packed_launch_of<T, PROBS, 16, 32, kWave>(B, gamma, 1);
            if (gamma >= 16 || rows > 8192) return packed_launch_of<T, PROBS, 32, 16>(B, gamma, 1);
            return packed_launch_of<T, PROBS, 64, 8, 16>(B, gamma, 1);
        } else {
            const bool here = gamma < 16 ? bf16 && (gamma >= 5 ? rows > 8192 : gamma == 4 && rows > (own_lengths ? 65536 : 24576))
                            : gamma < 24 ? !(bf16 && V <= 384 && B > 1200) : gamma < 32 && B <= kComputeUnits;
            if (here) return packed_launch_of<T, PROBS, 32, 16, ElemTraits<T>::kVec == 8 ? 0 : kWave>(B, gamma, 1);
        }
    }
    if constexpr (PROBS) {
        if (V > 32 * 16 && V <= 32 * 32) return rows > 3072 || gamma >= 16 ? packed_launch_of<T, PROBS, 32, 32>(B, gamma, 1) : packed_launch_of<T, PROBS, 64, 16, 16>(B, gamma, 1);
        const bool few_long = V > 64 * 24 && gamma >= (bf16 ? 12 : 10) && B <= (bf16 ? 32 : 64);
        if (V > 32 * 32 && V <= kSmallMaxRow && (gamma < 6 || rows <= 6000) && !few_long) return packed_launch_of<T, PROBS, 64, 32, 16>(B, gamma, 1);
    }
    return {};
}

// Probabilities as inputs: one to three launches, every element read once.  Scratch (rows of more than 2048 tokens): the staged path's areas
// (chunk partial sums where its row statistics go, the weights where its row constants go).
template <typename T, bool ALIGNED>
sv_status_t launch_probs(int algo, const void *target_v, const void *draft_v, const int32_t *tokens, const int32_t *draft_lens,
                         size_t tstride, size_t dstride, const float *uniforms, int B, int gamma, int V, const Layout &L,
                         char *ws, int32_t *accept_len, int32_t *next_token, float *debug_out, hipStream_t stream)
{
    const T *target = static_cast<const T *>(target_v);
    const T *draft = static_cast<const T *>(draft_v);
    const PackedLaunch packed = packed_launch<T, true>(B, gamma, V, tstride, draft_lens != nullptr, algo == kToken && !debug_out);
    if (packed.kernel) {
        FusedParams F = {};
        F.target = target; F.draft = draft; F.tokens = tokens; F.draft_lens = draft_lens; F.uniforms = uniforms;
        F.B = B; F.gamma = gamma; F.V = V; F.tstride = tstride; F.dstride = dstride; F.algo = algo;
        F.group_seqs = packed.seqs; F.inv_slots = (unsigned)(0x100000000ull / (unsigned)(gamma + 1)) + 1u;
        F.accept_len = accept_len; F.next_token = next_token; F.debug_out = debug_out;
        packed.kernel<<<packed.blocks, packed.threads, 0, stream>>>(F);
        report_form(SV_FORM_SEQUENCES, packed.lanes, packed.logits);
        return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
    }
    ProbsParams P = {};
    P.target = target; P.draft = draft; P.tstride = tstride; P.dstride = dstride;
    P.tokens = tokens; P.draft_lens = draft_lens; P.uniforms = uniforms;
    P.gamma = gamma; P.V = V; P.nchunks = L.nchunks; P.algo = algo;
    // (the words where the staged path has its row statistics, one for every chunk of all rows, and its residual partial sums)
    P.part = reinterpret_cast<u64 *>(ws + L.off_stats);
    P.part_last = P.part + 2 * (size_t)B * gamma * L.nchunks;
    P.check_last = reinterpret_cast<unsigned *>(ws + L.off_sspart);
    static_assert(sizeof(ProbWeight) <= sizeof(SeqCoef), "the weights reuse the staged path's row-constant area");
    ProbWeight *const weights = reinterpret_cast<ProbWeight *>(ws + L.off_coef);
    P.weights = weights;
    P.spin_limit = g_spin_limit.load();
    P.call = probs_call_number();
    P.accept_len = accept_len; P.next_token = next_token; P.debug_out = debug_out;
    const unsigned blocks = (unsigned)((size_t)B * (gamma + 1) * L.nchunks);
    // A position's weight: formed by each of its workgroups under its loads (B = 64, gamma = 8, V = 128256, bf16: 58 -> 51 us,
    // 1 sequence 18 -> 14; float32, B = 48 83 -> 69, 72 with the kernel in front), or by a kernel in front.  That is the better way where most workgroups have nothing to sum
    // (Alg. 1 unless every sum is reported: 25 us against 48 there, unless the call runs at once anyway: kProbsAtOnce) and where there are many of them with less to read
    // than the weight takes to form (kProbsFormMax).
    const int every_sum = P.every_sum = debug_out ? 1 : 0;
    const bool many_short = V <= kChunk / 2 && (long long)B * (gamma + 1) > kProbsFormMax;
    const size_t row_bytes = (size_t)blocks * (V < kChunk ? V : kChunk) * sizeof(T);       // the target rows' (the last chunk counted whole)
    const bool in_front = (algo == kToken && !every_sum && (blocks > kProbsAtOnce || row_bytes > kProbsAtOnceBytes)) || many_short;
    if (in_front)
        probs_weights_kernel<T><<<B, 64, 0, stream>>>(target, draft, tstride, dstride, tokens, draft_lens, gamma, algo, weights, uniforms, every_sum);
    const size_t kept_floats = (size_t)(gamma + 1) * L.nchunks * (algo == kGreedy ? 2 : 1);      // chunk sums (Alg. 4: and rejected masses)
    P.keep = kept_floats <= (size_t)kProbsKeepMax ? 1 : 0;
    const size_t lds = probs_finish_doubles(gamma) * sizeof(double) + (P.keep ? kept_floats * sizeof(float) : 0);
    static std::atomic<int> cap;
    const int resident = resident_workgroups(probs_residual_kernel<T, ALIGNED, false, true, true>, cap);
    if (resident < 1) return SV_ERR_HIP;
    // (the workgroup that finishes a sequence keeps its sums: no call this small has too many)
    // A recorded call has the same number every time it is replayed, and would take the words of the time before for its own: it has two launches.
    if (!in_front && P.keep && blocks <= probs_at_once(resident, gamma, ElemTraits<T>::kVec == 4, ALIGNED) && !being_captured(stream)) {
        (algo == kGreedy ? probs_residual_kernel<T, ALIGNED, true, true, true> : probs_residual_kernel<T, ALIGNED, false, true, true>)<<<blocks, kThreads, lds, stream>>>(P);
        return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
    }
    void (*const residual)(const ProbsParams) =
        algo == kGreedy ? (in_front ? probs_residual_kernel<T, ALIGNED, true, false, false> : probs_residual_kernel<T, ALIGNED, true, true, false>)
        : in_front ? probs_residual_kernel<T, ALIGNED, false, false, false> : probs_residual_kernel<T, ALIGNED, false, true, false>;
    // Rows of more than eight chunks whose weights are formed here, bf16: six workgroups on a compute unit instead of the eight that their registers allow, by LDS that they do
    // not use: more of them only pile up loads (eight / seven / six, us: B = 64, gamma = 8, V = 128256 49.7 / 49.1 / 49.0, five 50.0; 300 of 8 over 100000 151.6 / 148.7 / 145.7;
    // 100 of 8 over 250000 129.1 / 126.9 / 123.8; 200 of 8 over 65600 69.8 / 68.4 / 67.3).  Shorter ones need the places, the more the emptier a row's last workgroup is (200 of
    // 8 over 58000 69.8 / 70.0 / 70.2, over 50257 60.9 / 61.5 / 63.0; 548 ragged of 7 over 14016 39.5 / 41.2 / 42.9); float32 workgroups are five a unit (four: 200 of 4 over 128256
    // 132 / 130, 100 of 8 over 32000 in bf16 24.6 / 26.0).
    const bool long_rows = !in_front && ElemTraits<T>::kVec == 8 && L.nchunks > 8;
    residual<<<blocks, kThreads, long_rows ? kProbsSixPerUnit : 0, stream>>>(P);
    (algo == kGreedy ? probs_finish_kernel<T, ALIGNED, true> : probs_finish_kernel<T, ALIGNED, false>)<<<B, kThreads, lds, stream>>>(P);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

// Whether a sequence's 2 gamma + 1 rows fit the LDS of one workgroup.
bool tiny_ok(int gamma, int V) { return (size_t)(2 * gamma + 1) * (size_t)V <= (size_t)kTinyMaxFloats; }

// The kernel that keeps a sequence's rows in the registers of one workgroup, a wave per row pair or, in short rows, 4 or 16 lanes, and its launch, for the calls that
// packed_launch leaves (both sides' times there); none where the rows or their groups are too many.  As few logits per lane as the row allows: fewer registers,
// shorter chains (8192 sequences of 4 over 1000 bf16 logits: 58 us with sixteen per lane, 105 with 32; 32 / 24: float32 1000 of 4 over 1500 24.5 / 18.0, 2000 of 15 over
// 1030 88 / 77; bf16 300 of 16 over 1536 20.4 / 18.8, 5390 of 8 over 1244 150 / 147).
struct SmallLaunch {
    void (*kernel)(const FusedParams);
    unsigned blocks, threads;
    int lanes, logits;
};
template <typename T, int G, int LANE>
SmallLaunch small_launch_of(int B, int gamma)
{
    const int threads = ((gamma + 1) * G + kWave - 1) / kWave * kWave;           // a group per row pair and one for the last target row
    if constexpr (G * (SV_MAX_GAMMA + 1) > kTinyThreads && (G != kWave || LANE != 8)) {             // (those take no draft that fills the workgroup)
        if (threads > kTinyThreads && gamma * G <= kTinyThreads) return {small_verify_kernel<T, G, LANE, true>, (unsigned)B, kTinyThreads, G, LANE};
    }
    if (threads <= kTinyThreads) return {small_verify_kernel<T, G, LANE, false>, (unsigned)B, (unsigned)threads, G, LANE};
    return {};
}
template <typename T>
SmallLaunch small_launch(int B, int gamma, int V)
{
    if (V <= 4 * 8) return small_launch_of<T, 4, 8>(B, gamma);
    if (V <= 16 * 8) return small_launch_of<T, 16, 8>(B, gamma);
    if (V <= 64 * 8 && gamma < kTinyWaves) return small_launch_of<T, 64, 8>(B, gamma);
    if (V <= 16 * 32) return small_launch_of<T, 16, 32>(B, gamma);
    if (V <= 64 * 16) return small_launch_of<T, 64, 16>(B, gamma);
    if (V <= 64 * 24 && (tiny_ok(gamma, V) || B > kSmallMinWide)) return small_launch_of<T, 64, 24>(B, gamma);
    if (V <= kSmallMaxRow && (tiny_ok(gamma, V) || B > kSmallMinWide)) return small_launch_of<T, 64, 32>(B, gamma);
    return {};
}

// One workgroup per sequence (SV_ERR_UNSUPPORTED: the sequence does not fit one).
template <typename T>
sv_status_t launch_tiny(int algo, const void *target, const void *draft, const int32_t *tokens, const int32_t *draft_lens,
                        size_t tstride, size_t dstride, const float *uniforms, int B, int gamma, int V, float k, double kd,
                        int magic, char *ws, int32_t *accept_len, int32_t *next_token, float *debug_out, hipStream_t stream)
{
    const PackedLaunch packed = packed_launch<T, false>(B, gamma, V, tstride, draft_lens != nullptr, false);
    const SmallLaunch small = packed.kernel ? SmallLaunch{packed.kernel, packed.blocks, packed.threads, packed.lanes, packed.logits} : small_launch<T>(B, gamma, V);
    if (!small.kernel && !tiny_ok(gamma, V)) return SV_ERR_UNSUPPORTED;
    FusedParams P = {};
    P.target = target; P.draft = draft; P.tokens = tokens; P.draft_lens = draft_lens; P.uniforms = uniforms;
    P.B = B; P.gamma = gamma; P.V = V; P.tstride = tstride; P.dstride = dstride;
    P.k = k; P.kd = kd; P.k_eps = kd / (double)k - 1.0; P.algo = algo;
    P.magic = magic;
    P.inv_wpr = V > 1 ? (unsigned)(0x100000000ull / (unsigned)V) + 1u : 0u;
    P.group_seqs = packed.seqs; P.inv_slots = (unsigned)(0x100000000ull / (unsigned)(gamma + 1)) + 1u;
    P.header = reinterpret_cast<int *>(ws);
    P.accept_len = accept_len; P.next_token = next_token; P.debug_out = debug_out;
#ifdef SV_PROFILE
    P.prof = g_prof.load();
#endif
    report_form(packed.kernel ? SV_FORM_SEQUENCES : small.kernel ? SV_FORM_SEQUENCE : SV_FORM_SEQUENCE_IN_LDS, small.lanes, small.logits);
    if (small.kernel) small.kernel<<<small.blocks, small.threads, 0, stream>>>(P);
    else tiny_verify_kernel<T><<<(unsigned)B, kTinyThreads, 0, stream>>>(P);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

// The arguments that the kernels working through the control words share: the inputs, the outputs, the words.
FusedParams word_params(int algo, const void *target, const void *draft, const int32_t *tokens, const int32_t *draft_lens,
                        size_t tstride, size_t dstride, const float *uniforms, int B, int gamma, int V, float k, double kd, const Layout &L,
                        char *ws, int32_t *accept_len, int32_t *next_token, float *debug_out)
{
    FusedParams P = {};
    P.target = target; P.draft = draft; P.tokens = tokens; P.draft_lens = draft_lens; P.uniforms = uniforms;
    P.tstride = tstride; P.dstride = dstride;
    P.B = B; P.gamma = gamma; P.V = V; P.k = k; P.kd = kd; P.k_eps = kd / (double)k - 1.0; P.algo = algo;
    P.nu = L.nu;
    P.spin_limit = g_spin_limit.load();
    P.magic = workspace_magic(B, gamma, V);
    P.header = reinterpret_cast<int *>(ws);
    P.gen = reinterpret_cast<int *>(ws + L.off_gen);
    P.words.ratio = reinterpret_cast<u64 *>(ws + L.off_ratio);
    P.words.lw = reinterpret_cast<u64 *>(ws + L.off_lw);
    P.words.rowres = reinterpret_cast<u64 *>(ws + L.off_rowres);
    P.words.pstat = reinterpret_cast<u64 *>(ws + L.off_pstat);
    P.words.plast = reinterpret_cast<u64 *>(ws + L.off_plast);
    P.words.pgrp = reinterpret_cast<u64 *>(ws + L.off_pgrp);
    P.words.qgrp = reinterpret_cast<u64 *>(ws + L.off_qgrp);
    P.words.spart = reinterpret_cast<unsigned *>(ws + L.off_spart);
    P.words.lseen = reinterpret_cast<u64 *>(ws + L.off_lseen);
    P.copy_bytes = L.copy_bytes;
    P.accept_len = accept_len; P.next_token = next_token; P.debug_out = debug_out;
#ifdef SV_PROFILE
    P.prof = g_prof.load();
#endif
    return P;
}

// Rows that one workgroup holds (rows_verify_kernel); `P`: the arguments of the call, `in_chain`: how a position learns w_i (calls of few resident sets: from the
// ratios, see resident_sets; others by the large kernel's line, which holds here: 200 calls of 1.2 to 16 of its sets with the line / the ratios / the chain: 0.15 % over the faster of the two on
// average, eleven more than 1 % over, the worst 1064 ragged of 4 over 2301, Alg. 1, 15.2 / 14.6 / 15.2 us; 104 ragged of 16 over 2163 11.2 / 11.2 / 18.5, 1912 of 8 over 4736 60.5 /
// 64.7 / 60.4).
template <typename T, bool ALIGNED>
sv_status_t launch_rows(FusedParams P, bool in_chain, hipStream_t stream)
{
    static std::atomic<int> caps[2][3][65];              // (of each kernel: with and without the chain, by waves, by logits per lane)
    void (*kernel)(const FusedParams) = nullptr;
    const int waves = P.V <= 4096 ? 2 : P.V <= kThreads * 64 ? 4 : 8;
    int lane_logits = (P.V + waves * kWave - 1) / (waves * kWave);
    // (two waves or four or eight: 1200 sequences of 4 over 3000 19.1 / 21.1 us, 1000 of 8 over 4000 30.2 / 31.3, 800 of 8 over 5000 31.6 / 30.7, 2000 of 4 over 8192 51.6 / 50.4;
    // 512 of 8 over 16384 four 50.7, eight 52.8)
#define SV_FORM(W, LN) if (!kernel && waves == W && lane_logits <= LN) { \
        kernel = in_chain ? rows_verify_kernel<T, ALIGNED, W, LN, true> : rows_verify_kernel<T, ALIGNED, W, LN, false>; lane_logits = LN; }
    SV_FORM(2, 24) SV_FORM(2, 32) SV_FORM(4, 24) SV_FORM(4, 32) SV_FORM(4, 40) SV_FORM(4, 48) SV_FORM(4, 64) SV_FORM(8, 40)
#undef SV_FORM
    if (!kernel) return SV_ERR_UNSUPPORTED;
    const int capacity = resident_workgroups(kernel, caps[in_chain ? 1 : 0][waves / 4][lane_logits], waves * kWave);
    if (capacity < 1) return SV_ERR_HIP;
    // groups of sequences so large that one position of a group fills the device at least once
    const int groups = P.B / capacity > 1 ? P.B / capacity : 1;
    P.group_seqs = (P.B + groups - 1) / groups;
    const int n_groups = (P.B + P.group_seqs - 1) / P.group_seqs;
    P.inv_slots = (unsigned)(0x100000000ull / (unsigned)(P.gamma + 1)) + 1u;
    if ((size_t)n_groups * (P.gamma + 1) > 65535u) return SV_ERR_UNSUPPORTED;
    kernel<<<dim3((unsigned)P.group_seqs, (unsigned)(n_groups * (P.gamma + 1))), waves * kWave, 0, stream>>>(P);
    report_form(SV_FORM_ROW, waves * kWave, lane_logits);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

// The kernels for calls of few resident sets; SV_ERR_UNSUPPORTED for the calls they do not take (more workgroups than
// resident_sets() times what the device keeps resident - kResidentSetsForced where the testing hook asks for it and that is more -,
// rows of more than kResidentMaxGroups workgroups).
template <typename T, bool ALIGNED>
sv_status_t launch_resident(int algo, const void *target, const void *draft, const int32_t *tokens, const int32_t *draft_lens,
                            size_t tstride, size_t dstride, const float *uniforms, int B, int gamma, int V, float k, double kd, const Layout &L,
                            char *ws, int32_t *accept_len, int32_t *next_token, float *debug_out, hipStream_t stream)
{
    const int nwg = L.nu / kWaves;
    if (nwg > kResidentMaxGroups || B > 65535) return SV_ERR_UNSUPPORTED;
    static std::atomic<int> cap, cap_together;
    void (*kernel)(const FusedParams) = resident_verify_kernel<T, ALIGNED>;
    const int capacity = resident_workgroups(kernel, cap);
    if (capacity < 1) return SV_ERR_HIP;
    double sets = resident_sets(gamma, nwg, ElemTraits<T>::kVec == 4, draft_lens != nullptr, ALIGNED);
    const int path = g_path.load();
    if (path >= 7 && sets < kResidentSetsForced) sets = kResidentSetsForced;
    if ((double)((long long)nwg * B * (gamma + 1)) > sets * capacity) return SV_ERR_UNSUPPORTED;
    // (a rule without the report, which changes no decision)
    const bool together = path >= 8 ? path == 8
        : runs_together((long long)nwg * B * (gamma + 1), resident_workgroups(together_verify_kernel<T, ALIGNED, 1>, cap_together), nwg, gamma, ElemTraits<T>::kVec == 4);
    if (together)
        kernel = nwg <= 4 ? together_verify_kernel<T, ALIGNED, 0> : nwg <= 16 ? together_verify_kernel<T, ALIGNED, 1> : together_verify_kernel<T, ALIGNED, 2>;
    FusedParams P = word_params(algo, target, draft, tokens, draft_lens, tstride, dstride, uniforms, B, gamma, V, k, kd, L,
                                ws, accept_len, next_token, debug_out);
    // (where the row pairs are more than run at once: what leaves early makes room)
    P.prune = (long long)nwg * B * gamma > capacity ? 1 : 0;
    if (path == 0 && rows_alone((long long)nwg * B * (gamma + 1), resident_workgroups(together_verify_kernel<T, ALIGNED, 1>, cap_together), gamma, V,
                                ElemTraits<T>::kVec == 4, draft_lens != nullptr, together, algo == kToken)) {
        const sv_status_t st = launch_rows<T, ALIGNED>(P, false, stream);
        if (st == SV_OK) g_last_together.store(0);
        if (st != SV_ERR_UNSUPPORTED) return st;
    }
    kernel<<<dim3((unsigned)nwg, (unsigned)B, (unsigned)(gamma + 1)), kThreads, 0, stream>>>(P);
    g_last_together.store(together ? 1 : 0);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

template <typename T, bool ALIGNED>
sv_status_t launch_fused(int algo, const void *target, const void *draft, const int32_t *tokens, const int32_t *draft_lens,
                         size_t tstride, size_t dstride, const float *uniforms, int B, int gamma, int V, float k, double kd, const Layout &L,
                         char *ws, int32_t *accept_len, int32_t *next_token, float *debug_out,
                         hipStream_t stream)
{
    // Unit size: 32 logits per lane (5 waves per SIMD).  The kernel also exists with 64 per lane (3 waves per SIMD, half
    // as many workgroups per row to wait for; bf16 rows on the vector path), which used to be the faster one for very wide
    // rows; since the smaller units publish less it is not any more (B = 1024, gamma = 8, V = 256000: 1414 - 1424 us
    // against 1435 - 1439), and only the testing hook asks for it.
    // The workspace is laid out for the smaller units, whose words are a superset.
    constexpr bool kLargeOk = ALIGNED && ElemTraits<T>::kVec == 8;
    const bool large = kLargeOk && g_lane.load() == kLaneLarge;
    const int lane_logits = large ? kLaneLarge : kLaneSmall;
    const int nu = (V + kWaves * kWave * lane_logits - 1) / (kWaves * kWave * lane_logits) * kWaves;
    // the instantiations for this row width (one or two words of a row per lane of the collecting wave), with and without
    // the chain (the hook's larger units always have it), and their resident workgroups
    static std::atomic<int> cap[2], cap_chain[2][2];
    const int nwg = nu / kWaves;
    const int nw_log = nwg <= kWave ? 0 : 1;
    void (*ratios)(const FusedParams) = nullptr, (*chain)(const FusedParams) = nullptr;
#define SV_PICK(LN, CH) (nw_log == 0 ? fused_verify_kernel<T, ALIGNED, 1, LN, CH> : fused_verify_kernel<T, ALIGNED, 2, LN, CH>)
    if constexpr (kLargeOk) {
        if (large) chain = SV_PICK(kLaneLarge, true);
    }
    if (!large) { ratios = SV_PICK(kLaneSmall, false); chain = SV_PICK(kLaneSmall, true); }
#undef SV_PICK
    const int with_chain = resident_workgroups(chain, cap_chain[nw_log][large ? 1 : 0]), with_ratios = large ? with_chain : resident_workgroups(ratios, cap[nw_log]);
    const int capacity = with_ratios < with_chain ? with_ratios : with_chain;
    const int wpr = nwg;
    // a row's workgroups wait for each other and must fit on the device together, with room to spare
    if (capacity < 4 * wpr) return capacity < 1 ? SV_ERR_HIP : SV_ERR_UNSUPPORTED;
    FusedParams P = word_params(algo, target, draft, tokens, draft_lens, tstride, dstride, uniforms, B, gamma, V, k, kd, L,
                                ws, accept_len, next_token, debug_out);
    P.nu = nu;
    P.inv_slots = (unsigned)(0x100000000ull / (unsigned)(gamma + 1)) + 1u;
    P.inv_wpr = (unsigned)(0x100000000ull / (unsigned)(nu / kWaves)) + 1u;
    // groups of sequences so large that one position of a group fills the device at least once
    const int min_seqs = (capacity + wpr - 1) / wpr;
    const int groups = B / min_seqs > 1 ? B / min_seqs : 1;
    P.group_seqs = (B + groups - 1) / groups;
    const int n_groups = (B + P.group_seqs - 1) / P.group_seqs;
    if ((size_t)n_groups * (gamma + 1) > 65535u || P.group_seqs > 65535) return SV_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)wpr, (unsigned)P.group_seqs, (unsigned)(n_groups * (gamma + 1)));
    // (the testing hook's forced unit sizes also force the pruning, so that small test shapes exercise it)
    const double sets = (double)((size_t)wpr * P.group_seqs * n_groups * (gamma + 1)) / (double)capacity;
    P.prune = g_lane.load() != 0 || sets > 1.0 ? 1 : 0;
    P.skip_last = P.prune;
    // How a position learns w_i.  From the leader of the position before, one word handed on from position to position, where a
    // position takes longer than that trip (about 2 us): the least to read (B = 1024, gamma = 8, V = 256000 1369 us against 1401, B = 64,
    // V = 128256 50.1 against 52.9, host included).  Else from the ratios of all earlier positions, which their leaders publish without
    // waiting for each other: gamma = 16, V = 128256, bf16, 1.3 / 3.8 / 6.4 resident sets 20 / 35 / 51 us against 43 / 49 / 58 with the
    // chain, gamma = 8 21 / 37 / 52 against 29 / 37 / 50, gamma = 2 the same either way; half as many workgroups are
    // there to pass the time where sequences bring their own draft lengths (gamma = 8, 6.4 sets: 37 / 37).  Where every S_i is
    // reported nobody asks for w_i before the row's words are in, which favours the chain earlier (gamma = 8: 2.4 sets 30 / 30, 3.6 sets
    // 37 / 35); the line is the same nevertheless: the two ways round log2 w_i differently, and the report changes no decision.
    const int forced_chain = g_chain.load();
    const bool in_chain = large || (P.prune && (forced_chain >= 0 ? forced_chain != 0 : sets > (draft_lens ? 0.9 : 0.45) * gamma));
    if (g_path.load() == 0 && V <= kRowsMaxRow) {
        const sv_status_t st = launch_rows<T, ALIGNED>(P, in_chain, stream);
        if (st == SV_OK) g_last_chain.store(in_chain ? 1 : 0);
        if (st != SV_ERR_UNSUPPORTED) return st;
    }
    (in_chain ? chain : ratios)<<<grid, kThreads, 0, stream>>>(P);
    if (nu != L.nu) {
        P.nu = L.nu;
        clear_next_words_kernel<<<dim3((unsigned)B, (unsigned)(gamma + 1)), kWave, 0, stream>>>(P);
    }
    g_last_chain.store(in_chain ? 1 : 0);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

std::mutex g_null_stream_mutex;          // over the two launches of a drafting call on the null stream

// A number for a drafting call of one launch, never 0: other than that of the 2^32 calls before (see sample.hpp).
unsigned sample_call_number()
{
    static std::atomic<unsigned> next{1};
    unsigned n;
    do n = next.fetch_add(1); while (n == 0);
    return n;
}

// The drafting step: how many waves share a row.  (`split`: rows spread over the device, through `entries`, or NULL: the null stream's.)
template <typename T>
sv_status_t launch_sample(const void *logits_v, int rows, int V, float k, const float *uniforms, int32_t *tokens, bool split, SampleEntry *entries, hipStream_t stream)
{
    const T *logits = static_cast<const T *>(logits_v);
    if (split) {
        const int units = (V - 1) / kSampleUnit + 1;
        const dim3 grid((unsigned)((units - 1) / kWaves + 1), (unsigned)rows);
        if (!entries && units <= kSampleOneUnits && (long long)grid.x * rows <= kSampleOneLaunch) {
            sample_units_kernel<T, true><<<grid, kThreads, 0, stream>>>(logits, V, units, k, uniforms, tokens, nullptr, sample_call_number(), g_spin_limit.load());
        } else {
            std::unique_lock<std::mutex> lock(g_null_stream_mutex, std::defer_lock);
            if (!entries) lock.lock();
            sample_units_kernel<T, false><<<grid, kThreads, 0, stream>>>(logits, V, units, k, uniforms, tokens, entries, 0, 0);
            sample_finish_kernel<T><<<(unsigned)rows, kWave, 0, stream>>>(logits, V, units, k, uniforms, entries, tokens);
        }
        return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
    }
    // (no kernel that takes more than kSampleManyRows rows has more than 256 threads for one)
    constexpr int kStep = 1 << 23;
    static_assert((unsigned long long)kStep * kThreads <= kMaxLaunchThreads, "one launch per step");
    for (int left = rows; left > 0; left -= kStep) {
        const int n = left < kStep ? left : kStep;
        if (V <= kSampleSerial)
            sample_short_rows_kernel<T><<<(unsigned)((n - 1) / kThreads + 1), kThreads, 0, stream>>>(logits, n, V, k, uniforms, tokens);
        else if (V <= 16 * kLaneSmall)
            sample_small_rows_kernel<T, 16><<<(unsigned)((n - 1) / (kThreads / 16) + 1), kThreads, 0, stream>>>(logits, n, V, k, uniforms, tokens);
        else if (V <= kSampleUnit)
            sample_small_rows_kernel<T, 64><<<(unsigned)((n - 1) / kWaves + 1), kThreads, 0, stream>>>(logits, n, V, k, uniforms, tokens);
        else if (V <= 4 * kSampleUnit || rows >= kSampleManyRows)
            sample_rows_kernel<T, 4><<<(unsigned)n, 4 * kWave, 0, stream>>>(logits, V, k, uniforms, tokens);
        else
            sample_rows_kernel<T, 16><<<(unsigned)n, 16 * kWave, 0, stream>>>(logits, V, k, uniforms, tokens);
        if (hipGetLastError() != hipSuccess) return SV_ERR_HIP;
        logits += (size_t)n * V; uniforms += n; tokens += n;
    }
    return SV_OK;
}

sv_status_t verify_entry(int algo, bool probs, const void *target, const void *draft, const int32_t *tokens, const int32_t *draft_lens,
                         int64_t target_row_stride, int64_t draft_row_stride,
                         const float *uniforms, int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype,
                         float temperature, void *workspace, size_t workspace_bytes,
                         int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream_v)
{
    if (!target || !draft || !tokens || !uniforms || !workspace || !accept_len || !next_token)
        return SV_ERR_INVALID_ARG;
    if (B < 1 || gamma < 1 || V < 1) return SV_ERR_INVALID_ARG;
    if (!probs && (!(temperature > 0.f) || !isfinite(temperature))) return SV_ERR_INVALID_ARG;
    if (dtype != SV_DTYPE_F32 && dtype != SV_DTYPE_BF16) return SV_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SV_ERR_INVALID_ARG;
    Layout L;
    if (!make_layout(B, gamma, V, L)) return SV_ERR_UNSUPPORTED;
    if (workspace_bytes < L.total) return SV_ERR_WORKSPACE_TOO_SMALL;

    const double kd = 1.4426950408889634074 / (double)temperature;
    const float k = (float)kd;
    const size_t esize = dtype == SV_DTYPE_F32 ? 4 : 2;
    // rows are V logits, target_row_stride / draft_row_stride elements apart (0: dense, the stride is V)
    if (target_row_stride < 0 || draft_row_stride < 0) return SV_ERR_INVALID_ARG;
    const size_t tstride = target_row_stride ? (size_t)target_row_stride : (size_t)V;
    const size_t dstride = draft_row_stride ? (size_t)draft_row_stride : (size_t)V;
    if (tstride < (size_t)V || dstride < (size_t)V) return SV_ERR_INVALID_ARG;
    const bool aligned = ((reinterpret_cast<uintptr_t>(target) | reinterpret_cast<uintptr_t>(draft)) & 15u) == 0 &&
                         ((size_t)V * esize) % 16 == 0 && (tstride * esize) % 16 == 0 && (dstride * esize) % 16 == 0;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    char *ws = static_cast<char *>(workspace);
    g_last_form.store(0);
    // Launches of `threads` threads per sequence along x, as many as kMaxLaunchThreads asks for (nearly always one), equally
    // large: `launch` gets the arguments of its sequences.  What they leave in the scratch areas is their own.
    auto in_slices = [&](unsigned long long threads, auto launch) {
        if (threads > kMaxLaunchThreads) return SV_ERR_UNSUPPORTED;
        const long long most = (long long)(kMaxLaunchThreads / threads), slices = (B - 1) / most + 1, step = (B - 1) / slices + 1;
        for (long long b = 0; b < B; b += step) {
            const size_t t = (size_t)b * (gamma + 1), d = (size_t)b * gamma;
            const sv_status_t st = launch(static_cast<const void *>(static_cast<const char *>(target) + t * tstride * esize),
                                          static_cast<const void *>(static_cast<const char *>(draft) + d * dstride * esize), tokens + d,
                                          draft_lens ? draft_lens + b : nullptr, uniforms + t, (int)(b + step < B ? step : B - b),
                                          accept_len + b, next_token + b, debug_out ? debug_out + 3 * t : nullptr);
            if (st != SV_OK) return st;
        }
        return SV_OK;
    };
    // (what `launch` takes: the names of this function's arguments, of the slice)
#define SV_SLICE const void *target, const void *draft, const int32_t *tokens, const int32_t *draft_lens, const float *uniforms, \
                 int B, int32_t *accept_len, int32_t *next_token, float *debug_out
    const unsigned long long chunk_threads = (2ull * gamma + 1) * L.nchunks * kThreads;      // a workgroup per chunk of every row
    if (probs) {
#define SV_PROBS(TT, AL) launch_probs<TT, AL>(algo, target, draft, tokens, draft_lens, tstride, dstride, uniforms, B, gamma, V, \
                                              L, ws, accept_len, next_token, debug_out, stream)
        g_last_kernel.store(SV_KERNEL_PROBS);
        return in_slices(chunk_threads, [&](SV_SLICE) {
            return dtype == SV_DTYPE_F32 ? (aligned ? SV_PROBS(float, true) : SV_PROBS(float, false))
                                         : (aligned ? SV_PROBS(bf16_t, true) : SV_PROBS(bf16_t, false)); });
#undef SV_PROBS
    }
    const int path = g_path.load();
    if (path == 2 && !L.fused_ok) return SV_ERR_UNSUPPORTED;
    // sequences small enough for one workgroup each need nothing between workgroups (the testing hook asks for those of
    // them that fit LDS)
    if (path == 5 && !tiny_ok(gamma, V)) return SV_ERR_UNSUPPORTED;
    if (path == 5 || (path == 0 && !(V > kSmallMaxRow && (long long)B * (gamma + 1) > kTinyFewRows))) {
        const int magic = workspace_magic(B, gamma, V);
#define SV_TINY(TT) launch_tiny<TT>(algo, target, draft, tokens, draft_lens, tstride, dstride, uniforms, B, gamma, V, k, kd, magic, ws, \
                                    accept_len, next_token, debug_out, stream)
        const sv_status_t st = in_slices(kTinyThreads, [&](SV_SLICE) { return dtype == SV_DTYPE_F32 ? SV_TINY(float) : SV_TINY(bf16_t); });
#undef SV_TINY
        if (st != SV_ERR_UNSUPPORTED) { g_last_kernel.store(SV_KERNEL_TINY); return st; }
    }

#define SV_ARGS algo, target, draft, tokens, draft_lens, tstride, dstride, uniforms, B, gamma, V, k, kd, L, ws, \
                accept_len, next_token, debug_out, stream
#define SV_DISPATCH(FN)                                                                   \
    (dtype == SV_DTYPE_F32 ? (aligned ? FN<float, true>(SV_ARGS) : FN<float, false>(SV_ARGS)) \
                           : (aligned ? FN<bf16_t, true>(SV_ARGS) : FN<bf16_t, false>(SV_ARGS)))
    // calls of few resident sets: the kernels without a row leader's second look at the logits
    if ((path >= 7 || path == 0) && L.fused_ok) {
        const sv_status_t st = SV_DISPATCH(launch_resident);
        if (st == SV_OK) g_last_kernel.store(SV_KERNEL_RESIDENT);
        if (st != SV_ERR_UNSUPPORTED || path >= 7) return st;
    } else if (path >= 7) {
        return SV_ERR_UNSUPPORTED;
    }
    // the fused kernel (every logit read once) is the default; the staged kernels (every logit read twice)
    // take the shapes it does not: rows of more than kMaxUnitsPerRow wave chunks, or rows too wide to fit
    // four times into the device's resident set
    if (path != 1 && L.fused_ok) {
        const sv_status_t st = SV_DISPATCH(launch_fused);
        if (st == SV_OK) g_last_kernel.store(SV_KERNEL_FUSED);
        if (st != SV_ERR_UNSUPPORTED || path == 2) return st;
    } else if (path == 2) {
        return SV_ERR_UNSUPPORTED;
    }
    g_last_kernel.store(SV_KERNEL_STAGED);
    return in_slices(chunk_threads, [&](SV_SLICE) { return SV_DISPATCH(launch_staged); });
#undef SV_DISPATCH
#undef SV_ARGS
#undef SV_SLICE
}

// ---- the workspace of spec_verify_ex_noalloc: device memory that belongs to the library's code object, one copy per
// GPU that runs it, alive until the process ends.  The name below is only a handle for hipGetSymbolAddress: the
// address that kernels get is looked up once per device and kept.
__device__ __align__(256) unsigned char g_static_scratch[SV_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
struct StaticScratch {
    void *ptr = nullptr;                 // the array's address on this device
    int32_t B = 0, gamma = 0, V = 0;     // the shape its control words were last prepared for (0: never)
};
std::mutex g_static_mutex;
StaticScratch g_static[kMaxDevices];

}  // namespace

extern "C" {

size_t spec_verify_workspace_bytes(int32_t B, int32_t gamma, int32_t V)
{
    Layout L;
    return make_layout(B, gamma, V, L) ? L.total : 0;
}

sv_status_t spec_verify_workspace_init(void *workspace, size_t workspace_bytes,
                                       int32_t B, int32_t gamma, int32_t V, void *stream)
{
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return SV_ERR_INVALID_ARG;
    if (B < 1 || gamma < 1 || V < 1) return SV_ERR_INVALID_ARG;
    Layout L;
    if (!make_layout(B, gamma, V, L)) return SV_ERR_UNSUPPORTED;
    if (workspace_bytes < L.total) return SV_ERR_WORKSPACE_TOO_SMALL;
    const size_t blocks = (L.control_words + 255) / 256;
    const unsigned grid = (unsigned)(blocks < 65536 ? blocks : 65536);
    workspace_init_kernel<<<grid, 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<int *>(workspace), L.control_words, workspace_magic(B, gamma, V));
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

sv_status_t spec_verify_workspace_check(const void *workspace, int32_t B, int32_t gamma, int32_t V, void *stream)
{
    if (!workspace) return SV_ERR_INVALID_ARG;
    int words[2] = {0, 0};
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(words, workspace, sizeof(words), hipMemcpyDeviceToHost, s) != hipSuccess) return SV_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return SV_ERR_HIP;
    if (words[kHdrMagic] != workspace_magic(B, gamma, V)) return SV_ERR_INVALID_ARG;
    return words[kHdrError] == 0 ? SV_OK : SV_ERR_INTERNAL;
}

int32_t spec_verify_debug_last_kernel(void) { return g_last_kernel.load(); }

int32_t spec_verify_debug_last_chain(void) { return g_last_chain.load(); }

int32_t spec_verify_debug_last_together(void) { return g_last_together.load(); }

int32_t spec_verify_debug_last_form(void) { return g_last_form.load(); }

void spec_verify_debug_config(int32_t path, int32_t spin_limit)
{
    const bool fused_form = path == 3 || path == 4 || path == 6;
    g_path.store((path >= 0 && path <= 2) || path == 5 || (path >= 7 && path <= 9) ? path : fused_form ? 2 : 0);
    g_lane.store(path == 4 ? kLaneLarge : fused_form ? kLaneSmall : 0);
    g_chain.store(fused_form ? path != 6 : -1);
    g_spin_limit.store(spin_limit >= 0 ? spin_limit : kDefaultSpinLimit);
}

// Plain copy, 16 bytes per thread and step: what the HBM traffic counters are calibrated against.
namespace { __global__ __launch_bounds__(256) void copy_probe_kernel(uint4 *dst, const uint4 *src, size_t nvec)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (size_t)gridDim.x * 256) dst[i] = src[i];
} }

sv_status_t spec_verify_debug_copy(void *dst, const void *src, size_t bytes, void *stream)
{
    if (!dst || !src || bytes == 0 || bytes % 16 != 0) return SV_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15u) != 0) return SV_ERR_INVALID_ARG;
    const size_t nvec = bytes / 16;
    const size_t blocks = (nvec + 255) / 256;
    copy_probe_kernel<<<(unsigned)(blocks < 65536 ? blocks : 65536), 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<uint4 *>(dst), static_cast<const uint4 *>(src), nvec);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

// What a one-pass kernel of the fused kernel's launch shape can reach: one 256-thread workgroup per 2 x 16 KB (a wave
// reads 4 KB of each of two buffers with eight 16-byte loads per lane, all issued up front), the first sweep's
// arithmetic on bf16 (unpack, maximum, exp2, sum), no traffic between workgroups.  Its registers would let eight waves
// share a SIMD; the launch asks for kProbeLdsBytes of LDS per workgroup so that five workgroups fit a compute unit, as
// with the verifying kernel (five times 32 KiB do not fit beside what the hardware keeps of the 160 KiB for itself:
// 32768 bytes give four workgroups, 32000 give five - found by timing the probe with waits over a range of sizes).
constexpr unsigned kProbeLdsBytes = 32000;
namespace { __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
void stream_probe_kernel(const uint4 *a, const uint4 *b, float *out, int short_waits, int long_waits)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint4 *pa = a + (size_t)blockIdx.x * 1024 + wave * 256 + lane;
    const uint4 *pb = b + (size_t)blockIdx.x * 1024 + wave * 256 + lane;
    uint4 va[4], vb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) va[j] = load_streamed(pa + j * 64);
#pragma unroll
    for (int j = 0; j < 4; ++j) vb[j] = load_streamed(pb + j * 64);
    float res = 0.f;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint4 *v = r ? vb : va;
        float x[32];
#pragma unroll
        for (int j = 0; j < 4; ++j) unpack_vec<bf16_t>(v[j], x + j * 8);
        float shift;
        const u64 word = first_sweep_row(x, 1.8f, shift);
        res += stat_sum(word) + shift;
    }
    // the waits of a verifying kernel, modelled: a workgroup keeps its registers for a while after its sweep (the look
    // at log2 w_i; for one in four "rows" of 16 neighbouring workgroups the wait for the row and the second sweep)
    const int waits = ((blockIdx.x >> 4) & 3) == 0 ? long_waits : short_waits;
    if (waits > 0) {
        __syncthreads();
        for (int i = 0; i < waits; ++i) __builtin_amdgcn_s_sleep(8);        // 512 clocks each
        __syncthreads();
    }
    if (lane == 0) out[(size_t)blockIdx.x * 4 + wave] = res;
} }

sv_status_t spec_verify_debug_stream_probe(const void *a, const void *b, size_t bytes_each, float *out,
                                           int32_t short_waits, int32_t long_waits, void *stream)
{
    if (!a || !b || !out || bytes_each == 0 || bytes_each % 16384 != 0) return SV_ERR_INVALID_ARG;
    if (short_waits < 0 || long_waits < 0 || short_waits > 64 || long_waits > 64) return SV_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15u) != 0) return SV_ERR_INVALID_ARG;
    const size_t blocks = bytes_each / 16384;
    if (blocks > 0x7fffffffull) return SV_ERR_UNSUPPORTED;
    stream_probe_kernel<<<(unsigned)blocks, 256, kProbeLdsBytes, static_cast<hipStream_t>(stream)>>>(
        static_cast<const uint4 *>(a), static_cast<const uint4 *>(b), out, short_waits, long_waits);
    return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_HIP;
}

size_t spec_sample_workspace_bytes(int64_t rows, int32_t V)
{
    if (rows < 1 || V < 1) return 0;
    const int units = (V - 1) / kSampleUnit + 1;
    return units > kSampleMinSplit && units <= kSampleSplitUnits && rows <= (int64_t)kSampleSplitRows * units ? (size_t)rows * units * sizeof(SampleEntry) : 0;
}

sv_status_t spec_sample_tokens_ws(const void *logits, int64_t rows, int32_t V, sv_dtype_t dtype, float temperature,
                                  const float *uniforms, int32_t *tokens, void *workspace, size_t workspace_bytes, void *stream_v)
{
    if (!logits || !uniforms || !tokens) return SV_ERR_INVALID_ARG;
    if (rows < 1 || V < 1) return SV_ERR_INVALID_ARG;
    if (!(temperature > 0.f) || !isfinite(temperature)) return SV_ERR_INVALID_ARG;
    if (dtype != SV_DTYPE_F32 && dtype != SV_DTYPE_BF16) return SV_ERR_INVALID_ARG;
    if (rows > 0x7fffffffll) return SV_ERR_UNSUPPORTED;
    const size_t wanted = spec_sample_workspace_bytes(rows, V);
    if ((reinterpret_cast<uintptr_t>(workspace) & 15u) != 0) return SV_ERR_INVALID_ARG;
    if (workspace && workspace_bytes < wanted) return SV_ERR_WORKSPACE_TOO_SMALL;
    SampleEntry *const entries = static_cast<SampleEntry *>(workspace);
    const bool null_stream = !workspace && !stream_v && wanted && wanted <= (size_t)kSampleOwnEntries * sizeof(SampleEntry);
    const bool split = wanted && (workspace || null_stream);
    const float k = (float)(1.4426950408889634074 / (double)temperature);
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    return dtype == SV_DTYPE_F32
        ? launch_sample<float>(logits, (int)rows, V, k, uniforms, tokens, split, entries, stream)
        : launch_sample<bf16_t>(logits, (int)rows, V, k, uniforms, tokens, split, entries, stream);
}

sv_status_t spec_sample_tokens(const void *logits, int64_t rows, int32_t V, sv_dtype_t dtype, float temperature,
                               const float *uniforms, int32_t *tokens, void *stream_v)
{
    return spec_sample_tokens_ws(logits, rows, V, dtype, temperature, uniforms, tokens, nullptr, 0, stream_v);
}

#ifdef SV_PROFILE
void spec_verify_debug_profile(void *device_buffer)
{
    g_prof.store(static_cast<long long *>(device_buffer));
}
#endif

sv_status_t spec_verify_block(const void *target_logits, const void *draft_logits,
                              const int32_t *draft_tokens, const float *uniforms,
                              int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype,
                              float temperature, void *workspace, size_t workspace_bytes,
                              int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream)
{
    return verify_entry(kBlock, false, target_logits, draft_logits, draft_tokens, nullptr, 0, 0, uniforms, B, gamma, V, dtype,
                        temperature, workspace, workspace_bytes, accept_len, next_token, debug_out, stream);
}

sv_status_t spec_verify_token(const void *target_logits, const void *draft_logits,
                              const int32_t *draft_tokens, const float *uniforms,
                              int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype,
                              float temperature, void *workspace, size_t workspace_bytes,
                              int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream)
{
    return verify_entry(kToken, false, target_logits, draft_logits, draft_tokens, nullptr, 0, 0, uniforms, B, gamma, V, dtype,
                        temperature, workspace, workspace_bytes, accept_len, next_token, debug_out, stream);
}

sv_status_t spec_verify_greedy(const void *target_logits, const void *draft_logits,
                               const int32_t *draft_tokens, const float *uniforms,
                               int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype,
                               float temperature, void *workspace, size_t workspace_bytes,
                               int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream)
{
    return verify_entry(kGreedy, false, target_logits, draft_logits, draft_tokens, nullptr, 0, 0, uniforms, B, gamma, V, dtype,
                        temperature, workspace, workspace_bytes, accept_len, next_token, debug_out, stream);
}

sv_status_t spec_verify_ex(sv_algo_t algo, const void *target_logits, const void *draft_logits,
                           const int32_t *draft_tokens, const int32_t *draft_lens,
                           int64_t target_row_stride, int64_t draft_row_stride, const float *uniforms,
                           int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype,
                           float temperature, void *workspace, size_t workspace_bytes,
                           int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream)
{
    if (algo != SV_ALGO_BLOCK && algo != SV_ALGO_TOKEN && algo != SV_ALGO_GREEDY) return SV_ERR_INVALID_ARG;
    const int a = algo == SV_ALGO_BLOCK ? kBlock : algo == SV_ALGO_TOKEN ? kToken : kGreedy;
    return verify_entry(a, false, target_logits, draft_logits, draft_tokens, draft_lens, target_row_stride, draft_row_stride,
                        uniforms, B, gamma, V, dtype, temperature, workspace, workspace_bytes, accept_len, next_token,
                        debug_out, stream);
}

sv_status_t spec_verify_probs(sv_algo_t algo, const void *target_probs, const void *draft_probs,
                              const int32_t *draft_tokens, const int32_t *draft_lens,
                              int64_t target_row_stride, int64_t draft_row_stride, const float *uniforms,
                              int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype,
                              void *workspace, size_t workspace_bytes,
                              int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream)
{
    if (algo != SV_ALGO_BLOCK && algo != SV_ALGO_TOKEN && algo != SV_ALGO_GREEDY) return SV_ERR_INVALID_ARG;
    const int a = algo == SV_ALGO_BLOCK ? kBlock : algo == SV_ALGO_TOKEN ? kToken : kGreedy;
    return verify_entry(a, true, target_probs, draft_probs, draft_tokens, draft_lens, target_row_stride, draft_row_stride,
                        uniforms, B, gamma, V, dtype, 1.f, workspace, workspace_bytes, accept_len, next_token,
                        debug_out, stream);
}

sv_status_t spec_verify_ex_noalloc(sv_algo_t algo, const void *target_logits, const void *draft_logits,
                                   const int32_t *draft_tokens, const int32_t *draft_lens,
                                   int64_t target_row_stride, int64_t draft_row_stride, const float *uniforms,
                                   int32_t B, int32_t gamma, int32_t V, sv_dtype_t dtype, float temperature,
                                   int32_t *accept_len, int32_t *next_token, float *debug_out, void *stream)
{
    if (algo != SV_ALGO_BLOCK && algo != SV_ALGO_TOKEN && algo != SV_ALGO_GREEDY) return SV_ERR_INVALID_ARG;
    if (B < 1 || gamma < 1 || V < 1) return SV_ERR_INVALID_ARG;
    Layout L;
    if (!make_layout(B, gamma, V, L)) return SV_ERR_UNSUPPORTED;
    if (L.total > (size_t)SV_STATIC_SCRATCH_BYTES) return SV_ERR_STATIC_SCRATCH_TOO_SMALL;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SV_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return SV_ERR_UNSUPPORTED;
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_static_mutex);
        StaticScratch &st = g_static[dev];
        if (!st.ptr) {
            // once per device, with that device current: every GPU holds its own copy of the array at its own address
            void *p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)) != hipSuccess || !p) return SV_ERR_HIP;
            st.ptr = p;
        }
        ws = st.ptr;
        if (st.B != B || st.gamma != gamma || st.V != V) {
            // the array keeps what the last call left: its control words are prepared again whenever the shape changes
            // (a kernel on the caller's stream, in front of the verification's)
            const sv_status_t rc = spec_verify_workspace_init(ws, SV_STATIC_SCRATCH_BYTES, B, gamma, V, stream);
            if (rc != SV_OK) return rc;
            st.B = B; st.gamma = gamma; st.V = V;
        }
    }
    const int a = algo == SV_ALGO_BLOCK ? kBlock : algo == SV_ALGO_TOKEN ? kToken : kGreedy;
    return verify_entry(a, false, target_logits, draft_logits, draft_tokens, draft_lens, target_row_stride, draft_row_stride,
                        uniforms, B, gamma, V, dtype, temperature, ws, SV_STATIC_SCRATCH_BYTES, accept_len, next_token,
                        debug_out, stream);
}

sv_status_t spec_verify_call(const sv_call_t *c)
{
    if (!c) return SV_ERR_INVALID_ARG;
    const sv_algo_t algo = (sv_algo_t)c->algo;
    const sv_dtype_t dtype = (sv_dtype_t)c->dtype;
    switch (c->inputs) {
    case SV_CALL_LOGITS:
        return spec_verify_ex(algo, c->target, c->draft, c->draft_tokens, c->draft_lens, c->target_row_stride, c->draft_row_stride,
                              c->uniforms, c->B, c->gamma, c->V, dtype, (float)c->temperature, c->workspace, (size_t)c->workspace_bytes,
                              c->accept_len, c->next_token, c->debug_out, c->stream);
    case SV_CALL_PROBS:
        return spec_verify_probs(algo, c->target, c->draft, c->draft_tokens, c->draft_lens, c->target_row_stride, c->draft_row_stride,
                                 c->uniforms, c->B, c->gamma, c->V, dtype, c->workspace, (size_t)c->workspace_bytes,
                                 c->accept_len, c->next_token, c->debug_out, c->stream);
    case SV_CALL_LOGITS_NOALLOC:
        return spec_verify_ex_noalloc(algo, c->target, c->draft, c->draft_tokens, c->draft_lens, c->target_row_stride, c->draft_row_stride,
                                      c->uniforms, c->B, c->gamma, c->V, dtype, (float)c->temperature, c->accept_len, c->next_token,
                                      c->debug_out, c->stream);
    }
    return SV_ERR_INVALID_ARG;
}

const char *spec_verify_status_string(sv_status_t status)
{
    switch (status) {
    case SV_OK: return "ok";
    case SV_ERR_INVALID_ARG: return "invalid argument";
    case SV_ERR_UNSUPPORTED: return "unsupported size";
    case SV_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case SV_ERR_HIP: return "HIP call failed";
    case SV_ERR_INTERNAL: return "a bounded wait inside the kernel ran out";
    case SV_ERR_STATIC_SCRATCH_TOO_SMALL: return "the sizes need more than the library's built-in scratch memory";
    }
    return "unknown status";
}

}  // extern "C"
