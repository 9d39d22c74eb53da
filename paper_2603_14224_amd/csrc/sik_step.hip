// Host side of the one-launch decode step: which kernel variant a layout takes (step_plan), the one-time zeroing of
// the synchronisation words, and the launch (the kernel itself: sik_step_kernel.h).
#include <atomic>

#include "sik_scan.h"
#include "sik_select.h"
#include "sik_step_args.h"

namespace sik {

// ---- host side ---------------------------------------------------------------------------------------------------
// instantiated (tokens per thread with scores in registers, further tokens with scores in LDS); chunk = 1024 x sum
constexpr int kStepT[][2] = {{1, 0}, {2, 0}, {3, 0}, {4, 0}, {6, 0}};
// instantiated tokens per thread of the variant with the 16-bit first pass (two registers per token)
constexpr int kStepFx[] = {4, 8, 12, 16, 20};
// the same for the variant with two heads to a workgroup of 512 threads; chunk = 512 x sum
constexpr int kStepPair[][2] = {{16, 0}, {24, 0}, {24, 8}, {28, 8}, {32, 8}};
// the pairs instantiated for the 2-bit cache, and with a forced set for either cache
constexpr int kStepQ2[][2] = {{1, 0}, {2, 0}, {4, 0}, {8, 0}, {12, 0}, {12, 4}, {14, 4}, {16, 4}};
constexpr int kStepForced[][2] = {{1, 0}, {4, 0}, {12, 0}, {12, 4}, {14, 4}, {16, 4}};

size_t step_sync_need(const Dims& d) {
    return kSyncHeader + static_cast<size_t>(d.rows()) * kSyncPerRow + static_cast<size_t>(d.B) * kSyncPerSeq;
}

// At least kSyncReserve words whatever the layout: the words beyond a layout's own stay zero as well, so that a workspace
// that serves several layouts in turn has zeros where the largest of them looks (without this, what a small layout's
// scoring launch leaves behind its few counters would be taken for arrivals by a larger layout's one-launch step).
// The counters of a layout that needs more lie where a smaller one keeps its histograms.  Such a layout has thousands of
// head blocks, hence one chunk each, and uses the sequences' counters only, to publish appended rows: launch_leave_clear.
size_t step_sync_words(const Dims& d) {
    const size_t need = step_sync_need(d);
    return need < kSyncReserve ? kSyncReserve : need;
}

// Upper bound of the chunks per head block any one-launch plan of this layout uses (sizes the histogram area; of pairs a
// few more would be resident in places).
int step_max_chunks(const Dims& d) {
    const int hbs = d.units() * ((d.R + kHB - 1) / kHB);
    const int byc = 320 / hbs;  // no part of this family has more compute units
    return byc < 1 ? 1 : (byc > kMaxChunks ? kMaxChunks : byc);
}

static size_t step_dyn_bytes(int heads, int chunk, int TL, int k, int* listcap) {
    const size_t hb = static_cast<size_t>(heads);
    const int cap = ((chunk < k ? chunk : k) + 7) & ~7;
    *listcap = cap;
    const size_t lists = ((hb * cap * 2 + 15) & ~size_t(15)) + hb * kCandCap * 8 +
                         static_cast<size_t>(TL) * step_threads(heads) * hb * 4;
    const size_t tail = hb * (kCandCap + 8) * 8 + hb * 2 * kCandCap * 4;
    return lists > tail ? lists : tail;
}

// The variant of the one-launch step for this layout, as a code (kStepPairCode or kStepFxCode, plus T * 100 + TL: tokens
// per thread with their scores in registers and in LDS), or 0 when none applies: the smallest chunk whose grid fits the
// device (workgroups of a head block wait for each other, so they must all be resident: one of four heads to a compute
// unit, two of two heads); a single chunk per head block needs no wait and may exceed it.
//
// Chunks of 8192 tokens and more on 16-bit rows go to the variant with two heads to a workgroup, two workgroups to a
// compute unit: the scan is bound by LDS reads and vector instructions, the gather by HBM, and with one workgroup on
// every compute unit they ran one after the other over the whole chip.  Of two workgroups the one dispatched first is served
// first, by age, so it gathers while the other one still scans.  Scanning the codes once per pair instead of once per four
// heads costs less than that gives, and groups of 3, 5 or 6 heads leave fewer table entries empty.  Us, four heads against
// two: 32 x 8 x 16K with 4:1 (512 selected) 75.7 -> 69.7 ragged; 32 x 8 x 12K with 4:1 70.8 -> 66.0; 33 x 8 x 8K with 3:1
// 78.5 -> 62.8; 16 x 8 x 16K with 5:1 71.2 -> 61.7, 7:1 79.8 -> 72.6, 8:1 84.9 -> 77.1; 16 x 8 x 20K with 8:1 115 -> 106;
// 8 x 8 x 40K with 6:1 92.9 -> 86.6; 4 x 8 x 128K with 4:1 93.3 -> 90.7; 64 x 4 x 16K with 2:1 57.9 -> 53.7; none slower.
// On 2-bit records the gather is bound by vector instructions too and there is little to overlap: 32 x 8 x 16K 60.7 us with
// four heads, 64.2 with two.
// Where a grid of pairs is resident and one of four heads is not (5:1, 6:1, 9:1, one pair to a KV head), two launches against
// two chunks of pairs: 10 x 8 x 24000 with 5:1 83 -> 64, 9 x 8 x 36800 109 -> 86, 20 x 8 x 36000 with 2:1 101 -> 83, 12 x 4 x
// 30000 with 9:1 104 -> 80, lengths falling to a quarter 127 -> 86, one long 129 -> 62.
int step_plan(const Dims& d, int k, bool appended, int cus, bool fx, bool kvq, bool forced, bool single, int* nchunk_out, size_t* dyn_out,
              int* listcap_out) {
    if (d.R < 2 || d.R > 255 || cus < 1) return 0;
    auto fits = [&](int heads, int tokens, int tl) {
        const int hbs = d.units() * ((d.R + heads - 1) / heads);
        const int chunk = step_threads(heads) * tokens;
        const int nchunk = (d.Lmax + chunk - 1) / chunk;
        if (nchunk > kMaxChunks || nchunk > step_max_chunks(d)) return false;
        const bool resident = static_cast<int64_t>(hbs) * nchunk <= static_cast<int64_t>(cus) * (heads == kHB ? 1 : 2);
        if (nchunk != 1 && (single || !resident)) return false;
        int listcap;
        const size_t dyn = step_dyn_bytes(heads, chunk, tl, k, &listcap);
        if (dyn > step_lds_budget(heads)) return false;
        *nchunk_out = nchunk;
        *dyn_out = dyn;
        *listcap_out = listcap;
        return true;
    };
    if (fx) {
        if (kvq || forced) return 0;
        for (const int t : kStepFx)
            if (fits(kHB, t, 0)) return kStepFxCode + t * 100;
        return 0;
    }
    if (forced) {
        for (const auto& tt : kStepForced)
            if (fits(kHB, tt[0] + tt[1], tt[1])) return tt[0] * 100 + tt[1];
        return 0;
    }
    if (kvq) {
        for (const auto& tt : kStepQ2)
            if (fits(kHB, tt[0] + tt[1], tt[1])) return tt[0] * 100 + tt[1];
        return 0;
    }
    for (const auto& tt : kStepT)
        if (fits(kHB, tt[0] + tt[1], tt[1])) return tt[0] * 100 + tt[1];  // both numbers in one: T * 100 + TL
    for (const auto& pp : kStepPair) {
        if (!fits(kHBPair, pp[0] + pp[1], pp[1])) continue;
        // (larger budgets in chunks beyond 12288 tokens gain 10 to 15 % with equal lengths and lose as much or more with
        // unequal ones: 4 x 8 x 64K with 8:1, 3500 selected, 131 -> 111 us and, falling to a quarter, 164 -> 180;
        // 10 x 8 x 16K 129 -> 116 and, one long, 73 -> 95)
        if (pp[1] > 0 && k > 3072) return 0;
        return kStepPairCode + pp[0] * 100 + pp[1];
    }
    return 0;
}

// Tokens of a chunk, in units of 1024, of the variant that a plan code names.
int step_chunk_k(int code) {
    const int tokens = code % 100000 / 100 + code % 100;
    return code >= kStepPairCode ? tokens / 2 : tokens;
}

// Whether the one-launch step with a single chunk per head block, of kilo x 1024 tokens, beats the two launches.  Nothing
// in it waits for another workgroup; against the two launches it saves the boundary, the scores' way through memory
// and the last workgroup's exchange, and it loses where its workgroups (one per four heads, or two per four in pairs) are
// too few for the chip.  Measured on 256 compute units with 4 % of the context selected, two launches -> one launch, us,
// by head blocks (units x ceil(R / 4)) and context:
//   rows      1000: 8 blocks 15.9 -> 12.9, 256 19.3 -> 13.6      2000: 8 blocks 16.0 -> 15.7, 128 19.2 -> 16.0
//             4096: 64 blocks 20.2 -> 21.1, 80 22.9 -> 21.2, 128 25.4 -> 22.8, 192 34.2 -> 25.6
//             6000: 80 blocks 22.9 -> 25.9, 96 32.3 -> 26.8      8192: 32 blocks 20.7 -> 23.7, 64 26.2 -> 24.5, 128 38 -> 31
//             12288: 64 blocks 32.5 -> 33.2, 80 36.9 -> 31.6, 192 81 -> 54    16384: 64 blocks 39 -> 45, 80 41.5 -> 38.7
//             20000: 80 blocks 50.6 -> 52.3, 96 72 -> 58
//             8192, 2:1: 64 blocks 22.0 -> 23.7, 80 28.1 -> 23.8; 9:1: 72 blocks 29.5 -> 23.7
//   records   1000: 8 blocks 17.6 -> 14.9      2000: 8 blocks 17.6 -> 17.7, 64 20.8 -> 17.7
//             4096: 64 blocks 22.7 -> 24.6, 128 26.0 -> 24.6, 192 35.7 -> 24.7
//             8192: 128 blocks 35.4 -> 37.3, 192 48.2 -> 37.4    12288: 128 blocks 47.0 -> 50.3, 160 68.9 -> 51.8
//   64 forced tokens (chunks of 1, 4, 12, 16 and more x 1024, one workgroup per four heads)
//   rows      1000: 8 blocks 18.4 -> 15.7      2000: 32 blocks 19.4 -> 19.1, 64 21.7 -> 19.1
//             4096: 64 blocks 24.7 -> 24.6, 96 28.5 -> 25.2, 192 41 -> 31    8192: 128 blocks 41 -> 44, 160 55 -> 45
//             16384: 160 blocks 85 -> 76
//   records   1000: 8 blocks 21.0 -> 19.3      2000: 32 blocks 21.6 -> 22.8, 64 24.5 -> 22.5
//             4096: 64 blocks 26.6 -> 29.4, 96 30.6 -> 29.7, 192 40 -> 30    8192: 128 blocks 39.8 -> 43.5, 160 54 -> 44
//             4096, 5:1: 96 blocks 26.1 -> 28.1, 128 27.5 -> 28.2; 6:1: 128 29.1 -> 28.1
// With more blocks than compute units, and with long chunks of the variants of four heads, what counts is how much of
// what either form computes is padding: the one launch goes in rounds, four heads to a block (three take nearly as long
// as four, two three quarters), the two launches in chunks of a power of two, the last one padded beyond 8192 tokens.
// `room` is the ratio of the two, head x tokens that the rounds have room for over those that the chunks have; pairs of
// heads (rows, chunks from 8192) won everywhere.  Measured at 700 shapes of 257 to 1100 blocks and 2:1 to 13:1, by room:
//   rows      2000: 1.40 39.7 -> 33.6, 1.57 32.3 -> 33.2, 1.9 31.1 -> 32.7    4096: 1.31 60 -> 53, 1.60 50.6 -> 52.0, 3.0 39 -> 44
//             6000: 1.77 69 -> 63, 1.87 86 -> 93    forced: 8192: 1.77 93 -> 86, 2.7 69 -> 83    20000: 1.3 203 -> 177, 1.9 141 -> 166
//   records   2000: 1.9 38.3 -> 33.2, 2.05 32.5 -> 33.6    4096: 1.6 57 -> 48, 2.05 45.0 -> 47.6    8192: 1.6 65.8 -> 61, 1.9 62 -> 72
//             9500: 0.92 102 -> 82    12288, 2:1: 1.39 87 -> 76; 4:1: 1.45 93 -> 99    16384: 1.33 132 -> 127, 1.6 122 -> 128, 1.9 104 -> 126
//   up to 256 blocks, four heads, chunks of 16384: 1.8 83.9 -> 73 (rows, forced), 66 -> 63 (records), 2.0 58.1 -> 56.4, 2.4 55.9 -> 62.9;
//             of 18432 and 20480: 1.45 78 -> 75, 1.73 63.7 -> 69
bool step_single_pays(const Dims& d, int kilo, bool kvq, bool forced, int cus) {
    const int blocks = d.units() * ((d.R + kHB - 1) / kHB);
    const bool full = d.R % kHB == 0 || d.R % kHB == 3;  // (nearly) all of a block's table entries in use
    const bool pairs = kilo >= 8 && !kvq && !forced;
    const int rounds = (blocks + cus - 1) / cus;
    int chunks = 1, chunk = d.Lmax;
    if (d.Lmax > 8192) fused_plan(d, &chunks, &chunk);
    const double room = static_cast<double>(rounds) * cus * kHB * (d.R == 2 ? 0.75 : 1.0) / static_cast<double>(d.rows()) *
                        d.Lmax / (static_cast<double>(chunks) * chunk);
    if (blocks > cus) {
        if (pairs) return true;
        if (kvq) return room <= (kilo <= 2 ? 2.0 : (kilo <= 4 ? (forced ? 1.78 : 1.85) : (kilo <= 8 ? 1.72 : (kilo <= 12 ? 1.42 : 1.38))));
        return room <= (kilo <= 4 ? 1.595 : 1.8);
    }
    if (kilo > 12 && !pairs) return 2 * blocks > cus && (d.R < kHB || room <= (kilo == 16 ? 2.05 : 1.7));
    if (forced && kvq && kilo == 4 && d.R > kHB && !full && d.Lmax > 3072 && 3 * d.rows() < 4 * cus) return false;
    // (one pair to a KV head, half of the compute units at most: two chunks each, where the launch is large enough for that,
    // 16 x 8 x 19544 with 1563 selected 73 -> 64 us)
    if (pairs && kilo > 16 && d.R == kHBPair && 2 * blocks <= cus) return false;
    int least;  // in sixteenths of the compute units
    if (forced)
        least = kilo == 1 ? 0 : (kilo > 4 ? 10 : (d.Lmax <= 2048 ? 4 : 6));
    else if (kvq)
        least = kilo == 1 ? 0 : (kilo == 2 ? 2 : (kilo <= 4 ? 8 : 10));
    else
        least = kilo <= 2 ? 0 : (kilo == 8 ? (8 * d.rows() < 5 * cus ? 5 : 4) : (kilo == 6 || kilo > 16 ? 6 : 5));
    return 16 * blocks >= least * cus;
}

int device_compute_units() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

__global__ void fill_zero_kernel(uint32_t* p, size_t n) {
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<size_t>(gridDim.x) * blockDim.x)
        p[i] = 0u;
}

hipError_t launch_sync_init(const Dims& d, const Workspace& w, hipStream_t s) {
    const size_t n = step_sync_words(d);
    return launch_kernel(fill_zero_kernel, static_cast<int>((n + 255) / 256 > 64 ? 64 : (n + 255) / 256), 256, s,
                         w.sync, n);
}

hipError_t launch_leave_clear(const Dims& d, const Workspace& w, hipStream_t s) {
    const size_t n = static_cast<size_t>(d.B) * kSyncPerSeq;
    return launch_kernel(fill_zero_kernel, static_cast<int>((n + 255) / 256 > 64 ? 64 : (n + 255) / 256), 256, s,
                         w.sync + kSyncHeader + static_cast<size_t>(d.rows()) * kSyncPerRow, n);
}

hipError_t launch_step(const Dims& d, const Workspace& w, int T, int nchunk, size_t dyn, int listcap, const void* q,
                       const Append& ap, const float* codebook, const uint8_t* codes, int32_t* seq_len,
                       const void* K, const void* V, const void* kvq, const float* alpha, int k, const StepOptions& fo,
                       float scale, int32_t* idx_out, void* out, hipStream_t s) {
    StepArgs a{};
    a.k_per_mille = fo.k_per_mille;
    const int spin_limit = fo.spin_limit;
    a.k_new = ap.k_new, a.v_new = ap.v_new, a.Kw = ap.K, a.Vw = ap.V, a.mu = ap.mu, a.codes_w = ap.codes;
    a.kvq = static_cast<const uint2*>(kvq), a.kvq_w = static_cast<uint2*>(ap.kvq), a.alpha = alpha;
    a.forced_idx = fo.idx, a.n_forced = fo.n, a.fK = fo.fK, a.fV = fo.fV;
    if (fo.mu) a.mu = fo.mu;  // (the same vector the append uses)
    a.parthist = w.parthist, a.pool = w.cand, a.partial = w.partial, a.scores = w.scores, a.sync = w.sync;
    a.idx_out = idx_out, a.idx_ws = w.idx, a.out = out;
    a.sstride = w.sstride, a.k = k, a.spin_limit = spin_limit > 0 ? spin_limit : (1 << 20), a.listcap = listcap;
    a.scale_log2e = (scale > 0.0f ? scale : 1.0f / sqrtf(static_cast<float>(d.D))) * 1.4426950408889634f;
    const bool out_f32 = d.out_dtype == kF32;
    if (T >= kStepPairCode)
        return d.kv_dtype == kBF16
                   ? launch_step_pair_bf16(d, T, nchunk, dyn, q, codebook, codes, seq_len, K, V, a, out_f32, s)
                   : launch_step_pair_f16(d, T, nchunk, dyn, q, codebook, codes, seq_len, K, V, a, out_f32, s);
    return d.kv_dtype == kBF16 ? launch_step_bf16(d, T, nchunk, dyn, q, codebook, codes, seq_len, K, V, a, out_f32, s)
                               : launch_step_f16(d, T, nchunk, dyn, q, codebook, codes, seq_len, K, V, a, out_f32, s);
}


}  // namespace sik
