// Exact per-query-head top-k selection on gfx950 without sorting (the selection step after the
// retrieval equation in "Compressed-Domain Top-k Retrieval").
//
// Level 1: a 512-bin histogram of a monotone map of the score (built while scoring, or by the
// two stand-alone kernels below) locates the threshold bin b*: every token in a bin above b* is
// selected; tokens inside b* are candidates.
// Level 2: the candidates (typically L / 1000 of them) are gathered by all workgroups of the
// query head and ranked exactly by (score desc, index asc) by the last workgroup to finish, which
// fills the remaining k - c_gt slots.  A workgroup's place in the index list follows from the histograms of the
// chunks before its own, so the list has one order whatever the order of arrival.  If the threshold
// bin holds more than kCandCap tokens (degenerate score distributions, e.g. all scores equal) the same
// workgroup falls back to an 8-bit radix select over the bin's members, still exact (the list's order is then
// open among the members of that bin).
#include "sik_device.h"
#include "sik_internal.h"
#include "sik_select.h"

namespace sik {

SIK_TL_DEFINE(sik_dbg_tl_topk)

constexpr int kSelPer = 16;   // scores a thread of the select kernel holds in registers at a time
constexpr int kSelBig = 512;  // its workgroup size for chunks of more than kSelPer * kBlock scores

// ---- stand-alone level 1, pass A: min and max of the order-preserving keys of each chunk ----
// Also clears the counters of its row for the kernels that follow (chunk 0), so that no launch has to do it first: with
// what select_kernel gained, scoring, top-k and attention of 2 x 32 heads x 20000 as separate calls 39.6 -> 36.4 us
// (cards and runs differ by up to 2).
__global__ __launch_bounds__(kBlock) void minmax_kernel(const float* __restrict__ scores,
                                                        const int32_t* __restrict__ seq_len,
                                                        uint32_t* __restrict__ counters,
                                                        uint2* __restrict__ minmax, int Hq, int Lmax, int nchunk,
                                                        int chunk) {
    __shared__ uint32_t smin[kBlock / kWave], smax[kBlock / kWave];
    const int row = blockIdx.x / nchunk, c = blockIdx.x % nchunk, tid = threadIdx.x;
    int L = seq_len[row / Hq];
    L = L > Lmax ? Lmax : L;
    if (c == 0 && tid < 8) counters[row * 8 + tid] = 0u;
    const int start = c * chunk, end = min(L, start + chunk);
    if (start >= end) return;
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    const float* s = scores + static_cast<size_t>(row) * Lmax;
#pragma unroll 8
    for (int i = start + tid; i < end; i += kBlock) {
        const uint32_t key = float_to_key(s[i]);
        kmin = min(kmin, key);
        kmax = max(kmax, key);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        kmin = min(kmin, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmin), o, 64)));
        kmax = max(kmax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmax), o, 64)));
    }
    if ((tid & 63) == 0) {
        smin[tid >> 6] = kmin;
        smax[tid >> 6] = kmax;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) {
            kmin = min(kmin, smin[w]);
            kmax = max(kmax, smax[w]);
        }
        minmax[row * nchunk + c] = make_uint2(kmin, kmax);
    }
}

// ---- stand-alone level 1, pass B: per-chunk histograms over [min, max] -----------------------
__global__ __launch_bounds__(kBlock) void hist_kernel(const float* __restrict__ scores,
                                                      const int32_t* __restrict__ seq_len,
                                                      const uint2* __restrict__ minmax,
                                                      uint32_t* __restrict__ parthist,
                                                      float* __restrict__ binp, int Hq, int Lmax, int nchunk,
                                                      int chunk) {
    __shared__ uint32_t lhist[kBins];
    const int row = blockIdx.x / nchunk, c = blockIdx.x % nchunk, tid = threadIdx.x;
    int L = seq_len[row / Hq];
    L = L < 0 ? 0 : (L > Lmax ? Lmax : L);
    const int start = c * chunk, end = min(L, start + chunk);
    if (start >= L && c != 0) return;
    // one lane per chunk that holds tokens (at most kMaxChunks); every wavefront reduces the row's pairs itself
    static_assert(kMaxChunks <= kWave, "one lane per chunk");
    uint2 mm = make_uint2(0xffffffffu, 0u);
    if ((tid & 63) * static_cast<int64_t>(chunk) < L) mm = minmax[row * nchunk + (tid & 63)];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        mm.x = min(mm.x, static_cast<uint32_t>(__shfl_xor(static_cast<int>(mm.x), o, 64)));
        mm.y = max(mm.y, static_cast<uint32_t>(__shfl_xor(static_cast<int>(mm.y), o, 64)));
    }
    const float lo = key_to_float(mm.x);
    const float hi = key_to_float(mm.y);
    const float span = hi - lo;
    const float scale = (span > 1e-30f && span < 3.0e38f) ? static_cast<float>(kBins) / span : 0.0f;
    if (c == 0 && tid == 0) {
        binp[row * 2] = lo;
        binp[row * 2 + 1] = scale;
    }
    for (int e = tid; e < kBins; e += kBlock) lhist[e] = 0u;
    __syncthreads();
    const float* s = scores + static_cast<size_t>(row) * Lmax;
#pragma unroll 8
    for (int i = start + tid; i < end; i += kBlock) atomicAdd(&lhist[score_bin(s[i], lo, scale)], 1u);
    __syncthreads();
    publish_hist(lhist, parthist + (static_cast<size_t>(row) * nchunk + c) * kHistWords);
}

// ---- select: compaction against the threshold bin, exact resolution of the bin ---------------
// One workgroup per (row, chunk of the producer's histograms): where its tokens go in the index list is the number of
// selected ones in the chunks before it, which the histograms that it loads anyway say (a place reserved with an atomic
// made the order of the list, and with it the last bits of the softmax sums that follow it, depend on the order in which
// the workgroups arrived).  256 threads for chunks of up to 4096 scores; 512 for longer ones, whose scores pass through
// the registers in pieces of 8192, the next piece requested while one is placed (1024 threads: one workgroup per compute
// unit, sik_topk of 512 rows x 20000 57 us against 50).  Measured against chunks of at most 4096 with reserved places:
// 512 x 20000 52 -> 50 us, 32 x 131072 46 -> 31, 64 x 20000 16.5 -> 16.6; group-shared step on 4 x 8 x 64K with 8:1 GQA
// 42.8 -> 43.2.
template <int NT>
__global__ __launch_bounds__(NT, NT == kBlock ? 8 : 6) void select_kernel(
    // (the first 14 dwords arrive in scalar registers with the wavefront: what the first loads need comes first)
    const float* __restrict__ scores, const int32_t* __restrict__ seq_len, const uint32_t* __restrict__ parthist,
    const float* __restrict__ binp, int sstride, int Hq, int Lmax, int chunk, int nchunk,
    uint32_t* __restrict__ counters, uint32_t* __restrict__ cand, int32_t* __restrict__ idx, int k) {
    constexpr int kWaves = NT / kWave, kSpan = kSelPer * NT;
    // The candidate list shares its storage with the histogram staging of find_threshold (dead after the barrier that
    // follows it).
    static_assert((kBlock / kWave) * kBins <= 2 * kCandCap + 16, "the staging area fits the candidate list");
    __shared__ uint32_t h256[kBlock];
    __shared__ __align__(8) uint32_t red[2 * kCandCap + 16];
    uint32_t* const l_cand = red;
    __shared__ int s_flag, sthr[3];
    __shared__ uint32_t wsel[2][kWaves], wbefore[kBlock / kWave], s_ncand, sh[4];

    SIK_TL(8);
    const int row = blockIdx.x / nchunk, c = blockIdx.x % nchunk, tid = threadIdx.x;
    int L = seq_len[row / Hq];
    L = L < 0 ? 0 : (L > Lmax ? Lmax : L);
    const int start = c * chunk, end = min(L, start + chunk);
    if (start >= L && c != 0) return;  // chunk 0 always runs: it may have to pad the row
    const int kk = min(k, L);
    const float* s = scores + static_cast<size_t>(row) * sstride;
    int32_t* out = idx + static_cast<size_t>(row) * k;

    // threshold bin of this query head from the chunk histograms of the producing kernel
    const float lo = binp[row * 2], scale = binp[row * 2 + 1];
    if (tid == 0) s_ncand = 0u;
    const int nact = L > 0 ? (L + chunk - 1) / chunk : 1;  // chunks that hold tokens of this sequence
    // the scores of the first piece (nearly always the whole chunk) are requested together with the histograms, one
    // round trip for both: score x of this thread is token(base, x)
    const bool vec = (sstride & 3) == 0;  // rows are 16-byte aligned (base is a multiple of 256): vector loads
    auto token = [&](int base, int x) {
        return vec ? base + ((x >> 2) * NT + tid) * 4 + (x & 3) : base + x * NT + tid;
    };
    float v[kSelPer];
    auto load = [&](int base) {
        if (vec) {
            const float4* s4 = reinterpret_cast<const float4*>(s);
#pragma unroll
            for (int j = 0; j < kSelPer / 4; ++j) {
                const int i = token(base, 4 * j);
                const float4 f = i < end ? s4[i >> 2] : make_float4(0.f, 0.f, 0.f, 0.f);
                v[4 * j] = f.x, v[4 * j + 1] = f.y, v[4 * j + 2] = f.z, v[4 * j + 3] = f.w;
            }
        } else {
#pragma unroll
            for (int x = 0; x < kSelPer; ++x) v[x] = token(base, x) < end ? s[token(base, x)] : 0.0f;
        }
    };
    load(start);
    const PlacedHistLoads hl =
        load_chunk_hists_before(parthist + static_cast<size_t>(row) * nchunk * kHistWords, nact, c);
    const Threshold th = find_threshold<NT>(hl.all, kk, L, red, sh, sthr);
    const int bstar = th.bstar, cgt = th.cgt, nb = th.nb;
    const bool ranked = nb <= kCandCap;
    const int lane = tid & 63, wv = tid >> 6;
    // tokens of the chunks before this one that are selected (low 22 bits: at most kMaxLen) and that are candidates
    // (high 10 bits: at most kCandCap where they are ranked; that many before this chunk leave none for it)
    static_assert(kMaxLen < (1 << 22) && kCandCap <= (1 << 10), "two counts in one word");
    if (c != 0 && wv < kBlock / kWave) {
        uint32_t n = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int bin = 8 * lane + e;
            n += bin > bstar ? hl.before.cnt[e] : (bin == bstar ? hl.before.cnt[e] << 22 : 0u);
        }
        n = wave_sum(n);
        if (lane == 0) wbefore[wv] = n;
    }
    __syncthreads();
    SIK_TL(9);
    uint32_t before = 0u;
    if (c != 0) {
#pragma unroll
        for (int w = 0; w < kBlock / kWave; ++w) before += wbefore[w];
    }
    const uint32_t cand0 = before >> 22;
    uint32_t sel0 = before & ((1u << 22) - 1u);

    for (int base = start, piece = 0;; piece ^= 1) {
        // Selected scores become bits of a mask and their places follow from five ballots over the lanes' counts; a
        // counter in LDS per selected score cost a round trip for nearly every one of the kSelPer scores, as some lane
        // of the 64 has a selected one.  Candidates are rare and keep their counter: they are ranked, in any order.
        uint32_t smask = 0u;
#pragma unroll
        for (int x = 0; x < kSelPer; ++x) {
            const int i = token(base, x);
            const int bin = bstar < 0 ? 0 : score_bin(v[x], lo, scale);
            const bool in = i < end;
            smask |= (in && bin > bstar ? 1u : 0u) << x;
            if (in && bin == bstar && ranked) {
                const uint32_t pos = atomicAdd(&s_ncand, 1u);
                if (pos < static_cast<uint32_t>(kCandCap)) {
                    l_cand[2 * pos] = float_to_key(v[x]);
                    l_cand[2 * pos + 1] = static_cast<uint32_t>(i);
                }
            }
        }
        const int at0 = base;
        base += kSpan;
        // the next piece's scores travel while this one's places are found and written
        if (NT != kBlock && base < end) load(base);
        static_assert(kSelPer < 32, "a lane's count has five bits");
        const uint32_t mine = static_cast<uint32_t>(__popc(smask));
        uint32_t at = sel0, wtot = 0u;  // place of this lane's first one; selected in the wavefront
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            const uint64_t bal = __ballot((mine >> e) & 1u);
            at += static_cast<uint32_t>(__popcll(bal & ((1ull << lane) - 1ull))) << e;
            wtot += static_cast<uint32_t>(__popcll(bal)) << e;
        }
        if (lane == 0) wsel[piece][wv] = wtot;
        __syncthreads();  // (two sets of sums in turn: the next piece's are written before all have read these)
        SIK_TL(10);
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            at += w < wv ? wsel[piece][w] : 0u;
            sel0 += wsel[piece][w];
        }
        while (smask != 0u) {
            const int x = __ffs(static_cast<int>(smask)) - 1;
            smask &= smask - 1u;
            if (at < static_cast<uint32_t>(k)) out[at] = token(at0, x);
            ++at;
        }
        if (NT == kBlock || base >= end) break;
    }
    const uint32_t ncand = min(s_ncand, static_cast<uint32_t>(kCandCap));
    uint32_t* crow = cand + static_cast<size_t>(row) * kCandCap * 2;
    for (uint32_t j = tid; j < ncand; j += NT) {
        const uint32_t pos = cand0 + j;
        if (pos < static_cast<uint32_t>(kCandCap)) {
            st_agent(&crow[2 * pos], l_cand[2 * j]);
            st_agent(&crow[2 * pos + 1], l_cand[2 * j + 1]);
        }
    }

    SIK_TL(11);
    if (!last_arriver(&counters[row * 8 + 2], static_cast<uint32_t>(nact), &s_flag)) return;

    SIK_TL_ANY(12);
    // ---- last workgroup of this query head: resolve the threshold bin, pad the row ----------
    const int need = kk - min(cgt, kk);
    if (need > 0) {
        if (ranked) {
            const int n = min(nb, kCandCap);
            const int npad = (n + 7) & ~7;  // padding entries outrank nothing
            for (int j = tid; j < 2 * npad; j += NT)
                l_cand[j] = j < 2 * n ? ld_agent(&crow[j]) : ((j & 1) ? 0xffffffffu : 0u);
            __syncthreads();
            const uint2* lc2 = reinterpret_cast<const uint2*>(l_cand);
            for (int a = tid; a < n; a += NT) {
                const uint2 me = lc2[a];
                int rank = 0;
                for (int x = 0; x < npad; x += 8) {  // eight LDS reads in flight
                    uint2 o8[8];
#pragma unroll
                    for (int y = 0; y < 8; ++y) o8[y] = lc2[x + y];
#pragma unroll
                    for (int y = 0; y < 8; ++y) rank += (o8[y].x > me.x || (o8[y].x == me.x && o8[y].y < me.y)) ? 1 : 0;
                }
                if (rank < need) out[cgt + rank] = static_cast<int32_t>(me.y);
            }
        } else {
            radix_select_in_bin<NT>(s, L, lo, scale, bstar, need, out + cgt, h256, sh);
        }
    }
    for (int j = kk + tid; j < k; j += NT) out[j] = -1;
    SIK_TL_ANY(13);
}

// ---------------------------------------------------------------------------------------
// Chunks of the stand-alone histogram pass: at most kChunkCap tokens each (16-bit counts per bin and chunk) and
// at most kMaxChunks of them per row: max_len <= kMaxLen.
void hist_plan(const Dims& d, int* nchunk, int* chunk) {
    const int rows = d.rows();
    int want = (512 + rows - 1) / rows;
    if (want > kMaxChunks) want = kMaxChunks;
    int ch = (d.Lmax + want - 1) / want;
    ch = (ch + kBlock - 1) / kBlock * kBlock;
    if (ch < 2048) ch = 2048;
    if (ch > kChunkCap) ch = kChunkCap;
    *chunk = ch;
    *nchunk = (d.Lmax + ch - 1) / ch;
}

bool hist_plan_ok(const Dims& d) {
    int nchunk, chunk;
    hist_plan(d, &nchunk, &chunk);
    return chunk <= kChunkCap && nchunk <= kMaxChunks;
}

hipError_t launch_topk_hist(const Dims& d, const Workspace& w, const float* scores, const int32_t* seq_len,
                            hipStream_t s) {
    int nchunk, chunk;
    hist_plan(d, &nchunk, &chunk);
    const int grid = nchunk * d.rows();
    // the attention partials are not in use during a selection: [rows][nchunk] pairs fit their [rows][kMaxSplit] slots
    static_assert(kMaxChunks * 2 <= kMaxSplit * (kD + 2), "one (min, max) pair per chunk");
    uint2* minmax = reinterpret_cast<uint2*>(w.partial);
    minmax_kernel<<<grid, kBlock, 0, s>>>(scores, seq_len, w.counters, minmax, d.Hq, d.Lmax, nchunk, chunk);
    hist_kernel<<<grid, kBlock, 0, s>>>(scores, seq_len, minmax, w.parthist, w.binp, d.Hq, d.Lmax, nchunk,
                                        chunk);
    return hipGetLastError();
}

hipError_t launch_select(const Dims& d, const Workspace& w, bool hist_from_score, const float* scores,
                         const int32_t* seq_len, int k, int32_t* idx, hipStream_t s) {
    int nchunk, chunk, nhb;
    if (hist_from_score)
        score_plan(d, &nhb, &nchunk, &chunk);
    else
        hist_plan(d, &nchunk, &chunk);
    const bool small = chunk <= kSelPer * kBlock;
    return launch_kernel(small ? select_kernel<kBlock> : select_kernel<kSelBig>, nchunk * d.rows(), small ? kBlock : kSelBig,
                         s, scores, seq_len, w.parthist, w.binp, hist_from_score ? w.sstride : d.Lmax, d.Hq, d.Lmax,
                         chunk, nchunk, w.counters, w.cand, idx, k);
}

}  // namespace sik
