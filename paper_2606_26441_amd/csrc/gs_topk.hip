// Exact per-query top-k over the score arrays (paper Sec. 4.2: a top-k over
// each query's accumulator row; Sec. 4.3: the result is exact).
//
// Every document is ranked by the 64-bit composite key
//     c = (score bits << 32) | (uint32)~doc_id
// Non-negative fp32 and int32 scores are monotone in their bit patterns, and
// ~id reverses the id order, so "c descending" is exactly "score descending,
// then doc id ascending", and all composites are distinct: the k largest
// composites are the unique answer, ties included.
//
// Pipeline for a tile of queries (all launches fixed, no host round trip):
//  1. the first 11-bit digit histogram (built by the scoring kernel);
//  2. k_select: find the digit bucket holding the k-th composite; if the composites
//     at or above that bucket fit the candidate buffer the query is resolved,
//     otherwise its workgroup refines the bucket over the full score array, 11 more
//     bits of the score per pass, then by id (massive ties at the k-th score). A query
//     that fewer than k documents match needs no pass: its answer is every positive
//     document and documents among the first k (see k_select);
//  3. k_filter: append every composite >= the threshold to the candidate buffer
//     (wavefront ballot + popcount for the append slot);
//  4. k_final: histogram selection on the candidates in 2048 bins of their range
//     (narrowed while the bin of the k-th holds too many), the winners grouped by
//     bin in LDS and each placed by its rank inside its bin. Collections of at most
//     kCandCap documents skip 1 to 3: the score row itself is the candidate set.
// bf16 form: k_final also derives the error band of the k-th approximate score and
// lists the candidates in the band; k_rescore sums them again in fp64 from the fp32
// forward rows (ascending term order) on a grid over the listed documents, and
// k_band_topk ranks them. k_band_filter handles the rare case in which the band
// reaches below the candidate threshold (a fused query first gets the rows of its
// other tiles, scoring phase 5).
//
// Fused candidate filtering (doc-tiled kernels, searches of 32+ queries): the
// seed tiles (every 8th doc tile) are scored first; k_seed_bound derives from their
// histogram a lower bound of each query's k-th composite (a bin edge, refined over
// the seed rows where too many documents reach it); the other tiles append every
// composite at or above it while they are scored (then writing no score rows for
// them and not counting them in the histogram), and step 3 scans only the seed
// tiles. A query with too many appended falls back to the full row: it is listed,
// its other tiles are scored and counted again, and a second k_select pass redoes
// its step 2 from the complete histogram before steps 3 and 4.
//
// Wide-range check (fixed-point sums of the doc-tiled kernels, fp32 and bf16
// weights): a fixed-point sum is within an absolute bound E of the exact score,
// so a score far below the query's scale can miss the relative error budget. At
// step 2 the lower edge of the k-th composite's bucket (a lower bound of the
// k-th approximate score, also with fused filtering) is compared with the
// query's limit (E over the budget). Below it, the query is listed as wide
// range: every tile is scored again with fp64 accumulation of exact fp64
// products (its histogram counted anew), and the second k_select pass selects
// from those rows.
#include <algorithm>
#include <type_traits>

#include "gs_internal.h"

namespace gs {

namespace {

__device__ __forceinline__ unsigned long long comp_key(uint32_t key, uint32_t id) {
    return ((unsigned long long)key << 32) | (unsigned long long)(~id);
}

__device__ __forceinline__ int64_t kq_of(const DevBatch& qb, int q, int64_t N) {
    return min((int64_t)qb.k[q], N);
}

// The composite of score 0 and doc id kq - 1. Documents 0 .. kq - 1 are kq composites at or
// above it, so it never exceeds the kq-th largest composite, whatever the scores.
__device__ __forceinline__ unsigned long long zero_floor(int64_t kq) { return comp_key(0u, (uint32_t)(kq - 1)); }

constexpr int kSelBS = 512;  // workgroup of the selection kernels: four histogram bins per thread
static_assert(kHistBins == 4 * kSelBS, "four bins per thread");

// What scan_bins leaves for the workgroup: the bin of the need-th largest element, the number of
// elements in the bins above it and the number in it.
struct BinScan {
    uint32_t wsum[kSelBS / kWave];
    int d;
    uint32_t above, count;
};

// The whole workgroup finds the bin d holding the need-th largest element of a kHistBins
// histogram, above(d) < need <= above(d) + h[d] (thread t holds bins 2047 - 4 t .. 2044 - 4 t,
// given top bin first in c; e receives the number of elements above each). 1 <= need; with
// fewer elements than need, d is bin 0. Ends with a barrier.
__device__ __forceinline__ void scan_bins(const uint32_t (&c)[4], uint32_t (&e)[4], uint32_t need, BinScan& sh) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const uint32_t s = c[0] + c[1] + c[2] + c[3];
    uint32_t incl = s;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t v = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += v;
    }
    if (lane == kWave - 1) sh.wsum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - s;
#pragma unroll
    for (int w = 0; w < kSelBS / kWave; w++) run += w < wave ? sh.wsum[w] : 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        e[j] = run;
        const bool last = tid == kSelBS - 1 && j == 3;
        if ((run < need && need <= run + c[j]) || (last && run + c[j] < need)) {
            sh.d = kHistBins - 1 - 4 * tid - j;
            sh.above = run;
            sh.count = c[j];
        }
        run += c[j];
    }
    __syncthreads();
}

__device__ __forceinline__ void load_bins(const uint32_t* h, uint32_t (&c)[4]) {
    const uint4 v = reinterpret_cast<const uint4*>(h)[kSelBS - 1 - (int)threadIdx.x];
    c[0] = v.w; c[1] = v.z; c[2] = v.y; c[3] = v.x;
}

// The documents of a refinement, by ascending id: a whole row, or its seed tiles (document i of
// those is document at(i) of the row). Four from a multiple of 4 on are side by side in the row,
// which is padded to a multiple of 64.
struct WholeRow {
    uint32_t n;  // below 2^31
    __device__ __forceinline__ uint32_t at(uint32_t i) const { return i; }
};
struct SeedTiles {
    uint32_t n;
    int tile_shift, stride;
    __device__ __forceinline__ uint32_t at(uint32_t i) const {
        return (((i >> tile_shift) * (uint32_t)stride) << tile_shift) + (i & ((1u << tile_shift) - 1u));
    }
};

// Four scores of documents i .. i + 3 of a lane (the last aligned four where i is past them); those
// at or past n are replaced by `none`.
template <typename Docs>
__device__ __forceinline__ uint4 load_scores(const uint32_t* Sq, const Docs& docs, uint32_t i) {
    return *reinterpret_cast<const uint4*>(Sq + docs.at(min(i, (docs.n - 1) & ~3u)));
}
__device__ __forceinline__ void mask_past(uint4& v, uint32_t i, uint32_t n, uint32_t none) {
    if (i + 3 < n) return;
    if (i >= n) v.x = none;
    if (i + 1 >= n) v.y = none;
    if (i + 2 >= n) v.z = none;
    v.w = none;
}

// Histogram copies of a refinement, one per lane modulo their number, side by side per bin.
template <int R>
constexpr int refine_copies() {
    return R == 16 ? 4 : 1;
}

// Add the scores that lie in [s_lo, s_lo + s_width) to an LDS histogram of s_width >> nsh bins.
// R rounds of 16-byte loads are issued before the first count. A thread counts scores of one bin in
// a register until one of another comes: where a refinement is needed most scores are often equal,
// and 64 adds to one LDS word take 64 clocks. The copies are for a few values among the scores (4M
// scores of two values: 1.42 -> 0.95 ms a search).
template <int R, typename Docs>
__device__ __forceinline__ void count_scores(const uint32_t* Sq, const Docs& docs, uint32_t s_lo, uint32_t s_width,
                                             int nsh, uint32_t* hist) {
    constexpr int C = refine_copies<R>();
    uint32_t* const mine = hist + (threadIdx.x & (C - 1));
    uint32_t bin = 0, n = 0;
    for (uint32_t i = 4 * threadIdx.x; i < docs.n; i += 4 * kSelBS * R) {
        uint4 v[R];
#pragma unroll
        for (int r = 0; r < R; r++) v[r] = load_scores(Sq, docs, i + r * 4 * kSelBS);
#pragma unroll
        for (int r = 0; r < R; r++) {
            mask_past(v[r], i + r * 4 * kSelBS, docs.n, s_lo + s_width);
            const uint32_t vs[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint32_t u = vs[j] - s_lo, b = u >> nsh;
                const bool in = u < s_width;
                if (in && b != bin) {
                    if (n) atomicAdd(&mine[bin * C], n);
                    bin = b;
                    n = 0;
                }
                n += in ? 1u : 0u;
            }
        }
    }
    if (n) atomicAdd(&mine[bin * C], n);
}

// The need-th document of score s, in id order (they hold that many).
template <typename Docs>
__device__ __forceinline__ uint32_t nth_of_score(const uint32_t* Sq, const Docs& docs, uint32_t s, int need,
                                                 uint32_t* cnt, uint32_t* found) {
    constexpr int R = 4, NW = kSelBS / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    for (uint32_t wb = 0; wb < docs.n; wb += 4 * kSelBS * R) {
        const uint32_t i = wb + 4 * threadIdx.x;
        uint4 v[R];
        unsigned long long m[R][4];
#pragma unroll
        for (int r = 0; r < R; r++) v[r] = load_scores(Sq, docs, i + r * 4 * kSelBS);
#pragma unroll
        for (int r = 0; r < R; r++) {
            mask_past(v[r], i + r * 4 * kSelBS, docs.n, ~s);
            m[r][0] = __ballot(v[r].x == s);
            m[r][1] = __ballot(v[r].y == s);
            m[r][2] = __ballot(v[r].z == s);
            m[r][3] = __ballot(v[r].w == s);
            if (lane == 0)
                cnt[r * NW + wave] = (uint32_t)(__popcll(m[r][0]) + __popcll(m[r][1]) + __popcll(m[r][2]) + __popcll(m[r][3]));
        }
        __syncthreads();
        int run = 0, before[R];
#pragma unroll
        for (int r = 0; r < R; r++)
            for (int w = 0; w < NW; w++) {  // in id order
                if (w == wave) before[r] = run;
                run += (int)cnt[r * NW + w];
            }
        if (run >= need) {
            const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
            for (int r = 0; r < R; r++) {
                int at = before[r];  // documents of that score before this lane's
#pragma unroll
                for (int j = 0; j < 4; j++) at += __popcll(m[r][j] & below);
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    if (!((m[r][j] >> lane) & 1ull)) continue;
                    if (++at == need) *found = docs.at(i + r * 4 * kSelBS + j);
                }
            }
            __syncthreads();
            return *found;
        }
        need -= run;
        __syncthreads();  // cnt is read
    }
    return 0xFFFFFFFFu;
}

// A composite at or below the need-th largest of the composites of a query's documents whose scores
// lie in [s_lo, s_lo + s_width), such that fits(number of those at or above it) holds, or the
// need-th largest itself. 11 bits of the score per pass; among equal scores the ids decide: the
// documents are walked from the lowest id until enough hold that score (few are read where many do).
// One workgroup reads the row, so a pass takes one CU's time (4M scores: 0.35 ms). 2M equal scores
// among 4M, fp32: 0.79 ms a search; with the scores of a tie added one by one and the id's bits as
// further digits 5.0.
template <int R, typename Docs, typename Fits>
__device__ __forceinline__ unsigned long long refine(const uint32_t* Sq, const Docs& docs, uint32_t s_lo, uint32_t s_width,
                                                     int need, Fits fits, uint32_t* hist, BinScan& sh, uint32_t* found,
                                                     int* passes, int* kept) {
    int above = 0;  // composites of the range above [s_lo, s_lo + s_width)
    constexpr int C = refine_copies<R>();
    while (s_width > 1) {
        for (int i = threadIdx.x; i < kHistBins * C / 4; i += kSelBS)
            reinterpret_cast<uint4*>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
        const int nsh = max(0, 32 - __clz((int)(s_width - 1)) - kHistBits);
        __syncthreads();
        count_scores<R>(Sq, docs, s_lo, s_width, nsh, hist);
        __syncthreads();
        uint32_t c[4], e[4];
        if constexpr (C == 1) {
            load_bins(hist, c);
        } else {
            static_assert(C == 4, "a 16-byte load per bin");
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint4 v = reinterpret_cast<const uint4*>(hist)[kHistBins - 1 - 4 * (int)threadIdx.x - j];
                c[j] = v.x + v.y + v.z + v.w;
            }
        }
        scan_bins(c, e, (uint32_t)need, sh);
        const uint32_t off = (uint32_t)sh.d << nsh;
        s_lo += off;
        s_width = min(1u << nsh, s_width - off);
        above += (int)sh.above;
        need -= (int)sh.above;
        *passes += 1;
        *kept = above + (int)sh.count;
        if (fits(*kept)) return (unsigned long long)s_lo << 32;
        __syncthreads();  // sh is read
    }
    *passes += 1;
    *kept = above + need;
    return comp_key(s_lo, nth_of_score(Sq, docs, s_lo, need, hist, found));
}

// Bins below the k-th score's that hold the bf16 error band (2^-7 of the score, at most four
// bins, and the band's absolute part); below the digit's fine range one bin of 12.5 % does.
constexpr int kBandBins = 6;

// pass 0 runs once every tile is scored; pass 1 runs after phase 3 for the queries that
// fell back, whose histograms are complete only then (phase 2 counts the seed tiles of a
// fused query only). One workgroup per query: the first digit, then, for a query whose
// threshold bucket is too large for the candidate buffer, the refinement over its row (refine; in
// this launch: as launches of their own, twelve of them, they took 2 to 4.5 us
// each also when, as usual, no query needs one: 19 of the 57 us of a search of 10,000
// documents).
// A query that fewer than kq documents match: its k-th composite has score 0, and the
// documents that can win are the positive ones and those with id below kq (zero_floor). With
// the zero-score documents counted beside the histogram, that needs no pass over the row
// (four of them before, for every short query of a rare term).
// R: loads in flight per thread of the refinement. Sixteen where there is at most one query per CU (the
// tied query of refine: 1,026 / 842 / 790 us a search at 4 / 8 / 16); four otherwise, so that the
// registers let four workgroups share a CU (4,096 queries, none refined: 1,928 us a search at 8, 1,908
// at 4).
template <int R>
__global__ __launch_bounds__(kSelBS) __attribute__((amdgpu_waves_per_eu(R == 4 ? 8 : 2))) void k_select(
    DevBatch qb, int32_t q0, int64_t N, int precision, const uint32_t* __restrict__ S, int64_t ld,
    uint32_t* __restrict__ hist1, SelState* __restrict__ state, uint32_t* __restrict__ counters,
    int32_t* __restrict__ rescore_list, int pass, int wide_check) {
    __shared__ __align__(16) uint32_t hist[kHistBins * refine_copies<R>()];
    __shared__ BinScan sh;
    __shared__ uint32_t sh_found;
    __shared__ int sh_open;
    const int tid = threadIdx.x;
    const int ql = blockIdx.x, q = q0 + ql;
    SelState* st = state + ql;
    if (pass == 1 && st->rescore == 0) return;
    const int64_t kq = kq_of(qb, q, N);
    if (kq == 0) {
        if (tid == 0) st->resolved = 2;
        return;
    }
    uint32_t* h = hist1 + (int64_t)ql * kHistBins;
    // read before the barriers below: thread 0 changes it after them
    const unsigned long long bound = st->fused == 1 ? st->bound : 0ull;
    uint32_t c[4], e[4];
    load_bins(h, c);
    scan_bins(c, e, (uint32_t)kq, sh);
    const int d = sh.d;
    const FirstDigit fd = qb.first[q];
    const unsigned long long edge = first_edge(fd, d);
    if (pass == 0 && wide_check) {
        // a lower bound of the k-th composite's score: the lower edge of its bucket, or the seed bound
        const float s_lo = __uint_as_float((uint32_t)(max(edge, bound) >> 32));
        if ((double)s_lo < qb.q_wide_lim[q]) {
            // every lane has read its bins: the fp64 pass counts anew
            reinterpret_cast<uint4*>(h)[tid] = make_uint4(0u, 0u, 0u, 0u);
            if (tid == 0) {
                st->fused = 0;
                st->n_cand = 0;
                st->zeros = 0;
                st->resolved = 0;
                st->rescore = 2;
                rescore_list[atomicAdd(&counters[kCntListed], 1u)] = ql;
            }
            return;
        }
    }
    if (tid == 0) {
        const int64_t ge = (int64_t)sh.above + sh.count;
        int64_t kept = 0;  // composites at or above the filter threshold
        int resolved = 1;
        unsigned long long lo = 0;
        if (st->fused == 1) {  // the histogram counts the seed tiles alone
            lo = bound;
            kept = st->seed_kept;
        } else if (edge == 0ull) {  // the bin that holds score 0
            lo = zero_floor(kq);
            kept = N - st->zeros + min(kq, (int64_t)st->zeros);
        } else {
            lo = edge;
            kept = ge;
        }
        if (kept > kCandCap) resolved = 0;
        const int to = max(d - kBandBins, min(d, fd.low) - 1);
        if (precision == kBF16 && resolved && lo == edge && to > 0) {
            // a few bins lower: the bf16 error band below the k-th score then lies inside the candidates
            int64_t more = 0;
            for (int j = to; j < d; j++) more += h[j];
            if (st->n_cand + kept + more <= kCandCap) {
                lo = first_edge(fd, to);
                kept += more;
            }
        }
        // Fused filtering holds the appended candidates (every composite >= the seed bound
        // of the non-seed tiles; the bound is at least the threshold) and the filter then
        // scans the seed tiles only. With too many appended they are dropped and the whole
        // row is scanned.
        int open = resolved == 0;
        if (st->fused == 1 && (!resolved || st->fused_over || (int64_t)st->n_cand + kept > kCandCap)) {
            st->fused = 0;
            st->n_cand = 0;
            st->rescore = 1;  // its non-seed rows were not written: score them again
            rescore_list[atomicAdd(&counters[kCntListed], 1u)] = ql;
            open = 0;
        }
        st->resolved = resolved;
        st->lo = lo;
        sh_open = open;
    }
    __syncthreads();
    if (!sh_open) return;
    // the threshold inside the bin, from the row (no score reaches the top bin's upper edge: the
    // digit starts from the query's largest possible one)
    const uint32_t s_lo = (uint32_t)(edge >> 32), s_hi = (uint32_t)(first_edge(fd, d + 1) >> 32);
    const int above = (int)sh.above;
    int passes = 0, kept = 0;
    const unsigned long long lo = refine<R>(
        S + (int64_t)ql * ld, WholeRow{(uint32_t)N}, s_lo, s_hi - s_lo, (int)kq - above,
        [&](int n) { return above + n <= kCandCap; }, hist, sh, &sh_found, &passes, &kept);
    if (tid == 0) {
        st->passes += passes;
        st->resolved = 1;
        st->lo = lo;
    }
}

// Fused filtering, after the seed tiles are scored: the bound of a query is the lower edge of the
// first-digit bin that holds the k-th largest composite among the seed tiles' documents (from the
// histogram they built). The k-th largest over all documents is at least as large, so the bound
// never exceeds it; neither does zero_floor, which keeps a query matched by few documents from
// appending every zero-score one. With fewer than k seed documents there is no bound.
// Where so many seed documents reach the edge that the other tiles would append more than kSeedFit
// candidates (scores that tie, or in a bin of 12.5 %), the bound is refined over the seed rows until
// they would not: the appends would pass kFusedCap and the query be scored again from its lists. Only
// there: a second digit for every query took 54 us for 500 queries of 1M documents and 128 us for
// 4,096 of 250,000, and saved 3 % of the candidates. (100 queries of 1M documents with equal scores at
// the bound: 814 -> 298 us, fp32.)
constexpr int kSeedFit = kFusedCap * 2 / 3;

__global__ __launch_bounds__(kSelBS) __attribute__((amdgpu_waves_per_eu(8))) void k_seed_bound(
    DevBatch qb, int32_t q0, int64_t N, const uint32_t* __restrict__ S, int64_t ld, const uint32_t* __restrict__ hist1,
    SelState* __restrict__ state, int tile_shift, int stride) {
    __shared__ uint32_t hist[kHistBins];
    __shared__ BinScan sh;
    __shared__ uint32_t sh_found;
    const int ql = blockIdx.x, q = q0 + ql;
    SelState* st = state + ql;
    const int64_t kq = kq_of(qb, q, N);
    if (kq == 0) return;  // fused stays 0 (cleared)
    uint32_t c[4], e[4];
    load_bins(hist1 + (int64_t)ql * kHistBins, c);
    scan_bins(c, e, (uint32_t)kq, sh);
    const int above = (int)sh.above, d = sh.d;
    int kept = above + (int)sh.count;  // seed composites at or above the bound
    if (kept < kq) return;
    const int64_t n_tiles = (N + (1ll << tile_shift) - 1) >> tile_shift, seeds = (n_tiles + stride - 1) / stride;
    const int64_t docs = ((seeds - 1) << tile_shift) + min(1ll << tile_shift, N - (((seeds - 1) * stride) << tile_shift));
    auto fits = [&](int64_t n) { return n * (N - docs) <= kSeedFit * docs; };
    const FirstDigit fd = qb.first[q];
    unsigned long long b = first_edge(fd, d);
    const unsigned long long z = zero_floor(kq);
    int64_t reach = kept;  // of them in every tile alike
    int passes = 0;
    if (b == 0ull) {       // every positive document, and the zero-score ones below id kq (in the first tile)
        reach = docs - st->zeros;
        kept = (int)(reach + min(kq, (int64_t)st->zeros));
    }
    if (!fits(reach)) {
        int n = 0;
        const uint32_t s_lo = (uint32_t)(b >> 32), s_hi = (uint32_t)(first_edge(fd, d + 1) >> 32);
        b = refine<4>(
            S + (int64_t)ql * ld, SeedTiles{(uint32_t)docs, tile_shift, stride}, s_lo, s_hi - s_lo, (int)kq - above,
            [&](int m) { return fits(above + m); }, hist, sh, &sh_found, &passes, &n);
        kept = above + n;
    }
    if (threadIdx.x != 0) return;
    st->bound = b > z ? b : z;
    st->seed_kept = kept;
    st->passes = passes;
    st->fused = 1;
}

// Append every composite >= the query's threshold to its candidate buffer.
// Each lane reads four consecutive scores with one 16-byte load (rows are
// 64-aligned). A wavefront reserves slots for its hits (ballot + popcount) in
// a workgroup-local LDS stage, so the scan never waits on a global atomic; at
// the end the workgroup takes one range of the query's buffer and copies the
// stage out. Hits that find the stage full are appended to the global buffer
// directly (slot from a global atomic), so any number of hits is handled.
// Bound by the rows' reads: 5.3 TB/s at 2.2 GB (500 queries of 8.8M documents, seed tiles), 4 TB/s
// at 250 MB (62 us). Places for all of a wavefront's hits of a round from one atomic on the stage:
// 70 us there, though 9 -> 7.5 us at 48 queries of 262,147 documents.
constexpr int kFilterStage = 4096;

__device__ __forceinline__ void append_global(SelState* st, unsigned long long* C, bool take,
                                              unsigned long long c, int lane) {
    const unsigned long long m = __ballot(take);
    if (m == 0) return;
    int slot = 0;
    if (lane == 0) slot = atomicAdd(&st->n_cand, __popcll(m));
    slot = __shfl(slot, 0, kWave) + __popcll(m & ((1ull << lane) - 1ull));
    if (take) {
        if (slot < kCandCap) C[slot] = c;
        else st->overflow = 1;
    }
}

__global__ __launch_bounds__(512) void k_filter(int32_t q0, int64_t N, const uint32_t* __restrict__ S, int64_t ld,
                                                int per_block, SelState* __restrict__ state,
                                                unsigned long long* __restrict__ cand, int tile_shift,
                                                int seed_stride) {
    __shared__ unsigned long long stage[kFilterStage];
    __shared__ int n_stage, g_base;
    const int ql = blockIdx.y;
    SelState* st = state + ql;
    if (st->resolved != 1) return;
    const unsigned long long lo = st->lo;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    if (tid == 0) n_stage = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * per_block, b1 = min(N, b0 + per_block);  // per_block % 256 == 0
    const uint32_t* Sq = S + (int64_t)ql * ld;
    unsigned long long* C = cand + (int64_t)ql * kCandCap;
    // Four rounds of 16-byte loads are issued before the first test (a single load in flight
    // per lane left the scan at about half the HBM rate). A lane past the range reads the
    // range's last aligned four scores instead (no branch around the load) and tests nothing.
    auto scan = [&](int64_t d0, int64_t d1) {  // d0 % 256 == 0
        constexpr int R = 4;
        const int64_t last = (d1 - 1) & ~3ll;  // d + 3 < ld: rows are padded to 64
        for (int64_t wb = d0 + (int64_t)wave * kWave * 4; wb < d1; wb += 512 * 4 * R) {
            uint4 v[R];
#pragma unroll
            for (int r = 0; r < R; r++)
                v[r] = *reinterpret_cast<const uint4*>(Sq + min(wb + r * 2048 + (int64_t)lane * 4, last));
#pragma unroll
            for (int r = 0; r < R; r++) {
                const int64_t d = wb + r * 2048 + (int64_t)lane * 4;
                const uint32_t vs[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const unsigned long long c = comp_key(vs[j], (uint32_t)(d + j));
                    const bool take = d + j < d1 && c >= lo;
                    const unsigned long long m = __ballot(take);
                    if (m == 0) continue;
                    int slot = 0;
                    if (lane == 0) slot = atomicAdd(&n_stage, __popcll(m));
                    slot = __shfl(slot, 0, kWave) + __popcll(m & ((1ull << lane) - 1ull));
                    if (take && slot < kFilterStage) stage[slot] = c;
                    append_global(st, C, take && slot >= kFilterStage, c, lane);
                }
            }
        }
    };
    if (st->fused == 1 && seed_stride > 0) {
        // fused filtering: the other tiles' candidates were appended while they were
        // scored; only the seed tiles' documents are scanned here
        for (int64_t t = b0 >> tile_shift; (t << tile_shift) < b1; t++)
            if (t % seed_stride == 0) scan(max(b0, t << tile_shift), min(b1, (t + 1) << tile_shift));
    } else {
        scan(b0, b1);
    }
    __syncthreads();
    const int n = min(n_stage, kFilterStage);
    if (tid == 0) g_base = n ? atomicAdd(&st->n_cand, n) : 0;
    __syncthreads();
    const int base = g_base;
    for (int i = tid; i < n; i += 512) {
        if (base + i < kCandCap) C[base + i] = stage[i];
        else st->overflow = 1;
    }
}

// Candidates and winners held in LDS by k_final, band documents held by k_band_topk.
constexpr int kFinalCap = kMaxK + 512;
// Largest bin whose winners are ranked by comparisons among them (64 comparisons cost about as
// much as the bitonic sort of 1,000 winners that takes over past it).
constexpr int kFinalBin = 64;

// Smallest shift that maps offsets 0 .. range onto kHistBins bins.
__device__ __forceinline__ int range_shift(unsigned long long range) {
    return range == 0 ? 0 : max(0, 64 - __clzll((long long)range) - kHistBits);
}

__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long o = __shfl_xor(v, d, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// Largest of a workgroup's values, in *out (LDS, zero before).
__device__ __forceinline__ void block_max(uint32_t v, uint32_t* out) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, d, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(out, v);
    __syncthreads();
}

// Bitonic sort of m elements in LDS by the whole workgroup, with every comparator in the same
// direction (each merge opens with a mirrored step), so that m need not be a power of two:
// comparators past the end are left out. order(l, r) puts the elements l < r in order. The way
// out where one bin holds too many winners to rank them by comparisons (many equal scores).
// In steps of j <= 64 a wavefront's pairs stay inside its own 128 elements, so those steps need
// no workgroup barrier between them (1,000 elements: 49 of 55 barriers less).
template <typename F>
__device__ __forceinline__ void bitonic_sort(int m, F order) {
    for (int lk = 1; (1 << (lk - 1)) < m; lk++) {
        for (int lj = lk - 1; lj >= 0; lj--) {
            const int j = 1 << lj, pairs = ((m + 2 * j - 1) >> (lj + 1)) << lj;
            for (int t = threadIdx.x; t < pairs; t += kSelBS) {
                const int block = t >> lj, at = t & (j - 1);
                const int l = (block << (lj + 1)) + at;
                const int r = lj == lk - 1 ? (block << (lj + 1)) + 2 * j - 1 - at : l + j;
                if (r < m) order(l, r);
            }
            if (j > kWave || (lj == 0 ? (1 << lk) : j >> 1) > kWave) __syncthreads();
            else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        }
    }
    __syncthreads();
}

// Smallest and largest of the workgroup's values (given as per-thread extremes) in red[0], red[1].
__device__ __forceinline__ void block_range(unsigned long long mn, unsigned long long mx, unsigned long long* red) {
    mn = ~wave_max(~mn);
    mx = wave_max(mx);
    if (threadIdx.x == 0) {
        red[0] = ~0ull;
        red[1] = 0ull;
    }
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicMin(&red[0], mn);
        atomicMax(&red[1], mx);
    }
    __syncthreads();
}

// One wavefront walks a 256-bin histogram from the top bin down for the bin
// holding the need-th largest element; writes it and the count above it.
__device__ void walk256(const uint32_t* hist, uint32_t need, int* d_out, uint32_t* above_out) {
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t s = 0;
    for (int j = 0; j < 4; j++) s += hist[255 - lane * 4 - j];
    uint32_t incl = s;
    for (int dd = 1; dd < kWave; dd <<= 1) {
        const uint32_t v = __shfl_up(incl, dd, kWave);
        if (lane >= dd) incl += v;
    }
    const uint32_t excl = incl - s;
    const unsigned long long m = __ballot(excl < need && need <= incl);
    const int owner = m ? __ffsll((long long)m) - 1 : kWave - 1;
    if (lane == owner) {
        uint32_t run = excl;
        int dsel = 255 - lane * 4 - 3;
        uint32_t ab = run;
        for (int j = 0; j < 4; j++) {
            const uint32_t c = hist[255 - lane * 4 - j];
            if (run + c >= need) {
                dsel = 255 - lane * 4 - j;
                ab = run;
                break;
            }
            run += c;
        }
        *d_out = dsel;
        *above_out = ab;
    }
}

// The first kq band members by (fp64 score desc, doc id asc), written to ids /
// sc. Keys (score bits, ~doc id) are distinct and ordered like that pair (scores
// are >= 0, so their bits are monotone): a radix select with 8-bit digits (8 of
// the score, then 4 of ~id) finds the kq-th largest key, the kq keys at or above
// it are gathered into LDS, and each is placed by its rank among them.
// LDS used by band_topk: hist[256], wsc[kMaxK], wid[kMaxK] and three scalars
// (the caller may hand in arrays it no longer needs).
struct BandLds {
    uint32_t* hist;
    unsigned long long* wsc;
    int32_t* wid;
    int* d;
    uint32_t* above;
    int* cnt;
};

__device__ void band_topk(const double* bs, const int32_t* bid, int nb, int64_t kq, int32_t* ids, double* sc,
                          const BandLds& L) {
    const int tid = threadIdx.x, nt = blockDim.x;
    unsigned long long ph = 0, mh = 0;
    uint32_t pl = 0, ml = 0;
    uint32_t need = (uint32_t)min<int64_t>(kq, nb);
    if ((uint32_t)nb > need) {
        for (int d = 0; d < 12; d++) {
            for (int i = tid; i < 256; i += nt) L.hist[i] = 0u;
            __syncthreads();
            for (int i = tid; i < nb; i += nt) {
                const unsigned long long h = (unsigned long long)__double_as_longlong(bs[i]);
                const uint32_t l = ~(uint32_t)bid[i];
                if ((h & mh) == ph && (l & ml) == pl) {
                    const uint32_t dig = d < 8 ? (uint32_t)(h >> (56 - 8 * d)) & 255u : (l >> (88 - 8 * d)) & 255u;
                    atomicAdd(&L.hist[dig], 1u);
                }
            }
            __syncthreads();
            if (tid < kWave) walk256(L.hist, need, L.d, L.above);
            __syncthreads();
            const int dsel = *L.d;
            need -= *L.above;
            const uint32_t hd = L.hist[dsel];
            __syncthreads();
            if (d < 8) {
                ph |= (unsigned long long)dsel << (56 - 8 * d);
                mh |= 255ull << (56 - 8 * d);
            } else {
                pl |= (uint32_t)dsel << (88 - 8 * d);  // id digits: bits 31..24, ..., 7..0
                ml |= 255u << (88 - 8 * d);
            }
            if (hd == need) break;
        }
    }
    if (tid == 0) *L.cnt = 0;
    __syncthreads();
    for (int i = tid; i < nb; i += nt) {
        const unsigned long long h = (unsigned long long)__double_as_longlong(bs[i]);
        const uint32_t l = ~(uint32_t)bid[i];
        if (h > ph || (h == ph && l >= pl)) {
            const int pos = atomicAdd(L.cnt, 1);
            if (pos < kMaxK) {
                L.wsc[pos] = h;
                L.wid[pos] = bid[i];
            }
        }
    }
    __syncthreads();
    const int m = min(*L.cnt, kMaxK);
    for (int i = tid; i < m; i += nt) {
        const unsigned long long si = L.wsc[i];
        const int32_t di = L.wid[i];
        int r = 0;
        for (int j = 0; j < m; j++) {
            const unsigned long long sj = L.wsc[j];
            r += (sj > si) || (sj == si && L.wid[j] < di);
        }
        if (r < kq) {
            ids[r] = di;
            sc[r] = __longlong_as_double((long long)si);
        }
    }
}

// Band of the bf16 form. Every doc's approximate score satisfies
//   s(1-delta) - E <= approx <= s(1+delta) + E
// (delta: relative error of the stored bf16 weights and of the score's
// arithmetic; E: the fixed-point error bound). Then approx_k <= (1+delta) s_k + E,
// and every true top-k doc has
// approx >= s(1-delta) - E >= (approx_k - E)(1-delta)/(1+delta) - E = tau.
__device__ __forceinline__ double band_tau(float sk, double delta, double abs_err) {
    const double d = delta;
    const double t = ((double)sk - abs_err) * (1.0 - d) / (1.0 + d) - abs_err;
    return t > 0.0 ? t * (1.0 - 1e-12) : 0.0;
}

// Error terms of the bf16 band for a query: relative (delta) and absolute (E).
// Fixed-point sums: the stored-weight and final fp32 roundings, plus E. The fp64
// pass (wide range): exact products, an fp64 sum (relative error below 1e-13 for
// 256 terms) rounded once to fp32, no E. fp32 sums (global-atomic and
// document-parallel kernels): each product and addition rounds, so delta also
// covers gamma_m = m u / (1 - m u) with u = 2^-24 for m query terms; no E.
__device__ __forceinline__ void band_error(const DevBatch& qb, int q, int acc, int rescore, int m, double* rel,
                                           double* abs_err) {
    const double d = (double)qb.delta[q];
    if (rescore == 2) {
        *rel = d + 1e-12;
        *abs_err = 0.0;
    } else if (acc == kAccFloat) {
        const double mu = (double)(m + 1) * 0x1p-24;
        *rel = (1.0 + d) * (1.0 + mu / (1.0 - mu)) - 1.0;
        *abs_err = 0.0;
    } else {
        *rel = d;
        *abs_err = qb.q_abs_err[q];
    }
}

// One row of the per-query diagnostics (gs_batch_diagnostics).
__device__ __forceinline__ void write_diag(int32_t* diag, int q, const SelState& st) {
    if (diag == nullptr || threadIdx.x != 0) return;
    int32_t* o = diag + (int64_t)q * kDiagWords;
    o[0] = st.n_cand;
    o[1] = st.passes;
    o[2] = st.band;
    o[3] = st.overflow;
    o[4] = st.rescore;
    o[5] = st.fused == 1 ? 1 : 0;
    o[6] = st.pruned;
    o[7] = 0;
}

// The k best of a query's candidates, in order. ROW: the candidates are the documents of the
// score row themselves (collections of at most kCandCap documents; no selection state is read).
// A histogram of the candidates over 2048 equal bins of their range finds the bin of the k-th
// in one pass; while that bin is too large to be ranked by comparisons the range is narrowed to
// it and counted again. The winners are grouped by bin in LDS (the scanned histogram gives each
// bin's first place), so that each needs comparing only with its own bin. Before: up to eight
// 8-bit radix passes and a rank by comparison with all k winners (27 us for one query of
// 4M documents, k = 1000, now 8; 4,096 queries of 250,000 documents 300 us, now 73).
template <int P, bool ROW>
__global__ __launch_bounds__(kSelBS) void k_final(DevIndex ix, DevBatch qb, int32_t q0, SelState* __restrict__ state,
                                                  const unsigned long long* __restrict__ cand,
                                                  const uint32_t* __restrict__ S, int64_t ld,
                                                  int32_t* __restrict__ band_id, int32_t* __restrict__ out_ids,
                                                  void* __restrict__ out_scores, int acc,
                                                  uint32_t* __restrict__ counters, int32_t* __restrict__ rescore_list,
                                                  int32_t* __restrict__ diag) {
    static_assert(P != kBF16 || !ROW, "bf16 needs the selection state (error band)");
    __shared__ unsigned long long sel[kFinalCap];
    __shared__ uint32_t hist[kHistBins];
    __shared__ BinScan sh;
    __shared__ unsigned long long red[2];
    const int tid = threadIdx.x;
    const int ql = blockIdx.x, q = q0 + ql;
    SelState* st = state + ql;
    const int64_t kq = kq_of(qb, q, ix.n_docs);
    const int kmax = qb.k_max;
    int32_t* ids = out_ids + (int64_t)q * kmax;
    if (P != kBF16) {
        for (int i = tid; i < kmax; i += kSelBS) {
            if (i >= kq) {
                ids[i] = -1;
                ((uint32_t*)out_scores)[(int64_t)q * kmax + i] = 0u;
            }
        }
        if constexpr (ROW) {
            SelState d{};
            d.n_cand = kq > 0 ? (int32_t)ix.n_docs : 0;
            write_diag(diag, q, d);
        } else {
            write_diag(diag, q, *st);
        }
    }
    if (kq == 0) return;
    const int n = ROW ? (int)ix.n_docs : min(st->n_cand, kCandCap);
    if (n == 0) return;
    const unsigned long long* C = cand + (int64_t)ql * kCandCap;
    const uint32_t* Sq = S + (int64_t)ql * ld;
    auto get = [&](int i) { return ROW ? comp_key(Sq[i], (uint32_t)i) : C[i]; };
    // the first REG candidates of each thread stay in registers over the passes
    constexpr int REG = 16;
    unsigned long long reg[REG];
    unsigned long long mn = ~0ull, mx = 0ull;
#pragma unroll
    for (int r = 0; r < REG; r++) {
        const int i = tid + r * kSelBS;
        reg[r] = i < n ? get(i) : 0ull;
    }
    auto each = [&](auto f) {
#pragma unroll
        for (int r = 0; r < REG; r++)
            if (tid + r * kSelBS < n) f(reg[r]);
        for (int i = tid + REG * kSelBS; i < n; i += kSelBS) f(get(i));
    };
    each([&](unsigned long long c) {
        mn = c < mn ? c : mn;
        mx = c > mx ? c : mx;
    });
    block_range(mn, mx, red);
    mn = red[0];
    mx = red[1];
    unsigned long long lo = mn, hi = mx, thr;
    uint32_t above = 0;  // composites past hi
    const uint32_t need = (uint32_t)min((int64_t)n, kq);
    int s, total;
    uint32_t c4[4], e4[4];
    auto count = [&]() {  // composites of [lo, hi] per bin, and the bin of the (need - above)-th
        s = range_shift(hi - lo);
        reinterpret_cast<uint4*>(hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        each([&](unsigned long long c) {
            if (c >= lo && c <= hi) atomicAdd(&hist[(c - lo) >> s], 1u);
        });
        __syncthreads();
        load_bins(hist, c4);
        scan_bins(c4, e4, need - above, sh);
    };
    bool whole = true;  // hist spans every winner
    for (;;) {
        count();
        total = (int)(above + sh.above + sh.count);
        thr = lo + ((unsigned long long)sh.d << s);
        if (s == 0 || (total <= kFinalCap && sh.count <= (uint32_t)kFinalBin)) break;
        above += sh.above;
        hi = min(hi, thr + ((1ull << s) - 1ull));
        lo = thr;
        whole = false;
        __syncthreads();  // sh is read: the next scan may write it
    }
    if (!whole) {
        __syncthreads();
        lo = thr;
        hi = mx;
        above = 0;
        count();
    }
    // the largest bin among the winners' decides how they are put in order
    __syncthreads();  // sh is read
    if (tid == 0) sh.above = 0;
    __syncthreads();
    {
        uint32_t big = 0;
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (lo + ((unsigned long long)(kHistBins - 1 - 4 * tid - j) << s) >= thr) big = max(big, c4[j]);
        block_max(big, &sh.above);
    }
    const bool sorted = sh.above > (uint32_t)kFinalBin;
    // group the winners by bin: the scanned histogram (elements above each bin) is the cursor
    reinterpret_cast<uint4*>(hist)[kSelBS - 1 - tid] = make_uint4(e4[3], e4[2], e4[1], e4[0]);
    __syncthreads();
    each([&](unsigned long long c) {
        if (c >= thr) {
            const uint32_t pos = atomicAdd(&hist[(c - lo) >> s], 1u);
            if (pos < (uint32_t)kFinalCap) sel[pos] = c;
        }
    });
    __syncthreads();
    const int m = min(total, kFinalCap);
    if (sorted)
        bitonic_sort(m, [&](int l, int r) {
            const unsigned long long a = sel[l], b = sel[r];
            if (a < b) {
                sel[l] = b;
                sel[r] = a;
            }
        });
    // bin b now ends at hist[b] and starts where the bin above it ends
    auto ranked = [&](auto f) {
        for (int p = tid; p < m; p += kSelBS) {
            const unsigned long long c = sel[p];
            if (sorted) {
                f(p, c);
                continue;
            }
            const int b = (int)((c - lo) >> s);
            const int from = b + 1 < kHistBins ? (int)hist[b + 1] : 0, to = min((int)hist[b], m);
            int r = from;
            for (int j = from; j < to; j++) r += sel[j] > c;
            f(r, c);
        }
    };
    if constexpr (P != kBF16) {
        ranked([&](int r, unsigned long long c) {
            if (r < kq) {
                ids[r] = (int32_t)(~(uint32_t)c);
                ((uint32_t*)out_scores)[(int64_t)q * kmax + r] = (uint32_t)(c >> 32);
            }
        });
    } else {
        // bf16: exact k-th approximate score, then the error band
        __shared__ unsigned long long sh_kth;
        __shared__ int sh_cnt;
        if (tid == 0) {
            sh_kth = 0ull;
            sh_cnt = 0;
        }
        __syncthreads();
        int32_t* bid = band_id + (int64_t)ql * kCandCap;
        ranked([&](int r, unsigned long long c) {
            if (r == kq - 1) sh_kth = c;
        });
        __syncthreads();
        const float sk = __uint_as_float((uint32_t)(sh_kth >> 32));
        const int nq = (int)(qb.q_row_ptr[q + 1] - qb.q_row_ptr[q]);
        double rel_err, abs_err;
        band_error(qb, q, acc, st->rescore, nq, &rel_err, &abs_err);
        int nb;
        if (sk == 0.0f) {
            // fewer than k docs share a term with the query: the k winners are every doc with a
            // positive score plus the lowest-id zero-score docs. A zero approximate score is exact
            // here: from fp32 or fp64 sums (no product of admissible weights underflows to 0), or
            // from fixed point only if no positive product can round to 0 units (otherwise the
            // wide-range check sent the query to the fp64 pass: its k-th bucket starts at 0).
            ranked([&](int r, unsigned long long c) {
                if (r < kq) bid[r] = (int32_t)(~(uint32_t)c);
            });
            nb = (int)kq;
        } else {
            const double tau = band_tau(sk, rel_err, abs_err);
            // with fused filtering the other tiles' candidates start at the bound, the seed tiles' at lo
            const unsigned long long flo = st->fused == 1 ? max(st->lo, st->bound) : st->lo;
            const double lo_val = (double)__uint_as_float((uint32_t)(flo >> 32));
            const bool inside = tau > 0.0 && (((uint32_t)flo == 0u) ? (lo_val <= tau) : (lo_val < tau));
            if (!inside) {
                if (tid == 0) {
                    st->need_band_pass = 1;
                    st->tau = tau;
                    if (st->fused == 1) {  // its other tiles wrote no rows: score them for the band pass
                        st->rescore = 3;
                        rescore_list[atomicAdd(&counters[kCntListed], 1u)] = ql;
                    }
                }
                return;
            }
            each([&](unsigned long long c) {
                const double v = (double)__uint_as_float((uint32_t)(c >> 32));
                if (v > 0.0 && v >= tau) bid[atomicAdd(&sh_cnt, 1)] = (int32_t)(~(uint32_t)c);
            });
            __syncthreads();
            nb = sh_cnt;
        }
        if (tid == 0) st->band = nb;
    }
}

// fp64 rescoring of the listed band documents against their query, on a grid over the
// documents (a workgroup per query left 252 of 256 CUs idle for a call of four queries: its
// selection took 368 us). A wavefront takes 4 documents, 16 lanes each. Lane `sub` holds entries
// sub, sub + 16, ... of the document's forward row (sorted by term), eight of terms and eight of
// weights in flight, and finds each term in the query by a hash of its low bits: one LDS read
// and a compare each, without a branch. The products of the terms found are put side by side in
// LDS in row order (ascending term) and added by one lane, so the sum is the same sequence of
// fp64 additions as a serial walk of the row.
// Bound by the rows' reads, some 1,150 per query at k = 1,000 and in no order, as many
// wavefronts in flight as there can be: at 8, 6 and 5 a SIMD 159, 201 and 252 us (500 queries of
// 500,000 documents), so it is held to 64 VGPRs. A chain walk and a wait per lookup took 202 us
// there, and 18.5 us for 4 queries of 200,000 documents against 10.5.
constexpr int kRescoreBS = 512;
constexpr int kRescoreHash = 2048;
constexpr int kRescoreProds = 96;  // products of a document held at once

template <typename TT>
__global__ __launch_bounds__(kRescoreBS) __attribute__((amdgpu_waves_per_eu(8))) void k_rescore(
    DevIndex ix, const TT* __restrict__ fwd_term, DevBatch qb, int32_t q0, const SelState* __restrict__ state,
    double* __restrict__ band_s, const int32_t* __restrict__ band_id) {
    // a bucket's last query term: its upper bits << 10 | (512 if the bucket has more) | its place + 1
    // (at most 256), or 0
    __shared__ __align__(16) uint32_t head[kRescoreHash];
    __shared__ int32_t next[kMaxQueryNnz + 1];  // the bucket's other terms, by the same places
    __shared__ int32_t sq_t[kMaxQueryNnz + 1];
    __shared__ float sq_w[kMaxQueryNnz + 1];
    // per document, products in row order, then zeros up to a multiple of 4
    __shared__ __align__(16) double prod[kRescoreBS / 16][kRescoreProds + 4];
    constexpr int kBits = 11;
    static_assert(kRescoreHash == 1 << kBits && kMaxQueryNnz < 512, "bucket entries");
    const int ql = blockIdx.y, q = q0 + ql, tid = threadIdx.x;
    const SelState* st = state + ql;
    const int nb = st->overflow ? 0 : min(st->band, kCandCap);
    constexpr int per = kRescoreBS / 16;
    if ((int)blockIdx.x * per >= nb) return;
    for (int i = tid; i < kRescoreHash / 4; i += kRescoreBS) ((uint4*)head)[i] = make_uint4(0u, 0u, 0u, 0u);
    const int64_t qa = qb.q_row_ptr[q];
    const int nq = (int)(qb.q_row_ptr[q + 1] - qa);
    __syncthreads();
    for (int i = tid; i < nq; i += kRescoreBS) {
        const int32_t t = qb.q_term[qa + i];
        sq_t[i + 1] = t;
        sq_w[i + 1] = qb.q_w[qa + i];
        uint32_t* const h = &head[t & (kRescoreHash - 1)];
        const uint32_t before = atomicExch(h, ((uint32_t)t >> kBits) << 10 | (uint32_t)(i + 1));
        next[i + 1] = (int32_t)(before & 511u);
        if (before != 0u) atomicOr(h, 512u);
    }
    if (tid == 0) sq_w[0] = 0.0f;
    __syncthreads();
    const int32_t* bid = band_id + (int64_t)ql * kCandCap;
    double* bs = band_s + (int64_t)ql * kCandCap;
    const int lane = tid & (kWave - 1), wave = tid >> 6;
    const int grp = lane >> 4, sub = lane & 15, sh = (grp & 1) * 16;
    const uint32_t below = (1u << sub) - 1u;
    double* mine = prod[wave * 4 + grp];
    auto row = [&](int i, int64_t& a, int& len) {  // document i's forward row
        a = 0;
        len = 0;
        if (i < nb) {
            const int64_t doc = bid[i];
            a = ix.fwd_row_ptr[doc];
            len = (int)(ix.fwd_row_ptr[doc + 1] - a);
        }
    };
    int64_t a, a_next;
    int len, len_next, cnt;
    double s;
    // the held products into the sum, one lane adding them one by one, four read at once
    auto add = [&]() {
        if (sub < 4) mine[cnt + sub] = 0.0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // LDS of this wavefront only
        if (sub == 0)
            for (int p = 0; p < cnt; p += 4) {
                const double2 lo = *(const double2*)&mine[p], hi = *(const double2*)&mine[p + 2];
                s += lo.x;
                s += lo.y;
                s += hi.x;
                s += hi.y;
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        cnt = 0;
    };
    // entries [off, off + 16 U) of the four rows
    auto entries = [&](auto uc, int off, auto under) {
        constexpr int U = decltype(uc)::value;
        int t[U];
        float w[U];
        const TT* rt = fwd_term + (a + off + sub);
        const float* rw = ix.fwd_w + (a + off + sub);
        const int left = len - off - sub;
#pragma unroll
        for (int u = 0; u < U; u++) t[u] = 16 * u < left ? (int)rt[16 * u] : -1;
        // most of a row's cache lines hold a query term's weight: all are read beside the terms
#pragma unroll
        for (int u = 0; u < U; u++) w[u] = 16 * u < left ? rw[16 * u] : 0.0f;
        under();
        constexpr int H = U < 4 ? U : 4;
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += H) {
            uint32_t h[H];
            int j[H];
            float qw[H];
#pragma unroll
            for (int u = 0; u < H; u++) h[u] = head[t[u0 + u] & (kRescoreHash - 1)];
            bool more = false;
#pragma unroll
            for (int u = 0; u < H; u++) {
                const bool same = h[u] >> 10 == (uint32_t)t[u0 + u] >> kBits;  // never where t is -1
                j[u] = same ? (int)(h[u] & 511u) : 0;
                more |= !same && (h[u] & 512u) != 0u;
            }
            if (__any(more)) {  // two query terms in one bucket: rare
#pragma unroll
                for (int u = 0; u < H; u++)
                    if (j[u] == 0 && (h[u] & 512u) != 0u) {
                        j[u] = next[h[u] & 511u];
                        while (j[u] != 0 && sq_t[j[u]] != t[u0 + u]) j[u] = next[j[u]];
                    }
            }
#pragma unroll
            for (int u = 0; u < H; u++) qw[u] = sq_w[j[u]];
            if (__any(cnt > kRescoreProds - 16 * H)) add();
#pragma unroll
            for (int u = 0; u < H; u++) {
                const bool hit = j[u] != 0;
                const unsigned long long m = __ballot(hit);
                const uint32_t mm = (lane < 32 ? (uint32_t)m : (uint32_t)(m >> 32)) >> sh & 0xFFFFu;
                if (hit) mine[cnt + __popc(mm & below)] = (double)qw[u] * (double)w[u0 + u];
                cnt += __popc(mm);
            }
        }
    };
    const int step = (int)gridDim.x * per;
    row((int)blockIdx.x * per + wave * 4 + grp, a_next, len_next);
    for (int base = (int)blockIdx.x * per + wave * 4; base < nb; base += step) {
        const int i = base + grp;
        a = a_next;
        len = len_next;
        int maxlen = len;
        maxlen = max(maxlen, __shfl_xor(maxlen, 16, kWave));
        maxlen = __builtin_amdgcn_readfirstlane(max(maxlen, __shfl_xor(maxlen, 32, kWave)));
        s = 0.0;
        cnt = 0;
        auto next_row = [&]() { row(i + step, a_next, len_next); };  // under this one's loads
        entries(std::integral_constant<int, 8>(), 0, next_row);
        for (int off = 128; off < maxlen;) {
            if (maxlen - off > 32) {
                entries(std::integral_constant<int, 8>(), off, [] {});
                off += 128;
            } else {
                entries(std::integral_constant<int, 2>(), off, [] {});
                off += 32;
            }
        }
        add();
        if (sub == 0 && i < nb) bs[i] = s;
    }
}

__global__ __launch_bounds__(512) void k_band_filter(int32_t q0, int64_t N, const uint32_t* __restrict__ S,
                                                     int64_t ld, int per_block, SelState* __restrict__ state,
                                                     int32_t* __restrict__ band_id) {
    const int ql = blockIdx.y;
    SelState* st = state + ql;
    if (st->need_band_pass != 1) return;
    const double tau = st->tau;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int64_t d0 = (int64_t)blockIdx.x * per_block, d1 = min(N, d0 + per_block);
    const uint32_t* Sq = S + (int64_t)ql * ld;
    int32_t* B = band_id + (int64_t)ql * kCandCap;
    for (int64_t wb = d0 + wave * kWave; wb < d1; wb += 512) {
        const int64_t d = wb + lane;
        const double v = d < d1 ? (double)__uint_as_float(Sq[d]) : 0.0;
        const bool take = v > 0.0 && v >= tau;
        const unsigned long long m = __ballot(take);
        if (m == 0) continue;
        int slot = 0;
        if (lane == 0) slot = atomicAdd(&st->band, __popcll(m));
        slot = __shfl(slot, 0, kWave) + __popcll(m & ((1ull << lane) - 1ull));
        if (take) {
            if (slot < kCandCap) B[slot] = (int32_t)d;
            else st->overflow = 1;
        }
    }
}

// The kq best band documents of a query by (fp64 score desc, doc id asc): grouped by bins of
// the score bits in LDS and ranked inside their bin as in k_final; bands past kFinalCap
// documents (massive near-ties) go through the radix selection of band_topk.
__global__ __launch_bounds__(kSelBS) void k_band_topk(DevIndex ix, DevBatch qb, int32_t q0,
                                                      const SelState* __restrict__ state,
                                                      const double* __restrict__ band_s,
                                                      const int32_t* __restrict__ band_id,
                                                      int32_t* __restrict__ out_ids, double* __restrict__ out_scores,
                                                      int32_t* __restrict__ diag) {
    __shared__ uint32_t hist[kHistBins];
    __shared__ unsigned long long wsc[kFinalCap];
    __shared__ int32_t wid[kFinalCap];
    __shared__ BinScan sh;
    __shared__ unsigned long long red[2];
    __shared__ int sh_d, sh_cnt;
    __shared__ uint32_t sh_above;
    const int ql = blockIdx.x, q = q0 + ql, tid = threadIdx.x;
    const SelState* st = state + ql;
    const int64_t kq = kq_of(qb, q, ix.n_docs);
    int32_t* ids = out_ids + (int64_t)q * qb.k_max;
    double* sc = out_scores + (int64_t)q * qb.k_max;
    // a band that does not fit its buffer: the row is left as padding and flagged
    const bool lost = st->need_band_pass == 1 && st->overflow;
    for (int i = tid; i < qb.k_max; i += kSelBS) {
        if (i >= kq || lost) {
            ids[i] = -1;
            sc[i] = 0.0;
        }
    }
    write_diag(diag, q, *st);
    if (kq == 0 || lost) return;
    const int nb = min(st->band, kCandCap);
    const double* bs = band_s + (int64_t)ql * kCandCap;
    const int32_t* bid = band_id + (int64_t)ql * kCandCap;
    if (nb > kFinalCap) {
        band_topk(bs, bid, nb, kq, ids, sc, BandLds{hist, wsc, wid, &sh_d, &sh_above, &sh_cnt});
        return;
    }
    if (nb == 0) return;
    constexpr int R = kFinalCap / kSelBS;
    unsigned long long key[R];
    int32_t id[R];
    unsigned long long mn = ~0ull, mx = 0ull;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = tid + r * kSelBS;
        key[r] = i < nb ? (unsigned long long)__double_as_longlong(bs[i]) : 0ull;
        id[r] = i < nb ? bid[i] : 0;
        if (i < nb) {
            mn = key[r] < mn ? key[r] : mn;
            mx = key[r] > mx ? key[r] : mx;
        }
    }
    reinterpret_cast<uint4*>(hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
    block_range(mn, mx, red);
    mn = red[0];
    const int s = range_shift(red[1] - mn);
#pragma unroll
    for (int r = 0; r < R; r++)
        if (tid + r * kSelBS < nb) atomicAdd(&hist[(key[r] - mn) >> s], 1u);
    __syncthreads();
    uint32_t c4[4], e4[4];
    load_bins(hist, c4);
    scan_bins(c4, e4, (uint32_t)min((int64_t)nb, kq), sh);
    reinterpret_cast<uint4*>(hist)[kSelBS - 1 - tid] = make_uint4(e4[3], e4[2], e4[1], e4[0]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (tid + r * kSelBS >= nb) continue;
        const uint32_t pos = atomicAdd(&hist[(key[r] - mn) >> s], 1u);
        wsc[pos] = key[r];
        wid[pos] = id[r];
    }
    __syncthreads();
    const int m = min((int)(sh.above + sh.count), nb);  // the winners' bins come first
    const int d_last = sh.d;
    __syncthreads();
    if (tid == 0) sh.above = 0;
    __syncthreads();
    {
        uint32_t big = 0;
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (kHistBins - 1 - 4 * tid - j >= d_last) big = max(big, c4[j]);
        block_max(big, &sh.above);
    }
    const bool sorted = sh.above > (uint32_t)kFinalBin;
    if (sorted)
        bitonic_sort(m, [&](int l, int r) {
            const unsigned long long a = wsc[l], b = wsc[r];
            const int32_t ia = wid[l], ib = wid[r];
            if (a < b || (a == b && ia > ib)) {
                wsc[l] = b;
                wsc[r] = a;
                wid[l] = ib;
                wid[r] = ia;
            }
        });
    for (int p = tid; p < m; p += kSelBS) {
        const unsigned long long k = wsc[p];
        const int32_t di = wid[p];
        if (sorted) {
            if (p < kq) {
                ids[p] = di;
                sc[p] = __longlong_as_double((long long)k);
            }
            continue;
        }
        const int b = (int)((k - mn) >> s);
        const int from = b + 1 < kHistBins ? (int)hist[b + 1] : 0, to = (int)hist[b];
        int r = from;
        for (int j = from; j < to; j++) r += wsc[j] > k || (wsc[j] == k && wid[j] < di);
        if (r < kq) {
            ids[r] = di;
            sc[r] = __longlong_as_double((long long)k);
        }
    }
}

}  // namespace

hipError_t launch_seed_bound(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const Workspace& ws,
                             hipStream_t s, int tile_shift, int seed_stride) {
    hipLaunchKernelGGL(k_seed_bound, dim3(qt), dim3(kSelBS), 0, s, qb, q0, ix.n_docs, (const uint32_t*)ws.scores, ws.ld,
                       (const uint32_t*)ws.hist1, ws.state, tile_shift, seed_stride);
    GS_CHECK_LAUNCH("k_seed_bound");
    return hipSuccess;
}

hipError_t launch_select(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const Workspace& ws,
                         int32_t* out_ids, void* out_scores, int32_t* diag, hipStream_t s, int acc, int tile_shift,
                         int seed_stride, const ScoreOpts* phase3, bool wide, bool from_row) {
    const int64_t N = ix.n_docs;
    auto final_pass = [&]() -> hipError_t {
        auto go = [&](auto pc, auto row) {
            constexpr int P = decltype(pc)::value;
            hipLaunchKernelGGL((k_final<P, decltype(row)::value>), dim3(qt), dim3(kSelBS), 0, s, ix, qb, q0, ws.state,
                               (const unsigned long long*)ws.cand, (const uint32_t*)ws.scores, ws.ld, ws.band_id,
                               out_ids, out_scores, acc, ws.counters, ws.rescore_list, diag);
        };
        using FP32 = std::integral_constant<int, kFP32>;
        using BF16 = std::integral_constant<int, kBF16>;
        using U8 = std::integral_constant<int, kU8>;
        switch (ix.precision) {
            case kFP32:
                if (from_row) go(FP32(), std::true_type()); else go(FP32(), std::false_type());
                break;
            case kU8:
                if (from_row) go(U8(), std::true_type()); else go(U8(), std::false_type());
                break;
            default: go(BF16(), std::false_type()); break;
        }
        GS_CHECK_LAUNCH("k_final");
        return hipSuccess;
    };
    // bf16: the band's rescoring and ranking (also the padding and the diagnostics)
    auto band_pass = [&]() -> hipError_t {
        // Workgroups per query: one pass over the documents each for a band of 1.25 k where the
        // queries are few, more passes each (down to 4,096 workgroups in all) where they are many: a
        // workgroup sets up its query's hash first (500 queries: 190 us at 8 workgroups each, 221 at
        // 16, 201 at 4).
        const int x = std::max(1, std::min({64, (qb.k_max + qb.k_max / 4 + 31) / 32, 4096 / std::max(qt, 1)}));
        const dim3 grid((unsigned)x, (unsigned)qt);
        const SelState* st = ws.state;
        const int32_t* bid = ws.band_id;
        if (ix.fwd_term16)
            hipLaunchKernelGGL(k_rescore<uint16_t>, grid, dim3(kRescoreBS), 0, s, ix, ix.fwd_term16, qb, q0, st, ws.band_s, bid);
        else
            hipLaunchKernelGGL(k_rescore<int32_t>, grid, dim3(kRescoreBS), 0, s, ix, ix.fwd_term, qb, q0, st, ws.band_s, bid);
        GS_CHECK_LAUNCH("k_rescore");
        hipLaunchKernelGGL(k_band_topk, dim3(qt), dim3(kSelBS), 0, s, ix, qb, q0, (const SelState*)ws.state,
                           (const double*)ws.band_s, (const int32_t*)ws.band_id, out_ids, (double*)out_scores, diag);
        GS_CHECK_LAUNCH("k_band_topk");
        return hipSuccess;
    };
    if (N == 0) return ix.precision == kBF16 ? band_pass() : final_pass();  // empty collection: padding only
    if (from_row) return final_pass();
    // Rows are scanned by workgroups of 65536 documents, or fewer (down to 8192) where that
    // leaves the chip idle: below 1024 workgroups (four per CU) the range per workgroup, not
    // the memory, sets the scan's time (27 us at 200,000 documents x 4 queries).
    int per = 65536;
    while (per > 8192 && ((N + per - 1) / per) * qt < 1024) per >>= 1;
    const dim3 grid_scan((unsigned)((N + per - 1) / per), (unsigned)qt);
    const int wide_check = wide ? 1 : 0;
    auto select = [&](int pass) -> hipError_t {
        const auto k = qt <= 256 ? k_select<16> : k_select<4>;
        hipLaunchKernelGGL(k, dim3(qt), dim3(kSelBS), 0, s, qb, q0, N, ix.precision,
                           (const uint32_t*)ws.scores, ws.ld, ws.hist1, ws.state, ws.counters, ws.rescore_list, pass,
                           pass == 0 ? wide_check : 0);
        GS_CHECK_LAUNCH("k_select");
        return hipSuccess;
    };
    hipError_t e = select(0);
    if (e != hipSuccess) return e;
    if (phase3 || wide) {  // rows (and counts) of the listed queries: fused fallback, wide range
        if (phase3) e = launch_score_tiled(ix, qb, q0, qt, *phase3, ws, s, 3);
        if (e == hipSuccess && wide) e = launch_score_wide(ix, qb, q0, qt, ws, s);
        if (e == hipSuccess) e = select(1);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_filter, grid_scan, dim3(512), 0, s, q0, N, (const uint32_t*)ws.scores, ws.ld, per, ws.state,
                       ws.cand, seed_stride > 0 ? tile_shift : 16, seed_stride);
    GS_CHECK_LAUNCH("k_filter");
    e = final_pass();
    if (e != hipSuccess || ix.precision != kBF16) return e;
    if (phase3) {  // fused queries whose band reaches below their candidates: the other tiles' rows
        e = launch_score_tiled(ix, qb, q0, qt, *phase3, ws, s, 5);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_band_filter, grid_scan, dim3(512), 0, s, q0, N, (const uint32_t*)ws.scores, ws.ld, per,
                       ws.state, ws.band_id);
    GS_CHECK_LAUNCH("k_band_filter");
    return band_pass();
}

}  // namespace gs
