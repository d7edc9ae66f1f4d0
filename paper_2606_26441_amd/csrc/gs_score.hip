// Scoring kernels: fill one score array per query with
//   S[q][d] = sum over the query's terms t of w_q(t) * w_d(t)
// (paper Sec. 4.1: the score decomposes into one scatter-add per query term).
//
// Forms:
//  * k_score_tiled  - term-parallel, work = (query, doc tile). The query's commonest
//    terms are summed from rows that hold their weight for every document, in
//    registers; each other term's posting list is doc-sorted, so the postings that
//    fall into a doc tile are one contiguous segment (found in the per-term segment
//    table), streamed through coalesced loads and scatter-added into an LDS copy of
//    the tile with LDS atomics. The tile is then written once (coalesced) with the
//    histogram of the first selection digit, or leaves its candidates. No global
//    atomics on scores, no zeroing pass. This is the hybrid of scatter-add and
//    on-chip accumulation listed as future work (1) in Sec. 8. Items run tile by
//    tile, so that the queries of a batch share a tile's rows and postings in L2.
//  * k_score_group - pairs of queries per item, each posting chunk loaded once.
//  * k_score_pruned, k_score_listed - posting-only passes over a tile (score_tile):
//    block-max pruning; the rows of fused filtering's fallbacks; the fp64 pass.
//  * k_score_atomic - term-parallel, work = (query, term, chunk of postings);
//    global atomic adds into a zeroed score array, as in the paper's Sec. 5.2
//    kernel (one program per query term looping over posting chunks), with
//    long lists split into chunks so that head terms do not serialise.
//  * k_score_docpar - document-parallel (Sec. 5.3): per (query, doc) a gather
//    over the doc's forward row with the query's weights in a dense LDS table;
//    each output cell is written once, no atomics.
//
// Weight forms of the doc-tiled kernels: fp32 (products rounded to units of a
// per-query scale and summed exactly in 64-bit fixed point), bf16 (stored as the
// upper 16 bits of the fp32 pattern; 32-bit fixed point, then fp64 rescoring of
// the candidates) and uint8 impacts (int32 products and sums, exact). Doc ids are
// read as 16-bit offsets. With fused candidate filtering a search runs them in phases: the seed tiles, then the
// other tiles appending candidates at or above a bound while they flush, then a
// pass that writes the rows of the queries that fell back (k_score_listed; see
// gs_topk.hip).
#include <algorithm>
#include <type_traits>

#include "gs_internal.h"

namespace gs {

static inline int64_t score_ld(int64_t n_docs) { return (n_docs + 63) / 64 * 64; }

namespace {

template <int P> struct WF;
template <> struct WF<kFP32> {
    using Acc = float;
    static __device__ __forceinline__ float load(const void* p, int64_t i) { return ((const float*)p)[i]; }
    static __device__ __forceinline__ float from_fp32(float w) { return w; }
    static __device__ __forceinline__ float qweight(const DevBatch& qb, int64_t j) { return qb.q_w[j]; }
    static __device__ __forceinline__ uint32_t bits(float v) { return __float_as_uint(v); }
};
template <> struct WF<kBF16> {
    using Acc = float;
    static __device__ __forceinline__ float load(const void* p, int64_t i) {
        return __uint_as_float((uint32_t)((const uint16_t*)p)[i] << 16);
    }
    static __device__ __forceinline__ float from_fp32(float w) {
        // round to nearest even on the upper 16 bits (weights are finite and >= 0)
        uint32_t u = __float_as_uint(w);
        u += 0x7fffu + ((u >> 16) & 1u);
        return __uint_as_float(u & 0xffff0000u);
    }
    static __device__ __forceinline__ float qweight(const DevBatch& qb, int64_t j) { return qb.q_w[j]; }
    static __device__ __forceinline__ uint32_t bits(float v) { return __float_as_uint(v); }
};
template <> struct WF<kU8> {
    using Acc = int;
    static __device__ __forceinline__ int load(const void* p, int64_t i) { return ((const uint8_t*)p)[i]; }
    static __device__ __forceinline__ int from_fp32(float w) {
        double x = __builtin_rint((double)w * 85.0);
        return x > 255.0 ? 255 : (x > 0.0 ? (int)x : 0);
    }
    static __device__ __forceinline__ int qweight(const DevBatch& qb, int64_t j) { return qb.q_w8[j]; }
    static __device__ __forceinline__ uint32_t bits(int v) { return (uint32_t)v; }
};

// A wave-uniform double moved into scalar registers: the predicated per-posting
// blocks that use it then carry no wait on the LDS read that produced it.
__device__ __forceinline__ double uniform_f64(double v) {
    const long long b = __double_as_longlong(v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Lane l's value (l uniform), in scalar registers.
__device__ __forceinline__ unsigned long long read_lane64(unsigned long long v, int l) {
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long comp_key(uint32_t key, uint32_t id) {
    return ((unsigned long long)key << 32) | (unsigned long long)(~id);
}

__device__ __forceinline__ void glb_add(uint32_t* a, float v) { unsafeAtomicAdd(reinterpret_cast<float*>(a), v); }
__device__ __forceinline__ void glb_add(uint32_t* a, int v) { atomicAdd(reinterpret_cast<int*>(a), v); }

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// Fixed-point product of a query weight pre-scaled by 2^F (qd = w_q * 2^F, exact
// in fp64) and a stored document weight given by its fp32 bit pattern (bf16
// weights are widened first). One fp64 FMA forms qd * w_d + 2^52 with a single
// rounding; the per-query F keeps every product below 2^51, so the result lies in
// [2^52, 2^53) where the fp64 spacing is 1 and its low bits are the product
// rounded to the nearest integer (within half a unit of it). A product below half
// a unit becomes 0; the selection's wide-range check covers the queries where
// that could matter (their rows are summed again in fp64).
__device__ __forceinline__ unsigned long long fx_bits(double qd, uint32_t wbits) {  // exponent bits 0x433 on top
    constexpr double kTwo52 = 4503599627370496.0;
    const double wd = (double)__uint_as_float(wbits);
    return (unsigned long long)__double_as_longlong(__builtin_fma(qd, wd, kTwo52));
}
__device__ __forceinline__ unsigned long long fx_product(double qd, uint32_t wbits) {
    return fx_bits(qd, wbits) & 0x000fffffffffffffull;
}

// Write a finished LDS tile to the score array (fp32 bits or int32) and add its
// first-digit histogram (composite key (score bits, ~doc id), digit at fs).
// Accumulator forms: kAccInt (int32 sums, written as they are), kAccFx32 and
// kAccFx64 (unsigned fixed point in units of `scale`, written as fp32 bits), kAccF64
// (fp64 sums of exact fp64 products, the wide-range pass, written as fp32 bits).
enum AccForm { kAccInt = 0, kAccFx32 = 1, kAccFx64 = 2, kAccF64 = 3 };

// Fused candidate filtering: append the composites c >= bound of the lanes that
// take one to the query's candidate buffer (one atomic per wavefront). Past kFusedCap
// the query is flagged instead.
__device__ __forceinline__ void append_candidates(bool take, unsigned long long c, SelState* st,
                                                  unsigned long long* C) {
    const unsigned long long m = __ballot(take);
    if (m == 0) return;
    const int lane = threadIdx.x & (kWave - 1);
    int slot = 0;
    if (lane == 0) {
        slot = atomicAdd(&st->n_cand, __popcll(m));
        if (slot + __popcll(m) > kFusedCap) st->fused_over = 1;
    }
    slot = __shfl(slot, 0, kWave) + __popcll(m & ((1ull << lane) - 1ull));
    if (take && slot < kFusedCap) C[slot] = c;
}

// A document's score bits from its accumulator.
template <int AF, typename T>
__device__ __forceinline__ uint32_t score_bits(T acc, double scale) {
    if constexpr (AF == kAccInt) return acc;
    else if constexpr (AF == kAccF64) return __float_as_uint((float)acc);
    else return __float_as_uint((float)((double)acc * scale));
}

template <int AF>
using AccOf = std::conditional_t<AF == kAccFx64, unsigned long long, std::conditional_t<AF == kAccF64, double, uint32_t>>;

// Write a finished LDS tile to its score row (write) and, with count, add it to the query's
// first-digit histogram (hist: kHistLds words, zeroed by the caller) and its zero scores to the
// query's count of them.
template <int BS, int AF>
__device__ __forceinline__ void flush_tile(const void* acc_v, uint32_t* hist, int tile_n, uint32_t* Sq,
                                           FirstDigit fd, double scale, uint32_t* hist_out, SelState* st, bool write, bool count) {
    using T = AccOf<AF>;
    const T* acc = reinterpret_cast<const T*>(acc_v);
    const int tid = threadIdx.x, n4 = tile_n >> 2;
    int zc = 0;  // counted zero scores of this thread
    auto tally = [&](uint32_t v) {
        atomicAdd(&hist[first_digit<AF != kAccInt>(fd, v)], 1u);
        zc += v == 0u;
    };
    for (int i = tid; i < n4; i += BS) {
        T a[4];
        if constexpr (sizeof(T) == 4) {
            const uint4 u = reinterpret_cast<const uint4*>(acc)[i];
            a[0] = u.x; a[1] = u.y; a[2] = u.z; a[3] = u.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) a[j] = acc[4 * i + j];
        }
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = score_bits<AF>(a[j], scale);
        if (write) reinterpret_cast<uint4*>(Sq)[i] = make_uint4(v[0], v[1], v[2], v[3]);
        if (count)
#pragma unroll
            for (int j = 0; j < 4; j++) tally(v[j]);
    }
    for (int i = (n4 << 2) + tid; i < tile_n; i += BS) {
        const uint32_t v = score_bits<AF>(acc[i], scale);
        if (write) Sq[i] = v;
        if (count) tally(v);
    }
    if (!count) return;
    zc = wave_sum(zc);
    if ((tid & (kWave - 1)) == 0 && zc) atomicAdd(&hist[kHistBins], (uint32_t)zc);
    __syncthreads();
    for (int b = tid; b < kHistBins; b += BS)
        if (hist[b]) atomicAdd(&hist_out[b], hist[b]);
    if (tid == 0 && hist[kHistBins]) atomicAdd(&st->zeros, (int)hist[kHistBins]);
}

// Append a finished LDS tile's composites at or above the query's bound to its candidates (no
// row, no histogram). Few documents reach the bound (about 1 in 100), but nearly every
// wavefront holds some, so no conversion or compaction is done per document: each thread marks
// its documents whose raw sum can reach the bound in a bit mask (a compare and an add each),
// then the wavefront takes one marked document per lane at a time: exact composite, exact test,
// and a place in the wavefront's slice of an LDS stage (stage_cap entries for the workgroup),
// which goes to the query's buffer as one range; candidates past the slice go there directly.
// Converting every document of a wavefront with a hit took half of the kernel's vector
// instructions (fp32).
// Raw test: a document whose float score float(sum * scale) reaches the bound's score s_b has
// sum * scale >= s_b (1 - 2^-24), and converting the sum to double loses at most 2^-53 more, so
// a sum below t_lo (taken with margin) cannot reach it. A bound of score 0 takes zero-score
// documents up to the bound's id only, so a tile past that id marks positive sums alone.
template <int BS, int AF, int TILE>
__device__ __forceinline__ void flush_candidates(const void* acc_v, int tile_n, int64_t base, double scale,
                                                 unsigned long long bound, SelState* st, unsigned long long* C,
                                                 unsigned long long* stage, int stage_cap) {
    static_assert(AF != kAccF64, "integer sums");
    using T = AccOf<AF>;
    const T* acc = reinterpret_cast<const T*>(acc_v);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), per_w = stage_cap / (BS / kWave);
    unsigned long long* my_stage = stage + wv * per_w;
    int w_cnt = 0;  // staged candidates of the wavefront (uniform)
    T t_lo;
    if constexpr (AF == kAccInt) {
        t_lo = (uint32_t)(bound >> 32);
    } else {
        const double sb = (double)__uint_as_float((uint32_t)(bound >> 32));
        const double t = fmax(0.0, floor(sb * (1.0 - 0x1p-22) / scale));
        t_lo = AF == kAccFx64 ? (T)t : (T)fmin(t, 4294967295.0);
    }
    if (t_lo == 0 && base > (int64_t)(~(uint32_t)bound)) t_lo = 1;
    constexpr int D = TILE / BS, DB = D < 32 ? D : 32;  // documents per thread, per mask
#pragma unroll
    for (int d0 = 0; d0 < D; d0 += DB) {
        uint32_t mask = 0;  // bit DB - 1 - d: document d of this block
#pragma unroll
        for (int g = 0; g < DB / 4; g++) {
            const int i = tid + (d0 / 4 + g) * BS;  // documents 4 i ..
            T a[4];
            if constexpr (sizeof(T) == 4) {
                const uint4 u = reinterpret_cast<const uint4*>(acc)[i];
                a[0] = u.x; a[1] = u.y; a[2] = u.z; a[3] = u.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++) a[j] = acc[4 * i + j];
            }
#pragma unroll
            for (int j = 0; j < 4; j++) mask = mask + mask + (a[j] >= t_lo ? 1u : 0u);
        }
        while (__ballot(mask != 0u)) {
            const int d = DB - 1 - (31 - __clz((int)(mask | 1u)));  // this lane's next document
            const bool has = mask != 0u;
            if (has) mask &= ~(1u << (DB - 1 - d));
            const int doc = 4 * (tid + ((d0 + d) >> 2) * BS) + (d & 3);
            const unsigned long long c = comp_key(score_bits<AF>(acc[doc], scale), (uint32_t)(base + doc));
            const bool take = has && doc < tile_n && c >= bound;
            const unsigned long long m = __ballot(take);
            if (m == 0) continue;
            const int slot = w_cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (take && slot < per_w) my_stage[slot] = c;
            const int n = w_cnt + __popcll(m);
            if (n > per_w) append_candidates(take && slot >= per_w, c, st, C);  // past the slice
            w_cnt = min(n, per_w);
        }
    }
    if (w_cnt == 0) return;
    int b = 0;
    if (lane == 0) {
        b = atomicAdd(&st->n_cand, w_cnt);
        if (b + w_cnt > kFusedCap) st->fused_over = 1;
    }
    b = __builtin_amdgcn_readfirstlane(b);
    for (int i = lane; i < w_cnt; i += kWave)
        if (b + i < kFusedCap) C[b + i] = my_stage[i];
}

// ------------------------------------------------------------- tiled --
//
// One workgroup per (query, doc tile of 2^TS docs). LDS holds the tile's
// accumulators: unsigned fixed point for fp32 (64-bit) and bf16 (32-bit) weights
// (LDS integer atomics run far faster than LDS float atomics on this GPU, and
// integer sums do not depend on the order of the updates), int32 for uint8
// impacts.

// fp32 weights: 64-bit fixed point. Its error is absolute, (m+1) half-units of
// 2^-F with 2^-F about 2^-51 of the query's largest product: far inside the 1e-5
// relative rule for scores near the query's scale, not for scores many orders of
// magnitude below it. The selection checks each query's k-th score against that
// bound and sends the queries where it could fail to the fp64 pass (W).
// bf16 weights: 32-bit fixed point, whose scores only choose the candidates that
// are rescored in fp64 (the same check keeps the error band narrow). uint8
// impacts: int32, exact. W: fp64 accumulation of exact fp64 products.
template <int P, bool W = false>
constexpr int acc_form() {
    return W ? kAccF64 : (P == kFP32 ? kAccFx64 : (P == kBF16 ? kAccFx32 : kAccInt));
}

// Queries per work item of the group kernel. Two: 64 KiB of 32-bit accumulators over
// 8192 docs (bf16, uint8), so that two workgroups share a CU and one accumulates while the
// other flushes; 128 KiB of 64-bit ones (fp32). (Four queries with 32-bit sums, 128 KiB and
// one workgroup per CU, measured slower.)
template <int P>
constexpr int group_size() {
    return 2;
}

// Word 3 of a raw buffer descriptor on the gfx9 family (gfx950 included): no stride,
// no swizzle, 32-bit data format; the hardware range-checks each lane's byte offset
// against the record count and returns 0 past it.
constexpr int kRawBufferWord3 = 0x00020000;

// Segments of a (query, tile) work item of score_tile.
struct TileShared {
    int64_t seg_beg[kMaxQueryNnz];
    int32_t seg_len[kMaxQueryNnz];
    int32_t seg_cpre[kMaxQueryNnz + 1];
    double seg_qd[kMaxQueryNnz];   // w_q * 2^F (fixed point)
    uint32_t seg_q8[kMaxQueryNnz]; // uint8 query impact
    uint16_t seg_edge[kMaxQueryNnz];  // whole blocks: postings before | after the real segment << 8
    unsigned long long dmask[kMaxQueryNnz / kWave];  // (PR) essential terms per wavefront of the setup
    unsigned long long wmax[kMaxQueryNnz / kWave];   // pruning: largest bound sum per wavefront
    // what the flush needs of the query (its selection state and histogram scaling)
    unsigned long long fl_bound;
    double fl_scale;
    int fl_fused, fl_over;
    FirstDigit fl_first;
};
static_assert(kMaxQueryNnz <= 512 && kMaxQueryNnz % kWave == 0, "segment setup: one thread per query term");

// Chunk c of a tile's work (c is the same on every lane of the wavefront):
// segment index, first posting and length, kept in scalar registers. The
// segment comes from the chunk table when the tile has one, else from a binary
// search over the chunk prefix.
template <bool TAB>
__device__ __forceinline__ void chunk_at(const TileShared& sh, const uint8_t* tab, int nq, int c, int ch, int* seg,
                                         int64_t* p0, int* n, int* off_out) {
    int lo;
    if constexpr (TAB) {
        lo = tab[c];
    } else {
        lo = 0;
        int hi = nq - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (sh.seg_cpre[mid] <= c) lo = mid; else hi = mid - 1;
        }
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const int off = __builtin_amdgcn_readfirstlane((c - sh.seg_cpre[lo]) * ch);
    *off_out = off;
    *seg = lo;
    *n = __builtin_amdgcn_readfirstlane(min(ch, sh.seg_len[lo] - off));
    const int64_t p = sh.seg_beg[lo] + off;
    *p0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32) |
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p));
}

// Score one (query, doc tile) work item into LDS and flush it. Every thread of
// the workgroup calls this; it ends after the flush (callers that loop must
// synchronise before reusing the LDS). This is the form of the passes that score_item does
// not serve: W: the wide-range pass (fp64 products w_q * w_d, fp64 sums); the listed queries'
// rows; and
// PR: block-max pruning (MaxScore over 64-posting blocks) in the non-seed tiles of a query
// with a seed bound, for fp32 and uint8 weights. The query's
// terms with the smallest bounds w_q * maxw, as long as their bounds sum to less than the
// bound's raw score t_lo, are non-essential: no doc that holds none of the others can be a
// candidate. The essential terms are scored first; then each 64-doc group of the tile gets
// its largest partial sum, and a block of a non-essential term is skipped (not even read)
// when every doc it can hold has partial sum + the non-essential bounds' sum below t_lo. A
// doc of a skipped block can then not reach the bound, so it is no candidate, and every
// candidate's sum is complete: the result is exact.
template <int P, int TS, int CH, bool W = false, bool PR = false>
__device__ __forceinline__ void score_tile(const DevIndex& ix, const DevBatch& qb, int32_t q0, int64_t tile, int ql,
                                           uint32_t* __restrict__ S, int64_t ld, uint32_t* __restrict__ hist1,
                                           uint32_t* lds, TileShared& sh, int phase, SelState* state,
                                           unsigned long long* cand) {
    constexpr int BS = 512, NW = BS / kWave, TILE = 1 << TS, U = CH / kWave, GPT = TS - kGrainShift;
    constexpr bool FX = P != kU8;                  // fixed-point (or, W, fp64) products (fp32, bf16)
    constexpr int AF = acc_form<P, W>();
    constexpr int AW = (AF == kAccFx64 || AF == kAccF64) ? 2 : 1;  // accumulator words per doc
    unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(lds);  // [TILE] (fp32)
    uint32_t* acc32 = lds;                                                   // [TILE] (bf16, uint8)
    uint32_t* hist = lds + TILE * AW;                                        // [kHistLds]

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: chunk bookkeeping stays scalar
    const int q = q0 + ql;
    if (qb.k[q] == 0) return;  // nothing is selected for it (also every padding slot of a batch)
    if (phase == 3 && state[ql].rescore != 1) return;  // only the queries that fell back
    if (phase == 4 && state[ql].rescore != 2) return;  // only the wide-range queries
    if (phase == 5 && state[ql].rescore != 3) return;  // only the bf16 band passes of fused queries
    // What the flush needs of the query: one thread loads it now, so that the latency passes
    // under the setup, and leaves it in LDS (registers are what the accumulation runs short
    // of). The state is set before this launch; the cap flag may be set during it by other
    // workgroups, and a stale 0 only costs appends that the cap check drops.
    int fl_fused = 0, fl_over = 0;
    FirstDigit fl_first{0, 0};
    unsigned long long fl_bound = 0;
    double fl_scale = 1.0;
    if (threadIdx.x == BS - 1) {
        const SelState* stq0 = state + ql;
        fl_fused = stq0->fused;
        fl_over = stq0->fused_over;
        fl_bound = stq0->bound;
        fl_first = qb.first[q];
        fl_scale = (FX && !W) ? qb.q_scale[q] : 1.0;
    }
    const int64_t N = ix.n_docs;
    const int64_t base = tile << TS;
    const int tile_n = (int)min((int64_t)TILE, N - base);
    static_assert(TS <= 16, "a doc tile must lie inside one 65536-doc range");
    const int lbase = (int)(base & 0xFFFF);  // the tile's offset inside its 65536-doc range

    for (int i = tid; i < TILE * AW / 4; i += BS) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);

    const int64_t qa = qb.q_row_ptr[q];
    const int nq = (int)(qb.q_row_ptr[q + 1] - qa);
    const int64_t g0 = tile << GPT;
    const int64_t g1 = min(g0 + (int64_t)(1 << GPT), ix.n_grains);
    static_assert(!PR || (P != kBF16 && !W), "pruning: fp32 and uint8 fixed-point or integer sums");
    // Pruning applies to the non-seed tiles of a query whose seed bound is set; t_lo is the
    // bound's score as a raw sum (no sum below it can give a candidate, see flush_tile).
    bool prune_item = false;
    unsigned long long t_lo = 0;
    if constexpr (PR) {
        const SelState* stq = state + ql;
        if (phase == 2 && stq->fused == 1) {
            const uint32_t sb = (uint32_t)(stq->bound >> 32);
            if constexpr (P == kU8) t_lo = sb;
            else t_lo = (unsigned long long)fmax(0.0, floor((double)__uint_as_float(sb) * (1.0 - 0x1p-22) / qb.q_scale[q]));
            prune_item = t_lo > 0;
        }
    }
    // One thread per query term. With pruning the essential terms come first (exact segments)
    // and the non-essential ones after them (whole 64-posting blocks, each skipped or read).
    const int t = tid;
    const bool live = t < nq;
    int term = 0, a = 0, b = 0;
    bool first = false;  // (PR) an essential term
    unsigned long long ub_cum = 0;
    if (live) {
        term = qb.q_term[qa + t];
        const int32_t* row = ix.tile_off + (int64_t)term * (ix.n_grains + 1);
        a = row[g0];
        b = row[g1];
        if constexpr (PR) {
            ub_cum = qb.q_ub_cum[qa + t];
            first = !prune_item || !(ub_cum < t_lo);
        }
    }
    if (t < kMaxQueryNnz) {
        const unsigned long long m = __ballot(live && first);
        if (lane == 0) sh.dmask[wave] = m;
        if constexpr (PR) {
            // the bound sum of the non-essential terms: the largest cumulative bound among them
            unsigned long long v = (live && !first) ? ub_cum : 0ull;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                const unsigned long long o = __shfl_xor(v, d, kWave);
                v = o > v ? o : v;
            }
            if (lane == 0) sh.wmax[wave] = v;
        }
    }
    __syncthreads();
    if (live) {
        int before = 0, nd = 0;
#pragma unroll
        for (int w = 0; w < kMaxQueryNnz / kWave; w++) {
            const int pc = __popcll(sh.dmask[w]);
            nd += pc;
            if (w < wave) before += pc;
        }
        before += __popcll(sh.dmask[wave] & ((1ull << lane) - 1ull));
        const int slot = first ? before : nd + (t - before);
        bool zero_weight;
        if constexpr (FX) {
            const double qd = W ? (double)qb.q_w[qa + t] : qb.q_fx[qa + t];
            sh.seg_qd[slot] = qd;
            zero_weight = !(qd > 0.0);
        } else {
            const uint32_t q8 = (uint32_t)qb.q_w8[qa + t];
            sh.seg_q8[slot] = q8;
            zero_weight = q8 == 0u;
        }
        int beg = a, len = b - a, edge = 0;
        if (PR && !first && b > a) {  // whole blocks: lists start 64-aligned and are padded to 64
            beg = a & ~(kBlock - 1);
            const int end = (b + kBlock - 1) & ~(kBlock - 1);
            len = end - beg;
            edge = (a - beg) | ((end - b) << 8);
        }
        sh.seg_beg[slot] = ix.term_off[term] + beg;
        sh.seg_len[slot] = zero_weight ? 0 : len;  // a zero query weight adds nothing
        sh.seg_edge[slot] = (uint16_t)edge;
    }
    if (tid == BS - 1) {
        sh.fl_fused = fl_fused;
        sh.fl_over = fl_over;
        sh.fl_bound = fl_bound;
        sh.fl_first = fl_first;
        sh.fl_scale = fl_scale;
    }
    __syncthreads();
    {
        // Every wavefront computes the chunk prefix of all segments (lane l: segments
        // 4 l .. 4 l + 3) and writes its eighth of the chunk table; wavefront 0 also stores
        // the prefix.
        int c[4];
        int s = 0;
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int t = lane * 4 + u;
            c[u] = t < nq ? (sh.seg_len[t] + CH - 1) / CH : 0;
            s += c[u];
        }
        // Exclusive prefix of s over the lanes, one bit plane at a time: a ballot of bit b
        // and the count of the lower lanes that hold it (no cross-lane traffic through the
        // LDS, whose queue the other workgroup's atomics keep long).
        int run = 0, total = 0;
        for (int b = 0; __ballot((s >> b) != 0) != 0ull; b++) {
            const unsigned long long m = __ballot((s >> b) & 1);
            run += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) << b;
            total += __popcll(m) << b;
        }
        // Chunk table: during accumulation the histogram's LDS holds the segment index
        // of every chunk (one byte each), so a wavefront finds its chunk's segment with
        // one LDS read; tiles with more chunks than it holds fall back to a search.
        uint8_t* t8 = reinterpret_cast<uint8_t*>(hist);
        const bool table = total <= kHistBins * 4;
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (wave == 0) sh.seg_cpre[lane * 4 + u] = run;
            if (table)
                for (int j = wave; j < c[u]; j += NW) t8[run + j] = (uint8_t)(lane * 4 + u);
            run += c[u];
        }
        if (tid == 0) sh.seg_cpre[kMaxQueryNnz] = total;
    }
    __syncthreads();

    // Chunks go round-robin to the wavefronts. Each wavefront keeps two chunks in
    // flight: the loads of its next chunk are issued before the LDS adds of the
    // current one (two register sets, alternating).
    const int total = sh.seg_cpre[nq];
    const uint8_t* tab = total <= kHistBins * 4 ? reinterpret_cast<const uint8_t*>(hist) : nullptr;
    struct Chunk {
        uint32_t doc[U];  // doc id modulo 65536
        uint32_t w[U];    // stored weight as fp32 bits, or the uint8 impact
        int seg, n, lo;   // postings [lo, n) of the chunk are the segment's (lo > 0: first slot only)
        uint32_t skip;    // (pruned blocks) bit u: block u of the chunk is skipped
    };
    // Chunk forms: exact segment; non-essential term under pruning (whole blocks, skipped ones
    // not read).
    using FExact = std::integral_constant<bool, false>;
    using FPrune = std::integral_constant<bool, true>;
    // pruning: per 64-doc group of the tile, the largest sum of the essential terms (in the
    // histogram area's last 2 KiB, which the chunk table leaves free for pruned items)
    unsigned long long* gmax = reinterpret_cast<unsigned long long*>(hist) + (kHistBins / 2 - 256);
    unsigned long long u_n = 0;  // the bound sum of the non-essential terms
    const int tbase = __builtin_amdgcn_readfirstlane((int)base);
    using WT = std::conditional_t<P == kU8, uint8_t, std::conditional_t<P == kBF16, uint16_t, uint32_t>>;
    // Loads are straight-line (no branch around them, so the compiler can wait for
    // the older chunk only): lanes past the end of a chunk read 0, and an empty slot
    // reads nothing (record count 0). The chunk's base is wave-uniform (a buffer
    // descriptor in scalar registers), so no address arithmetic is done per posting.
    // The chunk lookup is branch-free with the chunk table (an invalid slot looks up
    // chunk 0 and gets length 0).
    auto load = [&](auto use_tab, auto form, int c, Chunk& k, bool valid) {
        constexpr bool PRUNED = decltype(form)::value;
        int64_t p0 = 0;
        int n = 0, off = 0;
        chunk_at<decltype(use_tab)::value>(sh, tab, nq, valid ? c : 0, CH, &k.seg, &p0, &n, &off);
        k.skip = 0u;
        if constexpr (PRUNED) {
            const int edge = __builtin_amdgcn_readfirstlane((int)sh.seg_edge[k.seg]);
            const int real_end = sh.seg_len[k.seg] - (edge >> 8) - off;
            k.lo = off == 0 ? (edge & 0xFF) : 0;
            k.n = valid ? min(n, real_end) : 0;
        } else {
            k.lo = 0;
            k.n = valid ? n : 0;
        }
        const int nblk = (n + kBlock - 1) >> 6;
        if constexpr (PRUNED) {
            // lane u < nblk decides block u: the docs it can hold are [its first doc, the next
            // block's first doc) inside the segment, the tile's end for the segment's last
            // block, clipped to the tile; it is skipped when every 64-doc group they touch has
            // essential sum + u_n below t_lo
            bool sk = false;
            if (valid && lane < nblk) {
                const int64_t blk = (p0 >> 6) + lane;
                const int64_t seg_end_blk = (sh.seg_beg[k.seg] + sh.seg_len[k.seg]) >> 6;
                const int first = ix.blk_first[blk];
                const int last = blk + 1 < seg_end_blk ? ix.blk_first[blk + 1] - 1 : tbase + tile_n - 1;
                const int lo = max(first - tbase, 0), hi = min(last - tbase, tile_n - 1);
                unsigned long long m = 0;
                for (int gi = lo >> 6; gi <= (hi >> 6); gi++) m = gmax[gi] > m ? gmax[gi] : m;
                sk = m + u_n < t_lo;
            }
            k.skip = (uint32_t)__ballot(sk);
            if (k.skip != 0u && lane == 0) atomicAdd(&state[ql].pruned, __popc(k.skip));
        }
        // Buffer loads over the chunk: the descriptor's record count is the chunk's bytes,
        // so lanes past its end read 0 without a clamp, and slot u's offset is the
        // instruction's immediate (one lane-offset register per chunk).
        const int nrec = valid ? n : 0;
        const void* lb = static_cast<const void*>(ix.post_lo + p0);
        // a skipped block's lanes get an offset past the record count: the hardware reads nothing
        auto far = [&](int u) { return PRUNED && ((k.skip >> u) & 1u) ? (1 << 30) : 0; };
        const void* wb = static_cast<const void*>(reinterpret_cast<const WT*>(ix.post_w) + p0);
        const __amdgpu_buffer_rsrc_t rid =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(lb), (short)0, nrec * 2, kRawBufferWord3);
        const __amdgpu_buffer_rsrc_t rw =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(wb), (short)0, nrec * (int)sizeof(WT), kRawBufferWord3);
        // z is 0 (posting offsets stay far below 2^48) but not a loop invariant, so the
        // compiler keeps one lane offset per chunk and each slot's offset in the
        // instruction, instead of holding a register per slot across the loop.
        const int z = (int)((uint64_t)p0 >> 48);
        const int vid = (lane << 1) + z;
        const int vw = lane * (int)sizeof(WT) + z;
#pragma unroll
        for (int u = 0; u < U; u++) {
            k.doc[u] = __builtin_amdgcn_raw_buffer_load_b16(rid, vid + far(u) + u * kWave * 2, 0, 0);
            uint32_t wv;
            if constexpr (sizeof(WT) == 4) wv = __builtin_amdgcn_raw_buffer_load_b32(rw, vw + far(u) + u * kWave * 4, 0, 0);
            else if constexpr (sizeof(WT) == 2) wv = __builtin_amdgcn_raw_buffer_load_b16(rw, vw + far(u) + u * kWave * 2, 0, 0);
            else wv = __builtin_amdgcn_raw_buffer_load_b8(rw, vw + far(u) + u * kWave, 0, 0);
            k.w[u] = P == kBF16 ? wv << 16 : wv;
        }
    };
    // Accumulators indexed by doc id modulo 65536: the tile's offset folded into the base.
    unsigned long long* acc64f = acc64 - lbase;
    uint32_t* acc32f = acc32 - lbase;
    // A full chunk (every lane holds a posting in every slot) adds without the
    // per-posting predicate; a segment's first (whole blocks) and last chunks are predicated.
    auto apply = [&](auto form, const Chunk& k) {
        constexpr bool PRUNED = decltype(form)::value;
        auto add = [&](auto pred) {
            constexpr bool PRED = decltype(pred)::value;
            auto ok = [&](int u) {
                return (!PRUNED || !((k.skip >> u) & 1u)) &&
                       (!PRED || ((u > 0 || lane >= k.lo) && lane + u * kWave < k.n));
            };
            if constexpr (AF == kAccFx64) {
                const double qd = uniform_f64(sh.seg_qd[k.seg]);
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (ok(u)) atomicAdd(acc64f + k.doc[u], fx_product(qd, k.w[u]));
            } else if constexpr (AF == kAccF64) {
                // products of two fp32 values (or fp32 and bf16) are exact in fp64
                double* acc = reinterpret_cast<double*>(acc64f);
                const double qd = uniform_f64(sh.seg_qd[k.seg]);
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (ok(u)) atomicAdd(acc + k.doc[u], qd * (double)__uint_as_float(k.w[u]));
            } else if constexpr (AF == kAccFx32) {
                // the query's scale keeps every doc's sum below 2^32 units
                const double qd = uniform_f64(sh.seg_qd[k.seg]);
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (ok(u)) atomicAdd(acc32f + k.doc[u], (uint32_t)fx_product(qd, k.w[u]));
            } else {
                const uint32_t q8v = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.seg_q8[k.seg]);
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (ok(u)) atomicAdd(acc32f + k.doc[u], __umul24(q8v, k.w[u]));  // both below 256: full rate
            }
        };
        if (k.n == CH && k.lo == 0) add(std::false_type());
        else add(std::true_type());
    };
    // Chunks c = wave, wave + NW, ... below `end`; returns the wavefront's first chunk at
    // or past `end`.
    auto run = [&](auto use_tab, auto form, int c, int end) -> int {
        Chunk A, B;
        load(use_tab, form, c, A, c < end);
        while (c < end) {
            const int cb = c + NW;
            load(use_tab, form, cb, B, cb < end);
            apply(form, A);
            if (cb >= end) return cb;
            const int ca = cb + NW;
            load(use_tab, form, ca, A, ca < end);
            apply(form, B);
            c = ca;
        }
        return c;
    };
    if constexpr (PR) {
        // The chunk table must leave the last 2 KiB of the histogram area to the group maxima;
        // otherwise nothing is skipped (t_lo 0), the non-essential blocks are all read.
        if (prune_item && total > kHistBins * 4 - 2048) {
            prune_item = false;
            t_lo = 0;
        }
        u_n = sh.wmax[0];
#pragma unroll
        for (int w = 1; w < kMaxQueryNnz / kWave; w++) u_n = sh.wmax[w] > u_n ? sh.wmax[w] : u_n;
    }
    if (total > 0) {
        int n_dense = 0;
#pragma unroll
        for (int w = 0; w < kMaxQueryNnz / kWave; w++) n_dense += __popcll(sh.dmask[w]);
        const int total_d = __builtin_amdgcn_readfirstlane(sh.seg_cpre[n_dense]);
        auto two_loops = [&](auto use_tab) {
            int c = wave;
            if constexpr (PR) {
                // essential terms, then the largest essential sum of every 64-doc group, then
                // the non-essential terms block by block
                c = total_d > 0 ? run(use_tab, FExact(), wave, total_d) : wave;
                if (total_d < total) {  // non-essential terms exist: whole-block segments
                    __syncthreads();
                    for (int gi = tid >> 2; gi < TILE / 64; gi += BS / 4) {
                        unsigned long long m = 0;
                        for (int j = 0; j < 16; j++) {
                            const int d = gi * 64 + (tid & 3) * 16 + j;
                            if (d < tile_n) {
                                const unsigned long long v =
                                    AF == kAccFx64 ? acc64[d] : (unsigned long long)acc32[d];
                                m = v > m ? v : m;
                            }
                        }
                        unsigned long long o = __shfl_xor(m, 1, kWave);
                        m = o > m ? o : m;
                        o = __shfl_xor(m, 2, kWave);
                        m = o > m ? o : m;
                        if ((tid & 3) == 0 && prune_item) gmax[gi] = m;
                    }
                    __syncthreads();
                    run(use_tab, FPrune(), c, total);
                }
            } else {
                run(use_tab, FExact(), c, total);
            }
        };
        if (tab) two_loops(std::true_type());
        else two_loops(std::false_type());
    }
    __syncthreads();
    for (int i = tid; i < kHistLds; i += BS) hist[i] = 0u;
    __syncthreads();
    // Fused filtering (the non-seed tiles of a query whose seed bound is set): append while
    // flushing, no appends once past the cap, and no score row. A query that falls back gets
    // its rows from phase 3; a bf16 query whose error band reaches below its candidates gets
    // them from phase 5, before the band pass.
    SelState* st = state + ql;
    if (phase == 2 && sh.fl_fused == 1) {
        if constexpr (AF != kAccF64)
            if (!sh.fl_over)
                flush_candidates<BS, AF, TILE>(lds, tile_n, base, sh.fl_scale, sh.fl_bound, st,
                                               cand + (int64_t)ql * kCandCap,
                                               reinterpret_cast<unsigned long long*>(hist), kHistBins / 2);
        return;
    }
    flush_tile<BS, AF>(lds, hist, tile_n, S + (int64_t)ql * ld + base, sh.fl_first, sh.fl_scale,
                       hist1 + (int64_t)ql * kHistBins, st, true, true);
}

// The tile's accumulators from the rows of the query's commonest terms (the first nr of its
// scoring terms; `rec` holds the first 64, one per lane): every thread sums a few documents in
// registers over all the rows and writes them to LDS, which starts the tile (zeros without
// rows). Two rows are in flight per wavefront (uint8: two steps of four).
// Why: a posting scatter-added into LDS costs 1/8 (32-bit) or 1/5.6 (64-bit) of a CU's clock,
// which bounded the batched search; with SPLADE-like term frequencies a few rows hold most of a
// query's postings (nine terms of thirty, nine postings of ten), and a row's document costs
// about 1/80 (uint8, four rows per dot4) to 1/20 clock (fp32: convert, FMA, 64-bit add) of
// vector arithmetic, with coalesced 16-byte loads and no doc ids. The integer sums are the
// same, whatever the order.
// The rows are stored grain by grain (8192 documents, all rows of a grain side by side: one or
// two memory pages per tile instead of one per row), and inside a grain in the order that the
// threads write them: a thread's 16-byte load holds fours of consecutive documents 2048 apart,
// so that each of its 16-byte LDS writes is next to its neighbours' and no bank conflicts.
template <int P, int TS>
__device__ __forceinline__ void sum_rows(const DevIndex& ix, const ScoreTerm* __restrict__ terms, ScoreTerm rec, int nr,
                                         int64_t base, uint32_t* lds) {
    using WT = std::conditional_t<P == kU8, uint8_t, std::conditional_t<P == kBF16, uint16_t, uint32_t>>;
    constexpr int BS = 512, TILE = 1 << TS;
    constexpr int DPL = 16 / (int)sizeof(WT);  // documents per 16-byte load
    constexpr int G = TILE / (BS * DPL);       // loads per thread and row
    constexpr int GM = (P == kFP32 ? 16 : 32) / DPL, GB = G < GM ? G : GM;  // of them in registers at once
    constexpr int R = P == kU8 ? 4 : 1;        // rows per step
    using Acc = std::conditional_t<P == kFP32, unsigned long long, uint32_t>;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    // grain by grain, all rows of one grain together
    constexpr int PER = (1 << kGrainShift) / (BS * DPL);  // loads per thread, row and grain
    const int64_t g_first = base >> kGrainShift, left = ix.n_grains - g_first;
    const int grain = ix.n_rows << kGrainShift;
    const int nrec = (((int)(left < (TILE >> kGrainShift) ? left : (TILE >> kGrainShift)) - 1) * grain +
                      (1 << kGrainShift)) * (int)sizeof(WT);
    const WT* rows = reinterpret_cast<const WT*>(ix.rows) + g_first * grain;
    struct Step {
        uint32_t w[R][GB][4];
        unsigned long long q[R];
    };
#pragma unroll
    for (int g0 = 0; g0 < G; g0 += GB) {
        ScoreTerm rr = rec;  // the 64 terms that the step's rows are among
        auto fetch = [&](int i0, Step& b) {
            if (i0 >= kWave && (i0 & (kWave - 1)) == 0 && i0 < nr) rr = terms[min(i0 + lane, nr - 1)];
#pragma unroll
            for (int r = 0; r < R; r++) {
                const bool have = i0 + r < nr;  // a missing row reads nothing (record count 0) and weighs 0
                const int l = (i0 + r) & (kWave - 1);
                const int64_t row = have ? __builtin_amdgcn_readlane(rr.row, l) : 0;
                b.q[r] = have ? read_lane64(rr.q, l) : 0ull;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<WT*>(rows + (row << kGrainShift)), (short)0, have ? nrec : 0, kRawBufferWord3);
#pragma unroll
                for (int g = 0; g < GB; g++) {
                    const int at = (g0 + g) / PER * grain * (int)sizeof(WT) + ((g0 + g) % PER * BS + tid) * 16;
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0);
#pragma unroll
                    for (int x = 0; x < 4; x++) b.w[r][g][x] = v[x];
                }
            }
        };
        Acc acc[GB * DPL];
#pragma unroll
        for (int i = 0; i < GB * DPL; i++)  // fp32: the exponent bits of the rows' products (see fx_bits) taken off
            acc[i] = P == kFP32 ? (Acc)(0ull - (unsigned long long)nr * 0x4330000000000000ull) : (Acc)0;
        auto add = [&](const Step& b) {
            if constexpr (P == kU8) {
                uint32_t q4 = 0;
#pragma unroll
                for (int r = 0; r < R; r++) q4 |= (uint32_t)b.q[r] << (8 * r);
#pragma unroll
                for (int g = 0; g < GB; g++)
#pragma unroll
                    for (int x = 0; x < 4; x++) {
                        // four rows' words of four documents each: transposed to a word per document
                        const uint32_t t0 = __builtin_amdgcn_perm(b.w[1][g][x], b.w[0][g][x], 0x05010400u);
                        const uint32_t t1 = __builtin_amdgcn_perm(b.w[3][g][x], b.w[2][g][x], 0x05010400u);
                        const uint32_t t2 = __builtin_amdgcn_perm(b.w[1][g][x], b.w[0][g][x], 0x07030602u);
                        const uint32_t t3 = __builtin_amdgcn_perm(b.w[3][g][x], b.w[2][g][x], 0x07030602u);
                        Acc* a = &acc[g * DPL + 4 * x];
                        a[0] = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(t1, t0, 0x05040100u), q4, a[0], false);
                        a[1] = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(t1, t0, 0x07060302u), q4, a[1], false);
                        a[2] = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(t3, t2, 0x05040100u), q4, a[2], false);
                        a[3] = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(t3, t2, 0x07060302u), q4, a[3], false);
                    }
            } else {
                const double qd = __longlong_as_double((long long)b.q[0]);
#pragma unroll
                for (int g = 0; g < GB; g++)
#pragma unroll
                    for (int d = 0; d < DPL; d++) {
                        if constexpr (P == kFP32) {
                            acc[g * DPL + d] += fx_bits(qd, b.w[0][g][d]);
                        } else {
                            const uint32_t x = b.w[0][g][d >> 1];
                            acc[g * DPL + d] += (uint32_t)fx_product(qd, (d & 1) ? x & 0xffff0000u : x << 16);
                        }
                    }
            }
        };
        if (nr > 0) {
            Step A, B;
            fetch(0, A);
            for (int i0 = 0; i0 < nr; i0 += 2 * R) {
                fetch(i0 + R, B);
                add(A);
                if (i0 + R >= nr) break;
                fetch(i0 + 2 * R, A);
                add(B);
            }
        }
#pragma unroll
        for (int g = 0; g < GB; g++) {
            const Acc* a = &acc[g * DPL];
#pragma unroll
            for (int m = 0; m < DPL / 4; m++) {
                const int at = (g0 + g) * (BS * DPL / 4) + m * BS + tid;  // documents 4 at ..
                if constexpr (P == kFP32) {
                    uint4* o = reinterpret_cast<uint4*>(lds) + 2 * at;
                    o[0] = make_uint4((uint32_t)a[0], (uint32_t)(a[0] >> 32), (uint32_t)a[1], (uint32_t)(a[1] >> 32));
                    o[1] = make_uint4((uint32_t)a[2], (uint32_t)(a[2] >> 32), (uint32_t)a[3], (uint32_t)(a[3] >> 32));
                } else {
                    reinterpret_cast<uint4*>(lds)[at] = make_uint4(a[4 * m], a[4 * m + 1], a[4 * m + 2], a[4 * m + 3]);
                }
            }
        }
    }
}

// The doc-tiled kernel: one workgroup per (query, doc tile) work item.
//  1. Rows: the sums of the query's commonest terms start the tile (sum_rows).
//  2. Postings: the segments of its other terms in this tile are scatter-added into LDS. Each
//     wavefront holds the segments of 64 terms in its lanes (no LDS table, no barrier) and takes
//     every eighth chunk of CH postings; the loads of its next chunk are issued before the LDS
//     adds of the current one. Ids and weights are read four postings per lane: one 8-byte load
//     of ids and one load of four weights (4, 8 or 16 bytes) cover a lane's postings 4 l ..
//     4 l + 3 of each 256 postings of the chunk, a quarter of the vector memory instructions of
//     one posting per lane. Segment starts are rounded down to a multiple of 4 (the postings
//     before the real start are masked).
//  3. Flush: candidates (flush_candidates), or row and histogram (flush_tile).
// A work item is a chain of dependent loads (item, terms, segments, postings) with little work
// behind each, and two workgroups share a CU, so the chain is kept short: the item and term
// records hold what the batch update knows (16 bytes each), the segment bounds are loaded under
// the rows, and only two barriers order the tile.
// Items run tile by tile, an eighth of them on each XCD (workgroups are dealt to the XCDs round
// robin), so that a tile's rows and postings are read from that XCD's L2 by most of the queries
// that need them; the items of a batch are ordered by descending work, dealt into eight runs
// (ScoreItem), so that equal eighths are equal work. One mapping for the TILED and SHARED forms.
template <int P, int TS, int CH>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_score_tiled(
    DevIndex ix, const ScoreItem* __restrict__ items, const ScoreTerm* __restrict__ all_terms,
    const FirstDigit* __restrict__ first, const double* __restrict__ q_scale, int32_t q0, int32_t qt,
    uint32_t* __restrict__ S, int64_t ld, uint32_t* __restrict__ hist1, int phase, int stride,
    SelState* __restrict__ state, unsigned long long* __restrict__ cand) {
    constexpr int BS = 512, NW = BS / kWave, TILE = 1 << TS, GPT = TS - kGrainShift;
    constexpr bool FX = P != kU8;
    constexpr int AF = acc_form<P>();
    constexpr int AW = AF == kAccFx64 ? 2 : 1;  // accumulator words per doc
    static_assert(CH % 256 == 0, "chunks of 256-posting rows");
    using WT = std::conditional_t<P == kU8, uint8_t, std::conditional_t<P == kBF16, uint16_t, uint32_t>>;
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t* hist = lds + TILE * AW;  // [kHistLds]; the candidates' stage of a flush that does not count
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: chunk bookkeeping stays scalar

    const uint32_t n_tiles = (uint32_t)phase_tiles(phase, stride, (ix.n_docs + TILE - 1) >> TS);
    const uint32_t total_items = n_tiles * (uint32_t)qt, per = (total_items + 7) / 8;
    const uint32_t in_xcd = blockIdx.y * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const uint32_t item = (blockIdx.x & 7) * per + in_xcd;
    if (in_xcd >= per || item >= total_items) return;
    // the division runs in vector registers: back to a scalar, so that all below it stays scalar
    const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)(item / (uint32_t)qt));
    const ScoreItem it = items[item - v * (uint32_t)qt];
    if (it.n < 0) return;  // nothing is selected for the query (also every padding slot of a batch)
    const int64_t tile = phase_tile(phase, stride, (int64_t)v);
    const int ql = it.q - q0, nt = it.n & 1023, nr = it.n >> 10;
    const int64_t base = tile << TS;
    const int tile_n = (int)min((int64_t)TILE, ix.n_docs - base);
    static_assert(TS <= 16, "a doc tile must lie inside one 65536-doc range");
    const int lbase = (int)(base & 0xFFFF);  // the tile's offset inside its 65536-doc range
    const int64_t g0 = tile << GPT;
    const int64_t g1 = min(g0 + (int64_t)(1 << GPT), ix.n_grains);

    // What the flush needs of the query. The state is set before this launch; the cap flag may be
    // set during it by other workgroups, and a stale 0 only costs appends that the cap check drops.
    SelState* st = state + ql;
    const int fl_fused = st->fused, fl_over = st->fused_over;
    const unsigned long long fl_bound = st->bound;
    const bool fused_q = phase == 2 && fl_fused == 1;
    // Fused filtering (the non-seed tiles of a query whose seed bound is set): append while
    // flushing, no appends once past the cap, and no score row or counts. A query that falls back
    // gets its rows and counts from phase 3; a bf16 query whose error band reaches below its
    // candidates gets its rows from phase 5, before the band pass.
    const bool count = !fused_q && phase != kPhaseRows;

    // the first 64 terms, one per lane, and the segments of those among them without a row here
    const ScoreTerm* terms = all_terms + it.start;
    ScoreTerm rec{0, 0, 0ull};
    if (lane < nt) rec = terms[lane];
    struct Seg {
        int a, b;
        int64_t off;
    };
    auto segment = [&](const ScoreTerm& t, bool live) {
        Seg s{0, 0, 0};
        if (live) {
            const int32_t* row = ix.tile_off + (int64_t)t.term * (ix.n_grains + 1);
            s.a = row[g0];
            s.b = row[g1];
            s.off = ix.term_off[t.term];
        }
        return s;
    };
    Seg seg = segment(rec, lane >= nr && lane < nt);
    if (count)
        for (int i = tid; i < kHistLds; i += BS) hist[i] = 0u;
    sum_rows<P, TS>(ix, terms, rec, nr, base, lds);
    __syncthreads();

    struct Chunk {
        uint32_t doc[CH / 128];                     // four 16-bit ids per 256 postings: doc modulo 65536
        uint32_t w[CH / 256 * (int)sizeof(WT)];     // their weights
        int n, lo;                                  // postings [lo, n) of the chunk are the segment's
        unsigned long long q;                       // w_q * 2^F as fp64 bits, or the uint8 impact
    };
    for (int grp = nr >> 6; grp * kWave < nt; grp++) {
        const int idx = grp * kWave + lane;
        if (grp > 0) {
            rec = ScoreTerm{0, 0, 0ull};
            if (idx < nt) rec = terms[idx];
            seg = segment(rec, idx >= nr && idx < nt);
        }
        // each lane's chunks, and the number before them: an exclusive prefix over the lanes one
        // bit plane at a time (a ballot and the count of the lower lanes that hold the bit)
        const int64_t beg = seg.off + (seg.a & ~3);
        const int len = seg.b > seg.a ? seg.b - (seg.a & ~3) : 0, cnt = (len + CH - 1) / CH, edge = seg.a & 3;
        int pre = 0, total = 0;
        for (int b = 0; __ballot((cnt >> b) != 0) != 0ull; b++) {
            const unsigned long long m = __ballot((cnt >> b) & 1);
            pre += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) << b;
            total += __popcll(m) << b;
        }
        // Straight-line loads (no branch around them): an empty slot reads nothing (record count
        // 0), and lanes past the end of a chunk read 0. The chunk's base is wave-uniform (a buffer
        // descriptor in scalar registers), so no address arithmetic is done per posting.
        auto fetch = [&](int c, Chunk& k) {
            const bool valid = c < total;
            const unsigned long long m = __ballot(c >= pre && c < pre + cnt);
            const int l = valid ? __ffsll((long long)m) - 1 : 0;
            const int off = valid ? (c - __builtin_amdgcn_readlane(pre, l)) * CH : 0;
            k.n = valid ? min(CH, __builtin_amdgcn_readlane(len, l) - off) : 0;
            k.lo = off == 0 ? __builtin_amdgcn_readlane(edge, l) : 0;
            k.q = read_lane64(rec.q, l);
            const int64_t p0 = (int64_t)read_lane64((unsigned long long)beg, l) + off;
            const int nrec = (k.n + 3) & ~3;  // up to 3 postings past the segment, inside the padded list
            const __amdgpu_buffer_rsrc_t rid = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint16_t*>(ix.post_lo + p0), (short)0, nrec * 2, kRawBufferWord3);
            const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<WT*>(reinterpret_cast<const WT*>(ix.post_w) + p0), (short)0, nrec * (int)sizeof(WT),
                kRawBufferWord3);
            // z is 0 (posting offsets stay far below 2^48) but not a loop invariant, so the compiler
            // keeps one lane offset per chunk and each row's offset in the instruction
            const int z = (int)((uint64_t)p0 >> 48);
            const int vid = lane * 8 + z;
            const int vw = lane * 4 * (int)sizeof(WT) + z;
#pragma unroll
            for (int r = 0; r < CH / 256; r++) {
                const auto d = __builtin_amdgcn_raw_buffer_load_b64(rid, vid + r * 512, 0, 0);
                k.doc[2 * r] = d[0];
                k.doc[2 * r + 1] = d[1];
                if constexpr (sizeof(WT) == 1) {
                    k.w[r] = __builtin_amdgcn_raw_buffer_load_b32(rw, vw + r * 256, 0, 0);
                } else if constexpr (sizeof(WT) == 2) {
                    const auto w = __builtin_amdgcn_raw_buffer_load_b64(rw, vw + r * 512, 0, 0);
                    k.w[2 * r] = w[0];
                    k.w[2 * r + 1] = w[1];
                } else {
                    const auto w = __builtin_amdgcn_raw_buffer_load_b128(rw, vw + r * 1024, 0, 0);
#pragma unroll
                    for (int x = 0; x < 4; x++) k.w[4 * r + x] = w[x];
                }
            }
        };
        auto apply = [&](const Chunk& k) {
            const double qd = __longlong_as_double((long long)k.q);
            auto add = [&](auto pred, int r) {
                constexpr bool PRED = decltype(pred)::value;
                // accumulators indexed by doc id modulo 65536: the tile's offset folded into the base
                unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(lds) - lbase;
                uint32_t* acc32 = lds - lbase;
                const int i0 = lane * 4 - k.lo;  // a posting is the segment's if its index less lo is below n - lo
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    if (PRED && (uint32_t)(i0 + r * 256 + j) >= (uint32_t)(k.n - k.lo)) continue;
                    const uint32_t dw = k.doc[2 * r + (j >> 1)];
                    const uint32_t at = (j & 1) ? (dw >> 16) : (dw & 0xffffu);
                    if constexpr (P == kFP32) {
                        atomicAdd(acc64 + at, fx_product(qd, k.w[4 * r + j]));
                    } else if constexpr (P == kBF16) {
                        const uint32_t h = k.w[2 * r + (j >> 1)];
                        atomicAdd(acc32 + at, (uint32_t)fx_product(qd, (j & 1) ? h & 0xffff0000u : h << 16));
                    } else {
                        atomicAdd(acc32 + at, __umul24((uint32_t)k.q, (k.w[r] >> (8 * j)) & 0xffu));
                    }
                }
            };
            // a full row of 256 adds without the per-posting predicate
#pragma unroll
            for (int r = 0; r < CH / 256; r++) {
                if (r * 256 >= k.n) break;
                if (r * 256 + 256 <= k.n && (r > 0 || k.lo == 0)) add(std::false_type(), r);
                else add(std::true_type(), r);
            }
        };
        Chunk A, B;
        fetch(wave, A);
        for (int c = wave; c < total; c += 2 * NW) {
            fetch(c + NW, B);
            apply(A);
            if (c + NW >= total) break;
            fetch(c + 2 * NW, A);
            apply(B);
        }
    }
    __syncthreads();
    const double scale = FX ? q_scale[it.q] : 1.0;
    if (!fused_q)
        flush_tile<BS, AF>(lds, hist, tile_n, S + (int64_t)ql * ld + base, first[it.q], scale,
                           hist1 + (int64_t)ql * kHistBins, st, true, count);
    else if (!fl_over)
        flush_candidates<BS, AF, TILE>(lds, tile_n, base, scale, fl_bound, st, cand + (int64_t)ql * kCandCap,
                                       reinterpret_cast<unsigned long long*>(hist), kHistBins / 2);
}

// The non-seed tiles with block-max pruning: grid (tiles, queries).
template <int P, int TS, int CH>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_score_pruned(
    DevIndex ix, DevBatch qb, int32_t q0, uint32_t* __restrict__ S, int64_t ld, uint32_t* __restrict__ hist1,
    int phase, int stride, SelState* __restrict__ state, unsigned long long* __restrict__ cand) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ TileShared sh;
    const int64_t tile = phase_tile(phase, stride, (int64_t)blockIdx.x);
    score_tile<P, TS, CH, false, true>(ix, qb, q0, tile, (int)blockIdx.y, S, ld, hist1, lds, sh, phase, state, cand);
}

// The rows of the listed queries scored again, a few workgroups per tile sharing the list (usually
// empty): those that fell back from fused filtering (phase 3), were found wide range (phase 4, W:
// fp64 accumulation) or need their band pass's rows (phase 5). score_tile skips the other kinds. A
// kernel of its own, so that the per-query kernel's registers hold one copy of the scoring loop.
template <int P, int TS, int CH, bool W = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_score_listed(
    DevIndex ix, DevBatch qb, int32_t q0, uint32_t* __restrict__ S, int64_t ld, uint32_t* __restrict__ hist1,
    int phase, int stride, SelState* __restrict__ state, unsigned long long* __restrict__ cand,
    const uint32_t* __restrict__ counters, const int32_t* __restrict__ rescore_list) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ TileShared sh;
    const int64_t tile = phase_tile(phase, stride, (int64_t)blockIdx.x);
    const int nres = (int)counters[kCntListed];
    for (int r = (int)blockIdx.y; r < nres; r += (int)gridDim.y) {
        score_tile<P, TS, CH, W>(ix, qb, q0, tile, rescore_list[r], S, ld, hist1, lds, sh, phase, state, cand);
        __syncthreads();
    }
}

// ------------------------------------------------------------- group --
//
// Shared traversal with explicit sharing: a work item is (doc tile, group of G
// queries), G = 2. The LDS holds G accumulator tiles of 8192 docs (64 KiB with
// 32-bit sums for bf16 and uint8, 128 KiB with 64-bit fixed point for fp32). The
// segments are those of the union of the group's terms (built on the host, with
// each member's weight per union term, 0 where the member lacks the term), so a
// posting chunk is loaded once and scatter-added into the tile of every member
// that holds its term. The items of a tile run on one XCD (tile-major), groups in
// the host's order (heaviest first).
template <int MT, int G>
struct GroupShared {
    union {
        struct {
            int64_t beg[MT];
            int32_t len[MT];
            int32_t cpre[MT + 1];
        } seg;
        uint32_t hist[kHistLds];  // the flush histogram, once the segments are no longer read
    };
    uint32_t w[MT][G];  // per union term, each member's w_q (fp32 bits) or uint8 impact
    uint16_t tab[kGroupChunkTab];  // chunk -> union term, when the item has at most that many chunks
    int32_t wave_sum[16];
    int64_t item;
};

template <int P, int CH>
__global__ __launch_bounds__(group_size<P>() * kMaxQueryNnz) __attribute__((amdgpu_waves_per_eu(4))) void k_score_group(
    DevIndex ix, DevBatch qb, uint32_t* __restrict__ counters, uint32_t* __restrict__ S, int64_t ld,
    uint32_t* __restrict__ hist1, int phase, int stride, SelState* __restrict__ state,
    unsigned long long* __restrict__ cand) {
    constexpr int G = group_size<P>();
    constexpr int MT = G * kMaxQueryNnz;  // most union terms of a group; one thread each
    constexpr int TS = kGroupTileShift, TILE = 1 << TS, BS = MT, NW = BS / kWave, U = CH / kWave;
    static_assert(NW <= 16, "wave sums");
    constexpr bool FX = P != kU8;
    constexpr int AF = acc_form<P>();
    constexpr int AW = AF == kAccFx64 ? 2 : 1;  // accumulator words per doc
    extern __shared__ __align__(16) uint32_t lds[];  // [G][TILE * AW]
    __shared__ GroupShared<MT, G> sh;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x = (int)(blockIdx.x & 7);
    const int64_t n_tiles = phase_tiles(phase, stride, (ix.n_docs + TILE - 1) >> TS);
    const int64_t tiles_x = n_tiles > x ? (n_tiles - x + 7) / 8 : 0;
    const int ng = qb.g_count[0];
    const int64_t items = tiles_x * ng;
    using WT = std::conditional_t<P == kU8, uint8_t, std::conditional_t<P == kBF16, uint16_t, uint32_t>>;
    for (;;) {
        if (tid == 0) sh.item = (int64_t)atomicAdd(&counters[cnt_base(phase) + x], 1u);
        __syncthreads();
        const int64_t item = sh.item;
        if (item >= items) break;
        const int64_t tile = phase_tile(phase, stride, x + 8 * (item / ng));
        const int g = (int)(item % ng);
        const int64_t base = tile << TS;
        const int tile_n = (int)min((int64_t)TILE, ix.n_docs - base);
        const int lbase = (int)(base & 0xFFFF);
        const int gr = qb.g_row[g], nu = qb.g_row[g + 1] - gr;
        for (int i = tid; i < G * TILE * AW; i += BS) lds[i] = 0u;
        // segments of the union terms in this tile; a term no member weighs adds nothing
        const int64_t g0 = tile << (TS - kGrainShift);
        const int64_t g1 = min(g0 + (int64_t)(1 << (TS - kGrainShift)), ix.n_grains);
        int c = 0;
        if (tid < nu) {
            const int term = qb.g_term[gr + tid];
            const int32_t* row = ix.tile_off + (int64_t)term * (ix.n_grains + 1);
            const int a = row[g0], b = row[g1];
            bool any = false;
#pragma unroll
            for (int m = 0; m < G; m++) {
                uint32_t wv;
                if constexpr (FX) wv = __float_as_uint(qb.g_wq[(int64_t)(gr + tid) * G + m]);
                else wv = (uint32_t)qb.g_w8[(int64_t)(gr + tid) * G + m];
                sh.w[tid][m] = wv;
                any |= wv != 0u;  // weights are >= 0: a zero bit pattern is a zero weight
            }
            sh.seg.beg[tid] = ix.term_off[term] + a;
            sh.seg.len[tid] = any ? b - a : 0;
            c = any ? (b - a + CH - 1) / CH : 0;
        }
        // exclusive prefix of the chunk counts over the union terms (one per thread)
        int incl = c;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int v = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += v;
        }
        if (lane == kWave - 1) sh.wave_sum[wave] = incl;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const int ws_ = sh.wave_sum[w];
            before += w < wave ? ws_ : 0;
            total += ws_;
        }
        if (tid < nu) sh.seg.cpre[tid] = before + incl - c;
        if (tid == 0) sh.seg.cpre[MT] = total;
        // chunk table: each union term writes its chunks' entries
        const bool use_tab = total <= kGroupChunkTab;
        if (use_tab && tid < nu)
            for (int j = 0; j < c; j++) sh.tab[before + incl - c + j] = (uint16_t)tid;
        __syncthreads();
        struct Chunk {
            uint32_t doc[U];
            uint32_t w[U];
            int seg, n;
        };
        auto load = [&](int cc, Chunk& k, bool valid) {
            // segment of chunk cc: the chunk table, else a binary search over the prefix
            const int want = valid ? cc : 0;
            int lo = 0;
            if (use_tab) {
                lo = total > 0 ? (int)sh.tab[want] : 0;
            } else {
                int hi = max(nu - 1, 0);
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (sh.seg.cpre[mid] <= want) lo = mid; else hi = mid - 1;
                }
            }
            lo = __builtin_amdgcn_readfirstlane(lo);
            const int off = __builtin_amdgcn_readfirstlane((want - sh.seg.cpre[lo]) * CH);
            const int n = valid ? __builtin_amdgcn_readfirstlane(min(CH, sh.seg.len[lo] - off)) : 0;
            const int64_t pp = sh.seg.beg[lo] + off;
            const int64_t p0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(pp >> 32)) << 32) |
                                         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)pp));
            k.seg = lo;
            k.n = n;
            const __amdgpu_buffer_rsrc_t rid = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint16_t*>(ix.post_lo + p0), (short)0, n * 2, kRawBufferWord3);
            const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<WT*>(reinterpret_cast<const WT*>(ix.post_w) + p0), (short)0, n * (int)sizeof(WT),
                kRawBufferWord3);
            const int z = (int)((uint64_t)p0 >> 48);  // 0, but not a loop invariant (see score_tile)
            const int vid = (lane << 1) + z;
            const int vw = lane * (int)sizeof(WT) + z;
#pragma unroll
            for (int u = 0; u < U; u++) {
                k.doc[u] = __builtin_amdgcn_raw_buffer_load_b16(rid, vid + u * kWave * 2, 0, 0);
                uint32_t wv;
                if constexpr (sizeof(WT) == 4) wv = __builtin_amdgcn_raw_buffer_load_b32(rw, vw + u * kWave * 4, 0, 0);
                else if constexpr (sizeof(WT) == 2) wv = __builtin_amdgcn_raw_buffer_load_b16(rw, vw + u * kWave * 2, 0, 0);
                else wv = __builtin_amdgcn_raw_buffer_load_b8(rw, vw + u * kWave, 0, 0);
                k.w[u] = P == kBF16 ? wv << 16 : wv;
            }
        };
        // the members' scales 2^F (fixed point): w_q * 2^F is then exact, as q_fx
        double inv_scale[G];
#pragma unroll
        for (int m = 0; m < G; m++) {
            const int ql = qb.g_member[g * G + m];
            inv_scale[m] = (FX && ql >= 0) ? 1.0 / qb.q_scale[ql] : 0.0;
        }
        // a chunk's postings into the tile of every member holding its term
        auto apply = [&](const Chunk& k) {
            auto add = [&](auto pred) {
                constexpr bool PRED = decltype(pred)::value;
                auto ok = [&](int u) { return !PRED || lane + u * kWave < k.n; };
#pragma unroll
                for (int m = 0; m < G; m++) {
                    const uint32_t wm = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.w[k.seg][m]);
                    if (wm == 0u) continue;
                    if constexpr (AF == kAccFx64) {
                        const double qd = (double)__uint_as_float(wm) * inv_scale[m];
                        unsigned long long* acc = reinterpret_cast<unsigned long long*>(lds) + m * TILE - lbase;
#pragma unroll
                        for (int u = 0; u < U; u++)
                            if (ok(u)) atomicAdd(acc + k.doc[u], fx_product(qd, k.w[u]));
                    } else if constexpr (AF == kAccFx32) {
                        const double qd = (double)__uint_as_float(wm) * inv_scale[m];
                        uint32_t* acc = lds + m * TILE - lbase;
#pragma unroll
                        for (int u = 0; u < U; u++)
                            if (ok(u)) atomicAdd(acc + k.doc[u], (uint32_t)fx_product(qd, k.w[u]));
                    } else {
                        const uint32_t q8v = wm;
                        uint32_t* acc = lds + m * TILE - lbase;
#pragma unroll
                        for (int u = 0; u < U; u++)
                            if (ok(u)) atomicAdd(acc + k.doc[u], __umul24(q8v, k.w[u]));
                    }
                }
            };
            if (k.n == CH) add(std::false_type());
            else add(std::true_type());
        };
        {
            int cc = wave;
            Chunk A, B;
            load(cc, A, cc < total);
            while (cc < total) {
                const int cb = cc + NW;
                load(cb, B, cb < total);
                apply(A);
                if (cb >= total) break;
                const int ca = cb + NW;
                load(ca, A, ca < total);
                apply(B);
                cc = ca;
            }
        }
        __syncthreads();
        // flush every member's tile (the histogram reuses the segment area)
        uint32_t* hist = sh.hist;
        for (int m = 0; m < G; m++) {
            const int ql = qb.g_member[g * G + m];
            if (ql < 0 || qb.k[ql] == 0) continue;  // uniform: read from global memory
            for (int i = tid; i < kHistLds; i += BS) hist[i] = 0u;
            __syncthreads();
            SelState* st = state + ql;
            const bool fused_q = phase == 2 && st->fused == 1;
            // as in score_tile: a fused query writes no row and counts no tile here; its
            // fallback (phase 3) or bf16 band pass (phase 5) scores these tiles again
            const uint32_t* tile_acc = lds + m * TILE * AW;
            const double scale = FX ? qb.q_scale[ql] : 1.0;
            if (!fused_q)
                flush_tile<BS, AF>(tile_acc, hist, tile_n, S + (int64_t)ql * ld + base, qb.first[ql], scale,
                                   hist1 + (int64_t)ql * kHistBins, st, true, phase != kPhaseRows);
            else if (!st->fused_over)
                flush_candidates<BS, AF, TILE>(tile_acc, tile_n, base, scale, st->bound, st, cand + (int64_t)ql * kCandCap,
                                               reinterpret_cast<unsigned long long*>(hist), kHistBins / 2);
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------ atomic --

// Exclusive prefix of posting chunks over the (query, term) pairs of a query tile.
__global__ __launch_bounds__(1024) void k_pair_prefix(DevIndex ix, DevBatch qb, int32_t q0, int32_t qt, int chunk,
                                                      int64_t* __restrict__ prefix, int32_t* __restrict__ pair_q) {
    __shared__ int64_t part[1024];
    const int tid = threadIdx.x;
    const int64_t a0 = qb.q_row_ptr[q0];
    const int64_t np = qb.q_row_ptr[q0 + qt] - a0;
    const int64_t per = (np + 1023) / 1024;
    const int64_t lo = min(np, tid * per), hi = min(np, lo + per);
    int64_t s = 0;
    for (int64_t p = lo; p < hi; p++) {
        const int term = qb.q_term[a0 + p];
        const int64_t padded = ix.term_off[term + 1] - ix.term_off[term];
        s += (padded + chunk - 1) / chunk;
    }
    part[tid] = s;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int64_t v = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t run = part[tid] - s;
    int ql = 0;
    for (int64_t p = lo; p < hi; p++) {
        while (qb.q_row_ptr[q0 + ql + 1] - a0 <= p) ql++;
        prefix[p] = run;
        pair_q[p] = ql;
        const int term = qb.q_term[a0 + p];
        const int64_t padded = ix.term_off[term + 1] - ix.term_off[term];
        run += (padded + chunk - 1) / chunk;
    }
    if (tid == 1023) prefix[np] = part[1023];
}

template <int P, int CH>
__global__ __launch_bounds__(256) void k_score_atomic(DevIndex ix, DevBatch qb, int32_t q0, int32_t qt,
                                                      const int64_t* __restrict__ prefix,
                                                      const int32_t* __restrict__ pair_q, uint32_t* __restrict__ S,
                                                      int64_t ld) {
    constexpr int NW = 256 / kWave, U = CH / kWave;
    using Acc = typename WF<P>::Acc;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t a0 = qb.q_row_ptr[q0];
    const int64_t np = qb.q_row_ptr[q0 + qt] - a0;
    const int64_t total = prefix[np];
    for (int64_t c = (int64_t)blockIdx.x * NW + (threadIdx.x >> 6); c < total; c += (int64_t)gridDim.x * NW) {
        int64_t lo = 0, hi = np - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (prefix[mid] <= c) lo = mid; else hi = mid - 1;
        }
        const int term = qb.q_term[a0 + lo];
        const Acc wq = WF<P>::qweight(qb, a0 + lo);
        const int64_t off = (c - prefix[lo]) * (int64_t)CH;
        const int64_t p0 = ix.term_off[term] + off;
        const int n = (int)min((int64_t)CH, ix.term_off[term + 1] - p0);  // a list ends on a 64-posting block
        uint32_t* Sq = S + (int64_t)pair_q[lo] * ld;
        int doc[U];
        Acc w[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int i = lane + u * kWave;
            doc[u] = -1;
            if (i < n) {
                doc[u] = ix.post_doc[p0 + i];
                w[u] = WF<P>::load(ix.post_w, p0 + i);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (doc[u] >= 0) glb_add(&Sq[doc[u]], wq * w[u]);
    }
}

// ------------------------------------------------------------ docpar --

// 1024 threads per (query, block of docs): the query's weights sit in a dense
// LDS table; a wavefront scores 4 documents at a time, 16 lanes per document,
// each lane walking its document's forward row with stride 16 and four loads
// of (term, weight) in flight, then a 16-lane reduction. Rows are contiguous,
// so the 4 x 16 lanes read 4 short coalesced runs per step. The table's size bounds the
// vocabulary far below 65,536 terms, so the rows' terms are always the 2-byte ones.
template <int P>
__global__ __launch_bounds__(1024) void k_score_docpar(DevIndex ix, DevBatch qb, int32_t q0, uint32_t* __restrict__ S,
                                                       int64_t ld, int docs_per_block) {
    using Acc = typename WF<P>::Acc;
    extern __shared__ __align__(16) uint32_t table[];  // [vocab] query weights (dense)
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int ql = blockIdx.y, q = q0 + ql;
    for (int i = tid; i < ix.vocab; i += 1024) table[i] = 0u;
    __syncthreads();
    const int64_t qa = qb.q_row_ptr[q], qn = qb.q_row_ptr[q + 1] - qa;
    for (int t = tid; t < qn; t += 1024) {
        Acc v = WF<P>::qweight(qb, qa + t);
        table[qb.q_term[qa + t]] = WF<P>::bits(v);
    }
    __syncthreads();
    if (qb.k[q] == 0) return;
    const Acc* tab = reinterpret_cast<const Acc*>(table);
    const int64_t d0 = (int64_t)blockIdx.x * docs_per_block;
    const int64_t d1 = min(ix.n_docs, d0 + docs_per_block);
    uint32_t* Sq = S + (int64_t)ql * ld;
    const int grp = lane >> 4, sub = lane & 15;
    for (int64_t dg = d0 + (int64_t)wave * 4; dg < d1; dg += 16 * 4) {
        const int64_t d = dg + grp;
        int64_t a = 0, b = 0;
        if (d < d1) {
            a = ix.fwd_row_ptr[d];
            b = ix.fwd_row_ptr[d + 1];
        }
        Acc s = 0;
        for (int64_t e = a + sub; e < b; e += 64) {
            int t[4];
            float w[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t eu = e + 16 * u;
                t[u] = eu < b ? ix.fwd_term16[eu] : 0;
                w[u] = eu < b ? ix.fwd_w[eu] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (e + 16 * u < b) s += tab[t[u]] * WF<P>::from_fp32(w[u]);
        }
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) s += __shfl_xor(s, o, kWave);
        if (sub == 0 && d < d1) Sq[d] = WF<P>::bits(s);
    }
}

// ------------------------------------------------------ hist / clear --

__global__ __launch_bounds__(512) void k_hist1(DevBatch qb, int32_t q0, int64_t N, const uint32_t* __restrict__ S,
                                               int64_t ld, int per_block, uint32_t* __restrict__ hist1,
                                               SelState* __restrict__ state) {
    __shared__ uint32_t hist[kHistLds];
    const int tid = threadIdx.x, ql = blockIdx.y;
    for (int i = tid; i < kHistLds; i += 512) hist[i] = 0u;
    __syncthreads();
    int zc = 0;  // zero scores
    const FirstDigit fd = qb.first[q0 + ql];
    const int64_t d0 = (int64_t)blockIdx.x * per_block, d1 = min(N, d0 + per_block);
    const uint32_t* Sq = S + (int64_t)ql * ld;
    for (int64_t d = d0 + tid; d < d1; d += 512) {
        atomicAdd(&hist[fd.low ? first_digit<true>(fd, Sq[d]) : first_digit<false>(fd, Sq[d])], 1u);
        zc += Sq[d] == 0u;
    }
    zc = wave_sum(zc);
    if ((tid & (kWave - 1)) == 0 && zc) atomicAdd(&hist[kHistBins], (uint32_t)zc);
    __syncthreads();
    for (int b = tid; b < kHistBins; b += 512)
        if (hist[b]) atomicAdd(&hist1[(int64_t)ql * kHistBins + b], hist[b]);
    if (tid == 0 && hist[kHistBins]) atomicAdd(&state[ql].zeros, (int)hist[kHistBins]);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Row blockIdx.y of the commonest terms: the stored weights of its posting list by document
// (the rows are zero before). A grain's postings lie in one 65536-document range. A grain's
// documents are stored so that the 16 bytes a thread of sum_rows loads (4, 8 or 16 weights) are
// fours of documents 2048 apart.
template <typename WT>
__global__ __launch_bounds__(256) void k_fill_rows(DevIndex ix, const int32_t* __restrict__ terms, int r0,
                                                   WT* __restrict__ rows) {
    constexpr int DPL = 16 / (int)sizeof(WT), B = 512 * DPL, G = 1 << kGrainShift;
    const int row = r0 + (int)blockIdx.y, term = terms[row];
    const int32_t* off = ix.tile_off + (int64_t)term * (ix.n_grains + 1);
    const int64_t p0 = ix.term_off[term];
    for (int64_t g = blockIdx.x; g < ix.n_grains; g += gridDim.x) {
        WT* to = rows + ((g * ix.n_rows + row) << kGrainShift);
        for (int i = off[g] + (int)threadIdx.x; i < off[g + 1]; i += 256) {
            const int d = ix.post_lo[p0 + i] & (G - 1), r = d & (B - 1);
            to[d - r + ((r & 2047) >> 2) * DPL + (r >> 11) * 4 + (r & 3)] = reinterpret_cast<const WT*>(ix.post_w)[p0 + i];
        }
    }
}

__global__ __launch_bounds__(256) void k_narrow(const int32_t* __restrict__ src, uint16_t* __restrict__ dst,
                                                int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        dst[i] = (uint16_t)src[i];
}

// The start of a search: its step counters, selection state and histograms, in one launch.
static_assert(sizeof(SelState) % 16 == 0, "cleared 16 bytes at a time");
__global__ __launch_bounds__(256) void k_clear(uint32_t* __restrict__ counters, uint4* __restrict__ state,
                                               int64_t n_state, uint4* __restrict__ h1, int64_t n1) {
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0 && threadIdx.x < kCounterWords) counters[threadIdx.x] = 0u;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_state + n1; i += (int64_t)gridDim.x * 256) {
        if (i < n_state) state[i] = z;
        else h1[i - n_state] = z;
    }
}

hipError_t fill_u32(void* p, int64_t n_words, hipStream_t s) { return launch_fill(p, n_words, 0u, s); }

template <typename F>
hipError_t by_precision(int p, F f) {
    switch (p) {
        case kFP32: return f(std::integral_constant<int, kFP32>());
        case kBF16: return f(std::integral_constant<int, kBF16>());
        case kU8: return f(std::integral_constant<int, kU8>());
    }
    return hipErrorInvalidValue;
}

// Dynamic LDS past the default limit, once per kernel.
hipError_t allow_lds(const void* kernel, size_t lds, const char* name) {
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) g_failed_launch = name;
    return e;
}

template <int P, int TS>
constexpr size_t tile_lds() {
    return (size_t)((1 << TS) * (acc_form<P>() == kAccFx64 ? 2 : 1) + kHistLds) * 4;
}

template <int P, int TS, int CH>
hipError_t launch_tiled_one(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                            const Workspace& ws, int64_t ld, hipStream_t s, int phase, int stride, int64_t n_tiles) {
    constexpr size_t lds = tile_lds<P, TS>();
    static const hipError_t attr =
        allow_lds((const void*)k_score_tiled<P, TS, CH>, lds, "hipFuncSetAttribute(k_score_tiled)");
    if (attr != hipSuccess) return attr;
    // an eighth of the items per XCD, padded to a rectangle of workgroups
    const int64_t per = (n_tiles * qt + 7) / 8, gx = std::min<int64_t>(per, 65536), gy = (per + gx - 1) / gx;
    const ScoreItem* items = o.whole ? qb.s_order : qb.s_item + q0;
    hipLaunchKernelGGL((k_score_tiled<P, TS, CH>), dim3((unsigned)(8 * gx), (unsigned)gy), dim3(512), lds, s, ix, items,
                       qb.s_term, qb.first, qb.q_scale, q0, qt, ws.scores, ld, ws.hist1,
                       phase, stride, ws.state, ws.cand);
    GS_CHECK_LAUNCH("k_score_tiled");
    return hipSuccess;
}

template <int P, int TS>
hipError_t launch_tiled(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                        const Workspace& ws, hipStream_t s, int phase) {
    const int stride = phase == 0 || phase == kPhaseRows ? 1 : o.seed_stride;
    const int64_t ld = score_ld(ix.n_docs);
    const int64_t n_tiles = phase_tiles(phase, stride, (ix.n_docs + (1 << TS) - 1) >> TS);
    if (n_tiles <= 0) return hipSuccess;
    constexpr size_t lds = tile_lds<P, TS>();
    if (phase == 3 || phase == 5) {
        static const hipError_t attr =
            allow_lds((const void*)k_score_listed<P, TS, kMaxChunk>, lds, "hipFuncSetAttribute(k_score_listed)");
        if (attr != hipSuccess) return attr;
        const dim3 grid((unsigned)n_tiles, (unsigned)listed_ways(n_tiles, qt));
        hipLaunchKernelGGL((k_score_listed<P, TS, kMaxChunk>), grid, dim3(512), lds, s, ix, qb, q0,
                           ws.scores, ld, ws.hist1, phase, stride, ws.state, ws.cand, (const uint32_t*)ws.counters,
                           (const int32_t*)ws.rescore_list);
        GS_CHECK_LAUNCH("k_score_listed");
        return hipSuccess;
    }
    // block-max pruning (non-seed tiles): the default tile and chunk of fp32 and uint8 only
    if constexpr ((P == kFP32 && TS == 13) || (P == kU8 && TS == 14)) {
        if (o.prune && phase == 2) {
            static const hipError_t attr =
                allow_lds((const void*)k_score_pruned<P, TS, kMaxChunk>, lds, "hipFuncSetAttribute(k_score_pruned)");
            if (attr != hipSuccess) return attr;
            hipLaunchKernelGGL((k_score_pruned<P, TS, kMaxChunk>), dim3((unsigned)n_tiles, (unsigned)qt), dim3(512), lds,
                               s, ix, qb, q0, ws.scores, ld, ws.hist1, phase, stride, ws.state, ws.cand);
            GS_CHECK_LAUNCH("k_score_pruned");
            return hipSuccess;
        }
    }
    switch (o.chunk) {  // the kernel reads rows of 256 postings: smaller chunks run as 256
        case 64:
        case 128:
        case 256: return launch_tiled_one<P, TS, 256>(ix, qb, q0, qt, o, ws, ld, s, phase, stride, n_tiles);
        case 512: return launch_tiled_one<P, TS, 512>(ix, qb, q0, qt, o, ws, ld, s, phase, stride, n_tiles);
        case 1024: return launch_tiled_one<P, TS, 1024>(ix, qb, q0, qt, o, ws, ld, s, phase, stride, n_tiles);
    }
    return hipErrorInvalidValue;
}

template <int P, int CH>
hipError_t launch_group_one(const DevIndex& ix, const DevBatch& qb, const Workspace& ws, int64_t ld, hipStream_t s,
                            int phase, int stride) {
    constexpr int TS = kGroupTileShift;
    const int64_t n_tiles = phase_tiles(phase, stride, (ix.n_docs + (1 << TS) - 1) >> TS);
    if (n_tiles <= 0) return hipSuccess;
    const size_t lds = (size_t)group_size<P>() * (1 << TS) * (acc_form<P>() == kAccFx64 ? 8 : 4);
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_score_group<P, CH>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr != hipSuccess) {
        g_failed_launch = "hipFuncSetAttribute(k_score_group)";
        return attr;
    }
    // resident workgroups (one per CU), a multiple of the 8 XCDs
    static const int grid = [&] {
        int dev = 0, per_cu = 0;
        hipDeviceProp_t p{};
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&p, dev) != hipSuccess) return 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)k_score_group<P, CH>,
                                                         group_size<P>() * kMaxQueryNnz, lds) !=
            hipSuccess)
            return 0;
        return std::max(8, (p.multiProcessorCount * std::max(per_cu, 1)) / 8 * 8);
    }();
    if (grid <= 0) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_score_group<P, CH>), dim3((unsigned)grid), dim3(group_size<P>() * kMaxQueryNnz), lds, s,
                       ix, qb, ws.counters,
                       ws.scores, ld, ws.hist1, phase, stride, ws.state, ws.cand);
    GS_CHECK_LAUNCH("k_score_group");
    return hipSuccess;
}

}  // namespace

// The launches of one weight form. A build may compile this file in parts (GS_SCORE_PART 0, 1
// and 2: one form each; 3: the rest): the kernels of the three forms take most of its time.
template <int P>
struct ScoreForm {
    static hipError_t tiled(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                            const Workspace& ws, hipStream_t s, int phase);
    static hipError_t group(const DevIndex& ix, const DevBatch& qb, const ScoreOpts& o, const Workspace& ws,
                            hipStream_t s, int phase);
    static hipError_t wide(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const Workspace& ws,
                           hipStream_t s);
};

#if !defined(GS_SCORE_PART) || GS_SCORE_PART != 3
template <int P>
hipError_t ScoreForm<P>::tiled(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                               const Workspace& ws, hipStream_t s, int phase) {
    switch (o.tile_shift) {
        case 13: return launch_tiled<P, 13>(ix, qb, q0, qt, o, ws, s, phase);
        case 14: return launch_tiled<P, 14>(ix, qb, q0, qt, o, ws, s, phase);
        case 15:
            if constexpr (acc_form<P>() != kAccFx64) return launch_tiled<P, 15>(ix, qb, q0, qt, o, ws, s, phase);
            return hipErrorInvalidValue;  // 32768 64-bit accumulators exceed one CU's LDS
    }
    return hipErrorInvalidValue;
}

template <int P>
hipError_t ScoreForm<P>::group(const DevIndex& ix, const DevBatch& qb, const ScoreOpts& o, const Workspace& ws,
                               hipStream_t s, int phase) {
    const int stride = phase == 0 || phase == kPhaseRows ? 1 : o.seed_stride;
    const int64_t ld = score_ld(ix.n_docs);
    switch (o.chunk) {
        case 256: return launch_group_one<P, 256>(ix, qb, ws, ld, s, phase, stride);
        case 512: return launch_group_one<P, 512>(ix, qb, ws, ld, s, phase, stride);
        case 1024: return launch_group_one<P, 1024>(ix, qb, ws, ld, s, phase, stride);
    }
    return hipErrorInvalidValue;
}

template <int P>
hipError_t ScoreForm<P>::wide(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const Workspace& ws,
                              hipStream_t s) {
    // 8192 docs of fp64 accumulators (64 KiB of LDS)
    constexpr int TS = 13, CH = 256;
    const int64_t n_tiles = (ix.n_docs + (1 << TS) - 1) >> TS;
    if (n_tiles <= 0) return hipSuccess;
    const size_t lds = (size_t)((1 << TS) * 2 + kHistLds) * 4;
    const int64_t ld = score_ld(ix.n_docs);
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_score_listed<P, TS, CH, true>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr != hipSuccess) {
        g_failed_launch = "hipFuncSetAttribute(k_score_listed, wide)";
        return attr;
    }
    const dim3 grid((unsigned)n_tiles, (unsigned)listed_ways(n_tiles, qt));
    hipLaunchKernelGGL((k_score_listed<P, TS, CH, true>), grid, dim3(512), lds, s, ix, qb, q0,
                       ws.scores, ld, ws.hist1, 4, 1, ws.state, ws.cand, (const uint32_t*)ws.counters,
                       (const int32_t*)ws.rescore_list);
    GS_CHECK_LAUNCH("k_score_listed (wide)");
    return hipSuccess;
}

#if !defined(GS_SCORE_PART) || GS_SCORE_PART == 2
template <>
hipError_t ScoreForm<kU8>::wide(const DevIndex&, const DevBatch&, int32_t, int32_t, const Workspace&, hipStream_t) {
    return hipSuccess;  // uint8 sums are exact
}
#endif
#endif

#if defined(GS_SCORE_PART) && GS_SCORE_PART < 3
template struct ScoreForm<GS_SCORE_PART>;
#else

hipError_t launch_fill(void* p, int64_t n_words, uint32_t v, hipStream_t s) {
    if (n_words <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n_words + 255) / 256, 8192);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)p, n_words, v);
    GS_CHECK_LAUNCH("k_fill_u32");
    return hipSuccess;
}

hipError_t launch_fill_rows(const DevIndex& ix, const int32_t* terms, void* rows, hipStream_t s) {
    if (ix.n_rows <= 0 || ix.n_docs <= 0) return hipSuccess;
    const int w = ix.precision == kFP32 ? 4 : ix.precision == kBF16 ? 2 : 1;
    const hipError_t e = fill_u32(rows, ((ix.n_grains * ix.n_rows) << kGrainShift) * w / 4, s);
    if (e != hipSuccess) return e;
    for (int32_t r0 = 0; r0 < ix.n_rows; r0 += 32768) {  // grid rows
        const dim3 grid((unsigned)std::min<int64_t>(ix.n_grains, 1024), (unsigned)std::min(ix.n_rows - r0, 32768));
        if (w == 4) hipLaunchKernelGGL(k_fill_rows<uint32_t>, grid, dim3(256), 0, s, ix, terms, r0, (uint32_t*)rows);
        else if (w == 2) hipLaunchKernelGGL(k_fill_rows<uint16_t>, grid, dim3(256), 0, s, ix, terms, r0, (uint16_t*)rows);
        else hipLaunchKernelGGL(k_fill_rows<uint8_t>, grid, dim3(256), 0, s, ix, terms, r0, (uint8_t*)rows);
        GS_CHECK_LAUNCH("k_fill_rows");
    }
    return hipSuccess;
}

hipError_t launch_narrow(const int32_t* src, uint16_t* dst, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_narrow, dim3((unsigned)blocks), dim3(256), 0, s, src, dst, n);
    GS_CHECK_LAUNCH("k_narrow");
    return hipSuccess;
}

hipError_t launch_clear(const Workspace& ws, int32_t qt, hipStream_t s) {
    const int64_t n_state = (int64_t)qt * (sizeof(SelState) / 16), n_hist = (int64_t)qt * (kHistBins / 4);
    const int64_t blocks = std::min<int64_t>((n_state + n_hist + 255) / 256, 2048);
    hipLaunchKernelGGL(k_clear, dim3((unsigned)blocks), dim3(256), 0, s, ws.counters, (uint4*)ws.state, n_state,
                       (uint4*)ws.hist1, n_hist);
    GS_CHECK_LAUNCH("k_clear");
    return hipSuccess;
}

hipError_t launch_score_tiled(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                              const Workspace& ws, hipStream_t s, int phase) {
    return by_precision(ix.precision, [&](auto pc) {
        return ScoreForm<decltype(pc)::value>::tiled(ix, qb, q0, qt, o, ws, s, phase);
    });
}

hipError_t launch_score_group(const DevIndex& ix, const DevBatch& qb, const ScoreOpts& o, const Workspace& ws,
                              hipStream_t s, int phase) {
    return by_precision(ix.precision, [&](auto pc) {
        return ScoreForm<decltype(pc)::value>::group(ix, qb, o, ws, s, phase);
    });
}

hipError_t launch_score_wide(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const Workspace& ws,
                             hipStream_t s) {
    return by_precision(ix.precision,
                        [&](auto pc) { return ScoreForm<decltype(pc)::value>::wide(ix, qb, q0, qt, ws, s); });
}

hipError_t launch_score_atomic(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                               const Workspace& ws, hipStream_t s) {
    const int64_t ld = score_ld(ix.n_docs);
    hipError_t e = fill_u32(ws.scores, (int64_t)qt * ld, s);
    if (e != hipSuccess) return e;
    int64_t* prefix = ws.work_prefix;
    int32_t* pair_q = ws.work_pair_q;
    hipLaunchKernelGGL(k_pair_prefix, dim3(1), dim3(1024), 0, s, ix, qb, q0, qt, o.chunk, prefix, pair_q);
    GS_CHECK_LAUNCH("k_pair_prefix");
    const dim3 grid(2048);
    e = by_precision(ix.precision, [&](auto pc) -> hipError_t {
        constexpr int P = decltype(pc)::value;
        switch (o.chunk) {
            case 64: hipLaunchKernelGGL((k_score_atomic<P, 64>), grid, dim3(256), 0, s, ix, qb, q0, qt, prefix, pair_q, ws.scores, ld); break;
            case 128: hipLaunchKernelGGL((k_score_atomic<P, 128>), grid, dim3(256), 0, s, ix, qb, q0, qt, prefix, pair_q, ws.scores, ld); break;
            case 256: hipLaunchKernelGGL((k_score_atomic<P, 256>), grid, dim3(256), 0, s, ix, qb, q0, qt, prefix, pair_q, ws.scores, ld); break;
            case 512: hipLaunchKernelGGL((k_score_atomic<P, 512>), grid, dim3(256), 0, s, ix, qb, q0, qt, prefix, pair_q, ws.scores, ld); break;
            case 1024: hipLaunchKernelGGL((k_score_atomic<P, 1024>), grid, dim3(256), 0, s, ix, qb, q0, qt, prefix, pair_q, ws.scores, ld); break;
            default: return hipErrorInvalidValue;
        }
        GS_CHECK_LAUNCH("k_score_atomic");
        return hipSuccess;
    });
    if (e != hipSuccess) return e;
    return launch_hist1(ix, qb, q0, qt, ws, s);
}

hipError_t launch_score_docpar(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const ScoreOpts& o,
                               const Workspace& ws, hipStream_t s) {
    (void)o;
    const int64_t ld = score_ld(ix.n_docs);
    const int per = 4096;
    const dim3 grid((unsigned)((ix.n_docs + per - 1) / per), (unsigned)qt);
    const size_t lds = (size_t)ix.vocab * 4;
    if (lds > 160 * 1024) return hipErrorInvalidValue;  // dense query table must fit one CU's LDS
    hipError_t e = by_precision(ix.precision, [&](auto pc) -> hipError_t {
        constexpr int P = decltype(pc)::value;
        if (lds > 65536) {
            const hipError_t a = hipFuncSetAttribute((const void*)k_score_docpar<P>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (a != hipSuccess) return a;
        }
        hipLaunchKernelGGL((k_score_docpar<P>), grid, dim3(1024), lds, s, ix, qb, q0, ws.scores, ld, per);
        GS_CHECK_LAUNCH("k_score_docpar");
        return hipSuccess;
    });
    if (e != hipSuccess) return e;
    return launch_hist1(ix, qb, q0, qt, ws, s);
}

hipError_t launch_hist1(const DevIndex& ix, const DevBatch& qb, int32_t q0, int32_t qt, const Workspace& ws,
                        hipStream_t s) {
    const int64_t ld = score_ld(ix.n_docs);
    const int per = 65536;
    const dim3 grid((unsigned)((ix.n_docs + per - 1) / per), (unsigned)qt);
    hipLaunchKernelGGL(k_hist1, grid, dim3(512), 0, s, qb, q0, ix.n_docs, (const uint32_t*)ws.scores, ld, per,
                       ws.hist1, ws.state);
    GS_CHECK_LAUNCH("k_hist1");
    return hipSuccess;
}

#endif  // GS_SCORE_PART < 3

}  // namespace gs
