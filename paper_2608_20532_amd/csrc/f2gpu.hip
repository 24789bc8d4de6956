// f2gpu.hip -- MI355X (gfx950) kernels and C ABI of the GF(2) affine-map learner.
//
// Fit (Sec. 2.2): every context is an independent streaming Gaussian
// elimination over GF(2) on augmented rows [phi | y] (Eq. 5).  Rows are taken
// in stream order in blocks of 64, one row per lane of a 64-wide wavefront:
//   1. block reduce: every row of the block is reduced against the retained
//      basis.  The basis is kept fully reduced (each pivot column is set only
//      in its own row), so the row's own bits at the pivot columns select the
//      basis rows to add, in one pass;
//   2. in-block elimination in stream order: a wavefront ballot finds the
//      earliest row with a nonzero feature residual; the rows before it are
//      redundant or contradictory (zero features, nonzero output: Eq. 8) and
//      are classified together; the earliest nonzero row gives the new pivot
//      (its highest-priority feature bit), is broadcast to the later rows that
//      hold that bit and to the retained rows that hold it (back-substitution
//      keeps the basis fully reduced), and is inserted.
// A plan kernel validates the contexts and sorts them into classes by feature
// words and length, each class list in decreasing order of estimated work.
// Contexts of up to 8 words keep a pivot-indexed basis in LDS: short ones of up to 4
// words are fitted by one wavefront each, the others by four together, which
// reduce four blocks at once; as far as one can hide behind the other they run side by
// side in one kernel, else the second kind in a kernel behind it.  Wider contexts take up
// to eight workgroups each, with the basis in HBM and the rows it needs staged in LDS.
//
// Encode (Sec. 2.3): T(phi) is the XOR of the canonical map columns over the
// set bits of phi = [x | 1]; the support test checks phi against the
// parity-check rows of the free (non-pivot) columns, which the fit writes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <stdlib.h>

#include <atomic>
#include <type_traits>

#include "../../include/f2gpu.h"

namespace {

constexpr int kSmallWaves = 8;  // small-batch fit
constexpr int kSmallThreads = 64 * kSmallWaves;
constexpr int kEncThreads = 256;

struct FitArgs {
    const uint64_t* rows;
    int64_t rows_words;
    const int64_t* row_off;
    int32_t num_ctx;
    const int32_t* n_bits;
    const int64_t* basis_off;
    const int64_t* piv_off;
    const int64_t* map_off;
    int64_t basis_words, piv_entries, map_words;
    uint64_t* basis;
    int32_t* pivots;
    uint64_t* maps;
    uint64_t* tables;
    int32_t* rank;
    uint32_t* ctx_flags;
    int32_t* n_contra;
    int64_t* first_contra;
    int32_t* plan;  // workspace: class list offsets, group barrier counters, context lists (k_fit_plan)
    int32_t coop;   // the wide kernel runs as a cooperative launch (all workgroups resident)
    int32_t max_n;  // host hint: largest width of the batch, -1 if unknown
    int32_t spin_limit;  // polls of a group barrier before it gives up (0: never wait)
};

struct EncArgs {
    int32_t num_ctx;
    const int32_t* n_bits;
    const int64_t* basis_off;
    const int64_t* piv_off;
    const uint64_t* basis;
    const int32_t* pivots;
    const int32_t* rank;
    const uint32_t* ctx_flags;
    const int64_t* map_off;
    const uint64_t* maps;
    const uint64_t* tables;  // parity-check rows, context c at basis_off[c]
    const int32_t* ctx_id;
    const uint64_t* x;
    int32_t stride;
    int32_t x16;  // x is 16-byte aligned (then even strides allow 16-byte loads of a query)
    int32_t wide; // contexts of more than kLaneFW feature words may occur (by the declared width bound)
    int64_t nq;
    uint64_t* words;
    uint8_t* qflags;
};

constexpr uint32_t kBadCtx = F2_CTX_BAD_SEGMENT | F2_CTX_BAD_WIDTH | F2_CTX_BAD_OUTPUT | F2_CTX_SYNC_TIMEOUT;

__host__ __device__ __forceinline__ int feat_words(int n) { return (n + 64) >> 6; }

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), lane);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src_lane) {
    const int lo = __builtin_amdgcn_ds_bpermute(src_lane << 2, static_cast<int>(static_cast<uint32_t>(v)));
    const int hi = __builtin_amdgcn_ds_bpermute(src_lane << 2, static_cast<int>(static_cast<uint32_t>(v >> 32)));
    return (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo);
}

__device__ __forceinline__ int ffs64(uint64_t v) { return __ffsll(static_cast<unsigned long long>(v)) - 1; }
__device__ __forceinline__ int msb64(uint64_t v) { return 63 - __clzll(static_cast<long long>(v)); }

// valid bits of the last feature word
__device__ __forceinline__ uint64_t top_mask(int n, int fw) {
    const int vb = n + 1 - 64 * (fw - 1);
    return vb >= 64 ? ~0ull : ((1ull << vb) - 1);
}

// ---------------------------------------------------------------------------
// context descriptor: width, row segment and the checks of its offsets against
// the buffer sizes (an invalid context is flagged and left at rank 0)
// ---------------------------------------------------------------------------
struct CtxDesc {
    int c, n;
    uint32_t bad;
    int64_t row0, m;
    int64_t bo, po, mo;  // output offsets: basis (and parity rows), pivots, map
};

__device__ __forceinline__ CtxDesc load_desc(const FitArgs& a, int64_t c) {
    CtxDesc ds{-1, -1, 0u, 0, 0, 0, 0, 0};  // c = -1: no context
    if (c >= a.num_ctx) return ds;
    ds.c = static_cast<int>(c);
    // every load first (one memory latency), then the checks in order
    const int n = a.n_bits[c];
    const int64_t bo = a.basis_off[c], po = a.piv_off[c], mo = a.map_off[c];
    const int64_t s0 = a.row_off[c], s1 = a.row_off[c + 1];
    ds.n = n;
    ds.bo = bo;
    ds.po = po;
    ds.mo = mo;
    if (n < 0 || n > F2_MAX_N_BITS || (a.max_n >= 0 && n > a.max_n)) {  // outside the supported or declared range
        ds.bad = F2_CTX_BAD_WIDTH;
        return ds;
    }
    const int d = n + 1;
    const int W = feat_words(n) + F2_Y_WORDS;
    if (bo < 0 || bo + static_cast<int64_t>(d) * W > a.basis_words || po < 0 || po + d > a.piv_entries || mo < 0 ||
        mo + 2 * static_cast<int64_t>(d) > a.map_words) {
        ds.bad = F2_CTX_BAD_OUTPUT;
        return ds;
    }
    if (s0 < 0 || s1 < s0 || s1 > a.rows_words || (s1 - s0) % W != 0) {
        ds.bad = F2_CTX_BAD_SEGMENT;
        return ds;
    }
    ds.row0 = s0;
    ds.m = (s1 - s0) / W;
    return ds;
}

__device__ __forceinline__ CtxDesc readlane_desc(const CtxDesc& v, int t) {
    CtxDesc ds;
    ds.c = __builtin_amdgcn_readlane(v.c, t);
    ds.n = __builtin_amdgcn_readlane(v.n, t);
    ds.bad = __builtin_amdgcn_readlane(v.bad, t);
    ds.row0 = static_cast<int64_t>(readlane64(static_cast<uint64_t>(v.row0), t));
    ds.m = static_cast<int64_t>(readlane64(static_cast<uint64_t>(v.m), t));
    ds.bo = static_cast<int64_t>(readlane64(static_cast<uint64_t>(v.bo), t));
    ds.po = static_cast<int64_t>(readlane64(static_cast<uint64_t>(v.po), t));
    ds.mo = static_cast<int64_t>(readlane64(static_cast<uint64_t>(v.mo), t));
    return ds;
}

// outputs of an invalid context (one thread)
__device__ __forceinline__ void write_bad_context(const FitArgs& a, const CtxDesc& ds) {
    a.rank[ds.c] = 0;
    a.n_contra[ds.c] = 0;
    a.first_contra[ds.c] = -1;
    a.ctx_flags[ds.c] = ds.bad;
    if (ds.bad == F2_CTX_BAD_SEGMENT) {
        const int64_t mo = a.map_off[ds.c];
        for (int j = 0; j < 2 * (ds.n + 1); ++j) a.maps[mo + j] = 0;
    }
}

// ---------------------------------------------------------------------------
// fit plan.  Contexts are validated (an invalid one gets rank 0 and its flag
// here), assigned to the kernel of their class, and each class list is sorted
// by an estimate of the elimination work, largest first:
//   short:    fw <= 3 and few rows, or rows x columns small  -> one wavefront
//   long:     fw <= 3, rows x columns moderate               -> kPivWaves wavefronts, or one beside
//             many short ones
//   one long: fw = 4, likewise                               -> kPivWaves wavefronts, or one with a
//             larger basis
//   one:      fw = 4, few rows                               -> one wavefront with a larger basis
//   group:    fw <= 8, whatever is longer or wider           -> kPivWaves wavefronts
//   large:    fw > 8                                         -> large-context kernel
// (which kernel takes the middle four depends on their numbers: piv_lists)
// A class kernel with G workgroups deals its list out in stripes of G entries,
// alternating direction from stripe to stripe, so that every workgroup gets a
// similar share of the work and the longest contexts start first.  The sort is
// a counting sort over (class, cost bucket) bins in two kernels (per-block
// histograms; a scatter that scans them) with no device-wide atomics: on a chip
// of eight dies those serialise far from the compute units.
// Workspace (int32): [0, kNumCls] list offsets per class, [kPivNext] the work counter
// of the LDS-basis kernel, [kBarHead, kPlanHead) progress of the wide kernel's
// workgroups, [kPlanHead, kPlanHead + C) the lists, then C sort keys and a
// kPlanBins histogram per plan block.
// ---------------------------------------------------------------------------
constexpr int kRegMaxFW = 3;
constexpr int kPivMaxFW = 8;
constexpr int kLongRows = 4096;  // contexts with more rows are the work of several wavefronts
// One wavefront's time grows with rows x columns (each block of 64 rows is reduced against up to
// `columns` records).  Up to kShortRows rows or kShortWork it is the better path in any batch
// (8,000 contexts of 300 rows, 41 columns: 114 us, by four wavefronts 190; 20 among 100 small
// ones, 181 columns of rank 126: of 300 rows 70 and 75 us, 350 78 and 85, 400 85 and 75, 570 100
// and 94; 121 columns: 38 and 37, 42 and 36, 45 and 42, 52 and 48; 31 columns, 570 rows: 20 and
// 18, 800 rows 24 and 20); up to kLongWork it
// ends before a large batch of short contexts does (80,000 contexts of a corpus, 353 us with the
// line at 65,536, 213 us at 131,072 and 275 us at 262,144, where the longest end last).
constexpr int kShortRows = 320, kShortWork = 20480, kLongWork = 131072;
enum { kClsShort = 0, kClsLong = 1, kClsOneLong = 2, kClsOne = 3, kClsGroup = 4, kClsLarge = 5, kNumCls = 6 };
constexpr int kPivNext = 8;                 // plan word: next list position for the LDS-basis kernel
constexpr int kRegNext = 9;                 // and for the shared tail of the one-wavefront kernel's list
constexpr int kBarHead = 16;                // plan words kBarHead ..: progress of the wide kernel's workgroups
constexpr int kMaxMembers = 256;
constexpr int kPlanHead = kBarHead + kMaxMembers;
constexpr int kBuckets = 170;
constexpr int kPlanBins = 1024;
constexpr int kPlanThreads = 1024;  // one context per thread; one bin per thread in the scan
static_assert(kNumCls * kBuckets <= kPlanBins && kPlanBins == kPlanThreads, "the scan gives one bin to each thread");

__device__ __forceinline__ int fit_class(const CtxDesc& ds, int long_rows = kLongRows) {
    const int fw = feat_words(ds.n);
    if (fw > kPivMaxFW) return kClsLarge;
    const int64_t work = ds.m > kShortRows ? ds.m * (ds.n + 1) : 0;  // (m is at most 2^60)
    if (ds.m > long_rows || fw > kRegMaxFW + 1 || work > kLongWork) return kClsGroup;
    if (fw == kRegMaxFW + 1) return ds.m > kShortRows ? kClsOneLong : kClsOne;
    return work > kShortWork ? kClsLong : kClsShort;
}

// log-scale bucket (4 per octave) of rows x min(rows, d) x row words
__device__ __forceinline__ int cost_bucket(const CtxDesc& ds) {
    const uint64_t d = static_cast<uint64_t>(ds.n) + 1, W = static_cast<uint64_t>(feat_words(ds.n)) + F2_Y_WORDS;
    const uint64_t m = ds.m < (1ll << 32) ? static_cast<uint64_t>(ds.m) : (1ull << 32);
    const uint64_t cost = m * (m < d ? m : d) * W + 1;
    const int e = 63 - __clzll(static_cast<long long>(cost));
    const int frac = e >= 2 ? static_cast<int>((cost >> (e - 2)) & 3) : 0;
    const int b = 4 * e + frac;
    return b < kBuckets ? b : kBuckets - 1;
}

struct PlanView {
    int32_t* cls_off;  // [kNumCls + 1]
    int32_t* order;    // [C]
    int32_t* key;      // [C]
    int32_t* hist;     // [blocks][kPlanBins]
};

__device__ __forceinline__ PlanView plan_view(const FitArgs& a) {
    PlanView v;
    v.cls_off = a.plan;
    v.order = a.plan + kPlanHead;
    v.key = v.order + a.num_ctx;
    v.hist = v.key + a.num_ctx;
    return v;
}

// what the fit kernels count in, and where they meet
__device__ __forceinline__ void plan_clear(const FitArgs& a) {
    const int tid = threadIdx.x;
    if (tid < kMaxMembers) a.plan[kBarHead + tid] = 0;
    if (tid < 2) a.plan[kPivNext + tid] = 0;
}

// a context's bin, or -1 and its outputs written where it is invalid
__device__ __forceinline__ int plan_bin(const FitArgs& a, const CtxDesc& ds) {
    if (ds.bad) {
        write_bad_context(a, ds);
        return -1;
    }
    const int cls = fit_class(ds);
    if (cls == kClsLarge) {  // the workgroups of a wide context add their counts and flags, and share a list
        a.ctx_flags[ds.c] = 0u;
        a.n_contra[ds.c] = 0;
        a.first_contra[ds.c] = -1;
        a.pivots[ds.po] = 0;
    }
    return cls * kBuckets + (kBuckets - 1 - cost_bucket(ds));
}

// exclusive scan of one bin per thread (sWave: a word per wavefront)
__device__ __forceinline__ int plan_scan(int total, int* sWave) {
    const int tid = threadIdx.x, lane = tid & 63;
    int x = total;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    if (lane == 63) sWave[tid >> 6] = x;
    __syncthreads();
    int base = 0;
    for (int w = 0; w < (tid >> 6); ++w) base += sWave[w];
    return base + x - total;
}
__device__ __forceinline__ void plan_offsets(const PlanView& P, int excl, int total) {
    const int tid = threadIdx.x;
    if (tid % kBuckets == 0 && tid < kNumCls * kBuckets) P.cls_off[tid / kBuckets] = excl;
    if (tid == kPlanThreads - 1) P.cls_off[kNumCls] = excl + total;
}

// the plan of up to kPlanThreads contexts, one per thread, in one launch (a fit of 1,000
// contexts: 41.9 us, with the two kernels below 45.4 us; four contexts per thread took 12 us on
// 4,096, the two kernels 9.6 us)
__global__ __launch_bounds__(kPlanThreads) void k_plan_one(FitArgs a) {
    __shared__ int sBin[kPlanBins];
    __shared__ int sWave[kPlanThreads / 64];
    const PlanView P = plan_view(a);
    const int tid = threadIdx.x;
    sBin[tid] = 0;
    plan_clear(a);
    const CtxDesc ds = load_desc(a, tid);  // (c = -1 past the end)
    __syncthreads();
    const int key = ds.c < 0 ? -1 : plan_bin(a, ds);
    if (key >= 0) atomicAdd(&sBin[key], 1);
    __syncthreads();
    const int total = sBin[tid];
    const int excl = plan_scan(total, sWave);
    plan_offsets(P, excl, total);
    sBin[tid] = excl;
    __syncthreads();
    if (key >= 0) P.order[atomicAdd(&sBin[key], 1)] = ds.c;
}

// (1) per context: validate, class and bin; per block: histogram of the bins
__global__ __launch_bounds__(kPlanThreads) void k_plan_count(FitArgs a) {
    __shared__ int sBin[kPlanBins];
    const PlanView P = plan_view(a);
    const int tid = threadIdx.x;
    sBin[tid] = 0;
    __syncthreads();
    if (blockIdx.x == 0) plan_clear(a);
    const int64_t c = static_cast<int64_t>(blockIdx.x) * kPlanThreads + tid;
    if (c < a.num_ctx) {
        const int k = plan_bin(a, load_desc(a, c));
        if (k >= 0) atomicAdd(&sBin[k], 1);
        P.key[c] = k;
    }
    __syncthreads();
    P.hist[static_cast<int64_t>(blockIdx.x) * kPlanBins + tid] = sBin[tid];
}

// (2) scatter.  Thread b of every block sums bin b over all blocks (its total) and
// over the blocks before this one; a block scan of the totals gives the bin bases.
// List position = bin base + earlier blocks' count + rank within the block.
__global__ __launch_bounds__(kPlanThreads) void k_plan_scatter(FitArgs a, int blocks) {
    __shared__ int sBin[kPlanBins];
    __shared__ int sWave[kPlanThreads / 64];
    const PlanView P = plan_view(a);
    const int tid = threadIdx.x;
    const int g0 = static_cast<int>(blockIdx.x);
    int total = 0, before = 0;
    constexpr int U = 32;  // loads in flight (79 blocks: 8.4 us; 9.0 us with 8)
    for (int g = 0; g < blocks; g += U) {
        int v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = g + k < blocks ? P.hist[static_cast<int64_t>(g + k) * kPlanBins + tid] : 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            before += g + k < g0 ? v[k] : 0;
            total += v[k];
        }
    }
    const int excl = plan_scan(total, sWave);
    if (g0 == 0) plan_offsets(P, excl, total);
    sBin[tid] = excl + before;
    __syncthreads();
    const int64_t c = static_cast<int64_t>(g0) * kPlanThreads + tid;
    if (c < a.num_ctx) {
        const int k = P.key[c];
        if (k >= 0) P.order[atomicAdd(&sBin[k], 1)] = static_cast<int32_t>(c);
    }
}

// ---------------------------------------------------------------------------
// parity-check rows, written by every fit kernel next to the canonical map:
// for the i-th free (non-pivot) column f in ascending order, row i (fw words,
// at the context's basis offset in the tables buffer) is h_f = e_f plus e_p for
// every pivot p whose basis row holds bit f.  Since the basis is fully reduced,
// the residual of reducing phi at column f is the parity of phi & h_f, so phi
// lies in the span exactly when every row has even overlap with it.  Word w of
// h_f is one ballot: lane b tests bit f of the basis row of pivot 64 w + b.
// The rows exist only when t = d - rank <= rank; a context with more free
// columns than basis rows is encoded by reducing phi with the basis itself.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool has_parity_rows(int d, int rank) { return d - rank <= rank; }
// orders a wavefront's own LDS accesses: used where a wavefront works alone on
// its LDS region, so that no workgroup barrier couples it to the others
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// one-wavefront fit (fw <= 4): the rows pass through in blocks of 64, one row per
// lane; the basis row of pivot p lies in LDS record p (fw feature words, 2 output
// words), the basis fully reduced at the end of every block.  (Basis rows kept in
// registers where they stood took every later pivot's step once per earlier block and held
// contexts to 256 rows.)
// ---------------------------------------------------------------------------
template <int FW>
__device__ __forceinline__ uint64_t word_at(const uint64_t (&f)[FW], int wi) {
    // word wi (uniform), by masks: a chain of selects becomes an indexed load, and f an array in scratch
    uint64_t v = f[0];
#pragma unroll
    for (int k = 1; k < FW; ++k) v ^= (f[0] ^ f[k]) & (0ull - static_cast<uint64_t>(wi == k));
    return v;
}

// all-ones when bit b of w is set, else zero (32-bit: one mask serves both halves)
__device__ __forceinline__ uint32_t bit_mask(uint64_t w, int b) {
    const uint32_t dw = (b & 32) ? static_cast<uint32_t>(w >> 32) : static_cast<uint32_t>(w);
    return static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(dw), b & 31, 1));  // sign of a 1-bit field
}

// 64 x 64 bit-matrix transpose across a wavefront: lane b holds row b; returned,
// lane f holds bit f of every row (bit b of the result = bit f of row b).  Six
// rounds that swap the off-diagonal blocks of size 32, 16, .., 1 with the partner
// lane (lane xor j).
// (All in registers: a swap of the halves between lanes 32 apart, then per half a row
// swap, DPP moves, and byte permutes or a rotate and a bit select.  About 35 VALU
// instructions; rounds of ds_bpermute took 70 and 12 LDS permutes.)
__device__ __forceinline__ uint32_t transpose32(uint32_t x, int lane) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);  // [0] even rows' values, [1] odd rows'
    x = __builtin_amdgcn_perm(r[1], r[0], (lane & 16) ? 0x07060302u : 0x05040100u);
    uint32_t p = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), 0x128, 0xf, 0xf, true));  // lane ^ 8
    x = __builtin_amdgcn_perm(p, x, (lane & 8) ? 0x03070105u : 0x06020400u);
    p = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), 0x141, 0xf, 0xf, true));           // lane ^ 7
    p = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(p), 0x1b, 0xf, 0xf, true));            // and ^ 3
    const auto mix = [](uint32_t x, uint32_t p, uint32_t rot, uint32_t m) {  // bits m from p rotated right
        p = __builtin_amdgcn_alignbit(p, p, rot);
        return (p & m) | (x & ~m);
    };
    x = mix(x, p, (lane & 4) ? 4u : 28u, (lane & 4) ? 0x0f0f0f0fu : 0xf0f0f0f0u);
    p = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), 0x4e, 0xf, 0xf, true));            // lane ^ 2
    x = mix(x, p, (lane & 2) ? 2u : 30u, (lane & 2) ? 0x33333333u : 0xccccccccu);
    p = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), 0xb1, 0xf, 0xf, true));            // lane ^ 1
    return mix(x, p, (lane & 1) ? 1u : 31u, (lane & 1) ? 0x55555555u : 0xaaaaaaaau);
}
__device__ __forceinline__ uint64_t transpose64(uint64_t v, int lane) {
    const auto r = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(v), static_cast<uint32_t>(v >> 32), false, false);
    return (static_cast<uint64_t>(transpose32(r[1], lane)) << 32) | transpose32(r[0], lane);
}

// f ^ (m & d) with m a 32-bit all-ones/zero mask: one v_bitop3 per half
__device__ __forceinline__ uint64_t xor_and(uint64_t f, uint32_t m, uint64_t d) {
    const uint32_t lo = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(f), m, static_cast<uint32_t>(d), 0x78);
    const uint32_t hi =
        __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(f >> 32), m, static_cast<uint32_t>(d >> 32), 0x78);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// a ^ b ^ c: one v_bitop3 per half
__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
    const uint32_t lo = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(a), static_cast<uint32_t>(b),
                                                    static_cast<uint32_t>(c), 0x96);
    const uint32_t hi = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(a >> 32), static_cast<uint32_t>(b >> 32),
                                                    static_cast<uint32_t>(c >> 32), 0x96);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

struct RegRows {  // row words of a block in flight, per lane
    uint64_t w0, w1, w2, w3, w4, w5;  // (named: an array handed through calls ends in scratch memory)
    __device__ __forceinline__ uint64_t word(int w) const {
        return w == 0 ? w0 : w == 1 ? w1 : w == 2 ? w2 : w == 3 ? w3 : w == 4 ? w4 : w5;
    }
};
constexpr int reg_words(int fw) { return 64 * fw * (fw + F2_Y_WORDS); }  // LDS words of a wavefront's basis
constexpr int kRegRec = reg_words(kRegMaxFW);

// 8-byte aligned words, moved 16 bytes at a time at a 32-bit offset from a uniform base
typedef unsigned long long u64x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
template <int W>
__device__ __forceinline__ void load_words(const uint64_t* base, uint32_t bytes, uint64_t (&v)[W]) {
    const char* p = reinterpret_cast<const char*>(base) + bytes;
#pragma unroll
    for (int w = 0; w + 1 < W; w += 2) {
        const u64x2_a8 q = *reinterpret_cast<const u64x2_a8*>(p + 8 * w);
        v[w] = q.x;
        v[w + 1] = q.y;
    }
    if constexpr (W & 1) v[W - 1] = *reinterpret_cast<const uint64_t*>(p + 8 * (W - 1));
}
template <int W>
__device__ __forceinline__ void store_words(uint64_t* base, uint32_t bytes, const uint64_t (&v)[W]) {
    char* p = reinterpret_cast<char*>(base) + bytes;
#pragma unroll
    for (int w = 0; w + 1 < W; w += 2) *reinterpret_cast<u64x2_a8*>(p + 8 * w) = u64x2_a8{v[w], v[w + 1]};
    if constexpr (W & 1) *reinterpret_cast<uint64_t*>(p + 8 * (W - 1)) = v[W - 1];
}

// the 64 rows from i0 on, one per lane (zero past row m <= kLongRows): W words each
template <int W>
__device__ __forceinline__ RegRows load_rows(const uint64_t* R, int m, int i0) {
    const int i = i0 + static_cast<int>(threadIdx.x & 63);
    RegRows r{0, 0, 0, 0, 0, 0};
    if (i < m) {
        uint64_t v[W];
        load_words<W>(R, static_cast<uint32_t>(i) * (8 * W), v);
        r.w0 = v[0];
        r.w1 = v[1];
        r.w2 = v[2];
        if constexpr (W > 3) r.w3 = v[3];
        if constexpr (W > 4) r.w4 = v[4];
        if constexpr (W > 5) r.w5 = v[5];
    }
    return r;
}

// feature words of a context: of its only word just the low half where NARROW (at most 31
// inputs); every high half is then a known zero and takes no instruction
template <bool NARROW>
__device__ __forceinline__ uint64_t feat_xor_and(uint64_t f, uint32_t m, uint64_t d) {
    if constexpr (NARROW)
        return static_cast<uint32_t>(__builtin_amdgcn_bitop3_b32(static_cast<int>(static_cast<uint32_t>(f)), static_cast<int>(m),
                                                                 static_cast<int>(static_cast<uint32_t>(d)), 0x78));
    else
        return xor_and(f, m, d);
}
template <bool NARROW>
__device__ __forceinline__ uint64_t feat_readlane(uint64_t f, int j) {
    if constexpr (NARROW) return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(f), j));
    else return readlane64(f, j);
}
template <bool NARROW>
__device__ __forceinline__ uint32_t feat_mask(uint64_t f, int b) {
    if constexpr (NARROW) return static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(static_cast<uint32_t>(f)), b, 1));
    else return bit_mask(f, b);
}

// elimination in stream order of a block of 64 rows, one per lane (those of `pending`): the
// earliest row with a nonzero feature residual becomes a basis row where it stands, and its
// pivot is cleared from every other row, so that the new rows end fully reduced among
// themselves; the others end with zero features.  newp: the new pivots.  Bound by a
// pivot's chain (ballot, row to scalar registers, first set bit, mask, additions, ballot).
template <int FW, bool NARROW = false>
__device__ __forceinline__ void eliminate_block(uint64_t (&f)[FW], uint64_t& y0, uint64_t& y1, uint64_t pending, int n,
                                                const uint64_t (&xm)[FW], uint64_t (&newp)[FW]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int w = 0; w < FW; ++w) newp[w] = 0;
    const auto nonzero = [&]() {
        uint64_t any = f[0];
#pragma unroll
        for (int w = 1; w < FW; ++w) any |= f[w];
        return __ballot(any != 0) & pending;
    };
    uint64_t nz = nonzero();
    while (nz) {
        const int j = ffs64(nz);
        uint64_t F[FW];
#pragma unroll
        for (int w = 0; w < FW; ++w) F[w] = feat_readlane<NARROW>(f[w], j);
        const uint64_t Y0 = readlane64(y0, j), Y1 = readlane64(y1, j);
        // pivot: highest-priority set feature bit (x_{n-1} .. x_0, else the
        // constant: the row is nonzero)
        int pw = FW == 1 ? 0 : n >> 6, pb = n & 63;
#pragma unroll
        for (int w = 0; w < FW; ++w) {
            const uint64_t v = F[w] & xm[w];
            // (undefined for zero, where it is not taken)
            const int b = NARROW ? 31 ^ __builtin_clz(static_cast<uint32_t>(v)) : 63 ^ __builtin_clzll(v);
            pb = v ? b : pb;
            if (FW > 1) pw = v ? w : pw;
        }
        const uint32_t mb = feat_mask<NARROW>(word_at<FW>(f, pw), pb);
        const uint32_t mm = lane == j ? 0u : mb;
#pragma unroll
        for (int w = 0; w < FW; ++w) f[w] = feat_xor_and<NARROW>(f[w], mm, F[w]);
        y0 = xor_and(y0, mm, Y0);
        y1 = xor_and(y1, mm, Y1);
#pragma unroll
        for (int w = 0; w < FW; ++w) newp[w] |= FW == 1 || w == pw ? 1ull << pb : 0ull;
        pending &= ~(1ull << j);
        nz = nonzero();
    }
}

// first set bit of a row (in pivot order), where it has one: a new basis row's pivot
template <int FW>
__device__ __forceinline__ int row_pivot(const uint64_t (&f)[FW], const uint64_t (&xm)[FW], int n) {
    int p = n;
#pragma unroll
    for (int w = 0; w < FW; ++w) {
        const uint64_t v = f[w] & xm[w];
        p = v ? 64 * w + msb64(v) : p;
    }
    return p;
}

// where a wavefront's lanes store a context's scalars, a dword each: rank, n_contra, the
// halves of first_contra, ctx_flags (one store of five lanes instead of four with an address each)
struct RegScalars {
    char* at;
    uint32_t step;  // bytes per context
};
__device__ __forceinline__ RegScalars reg_scalars(const FitArgs& a) {
    const int lane = threadIdx.x & 63;
    RegScalars r;
    r.at = reinterpret_cast<char*>(lane == 0   ? a.rank
                                   : lane == 1 ? a.n_contra
                                   : lane < 4  ? reinterpret_cast<int32_t*>(a.first_contra) + (lane - 2)
                                               : reinterpret_cast<int32_t*>(a.ctx_flags));
    r.step = lane == 2 || lane == 3 ? 8 : 4;
    return r;
}

// One context: c of width n with m <= kLongRows rows from R on.  raw holds its first block's rows
// on entry; `next(raw)` is called once, when the last block's rows have been taken, and fills raw
// with the rows to be fitted after it; `next.offsets` gives the context's output offsets.
template <int FW, bool NARROW = false, typename Next>
__device__ __forceinline__ void fit_ctx_reg(const FitArgs& a, const RegScalars& sc, int c, int n, int m, const uint64_t* R,
                                            uint64_t* sRec, RegRows& raw, Next& next) {
    constexpr int W = FW + F2_Y_WORDS;
    const int lane = threadIdx.x & 63;
    const int d = n + 1;
    const uint64_t tmask = top_mask(n, FW);
    const int cw = n >> 6;
    const uint64_t cbit = 1ull << (n & 63);
    uint64_t xm[FW];  // the x columns of each feature word (the constant column cleared)
    uint64_t pm[FW];  // pivots of the basis
#pragma unroll
    for (int w = 0; w < FW; ++w) {
        xm[w] = (w == cw) ? ~cbit : ~0ull;
        pm[w] = 0;
    }
    int ncontra = 0, first = -1;

    for (int b0 = 0;; b0 += 64) {
        uint64_t f[FW], y0, y1;
#pragma unroll
        for (int w = 0; w < FW; ++w) f[w] = raw.word(w);
        f[FW - 1] &= tmask;
        if constexpr (NARROW) f[0] = static_cast<uint32_t>(f[0]);
        y0 = raw.word(FW);
        y1 = raw.word(FW + 1);
        const bool last = b0 + 64 >= m;
        if (last) next(raw);
        else raw = load_rows<W>(R, m, b0 + 64);
        // (1) reduce against the basis: it is fully reduced, so the row's own (unreduced)
        //     bits at the pivot columns select the records to add; the selection masks do
        //     not depend on one another
        uint64_t f0[FW];
#pragma unroll
        for (int w = 0; w < FW; ++w) f0[w] = f[w];
#pragma unroll
        for (int h = 0; h < (NARROW ? 1 : 2 * FW); ++h) {
            uint32_t ps = static_cast<uint32_t>(pm[h / 2] >> (32 * (h & 1)));
            const int own = static_cast<int>(static_cast<uint32_t>(f0[h / 2] >> (32 * (h & 1))));
            const uint64_t* base = sRec + 32 * h * W;
            auto add = [&](int b, const uint64_t (&rv)[W]) {
                const uint32_t mm = static_cast<uint32_t>(__builtin_amdgcn_sbfe(own, b, 1));
#pragma unroll
                for (int w = 0; w < FW; ++w) f[w] = feat_xor_and<NARROW>(f[w], mm, rv[w]);
                y0 = xor_and(y0, mm, rv[FW]);
                y1 = xor_and(y1, mm, rv[FW + 1]);
            };
            while (ps & (ps - 1)) {  // two records at a time
                const int b = __ffs(ps) - 1, b2 = __ffs(ps & (ps - 1)) - 1;
                ps &= ps - 1;
                ps &= ps - 1;
                uint64_t rv[W], rw[W];
#pragma unroll
                for (int w = 0; w < W; ++w) rv[w] = base[b * W + w];
#pragma unroll
                for (int w = 0; w < W; ++w) rw[w] = base[b2 * W + w];
                add(b, rv);
                add(b2, rw);
            }
            if (ps) {
                const int b = __ffs(ps) - 1;
                uint64_t rv[W];
#pragma unroll
                for (int w = 0; w < W; ++w) rv[w] = base[b * W + w];
                add(b, rv);
            }
        }

        // (2) elimination in stream order: the earliest row with a nonzero feature
        //     residual becomes a basis row where it stands, and its pivot is cleared
        //     from every other row of the block, so that the new rows end fully reduced
        //     among themselves (and hold no older pivot)
        const uint64_t valid = m - b0 >= 64 ? ~0ull : m > b0 ? (1ull << (m - b0)) - 1 : 0ull;
        uint64_t newp[FW];
        eliminate_block<FW, NARROW>(f, y0, y1, valid, n, xm, newp);
        // (3) the rows that are left have zero features: redundant, or contradictory
        //     when their output is nonzero (Eq. 8)
        uint64_t any = f[0], grown = newp[0], old = pm[0];
#pragma unroll
        for (int w = 1; w < FW; ++w) {
            any |= f[w];
            grown |= newp[w];
            old |= pm[w];
        }
        const uint64_t cm = __ballot(any == 0 && (y0 | y1) != 0) & valid;
        if (cm) {
            if (ncontra == 0) first = b0 + ffs64(cm);
            ncontra += __popcll(cm);
        }
        // (4) the new rows join the basis; the older rows lose the new pivots (whose rows hold
        //     no other new pivot: an older row's bits, read once, select what to add)
        if (grown) {
            if (any != 0) {
                uint64_t* rec = sRec + row_pivot<FW>(f, xm, n) * W;
#pragma unroll
                for (int w = 0; w < FW; ++w) rec[w] = f[w];
                rec[FW] = y0;
                rec[FW + 1] = y1;
            }
            wave_sync();
            if (old) {
#pragma unroll
                for (int k = 0; k < FW; ++k) {
                    if (!pm[k]) continue;
                    uint64_t* rec = sRec + (64 * k + lane) * W;
                    uint64_t v[W], v0[FW];
#pragma unroll
                    for (int w = 0; w < W; ++w) v[w] = rec[w];
#pragma unroll
                    for (int w = 0; w < FW; ++w) v0[w] = v[w];
#pragma unroll
                    for (int w = 0; w < FW; ++w) {
                        uint64_t q = newp[w];
                        while (q) {
                            const int b = ffs64(q);
                            q &= q - 1;
                            const uint64_t* nr = sRec + (64 * w + b) * W;
                            const uint32_t mm = feat_mask<NARROW>(v0[w], b);
#pragma unroll
                            for (int u = 0; u < W; ++u) v[u] = u < FW ? feat_xor_and<NARROW>(v[u], mm, nr[u]) : xor_and(v[u], mm, nr[u]);
                        }
                    }
                    if ((pm[k] >> lane) & 1ull) {
#pragma unroll
                        for (int w = 0; w < W; ++w) rec[w] = v[w];
                    }
                }
                wave_sync();
            }
#pragma unroll
            for (int w = 0; w < FW; ++w) pm[w] |= newp[w];
        }
        if (last) break;
    }

    // what is to be fitted next has arrived before the outputs are stored: a load is waited
    // for together with the stores issued after it
    next.arrived(raw);

    // outputs: basis rows and pivots in descending priority, canonical map, parity-check
    // rows, scalars
    int rank = 0;
#pragma unroll
    for (int w = 0; w < FW; ++w) rank += __popcll(pm[w]);
    int64_t bo, po, mo;
    next.offsets(bo, po, mo);
#pragma unroll
    for (int k = 0; k < FW; ++k) {
        const int p = 64 * k + lane;
        const bool present = (pm[k] >> lane) & 1ull;
        uint64_t v[W];
#pragma unroll
        for (int w = 0; w < W; ++w) v[w] = present ? sRec[p * W + w] : 0ull;
        if (p < d) {
            const uint64_t y[2] = {v[FW], v[FW + 1]};
            store_words<2>(a.maps + mo, static_cast<uint32_t>(p) * 16, y);
        }
        if (present) {
            int kout = rank - 1;
            if (p != n) {  // pivots of higher priority: x bits above p
                kout = __popcll((pm[k] & xm[k]) >> lane) - 1;
#pragma unroll
                for (int w = k + 1; w < FW; ++w) kout += __popcll(pm[w] & xm[w]);
            }
            store_words<W>(a.basis + bo, static_cast<uint32_t>(kout) * (8 * W), v);
            (a.pivots + po)[static_cast<uint32_t>(kout)] = p;
        }
    }
    // Word v of the parity-check row of free column 64 w + f holds, at bit b, bit f of word w
    // of the basis row of pivot 64 v + b: with lane b holding word w of that basis row (zero
    // for a free column), a bit-matrix transpose across the wavefront gives lane f exactly
    // that word; the free lanes then store their rows in ascending order.
    uint64_t* H = a.tables + bo;
    if (has_parity_rows(d, rank)) {
        int base = 0;  // free columns in the words before w
#pragma unroll
        for (int w = 0; w < FW; ++w) {
            const uint64_t fr = ~pm[w] & (w == FW - 1 ? tmask : ~0ull);
            if (!fr) continue;  // no free column in this word (full rank: none at all)
            const bool mine = (fr >> lane) & 1ull;
            const uint32_t i = base + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(fr >> 32),
                                                                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(fr), 0));
#pragma unroll
            for (int v = 0; v < FW; ++v) {
                const bool piv = (pm[v] >> lane) & 1ull;
                const uint64_t col = transpose64(piv ? sRec[(64 * v + lane) * W + w] : 0ull, lane);
                if (mine) H[i * FW + v] = col | (v == w ? (1ull << lane) : 0ull);
            }
            base += __popcll(fr);
        }
    }
    if (lane < 5) {
        const int v = lane == 0   ? rank
                      : lane == 1 ? ncontra
                      : lane == 2 ? first
                      : lane == 3 ? first >> 31
                                  : static_cast<int>(ncontra ? F2_CTX_CONTRADICTION : 0u);
        *reinterpret_cast<int32_t*>(sc.at + static_cast<uint64_t>(static_cast<uint32_t>(c)) * sc.step) = v;
    }
    wave_sync();
}

// a context with none after it
template <int FW>
__device__ __forceinline__ void fit_ctx_alone(const FitArgs& a, const CtxDesc& ds, uint64_t* sRec) {
    struct {
        const CtxDesc& ds;
        __device__ __forceinline__ void operator()(RegRows&) {}
        __device__ __forceinline__ void arrived(RegRows&) {}
        __device__ __forceinline__ void offsets(int64_t& bo, int64_t& po, int64_t& mo) {
            bo = ds.bo;
            po = ds.po;
            mo = ds.mo;
        }
    } none{ds};
    const uint64_t* R = a.rows + ds.row0;
    const int m = static_cast<int>(ds.m);
    RegRows raw = load_rows<FW + F2_Y_WORDS>(R, m, 0);
    fit_ctx_reg<FW>(a, reg_scalars(a), ds.c, ds.n, m, R, sRec, raw, none);
}

// ---------------------------------------------------------------------------
// fit by several wavefronts: retained row of pivot p in LDS record p (fw + 2
// words), a pivot-column bitmask beside it, for contexts of 5-8 feature words
// and for long ones of fewer.  The next NW blocks of 64 rows are reduced
// in parallel, one per wavefront; the first block (in stream order) that still
// holds a nonzero feature residual runs the insertion loop in its own
// wavefront (in registers), the blocks before it are only classified, the
// blocks after it are redone against the grown basis; then every wavefront
// clears the new pivots from the retained records.  Once the basis stops
// growing every round completes NW blocks, and a large basis reduces through
// Four-Russians tables.
// ---------------------------------------------------------------------------
constexpr int kPivRec = kPivMaxFW + F2_Y_WORDS;  // record words
constexpr int kPivCap = 64 * kPivMaxFW;          // d <= 512
constexpr int kPivWaves = 4;
constexpr int kPivThreads = 64 * kPivWaves;

// Four-Russians tables for contexts of up to 4 feature words (d <= 256): their
// records use rec[0, 256), and the tables take the rest of rec plus tabx (the
// two are adjacent): table g holds the 16 XOR combinations of the retained rows
// of positions 4g .. 4g+3 (fw + 2 words each; absent pivots contribute zero)
constexpr int kPivTabExtra = 1480;  // keeps three workgroups per compute unit within the LDS
constexpr int kPivTabWords = (kPivCap / 2) * kPivRec + kPivTabExtra;
constexpr int kPivTabMinRank = 32;   // smaller bases reduce as fast record by record
constexpr int kPivTabMinRows = 512;  // tables are built only with two rounds of rows or more to go

struct alignas(16) PivShared {  // 16-byte aligned: the tables are read 16 bytes at a time
    uint64_t rec[kPivCap][kPivRec];
    uint64_t tabx[kPivTabExtra];  // continues rec (tables)
    uint64_t pm[kPivMaxFW];   // pivot columns of the retained rows
    uint64_t npm[kPivMaxFW];  // pivot columns of the rows the current round added
    int flag[8];  // per wavefront (up to 8)
    int contra, nnew;
    long long first, round_first;
};

// all threads: the tables of the first positions (as many as fit) from the records
template <int FW, int NW>
__device__ __forceinline__ int piv_build_tables(PivShared& S, int d) {
    constexpr int W = FW + F2_Y_WORDS;
    constexpr int cap = kPivTabWords / (16 * W);
    const int nt = (d + 3) / 4 < cap ? (d + 3) / 4 : cap;
    uint64_t* tab = &S.rec[kPivCap / 2][0];
    for (int t = threadIdx.x; t < nt * W; t += 64 * NW) {  // one (table, word) per step
        const int g = t / W, w = t - g * W;
        uint64_t* e = tab + g * 16 * W + w;  // entry k of table g at e[k W]
        e[0] = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int p = 4 * g + b;
            const bool piv = p < d && ((S.pm[p >> 6] >> (p & 63)) & 1ull);
            const uint64_t r = piv ? S.rec[p][w] : 0ull;
            for (int k = 0; k < (1 << b); ++k) e[((1 << b) + k) * W] = e[k * W] ^ r;
        }
    }
    return nt;
}

// one table entry of W words from LDS, 16 bytes per read where W is even (the
// entries then start 16-byte aligned)
typedef unsigned long long u64x2_t __attribute__((ext_vector_type(2)));
template <int W>
__device__ __forceinline__ void load_entry(const uint64_t* e, uint64_t (&v)[W]) {
    if constexpr (W % 2 == 0) {
#pragma unroll
        for (int u = 0; u < W / 2; ++u) {
            const u64x2_t p = reinterpret_cast<const u64x2_t*>(e)[u];
            v[2 * u] = p.x;
            v[2 * u + 1] = p.y;
        }
    } else {
#pragma unroll
        for (int u = 0; u < W; ++u) v[u] = e[u];
    }
}

// reduce this wavefront's block rows against the retained basis (one pass: the
// basis is fully reduced).  Positions [0, 4 ntab) by table lookups: the row's own
// 4 bits at positions 4g .. 4g+3, masked to the pivots, select entry of table g.
template <int FW, bool FAR>
__device__ __forceinline__ void piv_reduce(PivShared& S, int ntab, uint64_t (&f)[FW], uint64_t& y0, uint64_t& y1) {
    constexpr int W = FW + F2_Y_WORDS;
    uint64_t f0[FW];
#pragma unroll
    for (int w = 0; w < FW; ++w) f0[w] = f[w];
    if constexpr (FW <= 4) {
        const uint64_t* tab = &S.rec[kPivCap / 2][0];
#pragma unroll
        for (int w = 0; w < FW; ++w) {
            if (16 * w >= ntab) break;
            const uint64_t pmw = S.pm[w];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t half = h ? static_cast<uint32_t>(f0[w] >> 32) : static_cast<uint32_t>(f0[w]);
                const uint32_t pmh = h ? static_cast<uint32_t>(pmw >> 32) : static_cast<uint32_t>(pmw);
#pragma unroll
                for (int k = 0; k < 8; k += 4) {  // four tables per step: every entry read issued first
                    const int g = 16 * w + 8 * h + k;
                    if (g >= ntab) break;
                    uint64_t ev[4][W];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // past the last table: entry 0 of table g (zero)
                        const bool in = g + q < ntab;
                        const uint32_t iq = in ? __builtin_amdgcn_ubfe(half, 4 * (k + q), 4) &
                                                     ((pmh >> (4 * (k + q))) & 0xFu)
                                               : 0u;
                        load_entry<W>(tab + (16 * (in ? g + q : g) + static_cast<int>(iq)) * W, ev[q]);
                    }
#pragma unroll
                    for (int u = 0; u < FW; ++u) f[u] = xor3(xor3(f[u], ev[0][u], ev[1][u]), ev[2][u], ev[3][u]);
                    y0 = xor3(xor3(y0, ev[0][FW], ev[1][FW]), ev[2][FW], ev[3][FW]);
                    y1 = xor3(xor3(y1, ev[0][FW + 1], ev[1][FW + 1]), ev[2][FW + 1], ev[3][FW + 1]);
                }
            }
        }
    }
    const int done = FW <= 4 ? 4 * ntab : 0;  // positions below are reduced
#pragma unroll
    for (int h = 0; h < 2 * FW; ++h) {  // half a word of pivots at a time
        if (32 * h + 32 <= done) continue;
        uint32_t ps = __builtin_amdgcn_readfirstlane(reinterpret_cast<const uint32_t*>(S.pm)[h]);
        if (32 * h < done) ps &= ~0u << (done & 31);
        const int own = static_cast<int>(static_cast<uint32_t>(f0[h / 2] >> (32 * (h & 1))));  // unreduced
        // U records at a time (past the last, record 0 of the half with an empty mask)
        constexpr int U = FW <= 5 || FAR ? 4 : 2;
        while (ps) {
            uint32_t mk[U];
            uint64_t rv[U][W];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = ps ? __builtin_ctz(ps) : 0;
                mk[u] = ps ? static_cast<uint32_t>(__builtin_amdgcn_sbfe(own, b, 1)) : 0u;
                ps &= ps - 1;
                const uint64_t* rec = S.rec[32 * h + b];
#pragma unroll
                for (int w = 0; w < W; ++w) rv[u][w] = rec[w];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int w = 0; w < FW; ++w) f[w] = xor_and(f[w], mk[u], rv[u][w]);
                y0 = xor_and(y0, mk[u], rv[u][FW]);
                y1 = xor_and(y1, mk[u], rv[u][FW + 1]);
            }
        }
    }
}

// in-block elimination of one wavefront's block, in registers.  The block was reduced first,
// so the new rows hold no retained pivot.  The rows that are left are classified; the new
// rows go to their records, their pivots to npm and their count to nnew; the retained rows
// are cleared of the new pivots afterwards by all wavefronts (piv_backsub).
template <int FW>
__device__ __forceinline__ void piv_insert(PivShared& S, int n, int64_t b0, bool valid, uint64_t (&f)[FW], uint64_t& y0,
                                           uint64_t& y1, int& ncon, long long& firstc) {
    const int lane = threadIdx.x & 63;
    const int cw = n >> 6;
    const uint64_t cbit = 1ull << (n & 63);
    uint64_t xm[FW];  // the x columns of each feature word (the constant column cleared)
#pragma unroll
    for (int w = 0; w < FW; ++w) xm[w] = (w == cw) ? ~cbit : ~0ull;
    uint64_t newp[FW];
    eliminate_block<FW>(f, y0, y1, __ballot(valid), n, xm, newp);
    uint64_t any = f[0];
#pragma unroll
    for (int w = 1; w < FW; ++w) any |= f[w];
    const uint64_t cm = __ballot(valid && any == 0 && (y0 | y1) != 0);
    if (cm) {
        firstc = b0 + ffs64(cm);
        ncon = __popcll(cm);
    }
    if (valid && any != 0) {
        uint64_t* rec = S.rec[row_pivot<FW>(f, xm, n)];
#pragma unroll
        for (int w = 0; w < FW; ++w) rec[w] = f[w];
        rec[FW] = y0;
        rec[FW + 1] = y1;
    }
    int nnew = 0;
#pragma unroll
    for (int w = 0; w < FW; ++w) {
        nnew += __popcll(newp[w]);
        if (lane == w) S.npm[w] = newp[w];
    }
    if (lane == 0) S.nnew = nnew;
}

// clear the round's new pivots from the retained rows (records of S.pm), one
// record per thread.  The new rows hold no other new pivot, so a record's bits
// at the new pivots, read once before any addition, select the rows to add.
template <int FW, int NW>
__device__ __forceinline__ void piv_backsub(PivShared& S, int d, int fw) {
    for (int s = threadIdx.x; s < d; s += 64 * NW) {
        if (!((S.pm[s >> 6] >> (s & 63)) & 1ull)) continue;
        uint64_t* rec = S.rec[s];
        uint64_t R[FW + 2];
#pragma unroll
        for (int w = 0; w < FW + 2; ++w) R[w] = rec[w];
        uint64_t R0[FW];
#pragma unroll
        for (int w = 0; w < FW; ++w) R0[w] = R[w];
#pragma unroll
        for (int w = 0; w < FW; ++w) {
            if (w >= fw) break;
            uint64_t m = S.npm[w];
            auto fetch = [&](int& b, uint64_t (&r)[FW + 2]) {
                b = ffs64(m);
                m &= m - 1;
                const uint64_t* nr = S.rec[64 * w + b];
#pragma unroll
                for (int u = 0; u < FW + 2; ++u) r[u] = nr[u];
            };
            auto add = [&](int b, const uint64_t (&r)[FW + 2]) {
                const uint32_t mk = bit_mask(R0[w], b);
#pragma unroll
                for (int u = 0; u < FW + 2; ++u) R[u] = xor_and(R[u], mk, r[u]);
            };
            if (!m) continue;
            int ba, bb;
            uint64_t ra[FW + 2], rb[FW + 2];
            if constexpr (FW > 6) {  // (no registers to read ahead)
                while (m) {
                    fetch(ba, ra);
                    add(ba, ra);
                }
                continue;
            }
            fetch(ba, ra);
            for (;;) {  // the next new row is read while this one is added
                const bool more = m != 0;
                if (more) fetch(bb, rb);
                add(ba, ra);
                if (!more) break;
                const bool again = m != 0;
                if (again) fetch(ba, ra);
                add(bb, rb);
                if (!again) break;
            }
        }
#pragma unroll
        for (int w = 0; w < FW + 2; ++w) rec[w] = R[w];
    }
}

// the wavefronts of a workgroup, or some of them, wait for one another
struct BlockSync {
    // registers for four of the widest records at a time (k_fit_piv: 168, and 24 values that spill
    // in its outputs and between contexts)
    static constexpr bool kFar = true;
    __device__ __forceinline__ void operator()() { __syncthreads(); }
};
// NW wavefronts of a larger workgroup: a count in LDS that each adds to once per wait.  Every
// wavefront of a workgroup is resident and each of the NW passes the same waits, so each wait ends.
template <int NW>
struct PartSync {
    static constexpr bool kFar = false;
    int* count;   // zero before the first wait
    int target;
    __device__ __forceinline__ void operator()() {
        target += NW;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
};

template <int FW, int NW, typename Sync>
__device__ __forceinline__ void fit_ctx_piv(const FitArgs& a, const CtxDesc& ds, PivShared& S, Sync& sync) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = ds.c, n = ds.n, d = n + 1;
    const int fw = feat_words(n);  // <= FW; records keep FW feature words, then the two output words
    const int Wr = fw + F2_Y_WORDS;
    const int64_t m = ds.m;
    const uint64_t* R = a.rows + ds.row0;
    const uint64_t tmask = top_mask(n, fw);

    static_assert(NW > 1, "rounds of several wavefronts");
    if (tid < kPivMaxFW) {
        S.pm[tid] = 0;
        S.npm[tid] = 0;
    }
    if (tid == 0) {
        S.contra = 0;
        S.nnew = 0;
        S.first = -1;
    }
    sync();
    // the next round's block is loaded while this round runs, on the guess that
    // the round completes all NW blocks (it does once the basis stops growing);
    // not for the widest records, whose registers it would cost occupancy
    constexpr bool kPrefetch = FW <= 4;
    // raw words of this wavefront's row in the block at base, row index clamped
    // into the segment (lanes past its end are masked at use).  Up to 4 feature
    // words every load is issued (fw >= FW - 1 there, so word FW - 1 is still in
    // the row): a fixed count of loads in flight, which the wait for them can count.
    auto load_raw = [&](int64_t base, uint64_t (&raw)[FW + 2]) {
        const int64_t ii = base + 64 * wave + lane;
        const uint64_t* row = R + (ii < m ? ii : m - 1) * Wr;
#pragma unroll
        for (int w = 0; w < FW; ++w) raw[w] = (kPrefetch || w < fw) ? row[w] : 0ull;
        raw[FW] = row[fw];
        raw[FW + 1] = row[fw + 1];
    };
    uint64_t pre[FW + 2];
    int64_t pre_b0 = -1;
    int rank = 0;
    // valid tables (positions [0, 4 ntab)), 0: none.  Every wavefront keeps its own count: one in
    // LDS, set by the first wavefront to have built its part, could keep a late one from the
    // build and from the wait behind it.
    int ntab = 0;
    int64_t b0 = 0;
    while (b0 < m) {
        const int64_t bw = b0 + 64 * wave;  // this wavefront's block
        const int64_t i = bw + lane;
        const bool valid = i < m;
        uint64_t raw[FW + 2];
        if (kPrefetch && pre_b0 == b0) {
#pragma unroll
            for (int w = 0; w < FW + 2; ++w) raw[w] = pre[w];
        } else {
            load_raw(b0, raw);
        }
        if constexpr (kPrefetch) {  // issued unconditionally (a block past the end reads the last row)
            pre_b0 = b0 + 64 * NW;
            load_raw(pre_b0, pre);
        }
        uint64_t f[FW], y0, y1;
#pragma unroll
        for (int w = 0; w < FW; ++w) f[w] = (valid && w < fw) ? raw[w] : 0ull;
#pragma unroll
        for (int w = 0; w < FW; ++w)
            if (w == fw - 1) f[w] &= tmask;
        y0 = valid ? raw[FW] : 0ull;
        y1 = valid ? raw[FW + 1] : 0ull;
        if constexpr (FW <= 4) {  // a large basis that will serve two rounds or more: tables
            if (ntab == 0 && rank >= kPivTabMinRank && m - b0 >= kPivTabMinRows) {
                ntab = piv_build_tables<FW, NW>(S, d);
                sync();
            }
        }
        if (rank > 0) piv_reduce<FW, Sync::kFar>(S, ntab, f, y0, y1);
        uint64_t any = f[0];
#pragma unroll
        for (int w = 1; w < FW; ++w) any |= f[w];
        const bool has_nz = __ballot(valid && any != 0) != 0;
        if (lane == 0) S.flag[wave] = has_nz ? 1 : 0;
        if (tid == 0) S.round_first = 0x7fffffffffffffffll;
        sync();
        int wstar = NW;
        for (int w = NW - 1; w >= 0; --w)
            if (S.flag[w]) wstar = w;
        int ncon = 0;
        long long firstc = -1;
        if (wave < wstar) {  // every residual is zero: redundant or contradictory rows
            const uint64_t cm = __ballot(valid && (y0 | y1) != 0);
            if (cm) {
                ncon = __popcll(cm);
                firstc = bw + ffs64(cm);
            }
        } else if (wave == wstar) {
            piv_insert<FW>(S, n, bw, valid, f, y0, y1, ncon, firstc);
        }
        if (lane == 0 && ncon) {
            atomicAdd(&S.contra, ncon);
            atomicMin(&S.round_first, firstc);
        }
        sync();
        if (S.nnew) {  // retained rows lose the new pivots, then the new rows join them
            piv_backsub<FW, NW>(S, d, fw);
            sync();
            if (tid < fw) S.pm[tid] |= S.npm[tid];
            ntab = 0;  // the tables no longer match the basis
            sync();
        }
        if (tid == 0 && S.first < 0 && S.round_first != 0x7fffffffffffffffll) S.first = S.round_first;
        rank = 0;
        for (int w = 0; w < fw; ++w) rank += __popcll(S.pm[w]);
        sync();
        if (tid == 0) S.nnew = 0;
        b0 += 64 * static_cast<int64_t>(wstar < NW ? wstar + 1 : NW);
    }
    sync();

    // outputs: basis rows and pivots in descending priority, canonical map, encode table, scalars
    const int64_t bo = ds.bo, po = ds.po, mo = ds.mo;
    const int cw = n >> 6;
    const uint64_t cbit = 1ull << (n & 63);
    for (int j = tid; j < d; j += 64 * NW) {
        const bool present = (S.pm[j >> 6] >> (j & 63)) & 1ull;
        a.maps[mo + 2 * j] = present ? S.rec[j][FW] : 0ull;
        a.maps[mo + 2 * j + 1] = present ? S.rec[j][FW + 1] : 0ull;
        if (!present) continue;
        int k = rank - 1;
        if (j != n) {  // pivots of higher priority: x bits above j
            k = 0;
            for (int w = j >> 6; w < fw; ++w) {
                uint64_t v = S.pm[w];
                if (w == (j >> 6)) v &= (j & 63) == 63 ? 0ull : (~0ull << ((j & 63) + 1));
                if (w == cw) v &= ~cbit;
                k += __popcll(v);
            }
        }
        uint64_t* out = a.basis + bo + static_cast<int64_t>(k) * Wr;
#pragma unroll
        for (int w = 0; w < FW; ++w)
            if (w < fw) out[w] = S.rec[j][w];
        out[fw] = S.rec[j][FW];
        out[fw + 1] = S.rec[j][FW + 1];
        a.pivots[po + k] = j;
    }
    // parity-check rows of the free columns (word v of the row of free column 64 w + f
    // holds, at bit b, bit f of word w of the retained row of pivot 64 v + b): per word
    // pair (w, v), taken by wavefront v mod NW, a bit-matrix transpose of word w of the
    // retained rows 64 v .. 64 v + 63 (zero for free columns) gives lane f its word
    uint64_t* H = a.tables + bo;
    if (has_parity_rows(d, rank)) {
        const uint64_t lane_lt = (1ull << lane) - 1;
        int base = 0;  // free columns in the words before w
        for (int w = 0; w < fw; ++w) {
            const uint64_t fr = ~S.pm[w] & (w == fw - 1 ? tmask : ~0ull);
            if (!fr) continue;  // no free column in this word
            const bool mine = (fr >> lane) & 1ull;
            const int64_t i = base + __popcll(fr & lane_lt);
            for (int v = wave; v < fw; v += NW) {
                const bool piv = (S.pm[v] >> lane) & 1ull;
                const uint64_t col = transpose64(piv ? S.rec[64 * v + lane][w] : 0ull, lane);
                if (mine) H[i * fw + v] = col | (v == w ? (1ull << lane) : 0ull);
            }
            base += __popcll(fr);
        }
    }
    if (tid == 0) {
        a.rank[c] = rank;
        a.n_contra[c] = S.contra;
        a.first_contra[c] = S.first;
        a.ctx_flags[c] = S.contra ? F2_CTX_CONTRADICTION : 0u;
    }
    sync();
}

// ---------------------------------------------------------------------------
// large-context fit (fw > 8): G workgroups of 8 wavefronts per context (G a power of
// two, all resident: a cooperative launch), one compute unit each.  The rows go in
// blocks of 64; member g takes blocks g, g + G, ...
//
// The working basis is a list of batches in insertion order: the new rows of one
// block, fully reduced among themselves and against every earlier batch (but not
// against later ones).  A later batch has no bit at an earlier batch's pivots, so
// adding, batch by batch in insertion order, the rows that a vector's own bits at the
// batch's pivots select leaves the one representative of its coset that is zero at
// every pivot: the same residual that a fully reduced basis gives, hence the same
// pivots, kept rows and contradictions.  Nothing that was inserted is ever rewritten
// (a basis kept fully reduced rewrites every retained row for every block: its stores,
// and reading the rewritten rows back, took half the time of a block), and members
// read each other's batches as they appear, without barriers.  The fully reduced
// basis is made once, at the end.
//
// The list lives in the context's tables area (capacity d rows of fw + 2 words), its
// pivots, with the block they come from, in the context's pivots area; both are final
// outputs only later.
//
// A round takes rows of one batch alone, so a stream that adds a few rows per block would cost
// a round for each few rows.  Whoever completes a chunk of 32 list rows that holds the
// ends of four batches or more reduces its rows among themselves, into the chunk's place in the context's
// basis area, before its block counts as done: a batch like any other, with the pivots and the span of
// those it replaces.  Every member comes to the same from the list's entries, and reads the chunk
// there; at the end the merged chunks are copied into the list.  One new row per
// block of 64: 128 contexts of 601 columns and rank 256 6.8 ms, 52 ms round by round; 8 of
// 2,048 columns and rank 1,024 22 and 201 ms.  (Chunks of 16: 6.2 and 22 ms, and dense contexts 3% slower.)
//
//   (1) block reduce, 32 basis rows (half a batch) per round, with Four-Russians tables
//       (the method of Arlazarov, Dinic, Kronrod and Faradzev): four rows give a
//       16-entry LDS table of their XOR combinations, and a row's four bits at their
//       pivots select the entry to add.  A half wavefront holds one row, two feature
//       words per lane, so that one 16-byte LDS read serves two rows;
//   (2) a block whose residuals are all zero is done whatever the blocks before it
//       still add.  Otherwise the member waits for them, reduces by what they added, and
//   (3) eliminates in stream order on panels: one wavefront, a column per lane, works on
//       the two highest feature words that hold a bit (128 columns) and notes which rows
//       were added to which (a 64 x 64 matrix T); then all wavefronts apply T to the
//       whole rows.  Rows that the panel reduces to zero go on to the next panel;
//   (4) the new rows are published.
// Once the rank reaches d the basis is the identity on the features and the map alone
// remains: a triangular solve of the output words, word by word from the lowest
// priority up, then every remaining row is checked against the map.  Below d each
// batch is reduced by the later ones as in (1).
//
// 64 contexts, n = 4095, 8,192 rows: 10.27 ms with a basis kept fully reduced (groups
// of 4 workgroups exchanging partial sums), 4.25 ms with 16 wavefronts of 4 rows and
// loads one round ahead, 3.33 ms.  A round of 32 basis rows takes about 4,200 cycles:
// 2,700 of LDS bandwidth (a table lookup moves 512 bytes for four basis rows) and 2,000
// of VALU issue that two wavefronts per SIMD do not overlap further.
// ---------------------------------------------------------------------------
// 256 registers a wavefront: loads two rounds ahead.  The rounds keep all of theirs; 142 more
// values spill around them, in the code of a block and of its outputs (440 bytes of scratch a lane).
constexpr int kWdWaves = 8;
constexpr int kWdPairs = 64 / kWdWaves / 2;  // pairs of block rows per wavefront
constexpr int kWdThreads = 64 * kWdWaves;
constexpr int kWdRows = 64;                   // rows per block
constexpr int kWdMaxBlocks = (1 << 19) - 2;   // block numbers in a pivot's tag; contexts of more rows take one member
constexpr int kWdBar = 1 << 30;               // progress values from here on: past the blocks
constexpr int kPivLast = 1 << 12;             // the last pivot of a batch
constexpr int kPivMerged = 1 << 13;           // the first pivot of a merged chunk (in LDS only)
constexpr int kChunk = 32;                    // list rows that are merged where they came in small batches
constexpr int kChunkEnds = 4;                 // from as many batch ends within the chunk
constexpr int kRowPitch = 33;                 // elimination: 16-byte units per row in LDS (33: no bank conflicts down a column)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));  // rows are 8-byte aligned

struct WideShared {
    u32x4 tab[2][128][32];             // [buffer][16 table + entry][word pair]; other phases lay out their own data here
    uint32_t sel[kWdWaves][4][128];    // selection: four rows of a wavefront, as words
    uint16_t piv[4096];                // the list's pivots, insertion order, kPivLast on the last of each batch
    u32x4 ys[64];                      // output words: two rounds of 32 rows, or the block's 64 rows
    uint64_t T[kWdRows];               // elimination: block rows added into each row
    uint64_t pm[64];                   // pivot columns
    int above[64];                     // pivots (constant excluded) in words above w
    uint32_t wm[kWdWaves][2];          // nonzero even and odd words of each wavefront's rows
    uint64_t ins;                      // block rows that became basis rows
    uint64_t panel;                    // the ones of the current panel
    int more;                          // a pending row holds a bit: another panel follows
    int any[2];                        // nonzero residuals in the block (alternating)
    int nrows, next;                   // list length; every block below `next` is done
    int merged;                        // the list holds merged chunks
    int timeout;                       // a wait of this context gave up
};

__device__ __forceinline__ u32x4 xor_and4(u32x4 f, uint32_t m, u32x4 d) {
    u32x4 r;
    r.x = __builtin_amdgcn_bitop3_b32(f.x, m, d.x, 0x78);
    r.y = __builtin_amdgcn_bitop3_b32(f.y, m, d.y, 0x78);
    r.z = __builtin_amdgcn_bitop3_b32(f.z, m, d.z, 0x78);
    r.w = __builtin_amdgcn_bitop3_b32(f.w, m, d.w, 0x78);
    return r;
}
__device__ __forceinline__ u32x4 xor3_4(u32x4 a, u32x4 b, u32x4 c) {
    u32x4 r;
    r.x = __builtin_amdgcn_bitop3_b32(a.x, b.x, c.x, 0x96);
    r.y = __builtin_amdgcn_bitop3_b32(a.y, b.y, c.y, 0x96);
    r.z = __builtin_amdgcn_bitop3_b32(a.z, b.z, c.z, 0x96);
    r.w = __builtin_amdgcn_bitop3_b32(a.w, b.w, c.w, 0x96);
    return r;
}
__device__ __forceinline__ bool any4(u32x4 v) { return (v.x | v.y | v.z | v.w) != 0; }
__device__ __forceinline__ u32x4 shfl_xor4(u32x4 v, int o) {
    return u32x4{static_cast<uint32_t>(__shfl_xor(static_cast<int>(v.x), o)), static_cast<uint32_t>(__shfl_xor(static_cast<int>(v.y), o)),
                 static_cast<uint32_t>(__shfl_xor(static_cast<int>(v.z), o)), static_cast<uint32_t>(__shfl_xor(static_cast<int>(v.w), o))};
}

// device-scope (sc1) accesses through a buffer resource: what members exchange while
// the kernel runs goes past the caches that other dies do not see
constexpr int kDevScope = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dev_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, static_cast<int>(bytes), 0x00020000);
}
template <bool DEV>
__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, DEV ? kDevScope : 0);
}

__device__ __forceinline__ void put_dev(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_dev32(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// v with the rows of `rows` flipped where row q's bit is set (a column per lane)
__device__ __forceinline__ uint64_t xor_sel(uint64_t v, int q, uint64_t rows) { return xor_and(v, bit_mask(v, q), rows); }

// progress of a group's members: blocks done, or kWdBar + k past barrier k; one word per member,
// cleared by the plan and stored only by it.  A group fits one context (k_fit_wide), so the
// words serve once.
__device__ __forceinline__ void put_progress(int32_t* prog, int g, int done) {
    __hip_atomic_store(prog + g, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// one wavefront: the lowest block not known to be done (own blocks below blk are)
__device__ __forceinline__ int lowest_open(const int32_t* prog, int G, int g, int blk) {
    const int lane = threadIdx.x & 63;
    int nb = 0x7fffffff;
    if (lane < G && lane != g) {
        const int dn = __hip_atomic_load(prog + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (dn < kWdBar) nb = lane + G * dn;
    }
    if (lane == g) nb = blk;
    for (int o = 4; o > 0; o >>= 1) {  // G <= 8
        const int t = __shfl_xor(nb, o);
        nb = t < nb ? t : nb;
    }
    return __builtin_amdgcn_readfirstlane(nb);
}

// one wavefront: take the list entries of blocks below `open` (all published) into LDS;
// returns the new length.  A pivot's entry holds its block number + 1 above bit 13; the
// entry after the last one published holds zero there (the plan clears entry 0).
__device__ __forceinline__ int take_entries(WideShared& L, const int32_t* ent, int nrows, int d, int open) {
    const int lane = threadIdx.x & 63;
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the progress is in before the entries are read
    for (;;) {
        const int i = nrows + lane;
        uint32_t v = 0;
        if (i < d) v = static_cast<uint32_t>(__hip_atomic_load(ent + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const int blk1 = static_cast<int>(v >> 13);
        const uint64_t ok = __ballot(blk1 >= 1 && blk1 <= open);
        const int cnt = ok == ~0ull ? 64 : ffs64(~ok);
        if (lane < cnt) {
            int p = static_cast<int>(v & (kPivLast - 1));
            if (p >= d) p = d - 1;  // (only after a wait that gave up)
            L.piv[i] = static_cast<uint16_t>(p | (v & kPivLast));
        }
        nrows += cnt;
        if (cnt < 64 || nrows >= d) return nrows;
    }
}

// one wavefront: does chunk q (whole) hold many small batches?  (The flags inside a chunk are as published until it is marked.)
__device__ __forceinline__ bool chunk_small(const WideShared& L, int q) {
    const int lane = threadIdx.x & 63;
    const uint64_t ends = __ballot(lane < kChunk - 1 && (L.piv[kChunk * q + (lane & (kChunk - 1))] & kPivLast));
    return __popcll(ends) >= kChunkEnds;
}
// one wavefront: the chunks that list rows from .. to - 1 completed become a batch of their own where they are merged
__device__ __forceinline__ void mark_chunks(WideShared& L, int from, int to) {
    const int lane = threadIdx.x & 63;
    wave_sync();
    for (int q = from / kChunk; q < to / kChunk; ++q) {
        if (!chunk_small(L, q)) continue;
        if (lane < kChunk) {
            uint16_t* e = &L.piv[kChunk * q + lane];
            *e = static_cast<uint16_t>((*e & (kPivLast - 1)) | (lane == 0 ? kPivMerged : lane == kChunk - 1 ? kPivLast : 0));
        }
        if (lane == 0) {
            if (q) L.piv[kChunk * q - 1] |= kPivLast;
            L.merged = 1;
        }
        wave_sync();
    }
}

// the basis rows of one round: wavefront t takes rows 4 t .. 4 t + 3 of it
struct RoundRows {
    u32x4 f[2];  // two words per lane of row 2 i + h in half wavefront h
    u32x4 y;     // output words of row lane & 3
};
template <bool DEV>
__device__ __forceinline__ void load_rows(__amdgpu_buffer_rsrc_t X, int W, int fw, int start, int cnt, int t, int voff,
                                          int lane, RoundRows& r) {
    const int soff = start * W * 8;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = 4 * t + 2 * i + (lane >> 5);
        r.f[i] = load16<DEV>(X, (k < cnt ? k : cnt - 1) * W * 8 + voff, soff);
    }
    const int k = 4 * t + (lane & 3);
    r.y = load16<DEV>(X, ((k < cnt ? k : cnt - 1) * W + fw) * 8, soff);
}

// lower and upper half of v, each in both half wavefronts
__device__ __forceinline__ void spread_halves(u32x4 v, u32x4& lo, u32x4& hi) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(v[k], v[k], false, false);
        lo[k] = r[0];
        hi[k] = r[1];
    }
}

// block rows: wavefront w holds rows 8 w .. 8 w + 7, row 8 w + 2 i + h in half h of acc[i];
// the output words of row 8 w + (lane & 7) are the XOR of y over the lanes of equal lane & 7
struct BlockRows {
    u32x4 acc[kWdPairs];
    u32x4 y;
};

// rows [start, start + cnt) of the list: half `half` of the batch of K rows at pos; cnt 0: none
struct Round {
    int pos, K, half, cnt;
    int merged;  // a merged chunk: its rows are in Y
};

// reduce the block by list rows pos .. nrows - 1 (pos < nrows starts a batch)
__device__ __forceinline__ void wide_reduce(WideShared& L, __amdgpu_buffer_rsrc_t X, __amdgpu_buffer_rsrc_t Y, int W, int d,
                                            int pos, int nrows, BlockRows& b) {
    const int fw = W - F2_Y_WORDS;
    const int lane = threadIdx.x & 63, j = lane & 31, h = lane >> 5;
    const int t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int voff = 16 * (2 * j < fw ? j : 0);
    char* const tab = reinterpret_cast<char*>(&L.tab[0][0][0]);
    // the round after r, from the list entries behind r's batch (read ahead)
    auto entry_after = [&](const Round& r) {
        const int i = r.pos + r.K + lane;
        return static_cast<int>(L.piv[i < nrows ? i : nrows - 1]);
    };
    auto after = [&](const Round& r, int e) {
        if (r.half == 0 && r.K > 32) return Round{r.pos, r.K, 1, r.K - 32, 0};
        const int p0 = r.pos + r.K;
        if (p0 >= nrows) return Round{p0, 0, 0, 0, 0};
        const uint64_t last = __ballot(p0 + lane < nrows && (e & kPivLast));
        const int left = nrows - p0 < 64 ? nrows - p0 : 64;
        const int k = last ? ffs64(last) + 1 : 64, K = k < left ? k : left;
        return Round{p0, K, 0, K < 32 ? K : 32, __builtin_amdgcn_readfirstlane(e) & kPivMerged};
    };
    // always the same number of loads (past the list, its last row): the wait for one
    // round's rows then leaves the next round's in flight
    auto fetch = [&](const Round& r, RoundRows& rr) {
        const int start = r.cnt ? r.pos + 32 * r.half : nrows - 1, cnt = r.cnt ? r.cnt : 1;
        // The first rows of a batch may share a cache line with the batch before it, read
        // before they were written; so may the last two rows that the area holds with the first
        // of the area behind it, another context's, which another group may read on the same die.
        const __amdgpu_buffer_rsrc_t S = r.merged ? Y : X;
        if ((r.half == 0 && t == 0) || start + cnt > d - 2) load_rows<true>(S, W, fw, start, cnt, t, voff, lane, rr);
        else load_rows<false>(S, W, fw, start, cnt, t, voff, lane, rr);
    };
    // absent rows are never selected, and entry 0 of an absent table must be zero
    auto store_tables = [&](int buf, const RoundRows& r) {
        u32x4 f0, f1, f2, f3;
        spread_halves(r.f[0], f0, f1);
        spread_halves(r.f[1], f2, f3);
        const u32x4 b0 = f2 & (h ? ~0u : 0u), b1 = b0 ^ f3, f01 = f0 ^ f1;
        char* e = tab + 65536 * buf + ((16 * t + 4 * h) * 32 + j) * 16;  // half h: entries 4 h .. and 8 + 4 h ..
        *reinterpret_cast<u32x4*>(e) = b0;
        *reinterpret_cast<u32x4*>(e + 512) = b0 ^ f0;
        *reinterpret_cast<u32x4*>(e + 1024) = b0 ^ f1;
        *reinterpret_cast<u32x4*>(e + 1536) = b0 ^ f01;
        *reinterpret_cast<u32x4*>(e + 4096) = b1;
        *reinterpret_cast<u32x4*>(e + 4608) = b1 ^ f0;
        *reinterpret_cast<u32x4*>(e + 5120) = b1 ^ f1;
        *reinterpret_cast<u32x4*>(e + 5632) = b1 ^ f01;
        if (lane < 4) L.ys[32 * buf + 4 * t + lane] = r.y;
    };
    uint32_t sl[kWdPairs], sh[kWdPairs], yl, yh;  // selections of this lane's rows: batch rows 0-31, 32-63
    auto select = [&](const Round& r) {  // the rows' bits at the batch's pivots
        const int p = lane < r.K ? (L.piv[r.pos + lane] & (kPivLast - 1)) : 0;
        yl = yh = 0;
        static_assert(kWdPairs % 2 == 0, "two pairs of rows at a time");
#pragma unroll
        for (int i0 = 0; i0 < kWdPairs; i0 += 2) {
#pragma unroll
            for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4*>(&L.sel[t][2 * i + h][4 * j]) = b.acc[i0 + i];
            wave_sync();
            uint32_t dw[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) dw[i] = L.sel[t][i][p >> 5];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint64_t sr = __ballot(lane < r.K && ((dw[i] >> (p & 31)) & 1u));  // row 2 i0 + i of the wavefront
                const int k = i0 + i / 2;
                if (i % 2 == 0) {
                    sl[k] = static_cast<uint32_t>(sr);
                    sh[k] = static_cast<uint32_t>(sr >> 32);
                } else {
                    sl[k] = h ? static_cast<uint32_t>(sr) : sl[k];
                    sh[k] = h ? static_cast<uint32_t>(sr >> 32) : sh[k];
                }
                yl = (lane & 7) == 2 * i0 + i ? static_cast<uint32_t>(sr) : yl;
                yh = (lane & 7) == 2 * i0 + i ? static_cast<uint32_t>(sr >> 32) : yh;
            }
            wave_sync();
        }
    };
    auto apply = [&](const Round& r, int buf) {
        uint32_t sv[kWdPairs];
#pragma unroll
        for (int i = 0; i < kWdPairs; ++i) sv[i] = r.half ? sh[i] : sl[i];
        const char* lb = tab + 65536 * buf + 16 * j;
        auto two_tables = [&](int g) {
            u32x4 t0[kWdPairs], t1[kWdPairs];
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) {
                t0[i] = *reinterpret_cast<const u32x4*>(lb + (__builtin_amdgcn_ubfe(sv[i], 4 * g, 4) << 9) + g * 8192);
                t1[i] = *reinterpret_cast<const u32x4*>(lb + (__builtin_amdgcn_ubfe(sv[i], 4 * g + 4, 4) << 9) + (g + 1) * 8192);
            }
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) b.acc[i] = xor3_4(b.acc[i], t0[i], t1[i]);
        };
        // output words: lane (table, row) adds the table's selected rows
        const int ty = lane >> 3;
        const uint32_t nib = (r.half ? yh : yl) >> (4 * ty);
        u32x4 yr[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) yr[i] = L.ys[32 * buf + 4 * ty + i];
        if (r.cnt > 24) {  // every table: no branches between the reads, so that they overlap
            two_tables(0);
            two_tables(2);
            two_tables(4);
            two_tables(6);
        } else {
            two_tables(0);
            if (r.cnt > 8) two_tables(2);
            if (r.cnt > 16) two_tables(4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            b.y = xor_and4(b.y, static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(nib), i, 1)), yr[i]);
    };
    // rounds: tables of `cur` in LDS, rows of `nxt` in registers (or on their way), rows of
    // `nn` fetched in this step.  Each SIMD holds one wavefront that builds the next tables
    // before it applies the current ones and one that builds them after, so that the
    // table reads of the one (LDS bandwidth) overlap the other's latencies.
    Round cur = after(Round{pos, 0, 0, 0, 0}, entry_after(Round{pos, 0, 0, 0, 0}));
    Round nxt = after(cur, entry_after(cur));
    Round nn = after(nxt, entry_after(nxt));
    RoundRows ra, rb;
    fetch(cur, rb);
    fetch(nxt, ra);
    store_tables(0, rb);
    __syncthreads();
    const bool early = t >= kWdWaves / 2;
    auto step = [&](int buf, const RoundRows& have, RoundRows& get) {
        if (early) {
            store_tables(buf ^ 1, have);
            fetch(nn, get);
        }
        const int e = entry_after(nn);
        if (cur.half == 0) select(cur);
        apply(cur, buf);
        if (!early) {
            fetch(nn, get);
            store_tables(buf ^ 1, have);
        }
        cur = nxt;
        nxt = nn;
        nn = after(nn, e);
        __syncthreads();
    };
    for (;;) {
        step(0, ra, rb);
        if (!cur.cnt) break;
        step(1, rb, ra);
        if (!cur.cnt) break;
    }
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) b.y ^= shfl_xor4(b.y, o);  // every lane: the whole of its row
}

// full rank: the map by a triangular solve.  Row p (of pivot p) has its highest bit at p, so
// words are solved from the lowest priority up: the 64 rows of a word add what their
// bits in the words below select of the solved rows, through 16 tables of 16 entries per
// word (kept in LDS), then among themselves, in order, in one wavefront.  One 32-bit
// column u of the four of the output word (they are independent: the members share them
// out).  Eight lanes share a row, so its words are read in order; the next word's rows
// load meanwhile.  Bound by the latency of a word's steps.
__device__ __forceinline__ void solve_map(const FitArgs& a, const CtxDesc& ds, WideShared& L, const uint64_t* X, int u) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = ds.n, d = n + 1, fw = feat_words(n), W = fw + F2_Y_WORDS, cw = n >> 6;
    uint32_t* zt = reinterpret_cast<uint32_t*>(&L.tab[0][0][0]);                // [64][kPitch] tables
    constexpr int kPitch = 272;  // a word's tables start 16 banks after the last word's
    uint32_t* zf = zt + 64 * kPitch;                                            // [4096] solved
    uint64_t* ur = reinterpret_cast<uint64_t*>(zf + 4096);                      // [64] the word's own bits
    uint32_t* zr = reinterpret_cast<uint32_t*>(ur + 64);                        // [64] before the word's own steps
    uint16_t* inv = reinterpret_cast<uint16_t*>(zr + 64);                       // [4096] list index of pivot p
    static_assert(64 * kPitch * 4 + 4096 * 4 + 64 * 12 + 4096 * 2 <= static_cast<int>(sizeof(L.tab)), "fits the tables' place");
    __syncthreads();
    for (int i = tid; i < d; i += kWdThreads) inv[L.piv[i] & (kPivLast - 1)] = static_cast<uint16_t>(i);
    __syncthreads();
    const int q = lane & 7, k = 8 * wave + (lane >> 3);  // words q, q + 8, .. of row k of the word
    auto row_of = [&](int p) {
        const int idx = inv[p < d ? p : 0];
        return X + static_cast<int64_t>(idx < d ? idx : 0) * W;
    };
    const uint32_t zc = reinterpret_cast<const uint32_t*>(row_of(n) + fw)[u];  // the constant's row: its features are the constant alone
    if (tid == 0) zf[n] = zc;
    uint64_t v[8];  // each word reloaded for the next row as soon as it is used
    const uint64_t* row = row_of(k);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = row[0];
    uint64_t cn = row[cw];
    uint32_t yn = reinterpret_cast<const uint32_t*>(row + fw)[u];
    for (int w = 0; w < fw; ++w) {
        uint32_t z = q == 0 ? yn ^ (((cn >> (n & 63)) & 1ull) ? zc : 0u) : 0u;
        uint64_t own = v[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) own = (w >> 3) == i ? v[i] : own;
        const int wn = w + 1 < fw ? w + 1 : w;
        row = row_of(64 * wn + k);
        cn = row[cw];
        yn = reinterpret_cast<const uint32_t*>(row + fw)[u];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ww = 8 * i + q;
            if (8 * i > wn) break;
            if (ww < w) {
                const uint32_t* tw = zt + kPitch * ww;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const uint32_t vh = e < 8 ? static_cast<uint32_t>(v[i]) : static_cast<uint32_t>(v[i] >> 32);
                    z ^= tw[16 * e + __builtin_amdgcn_ubfe(vh, 4 * (e & 7), 4)];
                }
            }
            v[i] = row[ww <= wn ? ww : 0];
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) z ^= static_cast<uint32_t>(__shfl_xor(static_cast<int>(z), o));
        if (q == 0) zr[k] = z;
        if (q == (w & 7)) ur[k] = own;
        __syncthreads();
        if (wave == 0) {
            const bool in = 64 * w + lane < n;
            const uint64_t own = in ? ur[lane] & ~(1ull << lane) & (w == cw ? (1ull << (n & 63)) - 1 : ~0ull) : 0ull;
            uint32_t x = in ? zr[lane] : 0u;
#pragma unroll 16
            for (int bb = 0; bb < 64; ++bb) {  // bits above a row's own are zero
                const uint32_t vh = bb < 32 ? static_cast<uint32_t>(own) : static_cast<uint32_t>(own >> 32);
                const uint32_t m = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(vh), bb & 31, 1));
                x = __builtin_amdgcn_bitop3_b32(x, m, __builtin_amdgcn_readlane(x, bb), 0x78);
            }
            if (in) zf[64 * w + lane] = x;
            zr[lane] = x;
            wave_sync();
#pragma unroll
            for (int i = 0; i < 4; ++i) {  // entries 16 g + e of tables g = 4 i + lane / 16
                const int g = 4 * i + (lane >> 4);
                uint32_t e = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) e ^= ((lane >> r) & 1) ? zr[4 * g + r] : 0u;
                zt[kPitch * w + 64 * i + lane] = e;
            }
        }
        __syncthreads();
    }
    // columns of the map, and the output words of the basis rows (device-scope: other members read them)
    for (int p = tid; p < d; p += kWdThreads) {
        put_dev32(reinterpret_cast<uint32_t*>(a.maps + ds.mo + 2 * p) + u, zf[p]);
        reinterpret_cast<uint32_t*>(a.basis + ds.bo + static_cast<int64_t>(p < n ? n - 1 - p : n) * W + fw)[u] = zf[p];
    }
    __syncthreads();
}

// full rank: this member's remaining blocks (blk, blk + G, ...) lie in the span; a row's
// residual is y + M phi, from tables of the map's columns, four columns each, 32 words
// of phi (128 KB of tables) at a time.  Each thread takes up to two rows.
__device__ __forceinline__ void check_rows(const FitArgs& a, const CtxDesc& ds, WideShared& L, int blk, int G, int nblk,
                                           int& ncon, long long& firstc) {
    const int tid = threadIdx.x;
    const int n = ds.n, d = n + 1, fw = feat_words(n), W = fw + F2_Y_WORDS;
    const uint64_t tmask = top_mask(n, fw);
    const u32x4_a8* M = reinterpret_cast<const u32x4_a8*>(a.maps + ds.mo);
    u32x4* tab = &L.tab[0][0][0];  // [512][16]
    constexpr int kRowsPer = 2, kStep = kRowsPer * kWdWaves;  // blocks per pass
    for (int b0 = blk; b0 < nblk; b0 += kStep * G) {
        const uint64_t* row[kRowsPer];
        int64_t ri[kRowsPer];
        u32x4 z[kRowsPer];
#pragma unroll
        for (int k = 0; k < kRowsPer; ++k) {
            const int bk = b0 + G * (kWdWaves * k + (tid >> 6));
            ri[k] = bk < nblk ? static_cast<int64_t>(bk) * kWdRows + (tid & 63) : ds.m;
            row[k] = a.rows + ds.row0 + (ri[k] < ds.m ? ri[k] : 0) * W;
            z[k] = *reinterpret_cast<const u32x4_a8*>(row[k] + fw);
        }
        for (int w0 = 0; w0 < fw; w0 += 32) {
            __syncthreads();
            if (64 * w0 + 4 * tid < d) {
                u32x4 c[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = 64 * w0 + 4 * tid + q;
                    c[q] = u32x4{0, 0, 0, 0};
                    if (col < d) c[q] = M[col];
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    u32x4 v = {0, 0, 0, 0};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if ((e >> q) & 1) v ^= c[q];
                    tab[16 * tid + (e ^ (tid & 15))] = v;  // entries rotated by the table: fewer bank conflicts
                }
            } else {
                tab[16 * tid + (tid & 15)] = u32x4{0, 0, 0, 0};  // no columns: entry 0 is read all the same
            }
            __syncthreads();
            const int wend = w0 + 32 < fw ? w0 + 32 : fw;
            uint64_t nx[kRowsPer];
            auto load_word = [&](int w) {
#pragma unroll
                for (int k = 0; k < kRowsPer; ++k) nx[k] = row[k][w] & (w == fw - 1 ? tmask : ~0ull);
            };
            load_word(w0);
            for (int w = w0; w < wend; ++w) {  // (a row's cache line serves sixteen steps)
                uint64_t v[kRowsPer];
#pragma unroll
                for (int k = 0; k < kRowsPer; ++k) v[k] = nx[k];
                load_word(w + 1 < wend ? w + 1 : w);
                const u32x4* tw = tab + 256 * (w - w0);
#pragma unroll
                for (int q = 0; q < 16; q += 2)
#pragma unroll
                    for (int k = 0; k < kRowsPer; ++k)
                        z[k] = xor3_4(z[k], tw[16 * q + ((static_cast<uint32_t>(v[k] >> (4 * q)) & 15u) ^ q)],
                                      tw[16 * q + 16 + ((static_cast<uint32_t>(v[k] >> (4 * q + 4)) & 15u) ^ (q + 1))]);
            }
        }
#pragma unroll
        for (int k = 0; k < kRowsPer; ++k)
            if (ri[k] < ds.m && any4(z[k])) {
                ++ncon;
                if (ri[k] < firstc) firstc = ri[k];
            }
    }
}

// member g of the G workgroups that fit context ds together
__device__ __forceinline__ void fit_ctx_wide(const FitArgs& a, const CtxDesc& ds, WideShared& L, int G, int g, int32_t* prog) {
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = ds.c, n = ds.n, d = n + 1, fw = feat_words(n), W = fw + F2_Y_WORDS, cw = n >> 6;
    const int64_t m = ds.m;
    const uint64_t* R = a.rows + ds.row0;
    const uint64_t tmask = top_mask(n, fw), cbit = 1ull << (n & 63);
    uint64_t* Xp = a.tables + ds.bo;
    const __amdgpu_buffer_rsrc_t X = dev_rsrc(Xp, static_cast<uint32_t>(8 * d * W));
    const __amdgpu_buffer_rsrc_t Y = dev_rsrc(a.basis + ds.bo, static_cast<uint32_t>(8 * d * W));  // merged chunks
    int32_t* ent = a.pivots + ds.po;
    constexpr long long kNone = 0x7fffffffffffffffll;
    const int nblk = m > static_cast<int64_t>(kWdMaxBlocks) * kWdRows ? 0x7fffffff : static_cast<int>((m + kWdRows - 1) / kWdRows);
    if (nblk > kWdMaxBlocks) {  // block numbers past the tags: one member, which reads no tags
        if (g != 0) return;
        G = 1;
    }
    const int64_t blocks = (m + kWdRows - 1) / kWdRows;
    // valid bits of words 2 j and 2 j + 1, and the constant's bit
    const uint64_t v0 = 2 * j < fw ? (2 * j == fw - 1 ? tmask : ~0ull) : 0ull;
    const uint64_t v1 = 2 * j + 1 < fw ? (2 * j + 1 == fw - 1 ? tmask : ~0ull) : 0ull;
    const u32x4 vm = {static_cast<uint32_t>(v0), static_cast<uint32_t>(v0 >> 32), static_cast<uint32_t>(v1),
                      static_cast<uint32_t>(v1 >> 32)};
    auto load_block = [&](int64_t bk, BlockRows& b) {
        const uint64_t* rb = R + bk * kWdRows * W;
        const int nb = m - bk * kWdRows < kWdRows ? static_cast<int>(m - bk * kWdRows) : kWdRows;
#pragma unroll
        for (int i = 0; i < kWdPairs; ++i) {
            const int r = 8 * wave + 2 * i + h;
            b.acc[i] = *reinterpret_cast<const u32x4_a8*>(rb + static_cast<int64_t>(r < nb ? r : 0) * W + (2 * j < fw ? 2 * j : 0));
        }
        const int r = 8 * wave + (lane & 7);
        b.y = *reinterpret_cast<const u32x4_a8*>(rb + static_cast<int64_t>(r < nb ? r : 0) * W + fw);
    };
    if (tid == 0) {
        L.timeout = 0;
        L.nrows = 0;
        L.next = 0;
        L.any[0] = L.any[1] = 0;
        L.more = 0;
        L.merged = 0;
    }
    __syncthreads();
    int nrows = 0;
    int ncon = 0;
    long long firstc = kNone;
    int flip = 0;
    // one pass of this loop: a block of this member (phase 0), a chunk of the list that its new
    // rows completed, to be merged (phase 2), then, below full rank, a batch of the list
    // (phase 1) to be reduced by the later ones
    int phase = 0, bpos = 0, bidx = 0, bK = 0;
    int64_t blk = g;
    bool full = false;
    BlockRows nextb;  // the next block's rows, loaded ahead
    if (blk < blocks) load_block(blk, nextb);
    // wavefront 0: wait until every block below `until` is done (or, with bar > 0, every member
    // past that barrier), then take the list's new entries
    auto wait_for = [&](int64_t until, int bar) {
        if (wave == 0) {
            int open = 0;
            bool ok = false;
            if (!L.timeout) {
                for (int spin = 0; spin < a.spin_limit; ++spin) {
                    if (bar) {
                        bool behind = false;
                        if (lane < G && lane != g) {
                            behind = __hip_atomic_load(prog + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < kWdBar + bar;
                        }
                        ok = __ballot(behind) == 0;
                    } else {
                        open = lowest_open(prog, G, g, static_cast<int>(until));
                        ok = open >= until;
                    }
                    if (ok) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                if (!ok && lane == 0) L.timeout = 1;
            }
            if (bar) open = 0x7fffffff;
            if (bar < 2) {
                const int k = take_entries(L, ent, nrows, d, open);
                mark_chunks(L, nrows, k);
                if (lane == 0) L.nrows = k;
            }
        }
        __syncthreads();
        nrows = __builtin_amdgcn_readfirstlane(L.nrows);
    };
    auto end_block = [&]() {
        blk += G;
        if (G > 1 && tid == 0) put_progress(prog, g, static_cast<int>((blk - g) / G));
        if (blk < blocks) load_block(blk, nextb);
    };
    // what the members have written.  One workgroup alone needs no cache cleared for its own
    // (2,000 contexts of 513 columns and up to 3 rows: 341 us with the die's L2 invalidated twice for each, 215 without)
    auto acquire = [&]() {
        if (G > 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    for (;;) {
        if (phase == 0 && (blk >= blocks || nrows >= d)) {
            bpos = 0;
            if (G > 1) {  // every member past its blocks: the list is complete
                __syncthreads();
                if (tid == 0) put_progress(prog, g, kWdBar + 1);
                wait_for(0, 1);
            }
            if (__builtin_amdgcn_readfirstlane(L.merged)) {  // merged chunks to their places in the list (the outputs go where they are)
                const uint64_t* const Yp = a.basis + ds.bo;
                for (int q = 0; q < nrows / kChunk; ++q) {
                    if (!(L.piv[kChunk * q] & kPivMerged)) continue;
                    if (q % G == g)
                        for (int i = kChunk * q * W + tid; i < kChunk * (q + 1) * W; i += kWdThreads)
                            put_dev(Xp + i, __hip_atomic_load(Yp + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
                __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                for (int q = tid; q < nrows / kChunk; q += kWdThreads) L.piv[kChunk * q] &= ~kPivMerged;
                if (G > 1) {
                    if (tid == 0) put_progress(prog, g, kWdBar + 2);
                    wait_for(0, 2);
                }
            }
            acquire();  // no line of the list read before it was whole is read again
            phase = 1;
            full = nrows >= d;
            // pivot columns and the counts above each word (descending-priority positions)
            if (tid < 64) L.pm[tid] = 0;
            __syncthreads();
            for (int i = tid; i < nrows; i += kWdThreads) {
                const int p = L.piv[i] & (kPivLast - 1);
                atomicOr(reinterpret_cast<unsigned long long*>(&L.pm[p >> 6]), 1ull << (p & 63));
            }
            __syncthreads();
            if (wave == 0) {
                const uint64_t v = L.pm[lane] & ((lane == cw) ? ~cbit : ~0ull);
                const int cnt = lane < fw ? __popcll(v) : 0;
                int x = cnt;
                for (int o = 1; o < 64; o <<= 1) {
                    const int t = __shfl_down(x, o);
                    if (lane + o < 64) x += t;
                }
                L.above[lane] = x - cnt;
            }
            __syncthreads();
            if (full) break;
        }
        if (phase == 1) {  // the next batch of this member: every G-th
            bool found = false;
            while (bpos < nrows) {
                const bool in = bpos + lane < nrows;
                const uint64_t last = __ballot(in && (L.piv[in ? bpos + lane : 0] & kPivLast));
                const int left = nrows - bpos < 64 ? nrows - bpos : 64;
                const int k = last ? ffs64(last) + 1 : 64;
                bK = k < left ? k : left;
                if (bidx % G == g) {
                    found = true;
                    break;
                }
                bpos += bK;
                ++bidx;
            }
            if (!found) break;
        }
        BlockRows b;
        const int nb = phase ? bK : (m - blk * kWdRows < kWdRows ? static_cast<int>(m - blk * kWdRows) : kWdRows);
        if (phase == 0) {
            b = nextb;
        } else {
            const int voff = 16 * (2 * j < fw ? j : 0);
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) {
                const int r = 8 * wave + 2 * i + h;
                b.acc[i] = load16<true>(X, (bpos + (r < nb ? r : 0)) * W * 8 + voff, 0);
            }
            const int r = 8 * wave + (lane & 7);
            b.y = load16<true>(X, ((bpos + (r < nb ? r : 0)) * W + fw) * 8, 0);
        }
#pragma unroll
        for (int i = 0; i < kWdPairs; ++i) b.acc[i] &= vm & (8 * wave + 2 * i + h < nb ? ~0u : 0u);
        b.y &= lane < 8 && 8 * wave + lane < nb ? ~0u : 0u;
        // phase 2: a row without its own pivot's bit selects the later rows of the chunk alone
        auto flip_own = [&]() {
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) {
                const int r = 8 * wave + 2 * i + h;
                const int p = L.piv[bpos + (r < nb ? r : 0)] & (kPivLast - 1);
                const uint32_t bit = r < nb && (p >> 7) == j ? 1u << (p & 31) : 0u;
#pragma unroll
                for (int k = 0; k < 4; ++k) b.acc[i][k] ^= ((p >> 5) & 3) == k ? bit : 0u;
            }
        };
        if (phase == 2) flip_own();
        if (phase == 0 && G > 1) {  // what the other members have added meanwhile
            if (wave == 0) {
                const int open = lowest_open(prog, G, g, static_cast<int>(blk));
                const int k = take_entries(L, ent, nrows, d, open);
                mark_chunks(L, nrows, k);
                if (lane == 0) {
                    L.nrows = k;
                    L.next = open;
                }
            }
            __syncthreads();
            nrows = __builtin_amdgcn_readfirstlane(L.nrows);
        }
        int pos = phase == 1 ? bpos + bK : phase == 2 ? bpos : 0;
        const int past = bpos + bK;  // phase 2: the end of the chunk
        int open = G > 1 && phase == 0 ? __builtin_amdgcn_readfirstlane(L.next) : 0x7fffffff;
        bool anynz = false;
        for (;;) {
            if (pos < nrows) {
                wide_reduce(L, X, Y, W, d, pos, phase == 2 ? past : nrows, b);
                pos = nrows;
            } else {
#pragma unroll
                for (int o = 8; o < 64; o <<= 1) b.y ^= shfl_xor4(b.y, o);
            }
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) b.acc[i] &= vm;  // (the lanes past the row collected other words)
            if (phase) break;
            bool mine = false;
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) mine |= any4(b.acc[i]);
            if (__ballot(mine) && lane == 0) L.any[flip] = 1;
            if (tid == 0) L.any[flip ^ 1] = 0;
            __syncthreads();
            anynz = __builtin_amdgcn_readfirstlane(L.any[flip]) != 0;
            flip ^= 1;
            if (!anynz || open >= blk) break;
            wait_for(blk, 0);  // (ends the phase: every earlier block is done)
            open = 0x7fffffff;
            if (pos == nrows) break;
            b.y &= lane < 8 ? ~0u : 0u;
            // (a chunk merged since the block was reduced by its first rows: whole, which these no longer select)
            const int q = pos / kChunk;
            if (__builtin_amdgcn_readfirstlane(L.piv[kChunk * q]) & kPivMerged) pos = kChunk * q;
        }
        if (phase == 2) {
            flip_own();
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) {
                const int r = 8 * wave + 2 * i + h;
                const int off = (bpos + r) * W * 8 + 16 * j;
                if (r < nb) {
                    if (2 * j + 1 < fw) __builtin_amdgcn_raw_buffer_store_b128(b.acc[i], Y, off, 0, kDevScope);
                    else if (2 * j < fw) __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{b.acc[i].x, b.acc[i].y}, Y, off, 0, kDevScope);
                }
            }
            const int r = 8 * wave + lane;
            if (lane < 8 && r < nb) __builtin_amdgcn_raw_buffer_store_b128(b.y, Y, ((bpos + r) * W + fw) * 8, 0, kDevScope);
            __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (wave == 0) mark_chunks(L, bpos, nrows);
            __syncthreads();
            phase = 0;
            end_block();
            continue;
        }
        if (phase == 1) {  // fully reduced rows to their final places
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) {
                const int r = 8 * wave + 2 * i + h;
                if (r < nb) {
                    const int p = L.piv[bpos + r] & (kPivLast - 1);
                    int k = nrows - 1;
                    if (p != n) {
                        uint64_t v = L.pm[p >> 6];
                        if ((p >> 6) == cw) v &= ~cbit;
                        v &= (p & 63) == 63 ? 0ull : (~0ull << ((p & 63) + 1));
                        k = L.above[p >> 6] + __popcll(v);
                    }
                    uint64_t* out = a.basis + ds.bo + static_cast<int64_t>(k) * W;
                    if (2 * j < fw) put_dev(out + 2 * j, (static_cast<uint64_t>(b.acc[i].y) << 32) | b.acc[i].x);
                    if (2 * j + 1 < fw) put_dev(out + 2 * j + 1, (static_cast<uint64_t>(b.acc[i].w) << 32) | b.acc[i].z);
                }
            }
            const int r = 8 * wave + lane;
            if (lane < 8 && r < nb) {
                const int p = L.piv[bpos + r] & (kPivLast - 1);
                int k = nrows - 1;
                if (p != n) {
                    uint64_t v = L.pm[p >> 6];
                    if ((p >> 6) == cw) v &= ~cbit;
                    v &= (p & 63) == 63 ? 0ull : (~0ull << ((p & 63) + 1));
                    k = L.above[p >> 6] + __popcll(v);
                }
                uint64_t* out = a.basis + ds.bo + static_cast<int64_t>(k) * W + fw;
                const uint64_t y0 = (static_cast<uint64_t>(b.y.y) << 32) | b.y.x, y1 = (static_cast<uint64_t>(b.y.w) << 32) | b.y.z;
                out[0] = y0;
                out[1] = y1;
                a.maps[ds.mo + 2 * p] = y0;
                a.maps[ds.mo + 2 * p + 1] = y1;
            }
            bpos += bK;
            ++bidx;
            __syncthreads();
            continue;
        }
        // (3) elimination in stream order on panels
        const int before = nrows;
        uint64_t ins = 0;
        if (anynz && nrows < d) {
            u32x4* const Rm = &L.tab[0][0][0];                         // [64][kRowPitch]
            u32x4* const ET = &L.tab[0][0][0] + kWdRows * kRowPitch;   // [128][32]: 8 tables
            uint64_t pend = ~0ull;  // wavefront 0: rows not yet basis rows
            int mypiv = 0;
            for (;;) {
                // the rows, and which words the pending ones hold (the constant apart)
                uint32_t ev = 0, od = 0;
#pragma unroll
                for (int i = 0; i < kWdPairs; ++i) {
                    const int r = 8 * wave + 2 * i + h;
                    Rm[r * kRowPitch + j] = b.acc[i];
                    const bool pe = !((ins >> r) & 1ull);
                    const uint64_t w0 = ((static_cast<uint64_t>(b.acc[i].y) << 32) | b.acc[i].x) & (2 * j == cw ? ~cbit : ~0ull);
                    const uint64_t w1 = ((static_cast<uint64_t>(b.acc[i].w) << 32) | b.acc[i].z) & (2 * j + 1 == cw ? ~cbit : ~0ull);
                    const uint64_t be = __ballot(pe && w0 != 0), bo = __ballot(pe && w1 != 0);
                    ev |= static_cast<uint32_t>(be) | static_cast<uint32_t>(be >> 32);
                    od |= static_cast<uint32_t>(bo) | static_cast<uint32_t>(bo >> 32);
                    if (__ballot(pe && any4(b.acc[i])) && lane == 0) L.more = 1;
                }
                if (lane < 8) L.ys[8 * wave + lane] = b.y;
                if (lane == 0) {
                    L.wm[wave][0] = ev;
                    L.wm[wave][1] = od;
                }
                __syncthreads();
                if (!__builtin_amdgcn_readfirstlane(L.more)) break;  // no pending row holds a bit
                if (wave == 0) {
                    uint32_t v = lane < 2 * kWdWaves ? (&L.wm[0][0])[lane] : 0u;
                    for (int o = 2; o < 32; o <<= 1) v |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), o));
                    uint32_t ue = __builtin_amdgcn_readlane(v, 0), uo = __builtin_amdgcn_readlane(v, 1);
                    auto top_word = [&]() {  // the highest nonzero word, taken out; -1: none
                        const int te = ue ? 2 * (31 - __builtin_clz(ue)) : -1, to = uo ? 2 * (31 - __builtin_clz(uo)) + 1 : -1;
                        if (te > to) ue &= ~(1u << (te >> 1));
                        else if (to >= 0) uo &= ~(1u << (to >> 1));
                        return te > to ? te : to;
                    };
                    const uint64_t* Rw = reinterpret_cast<const uint64_t*>(Rm) + lane * (2 * kRowPitch);
                    const int wa = top_word(), wb = top_word();
                    uint64_t va, vb = 0;
                    if (wa >= 0) {
                        va = Rw[wa] & (wa == cw ? ~cbit : ~0ull);
                        if (wb >= 0) vb = Rw[wb];
                    } else {
                        va = (Rw[cw] & cbit) ? 1ull : 0ull;  // only the constant is left
                    }
                    // a column per lane (bit q: row q), so that a row's bits are one ballot and the
                    // rows that hold a pivot are one lane's word: row after row, a row with a bit in
                    // the panel takes its highest as pivot and is added to the other rows that hold it
                    const uint64_t todo = __ballot((va | vb) != 0) & pend;  // (rows without a bit get none)
                    va = transpose64(va, lane);
                    vb = transpose64(vb, lane);
                    uint64_t T = 1ull << lane, now = 0;
                    auto half_rows = [&](uint32_t left, auto hi) {  // rows 0-31 or 32-63
                        constexpr int sft = decltype(hi)::value ? 32 : 0;
                        auto bit_of = [&](uint64_t v, int q) {
                            return static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(static_cast<uint32_t>(v >> sft)), q, 1));
                        };
                        auto pivot = [&](int q, int word, uint64_t bits, uint64_t& v, uint64_t& v2) {
                            const int bit = 63 - __builtin_clzll(bits);
                            const uint64_t self = 1ull << (q + sft);
                            const uint64_t col = readlane64(v, bit) & ~self;  // rows to clear
                            const uint32_t m = bit_of(v, q), m2 = bit_of(v2, q), mt = bit_of(T, q);
                            v = xor_and(v, m, col);
                            v2 = xor_and(v2, m2, col);
                            T = xor_and(T, mt, col);
                            mypiv = lane == q + sft ? 64 * word + bit : mypiv;
                            now |= self;
                        };
                        while (left) {  // (kept small: code run once is bound by its own fetch)
                            const int q = __builtin_ctz(left);
                            left &= left - 1;
                            const uint64_t ra = __ballot(bit_of(va, q) != 0);
                            if (ra) {
                                pivot(q, wa, ra, va, vb);
                            } else {
                                const uint64_t rb = __ballot(bit_of(vb, q) != 0);
                                if (rb) pivot(q, wb, rb, vb, va);
                            }
                        }
                    };
                    half_rows(static_cast<uint32_t>(todo), std::false_type{});
                    half_rows(static_cast<uint32_t>(todo >> 32), std::true_type{});
                    if (wa < 0) mypiv = ((now >> lane) & 1ull) ? n : mypiv;
                    pend &= ~now;
                    L.T[lane] = transpose64(T, lane);
                    if (lane == 0) L.panel = now;
                }
                __syncthreads();
                if (tid == 0) L.more = 0;  // (read by all before the barrier above)
                const uint64_t now = L.panel;
                const uint64_t nowu = readlane64(now, 0);
                uint64_t tl[kWdPairs];
#pragma unroll
                for (int i = 0; i < kWdPairs; ++i) tl[i] = L.T[8 * wave + 2 * i + h];
                const uint64_t ty = L.T[8 * wave + (lane & 7)];
                if (__popcll(nowu) <= 12) {  // few new rows: each added where T says so
                    uint64_t left = nowu;
                    u32x4 na[kWdPairs], ny = b.y & bit_mask(ty, 8 * wave + (lane & 7));
#pragma unroll
                    for (int i = 0; i < kWdPairs; ++i) na[i] = b.acc[i] & bit_mask(tl[i], 8 * wave + 2 * i + h);
                    while (left) {
                        const int q = ffs64(left);
                        left &= left - 1;
                        const u32x4 f = Rm[q * kRowPitch + j], z = L.ys[q];
#pragma unroll
                        for (int i = 0; i < kWdPairs; ++i)  // (the row itself is in already)
                            na[i] = xor_and4(na[i], (8 * wave + 2 * i + h == q) ? 0u : bit_mask(tl[i], q), f);
                        ny = xor_and4(ny, (8 * wave + (lane & 7) == q) ? 0u : bit_mask(ty, q), z);
                    }
#pragma unroll
                    for (int i = 0; i < kWdPairs; ++i) b.acc[i] = na[i];
                    b.y = ny;
                } else {
                    u32x4 na[kWdPairs], ny = {0, 0, 0, 0};
#pragma unroll
                    for (int i = 0; i < kWdPairs; ++i) na[i] = u32x4{0, 0, 0, 0};
#pragma unroll 1
                    for (int hf = 0; hf < 2; ++hf) {  // 32 rows, 8 tables at a time
                        const u32x4* f = Rm + (32 * hf + 4 * wave) * kRowPitch + j;
                        const u32x4 f0 = f[0], f1 = f[kRowPitch], f01 = f0 ^ f1;
                        const u32x4 b0 = f[2 * kRowPitch] & (h ? ~0u : 0u), b1 = b0 ^ f[3 * kRowPitch];
                        u32x4* e = ET + (16 * wave + 4 * h) * 32 + j;
                        e[0] = b0;
                        e[32] = b0 ^ f0;
                        e[64] = b0 ^ f1;
                        e[96] = b0 ^ f01;
                        e[256] = b1;
                        e[288] = b1 ^ f0;
                        e[320] = b1 ^ f1;
                        e[352] = b1 ^ f01;
                        __syncthreads();
                        uint32_t th[kWdPairs];
#pragma unroll
                        for (int i = 0; i < kWdPairs; ++i) th[i] = static_cast<uint32_t>(hf ? tl[i] >> 32 : tl[i]);
#pragma unroll
                        for (int q = 0; q < 8; q += 2)
#pragma unroll
                            for (int i = 0; i < kWdPairs; ++i)
                                na[i] = xor3_4(na[i], ET[(16 * q + __builtin_amdgcn_ubfe(th[i], 4 * q, 4)) * 32 + j],
                                               ET[(16 * q + 16 + __builtin_amdgcn_ubfe(th[i], 4 * q + 4, 4)) * 32 + j]);
                        const int ly = lane >> 3;
                        const uint32_t nib = static_cast<uint32_t>(hf ? ty >> 32 : ty) >> (4 * ly);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            ny = xor_and4(ny, static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(nib), i, 1)),
                                          L.ys[32 * hf + 4 * ly + i]);
                        __syncthreads();
                    }
#pragma unroll
                    for (int i = 0; i < kWdPairs; ++i) b.acc[i] = na[i];
#pragma unroll
                    for (int o = 8; o < 64; o <<= 1) ny ^= shfl_xor4(ny, o);
                    b.y = ny;
                }
                ins |= nowu;
                __syncthreads();  // the rows are rewritten for the next panel
            }
            // (4) publish: pivots and rows behind the list
            int K = __popcll(ins);
            if (K > d - nrows) K = d - nrows;  // (only after a wait that gave up)
            if (wave == 0) {
                const int i = __popcll(ins & ((1ull << lane) - 1));
                if (((ins >> lane) & 1ull) && i < K) {
                    const int v = mypiv | (i == K - 1 ? kPivLast : 0);
                    L.piv[nrows + i] = static_cast<uint16_t>(v);
                    if (G > 1)
                        __hip_atomic_store(ent + nrows + i, v | (static_cast<int>(blk + 1) << 13), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
                if (G > 1 && lane == 0 && nrows + K < d)
                    __hip_atomic_store(ent + nrows + K, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int i = 0; i < kWdPairs; ++i) {
                const int r = 8 * wave + 2 * i + h;
                const int k = __popcll(ins & ((1ull << r) - 1));
                if (((ins >> r) & 1ull) && k < K) {
                    const int off = (nrows + k) * W * 8 + 16 * j;
                    if (2 * j + 1 < fw) __builtin_amdgcn_raw_buffer_store_b128(b.acc[i], X, off, 0, kDevScope);
                    else if (2 * j < fw) __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{b.acc[i].x, b.acc[i].y}, X, off, 0, kDevScope);
                }
            }
            {
                const int r = 8 * wave + lane;
                const int k = lane < 8 ? __popcll(ins & ((1ull << r) - 1)) : K;
                if (lane < 8 && ((ins >> r) & 1ull) && k < K)
                    __builtin_amdgcn_raw_buffer_store_b128(b.y, X, ((nrows + k) * W + fw) * 8, 0, kDevScope);
            }
            __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's stores performed
            nrows += K;
        }
        {  // the other rows: redundant, or contradictory when an output bit is left
            const int r = 8 * wave + lane;
            const uint64_t cm = __ballot(lane < 8 && r < nb && !((ins >> r) & 1ull) && any4(b.y));
            if (cm) {
                ncon += lane == 0 ? __popcll(cm) : 0;
                const long long f = blk * kWdRows + 8 * wave + ffs64(cm);
                if (lane == 0 && f < firstc) firstc = f;
            }
        }
        if (tid == 0) L.nrows = nrows;
        __syncthreads();
        const int q = before / kChunk;  // (further chunks that the new rows completed hold them alone)
        if (nrows / kChunk > q && chunk_small(L, q)) {
            bpos = kChunk * q;
            bK = kChunk;
            phase = 2;
        } else {
            end_block();
        }
    }
    // outputs
    const int64_t po = ds.po, mo = ds.mo;
    const int rank = nrows;
    if (full) {
        for (int u = g; u < 4; u += G) solve_map(a, ds, L, Xp, u);
        uint64_t* B = a.basis + ds.bo;
        for (int k = kWdWaves * g + wave; k < d; k += kWdWaves * G) {
            const int p = k < n ? n - 1 - k : n;
            if (lane < fw) B[static_cast<int64_t>(k) * W + lane] = lane == (p >> 6) ? 1ull << (p & 63) : 0ull;
        }
    } else {
        for (int p = kWdThreads * g + tid; p < d; p += kWdThreads * G)
            if (!((L.pm[p >> 6] >> (p & 63)) & 1ull)) {
                a.maps[mo + 2 * p] = 0;
                a.maps[mo + 2 * p + 1] = 0;
            }
    }
    // every member's part of the map and the basis written (what others read of it at
    // device scope: a release fence would write back a whole L2); the list is dead
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (G > 1) {
        if (tid == 0) put_progress(prog, g, kWdBar + 3);
        wait_for(0, 3);
    }
    acquire();
    if (full) {
        if (blk < blocks) check_rows(a, ds, L, static_cast<int>(blk), G, static_cast<int>(blocks), ncon, firstc);
    } else if (has_parity_rows(d, rank)) {
        // parity-check rows of the free columns: per word pair (w, v), a bit-matrix transpose of
        // word w of the basis rows of pivots 64 v .. 64 v + 63 (zero for free columns) gives lane f
        // word v of the row of free column 64 w + f
        const uint64_t lane_lt = (1ull << lane) - 1;
        const uint64_t* B = a.basis + ds.bo;
        int base = 0;  // free columns in the words before w
        for (int w = 0; w < fw; ++w) {
            const uint64_t fr = ~L.pm[w] & (w == fw - 1 ? tmask : ~0ull);
            if (!fr) continue;
            const bool mine = (fr >> lane) & 1ull;
            const int64_t i = base + __popcll(fr & lane_lt);
            for (int v = kWdWaves * g + wave; v < fw; v += kWdWaves * G) {
                const uint64_t pv = L.pm[v];
                const bool piv = (pv >> lane) & 1ull;
                int k = rank - 1;
                if (64 * v + lane != n) {
                    uint64_t hi = pv & (v == cw ? ~cbit : ~0ull);
                    hi &= lane == 63 ? 0ull : (~0ull << (lane + 1));
                    k = L.above[v] + __popcll(hi);
                }
                const uint64_t col = transpose64(piv ? B[static_cast<int64_t>(k) * W + w] : 0ull, lane);
                if (mine) Xp[i * fw + v] = col | (v == w ? (1ull << lane) : 0ull);
            }
            base += __popcll(fr);
        }
    }
    if (g == 0) {
        for (int i = tid; i < rank; i += kWdThreads) {
            const int p = L.piv[i] & (kPivLast - 1);
            int k = rank - 1;
            if (p != n) {
                uint64_t v = L.pm[p >> 6];
                if ((p >> 6) == cw) v &= ~cbit;
                v &= (p & 63) == 63 ? 0ull : (~0ull << ((p & 63) + 1));
                k = L.above[p >> 6] + __popcll(v);
            }
            if (k < d) a.pivots[po + k] = p;
        }
        if (tid == 0) a.rank[c] = rank;
    }
    // contradictions: counted by every member (the plan cleared the words)
    if (ncon) {
        atomicAdd(&a.n_contra[c], ncon);
        atomicMin(reinterpret_cast<unsigned long long*>(&a.first_contra[c]), static_cast<unsigned long long>(firstc));
        atomicOr(&a.ctx_flags[c], F2_CTX_CONTRADICTION);
    }
    if (tid == 0 && L.timeout) atomicOr(&a.ctx_flags[c], F2_CTX_SYNC_TIMEOUT);
    __syncthreads();
}

// One workgroup of kRegWaves wavefronts per compute unit, each wavefront fitting its own
// contexts in its own LDS region, largest first.  The first kPivWaves of a workgroup start
// with contexts that need more: the group ones and the long ones, one per workgroup, fitted by the
// four together (their LDS regions are one PivShared), then those of four feature words, one
// each in a larger region (piv_lists).  These are chains of 100-200 us that once ran in a kernel of their
// own behind this one and left the chip idle; here the other wavefronts work beside them.
// A wavefront runs a pipeline over its contexts: while one is in its last block, the next one's
// first rows, the descriptor of the one after and the list entry of the third are loading.
// A descriptor is one load, a dword per lane.  Bound by the elimination's chain (some 400
// cycles a pivot with four wavefronts on a SIMD, half of the time), then by the record by
// record reduce.  A corpus of 80,000 contexts: 207 us; the former kernels, one after the
// other, 170 us (contexts of up to 256 rows) and 264 us (the rest).
constexpr int kRegWaves = 16;
constexpr int kRegGrid = 256;

// a workgroup's part of the list
struct RegQueue {
    unsigned long long tail;  // of the shared tail: the next list index, and in the upper half where the chunk ends
    int next;                 // next position of the workgroup's share
    int done;                 // the tail has ended
};
// Which kernel takes the long, one and group contexts.
// - Where k_fit_reg has a workgroup for each, its first wavefronts fit them together: beside
//   short contexts that end sooner, a long one by one wavefront would be the batch's time
//   (4,000 contexts of 60 rows, 41 columns and 20 of 4,000 rows, 31 columns: 67 us, with one
//   wavefront for each of the 20 107).
// - Else the long ones go to one wavefront each beside the others, if four-word contexts, the longest
//   chains of one wavefront, run there anyway and k_fit_reg is full (3,000 contexts of 60-250 columns, 180 of
//   them long, 819 of four words: 295 us, in k_fit_piv 385; a corpus of 7,000: 150 and 203), or
//   if they are more than k_fit_piv holds at once (1,000 of 500 rows, 98 columns among 4,000: 73
//   us, in k_fit_piv behind them 114).  Otherwise they would end last (300 of 1,300 rows, 98
//   columns among 8,000: 143 us beside them, 81 in k_fit_piv), also where the short ones are too few
//   (1,000 contexts of 17-97 columns and 2,000 rows: 166 and 97 us).
// - Those of four words go singly with them (1,000 of 201 columns and 240 rows: 117 us, 255 in
//   k_fit_piv), but for a batch of mostly long ones that k_fit_piv holds at once (300 of 221
//   columns and 500 rows: 181 us singly, 145 there; 1,000: 184 and 315).
// - Of more group contexts than workgroups, up to twice as many, k_fit_reg takes the largest where it is
//   full anyway (a corpus of 200,000, 384 of them: 550 us, 620 with all in k_fit_piv), else none (600
//   of 301 columns: 144 us in k_fit_piv, where three workgroups share a compute unit; 7,400 among 15,000:
//   970 and 797 us).
// - A few short ones go to k_fit_piv with the rest (500 contexts of 17-97 columns, 20 rows a
//   column, 75 of them short: 53 us, 70 with the short ones before the others).
struct PivLists {
    int short_lo, short_n, long_lo, long_n;            // k_fit_reg: by one wavefront each
    int one_lo, one_n;                                 // by its first wavefronts, singly
    int group_lo, group_n, chain_lo, chain_n;          // and together: of the group list, of the long lists
    int piv_group_lo, piv_group, piv_one, piv_long, piv_short;  // k_fit_piv: how many of each, in this order
};
__device__ __forceinline__ PivLists piv_lists(const FitArgs& a) {
    const int G = a.num_ctx < kRegGrid ? a.num_ctx : kRegGrid;  // k_fit_reg's workgroups
    PivLists p;
    p.short_lo = a.plan[kClsShort];
    p.chain_lo = a.plan[kClsLong];
    p.group_lo = a.plan[kClsGroup];
    const int four_lo = a.plan[kClsOneLong], one_lo = a.plan[kClsOne];
    p.short_n = p.chain_lo - p.short_lo;
    const int nl = four_lo - p.chain_lo, nf = one_lo - four_lo, no = p.group_lo - one_lo, ng = a.plan[kClsLarge] - p.group_lo;
    const bool each = ng + nl + nf <= G, busy = p.short_n + kPivWaves * (nf + no) >= kRegWaves * G;
    p.chain_n = each ? nl + nf : 0;
    p.long_lo = p.chain_lo;  // (one list or the other)
    const int rest = each ? 0 : nl;
    const bool lone = !each && nf > no && ng + nf + no <= 3 * G && p.short_n <= (ng + nl + nf + no) / 4;
    const bool beside = !lone && (rest == 0 || (rest <= p.short_n / 4 && (rest > 3 * G || (busy && nf + no > 0))));
    p.group_n = !beside ? 0 : ng <= G ? ng : busy && ng <= 2 * G ? G : 0;
    p.long_n = beside ? rest : 0;
    p.one_lo = each ? one_lo : four_lo;
    const int ones = each ? no : nf + no;
    p.one_n = beside ? ones : 0;
    p.piv_group_lo = p.group_lo + p.group_n;
    p.piv_group = ng - p.group_n;
    p.piv_one = ones - p.one_n;
    p.piv_long = rest - p.long_n;
    p.piv_short = !beside && p.short_n <= (ng + nl + nf + no) / 4 ? p.short_n : 0;
    p.short_n -= p.piv_short;
    return p;
}

__global__ __launch_bounds__(64 * kRegWaves) void k_fit_reg(FitArgs a) {
    __shared__ union {
        PivShared piv;
        uint64_t basis[kPivWaves][reg_words(kRegMaxFW + 1)];
    } sPart;
    __shared__ __align__(16) uint64_t sBasis[kRegWaves - kPivWaves][kRegRec];
    __shared__ RegQueue sQueue;
    __shared__ int sWait;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // the first kPivWaves wavefronts first fit contexts of the other classes, where these are
    // few: long and wide ones together, those of 4 feature words one each
    const int g = static_cast<int>(blockIdx.x), G = static_cast<int>(gridDim.x);
    const PivLists pl = piv_lists(a);
    const int cnt = pl.long_n + pl.short_n;
    const int groups = pl.group_n + pl.chain_n;
    const bool parted = g < groups || G - 1 - g < pl.one_n;
    if (!parted && cnt == 0) return;
    if (tid == 0) {
        sQueue.next = parted ? kRegWaves - kPivWaves : kRegWaves;
        sQueue.tail = 0;
        sQueue.done = 0;
        sWait = 0;
    }
    __syncthreads();
    // the others start with one context each, in snake order over the four SIMDs
    // (wavefront w runs on SIMD w mod 4), largest first
    const int r = (wave >> 2) - (parted ? 1 : 0), simd = wave & 3;
    int start = 4 * r + ((r & 1) ? 3 - simd : simd);
    if (wave < kPivWaves && parted) {
        PartSync<kPivWaves> sync{&sWait, 0};
        __builtin_amdgcn_s_setprio(3);
        if (g < groups) {
            const int c = __builtin_amdgcn_readfirstlane(
                a.plan[kPlanHead + (g < pl.group_n ? pl.group_lo + g : pl.chain_lo + g - pl.group_n)]);
            const CtxDesc ds = readlane_desc(load_desc(a, c), 0);
            switch (feat_words(ds.n)) {
                case 1: fit_ctx_piv<1, kPivWaves>(a, ds, sPart.piv, sync); break;
                case 2: fit_ctx_piv<2, kPivWaves>(a, ds, sPart.piv, sync); break;
                case 3: case 4: fit_ctx_piv<4, kPivWaves>(a, ds, sPart.piv, sync); break;
                case 5: fit_ctx_piv<5, kPivWaves>(a, ds, sPart.piv, sync); break;
                case 6: fit_ctx_piv<6, kPivWaves>(a, ds, sPart.piv, sync); break;
                default: fit_ctx_piv<8, kPivWaves>(a, ds, sPart.piv, sync); break;
            }
        }
        // (workgroups that had no group context come first)
        for (int64_t i = wave * G + G - 1 - g; i < pl.one_n; i += kPivWaves * G) {
            const int c = __builtin_amdgcn_readfirstlane(a.plan[kPlanHead + pl.one_lo + i]);
            const CtxDesc ds = readlane_desc(load_desc(a, c), 0);
            fit_ctx_alone<kRegMaxFW + 1>(a, ds, sPart.basis[wave]);
        }
        __builtin_amdgcn_s_setprio(0);
        if (lane == 0) start = atomicAdd(&sQueue.next, 1);
        start = __builtin_amdgcn_readfirstlane(start);
    }
    uint64_t* basis = wave < kPivWaves ? sPart.basis[wave] : sBasis[wave - kPivWaves];
    // the share's list positions (the class bounds read once)
    // the list: the long contexts, then the short ones
    const int32_t* const longs = a.plan + kPlanHead + pl.long_lo;
    const int32_t* const shorts = a.plan + kPlanHead + pl.short_lo - pl.long_n;
    auto list = [&](int e) { return (e < pl.long_n ? longs : shorts)[e]; };
    const RegScalars sc = reg_scalars(a);
    // lane's dword of a context's descriptor: n; row_off of the context (2) and of the next
    // (low half: the difference of the class's contexts fits); basis, pivot and map offsets
    const char* src = reinterpret_cast<const char*>(lane < 1   ? a.n_bits
                                                    : lane < 3 ? reinterpret_cast<const int32_t*>(a.row_off) + (lane - 1)
                                                    : lane < 4 ? reinterpret_cast<const int32_t*>(a.row_off) + 2
                                                    : lane < 6 ? reinterpret_cast<const int32_t*>(a.basis_off) + (lane - 4)
                                                    : lane < 8 ? reinterpret_cast<const int32_t*>(a.piv_off) + (lane - 6)
                                                               : reinterpret_cast<const int32_t*>(a.map_off) + (lane & 1));
    const uint32_t step = lane < 1 ? 4 : 8;
    // The list is dealt to the workgroups in snake order.  Of a long one only the first half is;
    // the tail, its smaller contexts, goes to whichever is free, which evens out what the first
    // wavefronts' other contexts took: an eighth of a workgroup's part at a time through a counter
    // in memory (about 5 ns per addition to one address: each wavefront's own additions, four
    // contexts at a time, cost 20 us on 80,000 contexts), from there one at a time through LDS.
    // A chunk has to be worth the wait of 16 wavefronts for it: up to kTailFrom contexts per
    // workgroup everything is dealt (contexts of 60 rows, 41 columns: 8,000 70 us with a tail
    // in chunks of 2, 39 without; 17,000 77 and 63; 30,000 95 and 91; of 50-250 rows, 100-191
    // columns: 22,000 469 and 473; 30,000 603 and 622).
    constexpr int kTailFrom = 96;
    const int share = cnt <= kTailFrom * G ? (cnt + G - 1) / G : cnt / (2 * G);
    const int tail = share * G < cnt ? share * G : cnt;
    const int chunk = (cnt - tail) / (8 * G) + 1;
    auto load = [&](int c) {
        return *reinterpret_cast<const int32_t*>(src + static_cast<uint64_t>(c < 0 ? 0u : static_cast<uint32_t>(c)) * step);
    };
    struct Pipe {
        int c, n, m;        // the context at hand, then (after the call) the next one
        const uint64_t* R;
        int desc;           // its descriptor
        int out;            // the descriptor of the context at hand: its output offsets
        int c1, desc1;      // the one after, loading
        int id, at;         // the list entry of the third, loading; the fourth's position in the share, on its way
        __device__ __forceinline__ void arrived(RegRows& raw) {
            asm volatile("" ::"v"(raw.w0), "v"(raw.w1), "v"(raw.w2), "v"(raw.w3), "v"(raw.w4), "v"(desc1), "v"(id));
        }
        __device__ __forceinline__ int64_t pair(int v, int l) {
            return static_cast<int64_t>((static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(v, l + 1))) << 32) |
                                        static_cast<uint32_t>(__builtin_amdgcn_readlane(v, l)));
        }
        __device__ __forceinline__ void offsets(int64_t& bo, int64_t& po, int64_t& mo) {
            bo = pair(out, 4);
            po = pair(out, 6);
            mo = pair(out, 8);
        }
        // width, rows and first rows of the context of desc
        __device__ __forceinline__ void take(const FitArgs& a, RegRows& raw) {
            if (c < 0) return;
            n = __builtin_amdgcn_readlane(desc, 0);
            R = a.rows + pair(desc, 1);
            const uint32_t words = static_cast<uint32_t>(__builtin_amdgcn_readlane(desc, 3) - __builtin_amdgcn_readlane(desc, 1));
            switch (feat_words(n)) {
                case 1: raw = load_rows<3>(R, m = static_cast<int>(words / 3u), 0); break;
                case 2: raw = load_rows<4>(R, m = static_cast<int>(words / 4u), 0); break;
                default: raw = load_rows<5>(R, m = static_cast<int>(words / 5u), 0); break;
            }
        }
    };
    struct Step : Pipe {
        const FitArgs& a;
        decltype(load)& ld;
        decltype(list)& at_list;
        RegQueue& Q;
        int lane, G, g, share, tail, chunk, cnt;
        __device__ __forceinline__ int entry() {  // the next list entry, or -1
            const int v = __builtin_amdgcn_readfirstlane(this->at);
            if (v >= share) return tail_entry();
            if (lane == 0) this->at = atomicAdd(&Q.next, 1);
            const int e = v * G + ((v & 1) ? G - 1 - g : g);
            return e < cnt ? at_list(e) : -1;
        }
        __device__ __forceinline__ int tail_entry() {
            if (tail >= cnt) return -1;
            for (;;) {
                unsigned long long q = 0;
                if (lane == 0) q = atomicAdd(&Q.tail, 1ull);
                const int cur = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(q)));
                const int end = __builtin_amdgcn_readfirstlane(static_cast<int>(q >> 32));
                if (cur < end) return at_list(cur);
                if (cur == end) {  // one wavefront's part: the next chunk, or the news that there is none
                    uint32_t v = 0;  // (the counter may pass 2^31 by a few chunks)
                    if (lane == 0) v = static_cast<uint32_t>(atomicAdd(&a.plan[kRegNext], chunk)) + static_cast<uint32_t>(tail);
                    v = __builtin_amdgcn_readfirstlane(v);
                    if (v >= static_cast<uint32_t>(cnt)) {
                        __hip_atomic_store(&Q.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        return -1;
                    }
                    const unsigned long long stop = v + chunk < static_cast<uint32_t>(cnt) ? v + chunk : cnt;
                    __hip_atomic_store(&Q.tail, (stop << 32) | (v + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    return at_list(static_cast<int>(v));
                }
                // the wavefront that met the end stores one or the other
                if (__hip_atomic_load(&Q.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) return -1;
                __builtin_amdgcn_s_sleep(2);
            }
        }
        __device__ __forceinline__ void operator()(RegRows& raw) {
            this->out = this->desc;
            this->c = this->c1;
            this->desc = this->desc1;
            this->take(a, raw);
            this->c1 = __builtin_amdgcn_readfirstlane(this->id);
            this->desc1 = ld(this->c1);
            this->id = entry();
        }
    };
    RegRows raw{0, 0, 0, 0, 0, 0};
    Step P{{}, a, load, list, sQueue, lane, G, g, share, tail, chunk, cnt};
    P.at = start;
    P.c = __builtin_amdgcn_readfirstlane(P.entry());
    P.desc = load(P.c);
    P.c1 = __builtin_amdgcn_readfirstlane(P.entry());
    P.desc1 = load(P.c1);
    P.id = P.entry();
    P.take(a, raw);
    while (P.c >= 0) {
        switch (feat_words(P.n)) {
            case 1:
                if (P.n < 32) fit_ctx_reg<1, true>(a, sc, P.c, P.n, P.m, P.R, basis, raw, P);
                else fit_ctx_reg<1>(a, sc, P.c, P.n, P.m, P.R, basis, raw, P);
                break;
            case 2: fit_ctx_reg<2>(a, sc, P.c, P.n, P.m, P.R, basis, raw, P); break;
            default: fit_ctx_reg<3>(a, sc, P.c, P.n, P.m, P.R, basis, raw, P); break;
        }
    }
}

// the long, one and group contexts that k_fit_reg leaves: kPivWaves wavefronts per
// workgroup, several workgroups per compute unit.
// The list (largest first) is taken greedily: workgroup g starts at position g,
// then each takes the next free position from a counter as it finishes one (the
// fetch is issued when a context starts, so its latency hides behind the work).
__global__ __launch_bounds__(kPivThreads, 3) void k_fit_piv(FitArgs a) {
    __shared__ PivShared S;
    __shared__ int sNext;
    const PivLists pl = piv_lists(a);
    const int g1 = pl.piv_group, g2 = g1 + pl.piv_one, g3 = g2 + pl.piv_long, cnt = g3 + pl.piv_short;
    const int32_t* const order = a.plan + kPlanHead;
    BlockSync sync;
    for (int i = static_cast<int>(blockIdx.x); i < cnt;) {
        const int c = __builtin_amdgcn_readfirstlane(i < g1   ? order[pl.piv_group_lo + i]
                                                     : i < g2 ? order[pl.one_lo + i - g1]
                                                     : i < g3 ? order[pl.long_lo + i - g2]
                                                              : order[pl.short_lo + i - g3]);
        int next = 0;
        if (threadIdx.x == 0) next = atomicAdd(&a.plan[kPivNext], 1) + static_cast<int>(gridDim.x);
        const CtxDesc ds = readlane_desc(load_desc(a, c), 0);
        switch (feat_words(ds.n)) {
            case 1: fit_ctx_piv<1, kPivWaves>(a, ds, S, sync); break;
            case 2: fit_ctx_piv<2, kPivWaves>(a, ds, S, sync); break;
            case 3: case 4: fit_ctx_piv<4, kPivWaves>(a, ds, S, sync); break;
            case 5: fit_ctx_piv<5, kPivWaves>(a, ds, S, sync); break;
            case 6: fit_ctx_piv<6, kPivWaves>(a, ds, S, sync); break;
            default: fit_ctx_piv<8, kPivWaves>(a, ds, S, sync); break;
        }
        if (threadIdx.x == 0) sNext = next;
        __syncthreads();
        i = sNext;
        __syncthreads();
    }
}

// Small batches (up to kSmallBatch contexts, declared widths below 512): one
// launch, one workgroup of 8 wavefronts per context, the context's class choosing
// the path (one wavefront up to kSmallRows rows of up to 3 feature words, else all eight).
// No plan: its launch would cost more than the fit of a batch this size,
// and one workgroup per context needs no load balance.  Invalid contexts, and any
// wider than the declared bound, are flagged here.
constexpr int kSmallBatch = 64;
constexpr int kSmallRows = 256;
union SmallShared {
    uint64_t reg[kRegRec];
    PivShared piv;
};

__global__ __launch_bounds__(kSmallThreads) void k_fit_small(FitArgs a) {
    __shared__ SmallShared U;
    const CtxDesc ds = readlane_desc(load_desc(a, blockIdx.x), 0);
    if (ds.c < 0) return;
    if (ds.bad) {
        if (threadIdx.x == 0) write_bad_context(a, ds);
        return;
    }
    const int fw = feat_words(ds.n);
    BlockSync sync;
    switch (fit_class(ds, kSmallRows)) {
        case kClsShort:
            if (threadIdx.x < 64) {
                if (fw == 1) fit_ctx_alone<1>(a, ds, U.reg);
                else if (fw == 2) fit_ctx_alone<2>(a, ds, U.reg);
                else fit_ctx_alone<3>(a, ds, U.reg);
            }
            break;
        case kClsLarge:  // not launched for a batch that may hold one (the bound is below 512)
            break;
        default:
            switch (fw) {
                case 1: fit_ctx_piv<1, kSmallWaves>(a, ds, U.piv, sync); break;
                case 2: fit_ctx_piv<2, kSmallWaves>(a, ds, U.piv, sync); break;
                case 3: case 4: fit_ctx_piv<4, kSmallWaves>(a, ds, U.piv, sync); break;
                case 5: fit_ctx_piv<5, kSmallWaves>(a, ds, U.piv, sync); break;
                case 6: fit_ctx_piv<6, kSmallWaves>(a, ds, U.piv, sync); break;
                default: fit_ctx_piv<8, kSmallWaves>(a, ds, U.piv, sync); break;
            }
            break;
    }
}

// Wide contexts (class large): the fewer there are, the more workgroups fit one together
// (8, 4 or 2, while every context then has its own).  Under a cooperative launch every
// workgroup is resident, which the waits for one another need; otherwise every context
// takes one.  A group's workgroups are blockIdx values congruent mod 8, which the
// dispatcher places on one die (a shared L2 for the list they all read): for speed alone, the
// list is exchanged at device scope.
__global__ __launch_bounds__(kWdThreads) void k_fit_wide(FitArgs a) {
    __shared__ WideShared U;
    const int nl = a.plan[kClsLarge + 1] - a.plan[kClsLarge];
    const int nwg = static_cast<int>(gridDim.x);
    int G = 1;
    if (a.coop && nwg <= kMaxMembers)
        for (int k = 2; k <= 8 && k * nl <= nwg && nwg % (8 * k) == 0; k *= 2) G = k;
    const int x = static_cast<int>(blockIdx.x), idx = x / 8;
    const int g = idx % G, grp = (x % 8) + 8 * (idx / G), ngrp = nwg / G;
    // the list is dealt to the groups in snake order: one context each where G > 1 (G * nl <= nwg)
    for (int i = 0;; ++i) {
        const int64_t e = static_cast<int64_t>(i) * ngrp + ((i & 1) ? ngrp - 1 - grp : grp);
        if (e >= nl) break;
        const int c = __builtin_amdgcn_readfirstlane(a.plan[kPlanHead + a.plan[kClsLarge] + static_cast<int>(e)]);
        fit_ctx_wide(a, readlane_desc(load_desc(a, c), 0), U, G, g, a.plan + kBarHead + (G > 1 ? grp * G : 0));
    }
}

// ---------------------------------------------------------------------------
// encode (Sec. 2.3), one lane per query, queries in any order: the table
// entries of the set bits of phi = [x | 1] are XORed (the constant column is
// always set).  The z part is T(phi) = M phi; the h part is the reduction
// residual on the free columns and must vanish for phi to lie in the span.
// ---------------------------------------------------------------------------

// x words of a query, with bits past the stride read as zero
template <int SMAX>
struct QueryX {
    uint64_t xr[SMAX > 0 ? SMAX : 1];
    const uint64_t* xq;
    int S;
    __device__ __forceinline__ void load(const uint64_t* p, int stride) {
        xq = p;
        S = stride;
        if constexpr (SMAX > 0) {
#pragma unroll
            for (int k = 0; k < SMAX; ++k) xr[k] = k < S ? p[k] : 0ull;
        }
    }
    __device__ __forceinline__ uint64_t word(int w) const {
        if constexpr (SMAX > 0) {
            uint64_t v = 0;
#pragma unroll
            for (int k = 0; k < SMAX; ++k) v = (w == k) ? xr[k] : v;
            return v;
        } else {
            return w < S ? xq[w] : 0ull;
        }
    }
};

// any x bit at or above the width n: outside the context's ambient space
template <int SMAX>
__device__ __forceinline__ bool outside_width(const QueryX<SMAX>& x, int n) {
    bool outside = false;
    for (int w = (n >> 6); w < x.S; ++w) {
        const uint64_t v = x.word(w);
        const int lo = 64 * w;
        outside |= (lo >= n) ? (v != 0) : ((v >> (n - lo)) != 0);
    }
    return outside;
}

struct alignas(16) Word2 {
    uint64_t x, y;
};

// T(phi): XOR of the map columns of the set bits, four gathers in flight
template <int SMAX>
__device__ __forceinline__ void map_gather(const uint64_t* M, int n, const QueryX<SMAX>& x, uint64_t& z0,
                                           uint64_t& z1) {
    const Word2 zc = *reinterpret_cast<const Word2*>(M + 2 * n);  // constant column: always set
    z0 = zc.x;
    z1 = zc.y;
    const int fw = feat_words(n);
    const int xw = x.S < fw ? x.S : fw;
    for (int w = 0; w < xw; ++w) {
        const uint64_t v = x.word(w);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint32_t u = half ? static_cast<uint32_t>(v >> 32) : static_cast<uint32_t>(v);
            const uint64_t* Mh = M + 2 * (64 * w + 32 * half);
            while (u) {  // a missing gather re-reads the first column and is masked off
                int jj[4];
                uint64_t mk[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    mk[k] = u ? ~0ull : 0ull;
                    jj[k] = u ? __builtin_ctz(u) : jj[0];
                    u &= u - 1;
                }
                Word2 a[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) a[k] = *reinterpret_cast<const Word2*>(Mh + 2 * jj[k]);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    z0 ^= a[k].x & mk[k];
                    z1 ^= a[k].y & mk[k];
                }
            }
        }
    }
}

// support test: even overlap of phi = [x | 1] with every parity-check row (all rows are
// read, several at a time: no early exit to serialise the loads; past the last row the
// last is read again, which changes nothing).  A lane's life is its chain of loads: with one row of two words or more, and
// one word of a wide basis row, at a time, 1M queries on a corpus of 80,000 maps took 188 us in
// k_encode_lanes, 126 us with two to four rows in flight here and in basis_scan.
template <int SMAX>
__device__ __forceinline__ bool parity_ok(const uint64_t* H, int t, int n, const QueryX<SMAX>& x) {
    const int fw = feat_words(n), cw = n >> 6;
    const uint64_t cbit = 1ull << (n & 63);
    int odd = 0;  // bit 0 of an OR of popcounts is the OR of their parities
    if (fw == 1) {
        const uint64_t q = x.word(0) | cbit;
        for (int f = 0; f < t; f += 4) {
            uint64_t h[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) h[u] = H[f + u < t ? f + u : t - 1];
#pragma unroll
            for (int u = 0; u < 4; ++u) odd |= __popcll(h[u] & q);
        }
    } else if (fw == 2) {
        const uint64_t q0 = x.word(0), q1 = x.word(1) | cbit;
        for (int f = 0; f < t; f += 4) {
            u64x2_a8 h[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) h[u] = *reinterpret_cast<const u64x2_a8*>(H + 2 * (f + u < t ? f + u : t - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u) odd |= __popcll((h[u].x & q0) ^ (h[u].y & q1));
        }
    } else {
        for (int f = 0; f < t; f += 2) {
            const uint64_t* h0 = H + static_cast<int64_t>(f) * fw;
            const uint64_t* h1 = f + 1 < t ? h0 + fw : h0;
            uint64_t a0 = 0, a1 = 0;
            for (int w = 0; w < fw; w += 4) {
                uint64_t v0[4], v1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    v0[u] = w + u < fw ? h0[w + u] : 0ull;
                    v1[u] = w + u < fw ? h1[w + u] : 0ull;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint64_t qw = x.word(w + u);
                    if (w + u == cw) qw |= cbit;
                    a0 ^= v0[u] & qw;
                    a1 ^= v1[u] & qw;
                }
            }
            odd |= __popcll(a0) | __popcll(a1);
        }
    }
    return (odd & 1) == 0;
}

// low-rank contexts: reduce phi by the basis rows (descending priority); the
// rows whose pivot bit phi holds sum to [phi | T(phi)] exactly when phi is in the span
template <int SMAX>
__device__ __forceinline__ bool basis_scan(const uint64_t* B, const int32_t* piv, int rank, int n,
                                           const QueryX<SMAX>& x, uint64_t& z0, uint64_t& z1) {
    const int fw = feat_words(n), W = fw + F2_Y_WORDS, cw = n >> 6;
    const uint64_t cbit = 1ull << (n & 63);
    uint64_t diff = 0;  // features: phi XOR the selected rows, word by word
    z0 = z1 = 0;
    if (fw <= 4) {
        uint64_t acc[4] = {0, 0, 0, 0};
        auto add_row = [&](int p, const uint64_t (&rv)[6]) {
            uint64_t qw = x.word(p >> 6);
            if ((p >> 6) == cw) qw |= cbit;
            const uint64_t mk = 0ull - ((qw >> (p & 63)) & 1ull);
#pragma unroll
            for (int w = 0; w < 4; ++w) acc[w] ^= rv[w] & mk;
            z0 ^= rv[4] & mk;
            z1 ^= rv[5] & mk;
        };
        int k = 0;
        for (; k + 2 <= rank; k += 2) {  // two rows in flight (four cost a third of the occupancy of the per-lane passes)
            int p[2];
            uint64_t rv[2][6];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                p[u] = piv[k + u];
                const uint64_t* row = B + static_cast<int64_t>(k + u) * W;
#pragma unroll
                for (int w = 0; w < 4; ++w) rv[u][w] = w < fw ? row[w] : 0ull;
                rv[u][4] = row[fw];
                rv[u][5] = row[fw + 1];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) add_row(p[u], rv[u]);
        }
        for (; k < rank; ++k) {
            const uint64_t* row = B + static_cast<int64_t>(k) * W;
            uint64_t rv[6];
#pragma unroll
            for (int w = 0; w < 4; ++w) rv[w] = w < fw ? row[w] : 0ull;
            rv[4] = row[fw];
            rv[5] = row[fw + 1];
            add_row(piv[k], rv);
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w >= fw) break;
            uint64_t qw = x.word(w);
            if (w == cw) qw |= cbit;
            diff |= acc[w] ^ qw;
        }
    } else {
        // two words at a time (the two output words last), four rows in flight
        for (int w = 0; w < W; w += 2) {
            w = w > fw ? fw : w;
            const int w1 = w + 1 < fw || w == fw ? w + 1 : w;
            uint64_t a0 = 0, a1 = 0;
            for (int k = 0; k < rank; k += 4) {
                int p[4];
                uint64_t v0[4], v1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = k + u < rank ? k + u : rank - 1;
                    p[u] = piv[i];
                    const uint64_t* row = B + static_cast<int64_t>(i) * W;
                    v0[u] = row[w];
                    v1[u] = row[w1];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint64_t qw = x.word(p[u] >> 6);
                    if ((p[u] >> 6) == cw) qw |= cbit;
                    const uint64_t mk = k + u < rank ? 0ull - ((qw >> (p[u] & 63)) & 1ull) : 0ull;
                    a0 ^= v0[u] & mk;
                    a1 ^= v1[u] & mk;
                }
            }
            if (w == fw) {
                z0 = a0;
                z1 = a1;
                break;
            }
            uint64_t q0 = x.word(w), q1 = x.word(w1);
            if (w == cw) q0 |= cbit;
            if (w1 == cw) q1 |= cbit;
            diff |= (a0 ^ q0) | (a1 ^ q1);
        }
    }
    return diff == 0;
}

template <int SMAX>
__device__ __forceinline__ bool encode_query(const EncArgs& e, int c, const uint64_t* xq, uint64_t& z0,
                                             uint64_t& z1) {
    QueryX<SMAX> x;
    x.load(xq, e.stride);
    const int n = e.n_bits[c];
    if (outside_width(x, n)) return false;
    const int d = n + 1;
    const int r0 = e.rank[c];
    const int r = r0 < 0 ? 0 : (r0 > d ? d : r0);  // 0 <= rank <= d for a fitted context
    if (!has_parity_rows(d, r))
        return basis_scan(e.basis + e.basis_off[c], e.pivots + e.piv_off[c], r, n, x, z0, z1);
    map_gather(e.maps + e.map_off[c], n, x, z0, z1);
    return parity_ok(e.tables + e.basis_off[c], d - r, n, x);
}

// flags and word of one query of context id c
__device__ __forceinline__ uint8_t encode_one(const EncArgs& e, int c, int64_t q, uint64_t& z0, uint64_t& z1) {
    z0 = z1 = 0;
    if (c < 0 || c >= e.num_ctx || (e.ctx_flags[c] & kBadCtx)) return F2_Q_BAD_CTX;
    uint8_t fl = (e.ctx_flags[c] & F2_CTX_CONTRADICTION) ? F2_Q_CTX_CONTRADICTORY : 0;
    const uint64_t* xq = e.x + q * e.stride;
    const bool in = e.stride <= 4 ? encode_query<4>(e, c, xq, z0, z1) : encode_query<0>(e, c, xq, z0, z1);
    if (!in) {
        fl |= F2_Q_OUT_OF_SPAN;
        z0 = z1 = 0;
    }
    return fl;
}

// ---------------------------------------------------------------------------
// queries of wide contexts (more than kLaneFW feature words: widths from 512 on): the whole wavefront
// takes one query, lane w holding word w of phi.  One lane per query walks a wide
// context's rows word by word behind dependent 8-byte loads; here a basis row, 64
// map columns or a parity-check row is one coalesced load, and only the rows and
// columns that phi selects are read.  It is bound by the latency of those loads
// (one round trip for the scalars, one for x and the pivots, one per eight rows).
// 20,000 queries on 96 contexts of 513-1,500 bits at ranks around 24: 1,090 us with
// a lane per query, 36 us with a wavefront per query.
// ---------------------------------------------------------------------------
// The lanes of a wavefront take its queries of up to 8 words at once; one after the
// other those would cost more (1M queries on 80,000 contexts of up to 5 words, 0.05%
// of the contexts with 5: 125 us per lane, 310 us with a wavefront for each of those).
constexpr int kLaneFW = 8;

__device__ __forceinline__ uint32_t xor_lanes(uint32_t v) {
    for (int o = 32; o > 0; o >>= 1) v ^= static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), o));
    return v;
}

// query q of context c (both uniform; c valid): support in the return value, the word in every lane
__device__ __forceinline__ bool encode_wave(const EncArgs& e, int c, int64_t q, uint64_t& z0, uint64_t& z1) {
    const int lane = threadIdx.x & 63;
    const uint64_t* xq = e.x + q * e.stride;
    const int n = e.n_bits[c], d = n + 1, r0 = e.rank[c];
    const int64_t bo = e.basis_off[c], po = e.piv_off[c], mo = e.map_off[c];
    const int r = r0 < 0 ? 0 : (r0 > d ? d : r0);
    const int fw = feat_words(n), W = fw + F2_Y_WORDS, cw = n >> 6;
    const uint64_t xw = lane < e.stride ? xq[lane] : 0ull;
    bool outside = lane > cw ? xw != 0 : (lane == cw && (xw >> (n & 63)) != 0);  // x bits at or above n
    for (int w = 64 + lane; w < e.stride; w += 64) outside |= xq[w] != 0;
    z0 = z1 = 0;
    if (__ballot(outside)) return false;
    const uint64_t ph = xw | (lane == cw ? 1ull << (n & 63) : 0ull);  // zero past word cw = fw - 1
    // the basis rows that phi selects (r / 2 or so) sum to [phi | T(phi)] exactly inside
    // the span; the t = d - r parity-check rows are all read, so they serve while t <= r / 2
    if (2 * (d - r) > r) {
        const uint64_t* B = e.basis + bo;
        uint64_t acc = ph, y = 0;
        const int fl = lane < fw ? lane : 0, yl = fw + (lane & 1);
        for (int k0 = 0; k0 < r; k0 += 64) {
            const bool has = k0 + lane < r;
            const int p = has ? e.pivots[po + k0 + lane] : 0;
            const uint64_t pw = shfl64(ph, (p >> 6) & 63);
            uint64_t sel = __ballot(has && ((pw >> (p & 63)) & 1ull));
            while (sel) {  // eight rows in flight; a missing one re-reads the first and is masked off
                int k[8];
                uint64_t f[8], v[8], mk[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    mk[u] = sel ? ~0ull : 0ull;
                    k[u] = sel ? ffs64(sel) : k[0];
                    sel &= sel - 1;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint64_t* row = B + static_cast<int64_t>(k0 + k[u]) * W;
                    f[u] = row[fl];
                    v[u] = row[yl];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    acc ^= f[u] & mk[u];
                    y ^= v[u] & mk[u];
                }
            }
        }
        z0 = readlane64(y, 0);
        z1 = readlane64(y, 1);
        return __ballot(lane < fw && acc != 0) == 0;
    }
    // T(phi): the map columns of phi's set bits, 64 columns (a word of phi) per step
    uint64_t a0 = 0, a1 = 0;
    const Word2* M = reinterpret_cast<const Word2*>(e.maps + mo);
    for (int w0 = 0; w0 < fw; w0 += 4) {
        Word2 col[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t pw = readlane64(ph, (w0 + u) & 63);  // (past the last word: zero, or masked by the bound)
            const bool set = w0 + u < fw && ((pw >> lane) & 1ull);
            col[u].x = col[u].y = 0;
            if (set) col[u] = M[64 * (w0 + u) + lane];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a0 ^= col[u].x;
            a1 ^= col[u].y;
        }
    }
    // support: even overlap with every parity-check row, the lanes' partial overlaps counted by a ballot
    const uint64_t* H = e.tables + bo;
    const int t = d - r;
    int odd = 0;
    for (int f0 = 0; f0 < t; f0 += 8) {
        uint64_t h[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = (lane < fw && f0 + u < t) ? H[static_cast<int64_t>(f0 + u) * fw + lane] : 0ull;
#pragma unroll
        for (int u = 0; u < 8; ++u) odd |= __popcll(__ballot(__popcll(h[u] & ph) & 1));
    }
    if (odd & 1) return false;
    z0 = (static_cast<uint64_t>(xor_lanes(static_cast<uint32_t>(a0 >> 32))) << 32) | xor_lanes(static_cast<uint32_t>(a0));
    z1 = (static_cast<uint64_t>(xor_lanes(static_cast<uint32_t>(a1 >> 32))) << 32) | xor_lanes(static_cast<uint32_t>(a1));
    return true;
}

// context c valid, in good order and wide
__device__ __forceinline__ bool wide_ctx(const EncArgs& e, int c) {
    return c >= 0 && c < e.num_ctx && !(e.ctx_flags[c] & kBadCtx) && feat_words(e.n_bits[c]) > kLaneFW;
}

// the queries of the lanes in `todo` (context c, query q), a wavefront each; out is written in those lanes
__device__ __forceinline__ uint8_t encode_each(const EncArgs& e, uint64_t todo, int c, int64_t q, Word2& out) {
    uint8_t fl = 0;
    for (; todo; todo &= todo - 1) {
        const int j = ffs64(todo);
        const int cj = __builtin_amdgcn_readlane(c, j);
        uint64_t z0, z1;
        const bool in = encode_wave(e, cj, static_cast<int64_t>(readlane64(static_cast<uint64_t>(q), j)), z0, z1);
        if ((threadIdx.x & 63) == j) {
            fl = ((e.ctx_flags[cj] & F2_CTX_CONTRADICTION) ? F2_Q_CTX_CONTRADICTORY : 0) | (in ? 0 : F2_Q_OUT_OF_SPAN);
            out.x = in ? z0 : 0;
            out.y = in ? z1 : 0;
        }
    }
    return fl;
}

// Wide queries of (nearly) full rank are a lane's each where a wavefront holds many: their lanes gather
// columns of the same map side by side, and read the few parity-check rows together.  A million queries on 100
// contexts, wavefront each / lane each: 600 bits at full rank 1.04 / 0.52 ms, 16 parity-check rows
// 1.33 / 0.69; 3,000 bits 2.55 / 1.62, 16 rows 2.86 / 2.55, 32 rows 3.32 / 3.72.  A lane's chain is 8 words' trips to a
// wavefront's 1 (times the queries): some 14 queries of 600 bits, 21 of 1,500.
constexpr int kLaneParity = 16, kLaneParityMin = 16;

// whether this lane's query (of context c, if live) is a wavefront's (no lane may be inactive here)
__device__ __forceinline__ bool for_wavefront(const EncArgs& e, bool live, int c) {
    const bool wide = live && wide_ctx(e, c);
    const bool few = wide && e.n_bits[c] + 1 - e.rank[c] <= kLaneParity;
    return wide && !(__popcll(__ballot(few)) >= kLaneParityMin && few);
}

// One query per live lane (context c, query q), the wide ones a wavefront each (no lane may be inactive here).
// With share >= 0 only the wide ones share * kWideShare on, kWideShare of them, and with share 0 the
// others too; `live` then says which.
constexpr int kWideShare = 8;
template <bool WIDE>
__device__ __forceinline__ uint8_t encode_lanes(const EncArgs& e, bool& live, int c, int64_t q, Word2& out, int share = -1) {
    uint8_t fl = 0;
    bool wide = false;
    if constexpr (WIDE) {
        wide = for_wavefront(e, live, c);
        if (share >= 0) {
            const int rank = __popcll(__ballot(wide) & ((1ull << (threadIdx.x & 63)) - 1));
            live = live && (wide ? rank / kWideShare == share : share == 0);
            wide = wide && live;
        }
    }
    if (live && !wide) fl = encode_one(e, c, q, out.x, out.y);
    if constexpr (WIDE) {
        const uint8_t fw = encode_each(e, __ballot(wide), c, q, out);
        if (wide) fl = fw;
    }
    return fl;
}

// Small batches that may hold wide contexts.  The first lane_blocks workgroups take a query per
// lane and leave the wide ones; in the others `parts` wavefronts look at the same 64 queries
// and share out their wide ones, so many that the chip is full of wavefronts when all
// are wide, and gone at once when none is.  (A wavefront that took 1-64 queries of
// either kind left most of its lanes empty on narrow ones.  100,000 queries of 40 bits on 300
// contexts, no width declared: 18.4 us so, 7.8 now, 7.6 where the widths are declared narrow; on
// 20,000 contexts 24.7, 18.2 and 16.3; 50,000 queries on 96 contexts of 513-1,500 bits: 53 and 52.)
constexpr int kWideWaves = 8192;  // eight per SIMD
__global__ __launch_bounds__(kEncThreads) void k_encode_wide(EncArgs e, int lane_blocks, int parts) {
    const int lane = threadIdx.x & 63;
    const int b = static_cast<int>(blockIdx.x);
    Word2 out;
    if (b < lane_blocks) {
        const int64_t q = static_cast<int64_t>(b) * kEncThreads + threadIdx.x;
        if (q >= e.nq) return;
        const int c = e.ctx_id[q];
        if (wide_ctx(e, c)) return;
        const uint8_t fl = encode_one(e, c, q, out.x, out.y);
        *reinterpret_cast<Word2*>(e.words + 2 * q) = out;
        e.qflags[q] = fl;
        return;
    }
    // which of the 64 are wide: each of the workgroup's wavefronts looks at 16 of them
    __shared__ uint16_t sWide[kEncThreads / 64];
    const int wave = threadIdx.x >> 6, shares = parts / (kEncThreads / 64);
    const int part = (b - lane_blocks) % shares * (kEncThreads / 64) + wave;
    const int64_t q0 = static_cast<int64_t>((b - lane_blocks) / shares) * 64, q = q0 + lane;
    const int c = q < e.nq ? e.ctx_id[q] : -1;
    const uint64_t some = __ballot(lane / 16 == wave && wide_ctx(e, c));
    if (lane == 0) sWide[wave] = static_cast<uint16_t>(some >> (16 * wave));
    __syncthreads();
    uint64_t all = 0;
    for (int w = 0; w < kEncThreads / 64; ++w) all |= static_cast<uint64_t>(sWide[w]) << (16 * w);
    const bool wide = (all >> lane) & 1ull;
    const int rank = __popcll(all & ((1ull << lane) - 1));
    const bool mine = wide && (rank & (parts - 1)) == part;
    const uint8_t fl = encode_each(e, __ballot(mine), c, q, out);
    if (!mine) return;
    *reinterpret_cast<Word2*>(e.words + 2 * q) = out;
    e.qflags[q] = fl;
}

__global__ __launch_bounds__(kEncThreads) void k_encode(EncArgs e) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kEncThreads + threadIdx.x;
    if (q >= e.nq) return;
    Word2 out;
    const uint8_t fl = encode_one(e, e.ctx_id[q], q, out.x, out.y);
    *reinterpret_cast<Word2*>(e.words + 2 * q) = out;
    e.qflags[q] = fl;
}

// ---------------------------------------------------------------------------
// context-grouped encode for large batches.  In arbitrary order the lanes of a
// wavefront gather from as many maps as they hold contexts, one cache line per
// lane.  A counting sort by bin (2^k consecutive contexts per bin, at most
// kSortMaxBins bins, or kSortMaxBinsLarge for batches above kFineBinQueries
// (finer bins, an LDS histogram of up to 160 KB), one more bin for out-of-range
// ids) first groups the queries; the encode then runs over the sorted order,
// where the lanes of a wavefront share a few contexts and their gathers hit the
// same lines, and writes each result straight to its query.
//
// The batch is sorted window by window (bpw consecutive count blocks, about
// kWindowQueries queries): a query's sorted position stays inside its window.
// The sorted passes walk the positions in order, so the results they scatter
// at any time land in the queries of about one window (128 MB of words), which
// the last-level cache merges before they reach HBM; scattered 16-byte writes
// over a whole 100M-query batch run at a third of that rate.  The flag bytes
// are cleared in query order by the scatter; the sorted passes write only the
// nonzero ones.  The sort uses per-block LDS histograms and scans (no
// device-wide counters):
//   count (per block)  ->  column scan (per window and bin, over the window's
//   blocks)  ->  scatter (bin scan per block, query -> sorted position)  ->
//   sorted encode  ->  second pass over the positions it leaves
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 1024;
constexpr int kSortMaxBins = 8192;
constexpr int kSortMaxBinsLarge = 40000;  // 160,004 bytes of LDS histogram: up to two of 80,000 contexts per bin
constexpr int64_t kWindowQueries = int64_t{1} << 23;

constexpr int kRestMore = 26;  // (a chunk of 2^30 queries has 2^24 groups)
struct SortArgs {
    int32_t nb;       // bins, the last one for out-of-range context ids
    int32_t bin_shift;  // 2^bin_shift contexts per bin
    int32_t blocks;   // count / scatter blocks
    int32_t bpw;      // count / scatter blocks per window
    int64_t qc;       // queries per count / scatter block
    int32_t* hist;    // [blocks][nb], then exclusive offsets within each bin (of the block's window)
    int32_t* total;   // [windows][nb]
    int2* perm;       // [nq] sorted position -> (query, context id)
    int32_t regroup;  // 1: each chunk of kRegroupChunk positions regrouped by context (k_enc_regroup)
    int32_t staged;   // 1: k_encode_sorted stages the wavefronts' contexts; 0: every position per lane
    uint64_t* rest;   // [ceil(nq / 64)] positions the staged pass left to the second pass (bit per lane; set for the listed groups only)
    int32_t* rest_list;   // [ceil(nq / 64)] the 64-position groups with such positions, in no order;
                          // from bit kRestMore on, how many wavefronts more share its wide queries
    int32_t* rest_count;  // [1] entries of rest_list (cleared by the count)
};

__device__ __forceinline__ int query_bin(const EncArgs& e, const SortArgs& s, int c) {
    return (c < 0 || c >= e.num_ctx) ? s.nb - 1 : (c >> s.bin_shift);
}

__global__ __launch_bounds__(kSortThreads) void k_enc_count(EncArgs e, SortArgs s) {
    extern __shared__ int sBin[];  // [s.nb] (dynamic)
    const int tid = threadIdx.x;
    for (int b = tid; b < s.nb; b += kSortThreads) sBin[b] = 0;
    __syncthreads();
    const int64_t q0 = static_cast<int64_t>(blockIdx.x) * s.qc;
    const int64_t q1 = q0 + s.qc < e.nq ? q0 + s.qc : e.nq;
    // eight ids per thread and step, the next step's loaded before this step's
    // counts (sixteen loads in flight per thread)
    constexpr int U = 8;
    int64_t q = q0 + tid;
    if (q + (U - 1) * kSortThreads < q1) {
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = e.ctx_id[q + u * kSortThreads];
        for (;;) {
            const int64_t qn = q + U * kSortThreads;
            const bool more = qn + (U - 1) * kSortThreads < q1;
            int cn[U];
#pragma unroll
            for (int u = 0; u < U; ++u) cn[u] = e.ctx_id[more ? qn + u * kSortThreads : q];  // (a valid address)
#pragma unroll
            for (int u = 0; u < U; ++u) atomicAdd(&sBin[query_bin(e, s, c[u])], 1);
            q = qn;
            if (!more) break;
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = cn[u];
        }
    }
    for (; q < q1; q += kSortThreads) atomicAdd(&sBin[query_bin(e, s, e.ctx_id[q])], 1);
    if (blockIdx.x == 0 && tid == 0) *s.rest_count = 0;
    __syncthreads();
    int32_t* h = s.hist + static_cast<int64_t>(blockIdx.x) * s.nb;
    for (int b = tid; b < s.nb; b += kSortThreads) h[b] = sBin[b];
}

// exclusive prefix of each bin over the blocks of its window, in place, and the
// bin's total in the window.  A workgroup takes 64 bins of one window (a lane
// each) and splits the window's blocks among its kColWaves wavefronts, so every lane
// has all of its loads in flight at once.
constexpr int kColWaves = 8;  // 16: 39 us on 100M queries in 12 windows of ~21 blocks; 8: 32 us
constexpr int kMaxSortBlocks = 256;
constexpr int kColPerWave = kMaxSortBlocks / kColWaves;  // blocks per wavefront (at most)
__global__ __launch_bounds__(64 * kColWaves) void k_enc_colscan(SortArgs s) {
    __shared__ int sPart[kColWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int groups = (s.nb + 63) / 64;  // bin groups per window
    const int win = blockIdx.x / groups;
    const int b = (blockIdx.x - win * groups) * 64 + lane;
    const int bpw = s.bpw > 0 ? s.bpw : s.blocks;  // (no window size: one window of every block)
    const int wb0 = win * bpw;
    const int wblocks = s.blocks - wb0 < bpw ? s.blocks - wb0 : bpw;  // <= kMaxSortBlocks
    const int per = (wblocks + kColWaves - 1) / kColWaves;  // <= kColPerWave
    const int gb = wb0 + wave * per, ge = wb0 + wblocks;
    int v[kColPerWave];
#pragma unroll
    for (int k = 0; k < kColPerWave; ++k)
        v[k] = (b < s.nb && k < per && gb + k < ge) ? s.hist[static_cast<int64_t>(gb + k) * s.nb + b] : 0;
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kColPerWave; ++k) sum += v[k];
    sPart[wave][lane] = sum;
    __syncthreads();
    int run = 0, total = 0;
    for (int w = 0; w < kColWaves; ++w) {
        const int t = sPart[w][lane];
        run += w < wave ? t : 0;
        total += t;
    }
    if (b >= s.nb) return;
#pragma unroll
    for (int k = 0; k < kColPerWave; ++k)
        if (k < per && gb + k < ge) {
            s.hist[static_cast<int64_t>(gb + k) * s.nb + b] = run;
            run += v[k];
        }
    if (wave == 0) s.total[static_cast<int64_t>(win) * s.nb + b] = total;
}

// exclusive scan of the bin totals by one workgroup of kSortThreads threads,
// added into sBin, which holds the block's own offsets within each bin (h, copied
// here while the totals are loading).  Up to kBinsPerThread bins per thread the
// totals stay in registers; more bins (large batches) read them twice.
constexpr int kBinsPerThread = (kSortMaxBins + 1 + kSortThreads - 1) / kSortThreads;
__device__ __forceinline__ void bin_offsets(const SortArgs& s, const int32_t* h, const int32_t* total, int* sBin,
                                            int* sWave) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int per = (s.nb + kSortThreads - 1) / kSortThreads;
    const int b0 = tid * per;
    const bool in_regs = per <= kBinsPerThread;
    int tv[kBinsPerThread];
    int sum = 0;
    if (in_regs) {
#pragma unroll
        for (int k = 0; k < kBinsPerThread; ++k) tv[k] = (k < per && b0 + k < s.nb) ? total[b0 + k] : 0;
#pragma unroll
        for (int k = 0; k < kBinsPerThread; ++k) sum += tv[k];
    } else {
        for (int k = 0; k < per; ++k)
            if (b0 + k < s.nb) sum += total[b0 + k];
    }
    for (int b = tid; b < s.nb; b += kSortThreads) sBin[b] = h[b];
    int x = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    if (lane == 63) sWave[tid >> 6] = x;
    __syncthreads();
    int run = x - sum;
    for (int w = 0; w < (tid >> 6); ++w) run += sWave[w];
    if (in_regs) {
#pragma unroll
        for (int k = 0; k < kBinsPerThread; ++k)
            if (k < per && b0 + k < s.nb) {
                sBin[b0 + k] += run;
                run += tv[k];
            }
    } else {
        for (int k = 0; k < per; ++k)
            if (b0 + k < s.nb) {
                sBin[b0 + k] += run;
                run += total[b0 + k];
            }
    }
}

__global__ __launch_bounds__(kSortThreads) void k_enc_scatter(EncArgs e, SortArgs s) {
    extern __shared__ int sBin[];  // [s.nb] (dynamic)
    __shared__ int sWave[kSortThreads / 64];
    const int tid = threadIdx.x;
    const int win = blockIdx.x / s.bpw;
    // every block scans its window's bin totals itself (a few thousand words)
    // instead of a one-workgroup scan kernel between the column scan and the scatter
    bin_offsets(s, s.hist + static_cast<int64_t>(blockIdx.x) * s.nb, s.total + static_cast<int64_t>(win) * s.nb, sBin,
                sWave);
    __syncthreads();
    const int64_t q0 = static_cast<int64_t>(blockIdx.x) * s.qc;
    const int64_t q1 = q0 + s.qc < e.nq ? q0 + s.qc : e.nq;
    const int64_t base = static_cast<int64_t>(win) * s.bpw * s.qc;  // the window's first query and position
    // the flag bytes of the block's queries, cleared in order (the sorted passes
    // write the nonzero ones), 8 at a time from the first 8-byte aligned one
    {
        const int mis = static_cast<int>((0 - reinterpret_cast<uintptr_t>(e.qflags)) & 7u);  // qflags + mis is aligned
        const int64_t a0 = q0 + ((mis - q0) & 7);
        const int64_t a1 = a0 + (q1 > a0 ? ((q1 - a0) & ~int64_t{7}) : 0);
        if (a0 < q1) {
            for (int64_t w = tid; w < ((a1 - a0) >> 3); w += kSortThreads)
                reinterpret_cast<uint64_t*>(e.qflags + a0)[w] = 0;
            if (tid < a0 - q0) e.qflags[q0 + tid] = 0;
            if (tid < q1 - a1) e.qflags[a1 + tid] = 0;
        } else {
            for (int64_t q = q0 + tid; q < q1; q += kSortThreads) e.qflags[q] = 0;
        }
    }
    auto place = [&](int64_t q, int c, int p) { s.perm[base + p] = make_int2(static_cast<int>(q), c); };
    // four queries per thread and step, the next step's ids loaded before this
    // step's entries are stored and taken (bins computed) after them: the wait
    // for those loads then leaves the scattered stores in flight (the memory
    // counter retires in issue order), and the ids of the first step are taken
    // before the loop, so that no wait at its top covers the stores either
    int64_t q = q0 + tid;
    if (q + 3 * kSortThreads < q1) {
        int c[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = e.ctx_id[q + u * kSortThreads];
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = query_bin(e, s, c[u]);
        for (;;) {
            const int64_t qn = q + 4 * kSortThreads;
            const bool more = qn + 3 * kSortThreads < q1;
            int cn[4], p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) cn[u] = e.ctx_id[more ? qn + u * kSortThreads : q];  // (a valid address)
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = atomicAdd(&sBin[b[u]], 1);
#pragma unroll
            for (int u = 0; u < 4; ++u) place(q + u * kSortThreads, c[u], p[u]);
            q = qn;
            if (!more) break;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = cn[u];
                b[u] = query_bin(e, s, cn[u]);
            }
        }
    }
    for (; q < q1; q += kSortThreads) {
        const int c = e.ctx_id[q];
        place(q, c, atomicAdd(&sBin[query_bin(e, s, c)], 1));
    }
}

// A bin of 2^bin_shift contexts keeps its queries in batch order, so its contexts
// interleave.  With many queries per context the sorted positions are regrouped
// chunk by chunk (kRegroupChunk positions, in LDS): key = the bin's offset from
// the chunk's first bin (clamped) and the context's low bits, so within a chunk
// spanning few bins every context's entries end contiguous.  Entries only move
// inside their chunk (chunks never straddle a window).
constexpr int kRegroupThreads = 1024;
constexpr int kRegroupPer = 4;
constexpr int kRegroupChunk = kRegroupThreads * kRegroupPer;  // 4096 positions, 12-bit keys

__global__ __launch_bounds__(kRegroupThreads) void k_enc_regroup(EncArgs e, SortArgs s) {
    __shared__ int sCount[kRegroupChunk];
    __shared__ int sWave[kRegroupThreads / 64];
    __shared__ int2 sEnt[kRegroupChunk];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kRegroupChunk;
    const int n = e.nq - c0 < kRegroupChunk ? static_cast<int>(e.nq - c0) : kRegroupChunk;
    const int b0 = query_bin(e, s, s.perm[c0].y);
    const int lb = s.bin_shift < 12 ? s.bin_shift : 12;  // keys stay below kRegroupChunk
    const int span = (kRegroupChunk >> lb) - 1;
    int2 ent[kRegroupPer];
    int key[kRegroupPer], rank[kRegroupPer];
#pragma unroll
    for (int u = 0; u < kRegroupPer; ++u) {
        const int k = tid + u * kRegroupThreads;
        ent[u] = k < n ? s.perm[c0 + k] : make_int2(0, 0);
        sCount[k] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRegroupPer; ++u) {
        const int k = tid + u * kRegroupThreads;
        key[u] = 0;
        rank[u] = 0;
        if (k < n) {  // positions past the batch take no slot
            const int db = query_bin(e, s, ent[u].y) - b0;  // >= 0: the chunk is in bin order
            key[u] = ((db < span ? db : span) << lb) | (ent[u].y & ((1 << lb) - 1));
            rank[u] = atomicAdd(&sCount[key[u]], 1);
        }
    }
    __syncthreads();
    // exclusive scan of the 4096 key counts: four consecutive keys per thread
    int cnt[kRegroupPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kRegroupPer; ++u) {
        cnt[u] = sCount[kRegroupPer * tid + u];
        sum += cnt[u];
    }
    int x = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    if (lane == 63) sWave[wave] = x;
    __syncthreads();
    int base = x - sum;
    for (int w = 0; w < wave; ++w) base += sWave[w];
#pragma unroll
    for (int u = 0; u < kRegroupPer; ++u) {
        sCount[kRegroupPer * tid + u] = base;
        base += cnt[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRegroupPer; ++u) {
        const int k = tid + u * kRegroupThreads;
        if (k < n) sEnt[sCount[key[u]] + rank[u]] = ent[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRegroupPer; ++u) {
        const int k = tid + u * kRegroupThreads;
        if (k < n) s.perm[c0 + k] = sEnt[k];
    }
}

// In grouped order the lanes of a wavefront mostly share one context.  Such a
// context's map columns and parity-check rows (or, with few basis rows, its
// basis rows and pivots) are staged in LDS by the whole wavefront with coalesced
// loads, and each lane masks the broadcast columns with its own phi bits: one
// sign-extended bit per column, where the per-lane path gathers a column per
// set bit with divergent addresses.  Staging capacity: contexts of up to 2
// feature words (d <= 128); the positions of wider ones, and of wavefronts with
// more than kSharedCtxPerWave contexts, are left to a second pass (k_encode_rest),
// which keeps this kernel's registers and LDS small (more wavefronts in flight
// to cover its three dependent memory round trips: entry, context scalars, stage).
// The second pass stages, in a stage of up to 4 feature words, each context that
// holds at least kRestStageLanes of a wavefront's remaining lanes, and gathers per
// lane for the others.
//
// A stage of SFW feature words: 64 SFW map columns of 16 bytes at words
// [0, 128 SFW), the parity-check rows (fewer than d / 2 + 1 of up to SFW words)
// from word 128 SFW; or, with few basis rows (r < d / 2), the basis rows and then
// the pivots as words.
template <int SFW>
struct StageGeom {
    static constexpr int cols = 64 * SFW;
    static constexpr int rows = 2 * cols;                  // first word of the parity-check rows
    static constexpr int words = rows + cols / 2 * SFW;    // SFW = 2: 3 KB, SFW = 4: 8 KB
    static_assert((cols / 2 - 1) * (SFW + F2_Y_WORDS + 1) <= words, "few-basis-row contexts fit the stage too");
};
constexpr int kEncStageFW = 2;  // the staged pass
constexpr int kEncWideFW = 4;   // the second pass
struct EncStage {
    uint64_t w[kEncThreads / 64][StageGeom<kEncStageFW>::words];
};
struct EncStageWide {
    uint64_t w[kEncThreads / 64][StageGeom<kEncWideFW>::words];
};

// the staged context's geometry (uniform)
struct StageCtx {
    int n, d, fw, r;
    bool rows;  // parity-check rows (else: basis rows)
};

// a context's scalars, all loads issued together (c valid)
struct CtxScalars {
    uint32_t flags;
    int n, r0;
    int64_t mo, bo, po;
};
__device__ __forceinline__ CtxScalars ctx_scalars(const EncArgs& e, int c) {
    CtxScalars v;
    v.flags = e.ctx_flags[c];
    v.n = e.n_bits[c];
    v.r0 = e.rank[c];
    v.mo = e.map_off[c];
    v.bo = e.basis_off[c];
    v.po = e.piv_off[c];
    // all six values taken here: the six loads go out together (else each is
    // sunk to its first use, behind the branches on the ones before)
    __asm__ volatile("" : : "s"(v.flags), "s"(v.n), "s"(v.r0), "s"(v.mo), "s"(v.bo), "s"(v.po));
    return v;
}

// whole wavefront: stage the context of v (valid, fw <= SFW) in the wavefront's LDS area
template <int SFW>
__device__ __forceinline__ StageCtx stage_context(const EncArgs& e, const CtxScalars& v, uint64_t* st) {
    const int lane = threadIdx.x & 63;
    StageCtx g;
    g.n = v.n;
    g.d = g.n + 1;
    g.fw = feat_words(g.n);
    g.r = v.r0 < 0 ? 0 : (v.r0 > g.d ? g.d : v.r0);
    g.rows = has_parity_rows(g.d, g.r);
    // every load of the stage is issued before the first LDS store (one round trip)
    using G = StageGeom<SFW>;
    if (g.rows) {  // columns at words [0, 2d), the t fw words of parity-check rows from G::rows
        constexpr int NM = 2 * G::cols / 64, NH = (G::words - G::rows) / 64;  // words per lane (d <= cols, t <= d / 2)
        const uint64_t* M = e.maps + v.mo;
        const uint64_t* H = e.tables + v.bo;
        const int nm = 2 * g.d, nh = (g.d - g.r) * g.fw;
        uint64_t a[NM], b[NH];
#pragma unroll
        for (int u = 0; u < NM; ++u) a[u] = lane + 64 * u < nm ? M[lane + 64 * u] : 0ull;
#pragma unroll
        for (int u = 0; u < NH; ++u) b[u] = lane + 64 * u < nh ? H[lane + 64 * u] : 0ull;
#pragma unroll
        for (int u = 0; u < NM; ++u)
            if (lane + 64 * u < nm) st[lane + 64 * u] = a[u];
#pragma unroll
        for (int u = 0; u < NH; ++u)
            if (lane + 64 * u < nh) st[G::rows + lane + 64 * u] = b[u];
    } else {  // basis rows (r (fw + 2) words, r < d / 2), then the pivots as words
        constexpr int NB = (G::cols / 2 * (SFW + F2_Y_WORDS) + 63) / 64, NP = (G::cols / 2 + 63) / 64;
        const uint64_t* B = e.basis + v.bo;
        const int32_t* P = e.pivots + v.po;
        const int nw = g.r * (g.fw + F2_Y_WORDS);
        uint64_t a[NB];
        int32_t b[NP];
#pragma unroll
        for (int u = 0; u < NB; ++u) a[u] = lane + 64 * u < nw ? B[lane + 64 * u] : 0ull;
#pragma unroll
        for (int u = 0; u < NP; ++u) b[u] = lane + 64 * u < g.r ? P[lane + 64 * u] : 0;
#pragma unroll
        for (int u = 0; u < NB; ++u)
            if (lane + 64 * u < nw) st[lane + 64 * u] = a[u];
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (lane + 64 * u < g.r) st[nw + lane + 64 * u] = static_cast<uint64_t>(b[u]);
    }
    wave_sync();
    return g;
}

template <int FW, int SFW>
__device__ __forceinline__ bool encode_staged(const EncArgs& e, const StageCtx& g, const uint64_t* st,
                                              const uint64_t* xq, const uint64_t (&xv)[4], uint64_t& z0,
                                              uint64_t& z1) {
    const int S = e.stride, n = g.n, d = g.d, fw = g.fw, cw = n >> 6;
    const uint64_t cbit = 1ull << (n & 63);
    bool outside = false;  // x bits at or above n
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w >= S) break;
        if (w > cw) outside |= xv[w] != 0;
        else if (w == cw) outside |= (xv[w] >> (n & 63)) != 0;
    }
    for (int w = 4; w < S; ++w) outside |= xq[w] != 0;  // staged contexts have fw <= 4: all of these are outside
    uint64_t ph[FW];
#pragma unroll
    for (int w = 0; w < FW; ++w) ph[w] = (w < fw ? xv[w] : 0ull) | (w == cw ? cbit : 0ull);
    if (g.rows) {
        // T(phi): every staged column, masked by its bit of phi (the columns past
        // n hold stale words, and their mask is zero).  A loop over 32-column
        // steps, unrolled within a step: fully unrolled, the code of every width
        // runs to several KB per wavefront and instruction fetch bounds the pass.
        const uint4* col = reinterpret_cast<const uint4*>(st);
        uint32_t a0 = 0, a1 = 0, a2 = 0, a3 = 0;
#pragma unroll 1
        for (int j0 = 0; j0 < d; j0 += 32) {
            uint64_t pw = ph[0];
#pragma unroll
            for (int k = 1; k < FW; ++k) pw = (j0 >> 6) == k ? ph[k] : pw;
            const uint32_t half = static_cast<uint32_t>(pw >> (j0 & 32));
#pragma unroll
            for (int u0 = 0; u0 < 32; u0 += 8) {
                if (j0 + u0 >= d) break;
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u) {
                    const uint4 v = col[j0 + u];
                    const uint32_t mk = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(half), u, 1));
                    a0 = __builtin_amdgcn_bitop3_b32(a0, mk, v.x, 0x78);
                    a1 = __builtin_amdgcn_bitop3_b32(a1, mk, v.y, 0x78);
                    a2 = __builtin_amdgcn_bitop3_b32(a2, mk, v.z, 0x78);
                    a3 = __builtin_amdgcn_bitop3_b32(a3, mk, v.w, 0x78);
                }
            }
        }
        z0 = (static_cast<uint64_t>(a1) << 32) | a0;
        z1 = (static_cast<uint64_t>(a3) << 32) | a2;
        // support: even overlap with every parity-check row
        const uint64_t* H = st + StageGeom<SFW>::rows;
        const int t = d - g.r;
        uint32_t odd = 0;
        for (int f = 0; f < t; ++f) {
            uint64_t acc = 0;
#pragma unroll
            for (int w = 0; w < FW; ++w)
                if (w < fw) acc ^= H[f * fw + w] & ph[w];
            odd |= static_cast<uint32_t>(__popcll(acc));
        }
        return (odd & 1u) == 0 && !outside;
    }
    // few basis rows: the rows whose pivot bit phi holds sum to [phi | T(phi)]
    // exactly when phi is in the span
    const int W = fw + F2_Y_WORDS;
    const uint64_t* piv = st + g.r * W;
    uint64_t acc[FW];
#pragma unroll
    for (int w = 0; w < FW; ++w) acc[w] = 0;
    uint64_t y0 = 0, y1 = 0;
    for (int k = 0; k < g.r; ++k) {
        const int p = static_cast<int>(piv[k]);
        uint64_t pwd = ph[0];
#pragma unroll
        for (int w = 1; w < FW; ++w) pwd = (p >> 6) == w ? ph[w] : pwd;
        const uint32_t mk = bit_mask(pwd, p & 63);
        const uint64_t* row = st + k * W;
#pragma unroll
        for (int w = 0; w < FW; ++w)
            if (w < fw) acc[w] = xor_and(acc[w], mk, row[w]);
        y0 = xor_and(y0, mk, row[fw]);
        y1 = xor_and(y1, mk, row[fw + 1]);
    }
    uint64_t diff = 0;
#pragma unroll
    for (int w = 0; w < FW; ++w) diff |= acc[w] ^ ph[w];
    z0 = y0;
    z1 = y1;
    return diff == 0 && !outside;
}

constexpr int kSharedCtxPerWave = 8;  // contexts of a wavefront taken through the stage

// a query's first x words (up to 4), 16 bytes at a time where the stride and
// the alignment allow
__device__ __forceinline__ void load_x4(const EncArgs& e, const uint64_t* xq, uint64_t (&xv)[4]) {
    const int S = e.stride;
    if (e.x16 && (S == 2 || S == 4)) {  // a query's words start 16-byte aligned
        const uint4* x4 = reinterpret_cast<const uint4*>(xq);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k >= S / 2) break;
            const uint4 v = x4[k];
            xv[2 * k] = (static_cast<uint64_t>(v.y) << 32) | v.x;
            xv[2 * k + 1] = (static_cast<uint64_t>(v.w) << 32) | v.z;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < S) xv[k] = xq[k];
    }
}

__global__ __launch_bounds__(kEncThreads) void k_encode_sorted(EncArgs e, SortArgs s) {
    __shared__ EncStage sStage;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kEncThreads + threadIdx.x;
    const bool live = i < e.nq;
    const int2 qc = live ? s.perm[i] : make_int2(0, 0);
    uint64_t* st = sStage.w[threadIdx.x >> 6];
    Word2 out, fl;
    out.x = out.y = 0;
    fl.x = fl.y = 0;
    bool done = !live;
    // the query's x words (up to 4) are loaded first: their latency overlaps the
    // context's scalars and the staging
    const uint64_t* xq = e.x + static_cast<int64_t>(live ? qc.x : 0) * e.stride;
    uint64_t xv[4] = {0, 0, 0, 0};
    if (live) load_x4(e, xq, xv);
    for (int k = 0; k < kSharedCtxPerWave; ++k) {  // the wavefront's contexts, first lane's first
        const uint64_t todo = __ballot(!done);
        if (!todo) break;
        const int c0 = __builtin_amdgcn_readlane(qc.y, ffs64(todo));
        const bool valid = c0 >= 0 && c0 < e.num_ctx;
        const CtxScalars v = ctx_scalars(e, valid ? c0 : 0);
        if (!valid || (v.flags & kBadCtx)) {
            if (!done && qc.y == c0) {
                fl.x = F2_Q_BAD_CTX;
                done = true;
            }
            continue;
        }
        if (feat_words(v.n) > kEncStageFW) break;  // wider: per-lane pass
        const StageCtx g = stage_context<kEncStageFW>(e, v, st);
        if (!done && qc.y == c0) {
            fl.x = (v.flags & F2_CTX_CONTRADICTION) ? F2_Q_CTX_CONTRADICTORY : 0;
            const bool in = encode_staged<kEncStageFW, kEncStageFW>(e, g, st, xq, xv, out.x, out.y);
            if (!in) {
                fl.x |= F2_Q_OUT_OF_SPAN;
                out.x = out.y = 0;
            }
            done = true;
        }
        wave_sync();  // the stage is rewritten for the next context
    }
    const uint64_t left = __ballot(!done);  // lanes of further or wider contexts: second pass
    if (left) {  // a few percent of the groups (the second pass reads only these)
        const int n = e.wide ? __popcll(__ballot(for_wavefront(e, !done, qc.y))) : 0;
        const int more = n > kWideShare ? (n - 1) / kWideShare : 0;  // further shares of wide queries
        if ((threadIdx.x & 63) == 0) {
            s.rest[i >> 6] = left;
            s.rest_list[atomicAdd(s.rest_count, 1)] = static_cast<int32_t>(i >> 6) | (more << kRestMore);
        }
    }
    if (!done || !live) return;
    *reinterpret_cast<Word2*>(e.words + 2 * static_cast<int64_t>(qc.x)) = out;
    if (fl.x) e.qflags[qc.x] = static_cast<uint8_t>(fl.x);  // the scatter cleared the others
}

// the second pass over the grouped order: the positions the staged pass left
// (their groups in s.rest_list, their lanes in s.rest).  Each context of the
// group (up to kEncWideFW feature words) is staged in turn, however few of the
// group's lanes it holds: on 100M Zipf queries that is 0.55 ms against 0.64 with
// per-lane gathers for contexts of fewer than 16 lanes; bad contexts, those of 5-8
// words and wide ones of full rank go per lane.  A fixed grid whose wavefronts take the listed groups in turn: a grid
// over every position would launch (and allocate the stage for) a workgroup per
// 256 positions, almost all of them idle (1.2 against 0.42 ms on 100M queries).
// A group's wide queries are a wavefront's each, kWideShare of them in this wavefront and the rest shared
// out: a large batch may hold a few such groups, and 64 queries one after the other would be the
// kernel's time (3M queries on 3,000 narrow contexts and 20 of 700 bits at rank 560: 1,090 us so, 650 now, 742 with
// a lane for each).
constexpr int kRestStageLanes = 1;
constexpr int kRestCtxPerWave = 64;  // contexts of a wavefront considered for the stage (all of them)
constexpr int kRestGrid = 2048;     // workgroups of the listed-group pass (100M queries: 0.50 ms; 1,024: 0.54)

// one wavefront: the lanes of bits among positions i0 .. i0 + 63 (of the wide queries one share)
template <bool WIDE>
__device__ __forceinline__ void rest_group(const EncArgs& e, const SortArgs& s, uint64_t* st, int64_t i0,
                                           uint64_t bits, int share) {
    const int lane = threadIdx.x & 63;
    const int64_t i = i0 + lane;
    const bool live = i < e.nq && ((bits >> lane) & 1ull);
    if (!__ballot(live)) return;
    const int2 qc = live ? s.perm[i] : make_int2(0, 0);
    const uint64_t* xq = e.x + static_cast<int64_t>(live ? qc.x : 0) * e.stride;
    uint64_t xv[4] = {0, 0, 0, 0};
    if (live && share == 0) load_x4(e, xq, xv);
    Word2 out;
    out.x = out.y = 0;
    uint8_t fl = 0;
    bool done = !live, lane_path = false;
    for (int k = 0; k < (share == 0 ? kRestCtxPerWave : 0); ++k) {
        const uint64_t todo = __ballot(!done && !lane_path);
        if (!todo) break;
        const int c0 = __builtin_amdgcn_readlane(qc.y, ffs64(todo));
        const bool mine = !done && !lane_path && qc.y == c0;
        bool stage = c0 >= 0 && c0 < e.num_ctx && __popcll(__ballot(mine)) >= kRestStageLanes;
        CtxScalars v;
        if (stage) {
            v = ctx_scalars(e, c0);
            stage = !(v.flags & kBadCtx) && feat_words(v.n) <= kEncWideFW;
        }
        if (!stage) {  // few lanes, or a bad or wide context: per lane
            if (mine) lane_path = true;
            continue;
        }
        const StageCtx g = stage_context<kEncWideFW>(e, v, st);
        if (mine) {
            fl = (v.flags & F2_CTX_CONTRADICTION) ? F2_Q_CTX_CONTRADICTORY : 0;
            const bool in = encode_staged<kEncWideFW, kEncWideFW>(e, g, st, xq, xv, out.x, out.y);
            if (!in) {
                fl |= F2_Q_OUT_OF_SPAN;
                out.x = out.y = 0;
            }
            done = true;
        }
        wave_sync();  // the stage is rewritten for the next context
    }
    bool mine = !done;
    const uint8_t lf = encode_lanes<WIDE>(e, mine, qc.y, qc.x, out, share);
    if (mine) fl = lf;
    if (!mine && !(live && done)) return;
    *reinterpret_cast<Word2*>(e.words + 2 * static_cast<int64_t>(qc.x)) = out;
    if (fl) e.qflags[qc.x] = fl;
}

template <bool WIDE>
__global__ __launch_bounds__(kEncThreads) void k_encode_rest(EncArgs e, SortArgs s) {
    __shared__ EncStageWide sStage;
    const int wave = threadIdx.x >> 6;
    uint64_t* st = sStage.w[wave];
    const int cnt = *s.rest_count;
    const int waves = static_cast<int>(gridDim.x) * (kEncThreads / 64);
    for (int k = static_cast<int>(blockIdx.x) * (kEncThreads / 64) + wave; k < cnt; k += waves) {
        const int g = __builtin_amdgcn_readfirstlane(s.rest_list[k]) & ((1 << kRestMore) - 1);
        rest_group<WIDE>(e, s, st, static_cast<int64_t>(g) * 64, s.rest[g], 0);
    }
    if constexpr (WIDE) {  // the further shares; 64 (group, share) pairs looked at together
        const int lane = threadIdx.x & 63;
        const int64_t pairs = static_cast<int64_t>(cnt) * (64 / kWideShare - 1);
        for (int64_t k0 = static_cast<int64_t>(blockIdx.x) * (kEncThreads / 64) + wave; k0 < pairs; k0 += 64 * static_cast<int64_t>(waves)) {
            const int64_t k = k0 + static_cast<int64_t>(lane) * waves;
            const int share = k < pairs ? 1 + static_cast<int>(k / cnt) : 0;
            const int v = share ? s.rest_list[k % cnt] : 0;
            for (uint64_t todo = __ballot(share && (v >> kRestMore) >= share); todo; todo &= todo - 1) {
                const int l = ffs64(todo), g = __builtin_amdgcn_readlane(v, l) & ((1 << kRestMore) - 1);
                rest_group<true>(e, s, st, static_cast<int64_t>(g) * 64, s.rest[g], __builtin_amdgcn_readlane(share, l));
            }
        }
    }
}

// grouped order without the staged pass (bins of several contexts, not
// regrouped): every position per lane, the lanes of a wavefront gathering from
// the few maps of its bins
template <bool WIDE>
__global__ __launch_bounds__(kEncThreads) void k_encode_lanes(EncArgs e, SortArgs s) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kEncThreads + threadIdx.x;
    bool live = i < e.nq;
    const int2 qc = live ? s.perm[i] : make_int2(0, -1);
    Word2 out;
    const uint8_t fl = encode_lanes<WIDE>(e, live, qc.y, qc.x, out);
    if (!live) return;
    *reinterpret_cast<Word2*>(e.words + 2 * static_cast<int64_t>(qc.x)) = out;
    if (fl) e.qflags[qc.x] = fl;
}

// ---------------------------------------------------------------------------
// feature vectors of Eq. 1 as fit rows, and the post-encode word merges: plain
// streaming kernels, one output word (vectorize) or one 128-bit word (merge)
// per thread, reads and writes coalesced
// ---------------------------------------------------------------------------
constexpr int kStreamThreads = 256;

// each workgroup writes the kVecRows rows from blockIdx * kVecRows on; the row of
// an output word is its index in the workgroup's span times magic = ceil(2^32 / rw)
// (exact: the span is under 2^15 words and rw <= 66)
constexpr int kVecRows = 256;
// words in flight per thread (7.24M rows of 5 values: 199 us with 1, 175 with 2, 166 with 4 = 5.2 TB/s, 164 with 8, which
// more of a short row's span leaves empty)
constexpr int kVecStep = 4;

__global__ __launch_bounds__(kStreamThreads) void k_vectorize(const uint64_t* values, const uint64_t* y,
                                                              int64_t num_rows, int k, uint64_t keep0,
                                                              uint64_t keep1, uint64_t* rows, uint32_t magic) {
    const int rw = k + 3;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kVecRows;
    const int nr = num_rows - r0 < kVecRows ? static_cast<int>(num_rows - r0) : kVecRows;
    const uint64_t* vals = values + r0 * k;
    const uint64_t* yr = y ? y + 2 * r0 : nullptr;
    uint64_t* out = rows + r0 * rw;
    // kVecStep words per thread at a time, every load in flight before the first store
    for (int w0 = threadIdx.x; w0 < nr * rw; w0 += kVecStep * kStreamThreads) {
        uint64_t v[kVecStep];
#pragma unroll
        for (int u = 0; u < kVecStep; ++u) {
            const int w = w0 + u * kStreamThreads;
            const int r = static_cast<int>(__umulhi(static_cast<uint32_t>(w), magic));
            const int j = w - r * rw;
            v[u] = j == k ? 1 : 0;  // the constant feature; without outputs, zeros
            if (w < nr * rw && j < k) v[u] = vals[r * k + j];
            else if (w < nr * rw && j > k && yr) v[u] = yr[2 * r + (j - k - 1)] & (j == k + 1 ? keep0 : keep1);
        }
#pragma unroll
        for (int u = 0; u < kVecStep; ++u)
            if (w0 + u * kStreamThreads < nr * rw) out[w0 + u * kStreamThreads] = v[u];
    }
}

__global__ __launch_bounds__(kStreamThreads) void k_merge(const uint64_t* words, const uint64_t* field, int shift,
                                                          int width, uint64_t mask0, uint64_t mask1,
                                                          const uint64_t* state, int64_t n, uint64_t* out) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kStreamThreads + threadIdx.x;
    if (q >= n) return;
    const Word2 w = *reinterpret_cast<const Word2*>(words + 2 * q);
    uint64_t lo = w.x, hi = w.y;
    if (field) {
        const uint64_t f = width >= 64 ? field[q] : (field[q] & ((1ull << width) - 1));
        if (shift == 0) {
            lo ^= f;
        } else if (shift < 64) {
            lo ^= f << shift;
            hi ^= f >> (64 - shift);
        } else {
            hi ^= f << (shift - 64);
        }
    }
    uint64_t s0 = 0, s1 = 0;
    if (state) {
        const Word2 st = *reinterpret_cast<const Word2*>(state + 2 * q);
        s0 = st.x;
        s1 = st.y;
    }
    Word2 r;
    r.x = (lo & ~mask0) | (s0 & mask0);
    r.y = (hi & ~mask1) | (s1 & mask1);
    *reinterpret_cast<Word2*>(out + 2 * q) = r;
}

// ---------------------------------------------------------------------------
// basis pooling: contexts trained separately (one per exact group) are tested
// for one shared map by eliminating their bases together.  The members' basis
// rows are concatenated per pool (count -> scan -> copy) and fitted by the fit
// kernels as ordinary row streams; a pool is shared when that fit finds no
// contradiction and its members are valid, consistent and of equal width and
// output mask.
// ---------------------------------------------------------------------------
struct PoolArgs {
    int32_t num_ctx;  // members' model
    const int32_t* n_bits;
    const int64_t* basis_off;
    const uint64_t* basis;
    const int32_t* rank;
    const uint32_t* ctx_flags;
    const uint64_t* out_mask;  // [2 num_ctx] or null
    int32_t num_pools;
    const int64_t* pool_off;   // [num_pools + 1] into members
    const int32_t* members;
    int64_t num_members;
    const int32_t* pooled_n;   // widths of the pooled contexts
    const uint32_t* pooled_flags;
    uint32_t* pool_flags;
    int64_t* row_off;          // [num_pools + 1]: row words per pool, then their offsets
    uint64_t* rows;
    int64_t rows_cap;
    int64_t* blk;              // [ceil(num_pools / 256) + 1]: words per block of 256 pools, then their
                               // offsets; last: the total, or -1 when it exceeds rows_cap
};

constexpr uint32_t kPoolNoRows = F2_POOL_BAD_MEMBER | F2_POOL_WIDTH_MISMATCH;

__global__ __launch_bounds__(256) void k_pool_count(PoolArgs P) {
    const int p0 = blockIdx.x * 256 + threadIdx.x;
    const bool live = p0 < P.num_pools;
    const int p = live ? p0 : P.num_pools - 1;  // lanes past the end redo the last pool and store nothing
    const int64_t lo = P.pool_off[p], hi = P.pool_off[p + 1];
    const int n = P.pooled_n[p];
    const int64_t W = feat_words(n < 0 ? 0 : n) + F2_Y_WORDS;
    uint32_t fl = (lo < 0 || hi < lo || hi > P.num_members || n < 0 || n > F2_MAX_N_BITS) ? F2_POOL_BAD_MEMBER : 0u;
    int64_t words = 0;
    uint64_t m0 = 0, m1 = 0;
    for (int64_t e = lo; e < hi && !(fl & F2_POOL_BAD_MEMBER); ++e) {
        const int c = P.members[e];
        if (c < 0 || c >= P.num_ctx || P.ctx_flags[c] != 0) {  // out of range, malformed or contradictory
            fl |= F2_POOL_BAD_MEMBER;
            break;
        }
        if (P.n_bits[c] != n) fl |= F2_POOL_WIDTH_MISMATCH;
        if (P.out_mask) {
            const uint64_t a0 = P.out_mask[2 * c], a1 = P.out_mask[2 * c + 1];
            if (e == lo) {
                m0 = a0;
                m1 = a1;
            } else if (a0 != m0 || a1 != m1) {
                fl |= F2_POOL_MASK_MISMATCH;
            }
        }
        words += static_cast<int64_t>(P.rank[c]) * W;
    }
    if (live) {
        P.pool_flags[p] = fl;
        P.row_off[p] = (fl & kPoolNoRows) ? 0 : words;
    }
    // the block's words
    __shared__ int64_t sSum[4];
    int64_t v = (!live || (fl & kPoolNoRows)) ? 0 : words;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((threadIdx.x & 63) == 0) sSum[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < 4; ++w) t += sSum[w];
        P.blk[blockIdx.x] = t;
    }
}

// one workgroup: exclusive scan of the blocks' words (1024 blocks at a time,
// coalesced); the last entry gets the total, or -1 beyond the buffer (a context
// in several pools), which empties every pool and flags it
__global__ __launch_bounds__(1024) void k_pool_scan(PoolArgs P) {
    __shared__ int64_t sWave[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int nblk = (P.num_pools + 255) / 256;
    int64_t carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 1024) {
        const int b = b0 + tid;
        const int64_t v = b < nblk ? P.blk[b] : 0;
        int64_t x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(x, o);
            if (lane >= o) x += t;
        }
        if (lane == 63) sWave[tid >> 6] = x;
        __syncthreads();
        int64_t run = x - v, total = 0;
        for (int w = 0; w < 16; ++w) {
            total += sWave[w];
            if (w < (tid >> 6)) run += sWave[w];
        }
        if (b < nblk) P.blk[b] = carry + run;
        carry += total;
        __syncthreads();  // sWave is rewritten by the next chunk
    }
    if (tid == 0) P.blk[nblk] = carry > P.rows_cap ? -1 : carry;
}

// the pools' row offsets: the blocks before their own, plus the scan within the block.  Up to
// kPoolSumBlocks blocks (262,144 pools) each sums the others' words itself: at most four
// loads per thread, against the 4.4 us of a launch of the scan; beyond, the sums would grow with
// the square of the pools.
constexpr int kPoolSumBlocks = 1024;
__global__ __launch_bounds__(256) void k_pool_offsets(PoolArgs P, bool scanned) {
    __shared__ int64_t sWave[4], sBase[4], sTotal[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int p = blockIdx.x * 256 + tid;
    const int nblk = (P.num_pools + 255) / 256;
    const bool live = p < P.num_pools;
    const int64_t v = live ? P.row_off[p] : 0;
    int64_t total = 0, base = 0;
    if (scanned) {
        total = P.blk[nblk];
        base = P.blk[blockIdx.x];
    } else {
        for (int b = tid; b < nblk; b += 256) {
            const int64_t w = P.blk[b];
            total += w;
            base += b < static_cast<int>(blockIdx.x) ? w : 0;
        }
        for (int o = 32; o > 0; o >>= 1) {
            total += __shfl_down(total, o);
            base += __shfl_down(base, o);
        }
        if (lane == 0) {
            sTotal[tid >> 6] = total;
            sBase[tid >> 6] = base;
        }
        __syncthreads();
        total = sTotal[0] + sTotal[1] + sTotal[2] + sTotal[3];
        base = sBase[0] + sBase[1] + sBase[2] + sBase[3];
        if (total > P.rows_cap) total = -1;
    }
    int64_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    if (lane == 63) sWave[tid >> 6] = x;
    __syncthreads();
    int64_t run = base + x - v;
    for (int w = 0; w < (tid >> 6); ++w) run += sWave[w];
    const bool over = total < 0;
    if (live) {
        P.row_off[p] = over ? 0 : run;
        if (over) P.pool_flags[p] |= F2_POOL_BAD_MEMBER;
    }
    if (p == P.num_pools - 1) P.row_off[P.num_pools] = over ? 0 : total;
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int i) {
    return (static_cast<int64_t>(__builtin_amdgcn_readlane(static_cast<int32_t>(v >> 32), i)) << 32) |
           static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int32_t>(v), i));
}

// one wavefront per pool: the members' basis rows, in member order, each in its
// stored order.  Bound by the latency of a wavefront's loads: four words per lane in flight
// took the copy of 80,000 pools of 4 from 83 to 56 us (one word at a time before).  Up to 64 members at a time, one per lane (their ranks and
// offsets loaded together); every lane then copies words of the group's output,
// the member of each word found among the lanes' prefixes.
__global__ __launch_bounds__(256) void k_pool_copy(PoolArgs P) {
    const int lane = threadIdx.x & 63;
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (p >= P.num_pools) return;
    // (loaded together: a wavefront's life is its chain of loads)
    const uint32_t fl = P.pool_flags[p];
    const int64_t lo = P.pool_off[p], hi = P.pool_off[p + 1];
    const int n = P.pooled_n[p];
    int64_t dst = P.row_off[p];
    asm volatile("" ::"v"(fl), "v"(lo), "v"(hi), "v"(n), "v"(dst));
    if (fl & kPoolNoRows) return;
    const int64_t W = feat_words(n) + F2_Y_WORDS;
    for (int64_t e0 = lo; e0 < hi; e0 += 64) {
        const int64_t e = e0 + lane;
        int64_t words = 0, src = 0;
        if (e < hi) {
            const int c = P.members[e];
            words = static_cast<int64_t>(P.rank[c]) * W;
            src = P.basis_off[c];
        }
        int64_t x = words;  // inclusive prefix over the group's members
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(x, o);
            if (lane >= o) x += t;
        }
        const int64_t pre = x - words;
        const int64_t total = __shfl(x, 63);
        const int nm = hi - e0 < 64 ? static_cast<int>(hi - e0) : 64;
        // U words per lane at a time, their loads in flight together.  The member holding
        // output word k is the last with prefix <= k (its prefix and source offset, as
        // source - prefix, read from its lane by readlane, which, unlike a permute, also
        // reads lanes that a loop has left inactive).
        constexpr int U = 4;
        const int64_t from = src - pre;
        for (int64_t k0 = lane; k0 < total; k0 += U * 64) {
            int64_t at[U];
            uint64_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) at[u] = readlane64(from, 0);
            for (int i = 1; i < nm; ++i) {
                const int64_t pi = readlane64(pre, i), fi = readlane64(from, i);
#pragma unroll
                for (int u = 0; u < U; ++u) at[u] = k0 + u * 64 >= pi ? fi : at[u];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = k0 + u * 64 < total ? P.basis[at[u] + k0 + u * 64] : 0ull;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u * 64 < total) P.rows[dst + k0 + u * 64] = v[u];
        }
        dst += total;
    }
}

__global__ __launch_bounds__(256) void k_pool_finish(PoolArgs P) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= P.num_pools) return;
    uint32_t fl = P.pool_flags[p];
    if (P.pooled_flags[p] & F2_CTX_CONTRADICTION) fl |= F2_POOL_CONTRADICTION;
    P.pool_flags[p] = fl ? fl : F2_POOL_SHARED;
}


// ---------------------------------------------------------------------------
// interleaved-stream ingestion: the rows of many contexts arrive mixed, in
// stream order (Sec. 3: observations are gathered across a corpus); the fit takes
// each context's rows contiguous and in stream order.  A stable LSD radix sort of the row
// indices by context, 9 bits per pass (per-block LDS histograms, the column scan of the
// encode sort, a stable scatter that sorts a tile in LDS and writes runs), then one gather
// copies each row, trimmed to its context's row width, to its place.  Rows of an out-of-range
// context sort last and are dropped; a context whose width is outside [0, F2_MAX_N_BITS] or
// needs more words than the stride gives its rows no words.
// ---------------------------------------------------------------------------
constexpr int kGrpDigitBits = 9;  // two passes up to 2^18 - 1 contexts
constexpr int kGrpBins = 1 << kGrpDigitBits;
constexpr int kGrpThreads = 1024;
constexpr int kGrpWaves = kGrpThreads / 64;
constexpr int kGrpSteps = 16;  // scatter: 64-row steps per wavefront and tile
constexpr int kGrpTile = kGrpThreads * kGrpSteps;

struct GroupArgs {
    int32_t num_ctx;
    const int32_t* n_bits;
    const int32_t* ctx_id;
    const uint64_t* rows;
    int32_t stride;
    int64_t nr;             // rows
    int32_t blocks;
    int64_t qc;             // rows per count / scatter block
    int32_t shift;          // digit of this pass: (key >> shift) & (kGrpBins - 1)
    const int32_t* in;      // keys of the previous pass, or null (first pass: from ctx_id)
    const int32_t* in_row;  // and their rows (first pass: in stream order)
    int32_t* out;           // this pass's keys, sorted up to its digit
    int32_t* out_row;       // and their rows
    int32_t* hist;          // [blocks][kGrpBins]
    int32_t* total;         // [kGrpBins]
    int2* bound;            // [num_ctx] first sorted position and end (0: no rows) of each context;
                            // then GroupDest
    int64_t* blk;           // [ceil(num_ctx / 1024)] words per block of contexts (scanned: before it)
    uint64_t* rows_out;
    int64_t* row_off;       // [num_ctx + 1]
    int64_t* dropped;       // [1]
};

// the sort key of a row: its context, or num_ctx for a row of none.  (The width is left to the
// kernels that work per context: a lookup per row here took 25 us of 41 in the first
// count of 7.24M rows.)
__device__ __forceinline__ int group_key(const GroupArgs& g, int64_t r) {
    if (g.in) return g.in[r];
    const int c = g.ctx_id[r];
    return c < 0 || c >= g.num_ctx ? g.num_ctx : c;
}

// words of a row of context c, 0 where its rows are dropped
__device__ __forceinline__ int group_width(const GroupArgs& g, int c) {
    const int n = g.n_bits[c];
    if (n < 0 || n > F2_MAX_N_BITS) return 0;
    const int w = feat_words(n) + F2_Y_WORDS;
    return w <= g.stride ? w : 0;
}

// per-block histogram of the pass's digit; the first pass also clears what the later
// kernels write into.  Eight rows per thread and step, their loads in flight together.
__global__ __launch_bounds__(kGrpThreads) void k_grp_count(GroupArgs g) {
    __shared__ int sBin[kGrpBins];
    const int tid = threadIdx.x;
    if (tid < kGrpBins) sBin[tid] = 0;
    if (!g.in) {
        for (int64_t c = static_cast<int64_t>(blockIdx.x) * kGrpThreads + tid; c < g.num_ctx;
             c += static_cast<int64_t>(gridDim.x) * kGrpThreads)
            g.bound[c] = make_int2(0, 0);
        if (blockIdx.x == 0 && tid == 0) *g.dropped = 0;
    }
    __syncthreads();
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * g.qc;
    const int64_t r1 = r0 + g.qc < g.nr ? r0 + g.qc : g.nr;
    constexpr int U = 8;
    for (int64_t r = r0 + tid; r < r1; r += U * kGrpThreads) {
        int k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = r + u * kGrpThreads < r1 ? group_key(g, r + u * kGrpThreads) : -1;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k[u] >= 0) atomicAdd(&sBin[(k[u] >> g.shift) & (kGrpBins - 1)], 1);
    }
    __syncthreads();
    if (tid < kGrpBins) g.hist[static_cast<int64_t>(blockIdx.x) * kGrpBins + tid] = sBin[tid];
}

// a & ~(m ^ b): bit k of the truth table is the result for (a, m, b) = the bits of k
__device__ __forceinline__ uint32_t same_bit(uint32_t a, uint32_t m, int b) {
    return static_cast<uint32_t>(__builtin_amdgcn_bitop3_b32(static_cast<int>(a), static_cast<int>(m), b, 0x90));
}

// stable scatter of a block's rows, a tile of up to kGrpTile at a time: each wavefront
// ranks a contiguous stretch of the tile, 64 rows a step (ballots of the digit bits give a
// row's rank among equal digits of its 64, the wavefront's own counter those before
// them), one scan over wavefronts and digits places them in LDS in sorted order, and the tile
// goes out in runs of equal digits (a run is 32 keys, 128 bytes, when 512 digits are equally
// common).  Bound by the chain of a step.  7.24M rows: 47 us a pass; scattering (key,
// row) pairs straight from registers took 94 us (512 open lines per block, which the XCD's L2
// evicts partly written).
__global__ __launch_bounds__(kGrpThreads) void k_grp_scatter(GroupArgs g) {
    __shared__ int sKey[kGrpTile], sRow[kGrpTile];
    __shared__ alignas(16) uint16_t sCnt[kGrpWaves][kGrpBins];  // at most kGrpTile: fits
    __shared__ int sLoc[kGrpBins], sGlob[kGrpBins];
    __shared__ int sSum[kGrpBins / 64], sTot[kGrpBins / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * g.qc;
    const int64_t r1 = r0 + g.qc < g.nr ? r0 + g.qc : g.nr;
    const int tiles = static_cast<int>((g.qc + kGrpTile - 1) / kGrpTile);
    // 64-row steps of a wavefront per tile, equal over the tiles
    const int steps = static_cast<int>(((g.qc + tiles - 1) / tiles + kGrpThreads - 1) / kGrpThreads);
    const int tile = steps * kGrpThreads;
    // a digit's next position: the digits before it over every block, then the blocks before this one
    int next = 0, own = 0;
    if (tid < kGrpBins) {
        own = g.total[tid];
        int x = own;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(x, o);
            if (lane >= o) x += t;
        }
        if (lane == 63) sTot[wave] = x;
        next = x - own + g.hist[static_cast<int64_t>(blockIdx.x) * kGrpBins + tid];
    }
    __syncthreads();
    if (tid < kGrpBins)
        for (int w = 0; w < wave; ++w) next += sTot[w];
    uint16_t* cnt = sCnt[wave];
    for (int64_t t0 = r0; t0 < r1; t0 += tile) {
        const int n = static_cast<int>(r1 - t0 < tile ? r1 - t0 : tile);
        const int e0 = wave * steps * 64 + lane;  // this lane's first element of the tile
        int key[kGrpSteps];
        int row[kGrpSteps];
        int rank[kGrpSteps];
#pragma unroll
        for (int u = 0; u < kGrpSteps; ++u) key[u] = u < steps && e0 + u * 64 < n ? group_key(g, t0 + e0 + u * 64) : -1;
#pragma unroll
        for (int u = 0; u < kGrpSteps; ++u) {
            const int64_t r = t0 + e0 + u * 64;
            row[u] = key[u] >= 0 && g.in ? g.in_row[r] : static_cast<int>(r);
        }
        *reinterpret_cast<uint4*>(&cnt[lane * 8]) = uint4{0, 0, 0, 0};
        wave_sync();
#pragma unroll
        for (int u = 0; u < kGrpSteps; ++u) {
            const bool live = key[u] >= 0;
            const int dg = (key[u] >> g.shift) & (kGrpBins - 1);
            const uint64_t alive = __ballot(live);
            uint32_t lo = static_cast<uint32_t>(alive), hi = static_cast<uint32_t>(alive >> 32);
#pragma unroll
            for (int b = 0; b < kGrpDigitBits; ++b) {  // keep the lanes whose bit is this lane's
                const int own_bit = (dg << (31 - b)) >> 31;
                const uint64_t m = __ballot(own_bit != 0);
                lo = same_bit(lo, static_cast<uint32_t>(m), own_bit);
                hi = same_bit(hi, static_cast<uint32_t>(m >> 32), own_bit);
            }
            const int before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
            const int all = __popc(lo) + __popc(hi);
            rank[u] = live ? cnt[dg] + before : 0;
            wave_sync();
            if (live && before == all - 1) cnt[dg] = static_cast<uint16_t>(rank[u] + 1);  // the digit's last lane
            wave_sync();
        }
        __syncthreads();
        int sum = 0, x = 0;
        if (tid < kGrpBins) {
#pragma unroll
            for (int w = 0; w < kGrpWaves; ++w) {  // exclusive prefix over the wavefronts
                const int c = sCnt[w][tid];
                sCnt[w][tid] = static_cast<uint16_t>(sum);
                sum += c;
            }
            x = sum;
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(x, o);
                if (lane >= o) x += t;
            }
            if (lane == 63) sSum[wave] = x;
        }
        __syncthreads();
        if (tid < kGrpBins) {
            int loc = x - sum;
            for (int w = 0; w < wave; ++w) loc += sSum[w];
            sLoc[tid] = loc;
            sGlob[tid] = next - loc;
            next += sum;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kGrpSteps; ++u)
            if (key[u] >= 0) {
                const int dg = (key[u] >> g.shift) & (kGrpBins - 1);
                const int i = sLoc[dg] + cnt[dg] + rank[u];
                sKey[i] = key[u];
                sRow[i] = row[u];
            }
        __syncthreads();
        // (the next tile's first barrier stands between these reads and its writes)
        for (int i = tid; i < n; i += kGrpThreads) {
            const int k = sKey[i];
            const int pos = sGlob[(k >> g.shift) & (kGrpBins - 1)] + i;
            g.out[pos] = k;
            g.out_row[pos] = sRow[i];
        }
    }
}

// first position and end of each context, rows of none (cleared by the first count); four sorted positions per thread
__global__ __launch_bounds__(256) void k_grp_bounds(GroupArgs g) {
    const int64_t i0 = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4;
    if (i0 >= g.nr) return;
    int k[6];  // the positions before and after too
    k[0] = i0 > 0 ? g.out[i0 - 1] : -1;
#pragma unroll
    for (int u = 0; u < 5; ++u) k[u + 1] = i0 + u < g.nr ? g.out[i0 + u] : -1;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u;
        if (i >= g.nr) break;
        const int c = k[u + 1];
        const bool start = c != k[u];
        if (c == g.num_ctx) {
            if (start) *g.dropped = g.nr - i;
            continue;
        }
        if (start) g.bound[c].x = static_cast<int32_t>(i);
        if (c != k[u + 2]) g.bound[c].y = static_cast<int32_t>(i + 1);
    }
}

// where a context's rows go: sorted position p lies at word base + p * width, kept as
// base << 8 | width in the 8 bytes of its bounds.  base may be negative; |base| < 2^31 * 66.
__device__ __forceinline__ int64_t group_dest(int64_t row_off, int first, int width) {
    return ((row_off - static_cast<int64_t>(first) * width) << 8) | width;
}

// words per context (and the rows of contexts of a bad width, to the dropped) and per block of 1024 contexts
__global__ __launch_bounds__(1024) void k_grp_words(GroupArgs g) {
    __shared__ int64_t sW[16];
    const int c = blockIdx.x * 1024 + threadIdx.x;
    int64_t v = 0;
    if (c < g.num_ctx) {
        const int2 b = g.bound[c];
        const int w = group_width(g, c);
        v = static_cast<int64_t>(b.y ? b.y - b.x : 0) * w;
        if (w == 0 && b.y)
            atomicAdd(reinterpret_cast<unsigned long long*>(g.dropped), static_cast<unsigned long long>(b.y - b.x));
        g.row_off[c] = v;
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((threadIdx.x & 63) == 0) sW[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < 16; ++w) t += sW[w];
        g.blk[blockIdx.x] = t;
    }
}

// one workgroup: exclusive scan of the blocks' words
__global__ __launch_bounds__(1024) void k_grp_scan(GroupArgs g) {
    __shared__ int64_t sWave[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int nblk = (g.num_ctx + 1023) / 1024;
    int64_t carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 1024) {
        const int b = b0 + tid;
        const int64_t v = b < nblk ? g.blk[b] : 0;
        int64_t x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(x, o);
            if (lane >= o) x += t;
        }
        if (lane == 63) sWave[tid >> 6] = x;
        __syncthreads();
        int64_t run = x - v, total = 0;
        for (int w = 0; w < 16; ++w) {
            total += sWave[w];
            if (w < (tid >> 6)) run += sWave[w];
        }
        if (b < nblk) g.blk[b] = carry + run;
        carry += total;
        __syncthreads();
    }
}

// each context's word offset: the blocks before its own, plus the scan within the block; the
// dropped-row count out.  Up to kGrpSumBlocks blocks (1M contexts) each sums those before it
// itself: at most one load per thread, against the 4.8 us of a launch of the scan; beyond, the
// sums would grow with the square of the contexts.
constexpr int kGrpSumBlocks = 1024;
__global__ __launch_bounds__(1024) void k_grp_offsets(GroupArgs g, bool scanned, int64_t* dropped_out) {
    __shared__ int64_t sWave[16], sBase[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int c = blockIdx.x * 1024 + tid;
    int64_t before = 0;
    if (scanned) {
        if (tid == 0) before = g.blk[blockIdx.x];
    } else if (tid < static_cast<int>(blockIdx.x)) {
        before = g.blk[tid];
    }
    for (int o = 32; o > 0; o >>= 1) before += __shfl_down(before, o);
    const int64_t v = c < g.num_ctx ? g.row_off[c] : 0;
    int64_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    if (lane == 0) sBase[tid >> 6] = before;
    if (lane == 63) sWave[tid >> 6] = x;
    __syncthreads();
    int64_t run = x - v;
    for (int w = 0; w < 16; ++w) run += sBase[w] + (w < (tid >> 6) ? sWave[w] : 0);
    if (c < g.num_ctx) {
        g.row_off[c] = run;
        reinterpret_cast<int64_t*>(g.bound)[c] = group_dest(run, g.bound[c].x, group_width(g, c));
    }
    if (c == g.num_ctx - 1) g.row_off[g.num_ctx] = run + v;
    if (blockIdx.x == 0 && tid == 0) *dropped_out = g.nr > 0 ? *g.dropped : 0;
}

// no contexts: every row is dropped
__global__ __launch_bounds__(64) void k_grp_none(int64_t nr, int64_t* row_off, int64_t* dropped_out) {
    if (threadIdx.x == 0) {
        row_off[0] = 0;
        *dropped_out = nr;
    }
}

// output rows: a gather in sorted order, each row trimmed to its context's width.  A
// wavefront takes 64 rows: a lane each finds source and destination, then LANES lanes per
// row copy its words, every load in flight before the first store.  Bound by the lines that
// the random rows touch (one or two of 128 bytes for the 24-40 that are kept).  7.24M rows
// of 7 words: 205 us; eight lanes per row that each looked up context and offset took 340
// us, and a copy in stream order with scattered writes 326 us (lines written in parts).
template <int LANES>
__global__ __launch_bounds__(256, 8) void k_grp_copy(GroupArgs g) {
    __shared__ int64_t sDest[4][64];
    __shared__ int sRow[4][64];
    constexpr int RPS = 64 / LANES;  // rows per step
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane % LANES, k = lane / LANES;
    const int64_t* __restrict__ dest = reinterpret_cast<const int64_t*>(g.bound);
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * 256 + wave * 64;
    if (i0 >= g.nr) return;
    const int64_t i = i0 + lane;
    const int c = i < g.nr ? g.out[i] : g.num_ctx;
    sRow[wave][lane] = i < g.nr ? g.out_row[i] : 0;
    const int64_t d = c < g.num_ctx ? dest[c] : 0;
    sDest[wave][lane] = d + ((i * (d & 255)) << 8);
    wave_sync();
    const uint64_t* src[LANES];
    int64_t e[LANES];
    uint64_t v[LANES];
#pragma unroll
    for (int u = 0; u < LANES; ++u) {
        e[u] = sDest[wave][u * RPS + k];
        src[u] = g.rows + static_cast<int64_t>(sRow[wave][u * RPS + k]) * g.stride;
        v[u] = j < static_cast<int>(e[u] & 255) ? src[u][j] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < LANES; ++u) {
        const int W = static_cast<int>(e[u] & 255);
        uint64_t* __restrict__ dst = g.rows_out + (e[u] >> 8);
        if (j < W) dst[j] = v[u];
        for (int w = j + LANES; w < W; w += LANES) dst[w] = src[u][w];
    }
}

inline size_t align256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }


// workspace of the grouping: two buffers of keys and rows, histograms, per-context bounds
struct GroupPlan {
    int blocks;
    int64_t qc;
    size_t off_a, off_b, off_hist, off_total, off_bound, off_blk, off_drop, bytes;
};
GroupPlan group_workspace(int32_t num_ctx, int64_t nr) {
    GroupPlan p{};
    int64_t blocks = (nr + 8191) / 8192;
    if (blocks > kMaxSortBlocks) blocks = kMaxSortBlocks;
    if (blocks < 1) blocks = 1;
    p.qc = (nr + blocks - 1) / blocks;
    if (p.qc < 1) p.qc = 1;
    p.blocks = static_cast<int>((nr + p.qc - 1) / p.qc);
    if (p.blocks < 1) p.blocks = 1;
    size_t o = 0;
    p.off_a = o;
    o = align256(o + 2 * sizeof(int32_t) * static_cast<size_t>(nr));
    p.off_b = o;
    o = align256(o + 2 * sizeof(int32_t) * static_cast<size_t>(nr));
    p.off_hist = o;
    o = align256(o + sizeof(int32_t) * static_cast<size_t>(p.blocks) * kGrpBins);
    p.off_total = o;
    o = align256(o + sizeof(int32_t) * kGrpBins);
    p.off_bound = o;
    o = align256(o + sizeof(int2) * static_cast<size_t>(num_ctx));
    p.off_blk = o;
    o = align256(o + sizeof(int64_t) * static_cast<size_t>((static_cast<int64_t>(num_ctx) + 1023) / 1024));
    p.off_drop = o;
    o = align256(o + sizeof(int64_t));
    p.bytes = o;
    return p;
}

// workgroups of a fit class kernel: at most one per context, at most `cap`
unsigned fit_grid(int num_ctx, int cap) { return static_cast<unsigned>(num_ctx < cap ? num_ctx : cap); }

// encode workspace: empty for the gather path; the sort buffers when the batch is
// large enough for grouping by context to pay off
struct EncPlan {
    bool sorted;
    int windows;
    SortArgs s;
    size_t off_hist, off_total, off_perm, off_rest, off_rest_list, off_rest_count, bytes;
};

int64_t encode_window();

// batches above this take the fine bins (an LDS histogram of up to 160 KB)
constexpr int64_t kFineBinQueries = int64_t{1} << 22;

EncPlan encode_workspace(int32_t num_ctx, int64_t nq) {
    EncPlan p{};
    p.bytes = 256;
    // grouping pays from about 160k queries on (4,096 contexts of 17-97 bits: the
    // gather path takes 31 us for 131k queries, the grouped one 36 us; at 197k 45 and 42 us)
    p.sorted = nq >= 3 * (1 << 16) && nq >= 4 * static_cast<int64_t>(num_ctx) && nq <= 0x7fffffff;
    if (!p.sorted) return p;
    const int64_t C = num_ctx > 0 ? num_ctx : 1;
    int shift = 0;
    // finer bins for large batches (100M Zipf queries over 80,000 contexts in
    // windows of 8M: 6.44 ms with 4 contexts per bin, 6.19 with 2); smaller ones
    // keep the small histogram (a 160 KB one costs its occupancy there)
    const int maxb = nq > kFineBinQueries ? kSortMaxBinsLarge : kSortMaxBins;
    while ((C + (int64_t{1} << shift) - 1) >> shift > maxb) ++shift;
    p.s.bin_shift = shift;
    p.s.nb = static_cast<int>((C + (int64_t{1} << shift) - 1) >> shift) + 1;
    // about 256 count / scatter blocks in all (one per compute unit, each with its
    // histogram), of at least 8k queries: enough blocks for the scatter, few
    // histogram rows to scan (1M queries: 83 us with 8k, 86 with 16k, 88 with 4k).
    // Above the window size the blocks form windows of bpw blocks; their size is a
    // multiple of kRegroupChunk, so no regrouped chunk straddles two windows.
    const int64_t wq = encode_window();
    const int64_t windows = (nq + wq - 1) / wq;
    int64_t qc, bpw;
    if (windows <= 1) {
        int64_t blocks = (nq + 8191) / 8192;
        if (blocks > kMaxSortBlocks) blocks = kMaxSortBlocks;
        qc = (nq + blocks - 1) / blocks;
        bpw = blocks;
    } else {
        bpw = kMaxSortBlocks / windows > 1 ? kMaxSortBlocks / windows : 1;
        const int64_t per_window = (nq + windows - 1) / windows;
        qc = (per_window + bpw - 1) / bpw;
        qc = (qc + kRegroupChunk - 1) / kRegroupChunk * kRegroupChunk;
    }
    p.s.qc = qc;
    p.s.blocks = static_cast<int>((nq + qc - 1) / qc);
    p.s.bpw = static_cast<int>(bpw < p.s.blocks ? bpw : p.s.blocks);
    p.windows = (p.s.blocks + p.s.bpw - 1) / p.s.bpw;
    size_t o = 0;
    p.off_hist = o;
    o = align256(o + sizeof(int32_t) * static_cast<size_t>(p.s.blocks) * p.s.nb);
    p.off_total = o;
    o = align256(o + sizeof(int32_t) * static_cast<size_t>(p.windows) * p.s.nb);
    p.off_perm = o;
    o = align256(o + sizeof(int2) * static_cast<size_t>(nq));
    // above kFineBinQueries bins of up to 4 contexts go to the staged pass as they
    // come (no regroup: 6.95 against 7.09 ms on 100M Zipf queries over 80,000
    // contexts); smaller batches regroup when bins hold several contexts and
    // contexts average 16 queries or more
    const bool fine = nq > kFineBinQueries && shift <= 2;
    p.s.regroup = !fine && shift > 0 && nq >= 16 * C;
    // with one context per bin, fine bins, or after the regroup, a wavefront holds
    // a few contexts and the staged pass applies; otherwise every position goes per lane
    p.s.staged = shift == 0 || fine || p.s.regroup;
    p.off_rest = o;
    o = align256(o + sizeof(uint64_t) * static_cast<size_t>((nq + 63) / 64));
    p.off_rest_list = o;
    o = align256(o + sizeof(int32_t) * static_cast<size_t>((nq + 63) / 64));
    p.off_rest_count = o;
    o = align256(o + sizeof(int32_t));
    p.bytes = o > 256 ? o : 256;
    return p;
}

// every output buffer of a model present and its sizes non-negative
bool model_complete(const f2_model* m) {
    return m->n_bits && m->basis_off && m->piv_off && m->map_off && m->basis && m->pivots && m->maps && m->tables &&
           m->rank && m->ctx_flags && m->n_contra && m->first_contra_row && m->basis_words >= 0 &&
           m->piv_entries >= 0 && m->map_words >= 0;
}

// polls of a group barrier before it gives up: 2^24 (seconds), or the value of
// F2GPU_GROUP_SPIN_LIMIT (a test hook for the timeout report)
int group_spin_limit() {
    const char* v = getenv("F2GPU_GROUP_SPIN_LIMIT");
    if (!v || !*v) return 1 << 24;
    char* end = nullptr;
    const long x = strtol(v, &end, 10);
    if (*end != '\0' || x < 0) return 1 << 24;
    return x > (1 << 24) ? (1 << 24) : static_cast<int>(x);
}

// queries per encode chunk: the grouped path indexes a batch's positions in 32
// bits, so larger batches are encoded in chunks of 2^30 (each grouped on its own,
// one after the other through one chunk-sized workspace); F2GPU_ENCODE_CHUNK may
// set a smaller chunk (a test hook for the chunking)
constexpr int64_t kEncChunk = int64_t{1} << 30;
int64_t encode_chunk() {
    const char* v = getenv("F2GPU_ENCODE_CHUNK");
    if (!v || !*v) return kEncChunk;
    char* end = nullptr;
    const long long x = strtoll(v, &end, 10);
    if (*end != '\0' || x < 1 || x > kEncChunk) return kEncChunk;
    return x;
}

// queries per sort window: kWindowQueries, or the value of F2GPU_ENCODE_WINDOW
// (a test hook: several windows at sizes the oracle checks quickly), at least
// 2^16 so that the per-window bin totals stay a small part of the workspace
int64_t encode_window() {
    const char* v = getenv("F2GPU_ENCODE_WINDOW");
    if (!v || !*v) return kWindowQueries;
    char* end = nullptr;
    const long long x = strtoll(v, &end, 10);
    if (*end != '\0' || x < 1 || x > kEncChunk) return kWindowQueries;
    return x < (int64_t{1} << 16) ? (int64_t{1} << 16) : x;
}

FitArgs fit_args(const uint64_t* rows, int64_t rows_words, const int64_t* row_off, const f2_model* m, int32_t* plan) {
    FitArgs a;
    a.rows = rows;
    a.rows_words = rows_words;
    a.row_off = row_off;
    a.num_ctx = m->num_ctx;
    a.n_bits = m->n_bits;
    a.basis_off = m->basis_off;
    a.piv_off = m->piv_off;
    a.map_off = m->map_off;
    a.basis_words = m->basis_words;
    a.piv_entries = m->piv_entries;
    a.map_words = m->map_words;
    a.basis = m->basis;
    a.pivots = m->pivots;
    a.maps = m->maps;
    a.tables = m->tables;
    a.rank = m->rank;
    a.ctx_flags = m->ctx_flags;
    a.n_contra = m->n_contra;
    a.first_contra = m->first_contra_row;
    a.plan = plan;
    a.coop = 0;
    a.max_n = m->max_n_bits;
    a.spin_limit = group_spin_limit();
    return a;
}

// workgroups of the wide kernel that can be resident at once on the current
// device, or 0 where cooperative launches are unavailable (queried once per device)
int wide_resident_workgroups() {
    static std::atomic<int> cache[64];  // value + 1; 0 = not queried yet
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
    if (dev < 64) {
        const int v = cache[dev].load(std::memory_order_relaxed);
        if (v > 0) return v - 1;
    }
    int coop = 0, cus = 0, per_cu = 0;
    int r = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) == hipSuccess && coop &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(k_fit_wide), kWdThreads,
                                                     0) == hipSuccess)
        r = cus * per_cu;
    (void)hipGetLastError();
    if (dev < 64) cache[dev].store(r + 1, std::memory_order_relaxed);
    return r;
}

// the fit: the plan (one kernel up to kPlanThreads contexts, else two), then the class
// kernels, each with about as many workgroups as fit on the chip at once.  The wide kernel runs one
// workgroup per compute unit as a cooperative launch (so that a group of
// workgroups can fit one context together), else a plain launch of up to 256.
constexpr int kPivGrid = 768;  // LDS-basis workgroups: three per compute unit (LDS-bound)
void launch_fit(FitArgs a, hipStream_t s) {
    const int32_t C = a.num_ctx;
    if (C <= kSmallBatch && a.max_n >= 0 && a.max_n < 512) {
        a.coop = 0;
        hipLaunchKernelGGL(k_fit_small, dim3(static_cast<unsigned>(C)), dim3(kSmallThreads), 0, s, a);
        return;
    }
    const int plan_blocks = static_cast<int>((static_cast<int64_t>(C) + kPlanThreads - 1) / kPlanThreads);
    if (C <= kPlanThreads) {
        hipLaunchKernelGGL(k_plan_one, dim3(1), dim3(kPlanThreads), 0, s, a);
    } else {
        hipLaunchKernelGGL(k_plan_count, dim3(plan_blocks), dim3(kPlanThreads), 0, s, a);
        hipLaunchKernelGGL(k_plan_scatter, dim3(plan_blocks), dim3(kPlanThreads), 0, s, a, plan_blocks);
    }
    hipLaunchKernelGGL(k_fit_reg, dim3(fit_grid(C, kRegGrid)), dim3(64 * kRegWaves), 0, s, a);
    if (C > kRegGrid)  // (else k_fit_reg has a workgroup for every context)
        hipLaunchKernelGGL(k_fit_piv, dim3(fit_grid(C, kPivGrid)), dim3(kPivThreads), 0, s, a);
    // a batch whose declared widths stay below 512 holds no wide context (wider
    // ones are rejected by the plan), so the wide kernel is not launched at all
    if (a.max_n >= 0 && a.max_n < 512) return;
    const int res = wide_resident_workgroups();
    if (res >= 32) {
        a.coop = 1;
        void* args[] = {&a};
        if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_fit_wide), dim3(res < kMaxMembers ? res : kMaxMembers),
                                       dim3(kWdThreads), args, 0, s) == hipSuccess)
            return;
        (void)hipGetLastError();
    }
    a.coop = 0;
    hipLaunchKernelGGL(k_fit_wide, dim3(fit_grid(C, 256)), dim3(kWdThreads), 0, s, a);
}

}  // namespace

extern "C" {

const char* f2_status_string(int status) {
    switch (status) {
        case F2_OK: return "ok";
        case F2_EINVAL: return "invalid argument";
        case F2_EWORKSPACE: return "workspace missing or too small";
        case F2_EDEVICE: return "HIP error while enqueuing device work";
        case F2_ETOOWIDE: return "context width above F2_MAX_N_BITS";
        case F2_ESCRATCH: return "batch above the allocation-free fit's fixed plan size (F2_NOALLOC_MAX_CTX contexts)";
        default: return "unknown status";
    }
}

int f2_fit_layout(const int32_t* n_bits_host, int32_t num_ctx, int64_t* basis_off_host, int64_t* piv_off_host,
                  int64_t* map_off_host) {
    if (num_ctx < 0 || !basis_off_host || !piv_off_host || !map_off_host || (num_ctx > 0 && !n_bits_host))
        return F2_EINVAL;
    int64_t bo = 0, po = 0, mo = 0;
    for (int32_t c = 0; c < num_ctx; ++c) {
        const int n = n_bits_host[c];
        if (n < 0) return F2_EINVAL;
        if (n > F2_MAX_N_BITS) return F2_ETOOWIDE;
        const int64_t d = n + 1, W = (n + 64) / 64 + F2_Y_WORDS;
        basis_off_host[c] = bo;
        piv_off_host[c] = po;
        map_off_host[c] = mo;
        bo += d * W;
        po += d;
        mo += 2 * d;
    }
    basis_off_host[num_ctx] = bo;
    piv_off_host[num_ctx] = po;
    map_off_host[num_ctx] = mo;
    return F2_OK;
}

size_t f2_fit_workspace_bytes(int32_t num_ctx) {
    if (num_ctx < 0) return 0;
    const size_t blocks = (static_cast<size_t>(num_ctx) + kPlanThreads - 1) / kPlanThreads;
    return align256(sizeof(int32_t) * (kPlanHead + 2 * static_cast<size_t>(num_ctx) + kPlanBins * blocks));
}

}  // extern "C"

namespace {

// ---------------------------------------------------------------------------
// allocation-free fit: the plan lives in a fixed device array instead of a
// caller workspace.  The array's name is a host-side stand-in; its device address
// is looked up once per device (hipGetSymbolAddress with that device current)
// and kept, and only that address is handed to kernels.  Every call on a device
// shares its array: calls that overlap on one device race.  The plan kernels
// initialise every plan word they read, so nothing stale carries over.
// ---------------------------------------------------------------------------
constexpr int32_t kScratchMaxCtx = F2_NOALLOC_MAX_CTX;
constexpr size_t kScratchBytes =
    (sizeof(int32_t) * (kPlanHead + 2 * static_cast<size_t>(kScratchMaxCtx) +
                        kPlanBins * ((static_cast<size_t>(kScratchMaxCtx) + kPlanThreads - 1) / kPlanThreads)) +
     255) / 256 * 256;
constexpr int kScratchDevices = 64;

__device__ __align__(256) uint8_t scratch[kScratchBytes];

// device address of this device's scratch array, or nullptr if it cannot be found
void* scratch_address() {
    static std::atomic<void*> addr[kScratchDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchDevices) return nullptr;
    void* p = addr[dev].load(std::memory_order_acquire);
    if (p) return p;
    void* q = nullptr;
    if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) {
        (void)hipGetLastError();
        return nullptr;
    }
    addr[dev].store(q, std::memory_order_release);  // the same address whichever thread looks it up
    return q;
}

}  // namespace

extern "C" {

int f2_fit_batch_noalloc(const uint64_t* rows, int64_t rows_words, const int64_t* row_off, const f2_model* m,
                         void* stream) {
    if (!m || m->num_ctx < 0 || rows_words < 0) return F2_EINVAL;
    const int32_t C = m->num_ctx;
    if (C == 0) return F2_OK;
    if (!row_off || !model_complete(m) || (rows_words > 0 && !rows)) return F2_EINVAL;
    if (C > kScratchMaxCtx || f2_fit_workspace_bytes(C) > kScratchBytes) return F2_ESCRATCH;
    void* plan = scratch_address();
    if (!plan) return F2_EDEVICE;
    launch_fit(fit_args(rows, rows_words, row_off, m, static_cast<int32_t*>(plan)), static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

int f2_fit_batch(const uint64_t* rows, int64_t rows_words, const int64_t* row_off, const f2_model* m,
                 void* workspace, size_t workspace_bytes, void* stream) {
    if (!m || m->num_ctx < 0 || rows_words < 0) return F2_EINVAL;
    const int32_t C = m->num_ctx;
    if (C == 0) return F2_OK;
    if (!row_off || !model_complete(m) || (rows_words > 0 && !rows)) return F2_EINVAL;
    if (!workspace || workspace_bytes < f2_fit_workspace_bytes(C) ||
        (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return F2_EWORKSPACE;
    launch_fit(fit_args(rows, rows_words, row_off, m, static_cast<int32_t*>(workspace)), static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

size_t f2_encode_workspace_bytes(const f2_model* m, int64_t num_queries) {
    if (!m || m->num_ctx < 0 || num_queries < 0) return 0;
    const int64_t chunk = encode_chunk();
    return encode_workspace(m->num_ctx, num_queries < chunk ? num_queries : chunk).bytes;
}

}  // extern "C"

namespace {

// one chunk of at most encode_chunk() queries (arguments checked by the caller)
int encode_range(const f2_model* m, const int32_t* ctx_id, const uint64_t* x, int32_t x_stride_words,
                 int64_t num_queries, uint64_t* words_out, uint8_t* qflags_out, void* workspace, hipStream_t s) {
    EncArgs e;
    e.num_ctx = m->num_ctx;
    e.n_bits = m->n_bits;
    e.basis_off = m->basis_off;
    e.piv_off = m->piv_off;
    e.basis = m->basis;
    e.pivots = m->pivots;
    e.rank = m->rank;
    e.ctx_flags = m->ctx_flags;
    e.map_off = m->map_off;
    e.maps = m->maps;
    e.tables = m->tables;
    e.ctx_id = ctx_id;
    e.x = x;
    e.stride = x_stride_words;
    e.x16 = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    e.nq = num_queries;
    e.words = words_out;
    e.qflags = qflags_out;
    const int64_t blocks = (num_queries + kEncThreads - 1) / kEncThreads;
    if (blocks > 0x7fffffff) return F2_EINVAL;
    EncPlan p = encode_workspace(m->num_ctx, num_queries);
    e.wide = m->max_n_bits < 0 || m->max_n_bits >= 64 * kLaneFW;
    if (!p.sorted && e.wide) {
        constexpr int per_block = kEncThreads / 64;
        int parts = 64;
        while (parts > per_block && num_queries * parts / 128 >= kWideWaves) parts /= 2;
        const int64_t wide_blocks = (num_queries + 63) / 64 * (parts / per_block);
        if (blocks + wide_blocks > 0x7fffffff) return F2_EINVAL;
        hipLaunchKernelGGL(k_encode_wide, dim3(static_cast<unsigned>(blocks + wide_blocks)), dim3(kEncThreads), 0, s, e,
                           static_cast<int>(blocks), parts);
        return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
    }
    if (!p.sorted) {
        hipLaunchKernelGGL(k_encode, dim3(static_cast<unsigned>(blocks)), dim3(kEncThreads), 0, s, e);
        return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
    }
    char* ws = static_cast<char*>(workspace);
    p.s.hist = reinterpret_cast<int32_t*>(ws + p.off_hist);
    p.s.total = reinterpret_cast<int32_t*>(ws + p.off_total);
    p.s.perm = reinterpret_cast<int2*>(ws + p.off_perm);
    p.s.rest = reinterpret_cast<uint64_t*>(ws + p.off_rest);
    p.s.rest_list = reinterpret_cast<int32_t*>(ws + p.off_rest_list);
    p.s.rest_count = reinterpret_cast<int32_t*>(ws + p.off_rest_count);
    const size_t bin_lds = sizeof(int) * static_cast<size_t>(p.s.nb);
    hipLaunchKernelGGL(k_enc_count, dim3(p.s.blocks), dim3(kSortThreads), bin_lds, s, e, p.s);
    hipLaunchKernelGGL(k_enc_colscan, dim3(static_cast<unsigned>(p.windows) * ((p.s.nb + 63) / 64)),
                       dim3(64 * kColWaves), 0, s, p.s);
    hipLaunchKernelGGL(k_enc_scatter, dim3(p.s.blocks), dim3(kSortThreads), bin_lds, s, e, p.s);
    if (p.s.regroup)
        hipLaunchKernelGGL(k_enc_regroup, dim3(static_cast<unsigned>((num_queries + kRegroupChunk - 1) / kRegroupChunk)),
                           dim3(kRegroupThreads), 0, s, e, p.s);
    if (p.s.staged) {
        hipLaunchKernelGGL(k_encode_sorted, dim3(static_cast<unsigned>(blocks)), dim3(kEncThreads), 0, s, e, p.s);
        hipLaunchKernelGGL(e.wide ? k_encode_rest<true> : k_encode_rest<false>, dim3(static_cast<unsigned>(blocks < kRestGrid ? blocks : kRestGrid)),
                           dim3(kEncThreads), 0, s, e, p.s);
    } else {
        hipLaunchKernelGGL(e.wide ? k_encode_lanes<true> : k_encode_lanes<false>, dim3(static_cast<unsigned>(blocks)), dim3(kEncThreads), 0, s, e, p.s);
    }
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

}  // namespace

extern "C" {

int f2_encode_batch(const f2_model* m, const int32_t* ctx_id, const uint64_t* x, int32_t x_stride_words,
                    int64_t num_queries, uint64_t* words_out, uint8_t* qflags_out, void* workspace,
                    size_t workspace_bytes, void* stream) {
    if (!m || m->num_ctx < 0 || num_queries < 0 || x_stride_words < 1) return F2_EINVAL;
    if (num_queries == 0) return F2_OK;
    if (!ctx_id || !x || !words_out || !qflags_out) return F2_EINVAL;
    if (m->num_ctx > 0 && (!m->n_bits || !m->basis_off || !m->piv_off || !m->map_off || !m->basis || !m->pivots ||
                           !m->maps || !m->tables || !m->rank || !m->ctx_flags))
        return F2_EINVAL;
    if (!workspace || workspace_bytes < f2_encode_workspace_bytes(m, num_queries) ||
        (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return F2_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // chunks in stream order through the one workspace
    const int64_t chunk = encode_chunk();
    for (int64_t q0 = 0; q0 < num_queries; q0 += chunk) {
        const int64_t n = num_queries - q0 < chunk ? num_queries - q0 : chunk;
        const int st = encode_range(m, ctx_id + q0, x + q0 * x_stride_words, x_stride_words, n, words_out + 2 * q0,
                                    qflags_out + q0, workspace, s);
        if (st != F2_OK) return st;
    }
    return F2_OK;
}

int f2_vectorize_rows(const uint64_t* values, const uint64_t* y, int64_t num_rows, int32_t k,
                      const uint64_t* keep_host, uint64_t* rows_out, void* stream) {
    if (num_rows < 0 || k < 0 || k > 63 || !keep_host) return F2_EINVAL;
    if (num_rows == 0) return F2_OK;
    if ((k > 0 && !values) || !rows_out) return F2_EINVAL;
    const int64_t blocks = (num_rows + kVecRows - 1) / kVecRows;
    if (num_rows > (int64_t{1} << 56) || blocks > 0x7fffffff) return F2_EINVAL;
    const uint32_t rw = static_cast<uint32_t>(k + 3);
    const uint32_t magic = static_cast<uint32_t>(((uint64_t{1} << 32) + rw - 1) / rw);  // ceil(2^32 / rw)
    hipLaunchKernelGGL(k_vectorize, dim3(static_cast<unsigned>(blocks)), dim3(kStreamThreads), 0,
                       static_cast<hipStream_t>(stream), values, y, num_rows, k, keep_host[0], keep_host[1], rows_out,
                       magic);
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

int f2_merge_words(const uint64_t* words, const uint64_t* field, int32_t shift, int32_t width,
                   const uint64_t* mask_host, const uint64_t* state, int64_t num_words, uint64_t* out,
                   void* stream) {
    if (num_words < 0 || !mask_host) return F2_EINVAL;
    if (field && (width < 1 || width > 64 || shift < 0 || shift + width > 128)) return F2_EINVAL;
    if (num_words == 0) return F2_OK;
    if (!words || !out) return F2_EINVAL;
    const int64_t blocks = (num_words + kStreamThreads - 1) / kStreamThreads;
    if (blocks > 0x7fffffff) return F2_EINVAL;
    hipLaunchKernelGGL(k_merge, dim3(static_cast<unsigned>(blocks)), dim3(kStreamThreads), 0,
                       static_cast<hipStream_t>(stream), words, field, field ? shift : 0, field ? width : 64,
                       mask_host[0], mask_host[1], state, num_words, out);
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

size_t f2_pool_workspace_bytes(const f2_model* members_model, int32_t num_pools) {
    if (!members_model || members_model->basis_words < 0 || num_pools < 0) return 0;
    return align256(sizeof(int64_t) * (static_cast<size_t>(num_pools) + 1)) +
           align256(sizeof(uint64_t) * static_cast<size_t>(members_model->basis_words)) +
           align256(sizeof(int64_t) * (static_cast<size_t>((num_pools + 255) / 256) + 1)) +
           f2_fit_workspace_bytes(num_pools);
}

size_t f2_group_workspace_bytes(int32_t num_ctx, int64_t num_rows) {
    if (num_ctx < 0 || num_rows < 0 || num_rows > 0x7fffffff) return 0;
    return group_workspace(num_ctx, num_rows).bytes;
}

int f2_group_rows(const int32_t* ctx_id, const uint64_t* rows, int32_t row_stride_words, int64_t num_rows,
                  const int32_t* n_bits, int32_t num_ctx, uint64_t* rows_out, int64_t rows_out_words,
                  int64_t* row_off_out, int64_t* dropped_out, void* workspace, size_t workspace_bytes, void* stream) {
    if (num_ctx < 0 || num_rows < 0 || num_rows > 0x7fffffff || row_stride_words < F2_Y_WORDS + 1) return F2_EINVAL;
    if (!row_off_out || !dropped_out || (num_ctx > 0 && !n_bits)) return F2_EINVAL;
    if (num_rows > 0 && (!ctx_id || !rows || !rows_out || rows_out_words < num_rows * row_stride_words))
        return F2_EINVAL;
    if (!workspace || workspace_bytes < f2_group_workspace_bytes(num_ctx, num_rows) ||
        (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return F2_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const GroupPlan p = group_workspace(num_ctx, num_rows);
    char* ws = static_cast<char*>(workspace);
    GroupArgs g;
    g.num_ctx = num_ctx;
    g.n_bits = n_bits;
    g.ctx_id = ctx_id;
    g.rows = rows;
    g.stride = row_stride_words;
    g.nr = num_rows;
    g.blocks = p.blocks;
    g.qc = p.qc;
    g.hist = reinterpret_cast<int32_t*>(ws + p.off_hist);
    g.total = reinterpret_cast<int32_t*>(ws + p.off_total);
    g.bound = reinterpret_cast<int2*>(ws + p.off_bound);
    g.blk = reinterpret_cast<int64_t*>(ws + p.off_blk);
    g.rows_out = rows_out;
    g.row_off = row_off_out;
    g.dropped = reinterpret_cast<int64_t*>(ws + p.off_drop);
    int32_t* bufs[2] = {reinterpret_cast<int32_t*>(ws + p.off_a), reinterpret_cast<int32_t*>(ws + p.off_b)};
    // passes: kGrpDigitBits bits of the key (0 .. num_ctx) each
    int bits = 1;
    while ((int64_t{1} << bits) <= num_ctx) ++bits;
    const int passes = (bits + kGrpDigitBits - 1) / kGrpDigitBits;
    SortArgs cs{};
    cs.nb = kGrpBins;
    cs.blocks = p.blocks;
    cs.bpw = p.blocks;  // one window: every block
    cs.hist = g.hist;
    cs.total = g.total;
    g.in = nullptr;
    g.in_row = nullptr;
    g.out = nullptr;
    g.out_row = nullptr;
    if (num_ctx == 0) {
        hipLaunchKernelGGL(k_grp_none, dim3(1), dim3(64), 0, s, num_rows, row_off_out, dropped_out);
        return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
    }
    // (without rows one count clears what the bounds would write)
    for (int k = 0; k < (num_rows > 0 ? passes : 1); ++k) {
        g.shift = kGrpDigitBits * k;
        g.out = bufs[k & 1];
        g.out_row = g.out + num_rows;
        hipLaunchKernelGGL(k_grp_count, dim3(p.blocks), dim3(kGrpThreads), 0, s, g);
        if (num_rows == 0) break;
        hipLaunchKernelGGL(k_enc_colscan, dim3((kGrpBins + 63) / 64), dim3(64 * kColWaves), 0, s, cs);
        hipLaunchKernelGGL(k_grp_scatter, dim3(p.blocks), dim3(kGrpThreads), 0, s, g);
        g.in = g.out;
        g.in_row = g.out_row;
    }
    if (num_rows > 0)
        hipLaunchKernelGGL(k_grp_bounds, dim3(static_cast<unsigned>((num_rows + 1023) / 1024)), dim3(256), 0, s, g);
    const unsigned kb = static_cast<unsigned>((num_ctx + 1023) / 1024);
    hipLaunchKernelGGL(k_grp_words, dim3(kb), dim3(1024), 0, s, g);
    if (kb > kGrpSumBlocks) hipLaunchKernelGGL(k_grp_scan, dim3(1), dim3(1024), 0, s, g);
    hipLaunchKernelGGL(k_grp_offsets, dim3(kb), dim3(1024), 0, s, g, kb > kGrpSumBlocks, dropped_out);
    if (num_rows > 0) {
        const dim3 grid(static_cast<unsigned>((num_rows + 255) / 256));
        if (row_stride_words <= 4)
            hipLaunchKernelGGL(k_grp_copy<4>, grid, dim3(256), 0, s, g);
        else
            hipLaunchKernelGGL(k_grp_copy<8>, grid, dim3(256), 0, s, g);
    }
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

int f2_pool_bases(const f2_model* members_model, const uint64_t* out_mask, const int64_t* pool_off,
                  const int32_t* members, int64_t num_members, const f2_model* pooled, uint32_t* pool_flags,
                  void* workspace, size_t workspace_bytes, void* stream) {
    if (!members_model || !pooled || members_model->num_ctx < 0 || pooled->num_ctx < 0 || num_members < 0)
        return F2_EINVAL;
    const int32_t P = pooled->num_ctx;
    if (P == 0) return F2_OK;
    if (!pool_off || !pool_flags || (num_members > 0 && !members) || !model_complete(pooled)) return F2_EINVAL;
    if (members_model->num_ctx > 0 && (!members_model->n_bits || !members_model->basis_off || !members_model->basis ||
                                       !members_model->rank || !members_model->ctx_flags || members_model->basis_words < 0))
        return F2_EINVAL;
    if (!workspace || workspace_bytes < f2_pool_workspace_bytes(members_model, P) ||
        (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return F2_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    PoolArgs A;
    A.num_ctx = members_model->num_ctx;
    A.n_bits = members_model->n_bits;
    A.basis_off = members_model->basis_off;
    A.basis = members_model->basis;
    A.rank = members_model->rank;
    A.ctx_flags = members_model->ctx_flags;
    A.out_mask = out_mask;
    A.num_pools = P;
    A.pool_off = pool_off;
    A.members = members;
    A.num_members = num_members;
    A.pooled_n = pooled->n_bits;
    A.pooled_flags = pooled->ctx_flags;
    A.pool_flags = pool_flags;
    A.row_off = reinterpret_cast<int64_t*>(ws);
    const size_t off_rows = align256(sizeof(int64_t) * (static_cast<size_t>(P) + 1));
    A.rows = reinterpret_cast<uint64_t*>(ws + off_rows);
    A.rows_cap = members_model->basis_words;
    const size_t off_blk = off_rows + align256(sizeof(uint64_t) * A.rows_cap);
    const unsigned pb = static_cast<unsigned>((P + 255) / 256);
    A.blk = reinterpret_cast<int64_t*>(ws + off_blk);
    int32_t* plan = reinterpret_cast<int32_t*>(ws + off_blk + align256(sizeof(int64_t) * (static_cast<size_t>(pb) + 1)));
    hipLaunchKernelGGL(k_pool_count, dim3(pb), dim3(256), 0, s, A);
    if (pb > kPoolSumBlocks) hipLaunchKernelGGL(k_pool_scan, dim3(1), dim3(1024), 0, s, A);
    hipLaunchKernelGGL(k_pool_offsets, dim3(pb), dim3(256), 0, s, A, pb > kPoolSumBlocks);
    hipLaunchKernelGGL(k_pool_copy, dim3(static_cast<unsigned>((P + 3) / 4)), dim3(256), 0, s, A);
    launch_fit(fit_args(A.rows, A.rows_cap, A.row_off, pooled, plan), s);
    hipLaunchKernelGGL(k_pool_finish, dim3(pb), dim3(256), 0, s, A);
    return hipGetLastError() == hipSuccess ? F2_OK : F2_EDEVICE;
}

}  // extern "C"
