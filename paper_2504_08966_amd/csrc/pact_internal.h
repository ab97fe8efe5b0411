// Internal declarations shared by the HIP sources of libpact (gfx950 only).
// Paper notation: n tokens, q kept tokens ("p-space" = position of a kept token in the
// ascending kept list), C centres, d_c cutoff, d_n density normaliser, alpha recovery factor.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include "pact.h"
#include "pact_measure.h"

namespace pact {

// ---------------------------------------------------------------------------------------
// Batch descriptor: passed BY VALUE as a kernel argument (no device copy to manage).
struct Seg {
    int32_t base;     // first row of this sample in every token-indexed tensor
    int32_t n;        // tokens in this sample
    float lambda, d_c, d_n, alpha;
    int32_t fallback_T;
    uint32_t flags;
};
struct Batch {
    int32_t B;        // samples in this launch (<= PACT_MAX_BATCH)
    int32_t n_max;    // max tokens of one sample; pitch of per-sample workspace arrays
    int32_t W;        // 64-bit words per bitmap row = ceil(n_max / 64)
    int32_t total;    // tokens over all samples
    Seg s[PACT_MAX_BATCH];
};

// ---------------------------------------------------------------------------------------
// Workspace layout.  Offsets in bytes from the 256-aligned workspace base.
constexpr int QG_CHUNKS = 8;          // row chunks of the global-query column sum, at most; but of queries of
constexpr int QG_NARROW = 1024;       // columns or fewer, in samples of more than 1024 QG_CHUNKS tokens,
constexpr int QG_LONG_CHUNKS = 16;    // at most
constexpr int SCORE_TOK = 64;         // tokens per workgroup in the logits kernel
constexpr int PRED_CAP = 64;          // 16-bit slots per kept token: slot 0 = count, then up to 63 preceding neighbours
constexpr int GRAM_MAX_WORKGROUPS = 256; // workgroups of 8 wavefronts per sample in a Gram pass (one per CU)
constexpr int NEAR_CAP = 1 << 16;     // near-threshold pairs kept for fp64 re-evaluation, per sample
// The list of a sample is in parts of equal size, each with a counter on a cache line of its own.  (One counter answers a hundred atomics a microsecond: an image's density
// pass, 700 wavefronts with undecided pairs, waited 4 us for it at its end.  Whole calls with one part / 4 / 8 / 16, us: images 1500 tokens 76.2 / 75.5 / 75.4 / 75.7, 2500 82.4 / 80.6 / 79.7 / 80.4, 4500 97.5 / 94.7 / 94.3 /
// 95.0, 7290 119.8 / 117.6 / 116.9 / 117.1; with few such pairs 128-wide images 3093 73.1 / 73.4 / 73.3 / 73.4, videos 3093 78.8 / 78.9 / 79.5 / 79.1, 6272 103.0 / 103.6 / 102.8 / 103.1.)  Samples of up to 1024 tokens, whose workgroups
// are few, have one, and those of batches, whose workgroups are fewer and at it at other times.  (One / sixteen: 2 x 2916 106.5 / 107.0, 2 x 7290 197.4 / 196.9, 3 x 4374 168.7 / 169.5, 7290 beside 729 134.7 / 132.0; 4 x 2916 148.4 / 149.1,
// 5 x 2916 159.9 / 161.0, 16 ragged images 356.5 / 358.9: finding a pair's part is 1.6 us of their settling.)
constexpr int NEAR_PARTS = 8, NEAR_COUNTER = 32;      // (words of a counter: places taken, ordered pairs they stand for, unused)
__host__ __device__ inline int near_parts(int n_max, int batch) { return n_max > 1024 && batch <= 3 ? NEAR_PARTS : 1; }
constexpr uint32_t NEAR_MARK = 0x80000000u;     // in the places taken of all parts of a list: some pair had no place in any
constexpr uint32_t NEAR_MIRROR = 0x80000000u;   // flag in a listed pair's row: the pair (col, row) is meant as well
constexpr float EXACT_SUMS_D_N = 0.21f;      // from this d_n on the density sums are exact in any order (see add_density)
constexpr uint32_t ST_UNKNOWN = 0, ST_CENTER = 1, ST_NOT = 2;
constexpr int RHO_RECHECK_MAX = PACT_MAX_RHO_RECHECK;   // tokens per sample whose density is evaluated again in fp64
constexpr int RHO_RECHECK_CHUNK = 64;                   // kept tokens per partial sum of such an evaluation (16 or 32 where few are listed)
// Clusters of at least MERGE_BIG rows are merged first (a cluster of 30 rows takes several times
// as long as one of 2, and started in the last turn it alone would be the end of the kernel).
// The first MERGE_SLOTS members of a cluster are noted as they join it (one 128-byte line per
// cluster), so that the merge of a full reduction needs no pass that builds member lists.
constexpr int MERGE_BIG = 12, MERGE_SLOTS = 32;
constexpr int32_t OVERFLOW_NEAR_LIST = 1, OVERFLOW_RHO_RECHECK = 2;   // bits of pact_report.refine_overflow

struct WsLayout {
    size_t qg_part, logits, hnorm, sm_part;            // score
    size_t nn, rinv;                                   // key norms, per token (global row index)
    size_t ident;                                      // identity index list (idx == NULL)
    size_t adj;                                        // [B][n_max][W] u64: rows < q adjacency; from row q on: candidate words [Wc][n_pruned]
    size_t cbest;                                      // [B][W][n_max] f32: largest cosine per (group of 64 centres, pruned token)
    size_t rho, status, cnum, cmask;                   // per sample, pitch n_max (cmask: W)
    size_t qg_long;                                    // [B][chunks][qcols] f64: more chunk sums than QG_CHUNKS (in the place of preds)
    size_t preds, heads;                               // [B][n_max][PRED_CAP] u16, [B][n_max] 4 x u16 (count + first 3; until those are
                                                       // built, the low parts of the densities: see add_density)
    size_t ksplit;                                     // [total]: fp32 clustering keys as int8 planes, [dk/64 rounded up][3][64] and [dk/64 rounded up][64]
    size_t near_list, near_cnt, stat;                  // refine list, counter; [B][workgroups * 8] most negative density exponent seen
    size_t tie_list, tie_cnt;                          // [B][RHO_RECHECK_MAX] kept positions whose density is re-evaluated; [B][4]: count, ticket
    size_t rho_fix;                                    // [B][min(RHO_RECHECK_MAX, n_max)][ceil(n_max / RHO_RECHECK_CHUNK)][2] f64 partial sums of those
    size_t offsets, members, big;                      // merge CSR (global row index); ids of the large clusters
    size_t slots;                                      // [total][MERGE_SLOTS] i32: first members of each cluster, in the order they joined (in the place of preds)
    size_t zeros;                                      // 256 zero bytes
    size_t total;
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
__host__ __device__ inline int64_t rho_fix_tokens(int64_t n_max) { return n_max < RHO_RECHECK_MAX ? n_max : RHO_RECHECK_MAX; }
__host__ __device__ inline int64_t rho_fix_chunks(int64_t n_max) { return (n_max + RHO_RECHECK_CHUNK - 1) / RHO_RECHECK_CHUNK; }

// Bytes of one token's clustering key as the Gram passes read it: bf16 as it is, fp32 as four int8 planes (padded with zeros to a
// multiple of 64 elements): the upper three interleaved, 192 bytes per 64 elements, then the lowest, 64 bytes per 64 elements.
inline size_t gram_token_bytes(int64_t dk, int k_dt) { return k_dt == PACT_F32 ? (size_t)((dk + 63) / 64) * 256 : (size_t)dk * 2; }

// dk: width of the clustering keys (0 for calls that run no Gram pass); k_dt: their type (only
// fp32 keys have a copy)
inline WsLayout make_layout(int64_t n_max, int64_t B, int64_t total, int64_t qcols, int64_t n_q, int64_t dk,
                            int k_dt) {
    WsLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const int64_t W = (n_max + 63) / 64;
    const int64_t smwg = (n_max + SCORE_TOK - 1) / SCORE_TOK;
    L.qg_part = take(sizeof(double) * B * QG_CHUNKS * qcols);
    L.logits = take(sizeof(double) * total * n_q);
    L.hnorm = take(sizeof(double) * total);
    L.sm_part = take(sizeof(double) * B * smwg * n_q * 2);
    L.nn = take(sizeof(double) * total);
    L.rinv = take(sizeof(float) * total);
    L.ident = take(sizeof(int32_t) * total);
    L.adj = take(sizeof(uint64_t) * B * n_max * W);
    L.cbest = take(sizeof(float) * B * W * n_max);
    L.rho = take(sizeof(double) * B * n_max);
    L.status = take(sizeof(uint32_t) * B * n_max);
    L.cnum = take(sizeof(int32_t) * B * n_max);
    L.cmask = take(sizeof(uint64_t) * B * W);
    L.preds = take(sizeof(uint16_t) * B * n_max * PRED_CAP);
    // (the sums are used up by the logits, before the lists are made)
    static_assert(sizeof(double) * QG_LONG_CHUNKS * QG_NARROW <= sizeof(uint16_t) * PRED_CAP * 1024 * QG_CHUNKS,
                  "the sums of a sample of that many tokens take no more room than its lists");
    L.qg_long = L.preds;
    L.heads = take(sizeof(uint16_t) * 4 * B * n_max);
    L.near_list = take(sizeof(uint32_t) * 2 * B * NEAR_CAP);
    L.near_cnt = take(sizeof(int32_t) * NEAR_COUNTER * NEAR_PARTS * B);
    L.stat = take(sizeof(uint32_t) * B * GRAM_MAX_WORKGROUPS * 8);   // Shape::STAT_WORDS of each workgroup of the density pass
    L.tie_list = take(sizeof(int32_t) * B * RHO_RECHECK_MAX);
    L.tie_cnt = take(sizeof(int32_t) * 4 * B);
    L.rho_fix = take(sizeof(double) * 2 * B * rho_fix_tokens(n_max) * rho_fix_chunks(n_max));
    L.offsets = take(sizeof(int32_t) * (total + B));
    L.members = take(sizeof(int32_t) * total);
    L.big = take(sizeof(int32_t) * total);
    // (the selection is over with the lists when the first member joins a cluster)
    static_assert(sizeof(int32_t) * MERGE_SLOTS == sizeof(uint16_t) * PRED_CAP, "a token's list and a cluster's slots take the same room");
    L.slots = L.preds;
    L.zeros = take(256);
    L.ksplit = take(k_dt == PACT_F32 ? total * gram_token_bytes(dk, k_dt) : 0);
    L.total = off;
    return L;
}

// Resolved device pointers for one call.
struct Ws {
    double* qg_part; double* qg_long; double* logits; double* hnorm; double* sm_part;
    double* nn; float* rinv; int32_t* ident;
    uint64_t* adj; float* cbest; double* rho; uint32_t* status;
    int32_t* cnum; uint64_t* cmask; uint16_t* preds; uint2* heads; double* rho_lo; uint32_t* near_list; int32_t* near_cnt; uint32_t* stat;
    int32_t* tie_list; int32_t* tie_cnt; double* rho_fix;
    int32_t* offsets; int32_t* members; int32_t* big; int32_t* slots; uint32_t* zeros; char* ksplit;
};

inline Ws resolve(void* base, const WsLayout& L) {
    char* p = (char*)base;
    Ws w;
    w.qg_part = (double*)(p + L.qg_part); w.qg_long = (double*)(p + L.qg_long);
    w.logits = (double*)(p + L.logits); w.hnorm = (double*)(p + L.hnorm);
    w.sm_part = (double*)(p + L.sm_part);
    w.nn = (double*)(p + L.nn); w.rinv = (float*)(p + L.rinv); w.ident = (int32_t*)(p + L.ident);
    w.adj = (uint64_t*)(p + L.adj); w.cbest = (float*)(p + L.cbest);
    w.rho = (double*)(p + L.rho);
    w.status = (uint32_t*)(p + L.status); w.cnum = (int32_t*)(p + L.cnum);
    w.preds = (uint16_t*)(p + L.preds); w.heads = (uint2*)(p + L.heads); w.rho_lo = (double*)(p + L.heads);
    w.cmask = (uint64_t*)(p + L.cmask); w.near_list = (uint32_t*)(p + L.near_list);
    w.near_cnt = (int32_t*)(p + L.near_cnt); w.stat = (uint32_t*)(p + L.stat);
    w.tie_list = (int32_t*)(p + L.tie_list); w.tie_cnt = (int32_t*)(p + L.tie_cnt);
    w.rho_fix = (double*)(p + L.rho_fix);
    w.offsets = (int32_t*)(p + L.offsets); w.big = (int32_t*)(p + L.big);
    w.members = (int32_t*)(p + L.members); w.slots = (int32_t*)(p + L.slots); w.zeros = (uint32_t*)(p + L.zeros);
    w.ksplit = p + L.ksplit;
    return w;
}

// ---------------------------------------------------------------------------------------
// Kernel launch bookkeeping (optional per-kernel events).
void prof_begin(const char* name, hipStream_t s);
void prof_end(hipStream_t s);

#define PACT_LAUNCH(name, kernel, grid, block, stream, ...)                        \
    do {                                                                           \
        ::pact::prof_begin(name, stream);                                          \
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);           \
        ::pact::prof_end(stream);                                                  \
        if (hipGetLastError() != hipSuccess) return PACT_ERR_HIP;                  \
    } while (0)

#define PACT_LAUNCH_SHMEM(name, kernel, grid, block, shmem, stream, ...)          \
    do {                                                                           \
        ::pact::prof_begin(name, stream);                                          \
        hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);       \
        ::pact::prof_end(stream);                                                  \
        if (hipGetLastError() != hipSuccess) return PACT_ERR_HIP;                  \
    } while (0)

// ---------------------------------------------------------------------------------------
// Stage launchers (host).  Each enqueues on `st` and returns a pact_status.
struct ScoreIn {
    const void* hidden; pact_dtype h_dt; int32_t h;
    const void* keys_pre; pact_dtype k_dt; int32_t n_kv, d_h;
    const void* q; pact_dtype q_dt; int32_t q_per_token; int32_t n_q;   // q_per_token: 1 = [total, ..], 0 = [B, ..]
};

struct KeysIn { const void* keys; pact_dtype k_dt; int32_t dk; };      // clustering keys
struct ReductionIn { KeysIn keys; pact_report* rep; int32_t *cluster_id, *cluster_counts; };

// First kernel of a clustering or recovery called alone: key norms, cleared bitmap rows, per-token initial state.  (In a reduction launch_score or
// launch_score_prune does it.)
int launch_front(const Batch& bt, const Ws& w, const KeysIn& keys, pact_report* rep, int32_t* cluster_id, int mode,
                 const int32_t* n_idx_dev, hipStream_t st);
int launch_score(const Batch& bt, const Ws& w, const ScoreIn& in, float* scores, const ReductionIn* red, hipStream_t st);
int launch_score_prune(const Batch& bt, const Ws* w, const ScoreIn* in, float* scores, const ReductionIn* red, int32_t* kept_idx, int32_t* pruned_idx,
                       pact_report* rep, hipStream_t st);
// want_stat: also record the largest key distance; *stat_words = words per sample the kernel
// wrote to w.stat (0 if not wanted), to be handed to launch_centres.
int launch_gram_density(const Batch& bt, const Ws& w, const void* keys, pact_dtype k_dt, int32_t dk,
                        const int32_t* idx, pact_report* rep, bool want_stat, int* stat_words, hipStream_t st);
// (diagnostic) the map of workgroup slots to samples that the Gram passes of a batch use
int plan_gram_workgroups(const int32_t* tiles, int32_t batch, uint16_t* wg_map, uint16_t* wg_count);
int launch_centres(const Batch& bt, const Ws& w, const void* keys, pact_dtype k_dt, int32_t dk,
                   const int32_t* idx, int32_t* center_idx, int32_t* cluster_id,
                   int32_t* cluster_counts, pact_report* rep, double* rho_opt, int32_t* rank_opt,
                   int stat_words, bool assign_now, hipStream_t st);
int launch_reincorporate(const Batch& bt, const Ws& w, const void* keys, pact_dtype k_dt, int32_t dk,
                         const int32_t* pruned_idx, const int32_t* center_idx, int32_t* cluster_id,
                         int32_t* cluster_counts, pact_report* rep, bool count_totals,
                         const int32_t* kept_idx, hipStream_t st);
int launch_merge(const Batch& bt, const Ws& w, const void* hidden, pact_dtype h_dt, int32_t h,
                 const int32_t* cluster_id, const int32_t* center_idx, pact_report* rep,
                 void* merged, pact_dtype out_dt, int32_t* cluster_counts, bool recount,
                 hipStream_t st);

int launch_handoff(const Batch& bt, const int32_t* center_idx, const int32_t* cluster_counts,
                   const pact_report* rep, const int32_t* positions, int32_t* positions_out,
                   float* log_weight, hipStream_t st);

// init modes
// m of Eq. 3 / 4: the threshold is the (m+1)-th smallest score, m = min(floor(lambda n), n-1);
// the m tokens below it are pruned, all of them when no other score equals the threshold.
__host__ __device__ inline int prune_rank(float lambda, int n) {
    int m = (int)floor((double)lambda * (double)n);
    if (m > n - 1) m = n - 1;
    return m < 0 ? 0 : m;
}
// Tokens of a sample, and of all samples, that a call will keep (the exact number of a sample is known on the device only: ties).
inline long kept_estimate(const Seg& sg) { return sg.n - prune_rank(sg.lambda, sg.n); }
inline long kept_estimate(const Batch& bt) {
    long n = 0;
    for (int b = 0; b < bt.B; ++b) n += kept_estimate(bt.s[b]);
    return n;
}

enum { INIT_REDUCE = 0, INIT_DBDPC_ALL = 1, INIT_DBDPC_SUBSET = 2, INIT_REINC = 3 };

// Worst-case error of a cosine from the matrix passes.  bf16 keys: rounding of the fp32 accumulation of
// dk products, plus slack for the scaling multiplies.  fp32 keys: bytes left out of the elements (at most
// sqrt(dk) 2^-23: all below 2^-24 of a row's largest), byte products left out (below dk 2^-23: order 3), the fp32
// combination of the rest.  Decisions closer than this to a threshold are re-made in fp64.
inline double cos_margin(int dk, int k_dt) {
    const double extra = k_dt == PACT_F32 ? sqrt((double)dk) : 0.0;
    return ((double)dk + extra + 16.0) * (1.0 / 8388608.0) + 2.5e-6;
}

// Internal element type of the Gram kernel for fp32 keys: each row as 32-bit integers in four int8 planes.
enum { PACT_I8X4 = 2 };

}  // namespace pact

// ---------------------------------------------------------------------------------------
// Device helpers
#ifdef __HIPCC__
namespace pact {

// LDS-qualified pointer types: accesses through them compile to ds_* instructions even when
// the pointer travels through function arguments (a generic pointer would give flat_*).
typedef __attribute__((address_space(3))) volatile unsigned char lds_vu8;
typedef __attribute__((address_space(3))) int lds_i32;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t hi16) { return __uint_as_float(hi16 << 16); }

// The cache lines of a kernel's arguments (a Batch, then `bytes` of others; up to the last of them, no kernel's segment need go on behind it), and that of sample b,
// are asked for together, ahead of everything else.  A scalar load comes where the compiler first needs it, behind the branches that decide on it, and each new line was a
// trip of its own to memory the first time: four to eight in turn ahead of a kernel's first vector load.  What is returned has to be waited for: in kernels whose counts and list heads, written
// by kernels before, come by scalar loads, by a statement that is not volatile, as an input beside the workgroup's number (behind a volatile one the compiler takes memory as written and uses vector
// loads: merge of 64 x 1458 tokens 896 wide 294.6 -> 298.6 us a call, searches of 64 x 196 97.4 -> 98.7); elsewhere by touch_args.
template <int BYTES> __device__ __forceinline__ uint32_t args_asked_for(int b) {
    const __attribute__((address_space(4))) char* args = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    asm("" : "+s"(args));
    auto word = [&](int at) __attribute__((always_inline)) { return *(const __attribute__((address_space(4))) uint32_t*)(args + at); };
    uint32_t t = word(0) ^ word(16 + (int)sizeof(Seg) * b);
#pragma unroll
    for (int at = 0; at < BYTES + 64; at += 64) t ^= word((int)sizeof(Batch) + (at < BYTES ? at : BYTES - 4));
    return t;
}
template <int BYTES> __device__ __forceinline__ void touch_args(int b) { asm volatile("" :: "s"(args_asked_for<BYTES>(b))); }
// Counts read back from a device-side report are clamped to the sample size, so that a report
// the caller never initialised cannot send a kernel out of bounds.
__device__ __forceinline__ int clamp_count(int v, int n) { return v < 0 ? 0 : (v > n ? n : v); }

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;   // NaN stays NaN
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// 16 bytes of a row -> up to 8 doubles.  EPL = elements per 16-byte load.
template <int DT> struct Elem;
template <> struct Elem<PACT_BF16> {
    static constexpr int EPL = 8;
    static constexpr int BYTES = 2;
    __device__ static __forceinline__ void widen(const uint4& v, double* out) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = (double)__uint_as_float(w[i] << 16);
            out[2 * i + 1] = (double)__uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    __device__ static __forceinline__ void widenf(const uint4& v, float* out) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
};
template <> struct Elem<PACT_F32> {
    static constexpr int EPL = 4;
    static constexpr int BYTES = 4;
    __device__ static __forceinline__ void widen(const uint4& v, double* out) {
        out[0] = (double)__uint_as_float(v.x); out[1] = (double)__uint_as_float(v.y);
        out[2] = (double)__uint_as_float(v.z); out[3] = (double)__uint_as_float(v.w);
    }
    __device__ static __forceinline__ void widenf(const uint4& v, float* out) {
        out[0] = __uint_as_float(v.x); out[1] = __uint_as_float(v.y);
        out[2] = __uint_as_float(v.z); out[3] = __uint_as_float(v.w);
    }
};

// Reductions over each group of `width` neighbouring lanes (a power of two), left in every lane
// of the group: lane l combines with lane l ^ 1, l ^ 2, ... in turn.  Inside a row of 16 lanes the
// partner's value comes through the data-parallel lane permutes of the vector unit (for a sum or
// a maximum a mirror image of the group of 8 or 16 serves as well as the exchange of its halves:
// the partner holds the same partial result, so the values are those of the exchange, bit for bit),
// beyond that through a shuffle; a shuffle of a double is two trips through the LDS crossbar, and
// 28 of them per wavefront were a quarter of the logits kernel with 28 query heads.
template <int CTRL> __device__ __forceinline__ float dpp_f32(float v) {
    const int u = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)u, (int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(u >> 32), (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// the value of the lane 4 apart, inside a row of 16: from above for the lanes with bit 2 clear (banks of four 0 and 2), from below for the others
__device__ __forceinline__ double dpp_xor4_f64(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    uint32_t r[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int x = (int)(uint32_t)(u >> (32 * w));
        const int t = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xF, 0x5, false);      // row_shl:4
        r[w] = (uint32_t)__builtin_amdgcn_update_dpp(t, x, 0x114, 0xF, 0xA, false);   // row_shr:4
    }
    return __builtin_bit_cast(double, ((uint64_t)r[1] << 32) | r[0]);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;   // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror
__device__ __forceinline__ double group_sum_f64(double v, int width) {
    if (width > 1) v += dpp_f64<DPP_XOR1>(v);
    if (width > 2) v += dpp_f64<DPP_XOR2>(v);
    if (width > 4) v += dpp_f64<DPP_HALF_MIRROR>(v);
    if (width > 8) v += dpp_f64<DPP_MIRROR>(v);
    for (int sft = 16; sft < width; sft <<= 1) v += __shfl_xor(v, sft, 64);
    return v;
}
template <int WIDTH> __device__ __forceinline__ double group_max_f64(double v) {
    static_assert(WIDTH == 8 || WIDTH == 16, "within a row of 16 lanes");
    v = fmax(v, dpp_f64<DPP_XOR1>(v));
    v = fmax(v, dpp_f64<DPP_XOR2>(v));
    v = fmax(v, dpp_f64<DPP_HALF_MIRROR>(v));
    if (WIDTH > 8) v = fmax(v, dpp_f64<DPP_MIRROR>(v));
    return v;
}
template <int WIDTH> __device__ __forceinline__ float group_sum_f32(float v) {
    static_assert(WIDTH == 8 || WIDTH == 16, "within a row of 16 lanes");
    v += dpp_f32<DPP_XOR1>(v);
    v += dpp_f32<DPP_XOR2>(v);
    v += dpp_f32<DPP_HALF_MIRROR>(v);
    if (WIDTH > 8) v += dpp_f32<DPP_MIRROR>(v);
    return v;
}
template <int WIDTH> __device__ __forceinline__ float group_max_f32(float v) {
    static_assert(WIDTH == 8 || WIDTH == 16, "within a row of 16 lanes");
    v = fmaxf(v, dpp_f32<DPP_XOR1>(v));
    v = fmaxf(v, dpp_f32<DPP_XOR2>(v));
    v = fmaxf(v, dpp_f32<DPP_HALF_MIRROR>(v));
    if (WIDTH > 8) v = fmaxf(v, dpp_f32<DPP_MIRROR>(v));
    return v;
}

// Inclusive prefix sum over the 64 lanes of a wavefront (all active), on the vector unit's lane
// permutes: shifts by 1, 2, 4 and 8 inside each row of 16, then lane 15 of rows 0 and 2 to rows 1
// and 3, then lane 31 to rows 2 and 3.  Six dependent vector instructions instead of six trips
// through the LDS crossbar.
__device__ __forceinline__ int wave_scan_incl_i32(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);     // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);     // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);     // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);     // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);     // row_bcast:15 -> rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);     // row_bcast:31 -> rows 2, 3
    return v;
}
// value of lane 0 / lane 63 of a wavefront-wide register, as a scalar
__device__ __forceinline__ int lane0_of(int v) { return __builtin_amdgcn_readlane(v, 0); }
__device__ __forceinline__ int lane63_of(int v) { return __builtin_amdgcn_readlane(v, 63); }

// Over the whole wavefront (all 64 lanes active): neighbours first, inside the rows of 16 lanes through
// the lane permutes, then the four rows through two shuffles - 4 trips through the LDS crossbar instead
// of 12, which is half a microsecond in a wavefront that waits for the result.
__device__ __forceinline__ double wave_sum_f64(double v) {
    return group_sum_f64(v, 64);   // butterfly: every lane ends with the bit-identical total
}
__device__ __forceinline__ double wave_max_f64(double v) {
    v = group_max_f64<16>(v);
    v = fmax(v, __shfl_xor(v, 16, 64));
    return fmax(v, __shfl_xor(v, 32, 64));
}

// fp64 dot product of two rows of dk elements, computed by one full wavefront; the partition
// of elements over lanes and the reduction tree are fixed, so dot(a,b) of bit-identical rows
// equals dot(a,a) bit for bit.
template <int DT>
__device__ __forceinline__ double wave_dot64(const char* ra, const char* rb, int dk, int lane) {
    constexpr int EPL = Elem<DT>::EPL;
    double acc = 0.0;
    for (int e = lane * EPL; e < dk; e += 64 * EPL) {
        const uint4 va = *(const uint4*)(ra + (size_t)e * Elem<DT>::BYTES);
        const uint4 vb = *(const uint4*)(rb + (size_t)e * Elem<DT>::BYTES);
        double a[8], b[8];
        Elem<DT>::widen(va, a);
        Elem<DT>::widen(vb, b);
#pragma unroll
        for (int i = 0; i < EPL; ++i) acc = fma(a[i], b[i], acc);
    }
    return wave_sum_f64(acc);
}

// 16 bytes that this launch touches once: loads and stores with the streaming hint.  Used when a
// call's hidden states are larger than what the 256 MB last-level cache can keep between the norm
// pass and the merge anyway; for smaller calls the hint costs those later hits (one 7290-token
// image: +4 us per call with it, 8 videos of 6272 tokens: -30 us; batches of 2 to 6 such videos,
// 43 MiB each: +8, +4, -6, -13, -20 us, hence the 150 MiB).
inline bool hidden_streams(long total_tokens, int h, int elem_bytes) {
    return (double)total_tokens * (double)h * (double)elem_bytes > 150.0 * 1024.0 * 1024.0;
}
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_once16(const void* p) {
    const u32x4_t v = __builtin_nontemporal_load((const u32x4_t*)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_once16(void* p, uint4 w) {
    const u32x4_t v = {w.x, w.y, w.z, w.w};
    __builtin_nontemporal_store(v, (u32x4_t*)p);
}

// Eq. 5 in fp64 from a dot product and the two squared norms; zero vector -> cosine 0.
__device__ __forceinline__ double cos_dist64(double dot, double nna, double nnb) {
    const double den = sqrt(nna * nnb);
    const double c = den > 0.0 ? dot / den : 0.0;
    return fmin(fmax(1.0 - c, 0.0), 2.0);
}

// Recovery (Eq. 8/9): the smallest fp32 cosine of a centre that may be within alpha d_c.
__device__ __forceinline__ float recovery_reach(const Seg& sg, float margin) { return (1.0f - sg.alpha * sg.d_c) - margin; }
// One pruned token and a group of 64 centres: `top`, the largest of the products that carry the centres' reciprocal norms only, becomes the group's
// largest cosine (never NaN); returned is the cut from which on such a product is a candidate: within reach, and at most 2 * margin below that
// cosine.  The column's factor rj is divided out of it, with more to spare than the roundings take: a bit more there is one more look in fp64.
__device__ __forceinline__ float candidate_cut(float& top, float rj, float margin, float reach) {
    top = fmaxf(top * rj, -INFINITY);
    const float cut = fmaxf(top - 2.0f * margin, reach), inv = __builtin_amdgcn_rcpf(rj), at = cut * inv;
    const float cutv = at - fmaxf(fabsf(at) * 0x1p-20f, inv * 1e-37f);
    return fabsf(cutv) < INFINITY ? cutv : -INFINITY;          // (a zero vector, or nearly infinite ones: all are candidates)
}

// What settling a sample's undecided pairs reports.  overflow: the list held not all of them, ordered: ordered pairs they stand for (a pair that stands for
// both orders counts twice).  far_bits: of the most negative exponent -(d / d_n) log2(e) that the density pass saw (negative floats order
// like their bits), 0 where it was not asked to look.
__device__ __forceinline__ void report_settled(pact_report* rep, bool overflow, int ordered, uint32_t far_bits, float d_n) {
    rep->dc_checked_pairs = overflow ? NEAR_CAP : ordered;
    rep->refine_overflow = overflow ? OVERFLOW_NEAR_LIST : 0;
    rep->max_key_distance = far_bits ? fminf(-__uint_as_float(far_bits) * d_n * 0.6931471805599453f, 2.0f) : 0.0f;
}
// ... and what a pair's fp64 distance decides: no neighbours beyond d_c; how many near-ties to count.
__device__ __forceinline__ bool beyond_cutoff(double d, double d_c) { return d > d_c; }
__device__ __forceinline__ int near_ties_of(double d, double d_c, bool both_orders) { return fabs(d - d_c) <= 1e-6 ? (both_orders ? 2 : 1) : 0; }

}  // namespace pact
#endif
