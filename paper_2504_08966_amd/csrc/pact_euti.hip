// EUTI (Alg. 1): global query (Eq. 1), importance score (Eq. 2), percentile split (Eq. 3/4),
// plus the per-token preparation of the clustering keys (norms, cleared bitmap rows).
// All arithmetic of the score is fp64 (the stage is bound by reading H from HBM, the ALU work
// is free), rounded once to fp32; the split then compares fp32 bit patterns exactly.
#include <type_traits>

#include "pact_internal.h"

namespace pact {

// ------------------------------------------------------------------------------------------
// What depends on the inputs alone:
//   query sums    : Eq. 1 pass 1, column sums of one row chunk of Q and 128 bytes of
//                   its columns (32 row lanes x 8 lanes of 16 bytes; eight rows in
//                   flight per lane).  Few chunks (query_chunks()): the logits kernel
//                   adds them up again in every workgroup;
//   clustering keys: squared norm (fp64), reciprocal norm (fp32), fp32 keys' int8
//                   planes, cleared bitmap row, per-token initial state (status,
//                   cluster id, counts); 16 to 64 lanes per token by the row's width;
//   |h_i|_2 in fp64: one wavefront per token or, for rows of at most 4 KB, several tokens per wavefront (eight loads in flight per lane).
// Keys and hidden states are walked by token of the whole batch (no blocks for the tokens that shorter samples do not have).
// The first launch of a reduction is the query sums (none if the query is given as its mean), the second the logits, both short of work: the hidden states' norms, most of a
// call's bytes, are in either or dealt to both (norms_first()), and the keys in one of these or beside the percentile split (keys_launch()).  A clustering alone has its keys in a launch of their own.
constexpr int FRONT_THREADS = 256;
struct KeyArgs {
    const char* keys; int32_t dk;
    double* nn; float* rinv; uint64_t* adj; double* rho; double* rho_lo;
    uint32_t* status; int32_t* ident; int32_t* near_cnt; int32_t* tie_cnt;
    pact_report* rep; int32_t* cluster_id; int32_t* cluster_counts;
    const int32_t* n_idx_dev; uint32_t* zeros;
    char* ksplit;                            // fp32 keys only: the int8 planes for the Gram passes
    int32_t mode, key_lanes, rows_each;      // lanes per row; rows per group of them
};
// Row chunks of a sample's query sum: of 128 rows, 8 at most, of wide queries, which have strips enough, 4 up to 4096 tokens (every workgroup of the logits
// kernel reads its columns of all chunks, 32 KB); 16 at most of long ones with narrow queries, whose few
// blocks would each be a chain of trips of 256 rows (16384 tokens, 512 fp32 columns: 8 chunks of 2048 rows were 128 blocks of 8 trips, 22 us for 34 MB).  Each sample its own number: with the longest
// one's for all, 32768 tokens beside 31 of 729, 14 query heads, both launches were a third longer.  And the number of a call of its own, so that its sums are the same there.  (28 query heads, whole calls with four chunks / eight, us: 4500 tokens
// 110.4 / 109.9, 7290 136.1 / 134.6, 10001 181.8 / 179.4, 32768 727 / 722, 4 x 5001 248.8 / 246.4, 3 x 7290 285.1 / 285.1; 2 x 4500 145.0 / 146.7, 8 x 6272 488.8 / 492.9, 7290 with fp32 keys 196.6 / 197.7.)
__host__ __device__ inline int query_chunks(int n, int qcols) {
    const bool wide = qcols > QG_NARROW;
    if (!wide && n > 1024 * QG_CHUNKS) return n > 1024 * QG_LONG_CHUNKS ? QG_LONG_CHUNKS : (n + 1023) / 1024;
    const int most = wide && n <= 4096 ? QG_CHUNKS / 2 : QG_CHUNKS, want = (n + 127) / 128;
    return want < most ? want : most;
}
// Where the chunks' sums are.
static double* query_sums(const Ws& w, int chunks) { return chunks > QG_CHUNKS ? w.qg_long : w.qg_part; }

// |h_g|_2 in fp64 of TPW consecutive tokens by one wavefront, 8 / TPW independent 16-byte loads in flight per
// lane and token.
template <int HDT, int TPW>
__device__ __forceinline__ void hnorm_rows(const char* __restrict__ hidden, int h, int g0, int total, int lane,
                                           double* __restrict__ hnorm, bool stream) {
    constexpr int HE = Elem<HDT>::EPL, U = 8 / TPW;
    double ss[TPW][4];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) ss[t][k] = 0.0;
    for (int e0 = lane * HE; e0 < h; e0 += U * 64 * HE) {
        uint4 v[TPW][U];
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const char* hp = hidden + (size_t)min(g0 + t, total - 1) * (size_t)h * Elem<HDT>::BYTES;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * 64 * HE;
                v[t][u] = (e >= h) ? make_uint4(0, 0, 0, 0)
                        : stream ? load_once16(hp + (size_t)e * Elem<HDT>::BYTES)
                                 : *(const uint4*)(hp + (size_t)e * Elem<HDT>::BYTES);
            }
        }
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                double x[8];
                Elem<HDT>::widen(v[t][u], x);
#pragma unroll
                for (int k = 0; k < HE; ++k) ss[t][u & 3] = fma(x[k], x[k], ss[t][u & 3]);
            }
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const double sst = wave_sum_f64((ss[t][0] + ss[t][1]) + (ss[t][2] + ss[t][3]));
        if (lane == 0 && g0 + t < total) hnorm[g0 + t] = sqrt(sst);
    }
}
// tokens per wavefront for a row of h elements
__host__ __device__ inline int hnorm_tokens(int h, int elem_bytes) {
    const int loads = (h * elem_bytes + 1023) / 1024;      // 16-byte loads per lane and row
    return loads <= 2 ? 4 : loads <= 4 ? 2 : 1;
}
struct NormArgs { const char* hidden; double* hnorm; int32_t h, h_bf16, stream, from, to; };      // tokens [from, to) of the batch
template <int HDT>
__device__ __forceinline__ void hnorm_job(const NormArgs& a, int wave_no, int lane) {
    const int tpw = hnorm_tokens(a.h, Elem<HDT>::BYTES), g0 = a.from + wave_no * tpw;
    if (g0 >= a.to) return;
    if (tpw == 4) hnorm_rows<HDT, 4>(a.hidden, a.h, g0, a.to, lane, a.hnorm, a.stream != 0);
    else if (tpw == 2) hnorm_rows<HDT, 2>(a.hidden, a.h, g0, a.to, lane, a.hnorm, a.stream != 0);
    else hnorm_rows<HDT, 1>(a.hidden, a.h, g0, a.to, lane, a.hnorm, a.stream != 0);
}
__device__ __forceinline__ void norm_block(const NormArgs& a, int wave_no, int lane) {
    if (a.h_bf16) hnorm_job<PACT_BF16>(a, wave_no, lane);
    else hnorm_job<PACT_F32>(a, wave_no, lane);
}

// Sample that token g of the batch belongs to (g the same for the wavefront: scalar loads, a vector load of an argument is a trip to memory).
__device__ __forceinline__ int sample_of(const Batch& bt, int g) {
    g = __builtin_amdgcn_readfirstlane(g);
    int b = 0;
    for (int step = PACT_MAX_BATCH / 2; step; step >>= 1)
        if (b + step < bt.B && bt.s[b + step].base <= g) b += step;
    return b;
}

// The bitmap is used over (kept tokens) x (kept tokens).  In a full reduction that is
// n - m rows and columns unless scores tie at the threshold (Eq. 3 / 4); the split
// clears the rest itself in that case.  Token i of sample b, by KL lanes.
template <int KL>
__device__ __forceinline__ void clear_bits(const Batch& bt, const KeyArgs& a, int b, const Seg& sg, int i, int kl) {
    uint64_t* arow = a.adj + ((size_t)b * bt.n_max + i) * bt.W;
    const int side = (a.mode == INIT_REDUCE) ? sg.n - prune_rank(sg.lambda, sg.n) : sg.n;
    const int Wn = (i < side) ? (side + 63) >> 6 : 0;
    for (int k = kl; k < Wn; k += KL) arow[k] = 0ull;
}
__device__ __forceinline__ void start_token(const Batch& bt, const KeyArgs& a, int b, const Seg& sg, int i, double v, float rinv) {
    const size_t g = (size_t)sg.base + i;
    a.nn[g] = v;
    a.rinv[g] = rinv;
    if (a.mode == INIT_REDUCE || a.mode == INIT_DBDPC_ALL || a.mode == INIT_DBDPC_SUBSET) {
        a.status[(size_t)b * bt.n_max + i] = ST_UNKNOWN;
        a.rho[(size_t)b * bt.n_max + i] = 0.0;
        if (sg.d_n < EXACT_SUMS_D_N) a.rho_lo[(size_t)b * bt.n_max + i] = 0.0;
        a.ident[g] = i;
        a.cluster_id[g] = -1;
        if (a.cluster_counts) a.cluster_counts[g] = 0;
    }
}

// A row of fp32 keys as 32-bit integers X = rint(x S) (S: its largest element becomes 2139062143 = 0x7F7F7F7F, or a power of
// four less for rows of more than 2^17 elements, whose order-0 sums would not fit an int32), split
// into four signed bytes: the upper three in turn, 64 elements of each, then all of the lowest; padded with zeros.
// The Gram passes' products are in units of 2^24, so that the reciprocal norm is 4096 / |X|.  It is rounded up to fp32 and S is
// taken from what that is the reciprocal of: it is then exact.  v: squared norm, top: largest element.
__device__ __forceinline__ double bytes_scale(double v, float top, int dk, float& rinv) {
    double most = 2139062143.0;
    for (int64_t d = dk; d > 131072; d >>= 2) most *= 0.5;
    double S = top > 0.0f ? most / (double)top : 0.0;
    if (v > 0.0) {
        const double len = sqrt(v);
        rinv = __double2float_ru(4096.0 / (S * len));
        if (v < INFINITY) S = 4096.0 / ((double)rinv * len);
    }
    return S;
}
// Four elements from element e on, to the planes at sp.  X + 0x80808080 has the signed bytes of X, each 128 more, as its
// unsigned ones (|X| <= 0x7F7F7F7F); then bytes of four words to four words of a byte each.
__device__ __forceinline__ void store_bytes(char* sp, int groups, int e, const float (&x)[8], double S) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = ((uint32_t)(int)rint((double)x[k] * S) + 0x80808080u) ^ 0x80808080u;
    const uint32_t a01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t a23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), b23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    char* at = sp + (size_t)(e >> 6) * 192 + (e & 63);
    *(uint32_t*)at = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
    *(uint32_t*)(at + 64) = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
    *(uint32_t*)(at + 128) = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
    *(uint32_t*)(sp + (size_t)groups * 192 + e) = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
}

// One clustering key by KL lanes (16, 32 or 64; a row of at most KL 16-byte chunks for KL < 64): the
// values are those of wave_dot64 whatever KL (the lanes it leaves out would add zeros).
template <int KDT, int KL>
__device__ __forceinline__ void key_job(const Batch& bt, const KeyArgs& a, int wave_no, int lane) {
    constexpr int EPL = Elem<KDT>::EPL;
    const int kl = lane & (KL - 1);
    const int g0 = wave_no * (64 / KL);
    if (g0 >= bt.total) return;
    const int b0 = sample_of(bt, g0);
    const int gi = g0 + lane / KL;
    if (gi >= bt.total) return;
    // (the tokens of a wavefront may straddle samples)
    int b = b0;
    if (KL < 64) while (b + 1 < bt.B && bt.s[b + 1].base <= gi) ++b;
    const Seg sg = bt.s[b];
    const size_t g = (size_t)gi;
    const int i = gi - sg.base;
    const char* row = a.keys + g * (size_t)a.dk * Elem<KDT>::BYTES;
    // (the first two chunks per lane stay in registers: fp32 rows of up to 2 KB are read once for all three of their uses)
    const uint4 none = make_uint4(0, 0, 0, 0);
    const uint4 c0 = kl * EPL < a.dk ? *(const uint4*)(row + (size_t)kl * 16) : none;
    const uint4 c1 = (kl + KL) * EPL < a.dk ? *(const uint4*)(row + (size_t)(kl + KL) * 16) : none;
    auto chunk = [&](int e) __attribute__((always_inline)) {                 // at element e, a multiple of EPL
        return e < KL * EPL ? c0 : e < 2 * KL * EPL ? c1 : e < a.dk ? *(const uint4*)(row + (size_t)e * Elem<KDT>::BYTES) : none;
    };
    double acc = 0.0;
    for (int e = kl * EPL; e < a.dk; e += KL * EPL) {
        double x[8];
        Elem<KDT>::widen(chunk(e), x);
#pragma unroll
        for (int k = 0; k < EPL; ++k) acc = fma(x[k], x[k], acc);
    }
    const double v = group_sum_f64(acc, KL);
    float rinv = v > 0.0 ? (float)(1.0 / sqrt(v)) : 0.0f;
    if constexpr (KDT == PACT_F32) {
        float top = 0.0f;
        for (int e = kl * 4; e < a.dk; e += 4 * KL) {
            float x[8];
            Elem<KDT>::widenf(chunk(e), x);
            top = fmaxf(fmaxf(top, fmaxf(fabsf(x[0]), fabsf(x[1]))), fmaxf(fabsf(x[2]), fabsf(x[3])));
        }
        top = group_max_f32<16>(top);
#pragma unroll
        for (int sft = 16; sft < KL; sft <<= 1) top = fmaxf(top, __shfl_xor(top, sft, 64));
        const double S = bytes_scale(v, top, a.dk, rinv);
        const int groups = (a.dk + 63) / 64;
        char* sp = a.ksplit + g * (size_t)groups * 256;
        for (int e = kl * 4; e < groups * 64; e += 4 * KL) {
            float x[8];
            Elem<KDT>::widenf(chunk(e), x);                            // (zeros past the row's end)
            store_bytes(sp, groups, e, x, S);
        }
    }
    clear_bits<KL>(bt, a, b, sg, i, kl);
    if (kl == 0) start_token(bt, a, b, sg, i, v, rinv);
}

// Values of T rows per lane (v[t]: row t), each combined over KL lanes as group_sum_f64 does it (neighbours, then pairs 2, 4, 8, 16 and 32
// apart; the same pairs, so the same bits): a lane gives up half of its rows at each step until it is left with row
// lane % T.  T = 4: half the instructions of four sums.
template <int T, int KL, class V, class F, class X> __device__ __forceinline__ V over_lanes(V (&v)[T], int lane, F&& join, X&& from) {
    static_assert(T == 2 || T == 4 || T == 8 || T == 16, "a row per lane in the end, inside a row of 16 lanes");
#pragma unroll
    for (int s = 0, left = T; (1 << s) < KL; ++s) {
        if (left > 1) {
            const bool low = ((lane >> s) & 1) == 0;
            left >>= 1;
#pragma unroll
            for (int k = 0; k < left; ++k) {
                const V own = low ? v[2 * k] : v[2 * k + 1], give = low ? v[2 * k + 1] : v[2 * k];
                v[k] = join(own, from(give, s));
            }
        } else v[0] = join(v[0], from(v[0], s));
    }
    return v[0];
}
__device__ __forceinline__ double apart_f64(double d, int s) {
    return s == 0 ? dpp_f64<DPP_XOR1>(d) : s == 1 ? dpp_f64<DPP_XOR2>(d) : s == 2 ? dpp_xor4_f64(d) : s == 3 ? dpp_f64<0x128>(d) : __shfl_xor(d, 1 << s, 64);      // (row_ror:8)
}

// T rows per group of KL lanes, U 16-byte chunks a lane, which are requested together; what is one value per row -
// the square root, the reciprocals, the stores - is done for all of them at once, a row per lane.  (Row by row that is 150
// instructions of a whole wavefront for each token, as much as the hidden states' part was: 8 x 6272 tokens 512 wide, keys and hidden states
// 77.5 -> 65 us, one image 13.8 -> 11.7.)
template <int KDT, int KL, int T, int U>
__device__ __forceinline__ void many_keys_job(const Batch& bt, const KeyArgs& a, int wave_no, int lane) {
    constexpr int EPL = Elem<KDT>::EPL, ROWS = 64 / KL;
    const int kl = lane & (KL - 1);
    const int g0 = wave_no * (ROWS * T);
    if (g0 >= bt.total) return;
    const int grp = KL < 64 ? lane / KL : 0;                         // this group's rows: g0 + grp + ROWS t
    const uint4 none = make_uint4(0, 0, 0, 0);
    const size_t row_bytes = (size_t)a.dk * Elem<KDT>::BYTES;
    uint4 c[T][U];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const char* row = a.keys + (size_t)min(g0 + grp + ROWS * t, bt.total - 1) * row_bytes;
#pragma unroll
        for (int u = 0; u < U; ++u) c[t][u] = (u * KL + kl) * EPL < a.dk ? *(const uint4*)(row + (size_t)(u * KL + kl) * 16) : none;
    }
    const int b0 = sample_of(bt, g0);
    double acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        acc[t] = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double x[8];
            Elem<KDT>::widen(c[t][u], x);
#pragma unroll
            for (int k = 0; k < EPL; ++k) acc[t] = fma(x[k], x[k], acc[t]);
        }
    }
    const double v = over_lanes<T, KL>(acc, lane, [](double x, double y) { return x + y; }, apart_f64);    // from here on a lane has row lane % T of its group's
    float rinv = v > 0.0 ? (float)(1.0 / sqrt(v)) : 0.0f;
    if constexpr (KDT == PACT_F32) {
        float tops[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            tops[t] = 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float x[8];
                Elem<KDT>::widenf(c[t][u], x);
                tops[t] = fmaxf(fmaxf(tops[t], fmaxf(fabsf(x[0]), fabsf(x[1]))), fmaxf(fabsf(x[2]), fabsf(x[3])));
            }
        }
        const float top = over_lanes<T, KL>(tops, lane, [](float x, float y) { return fmaxf(x, y); },
                                            [](float d, int s) { return __shfl_xor(d, 1 << s, 64); });
        const double S = bytes_scale(v, top, a.dk, rinv);
        const int groups = (a.dk + 63) / 64;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int g = g0 + grp + ROWS * t;
            const double St = __shfl(S, (lane & ~(KL - 1)) | t, 64);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = (u * KL + kl) * 4;
                float x[8];
                Elem<KDT>::widenf(c[t][u], x);
                if (g < bt.total && e < groups * 64) store_bytes(a.ksplit + (size_t)g * groups * 256, groups, e, x, St);
            }
        }
    }
    const int mine = g0 + grp + ROWS * (lane & (T - 1));
    const int end = b0 + 1 < bt.B ? bt.s[b0 + 1].base : bt.total;
    if (g0 + ROWS * T <= end) {                                      // all of one sample (uniform)
        const Seg sg = bt.s[b0];
#pragma unroll 4
        for (int t = 0; t < T; ++t) clear_bits<KL>(bt, a, b0, sg, g0 + grp + ROWS * t - sg.base, kl);
        if (kl < T) start_token(bt, a, b0, sg, mine - sg.base, v, rinv);
        return;
    }
    auto sample_from = [&](int g) __attribute__((always_inline)) {
        int b = b0;
        while (b + 1 < bt.B && bt.s[b + 1].base <= g) ++b;
        return b;
    };
#pragma unroll 1
    for (int t = 0; t < T; ++t) {
        const int g = g0 + grp + ROWS * t;
        if (g < bt.total) {
            const int b = sample_from(g);
            clear_bits<KL>(bt, a, b, bt.s[b], g - bt.s[b].base, kl);
        }
    }
    if (kl < T && mine < bt.total) {
        const int b = sample_from(mine);
        start_token(bt, a, b, bt.s[b], mine - bt.s[b].base, v, rinv);
    }
}

// Block `blk` of those of the clustering keys (WAVES wavefronts each), of which the first also clears counters and starts the reports.
template <int KDT, int WAVES>
__device__ __forceinline__ void key_block(const Batch& bt, const KeyArgs& a, int blk, int wave, int lane) {
    if (blk == 0) {
        if (threadIdx.x < 64) a.zeros[threadIdx.x] = 0u;
        for (int k = (int)threadIdx.x; k < bt.B * NEAR_PARTS; k += 64 * WAVES) *(int2*)(a.near_cnt + k * NEAR_COUNTER) = make_int2(0, 0);
        const int b = (int)threadIdx.x;
        if (b < bt.B) {
#pragma unroll
            for (int k = 0; k < 4; ++k) a.tie_cnt[4 * b + k] = 0;
            pact_report* rp = a.rep + b;
            const int mode = a.mode, n = bt.s[b].n;
            if (mode == INIT_REDUCE || mode == INIT_DBDPC_ALL || mode == INIT_DBDPC_SUBSET) {
                if (mode != INIT_REDUCE) {
                    const int k = (mode == INIT_DBDPC_ALL) ? n : min(max(*a.n_idx_dev, 0), n);
                    rp->n_kept = k;
                    rp->n_pruned = (mode == INIT_DBDPC_ALL) ? 0 : n - k;
                }
                rp->n_centers = 0; rp->rounds = 0; rp->dc_checked_pairs = 0; rp->dc_near_ties = 0;
                rp->refine_overflow = 0; rp->n_reincorporated = 0; rp->n_dropped = 0;
                rp->zero_norm_seen = 0;     // counted by the assignment kernels, which run later
                rp->max_key_distance = 0.0f;
                rp->rho_rechecked = 0; rp->rho_near_ties = 0;
                // (the split's two counters: a clustering call on a subset adds to them, in a reduction the split writes them, in this launch)
                if (mode == INIT_DBDPC_ALL) { rp->score_near_ties = 0; rp->nonfinite_seen = 0; }
                rp->reserved[0] = 0;
            }
            if (mode == INIT_REINC) { rp->n_reincorporated = 0; rp->n_dropped = 0; }
        }
    }
    const int wave_no = blk * WAVES + wave;
    if (a.rows_each > 1) {
        constexpr int T = KDT == PACT_BF16 ? 4 : 2;
        if (a.key_lanes == 16) many_keys_job<KDT, 16, T, 1>(bt, a, wave_no, lane);
        else if (a.key_lanes == 32) many_keys_job<KDT, 32, T, 1>(bt, a, wave_no, lane);
        else if (KDT == PACT_BF16 && a.rows_each == 8) many_keys_job<PACT_BF16, 64, 8, 1>(bt, a, wave_no, lane);
        else many_keys_job<KDT, 64, T, 2>(bt, a, wave_no, lane);
    }
    else if (a.key_lanes == 16) key_job<KDT, 16>(bt, a, wave_no, lane);
    else if (a.key_lanes == 32) key_job<KDT, 32>(bt, a, wave_no, lane);
    else key_job<KDT, 64>(bt, a, wave_no, lane);
}

// The keys of a clustering or recovery that is called alone.  grid (blocks), block 256.
template <int KDT>
__global__ __launch_bounds__(256) void front_kernel(Batch bt, KeyArgs a) {
    key_block<KDT, 4>(bt, a, blockIdx.x, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
}

// The query sums: first launch of a reduction with per-token queries; and, behind their blocks, keys and hidden states' norms.
// grid (strips of columns x chunks x B + keys' + norms'), block FRONT_THREADS.
struct QueryArgs { const char* q; double* qg_part; int32_t qcols, q_chunks, blocks, key_blocks; NormArgs norm; KeyArgs key; };
template <int KDT, int QDT>
__global__ __launch_bounds__(FRONT_THREADS) void query_sums_kernel(Batch bt, QueryArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int blk = blockIdx.x;
    if (blk >= a.blocks) {
        const int at = blk - a.blocks;
        if (at < a.key_blocks) return key_block<KDT, FRONT_THREADS / 64>(bt, a.key, at, wave, lane);
        return norm_block(a.norm, (at - a.key_blocks) * (FRONT_THREADS / 64) + wave, lane);
    }
    constexpr int EPL = Elem<QDT>::EPL, CW = 8 * EPL, RL = FRONT_THREADS / 8, U = 8;      // columns of a block, rows in a step, steps in flight
    __shared__ double s_part[FRONT_THREADS / 64][CW];
    const int ngroups = (a.qcols + CW - 1) / CW;
    const int cgroup = blk % ngroups, bc = blk / ngroups;
    // (q_chunks: those of the longest sample.  A single one has them; its blocks are the launch's longest chains, and this is ahead of their first loads)
    int b = 0, chunk = bc, own = a.q_chunks;
    if (bt.B > 1) {
        b = bc / a.q_chunks;
        chunk = bc - b * a.q_chunks;
        own = query_chunks(bt.s[b].n, a.qcols);
        if (chunk >= own) return;
    }
    const Seg sg = bt.s[b];
    const int rows_per = (sg.n + own - 1) / own;
    const int r0 = chunk * rows_per, r1 = min(sg.n, r0 + rows_per);
    const int rl = threadIdx.x >> 3, cl = threadIdx.x & 7;
    const int c = cgroup * CW + cl * EPL;
    const bool act = c < a.qcols;
    const size_t row_bytes = (size_t)a.qcols * Elem<QDT>::BYTES;
    const char* base = a.q + (size_t)sg.base * row_bytes + (size_t)(act ? c : 0) * Elem<QDT>::BYTES;
    double acc[EPL];
#pragma unroll
    for (int k = 0; k < EPL; ++k) acc[k] = 0.0;
    for (int rb = r0; rb < r1; rb += RL * U) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (rb + RL * u >= r1) break;                        // (uniform)
            v[u] = rb + RL * u + rl < r1 ? *(const uint4*)(base + (size_t)(rb + RL * u + rl) * row_bytes) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (rb + RL * u >= r1) break;
            double x[8];
            Elem<QDT>::widen(v[u], x);
#pragma unroll
            for (int k = 0; k < EPL; ++k) acc[k] += x[k];
        }
    }
    // over the wavefront's eight row lanes (lane bits 3 to 5): a lane gives up half of its columns at each step, as long as it has two
    int own_c = 0;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int left = EPL >> s;
        const bool up = ((lane >> (3 + s)) & 1) != 0;
        if (left >= 2) {
#pragma unroll
            for (int k = 0; k < left / 2; ++k) {
                const double keep = up ? acc[k + left / 2] : acc[k], give = up ? acc[k] : acc[k + left / 2];
                acc[k] = keep + __shfl_xor(give, 8 << s, 64);
            }
            own_c += up ? left / 2 : 0;
        } else acc[0] += __shfl_xor(acc[0], 8 << s, 64);
    }
    s_part[wave][cl * EPL + own_c] = acc[0];
    __syncthreads();
    const int oc = cgroup * CW + (int)threadIdx.x;
    if ((int)threadIdx.x < CW && oc < a.qcols) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < FRONT_THREADS / 64; ++k) t += s_part[k][threadIdx.x];
        a.qg_part[((size_t)b * a.q_chunks + chunk) * a.qcols + oc] = t;
    }
}

// ------------------------------------------------------------------------------------------
// Eq. 1, pass 2 and Eq. 2, pass 1.  A workgroup takes SCORE_TOK tokens and one key head (BY_MFMA) or a group of
// them: it adds up the chunk sums of its columns of the global query (or widens the one the caller
// passed) into LDS, computes the logits k_i^(g(j)) . Qg^(j) and leaves, per query head, the largest logit of
// its tokens, the sum of exp(logit - largest), and every token's exp(logit - largest).
// BY_MFMA (three to 16 query heads per key head, heads of whole 64-byte quarters): 16 tokens x 16 query heads per
// wavefront on v_mfma_f64_16x16x4_f64; lane l supplies token (query head) l % 16, elements of quarter l / 16
// of the head.  The vector units spent four instructions on conversion, LDS and lane sums for every
// multiplication (28 query heads over 4: 17.7 -> 13.2 us); with one query head per key head they are the faster way
// (8 videos 27.6 against 23.6 us).
// BY_LANES (one query head per key head, a power-of-two number of 16-byte chunks per head, at most 64): the
// lanes that hold a token's keys of the group multiply by elements of the global query in their registers; 64 / LT tokens at a time.
// BY_HEAD: any shape; a token per wavefront, one head after the other (and if a key head's columns do not fit
// the LDS, the chunk sums are added up where they are used: columns that many come in few chunks; a loop over more of them there cost
// all of BY_HEAD 97 spilled scalar registers, 729 tokens, four heads of 72 with 28 query heads, 271 -> 289 us).
// A launch of its own that added the chunk sums up cost 2.3 us and hid the norms' stream from the keys'.
// Behind the workgroups of the logits, which are bound by latency, those of hidden states' norms, bound by HBM, and of the clustering keys.
// grid (ceil(n_max / SCORE_TOK) x groups x B + norms' + keys'), block 256.
constexpr int LOGITS_COLS_ANY = 15360;   // columns of the global query that fit the LDS
static_assert(LOGITS_COLS_ANY >= QG_NARROW, "columns that do not fit the LDS come in QG_CHUNKS chunks at most");
constexpr int LOGITS_HEADS = 16;         // query heads of a workgroup, but for BY_HEAD
enum { BY_HEAD = 0, BY_LANES = 1, BY_MFMA = 2 };
struct LogitsArgs {
    const char* keys; int32_t n_kv, d_h, n_q;
    const double* qg_part; const char* q_given; int32_t q_bf16, q_chunks;     // q_given: the caller's global query
    double* expl; double* sm_part;
    int32_t kv_heads, qg_lds;            // key heads per group; whether their columns are in LDS
    int32_t blocks, logits_blocks;       // workgroups of a sample; of all samples
};
struct LogitsMoreArgs {
    NormArgs norm;
    KeyArgs key; int32_t key_blocks;
    uint32_t key_share;                  // key blocks among those behind the logits', in units of 2^-32, rounded up; 0: all of them first
};
// Key heads per workgroup of BY_HEAD.
static int logits_kv_heads_any(int n_kv, int n_q, int d_h) {
    for (int k = n_kv; k > 1; --k)
        if (n_kv % k == 0 && k * (n_q / n_kv) * d_h <= LOGITS_COLS_ANY) return k;
    return 1;
}
static int logits_way(int n_kv, int n_q, int d_h, int elem_bytes) {
    const int lph = d_h * elem_bytes / 16, rep = n_q / n_kv;
    if (rep == 1 && lph * 16 == d_h * elem_bytes && lph >= 1 && lph <= 64 && (lph & (lph - 1)) == 0) return BY_LANES;
    if (d_h * elem_bytes % 64 == 0 && rep <= LOGITS_HEADS && rep * (d_h + 8) <= LOGITS_COLS_ANY) return BY_MFMA;
    return BY_HEAD;
}

// Key heads per workgroup of BY_LANES: as many as the lanes hold, but 512 workgroups where the call has them (one image:
// 11.7 us with four heads a workgroup).
static int logits_kv_heads_lanes(const Batch& bt, int n_kv, int lph) {
    const long blocks = (bt.total + SCORE_TOK - 1) / SCORE_TOK;
    int best = 1;
    for (int k = 2; k <= n_kv && k <= LOGITS_HEADS && k * lph <= 64; ++k)
        if (n_kv % k == 0 && blocks * (n_kv / k) >= 512) best = k;
    return best;
}

template <int KDT, int WAY>
__device__ __forceinline__ void logits_block(const Batch& bt, const LogitsArgs& a) {
    constexpr int EPL = Elem<KDT>::EPL;
    constexpr int HEADS = WAY == BY_HEAD ? PACT_MAX_QHEADS : LOGITS_HEADS;
    extern __shared__ double s_qg[];     // BY_MFMA: [rep][4 quarters, padded]; otherwise [columns]
    __shared__ double s_l[HEADS][SCORE_TOK + 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int b = 0, blk = blockIdx.x;
    if (bt.B > 1) {
        b = (uint32_t)blk / (uint32_t)a.blocks;
        blk -= b * a.blocks;
    }
    const Seg sg = bt.s[b];
    const int n_groups = a.n_kv / a.kv_heads;
    const int tb = (uint32_t)blk / (uint32_t)n_groups, kv0 = (blk - tb * n_groups) * a.kv_heads;
    const int t0 = tb * SCORE_TOK;
    if (t0 >= sg.n) return;
    const int rep = a.n_q / a.n_kv, qcols = a.n_q * a.d_h;
    const int j0 = kv0 * rep, heads = a.kv_heads * rep, cols = heads * a.d_h;     // this workgroup's query heads and columns
    const size_t krow = (size_t)a.n_kv * a.d_h * Elem<KDT>::BYTES;
    // this lane's first keys are requested ahead of the global query.  BY_MFMA: its quarter of its token's row (8 chunks of it);
    // BY_LANES: its chunk of the rows of 8 tokens
    const int l16 = lane & 15, quarter = lane >> 4;
    const int qlen = a.d_h >> 2, qchunks = qlen / EPL;
    const int LT = WAY == BY_LANES ? a.kv_heads * (a.d_h / EPL) : 64, tpp = 64 / LT, tin = lane / LT, lt = lane - tin * LT;
    const char* kq = a.keys + ((size_t)sg.base + min(t0 + wave * 16 + l16, sg.n - 1)) * krow +
                     (size_t)(kv0 * a.d_h + quarter * qlen) * Elem<KDT>::BYTES;
    uint4 kv[8];
    auto fetch = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if constexpr (WAY == BY_MFMA) kv[u] = i0 + u < qchunks ? *(const uint4*)(kq + (i0 + u) * 16) : make_uint4(0, 0, 0, 0);
            if constexpr (WAY == BY_LANES) {
                const int t = t0 + wave * 16 + (i0 + u) * tpp + tin;
                kv[u] = tin < tpp && (i0 + u) * tpp < 16 && t < sg.n
                    ? *(const uint4*)(a.keys + ((size_t)sg.base + t) * krow + (size_t)(kv0 * a.d_h + lt * EPL) * Elem<KDT>::BYTES)
                    : make_uint4(0, 0, 0, 0);
            }
        }
    };
    fetch(0);
    // column j0 d_h + c of the global query; `further`: there may be more than QG_CHUNKS chunks
    auto query = [&](int c, auto further) __attribute__((always_inline)) {
        if (a.q_given) {
            const size_t at = (size_t)b * qcols + j0 * a.d_h + c;
            return a.q_bf16 ? (double)__uint_as_float((uint32_t)((const uint16_t*)a.q_given)[at] << 16) : (double)((const float*)a.q_given)[at];
        }
        const double* in = a.qg_part + (size_t)b * a.q_chunks * qcols + j0 * a.d_h + c;
        const int own = query_chunks(sg.n, qcols);
        double v = 0.0;
        auto add = [&](int k0) __attribute__((always_inline)) {
            double p[QG_CHUNKS];
#pragma unroll
            for (int k = 0; k < QG_CHUNKS; ++k) p[k] = k0 + k < own ? in[(size_t)(k0 + k) * qcols] : 0.0;
#pragma unroll
            for (int k = 0; k < QG_CHUNKS; ++k) v += p[k];
        };
        if constexpr (decltype(further)::value) {
#pragma unroll 1
            for (int k0 = 0; k0 < own; k0 += QG_CHUNKS) add(k0);
        } else add(0);
        return v / (double)sg.n;
    };
    // (a head's quarters one word apart from whole multiples of the LDS banks, the heads another: 64 different banks)
    const int qpitch = qlen + 1, hpitch = 4 * qpitch + 1;
    if (WAY != BY_HEAD || a.qg_lds) {
#pragma unroll 2
        for (int c = threadIdx.x; c < cols; c += 256) {
            const double v = query(c, std::true_type{});
            if constexpr (WAY == BY_MFMA) {
                const int r = c / a.d_h, e = c - r * a.d_h, qt = e / qlen;
                s_qg[r * hpitch + qt * qpitch + (e - qt * qlen)] = v;
            } else s_qg[c] = v;
        }
    }
    __syncthreads();
    if constexpr (WAY == BY_LANES) {
        const int lph = a.d_h / EPL;
        double qv[EPL];
#pragma unroll
        for (int k = 0; k < EPL; ++k) qv[k] = s_qg[lt * EPL + k];
#pragma unroll 1
        for (int i0 = 0; i0 * tpp < 16; i0 += 8) {
            if (i0 > 0) fetch(i0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if ((i0 + u) * tpp >= 16) break;                         // (uniform)
                double x[8], acc = 0.0;
                Elem<KDT>::widen(kv[u], x);
#pragma unroll
                for (int k = 0; k < EPL; ++k) acc = fma(x[k], qv[k], acc);
                acc = group_sum_f64(acc, lph);
                const int tl = (i0 + u) * tpp + tin;
                if (tin < tpp && tl < 16 && (lt & (lph - 1)) == 0) s_l[lt / lph][wave * 16 + tl] = acc;
            }
        }
    } else if constexpr (WAY == BY_MFMA) {
        typedef double f64x4_t __attribute__((ext_vector_type(4)));
        f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
        const double* qv = s_qg + min(l16, rep - 1) * hpitch + quarter * qpitch;
        for (int c0 = 0; c0 < qchunks; c0 += 8) {
            if (c0 > 0) fetch(c0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (c0 + u >= qchunks) break;                            // (uniform)
                double x[8];
                Elem<KDT>::widen(kv[u], x);
#pragma unroll
                for (int k = 0; k < EPL; ++k)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], qv[(c0 + u) * EPL + k], acc, 0, 0, 0);
            }
        }
        // this lane's results: tokens 4 v + lane / 16 of the wavefront's sixteen, query head lane % 16
        if (l16 < rep) {
#pragma unroll
            for (int v = 0; v < 4; ++v) s_l[l16][wave * 16 + 4 * v + quarter] = acc[v];
        }
    } else {
        for (int tl = wave; tl < SCORE_TOK && t0 + tl < sg.n; tl += 4) {
            const char* kp = a.keys + ((size_t)sg.base + t0 + tl) * krow;
            for (int jl = 0; jl < heads; ++jl) {
                const int kvh = (j0 + jl) / rep;
                double acc = 0.0;
                for (int e = lane * EPL; e < a.d_h; e += 64 * EPL) {
                    double x[8];
                    Elem<KDT>::widen(*(const uint4*)(kp + (size_t)(kvh * a.d_h + e) * Elem<KDT>::BYTES), x);
#pragma unroll
                    for (int k = 0; k < EPL; ++k) {
                        const int c = jl * a.d_h + e + k;
                        acc = fma(x[k], a.qg_lds ? s_qg[c] : query(c, std::false_type{}), acc);
                    }
                }
                acc = wave_sum_f64(acc);
                if (lane == 0) s_l[jl][tl] = acc;
            }
        }
    }
    __syncthreads();
    static_assert(SCORE_TOK == 64, "a lane per token, 16 tokens per wavefront");
    const bool have = t0 + lane < sg.n;
    const size_t part0 = ((size_t)b * ((bt.n_max + SCORE_TOK - 1) / SCORE_TOK) + tb) * a.n_q + j0;
    for (int jl = wave; jl < heads; jl += 4) {
        const double l = have ? s_l[jl][lane] : -INFINITY;
        const double m = wave_max_f64(l);
        const double e = have ? exp(l - m) : 0.0;
        const double z = wave_sum_f64(e);
        // (transposed through the same LDS words, so that a token's heads are stored together)
        s_l[jl][lane] = e;
        if (lane == 0) *(double2*)(a.sm_part + (part0 + jl) * 2) = make_double2(m, z);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < heads * SCORE_TOK; k += 256) {
        const int tl = k / heads, jl = k - tl * heads;
        if (t0 + tl < sg.n) a.expl[((size_t)sg.base + t0 + tl) * a.n_q + j0 + jl] = s_l[jl][tl];
    }
}

template <int KDT, int WAY>
__global__ __launch_bounds__(256) void score_logits_kernel(Batch bt, LogitsArgs a) {
    touch_args<sizeof(LogitsArgs)>(0);
    logits_block<KDT, WAY>(bt, a);
}
// With keys or hidden states behind them.
template <int KDT, int WAY>
__global__ __launch_bounds__(256) void score_logits_more_kernel(Batch bt, LogitsArgs a, LogitsMoreArgs m) {
    if ((int)blockIdx.x < a.logits_blocks) return logits_block<KDT, WAY>(bt, a);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // key blocks: ahead of those of the hidden states, or evenly among them (see launch_logits)
    const uint32_t at = blockIdx.x - (uint32_t)a.logits_blocks;
    uint32_t key_no = min(at, (uint32_t)m.key_blocks);
    bool keys_here = at < (uint32_t)m.key_blocks;
    if (m.key_share) {
        key_no = __umulhi(at, m.key_share);
        keys_here = __umulhi(at + 1, m.key_share) != key_no;
    }
    if (keys_here) key_block<KDT, 4>(bt, m.key, (int)key_no, wave, lane);
    else norm_block(m.norm, (int)(at - key_no) * 4 + wave, lane);
}

// ------------------------------------------------------------------------------------------
// Eq. 2, pass 2: the softmax statistics of every head from the token blocks' partials, and from them the
// factor exp(m_block - M) / Z of each (block, head); then s_i = |h_i| (1/n_q) sum_j e_ij factor_j.
// Workgroup-wide helpers, 1024 threads.
//   factors of blocks tb0 .. tb0 + nblk - 1: s_f[blk][n_q].  (Of the exponentials that Z is summed from, a lane holds its blocks'.)
__device__ __forceinline__ void softmax_factors(const Batch& bt, const Seg& sg, int b, int n_q, const double* __restrict__ sm_part,
                                                int tb0, int nblk, double* s_f, int tid) {
    const int lane = tid & 63;
    const int ntb_max = (bt.n_max + SCORE_TOK - 1) / SCORE_TOK, ntb = (sg.n + SCORE_TOK - 1) / SCORE_TOK;
    const double* part = sm_part + (size_t)b * ntb_max * n_q * 2;
    // 32 lanes per head; 8 partials per lane stay in registers between the two steps (16384 tokens)
    const int l32 = lane & 31;
    for (int j = tid >> 5; j < n_q; j += 32) {
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = l32 + 32 * u < ntb ? *(const double2*)(part + ((size_t)(l32 + 32 * u) * n_q + j) * 2) : make_double2(-INFINITY, 0.0);
        double m = v[0].x;
#pragma unroll
        for (int u = 1; u < 8; ++u) m = fmax(m, v[u].x);
        for (int k = l32 + 256; k < ntb; k += 32) m = fmax(m, part[((size_t)k * n_q + j) * 2]);
        m = group_max_f64<16>(m);
        m = fmax(m, __shfl_xor(m, 16, 64));
        double z = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (32 * u >= ntb) break;                                // (uniform)
            const double e = exp(v[u].x - m);
            z += v[u].y != 0.0 ? v[u].y * e : 0.0;
            v[u].x = e;
        }
        for (int k = l32 + 256; k < ntb; k += 32) {
            const double2 w = *(const double2*)(part + ((size_t)k * n_q + j) * 2);
            z += w.y != 0.0 ? w.y * exp(w.x - m) : 0.0;
        }
        z = group_sum_f64(z, 32);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int blk = l32 + 32 * u - tb0;
            if (blk >= 0 && blk < nblk) s_f[blk * n_q + j] = blk + tb0 < ntb ? v[u].x / z : 0.0;
        }
        for (int k = l32 + 256; k < tb0 + nblk; k += 32)
            if (k >= tb0) s_f[(k - tb0) * n_q + j] = k < ntb ? exp(part[((size_t)k * n_q + j) * 2] - m) / z : 0.0;
    }
    __syncthreads();
}
// the two ablations of Eq. 2: without the norm; norm only (softmax term -> 1/n)
__device__ __forceinline__ float finish_score(const Seg& sg, int n_q, double sum, double hn) {
    const double p = (sg.flags & PACT_FLAG_SCORE_NORM_ONLY) ? 1.0 / (double)sg.n : sum / (double)n_q;
    return (float)((sg.flags & PACT_FLAG_SCORE_NO_NORM) ? p : hn * p);
}

// grid (ceil(n_max/FINAL_TOK), B), block 1024: FINAL_PARTS threads per token (heads part, part + FINAL_PARTS, ...).
// 256 tokens a workgroup, or 128 from nine query heads on (28 heads: 10.8 -> 8.6 us; with four heads it is 2.3 us longer for 8 videos).
template <int FINAL_TOK>
__global__ __launch_bounds__(1024) void score_final_kernel(Batch bt, int n_q, const double* __restrict__ expl,
                                                           const double* __restrict__ hnorm,
                                                           const double* __restrict__ sm_part,
                                                           float* __restrict__ scores) {
    constexpr int NBLK = FINAL_TOK / SCORE_TOK, FINAL_PARTS = 1024 / FINAL_TOK;
    __shared__ double s_f[NBLK * PACT_MAX_QHEADS];
    __shared__ double s_acc[FINAL_PARTS - 1][FINAL_TOK];
    const int b = blockIdx.y;
    touch_args<40>(b);
    const Seg sg = bt.s[b];
    if ((int)blockIdx.x * FINAL_TOK >= sg.n) return;
    const int tid = threadIdx.x, tok = tid & (FINAL_TOK - 1), part = tid / FINAL_TOK;
    const int i = blockIdx.x * FINAL_TOK + tok;
    const size_t g = (size_t)sg.base + min(i, sg.n - 1);
    // this thread's values are requested before the partials are combined (they do not depend on them)
    const double hn = hnorm[g];
    double e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = part + FINAL_PARTS * u < n_q ? expl[g * n_q + part + FINAL_PARTS * u] : 0.0;
    softmax_factors(bt, sg, b, n_q, sm_part, blockIdx.x * NBLK, NBLK, s_f, tid);
    const double* f = s_f + (tok / SCORE_TOK) * n_q;
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (part + FINAL_PARTS * u < n_q) acc = fma(e[u], f[part + FINAL_PARTS * u], acc);
    for (int j = part + 4 * FINAL_PARTS; j < n_q; j += FINAL_PARTS) acc = fma(expl[g * n_q + j], f[j], acc);
    if (part > 0) s_acc[part - 1][tok] = acc;
    __syncthreads();
    if (part > 0 || i >= sg.n) return;
#pragma unroll
    for (int k = 0; k < FINAL_PARTS - 1; ++k) acc += s_acc[k][tok];
    scores[g] = finish_score(sg, n_q, acc, hn);
}

// ------------------------------------------------------------------------------------------
// Eq. 3/4, one workgroup of 1024 per sample, on the finished fp32 scores:
//   (a) the scores become order-preserving integer keys, in registers: wavefront w owns a contiguous range of tokens, 64 KREG at most;
//   (b) exact selection of the (m+1)-th smallest key, m = min(floor(lambda n), n-1);
//   (c) ordered compaction into the kept / pruned index lists.
// FINISH: samples of at most 1024 tokens finish their scores here as well (a thread per token; one launch
// fewer).  More values per sample than FUSE_VALUES are too much for one compute unit to fetch: they have score_final_kernel.
// Bound by its chain of barriers and LDS trips, on one CU.  The keys of a token stay in one lane from the scores to the lists (they were in LDS, the lists'
// order another one than the selection's); maxima and sums over wavefronts are lane permutes instead of shuffles and loops (event
// brackets, us): 196 tokens with FINISH 11.4 -> 8.8, 2915 tokens 10.4 -> 7.8, 7290 12.8 -> 10.4, 16384 21.5 -> 16.1.
constexpr int FUSE_TOKENS = 1024, FUSE_VALUES = 12288;
struct FinishArgs { const double *expl, *hnorm, *sm_part; int32_t n_q; };
__device__ __forceinline__ uint32_t ordered_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
// Largest value of a row of 16 lanes, in all of them / of the wavefront.
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v) {
    auto step = [&](uint32_t x) { v = max(v, x); };
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_XOR1, 0xF, 0xF, true));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_XOR2, 0xF, 0xF, true));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_HALF_MIRROR, 0xF, 0xF, true));
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_MIRROR, 0xF, 0xF, true));
    return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = row_max_u32(v);
    auto at = [&](int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    return max(max(at(0), at(16)), max(at(32), at(48)));
}
// Sums of 16 wavefronts' counts in LDS: of all of them; of those before wavefront `wave` (scalar).
__device__ __forceinline__ int counts_before(const int* s_cnt, int lane, int wave, int& all) {
    const int own = lane < 16 ? s_cnt[lane] : 0, inc = wave_scan_incl_i32(own);
    all = __builtin_amdgcn_readlane(inc, 15);
    return __builtin_amdgcn_readlane(inc - own, wave);
}

template <bool FINISH, int KREG>
__device__ __forceinline__ void prune_block(const Batch& bt, const FinishArgs& fin, float* scores,
                                            uint64_t* __restrict__ adj,
                                            int32_t* __restrict__ kept_idx,
                                            int32_t* __restrict__ pruned_idx,
                                            pact_report* __restrict__ rep) {
    __shared__ __align__(16) int s_hist[256 * 16];           // (cleared and scanned four bins at a time)
    __shared__ int s_bin[256];
    __shared__ int s_sel[2][2];
    __shared__ int s_wtot[2][16];
    __shared__ int s_odd[2];             // scores next to the threshold without being equal to it; non-finite scores
    __shared__ uint32_t s_mm[2][16], s_cand[64];
    __shared__ int s_ncand;
    const int b = blockIdx.x;
    const Seg sg = bt.s[b];
    const int n = sg.n;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* s = scores + sg.base;

    // this thread's tokens: i0 + 64 u + lane, below i1
    const int per_wave = ((n + 15) / 16 + 63) / 64 * 64;
    const int i0 = min(n, wave * per_wave), i1 = min(n, i0 + per_wave);
    uint32_t kreg[KREG];
    auto have = [&](int u) __attribute__((always_inline)) { return i0 + 64 * u + lane < i1; };
    {
        float sv[KREG];
        if constexpr (FINISH) {
            static_assert(KREG == 1, "a thread per token");
            constexpr int NBLK = FUSE_TOKENS / SCORE_TOK;
            __shared__ double s_f[NBLK * PACT_MAX_QHEADS];
            const int n_q = fin.n_q;
            const size_t g = (size_t)sg.base + min(tid, n - 1);
            const double hn = fin.hnorm[g];
            double e[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) e[u] = u < n_q ? fin.expl[g * n_q + u] : 0.0;
            softmax_factors(bt, sg, b, n_q, fin.sm_part, 0, NBLK, s_f, tid);
            const double* f = s_f + (tid / SCORE_TOK) * n_q;
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (u < n_q) acc[u & 3] = fma(e[u], f[u], acc[u & 3]);
            for (int j = 16; j < n_q; ++j) {
                const double v = fin.expl[g * n_q + j] * f[j];
                acc[0] += (j & 3) == 0 ? v : 0.0; acc[1] += (j & 3) == 1 ? v : 0.0;
                acc[2] += (j & 3) == 2 ? v : 0.0; acc[3] += (j & 3) == 3 ? v : 0.0;
            }
            sv[0] = finish_score(sg, n_q, (acc[0] + acc[1]) + (acc[2] + acc[3]), hn);
            if (tid < n) s[tid] = sv[0];
        } else {
#pragma unroll
            for (int u = 0; u < KREG; ++u) sv[u] = have(u) ? s[i0 + 64 * u + lane] : 0.0f;   // all in flight
        }
#pragma unroll
        for (int u = 0; u < KREG; ++u) kreg[u] = ordered_key(sv[u]);
    }

    const int m_rank = prune_rank(sg.lambda, n);
    int k = m_rank;
    uint32_t prefix = 0, mask = 0;
    // Selection in one histogram where that works: the keys of a sample share their leading bits
    // (scores of one image lie within a few binades), so the 4096 bins are laid over the range the
    // keys actually span, [smallest, largest]; the bin that holds rank k then has a handful of keys,
    // among which every wavefront finds the wanted one.  More than 64 keys in that bin
    // (ties, non-finite values that stretch the range): the radix select below does the whole job.
    bool selected = false, finite;
    {
        uint32_t kinv = 0u, kmax = 0u;                                       // (largest complement: the smallest key)
#pragma unroll
        for (int r = 0; r < KREG; ++r)
            if (have(r)) { kinv = max(kinv, ~kreg[r]); kmax = max(kmax, kreg[r]); }
        kinv = wave_max_u32(kinv);
        kmax = wave_max_u32(kmax);
        if (lane == 0) { s_mm[0][wave] = kinv; s_mm[1][wave] = kmax; }
        *(int4*)&s_hist[4 * tid] = make_int4(0, 0, 0, 0);
        if (tid == 0) { s_ncand = 0; s_odd[0] = 0; s_odd[1] = 0; }
        __syncthreads();
        const uint32_t kmin = ~(uint32_t)lane0_of((int)row_max_u32(s_mm[0][lane & 15]));
        kmax = (uint32_t)lane0_of((int)row_max_u32(s_mm[1][lane & 15]));
        finite = kmin > ordered_key(-INFINITY) && kmax < ordered_key(INFINITY);        // (NaN is beyond either)
        const uint32_t range = kmax - kmin;
        const int nbits = range ? 32 - __builtin_clz(range) : 0;
        const int bshift = nbits > 12 ? nbits - 12 : 0;                  // (key - kmin) >> bshift < 4096
#pragma unroll
        for (int r = 0; r < KREG; ++r)
            if (have(r)) atomicAdd(&s_hist[(kreg[r] - kmin) >> bshift], 1);
        __syncthreads();
        // exclusive scan over the bins, four per thread
        const int4 c4 = *(const int4*)&s_hist[4 * tid];
        const int c[4] = {c4.x, c4.y, c4.z, c4.w};
        const int loc = c4.x + c4.y + c4.z + c4.w;
        const int inc = wave_scan_incl_i32(loc);
        if (lane == 63) s_wtot[0][wave] = inc;
        __syncthreads();
        int all;
        int e = counts_before(s_wtot[0], lane, wave, all) + inc - loc;
        if (k >= e && k < e + loc) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (k >= e && k < e + c[t]) { s_sel[0][0] = 4 * tid + t; s_sel[0][1] = k - e; s_sel[1][0] = c[t]; }
                e += c[t];
            }
        }
        __syncthreads();
        const int sel = lane0_of(s_sel[0][0]), kk = lane0_of(s_sel[0][1]), ncand = lane0_of(s_sel[1][0]);
        if (ncand <= 64) {                                                   // (uniform)
#pragma unroll
            for (int r = 0; r < KREG; ++r)
                if (have(r) && (int)((kreg[r] - kmin) >> bshift) == sel) s_cand[atomicAdd(&s_ncand, 1)] = kreg[r];
            __syncthreads();
            // (counted one by one: by the bits in which they can differ, a ballot each, took 1.3 us longer for 3 candidates and 0.4 less for 40)
            const uint32_t v = lane < ncand ? s_cand[lane] : 0xFFFFFFFFu;
            int below = 0, equal = 0;
            for (int j = 0; j < ncand; ++j) {
                const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)v, j);
                below += u < v;
                equal += u == v;
            }
            const uint64_t found = __ballot(lane < ncand && below <= kk && kk < below + equal);      // (lanes of the same value)
            prefix = (uint32_t)__builtin_amdgcn_readlane((int)v, found ? __builtin_ctzll(found) : 0);
            selected = true;
        } else __syncthreads();            // (s_hist and s_sel are used again below)
    }
    if (!selected) {
    // Radix select, 8 bits per pass from the top.  Scores of one image share their leading bits,
    // so a plain histogram would serialise thousands of atomics on a handful of LDS words: every
    // bin has 16 copies (one per lane & 15, in 16 different banks), summed after the pass.
    for (int i = tid; i < 256 * 16; i += 1024) s_hist[i] = 0;
    __syncthreads();
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
#pragma unroll
        for (int r = 0; r < KREG; ++r) {
            const uint32_t u = kreg[r];
            if (have(r) && (u & mask) == prefix)
                atomicAdd(&s_hist[(((u >> shift) & 255) << 4) + (lane & 15)], 1);
        }
        __syncthreads();
        if (tid < 256) {                   // sum the 16 copies of a bin and leave them cleared for the next pass
            int t = 0;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const int a = (tid << 4) + ((c + tid) & 15);   // (rotated: spreads the banks)
                t += s_hist[a];
                s_hist[a] = 0;
            }
            s_bin[tid] = t;
        }
        __syncthreads();
        if (tid < 64) {
            const int c0 = s_bin[4 * tid], c1 = s_bin[4 * tid + 1];
            const int c2 = s_bin[4 * tid + 2], c3 = s_bin[4 * tid + 3];
            const int loc = c0 + c1 + c2 + c3;
            const int inc = wave_scan_incl_i32(loc);
            int e = inc - loc;   // keys with a smaller digit
            const int c[4] = {c0, c1, c2, c3};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (k >= e && k < e + c[t]) { s_sel[pass & 1][0] = 4 * tid + t; s_sel[pass & 1][1] = k - e; }
                e += c[t];
            }
        }
        __syncthreads();                   // (s_sel alternates, so no barrier is needed after reading it)
        prefix |= (uint32_t)s_sel[pass & 1][0] << shift;
        mask |= 255u << shift;
        k = s_sel[pass & 1][1];
    }
    }
    const uint32_t tau = prefix;

    // Ordered split (Eq. 3 / 4): a ballot per 64 tokens gives each its place, so both index lists are written in coalesced runs.
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < KREG; ++r) cnt += __popcll(__ballot(have(r) && kreg[r] >= tau));
    if (lane == 0) s_wtot[1][wave] = cnt;
    __syncthreads();
    // the threshold as a score again (inverse of ordered_key), for the two counters of the report
    const float tau_f = __uint_as_float((tau & 0x80000000u) ? (tau & 0x7FFFFFFFu) : ~tau);
    const double tau_band = 1e-6 * fabs((double)tau_f);
    int n_near = 0, n_bad = 0, total;
    int kp = counts_before(s_wtot[1], lane, wave, total);
    int32_t* ko = kept_idx + sg.base;
    int32_t* po = pruned_idx + sg.base;
#pragma unroll
    for (int r = 0; r < KREG; ++r) {
        if (i0 + 64 * r >= i1) break;                            // (uniform)
        const int t = i0 + 64 * r + lane;
        const bool in = have(r);
        const uint32_t key = in ? kreg[r] : tau;
        const bool keep = in && key >= tau;
        const uint64_t m = __ballot(keep);
        const int below = __popcll(m & ((1ull << lane) - 1ull));
        if (keep) ko[kp + below] = t;
        else if (in) po[t - (kp + below)] = t;
        kp += __popcll(m);
        const float f = __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
        // (the band in fp32 with something to spare first: hardly any score is inside it)
        const bool maybe = key != tau && !(fabsf(f - tau_f) > 1.01e-6f * fabsf(tau_f));
        if (__any(maybe)) n_near += __popcll(__ballot(maybe && fabs((double)f - (double)tau_f) <= tau_band));
        if (!finite) n_bad += __popcll(__ballot(in && !isfinite(f)));
    }
    if (lane == 0 && (n_near | n_bad)) { atomicAdd(&s_odd[0], n_near); atomicAdd(&s_odd[1], n_bad); }
    __syncthreads();
    if (tid == 0) {
        rep[b].n_kept = total;
        rep[b].n_pruned = n - total;
        rep[b].score_near_ties = s_odd[0];
        rep[b].nonfinite_seen = s_odd[1];
    }
    // Scores tied at the threshold: more tokens are kept than the n - m whose bitmap rows and
    // words were cleared along with the key norms; clear what the clustering will use.
    if (adj && total > n - m_rank) {
        uint64_t* rows = adj + (size_t)b * bt.n_max * bt.W;
        const int Wq = (total + 63) >> 6;
        for (int r = wave; r < total; r += 16)
            for (int w = lane; w < Wq; w += 64) rows[(size_t)r * bt.W + w] = 0ull;
    }
}

struct PruneArgs { FinishArgs fin; float* scores; uint64_t* adj; int32_t *kept_idx, *pruned_idx; pact_report* rep; };
template <bool FINISH, int KREG>
__global__ __launch_bounds__(1024) void score_prune_kernel(Batch bt, PruneArgs a) {
    touch_args<sizeof(PruneArgs)>(blockIdx.x);
    prune_block<FINISH, KREG>(bt, a.fin, a.scores, a.adj, a.kept_idx, a.pruned_idx, a.rep);
}
// With the clustering keys of the call (KDT: their type) behind the samples' workgroups.  (The split alone is half a microsecond longer with their code.)
template <bool FINISH, int KREG, int KDT>
__global__ __launch_bounds__(1024) void score_prune_keys_kernel(Batch bt, PruneArgs a, KeyArgs key) {
    touch_args<sizeof(PruneArgs) + sizeof(KeyArgs)>(min((int)blockIdx.x, PACT_MAX_BATCH - 1));
    if ((int)blockIdx.x < bt.B) prune_block<FINISH, KREG>(bt, a.fin, a.scores, a.adj, a.kept_idx, a.pruned_idx, a.rep);
    else key_block<KDT, 16>(bt, key, (int)blockIdx.x - bt.B, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
}

// ------------------------------------------------------------------------------------------
static hipError_t raise_lds_limit(const void* fn, size_t bytes) {
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// The launch that prepares the clustering keys: the query sums', the logits' or the split's of a reduction, or one of their own.
enum { KEYS_FIRST, KEYS_LOGITS, KEYS_SPLIT, KEYS_ALONE };
constexpr int CUS = 256;

// How they are dealt there: lanes per row, rows per group of lanes, workgroups (of 1024 threads beside the split, otherwise of 256).
struct KeyPlan { int lanes, rows, blocks; };
static KeyPlan key_plan(const Batch& bt, pact_dtype k_dt, int32_t dk, int where) {
    static_assert(FRONT_THREADS == 256, "four wavefronts");
    const bool bf16 = k_dt == PACT_BF16, among_splits = where == KEYS_SPLIT && bt.B > 1;
    const int chunks = dk * (bf16 ? 2 : 4) / 16, lanes = chunks <= 16 ? 16 : chunks <= 32 ? 32 : 64;
    auto blocks = [&](int rows) { const int each = (where == KEYS_SPLIT ? 16 : 4) * (64 / lanes) * rows; return (bt.total + each - 1) / each; };
    // Several rows per group of lanes, where there are rows enough: of few the launch is one wavefront's chain, which more rows make longer.  Whole calls, a row at a time / four (fp32 keys: two), us:
    // * Single samples: hardly a difference (128 wide 2500 tokens 71.2 / 70.7, 6500 87.3 / 87.2; 512 wide 860 69.5 / 69.4, 2000 81.7 / 81.7; fp32 keys 128 wide 2500 76.1 / 75.8, 512 wide 5001 127.3 / 126.7).
    // * Batches, beside the logits (rows of four in two samples, which look for their samples one by one, are likely the last ones): 512 wide 2 of 1500 86.5 / 86.2, of 3250 113.3 / 110.7, 128 wide
    //   2 of 1500 72.9 / 73.3, of 2250 76.2 / 76.3, 1024 wide 4 of 1125 124.1 / 122.5, of 1625 143.5 / 140.4; fp32 keys 512 wide 4 of 1458 123.3 / 121.2, 8 of 2688 286.7 / 283.2.
    // * Batches, beside the splits, whose workgroups are one to a CU (that many, a row at a time): 512 wide 16 of 190 (204) 94.8 / 96.1, of 400 (422) 105.8 / 106.4, of 560 (578) 117.7 / 116.2; 1024 wide 8 of
    //   750 (383) 133.1 / 135.9, 16 of 560 (578) 148.2 / 146.9; 128 wide 32 of 440 (251) 90.5 / 91.9, 16 of 1000 (266) 97.3 / 98.1, 32 of 720 (391) 110.5 / 110.7 and with 14 query heads 121.5 / 120.1, of 1000 (532) 132.5 / 130.2; fp32 keys
    //   128 wide 16 of 400 (219) 78.9 / 79.7, of 560 (297) 89.3 / 86.8, 512 wide 4 of 750 (192) 95.1 / 97.1, 8 of 750 (383) 118.6 / 116.3.
    // * Keys alone (the kernel itself): where one row each is nearly the wavefronts that the chip holds (512 wide, 6272 tokens 6.6 / 7.5, 7290 6.7 / 6.2, 16384 13.0 / 10.0; 128 wide, 16384 8.2 / 15.4,
    //   32768 22.3 / 20.8).
    const int rows_enough = chunks > 64 ? 5000 : chunks > 32 ? (bt.B > 1 ? 3000 : 1200) : bt.B > 1 ? 5000 : 2500;
    const bool many = chunks > 128           ? false
                    : where == KEYS_ALONE    ? bf16 && (long)bt.total * lanes / 64 >= 7000
                    : among_splits           ? blocks(1) + bt.B > (!bf16 ? CUS : lanes == 16 ? CUS * 3 / 2 : CUS * 7 / 4)
                                             : bt.total >= rows_enough;
    // (bf16, eight rows / four: 2 x 6272 tokens 512 wide 189.5 / 191.4, 9 x 1458 149.5 / 151.2, 32 x 720 200.5 / 201.9, 8 x 6272 436.2 / 435.0; alone beside the split 12001 198.7 / 198.1, 14001 228.9 / 230.2, 16384
    // 276.3 / 279.0; beside the splits of a batch 16 x 875 162.3 / 158.1)
    const int rows = !many ? 1 : !bf16 ? 2 : chunks > 32 && chunks <= 64 && bt.total >= 12000 && !among_splits ? 8 : 4;
    return {lanes, rows, blocks(rows)};
}

// What their workgroups need; the number of those.
static int key_args(KeyArgs& a, const Batch& bt, const Ws& w, const ReductionIn& red, int mode, const int32_t* n_idx_dev, int where) {
    const KeysIn& in = red.keys;
    a.keys = (const char*)in.keys; a.dk = in.dk;
    a.nn = w.nn; a.rinv = w.rinv; a.adj = w.adj; a.rho = w.rho; a.rho_lo = w.rho_lo;
    a.status = w.status; a.ident = w.ident; a.near_cnt = w.near_cnt; a.tie_cnt = w.tie_cnt;
    a.rep = red.rep; a.cluster_id = red.cluster_id; a.cluster_counts = red.cluster_counts; a.n_idx_dev = n_idx_dev;
    a.zeros = w.zeros; a.ksplit = w.ksplit;
    a.mode = mode;
    const KeyPlan plan = key_plan(bt, in.k_dt, in.dk, where);
    a.key_lanes = plan.lanes; a.rows_each = plan.rows;
    return plan.blocks;
}

int launch_front(const Batch& bt, const Ws& w, const KeysIn& keys, pact_report* rep, int32_t* cluster_id, int mode,
                 const int32_t* n_idx_dev, hipStream_t st) {
    KeyArgs a = {};
    const dim3 grid(key_args(a, bt, w, ReductionIn{keys, rep, cluster_id, nullptr}, mode, n_idx_dev, KEYS_ALONE));
    if (keys.k_dt == PACT_BF16) PACT_LAUNCH("front", front_kernel<PACT_BF16>, grid, dim3(256), st, bt, a);
    else PACT_LAUNCH("front", front_kernel<PACT_F32>, grid, dim3(256), st, bt, a);
    return PACT_OK;
}

static int launch_query_sums(const Batch& bt, const Ws& w, const ScoreIn& in, const NormArgs& norm, const KeyArgs* key, int key_blocks, hipStream_t st) {
    QueryArgs a = {};
    a.q = (const char*)in.q; a.qcols = in.n_q * in.d_h;
    const int cw = 128 / (in.q_dt == PACT_BF16 ? 2 : 4), strips = (a.qcols + cw - 1) / cw;
    a.q_chunks = query_chunks(bt.n_max, a.qcols);
    a.qg_part = query_sums(w, a.q_chunks);
    a.blocks = strips * a.q_chunks * bt.B;
    a.norm = norm;
    const int per_block = FRONT_THREADS / 64 * hnorm_tokens(norm.h, norm.h_bf16 ? 2 : 4);
    if (key) { a.key = *key; a.key_blocks = key_blocks; }
    const dim3 grid(a.blocks + a.key_blocks + (norm.to - norm.from + per_block - 1) / per_block);
#define PACT_QUERY(KDT, QDT) PACT_LAUNCH("front", (query_sums_kernel<KDT, QDT>), grid, dim3(FRONT_THREADS), st, bt, a)
    if (in.k_dt == PACT_BF16) {
        if (in.q_dt == PACT_BF16) PACT_QUERY(PACT_BF16, PACT_BF16);
        else PACT_QUERY(PACT_BF16, PACT_F32);
    } else {
        if (in.q_dt == PACT_BF16) PACT_QUERY(PACT_F32, PACT_BF16);
        else PACT_QUERY(PACT_F32, PACT_F32);
    }
#undef PACT_QUERY
    return PACT_OK;
}

// Scores of every sample, up to the token blocks' softmax partials, and the norms of the hidden states `norm` names.  The query sums must be there.
// key: the call's clustering keys, if they are in this launch, or nullptr.
static int launch_logits(const Batch& bt, const Ws& w, const ScoreIn& in, const NormArgs& norm, const KeyArgs* key, int key_blocks, hipStream_t st) {
    LogitsArgs a = {};
    a.keys = (const char*)in.keys_pre; a.n_kv = in.n_kv; a.d_h = in.d_h; a.n_q = in.n_q;
    a.q_given = in.q_per_token ? nullptr : (const char*)in.q; a.q_bf16 = in.q_dt == PACT_BF16;
    a.q_chunks = query_chunks(bt.n_max, in.n_q * in.d_h);
    a.qg_part = query_sums(w, a.q_chunks);
    a.expl = w.logits; a.sm_part = w.sm_part;
    const int way = logits_way(in.n_kv, in.n_q, in.d_h, in.k_dt == PACT_BF16 ? 2 : 4), r = in.n_q / in.n_kv;
    a.kv_heads = way == BY_MFMA ? 1 : way == BY_LANES ? logits_kv_heads_lanes(bt, in.n_kv, in.d_h / (in.k_dt == PACT_BF16 ? 8 : 4))
                                       : logits_kv_heads_any(in.n_kv, in.n_q, in.d_h);
    const int cols = way == BY_MFMA ? r * (4 * (in.d_h / 4 + 1) + 1) : a.kv_heads * r * in.d_h;
    a.qg_lds = cols <= LOGITS_COLS_ANY;
    a.blocks = (bt.n_max + SCORE_TOK - 1) / SCORE_TOK * (in.n_kv / a.kv_heads);
    a.logits_blocks = a.blocks * bt.B;
    LogitsMoreArgs m = {};
    m.norm = norm;
    if (key) { m.key = *key; m.key_blocks = key_blocks; }
    const int per_block = 4 * hnorm_tokens(norm.h, norm.h_bf16 ? 2 : 4), h_blocks = (norm.to - norm.from + per_block - 1) / per_block;
    // Key blocks ahead of those of the hidden states, but evenly among them in large batches whose clustering keys are the tensor that the logits read, as bf16: its rows, read
    // a second time, are then spread over the launch.  (Whole call, first / among, us.  One tensor: 16 x 2688 tokens 301.3 / 299.1, 8 x 6272 385.7 / 382.1, 16 ragged images 357.0 / 355.9 and with
    // 28 query heads 439.6 / 437.9, 16 x 4095 514.1 / 510.8, 12 x 2688 257.4 / 256.3, 8 x 3645 269.6 / 269.0; 4 x 6272 238.5 / 239.1, 2 x 2915 106.1 / 106.7, 5 x 1458 109.9 / 110.8.  Two tensors: 16 x 2688 299.2 / 300.6 and with 28 query
    // heads 385.0 / 388.7, 8 x 6272 390.6 / 392.7, ragged 360.7 / 362.4, 3 x 7290 256.2 / 258.3.)
    const uint64_t rest = (uint64_t)m.key_blocks + h_blocks;
    const bool among = key && in.k_dt == PACT_BF16 && key->keys == (const char*)in.keys_pre && bt.total > 26000;
    m.key_share = among ? (uint32_t)((((uint64_t)m.key_blocks << 32) + rest - 1) / rest) : 0u;       // (no hidden states here: 2^32, which is 0)
    const bool more = rest > 0;
    dim3 grid(a.logits_blocks + (unsigned)rest);
    const size_t lds = a.qg_lds ? sizeof(double) * cols : 0;
    if (lds > 24 * 1024) {
        static size_t raised[12] = {};
        const int di = (in.k_dt == PACT_BF16 ? 1 : 0) + 2 * way + (more ? 6 : 0);
#define PACT_LOGITS_OF(KERNEL)                                                                                                \
    (const void*)KERNEL<PACT_F32, BY_HEAD>, (const void*)KERNEL<PACT_BF16, BY_HEAD>, (const void*)KERNEL<PACT_F32, BY_LANES>, \
        (const void*)KERNEL<PACT_BF16, BY_LANES>, (const void*)KERNEL<PACT_F32, BY_MFMA>, (const void*)KERNEL<PACT_BF16, BY_MFMA>
        const void* fns[12] = {PACT_LOGITS_OF(score_logits_kernel), PACT_LOGITS_OF(score_logits_more_kernel)};
#undef PACT_LOGITS_OF
        if (lds > raised[di]) {
            if (raise_lds_limit(fns[di], lds) != hipSuccess) return PACT_ERR_HIP;
            raised[di] = lds;
        }
    }
#define PACT_LOGITS(KDT, WAY)                                                                                                     \
    do {                                                                                                                          \
        if (more) PACT_LAUNCH_SHMEM("score_logits", (score_logits_more_kernel<KDT, WAY>), grid, dim3(256), lds, st, bt, a, m);    \
        else PACT_LAUNCH_SHMEM("score_logits", (score_logits_kernel<KDT, WAY>), grid, dim3(256), lds, st, bt, a);                 \
    } while (0)
    if (in.k_dt == PACT_BF16) {
        if (way == BY_MFMA) PACT_LOGITS(PACT_BF16, BY_MFMA);
        else if (way == BY_LANES) PACT_LOGITS(PACT_BF16, BY_LANES);
        else PACT_LOGITS(PACT_BF16, BY_HEAD);
    } else {
        if (way == BY_MFMA) PACT_LOGITS(PACT_F32, BY_MFMA);
        else if (way == BY_LANES) PACT_LOGITS(PACT_F32, BY_LANES);
        else PACT_LOGITS(PACT_F32, BY_HEAD);
    }
#undef PACT_LOGITS
    return PACT_OK;
}

static bool finish_in_prune(const Batch& bt, int n_q) {
    return bt.n_max <= FUSE_TOKENS && (long)bt.n_max * n_q <= FUSE_VALUES;
}

constexpr int KEYS_SHORT = 4096;         // tokens of a single sample whose keys are never beside the split
// Single samples of more than 4096 tokens with narrow queries and little to read otherwise have all of it in the first launch.  (Whole call, all first / as below, us.  Four query heads, hidden states 3584 wide: 4374
// tokens 94.5 / 93.7, 5832 110.9 / 110.7, 6561 116.0 / 117.6, 7290 123.0 / 124.9, 8748, 81 MB, 150.2 / 151.5; 9701, 89 MB, 164.9 / 165.0; 10501, 97 MB, 171.3 / 169.4, 14001 232.7 / 229.4.  fp32 keys 4200
// 110.3 / 111.9, 5001 127.4 / 129.4, 7290, 82 MB, 174.7 / 175.1, 9001, 101 MB, 220.2 / 220.1.  896 wide: 4200 82.1 / 83.5, 7290 96.6 / 97.2.  Wide queries, 28 heads: 2915 89.6 / 89.5, 5001 112.4 / 111.4, 7290, 112 MB, 138.1 /
// 134.8.  Up to 4096 tokens, where the keys would be beside the logits and not the split: 729 50.9 / 50.2 and 75.3 / 74.5 with fp32 keys, 2187 83.3 / 82.7, 3645 90.1 / 89.5.)
static bool inputs_first(const Batch& bt, const ScoreIn& in) {
    const int64_t kb = in.k_dt == PACT_BF16 ? 2 : 4, qb = in.q_dt == PACT_BF16 ? 2 : 4, hb = in.h_dt == PACT_BF16 ? 2 : 4;
    return bt.B == 1 && in.q_per_token && bt.n_max > KEYS_SHORT && in.n_q * in.d_h <= QG_NARROW &&
           bt.total * (in.h * hb + (int64_t)in.n_q * in.d_h * qb + (int64_t)in.n_kv * in.d_h * kb) < (int64_t)90e6;
}
// Which launch prepares a reduction's keys: the first; the split's of long single samples, and of batches whose scores are finished there too as long as its workgroups, one to a CU, are one turn; otherwise that of the
// logits.  (Whole calls, beside the logits / beside the split, us.  Single samples: a query given as its mean 1500 tokens 72.1 / 74.4, 2915 82.5 / 83.8, 4095 91.4 / 92.6, 5001 97.4 / 98.0, 7290 117.8 / 115.6, 16384 280.9 / 275.5,
// with fp32 keys 7290 174.7 / 169.6 and 16384 477.0 / 479.1; 28 query heads 4500 110.5 / 109.4, 7290 137.4 / 134.9, 16384 311.8 / 308.0; four 10001 168.3 / 166.4, 32768 690.0 / 682.0.  Batches, with the workgroups
// that the split then has: 512 wide 16 of 875 (235) 161.1 / 157.7, 16 of 1000 (266) 163.9 / 167.2, 32 of 720 (392) 201.9 / 203.5, 64 of 220 (283) 163.4 / 167.5, of 470 (533) 237.9 / 244.2; 256 wide 32 of 720 (212)
// 174.7 / 173.4, 64 of 470 (299) 211.7 / 214.2; 128 wide, 14 query heads, 32 of 720 (122) 123.7 / 122.2, 64 of 720 (244) 174.7 / 172.2, two heads 64 of 940 (299) 188.9 / 191.7; 1024 wide 16 of 875 (235) 186.5 / 184.4, 32 of
// 720 (392) 238.7 / 242.0; fp32 keys 512 wide 16 of 400 (219) 121.9 / 120.0, of 560 (298) 138.1 / 142.2, 128 wide 32 of 440 (251) 100.1 / 98.2, 64 of 220 (283) 101.8 / 104.1.)
// (Where the logits go head by head their launch is a call's longest, and the keys belong there whatever the size, up to the first rule: beside the logits / beside the split, 8 heads of 72, one query head each, 32 of 406 tokens
// 203.3 / 221.9, 32 of 812 281.0 / 287.4; seven each, 6000 568.4 / 595.2; 8 of 80, two each, 32 of 406 268.3 / 286.0, 6000 244.2 / 256.8; 4 of 72, one each, 32 of 812 221.8 / 227.5.)
static int keys_launch(const Batch& bt, const ScoreIn& in) {
    if (inputs_first(bt, in)) return KEYS_FIRST;
    if (logits_way(in.n_kv, in.n_q, in.d_h, in.k_dt == PACT_BF16 ? 2 : 4) == BY_HEAD) return KEYS_LOGITS;
    if (bt.B == 1) return bt.n_max > KEYS_SHORT ? KEYS_SPLIT : KEYS_LOGITS;
    return finish_in_prune(bt, in.n_q) && key_plan(bt, in.k_dt, in.n_kv * in.d_h, KEYS_SPLIT).blocks + bt.B <= CUS ? KEYS_SPLIT : KEYS_LOGITS;
}
// Hidden states, of the whole batch, whose norms are in the first launch.  Of batches such that both launches read as much (16 ragged images 74.6 us with none, 74.9, 8 x 6272 87.4 and 85.8), also beside BY_HEAD, whose LDS leaves a CU room for two
// to four of their workgroups: four heads of 72 with 28 query heads, whole calls, all in the first launch / as here, 16384 tokens 484.7 / 474.6, 8 x 1458 368.8 / 362.4, 16 x 2688 608.0 / 577.5, 8 x 6272 898.2 / 870.3, 64 query heads over two of 96
// 7290 654.0 / 647.0.  Of single samples of more than 4096 tokens too where the queries are little beside them, of others none.  (Whole calls, none / half, us: four query heads 10501 tokens 167.1 / 165.0, 12001 197.1 / 195.2, 32768 645.2 / 639.5;
// fp32 hidden states 8124 163.0 / 161.7, 16384 302.8 / 301.0, 7000 and two heads of 64 119.0 / 116.2, 13001 188.0 / 185.7.  fp32 queries 16384 466.7 / 468.6; 28 heads 7290 132.9 / 133.8, 12001 213.2 / 212.6, with fp32 hidden states
// 7290 146.6 / 148.2; up to 4096 tokens 3000 92.8 / 93.0, 1458 83.2 / 83.6.)
static int norms_first(const Batch& bt, const ScoreIn& in, int keys_launch) {
    if (inputs_first(bt, in)) return bt.total;
    const int kb = in.k_dt == PACT_BF16 ? 2 : 4;
    const int64_t row = (int64_t)in.h * (in.h_dt == PACT_BF16 ? 2 : 4), queries = (int64_t)in.n_q * in.d_h * (in.q_dt == PACT_BF16 ? 2 : 4);
    if (bt.B == 1 && (bt.n_max <= KEYS_SHORT || 4 * queries > row)) return 0;
    const int64_t keys = (int64_t)in.n_kv * in.d_h * kb * (keys_launch == KEYS_LOGITS ? 2 : keys_launch == KEYS_FIRST ? 0 : 1);     // (the logits' read, and that of their preparation)
    const int64_t share = (row + keys - queries) / 2;      // (bytes of each token's that the first launch has yet to read)
    return share <= 0 ? 0 : share >= row ? bt.total : (int)(bt.total * share / row) & ~15;
}

// The scores themselves; with `red` (what a reduction has beside them) small samples leave them to launch_score_prune.
int launch_score(const Batch& bt, const Ws& w, const ScoreIn& in, float* scores, const ReductionIn* red, hipStream_t st) {
    KeyArgs key = {};
    const int where = red ? keys_launch(bt, in) : KEYS_SPLIT;
    const int key_blocks = where == KEYS_SPLIT ? 0 : key_args(key, bt, w, *red, INIT_REDUCE, nullptr, where);
    const int hb = in.h_dt == PACT_BF16 ? 2 : 4;
    NormArgs norm{(const char*)in.hidden, w.hnorm, in.h, in.h_dt == PACT_BF16, hidden_streams(bt.total, in.h, hb) ? 1 : 0, 0, bt.total};
    if (in.q_per_token) {
        const int first = norms_first(bt, in, where);
        norm.to = first;
        if (const int rc = launch_query_sums(bt, w, in, norm, where == KEYS_FIRST ? &key : nullptr, key_blocks, st)) return rc;
        norm.from = first;
        norm.to = bt.total;
    }
    if (const int rc = launch_logits(bt, w, in, norm, where == KEYS_LOGITS ? &key : nullptr, key_blocks, st)) return rc;
    if (red && finish_in_prune(bt, in.n_q)) return PACT_OK;
    if (in.n_q > 8)
        PACT_LAUNCH("score_final", score_final_kernel<128>, dim3((bt.n_max + 127) / 128, bt.B), dim3(1024), st, bt,
                    in.n_q, w.logits, w.hnorm, w.sm_part, scores);
    else
        PACT_LAUNCH("score_final", score_final_kernel<256>, dim3((bt.n_max + 255) / 256, bt.B), dim3(1024), st, bt,
                    in.n_q, w.logits, w.hnorm, w.sm_part, scores);
    return PACT_OK;
}

// Splits the scores of every sample (Eq. 3 / 4).  red: what a reduction has beside them, or nullptr (the split alone): small samples' scores are
// then finished here, and its keys prepared for their clustering, if they are not yet.
int launch_score_prune(const Batch& bt, const Ws* w, const ScoreIn* in, float* scores, const ReductionIn* red, int32_t* kept_idx, int32_t* pruned_idx,
                       pact_report* rep, hipStream_t st) {
    KeyArgs key = {};
    uint64_t* adj = red ? w->adj : nullptr;
    const bool f32 = red && red->keys.k_dt == PACT_F32, keys_here = red && keys_launch(bt, *in) == KEYS_SPLIT;
    const dim3 grid(bt.B + (keys_here ? key_args(key, bt, *w, *red, INIT_REDUCE, nullptr, KEYS_SPLIT) : 0));
    PruneArgs a{{}, scores, adj, kept_idx, pruned_idx, rep};
#define PACT_PRUNE(FINISH, KREG)                                                                                                                \
    do {                                                                                                                                        \
        if (!keys_here) PACT_LAUNCH("score_prune", (score_prune_kernel<FINISH, KREG>), grid, dim3(1024), st, bt, a);                            \
        else if (f32) PACT_LAUNCH("score_prune", (score_prune_keys_kernel<FINISH, KREG, PACT_F32>), grid, dim3(1024), st, bt, a, key);          \
        else PACT_LAUNCH("score_prune", (score_prune_keys_kernel<FINISH, KREG, PACT_BF16>), grid, dim3(1024), st, bt, a, key);                  \
    } while (0)
    static_assert(PACT_MAX_TOKENS <= 1024 * 32, "a sample's keys in the registers of one workgroup");
    if (red && finish_in_prune(bt, in->n_q)) {
        a.fin = FinishArgs{w->logits, w->hnorm, w->sm_part, in->n_q};
        PACT_PRUNE(true, 1);
    }
    else if (bt.n_max <= 1024 * 4) {
        static_assert(KEYS_SHORT == 1024 * 4, "keys_launch gives the split of such samples no keys: there is no build for it");
        if (keys_here) return PACT_ERR_HIP;
        PACT_LAUNCH("score_prune", (score_prune_kernel<false, 4>), grid, dim3(1024), st, bt, a);
    }
    else if (bt.n_max <= 1024 * 8) PACT_PRUNE(false, 8);
    else if (bt.n_max <= 1024 * 16) PACT_PRUNE(false, 16);
    else PACT_PRUNE(false, 32);
#undef PACT_PRUNE
    return PACT_OK;
}

}  // namespace pact
