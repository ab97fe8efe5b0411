// DBDPC after the Gram pass (Alg. 2): density order, centre selection under the bound d_c
// by parallel looks (same centres as the sequential loop; cf. the recursive scheme of
// appendix D), nearest-centre assignment; and the recovery of pruned tokens (Eq. 8/9).
//
// Centre selection.  Token j "precedes" i when rho_j > rho_i, or rho_j == rho_i and j < i
// (the stable descending density order of Alg. 2).  Alg. 2 makes i a centre iff no centre
// that precedes it lies within d_c.  With adj[i][j] = (d_ij <= d_c) this is a fixed point
// every token can evaluate on its own from its list of preceding neighbours:
//     a preceding neighbour is a centre            -> i is not a centre
//     every preceding neighbour is known not to be -> i is a centre
// Every wavefront evaluates this for its undecided tokens again and again, on statuses that the others
// change meanwhile.  The lists come from one order of the tokens, so the densest undecided token can always
// be decided and the looks end; what a token becomes does not depend on how stale the statuses are that were read.
#include <cstring>
#include <type_traits>

#include "pact_internal.h"

namespace pact {

constexpr int KP = PRED_CAP - 1;   // preceding neighbours kept per token (slot 0 holds the count); more -> bitmap fallback

__device__ __forceinline__ int lanes_below(uint64_t mask, int lane) {
    return __popcll(mask & ((1ull << lane) - 1ull));
}

// A clustering key whose squared norm is zero, or not a finite number, is counted in the report.
__device__ __forceinline__ void note_odd_norm(pact_report* rp, double nn) {
    if (nn > 0.0 && nn < INFINITY) return;
    if (nn == 0.0) atomicAdd(&rp->zero_norm_seen, 1);
    else atomicAdd(&rp->nonfinite_seen, 1);
}

__device__ __forceinline__ bool precedes(double rho_j, int j, double rho_i, int i) {
    return rho_j > rho_i || (rho_j == rho_i && j < i);
}

// Eq. 5 in fp64 (as wave_dot64 computes it) between the token's row `mine` and the rows of its na candidates (tokens in ctok), by one
// wavefront, two candidates and CH 16-byte chunks of each row at a time.
template <int DT, int CH>
__device__ __forceinline__ void nearest_fp64(const lds_i32* cand, const lds_i32* ctok, int na, const char* mine, double nnp,
                                             const char* kb, size_t row_bytes, const double* nnb, int dk, int lane, double thr,
                                             double& best, int& bestc) {
    constexpr int EPL = Elem<DT>::EPL, STEP = 64 * EPL;
    for (int k = 0; k < na; k += 2) {
        const int k1 = min(k + 1, na - 1);
        const int c0 = cand[k], c1 = cand[k1];
        const int t0 = ctok[k], t1 = ctok[k1];
        const char* r0 = kb + (size_t)t0 * row_bytes;
        const char* r1 = kb + (size_t)t1 * row_bytes;
        const double n0 = nnb[t0], n1 = nnb[t1];
        double a0 = 0.0, a1 = 0.0;
        for (int e0 = lane * EPL; e0 < dk; e0 += CH * STEP) {
            uint4 va[CH], v0[CH], v1[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const size_t o = (size_t)(u == 0 || e0 + u * STEP < dk ? e0 + u * STEP : e0) * Elem<DT>::BYTES;
                va[u] = *(const uint4*)(mine + o);
                v0[u] = *(const uint4*)(r0 + o);
                v1[u] = *(const uint4*)(r1 + o);
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                if (u > 0 && e0 + u * STEP >= dk) break;
                double a[8], x[8];
                Elem<DT>::widen(va[u], a);
                Elem<DT>::widen(v0[u], x);
#pragma unroll
                for (int i = 0; i < EPL; ++i) a0 = fma(a[i], x[i], a0);
                Elem<DT>::widen(v1[u], x);
#pragma unroll
                for (int i = 0; i < EPL; ++i) a1 = fma(a[i], x[i], a1);
            }
        }
        const double d0 = cos_dist64(wave_sum_f64(a0), nnp, n0);
        const double d1 = cos_dist64(wave_sum_f64(a1), nnp, n1);
        if (d0 < thr && (d0 < best || (d0 == best && c0 < bestc))) { best = d0; bestc = c0; }
        if (k1 != k && d1 < thr && (d1 < best || (d1 == best && c1 < bestc))) { best = d1; bestc = c1; }
    }
}

// Nearest of `ncand` candidates (ids in LDS) of one token, by one wavefront; only distances
// < thr compete, ties go to the lower candidate id; (best, bestc) are updated, identical in
// every lane.  tok_of(c) maps a candidate id to its token.
//
// What such a search costs is the conversion of the rows to fp64, so it screens in fp32 first:
//  1. fp32 cosines of all candidates, eight at a time (the wavefront splits into eight groups
//     of 8 lanes, one candidate row each; lane `sub` takes the 16-byte chunks sub, sub + 8, ...
//     of the candidate's row against the token's own, four chunks of either in flight per lane);
//  2. a candidate whose fp32 cosine is more than 2 * margin below the largest one cannot be the
//     nearest (margin bounds the error of an fp32 cosine), so only the others - usually one -
//     are evaluated in fp64, each by the whole wavefront (Eq. 5 as wave_dot64 computes it: a
//     copy of the token's row is at distance exactly 0);
//  3. if a single candidate is left, `complete` says that the call sees all candidates of the
//     token, and its fp32 cosine is more than margin away from the threshold, it is decided
//     without fp64: `best` is then only a placeholder that no other call will be compared with.
template <int DT, typename TokOf>
__device__ __forceinline__ void nearest_candidate(lds_i32* cand, lds_i32* ctok, lds_f32* ccos, int ncand,
                                                  bool complete, const char* mine, double nnp,
                                                  const char* kb, size_t row_bytes, const double* nnb,
                                                  int dk, int lane, double thr, float margin, TokOf tok_of,
                                                  double& best, int& bestc) {
    constexpr int EPL = Elem<DT>::EPL;
    const int grp = lane >> 3, sub = lane & 7;
    const int nchunk = dk / EPL;                       // 16-byte chunks per row (rows are 16-byte multiples)
    // the tokens of all candidates in one round trip (not one per batch of eight)
    for (int i = lane; i < ncand; i += 64) ctok[i] = tok_of(cand[i]);
    // 1. fp32 cosines
    float top = -INFINITY;
    for (int c0 = 0; c0 < ncand; c0 += 8) {
        const int ci = c0 + grp;
        const bool valid = ci < ncand;
        const int tok = ctok[valid ? ci : c0];
        const char* rb = kb + (size_t)tok * row_bytes;
        const double nnc = nnb[tok];
        float acc = 0.0f;
        for (int k0 = sub; k0 < nchunk; k0 += 32) {    // 4 chunks of either row per lane per pass
            uint4 vb[4], va[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 8 * u;
                const size_t o = (size_t)(k < nchunk ? k : k0) * 16;
                vb[u] = *(const uint4*)(rb + o);
                va[u] = *(const uint4*)(mine + o);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (k0 + 8 * u < nchunk) {
                    float a[8], x[8];
                    Elem<DT>::widenf(va[u], a);
                    Elem<DT>::widenf(vb[u], x);
#pragma unroll
                    for (int i = 0; i < EPL; ++i) acc = fmaf(a[i], x[i], acc);
                }
            }
        }
        acc = group_sum_f32<8>(acc);
        const double den = sqrt(nnp * nnc);
        float cv = den > 0.0 ? (float)((double)acc / den) : 0.0f;
        if (valid && sub == 0) ccos[ci] = cv;
        if (!valid) cv = -INFINITY;
        // (the eight lanes of a candidate hold the same value: the other candidate of the row of 16 through a rotation)
        cv = fmaxf(cv, dpp_f32<0x128>(cv));                  // row_ror:8
#pragma unroll
        for (int s = 16; s <= 32; s <<= 1) cv = fmaxf(cv, __shfl_xor(cv, s, 64));
        top = fmaxf(top, cv);
    }
    // 2. the candidates that can still be the nearest, compacted in place (order kept)
    const float floor32 = top - 2.0f * margin;
    int na = 0;
    for (int i0 = 0; i0 < ncand; i0 += 64) {
        const int i = i0 + lane;
        const bool amb = i < ncand && ccos[i] >= floor32;
        const int c = amb ? cand[i] : 0, t = amb ? ctok[i] : 0;
        const uint64_t m = __ballot(amb);
        if (amb) { cand[na + lanes_below(m, lane)] = c; ctok[na + lanes_below(m, lane)] = t; }
        na += __popcll(m);
    }
    // 3. decided by the fp32 screen alone?
    const double cthr = 1.0 - thr;                     // d < thr  <=>  cosine > 1 - thr
    if (complete && na == 1 && (double)top - cthr > (double)margin) {
        best = fmax(1.0 - (double)top, 0.0);
        bestc = cand[0];
        return;
    }
    if ((double)top < cthr - (double)margin) return;   // nothing can pass the threshold
    nearest_fp64<DT, 1>(cand, ctok, na, mine, nnp, kb, row_bytes, nnb, dk, lane, thr, best, bestc);
}

// ------------------------------------------------------------------------------------------
// After the density pass: the pairs its epilogue could not decide in fp32.  Eq. 5 in fp64, the bit
// cleared where the distance exceeds d_c.  One wavefront per listed pair and turn, so that the pairs are
// spread evenly (near d_c the pairs of a row come in clumps: settled by the wavefronts that build the rows'
// lists, or by workgroups of 32 rows, they took 3 to 13 us longer); a wavefront's pairs, tokens and norms arrive in three
// trips, then one trip per pair brings both rows (up to eight chunks of either per lane in flight).
// Rows of more than 2 KB are screened in fp32 (bf16 on v_dot2_f32_bf16): a lane's chain is a 64th of the row, so its error is a fortieth of the margin that
// listed the pair and nearly all are decided by it, without the conversions to fp64.  And they are bound by what their rows take to come (340 MB for 23 700 pairs of 7 KB
// rows), so the pairs of a tile of the density pass, which share rows, stay on one XCD.  7290 rows of 7 KB, bracket 51.6 us, by XCD 41, with the screen 36.6,
// on the dot instruction 32.6, 1024 workgroups (what the chip holds) instead of 768 31; 2000 rows 27 -> 21; 7290 fp32 rows 69.5 -> 44.5.  Short
// rows: 16 ragged images 10.2 -> 10.9 by XCD, 11.6 with 1024.
// PARTS: parts of the pairs' list (near_parts).  A list in one part has a build of its own: with the search for a pair's part and a vector load of the counter in it, 16 ragged images took 10.3 us
// instead of 8.7, 8 videos 7.1 instead of 6.1.
// grid (settle_blocks(), B), block 256.
static int settle_blocks(int n_max, bool wide) { return n_max >= 6144 ? (wide ? 1024 : 768) : n_max < 512 ? 64 : n_max / 64 * 8; }   // (the benchmark image: a pair per wavefront)

template <int DT, int CH, int PARTS>
__global__ __launch_bounds__(256) void settle_kernel(Batch bt, const char* __restrict__ keys, int dk,
                                                     const int32_t* __restrict__ idx,
                                                     const double* __restrict__ nn,
                                                     const uint32_t* __restrict__ near_list,
                                                     const int32_t* __restrict__ near_cnt,
                                                     const uint32_t* __restrict__ far_bits, int far_words,
                                                     double* __restrict__ rho, const double* __restrict__ rho_lo,
                                                     uint64_t* adj, pact_report* rep) {
    const int b = blockIdx.y;
    const Seg sg = bt.s[b];
    if (sg.d_n < EXACT_SUMS_D_N)                               // densities that came in two parts (add_density)
        for (int p = blockIdx.x * 256 + threadIdx.x; p < sg.n; p += gridDim.x * 256)
            rho[(size_t)b * bt.n_max + p] += rho_lo[(size_t)b * bt.n_max + p];
    constexpr bool SCREEN = CH > 2;                            // wide rows
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int gw = blockIdx.x * 4 + wave;
    // the parts' counters, a lane each, and where in the list as a whole each part begins; the only one of a list in one part by a scalar load
    constexpr int room = NEAR_CAP / PARTS;
    const int32_t* counters = near_cnt + b * NEAR_PARTS * NEAR_COUNTER;
    uint2 taken = make_uint2(0u, 0u);
    int in_part, ends, cnt_all;
    if constexpr (PARTS == 1) {
        taken = make_uint2((uint32_t)counters[0], (uint32_t)counters[1]);
        in_part = ends = cnt_all = (int)min(taken.x, (uint32_t)room);
    } else {
        if (lane < PARTS) taken = *(const uint2*)(counters + lane * NEAR_COUNTER);
        in_part = (int)min(taken.x, (uint32_t)room);
        ends = wave_scan_incl_i32(in_part);
        cnt_all = __builtin_amdgcn_readlane(ends, 63);
    }
    auto place = [&](int e) __attribute__((always_inline)) {         // of entry e of the list as a whole
        if constexpr (PARTS == 1) return e;
        int part = 0;
#pragma unroll
        for (int k = 0; k < PARTS - 1; ++k) part += e >= __builtin_amdgcn_readlane(ends, k) ? 1 : 0;
        return part * room + e - __shfl(ends - in_part, part, 64);
    };
    // wide rows: an eighth of the list per XCD (workgroups are dealt to them round-robin; the grid is a multiple of 8): neighbouring pairs are of one tile of the
    // density pass and share rows, which its L2 then holds
    const int xcd = blockIdx.x & 7;
    const int from = SCREEN ? (int)((long)cnt_all * xcd >> 3) : 0, cnt = SCREEN ? (int)((long)cnt_all * (xcd + 1) >> 3) : cnt_all;
    const int first = SCREEN ? from + (int)(blockIdx.x >> 3) * 4 + wave : gw, nw = SCREEN ? (int)(gridDim.x >> 3) * 4 : (int)gridDim.x * 4;
    if (gw == 0) {
        // largest key distance: the wavefronts of the density pass each left theirs
        uint32_t fb = 0u;
        for (int k0 = lane; k0 < far_words; k0 += 16 * 64) {       // (16 words per lane and trip)
            uint32_t v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = k0 + 64 * u < far_words ? far_bits[(size_t)b * far_words + k0 + 64 * u] : 0u;
#pragma unroll
            for (int u = 0; u < 16; ++u) fb = max(fb, v[u]);
        }
#pragma unroll
        for (int sft = 32; sft >= 1; sft >>= 1) fb = max(fb, (uint32_t)__shfl_xor((int)fb, sft, 64));
        const bool overflow = __ballot(lane < PARTS && taken.x <= (uint32_t)room) == 0;
        int ordered = (int)taken.y;
        if constexpr (PARTS > 1) {
#pragma unroll
            for (int sft = 32; sft >= 1; sft >>= 1) ordered += __shfl_xor(ordered, sft, 64);
        }
        if (lane == 0) report_settled(rep + b, overflow, ordered, fb, sg.d_n);
    }
    constexpr int EPL = Elem<DT>::EPL;
    const size_t row_bytes = (size_t)dk * Elem<DT>::BYTES;
    const char* kb = keys + (size_t)sg.base * row_bytes;
    const int32_t* ix = idx + sg.base;
    const double* nnb = nn + sg.base;
    const double d_c = (double)sg.d_c;
    // error of a lane's chain of dk / 64 fp32 additions, with a near-tie's 1e-6 on top.  (Against fp64, 4096 pairs each of neighbours, unrelated rows, rows of one sign, rows that cancel, rows that
    // are mostly one element or of very unequal ones, 1032 to 8192 wide, the dot instruction's sums are off by at most 7% of the first term.)
    const double screen = ((double)dk / 64.0 + 24.0) * (1.0 / 8388608.0) + 1.1e-6;
    int ties = 0;
    for (int e0 = first; e0 < cnt; e0 += 64 * nw) {
        // lane l takes this wavefront's l-th pair (e0 + l * nw)
        const int my_e = e0 + lane * nw;
        uint32_t my_pi = 0, my_pj = 0;
        int my_ti = 0, my_tj = 0;
        double my_ni = 0.0, my_nj = 0.0;
        const int at = place(min(my_e, cnt - 1));
        if (my_e < cnt) {
            const uint2 pr = *(const uint2*)(near_list + ((size_t)b * NEAR_CAP + at) * 2);
            my_pi = pr.x; my_pj = pr.y;
            my_ti = ix[my_pi & ~NEAR_MIRROR]; my_tj = ix[my_pj];
            my_ni = nnb[my_ti]; my_nj = nnb[my_tj];
        }
        const int mine = min(64, (cnt - e0 + nw - 1) / nw);     // pairs of this wavefront
        for (int k = 0; k < mine; ++k) {
            // (k is the same in every lane: scalar lane reads)
            const uint32_t pi_raw = (uint32_t)__builtin_amdgcn_readlane((int)my_pi, k), pj = (uint32_t)__builtin_amdgcn_readlane((int)my_pj, k);
            const uint32_t pi = pi_raw & ~NEAR_MIRROR;
            const bool both = (pi_raw & NEAR_MIRROR) != 0;
            double d = 0.0;
            if (pi != pj) {
                const char* ri = kb + (size_t)__builtin_amdgcn_readlane(my_ti, k) * row_bytes;
                const char* rj = kb + (size_t)__builtin_amdgcn_readlane(my_tj, k) * row_bytes;
                // both rows, CH chunks of either per lane and trip
                auto over_rows = [&](auto&& use) __attribute__((always_inline)) {
                    for (int c0 = lane * EPL; c0 < dk; c0 += CH * 64 * EPL) {
                        uint4 va[CH], vb[CH];
#pragma unroll
                        for (int u = 0; u < CH; ++u) {
                            const size_t o = (size_t)(c0 + u * 64 * EPL < dk ? c0 + u * 64 * EPL : c0) * Elem<DT>::BYTES;
                            va[u] = *(const uint4*)(ri + o);
                            vb[u] = *(const uint4*)(rj + o);
                        }
#pragma unroll
                        for (int u = 0; u < CH; ++u)
                            if (c0 + u * 64 * EPL < dk) use(va[u], vb[u]);
                    }
                };
                bool decided = false;
                if constexpr (SCREEN) {
                    float acc = 0.0f;
                    over_rows([&](const uint4& va, const uint4& vb) __attribute__((always_inline)) {
                        if constexpr (DT == PACT_BF16) {
                            typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
                            const uint32_t a[4] = {va.x, va.y, va.z, va.w}, x[4] = {vb.x, vb.y, vb.z, vb.w};
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a[i]), __builtin_bit_cast(bf16x2_t, x[i]), acc, false);
                        } else {
                            float a[8], x[8];
                            Elem<DT>::widenf(va, a);
                            Elem<DT>::widenf(vb, x);
#pragma unroll
                            for (int i = 0; i < EPL; ++i) acc = fmaf(a[i], x[i], acc);
                        }
                    });
                    const double ni = __shfl(my_ni, k, 64), nj = __shfl(my_nj, k, 64);
                    d = cos_dist64(wave_sum_f64((double)acc), ni, nj);
                    const double len = sqrt(ni * nj);        // (products that overflow or vanish in fp32: fp64)
                    decided = len > 1e-15 && len < 1e30 && fabs(d - d_c) > screen;
                }
                if (!decided) {                              // (the same in every lane)
                    double acc = 0.0;                        // (the order of operations of wave_dot64)
                    over_rows([&](const uint4& va, const uint4& vb) __attribute__((always_inline)) {
                        double a[8], x[8];
                        Elem<DT>::widen(va, a);
                        Elem<DT>::widen(vb, x);
#pragma unroll
                        for (int i = 0; i < EPL; ++i) acc = fma(a[i], x[i], acc);
                    });
                    d = cos_dist64(wave_sum_f64(acc), __shfl(my_ni, k, 64), __shfl(my_nj, k, 64));
                }
            }
            if (lane == 0) {
                if (beyond_cutoff(d, d_c)) {
                    atomicAnd((unsigned long long*)&adj[((size_t)b * bt.n_max + pi) * bt.W + (pj >> 6)],
                              ~(1ull << (pj & 63)));
                    if (both)
                        atomicAnd((unsigned long long*)&adj[((size_t)b * bt.n_max + pj) * bt.W + (pi >> 6)],
                                  ~(1ull << (pi & 63)));
                }
                ties += near_ties_of(d, d_c, both);
            }
        }
    }
    if (lane == 0 && ties) atomicAdd(&rep[b].dc_near_ties, ties);
}

// Optional output: position of every kept token in the density order, by enumeration.
// grid (ceil(n_max/64), B), block 1024 = 64 tokens x 16 slices of the j range.
__global__ __launch_bounds__(1024) void rank_kernel(Batch bt, const pact_report* __restrict__ rep,
                                                    const double* __restrict__ rho, int32_t* rank_opt) {
    __shared__ int s_cnt[16][64];
    const int b = blockIdx.y;
    const int q = clamp_count(rep[b].n_kept, bt.s[b].n);
    if (blockIdx.x * 64 >= q) return;
    const int lane = threadIdx.x & 63;
    const int slice = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = blockIdx.x * 64 + lane;
    const double* r = rho + (size_t)b * bt.n_max;
    const double mine = (p < q) ? r[p] : 0.0;
    const int per = (q + 15) / 16;
    const int j0 = slice * per, j1 = min(q, j0 + per);
    int cnt = 0;
    for (int j = j0; j < j1; ++j) cnt += precedes(r[j], j, mine, p);
    s_cnt[slice][lane] = cnt;
    __syncthreads();
    if (threadIdx.x < 64 && p < q) {
        int tot = 0;
#pragma unroll
        for (int s = 0; s < 16; ++s) tot += s_cnt[s][lane];
        rank_opt[bt.s[b].base + p] = tot;
    }
}

// ------------------------------------------------------------------------------------------
// Lock-step extraction of the set bits of one 64-bit word per lane: each call of `step`
// pops at most one bit per lane and reports, wave-wide, how many lanes popped one.
struct BitPop {
    uint64_t word;
    __device__ __forceinline__ bool any() const { return __any(word != 0ull); }
    // returns true if this lane popped bit `bit`
    __device__ __forceinline__ bool pop(int& bit) {
        const bool has = word != 0ull;
        bit = has ? __builtin_ctzll(word) : 0;
        if (has) word &= word - 1;
        return has;
    }
};

// Density order between neighbours (Alg. 2 sorts by density; only the order of tokens within
// d_c of each other can change which of them becomes a centre).  The densities summed by the
// matrix pass are fp64 sums of fp32 terms: each term carries the rounding of its exponent
// (matrix-core accumulation, scaling products, one fused multiply-add; a = log2(e) / d_n is the
// factor that turns a cosine error into an exponent error) and of the hardware exponential,
// independent from term to term, so the error of a sum grows like the square root of the number
// of terms that matter.  Two neighbours whose sums differ by less than
//     2^-20 (1 + 4a) sqrt(max(rho_i, rho_j))
// are both listed, and their densities are evaluated again entirely in fp64 before the order
// between them is used.  Measured against fp64, difference of two neighbours' sums, standard error / largest seen /
// the band, bf16 keys and fp32 keys, 512 wide:
//   4010 tokens of an image   d_n = 0.25  1.4e-5 / 7.5e-5 / 2.6e-4   9.4e-6 / 4.7e-5 / 2.6e-4   (rho = 120)
//                             d_n = 0.5   7.0e-6 / 3.5e-5 / 2.9e-4   4.2e-6 / 2.1e-5 / 2.9e-4   (rho = 590)
//                             d_n = 2     2.5e-6 / 1.1e-5 / 1.8e-4   2.2e-6 / 0.9e-5 / 1.8e-4   (rho = 2450)
//                             d_n = 8     1.7e-6 / 0.7e-5 / 9.8e-5   1.7e-6 / 0.7e-5 / 9.8e-5   (rho = 3540)
//   8000 of a video           d_n = 2     2.8e-6 / 1.3e-5 / 2.6e-4   2.8e-6 / 1.3e-5 / 2.6e-4   (rho = 4980)
// i.e. a band of twenty to a hundred standard errors.  It is a statistical bound, not a worst-case one (that of an fp32 cosine would list
// half the tokens of an image), and it does not hold everywhere: the rounding of a token's reciprocal norm is shared by all
// its terms, and where nearly all tokens are alike (cosines near 1) the errors add up.  Half of 4010 tokens nearly alike: largest error 0.9 of
// the band at d_n = 2, 1.5 at 0.25; all of 7290: 2.4 and 3.0 (more than 1024 tokens are listed there, which is reported).  The
// order between two such neighbours may then be that of the sums; whatever it is, it is one order (order_changed).
__device__ __forceinline__ double recheck_band2(float d_n) {
    const double a = 1.4426950408889634 / (double)d_n;
    const double c = (1.0 / 1048576.0) * (1.0 + 4.0 * a);
    return c * c;                          // compared with (rho_i - rho_j)^2 / max(rho_i, rho_j)
}

// For every kept token: the list of its neighbours (bitmap row) that precede it in the
// density order, as 16-bit positions in slots 1..KP of its PRED_CAP-slot record; slot 0 holds
// the list length, or KP+1 if the list did not fit (the token is then evaluated from its
// bitmap row).  The first four slots are also written to the token's 8-byte head: most tokens
// have at most three preceding neighbours, and the kernel that runs the rounds - a single
// workgroup - then has 8 bytes per token to fetch instead of 32.  The head of a longer list starts with the densest
// neighbour instead (the first of the list as it is ordered by position): it is a centre more often than not, and
// the token is then decided without its record.
// GL lanes of a wavefront per token (16: four tokens per wavefront, most tokens have fewer
// neighbours than that; 64: one).  Every lane of the wavefront takes part, with p < 0 for no token.
// `odd` counts, per token, the neighbours whose density is too close to this token's: DETECT:
// inside the band above; otherwise (second pass, on fp64 densities): lower-numbered neighbours with
// a different density within 1e-11 of the sum.
constexpr int HEAD_PREDS = 3;
__host__ __device__ inline int positions(int n_max) { return (n_max + 63) / 64 * 64; }
constexpr int PREDS_SPREAD = 256;      // set bits of a wavefront's row words that are spread over the lanes through LDS
template <bool DETECT, int GL>
__device__ __forceinline__ int preds_of_row(int p, int q, const double* r, const uint64_t* row, uint16_t* out,
                                            uint16_t* head, volatile uint16_t* nb_wave, int lane, double band2) {
    static_assert(GL == 16 || GL == 64, "a row of lanes or the wavefront");
    constexpr int WPL = 64 / GL;                       // words per lane and turn
    constexpr int CAP = PREDS_SPREAD / WPL;            // list entries per token
    const int gl = lane & (GL - 1), gbase = lane & ~(GL - 1);
    volatile uint16_t* nb = nb_wave + (lane / GL) * CAP;
    const bool on = p >= 0;
    const double rp = on ? r[p] : 0.0;
    const int Wq = (q + 63) >> 6;
    int total = 0, odd = 0;
    float best = -1.0f;                                // densest predecessor this lane has seen, and its position
    int best_j = 0;
    auto group_bits = [&](bool v) __attribute__((always_inline)) {          // ballot of this token's lanes
        const uint64_t m = __ballot(v);
        return GL == 64 ? m : (m >> gbase) & ((1ull << (GL & 63)) - 1ull);
    };
    auto group_scan = [&](int v) __attribute__((always_inline)) {           // inclusive prefix sum over them
        v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
        if (GL == 64) {
            v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
            v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
        }
        return v;
    };
    auto last_of = [&](int v) __attribute__((always_inline)) { return GL == 64 ? lane63_of(v) : __shfl(v, gbase + GL - 1, 64); };
    // A token's neighbours are mostly close to it in the sequence, i.e. their bits sit in one or
    // two words of the row: lane by lane, a word's bits would be looked up one after the other,
    // each look-up (the neighbour's density) a trip to memory.  So the set bits of 64 words are
    // first spread over the lanes - the k-th set bit to lane k, through a small LDS list - and
    // the densities of up to GL neighbours are fetched in one trip.
    for (int w0 = 0; w0 < Wq; w0 += 64) {
        uint64_t word[WPL];
#pragma unroll
        for (int u = 0; u < WPL; ++u) word[u] = on && w0 + gl + GL * u < Wq ? row[w0 + gl + GL * u] : 0ull;
        while (true) {
            // (all of a lane's bits; CAP / GL at a time where a token's words hold more than its list does)
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < WPL; ++u) cnt += __popcll(word[u]);
            int inc = group_scan(cnt);
            if (__any(last_of(inc) > CAP)) {
                cnt = min(cnt, CAP / GL);
                inc = group_scan(cnt);
            }
            const int nbits = last_of(inc);
            if (__all(nbits == 0)) break;
            int at = inc - cnt;
#pragma unroll
            for (int u = 0; u < WPL; ++u)
                while (word[u] && at < inc) {                // (no memory access in this loop)
                    const int bit = __builtin_ctzll(word[u]);
                    nb[at++] = (uint16_t)(((w0 + gl + GL * u) << 6) + bit);
                    word[u] &= word[u] - 1;
                }
            __builtin_amdgcn_wave_barrier();
            // (wave-uniform trip count; the densities of WPL entries per lane arrive together)
            for (int k0 = 0; __any(k0 < nbits); k0 += WPL * GL) {
                int j[WPL];
                double rj[WPL];
                bool has[WPL];
#pragma unroll
                for (int u = 0; u < WPL; ++u) {
                    const int k = k0 + gl + GL * u;
                    has[u] = k < nbits;
                    j[u] = has[u] ? nb[k] : 0;
                    has[u] = has[u] && j[u] < q;
                    rj[u] = has[u] ? r[j[u]] : rp;
                }
#pragma unroll
                for (int u = 0; u < WPL; ++u) {
                    if (u > 0 && !__any(k0 + GL * u < nbits)) break;
                    const uint64_t m = group_bits(has[u] && precedes(rj[u], j[u], rp, p));
                    const bool pre = (m >> gl) & 1ull;
                    const int slot = total + __popcll(m & ((1ull << gl) - 1ull));
                    if (pre && slot < KP) out[1 + slot] = (uint16_t)j[u];
                    if (pre && slot < HEAD_PREDS) head[1 + slot] = (uint16_t)j[u];
                    total += __popcll(m);
                    if (pre && (float)rj[u] > best) { best = (float)rj[u]; best_j = j[u]; }
                    const double d = rj[u] - rp;
                    const bool close = DETECT ? j[u] != p && d * d <= band2 * fmax(rj[u], rp)
                                              : j[u] < p && d != 0.0 && fabs(d) <= 1e-11 * (rj[u] + rp);
                    odd += __popcll(group_bits(has[u] && close));
                }
            }
            __builtin_amdgcn_wave_barrier();                 // the list is rewritten
        }
    }
    if (__any(total > HEAD_PREDS)) {
        float top = group_max_f32<16>(best);
        if (GL == 64) {
            top = fmaxf(top, __shfl_xor(top, 16, 64));
            top = fmaxf(top, __shfl_xor(top, 32, 64));
        }
        const uint64_t m = group_bits(best == top);
        if (total > HEAD_PREDS && gl == __builtin_ctzll(m)) head[1] = (uint16_t)best_j;
    }
    if (gl == 0 && on) {
        const uint16_t c = (uint16_t)(total > KP ? KP + 1 : total);
        out[0] = c;
        head[0] = c;
    }
    return odd;
}

// grid (ceil(n_max * GL / 256), B), block 256: GL lanes per kept token (see launch_centres).  Tokens with a neighbour
// inside the band are appended to the sample's list, as position | token << 16 (tie_cnt[4b]
// counts them, also past the list's end: the re-evaluation is then skipped and reported).
template <int GL>
__global__ __launch_bounds__(256) void build_preds_kernel(Batch bt, const pact_report* __restrict__ rep,
                                                          const uint64_t* __restrict__ adj,
                                                          const double* __restrict__ rho, double* __restrict__ rho_opt,
                                                          uint16_t* __restrict__ preds,
                                                          uint2* __restrict__ heads,
                                                          const int32_t* __restrict__ idx,
                                                          int32_t* __restrict__ tie_list,
                                                          int32_t* __restrict__ tie_cnt) {
    __shared__ uint16_t s_nb[4][PREDS_SPREAD];
    const int b = blockIdx.y;
    const Seg sg = bt.s[b];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int TPW = 64 / GL;
    const int pw = (blockIdx.x * 4 + wave) * TPW;          // the wavefront's first token
    const int q = clamp_count(rep[b].n_kept, sg.n);
    if (pw >= q) return;
    const int p = pw + lane / GL < q ? pw + lane / GL : -1, pr = p < 0 ? pw : p;
    const double* r = rho + (size_t)b * bt.n_max;
    const int odd = preds_of_row<true, GL>(p, q, r, adj + ((size_t)b * bt.n_max + pr) * bt.W,
                                           preds + ((size_t)b * bt.n_max + pr) * PRED_CAP,
                                           (uint16_t*)(heads + (size_t)b * bt.n_max + pr), s_nb[wave], lane,
                                           recheck_band2(sg.d_n));
    if ((lane & (GL - 1)) != 0 || p < 0) return;
    if (rho_opt) rho_opt[sg.base + p] = r[p];
    if (odd) {
        // position and token in one word (both below 2^15), so that the re-evaluation finds the
        // token's key without another look-up
        static_assert(PACT_MAX_TOKENS <= 32768, "two 15-bit numbers per list entry");
        const int slot = atomicAdd(&tie_cnt[4 * b], 1);
        if (slot < RHO_RECHECK_MAX) tie_list[(size_t)b * RHO_RECHECK_MAX + slot] = p | (idx[sg.base + p] << 16);
    }
}

// All rounds of the centre selection in one workgroup per sample, statuses in LDS; then the
// centres are numbered in ascending token order and published.
//  * The first round needs no look-ups: nothing is decided yet, so exactly the tokens without a
//    preceding neighbour become centres.  It is folded into the set-up.
//  * The second looks at the predecessors that the token's head names, still in registers: all of them for a token
//    with one to HEAD_PREDS, the densest one and two others for the rest.
//  * From then on there are no rounds: every wavefront looks at its undecided tokens again and again until
//    all are decided, at statuses that the others change meanwhile.  (That ends: of the undecided tokens the first in
//    the order has decided predecessors only, and its wavefront decides it at its next look.  What a token becomes does not
//    depend on when it is looked at.)
//  * Undecided tokens with more than HEAD_PREDS preceding neighbours are dealt out to groups of eight lanes, which keep
//    their records.
//  * Tokens whose list overflowed the record are evaluated from their bitmap row by a whole
//    wavefront.
// Bound by the instructions of one compute unit and chains of dependent accesses: 4010 / 7290 / 16384 kept tokens 12.4 / 24 / 29 us from the kernel's first instruction,
// of which the second look 2.0 / 3.9 / 8.7 and the later ones 2.3 / 7.4 / 2.3 (a comparison and a mask for every predecessor: 14.3 / 30.6 / 36 us).  Rounds between barriers, with work lists of the undecided tokens, took 1.7 us
// each, at least four of them; statuses were read one after the other, a long record by one lane.  (The times are at the kernel.)
// The code is loops rather than unrolled: it runs once, from a cold instruction cache.
// dynamic LDS: rounds_lds below.
// Tokens whose heads are kept in LDS, and whether the token numbers are.
__host__ __device__ inline int lds_heads(int qpad) { return qpad <= 8192 ? qpad : qpad <= 16384 ? 8192 : 4096; }
__host__ __device__ inline bool lds_tokens(int qpad) { return qpad <= 16384; }
static size_t rounds_lds(int n_max, int W) {
    const int qpad = positions(n_max);
    return (size_t)lds_heads(qpad) * 8 + ((size_t)W + 1) * 4 + (size_t)qpad * (lds_tokens(qpad) ? 5 : 3) + 4;
}

struct CentresArgs {
    const char* keys; int32_t dk;
    const int32_t* idx; const double* nn;
    pact_report* rep;
    const uint64_t* adj;
    double* rho; double* rho_opt;
    uint16_t* preds; uint2* heads;
    int32_t* tie_list; int32_t* tie_cnt;
    double* rho_fix;
    uint32_t* status; int32_t* cnum; uint64_t* cmask; int32_t* center_idx;
    int32_t write_rho;                   // whether `rho` itself has to end with the fp64 densities
    const int32_t* idx_ahead;            // idx where it has room for all n tokens; else (a caller's subset: n_kept entries, and that is not known yet) any other list that has
};

// The value again, by another name: what the compiler derives from it stays where it is used, instead of being kept in
// registers across the parts of a kernel that takes all of them (the first version spilled 13).
__device__ __forceinline__ int fresh_v(int v) { asm volatile("" : "+v"(v)); return v; }
__device__ __forceinline__ int fresh_s(int v) { asm volatile("" : "+s"(v)); return v; }

// Counts the workgroup in; what was there before.  Every wavefront waits for its own stores before the barrier: the one that
// counts releases what has reached the L2, and a workgroup barrier alone does not wait for that.
__device__ __forceinline__ void stores_done() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}
__device__ __forceinline__ int count_in(int* counter, int add, int& s_got) {
    stores_done();
    if (threadIdx.x == 0) s_got = __hip_atomic_fetch_add(counter, add, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return lane0_of(s_got);
}

__device__ __forceinline__ void run_rounds(const Batch& bt, const CentresArgs& a, int b, unsigned char* s_raw,
                                           int& s_count, int& s_looks) {
    const Seg sg = bt.s[b];
    const int tid = fresh_v(threadIdx.x);
    const int lane = tid & 63;
    const int wave = tid >> 6;
    pact_report* rep = a.rep;
    const int32_t* ix = a.idx + sg.base;
    const uint2* hd = a.heads + (size_t)b * bt.n_max;
    const int q = clamp_count(rep[b].n_kept, sg.n);
    const int qpad = positions(bt.n_max), Wq = (q + 63) >> 6, n_heads = lds_heads(qpad);
    const bool tok_lds = lds_tokens(qpad);
    typedef __attribute__((address_space(3))) unsigned char lds_u8;
    typedef uint32_t head_t __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) head_t lds_head;
    lds_head* s_head = (lds_head*)s_raw;                         // [n_heads]
    lds_i32* s_wcnt = (lds_i32*)(s_raw + (size_t)n_heads * 8); // [W + 1]
    lds_u16* s_list = (lds_u16*)(s_wcnt + bt.W + 1);                               // [qpad] undecided tokens: short lists from the front, others from the back
    lds_u16* s_ix = s_list + qpad;                               // [qpad] token numbers (tok_lds)
    // [qpad + 1] 1: undecided, 2: centre, 0: not one, as is the position behind the last, which stands for no predecessor: the statuses of several joined by OR say
    // whether one is a centre and whether one is undecided.  (One compute unit does all of this, and is bound by its instructions: with a comparison
    // for each predecessor the second look took 3 us for 4000 tokens, a later one 0.5.)
    lds_vu8* s_st = (lds_vu8*)(tok_lds ? s_ix + qpad : s_ix);
    constexpr unsigned char OPEN = 1, CENTRE = 2, NONE = 0;
    const lds_u8* s_rd = (const lds_u8*)s_st;                    // plain reads: independent look-ups go out together
    const uint4* rec = (const uint4*)(a.preds + (size_t)b * bt.n_max * PRED_CAP);   // 8 pieces per token
    if (tid == 0) { s_count = 0; s_looks = 0; s_st[qpad] = NONE; }
    // a head with the position behind the last in the slots that name nobody
    auto padded = [&](const uint2& v) __attribute__((always_inline)) {
        const uint32_t c = v.x & 0xFFFFu, none = (uint32_t)qpad;
        const uint32_t y = c > 1 ? v.y : none;
        return head_t{c > 0 ? v.x : none << 16, c > 2 ? y : (y & 0xFFFFu) | none << 16};
    };
    // round 1.  (The first heads are requested before the number of kept tokens is known: they lie inside the workspace.  So are the token
    // numbers, and again where the list may end with the last kept one.)
    for (int p0 = 0; p0 < sg.n; p0 += 4096) {
        uint2 hv[4];
        int tok[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) hv[u] = hd[min(p0 + 1024 * u + tid, sg.n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) tok[u] = a.idx_ahead[sg.base + min(p0 + 1024 * u + tid, sg.n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int p = p0 + 1024 * u + tid;
            if (p < q) {
                s_st[p] = (hv[u].x & 0xFFFFu) == 0 ? CENTRE : OPEN;
                if (p < n_heads) s_head[p] = padded(hv[u]);
            }
        }
        if (a.idx_ahead != a.idx) {
#pragma unroll
            for (int u = 0; u < 4; ++u) if (p0 + 1024 * u + tid < q) tok[u] = ix[p0 + 1024 * u + tid];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) if (tok_lds && p0 + 1024 * u + tid < q) s_ix[p0 + 1024 * u + tid] = (uint16_t)tok[u];
        if (p0 + 4096 >= q) break;
    }
    __syncthreads();
    auto head_of = [&](int p) __attribute__((always_inline)) {
        if (p < n_heads) return (head_t)s_head[p];
        return padded(hd[p]);
    };
    // one look at the up to three predecessors that a token's head names
    auto look = [&](head_t hv) __attribute__((always_inline)) {
        return (uint32_t)s_rd[hv.x >> 16] | s_rd[hv.y & 0xFFFFu] | s_rd[hv.y >> 16];
    };
    auto decide = [&](int p, uint32_t seen) __attribute__((always_inline)) {      // whether it stays undecided
        if (seen != OPEN) s_st[p] = seen & CENTRE ? NONE : CENTRE;
        return seen == OPEN;
    };
    // the second, and the two token lists (a wavefront's entries at once)
#pragma unroll 1
    for (int p0 = 0; p0 < q; p0 += 2048) {                       // (wave-uniform trip count)
        head_t hv[2];
        int c[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int p = p0 + 1024 * u + tid;
            hv[u] = head_of(min(p, q - 1));
            c[u] = p < q ? hv[u].x & 0xFFFF : 0;
        }
        if (!__any(c[0] + c[1] > 0)) continue;                   // (centres already, or past the last)
        uint64_t ms[2], ml[2];
        int n = 0;                                               // short ones, long ones << 16
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t seen = look(hv[u]);
            const bool lng = c[u] > HEAD_PREDS && !(seen & CENTRE);
            bool shrt = false;
            if (c[u] > 0 && !lng) shrt = decide(p0 + 1024 * u + tid, seen);
            ms[u] = __ballot(shrt);
            ml[u] = __ballot(lng);
            n += __popcll(ms[u]) + (__popcll(ml[u]) << 16);
        }
        if (n == 0) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_count, n);
        at = lane0_of(at);
        int at_s = at & 0xFFFF, at_l = (int)((uint32_t)at >> 16);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int p = p0 + 1024 * u + tid;
            if ((ms[u] >> lane) & 1ull) s_list[at_s + lanes_below(ms[u], lane)] = (uint16_t)p;
            if ((ml[u] >> lane) & 1ull) s_list[qpad - 1 - (at_l + lanes_below(ml[u], lane))] = (uint16_t)p;
            at_s += __popcll(ms[u]);
            at_l += __popcll(ml[u]);
        }
    }
    __syncthreads();
    const int nshort = s_count & 0xFFFF, nlong = (int)((uint32_t)s_count >> 16);
    // A long list's token, by eight lanes, a 16-byte piece of its record each, in which the position behind the last stands where there is no predecessor.
    // Whether the token stays undecided.
    const int sub = lane & 7;
    auto piece_of = [&](const uint4& v, int c) __attribute__((always_inline)) {      // of the positions 1 .. c
        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
        uint32_t out[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = 8 * sub + 2 * t;
            out[t] = (k >= 1 && k <= c ? wv[t] & 0xFFFFu : (uint32_t)qpad) | (k + 1 <= c ? wv[t] & 0xFFFF0000u : (uint32_t)qpad << 16);
        }
        return make_uint4(out[0], out[1], out[2], out[3]);
    };
    auto look_long = [&](const uint4& v, int p) __attribute__((always_inline)) {
        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
        uint32_t seen = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) seen |= (uint32_t)s_rd[wv[t] & 0xFFFFu] | s_rd[wv[t] >> 16];
        const bool b8 = ((__ballot((seen & CENTRE) != 0) >> (lane & 56)) & 0xFFull) != 0, p8 = ((__ballot((seen & OPEN) != 0) >> (lane & 56)) & 0xFFull) != 0;
        if (p >= 0 && sub == 0) decide(p, b8 ? CENTRE : p8 ? OPEN : NONE);
        return !b8 && p8;
    };
    // A token whose list overflowed the record, by the whole wavefront.
    auto decide_row = [&](int p) __attribute__((always_inline)) {
        const double* r = a.rho + (size_t)b * bt.n_max;
        const double rp = r[p];
        const uint64_t* row = a.adj + ((size_t)b * bt.n_max + p) * bt.W;
        bool blocked = false, pending = false;
        for (int w = lane; w < Wq; w += 64) {
            uint64_t word = row[w];
            while (word) {
                const int bit = __builtin_ctzll(word);
                word &= word - 1;
                const int j = (w << 6) + bit;
                if (j < q && precedes(r[j], j, rp, p)) {
                    const unsigned char sj = s_st[j];
                    blocked |= sj == CENTRE;
                    pending |= sj == OPEN;
                }
            }
        }
        blocked = __any(blocked);
        pending = __any(pending);
        if (lane == 0 && (blocked || !pending)) s_st[p] = blocked ? NONE : CENTRE;
        return !blocked && pending;
    };
    // (tokens are dealt out to all wavefronts)
    const int mine = lane * 16 + wave, mine8 = (lane >> 3) * 16 + wave;
    constexpr int HELD = 4;                                      // long-list tokens a group keeps in its registers
    int sp = -1, lp[HELD];                                       // this thread's short-list token, its group's long-list tokens
    bool over[HELD];                                             // (one whose list overflowed)
    head_t sh = {0, 0};
    uint4 lv[HELD];
#pragma unroll
    for (int k = 0; k < HELD; ++k) {
        lp[k] = -1;
        over[k] = false;
        lv[k] = piece_of(make_uint4(0, 0, 0, 0), 0);             // (no predecessors: a group without a token looks with the others of its wavefront)
        if (mine8 + 128 * k < nlong) {
            lp[k] = s_list[qpad - 1 - (mine8 + 128 * k)];
            lv[k] = rec[(size_t)lp[k] * 8 + sub];
            const int c = head_of(lp[k]).x & 0xFFFF;
            over[k] = c > KP;
            lv[k] = piece_of(lv[k], over[k] ? 0 : c);
        }
    }
    if (mine < nshort) {
        sp = s_list[mine];
        sh = head_of(sp);
    }
    int looks = 2;
    bool more_short = nshort > 1024, more_long = nlong > 128 * HELD;
    auto held = [&]() __attribute__((always_inline)) {
        int any = -1;
#pragma unroll
        for (int k = 0; k < HELD; ++k) any = max(any, lp[k]);
        return any >= 0;
    };
    while (__any(sp >= 0 || held() || more_short || more_long)) {
        asm volatile("" ::: "memory");                           // (the statuses are read again)
        ++looks;
        if (sp >= 0) {
            if (!decide(sp, look(sh))) sp = -1;
        }
        if (more_short) {
            more_short = false;
#pragma unroll 1
            for (int i = tid + 1024; i < nshort; i += 1024) {
                const int p = s_list[i];
                if (s_st[p] != OPEN) continue;
                more_short |= decide(p, look(head_of(p)));
            }
        }
#pragma unroll
        for (int k = 0; k < HELD; ++k) {
            if (__any(lp[k] >= 0)) {
                const bool stays = look_long(lv[k], over[k] ? -1 : lp[k]);
                if (!over[k] && !stays) lp[k] = -1;
                uint64_t mo = __ballot(lp[k] >= 0 && over[k] && sub == 0);
                while (mo) {
                    const int l = __builtin_ctzll(mo);
                    mo &= mo - 1;
                    if (!decide_row(__builtin_amdgcn_readlane(lp[k], l)) && (lane & 56) == l) lp[k] = -1;
                }
            }
        }
        if (__any(more_long)) {                                  // more of them than groups hold
            more_long = false;
#pragma unroll 1
            for (int i0 = 128 * HELD; i0 < nlong; i0 += 128) {          // (wave-uniform trip count)
                const int i = i0 + mine8, p = i < nlong ? s_list[qpad - 1 - i] : 0;
                const bool on = i < nlong && s_st[p] == OPEN;
                if (!__any(on)) continue;
                const uint4 v = rec[(size_t)p * 8 + sub];
                const int c = on ? (int)(head_of(p).x & 0xFFFF) : 0;
                const bool ov = c > KP;
                const bool stays = look_long(piece_of(v, ov ? 0 : c), on && !ov ? p : -1);
                more_long |= on && !ov && stays;
                uint64_t mo = __ballot(ov && sub == 0);
                while (mo) {
                    const int l = __builtin_ctzll(mo);
                    mo &= mo - 1;
                    more_long |= decide_row(__builtin_amdgcn_readlane(p, l));
                }
            }
        }
    }
    if (lane == 0) atomicMax(&s_looks, looks);
    __syncthreads();
    // Publish: one ballot per 64 tokens gives the centre mask word; the centres are numbered in
    // ascending p (= ascending token index) from the running sum of the words' popcounts.
    uint64_t* cm = a.cmask + (size_t)b * bt.W;
#pragma unroll 1
    for (int w = wave; w < Wq; w += 16) {
        const int p = (w << 6) + lane;
        const uint64_t m = __ballot(p < q && s_rd[p] == CENTRE);
        if (lane == 0) { cm[w] = m; s_wcnt[w] = __popcll(m); }
    }
    __syncthreads();
    if (wave == 0) {                                          // exclusive scan over the words
        int run = 0;
        for (int w0 = 0; w0 < Wq; w0 += 64) {
            const int w = w0 + lane;
            const int v = (w < Wq) ? s_wcnt[w] : 0;
            const int inc = wave_scan_incl_i32(v);
            if (w < Wq) s_wcnt[w] = run + inc - v;
            run += lane63_of(inc);
        }
        if (lane == 0) {
            s_wcnt[Wq] = run;
            rep[b].n_centers = run;
            rep[b].rounds = s_looks;
        }
    }
    __syncthreads();
    uint32_t* st = a.status + (size_t)b * bt.n_max;
    int32_t* cn = a.cnum + (size_t)b * bt.n_max;
    int32_t* co = a.center_idx + sg.base;
#pragma unroll 1
    for (int p0 = 0; p0 < q; p0 += 1024) {                       // (64 consecutive positions per wavefront)
        const int p = p0 + tid;
        const bool isc = p < q && s_rd[p] == CENTRE;
        const uint64_t m = __ballot(isc);
        if (p < q) {
            const int c = s_wcnt[p >> 6] + lanes_below(m, lane);
            st[p] = isc ? ST_CENTER : ST_NOT;
            cn[p] = isc ? c : -1;
            if (isc) co[c] = tok_lds ? s_ix[p] : ix[p];
        }
    }
}

// Densities of the listed tokens again, entirely in fp64 (Eq. 5 and Eq. 6 as they are written: dot product, two
// norms, one division, one exponential per pair, the term of the token itself exactly 1).
// A work item is 16 listed tokens x 16 * tiles kept ones.  Wavefront w forms the 16 x 16 dot products with the kept
// tokens of tile w % tiles over the w / tiles-th part of the 64-byte pieces of the rows, on v_mfma_f64_16x16x4_f64: lane l
// supplies row l % 16 of either operand, the l / 16-th 16-byte chunk of the piece, and receives the products of listed
// tokens 4 v + l / 16 with kept token l % 16.  (The order of the summands of a dot product is the same for every pair: equal rows give
// equal dot products.)  The parts meet in LDS; a thread per pair takes them from there.  The next item's first rows are requested
// before that.  Four tiles; two or one where a wavefront would have more than two steps of 32 multiplications (bf16) to
// do and the items are so few that every workgroup still gets at most one (3584-wide rows, 6 listed tokens: 40 -> 25 us) - up to eight steps only if
// they are for three quarters of the workgroups, all of which have to be counted in: 4010 rows of 1 KB with two / eight listed tokens, 126 items instead of 63,
// the launch 20.0 -> 18.4 / 18.9 us, 27 samples of up to 1649 with a few 20.1 -> 17.7; 7586 rows, 238 items, 22.3 -> 23.2; one tile 20.4.
// The sums are exact, hence the same in any order and for any two tokens with the same terms (two tokens at
// equal distances from everything else tie exactly, as they do for a correctly rounded sum, and the index
// decides): every term t in (0, 1] is split into hi = t rounded to a multiple of 2^-30 and lo = t - hi; sums of at
// most 32768 such hi, and of such lo as long as t >= 2^-17 (d_n >= 0.17), fit the 53 bits of an fp64 whatever
// their order, and the density is hi_total + lo_total, rounded once.
__device__ __forceinline__ int items_wanted(int workers, int nchunk, int tiles) { return nchunk * tiles > 8 * 64 ? workers : workers - workers / 4; }
typedef double f64x4_t __attribute__((ext_vector_type(4)));
constexpr int RECHECK_LDS = 4 * 16 * 64 * 8;
template <int DT>
__device__ __forceinline__ void recheck_items(const Batch& bt, const CentresArgs& a, int b, int T, int q, int from, int to,
                                              int tiles, double* s_dot) {
    constexpr int EPL = Elem<DT>::EPL, NBT = 4;
    const Seg sg = bt.s[b];
    const int tid = fresh_v(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const int chunk = 16 * tiles, parts = 16 / tiles;
    const int nch = (q + chunk - 1) / chunk;
    const size_t row_bytes = (size_t)a.dk * Elem<DT>::BYTES;
    const int nchunk = (int)(row_bytes / 16), steps = (nchunk + 4 * parts - 1) / (4 * parts);
    const char* kb = a.keys + (size_t)sg.base * row_bytes;
    const double* nnb = a.nn + sg.base;
    const int32_t* ix = a.idx + sg.base;
    const int32_t* list = a.tie_list + (size_t)b * RHO_RECHECK_MAX;
    double* part_b = a.rho_fix + (size_t)b * 2 * rho_fix_tokens(bt.n_max) * rho_fix_chunks(bt.n_max);   // [T][nch][2]
    const double d_n = (double)sg.d_n;
    const int i16 = lane & 15, kq = lane >> 4, part = wave / tiles, tile = wave - part * tiles;
    // this thread's rows of the products, and its pair of the second half (none beyond 16 x chunk threads)
    const int te = tid / chunk, ke = tid - te * chunk;
    int tokA, tokB, ent_end, tok_end;
    auto tokens_of = [&](int item) __attribute__((always_inline)) {
        const int rt = item / nch, c = item - rt * nch;
        tokA = list[min(rt * 16 + i16, T - 1)] >> 16;
        tokB = ix[min(c * chunk + tile * 16 + i16, q - 1)];
        ent_end = list[min(rt * 16 + te, T - 1)];
        tok_end = ix[min(c * chunk + ke, q - 1)];
    };
    uint4 va[NBT], vb[NBT];
    const char *ra, *rb;
    auto fetch = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NBT; ++u) {
            const size_t o = (size_t)min(((s0 + u) * parts + part) * 4 + kq, nchunk - 1) * 16;
            va[u] = *(const uint4*)(ra + o);
            vb[u] = *(const uint4*)(rb + o);
        }
    };
    auto begin = [&]() __attribute__((always_inline)) {
        ra = kb + (size_t)min(max(tokA, 0), sg.n - 1) * row_bytes;
        rb = kb + (size_t)tokB * row_bytes;
        fetch(0);
    };
    tokens_of(from);
    begin();
    for (int item = from; item < to; ++item) {
        const int rt = item / nch, c = item - rt * nch;
        const int t_end = rt * 16 + te, pk_end = c * chunk + ke, p_end = ent_end & 0xFFFF;
        const double nnA = nnb[min(max(ent_end >> 16, 0), sg.n - 1)], nnB = nnb[tok_end];
        if (item + 1 < to) tokens_of(item + 1);
        f64x4_t acc = {0.0, 0.0, 0.0, 0.0};                 // (four wavefronts share a matrix unit)
#pragma unroll 1
        for (int s0 = 0; s0 < steps; s0 += NBT) {
#pragma unroll
            for (int u = 0; u < NBT; ++u) {
                if (s0 + u < steps) {                       // (uniform)
                    if (((s0 + u) * parts + part) * 4 + kq >= nchunk) va[u] = vb[u] = make_uint4(0, 0, 0, 0);
                    double x[8], y[8];
                    Elem<DT>::widen(va[u], x);
                    Elem<DT>::widen(vb[u], y);
#pragma unroll
                    for (int e = 0; e < EPL; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[e], y[e], acc, 0, 0, 0);
                }
            }
            if (s0 + NBT < steps) fetch(s0 + NBT);
        }
        if (item + 1 < to) begin();
        __syncthreads();                                    // (the previous item's products have been read)
#pragma unroll
        for (int v = 0; v < 4; ++v) s_dot[(part * 16 + 4 * v + kq) * chunk + tile * 16 + i16] = acc[v];
        __syncthreads();
        if (tid < 16 * chunk) {                             // (whole wavefronts)
            double dot = 0.0;
            for (int k = 0; k < parts; ++k) dot += s_dot[k * 16 * chunk + tid];
            const double d = cos_dist64(dot, nnA, nnB);
            const double term = pk_end >= q ? 0.0 : (pk_end == min(p_end, q - 1) ? 1.0 : exp(-d / d_n));
            const double hi = rint(term * 1073741824.0) * (1.0 / 1073741824.0);
            const double vh = group_sum_f64(hi, chunk), vl = group_sum_f64(term - hi, chunk);
            if (ke == 0 && t_end < T) *(double2*)(part_b + ((size_t)t_end * nch + c) * 2) = make_double2(vh, vl);
        }
    }
}

// The fp64 densities of the listed tokens from their partial sums, and what they change: ORDER_PAIRS where two listed
// neighbours change their order, ORDER_BAND where a listed token moves by more than the band.  A neighbour that is not listed
// is further away than the band at the larger of the two densities, hence on the same side of a token that moves by no more than the
// band at its own: without ORDER_BAND only pairs of listed tokens can change.  With it any list of the sample may be out of date; a
// list that still names a neighbour which by now follows the token would let the two wait for each other for good.  (The band is
// a statistical bound, and tokens that are nearly all alike pass it: their terms share the rounding of the
// token's reciprocal norm.)  The densities are left in front of the partial sums.
enum { ORDER_PAIRS = 2, ORDER_BAND = 8 };
__device__ __forceinline__ int order_changed(const Batch& bt, const CentresArgs& a, int b, int T, int q, int tiles,
                                              unsigned char* s_raw, int* s_flag) {
    const Seg sg = bt.s[b];
    const int tid = fresh_v(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    double* s_new = (double*)s_raw;
    double* s_old = s_new + RHO_RECHECK_MAX;
    int* s_pos = (int*)(s_old + RHO_RECHECK_MAX);
    const int32_t* list = a.tie_list + (size_t)b * RHO_RECHECK_MAX;
    double* part_b = a.rho_fix + (size_t)b * 2 * rho_fix_tokens(bt.n_max) * rho_fix_chunks(bt.n_max);
    const double* rho_b = a.rho + (size_t)b * bt.n_max;
    const uint64_t* adj_b = a.adj + (size_t)b * bt.n_max * bt.W;
    const int nch = (q + 16 * tiles - 1) / (16 * tiles);
    static_assert(RHO_RECHECK_MAX <= 1024, "a listed token per thread");
    __syncthreads();
    if (tid == 0) s_flag[0] = s_flag[1] = fresh_v(0);
    if (tid < T) {
        const int p = min(list[tid] & 0xFFFF, q - 1);
        s_pos[tid] = p;
        s_old[tid] = rho_b[p];
    }
    for (int t0 = 0; t0 < T; t0 += 64) {                // 16 lanes per token
        const int t = t0 + wave * 4 + (lane >> 4);
        double ah = 0.0, al = 0.0;
        if (t < T) {
            for (int c = lane & 15; c < nch; c += 128) {
                double2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    v[u] = c + 16 * u < nch ? *(const double2*)(part_b + ((size_t)t * nch + c + 16 * u) * 2) : make_double2(0.0, 0.0);
#pragma unroll
                for (int u = 0; u < 8; ++u) { ah += v[u].x; al += v[u].y; }
            }
        }
        const double acc = group_sum_f64(ah, 16) + group_sum_f64(al, 16);
        if (t < T && (lane & 15) == 0) s_new[t] = acc;
    }
    __syncthreads();
    bool changed = false, far = false;
    int fine = 0;
    if (tid < T) {
        const double d = s_new[tid] - s_old[tid];
        far = !(d * d <= recheck_band2(sg.d_n) * s_old[tid]);           // (the comparison that lists tokens)
    }
    constexpr int UN = 4;
    for (int e0 = tid; e0 < T * T; e0 += 1024 * UN) {
        int i[UN], j[UN];
        uint64_t word[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int e = min(e0 + 1024 * u, T * T - 1);
            i[u] = e / T;
            j[u] = e - i[u] * T;
            word[u] = adj_b[(size_t)s_pos[i[u]] * bt.W + (s_pos[j[u]] >> 6)];
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int pi = s_pos[i[u]], pj = s_pos[j[u]];
            if (e0 + 1024 * u >= T * T || pj >= pi || !((word[u] >> (pj & 63)) & 1ull)) continue;
            const double ni = s_new[i[u]], nj = s_new[j[u]], d = nj - ni;
            changed |= precedes(nj, pj, ni, pi) != precedes(s_old[j[u]], pj, s_old[i[u]], pi);
            fine += d != 0.0 && fabs(d) <= 1e-11 * (nj + ni);
        }
    }
    if (changed) atomicOr(&s_flag[0], (int)ORDER_PAIRS);
    if (far) atomicOr(&s_flag[0], (int)ORDER_BAND);
    if (fine) atomicAdd(&s_flag[1], fine);
    if (tid < T) {
        part_b[tid] = s_new[tid];
        if (a.rho_opt) a.rho_opt[sg.base + s_pos[tid]] = s_new[tid];
    }
    __syncthreads();
    if (tid == 0) {
        if (s_flag[1]) atomicAdd(&a.rep[b].rho_near_ties, s_flag[1]);
        a.rep[b].rho_rechecked = T;
    }
    return lane0_of(s_flag[0]);
}

// The fp64 densities take their places; the predecessor lists are made again from them: those of the listed tokens, or all of
// the sample's (`changed`: what order_changed found).
__device__ __forceinline__ void replace_densities(const Batch& bt, const CentresArgs& a, int b, int T, int q, int changed,
                                                  uint16_t* s_nb) {
    const int tid = fresh_v(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const int32_t* list = a.tie_list + (size_t)b * RHO_RECHECK_MAX;
    const double* part_b = a.rho_fix + (size_t)b * 2 * rho_fix_tokens(bt.n_max) * rho_fix_chunks(bt.n_max);
    double* rho_b = a.rho + (size_t)b * bt.n_max;
    __syncthreads();
    if (tid < T) rho_b[min(list[tid] & 0xFFFF, q - 1)] = part_b[tid];
    __syncthreads();                                   // (the values are read back by this workgroup only)
    if (!changed) return;
    const bool all = (changed & ORDER_BAND) != 0;
    const int n_lists = all ? q : T;
    for (int t = wave; t < n_lists; t += 16) {
        const int p = all ? t : min(list[t] & 0xFFFF, q - 1);
        preds_of_row<false, 64>(p, q, rho_b, a.adj + ((size_t)b * bt.n_max + p) * bt.W, a.preds + ((size_t)b * bt.n_max + p) * PRED_CAP,
                                (uint16_t*)(a.heads + (size_t)b * bt.n_max + p), s_nb + wave * PREDS_SPREAD, lane, 0.0);
    }
    __syncthreads();
}

// Centre rounds and fp64 densities side by side: workgroup b < B runs the rounds of sample b in the order of the
// densities that it finds; the others share out the batch's work items of listed tokens, and the one that
// finishes a sample's last item looks whether two neighbours change their order.  They hardly ever do (the band that lists tokens is
// twenty and more standard errors wide); if so, the later of that workgroup and the sample's first one puts the fp64
// densities in place and runs the rounds again.  Nobody waits for anybody: counters say who is last.
// As two launches, rounds with barriers after the re-evaluation (event brackets, of which either launch has 2.5 us): 4010-token
// image 29 -> 20 us, 8 videos of 3450 tokens 48 -> 42 us, 16 ragged images 34 -> 21 us, 7290 rows of 7 KB 96 -> 36 us, 16384 tokens with fp32
// keys 151 -> 77 us (the fp64 products of 70 listed tokens).  Bound by the selection of a sample on one CU, and where tokens are listed by their chain
// (an image with two: first rows at 4 us, the products of an item 2, counted in at 12.7, looked at 15, 15.9), for the videos and the long
// rows by the products themselves (four wavefronts per SIMD, 9 us an item of four tiles).
// tie_cnt[4b]: listed tokens; [4b + 1]: work items done; [4b + 2]: 1 looked at, ORDER_PAIRS, ORDER_BAND, 4 rounds run.
// grid (B + workers), block 1024, dynamic LDS: what run_rounds takes, at least RECHECK_LDS.
template <int DT>
__global__ __launch_bounds__(1024) void centres_kernel(Batch bt, CentresArgs a) {
    extern __shared__ double s_dyn[];
    __shared__ int s_flag[2], s_count, s_looks, s_got, s_tiles;
    __shared__ int s_T[PACT_MAX_BATCH], s_q[PACT_MAX_BATCH], s_items[PACT_MAX_BATCH + 1];
    static_assert(PACT_MAX_BATCH <= 64, "a sample per lane");
    const bool resolver = (int)blockIdx.x < bt.B;
    int item = 0, item_end = 0, b = blockIdx.x, T = 0, q = 0, tiles = 4;
    if (!resolver) {
        const int workers = gridDim.x - bt.B;
        if (threadIdx.x < 64) {
            const int k = threadIdx.x;
            int Tk = 0, qk = 0;
            if (k < bt.B) {
                Tk = a.tie_cnt[4 * k];
                qk = clamp_count(a.rep[k].n_kept, bt.s[k].n);
                s_T[k] = Tk;
                s_q[k] = qk;
                if (Tk > RHO_RECHECK_MAX) Tk = 0;
            }
            // tiles of kept tokens per item; the room for partial sums is that of four tiles, for the most listed tokens
            const int nchunk = a.dk * Elem<DT>::BYTES / 16;
            int tiles = 4, inc = wave_scan_incl_i32(((Tk + 15) >> 4) * ((qk + 63) >> 6));
            while (tiles > 1 && nchunk * tiles > 2 * 64) {
                const int half = 8 * tiles, inc2 = wave_scan_incl_i32(((Tk + 15) >> 4) * ((qk + half - 1) / half));
                if (lane63_of(inc2) > items_wanted(workers, nchunk, tiles) || __any(Tk * (64 / half) > rho_fix_tokens(bt.n_max))) break;
                tiles >>= 1;
                inc = inc2;
            }
            s_items[k + 1] = inc;
            if (k == 0) { s_items[0] = 0; s_tiles = tiles; }
        }
        __syncthreads();
        tiles = lane0_of(s_tiles);
        const int total = lane0_of(s_items[bt.B]), w = (int)blockIdx.x - bt.B;
        item = (int)((long)total * w / workers);
        item_end = (int)((long)total * (w + 1) / workers);
        b = 0;
    }
    auto meet = [&](int* counter, int add) __attribute__((always_inline)) { return count_in(counter, add, s_got); };
    bool again = false;
    int changed = 0;
    while (true) {
        if (!resolver) {
            if (item >= item_end) return;
            while (item >= lane0_of(s_items[b + 1])) ++b;
            const int from = lane0_of(s_items[b]), next = lane0_of(s_items[b + 1]), to = min(item_end, next), all = next - from, mine = to - item;
            T = lane0_of(s_T[b]);
            q = lane0_of(s_q[b]);
            recheck_items<DT>(bt, a, fresh_s(b), fresh_s(T), fresh_s(q), fresh_s(item - from), fresh_s(to - from), tiles, s_dyn);
            item = to;
            if (meet(&a.tie_cnt[4 * b + 1], mine) != all - mine) continue;
            changed = order_changed(bt, a, fresh_s(b), fresh_s(T), fresh_s(q), tiles, (unsigned char*)s_dyn, s_flag);
            if (!(meet(&a.tie_cnt[4 * b + 2], changed | 1) & 4)) continue;        // the rounds still run
            again = changed || a.write_rho;
            if (!again) continue;
        }
        const int bs = fresh_s(b);
        if (again) replace_densities(bt, a, bs, T, q, changed, (uint16_t*)s_dyn);
        if (!again || changed) run_rounds(bt, a, bs, (unsigned char*)s_dyn, s_count, s_looks);
        if (!resolver) continue;
        if (again) return;
        T = a.tie_cnt[4 * bs];
        if (T <= 0) return;
        if (T > RHO_RECHECK_MAX) {
            if (threadIdx.x == 0) atomicOr(&a.rep[bs].refine_overflow, OVERFLOW_RHO_RECHECK);
            return;
        }
        q = clamp_count(a.rep[bs].n_kept, bt.s[bs].n);
        const int seen = meet(&a.tie_cnt[4 * bs + 2], 4);
        if (!(seen & 1)) return;                       // that workgroup will find the rounds run
        changed = seen & (ORDER_PAIRS | ORDER_BAND);
        again = changed || a.write_rho;
        if (!again) return;
    }
}

// ------------------------------------------------------------------------------------------
// Samples of at most SMALL_TOKENS: settling, order and selection in one launch.  One workgroup per sample, the sample's bitmap in LDS
// (1024 tokens: 139 KB, rows an odd number of words apart):
//  1. the undecided pairs are evaluated as settle_kernel does it, by groups of lanes that hold a row in one 16-byte chunk each (wide rows: by
//     settle_kernel, ahead); bits are cleared in LDS, and in memory, where the assignment reads them;
//  2. one to eight threads per kept token go through the set bits of its row, 32 at a time, and leave those of preceding neighbours.
//     Densities are compared in fp32 where that decides, near-ties are listed;
//  3. a thread per token, every wavefront looks at its undecided tokens until none is left.  Its 64 tokens are one word of the masks of
//     centres and of undecided tokens, so it alone writes that word, centres ahead of undecided; whoever reads the other
//     way round never misses a centre.  Two words of predecessors are in registers.
// Listed tokens (a tenth of the samples have two; all where tokens are copies of each other): their fp64 densities are work items that the
// launch's other workgroups wait for and take by ticket, and so does the sample's own workgroup once its selection is
// through: a worker's wait is bounded, and without workers the items are done all the same.  What follows from them is
// as in centres_kernel.  Of many items (128 and more: tokens nearly all copies) four are a ticket (32 samples of 729 copies of 5 tokens 681 -> 620 us).
// Waiting workers keep 1024 threads each and the launch's LDS from other streams for the 7 us to the lists.  So there is one per 32 tokens, or
// where that is more than 96, as many as do the items of two listed tokens in each sample in one turn, 96 at least.  With one per 32 tokens -> these -> the
// three launches of larger samples, calls alone (some samples with two listed tokens) / 40 copies of 256 MB on another stream beside 50 calls: 8 of 729 tokens 82.5 ->
// 82.1 -> 84.5 us / 5.4 -> 4.7 -> 4.5 ms, 16: 94.6 -> 93.7 -> 95.7 / 5.7 -> 4.8 -> 4.8, 32: 118.7 -> 118.7 -> 121.6 / 5.1 -> 5.0 -> 4.7 (128 workers: 8 of 729
// 5.4).  Workers that went on to other samples were no faster with 96 of them for 32 samples (119.0 -> 121).
// Bound by its chain: arguments, one trip for everything, one for the undecided pairs' rows (3 + 1.4 us), then instructions of few wavefronts (lists
// 2 to 3, selection 2 us).  The three launches of larger samples were mostly their beginnings and ends; event brackets: one frame of 196
// tokens 5.5 + 7.5 + 10.9 -> 12.7 us, a crop of 729 with fp32 keys 6 + 7 + 9.6 -> 14.8, 32 crops 7.3 + 8.6 + 16.4 -> 25 (ten of which are the listed tokens').
// tie_cnt[4b + 1]: work items done; [4b + 2]: as in centres_kernel; [4b + 3]: tickets taken | listed tokens << 16 | READY.
constexpr int SMALL_TOKENS = 1024, SMALL_READY = 1 << 30, SMALL_POLLS = 1 << 12, SMALL_WORKERS = 96;
struct SmallArgs {
    const uint32_t* near_list; const int32_t* near_cnt;          // near_list == nullptr: settle_kernel has run
    const uint32_t* far_bits; int32_t far_words;
    const double* rho_lo;
};
// Rows of more than 512 bytes are left to settle_kernel: one compute unit would fetch them for 5 us and more (835 tokens, fp32 keys 512
// wide, 158 pairs: event bracket 30 us).
constexpr int SMALL_SETTLE_CHUNKS = 32;
// Where one launch is the faster way: up to 512 kept tokens, and where settle_kernel has to come first up to 256 of a single sample.  Settling to
// selection, brackets without their 2.5 us a launch, three launches -> here, nothing listed / two tokens listed in a sample: width
// 128, images of 160 tokens 15.8 / - -> 9.0 / -, 300: 16.2 -> 11.4, 729: 16.6 / 20.1 -> 14.0 / 21.2, 1000 (550 kept): 17.2 -> 19.7; 8 of 300 18.3 / 21.2 -> 11.6 /
// 19; 8 of 729 18.3 / 21 -> 14.7 / 23; 32 of 729 25 -> 23; width 512: 160: 14.0 -> 11.0, 300: 15.5 / 23.3 -> 12.8 / 25.2, 729: 15.2 / 24.4 -> 14.8 / 27.2,
// 8 of 729 - / 24.5 -> - / 28.5.  A tenth of the samples have listed tokens; whole calls, with none / with some: 729 tokens 61.3 / 66.5 -> 57.5 / 67.2, 2 of 729
// 65.0 / 69.1 -> 60.3 / 69.8, 4: 69.7 / 71.9 -> 65.0 / 72.8, 8: 83.7 / 84.8 -> 77.8 / 82.9, 16: 95.3 / 97.4 -> 89.6 / 95.3, 32: - / 123.6 -> - / 120.7; 8 of 300 68.2 / 72.7 ->
// 61.2 / 70.1: where listed tokens are, up to four samples lose 1 us, against 4 to 5 won where none are.
static bool selects_in_one(const Batch& bt, bool settle_there) {
    if (bt.n_max > SMALL_TOKENS || (!settle_there && bt.B > 1)) return false;
    for (int b = 0; b < bt.B; ++b)
        if (bt.s[b].n - prune_rank(bt.s[b].lambda, bt.s[b].n) > (settle_there ? 512 : 256)) return false;
    return true;
}
static size_t small_lds(int W) { return (size_t)W * 64 * (((W | 1) + 1) * sizeof(uint64_t) + sizeof(float)); }

typedef __attribute__((address_space(3))) uint64_t lds_u64;
typedef __attribute__((address_space(3))) volatile uint64_t lds_vu64;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) double lds_f64;
struct SmallShared {
    uint64_t centre[16], open[16], odd[16];  // masks of centres, of undecided tokens, of tokens with a near-tie
    uint32_t far[16];
    int looks, near_ties, got;
    int flag[2];
    uint16_t tok[SMALL_TOKENS];
};

// The selection of sample b.  first: with the settling and the list of near-ties; otherwise on the bitmap and the densities as they
// are by now.  Returns the number of listed tokens (first).
template <int DT>
__device__ __forceinline__ int select_sample(const Batch& bt, const CentresArgs& a, const SmallArgs& sa, int b, bool first,
                                             unsigned char* s_raw, SmallShared& sh) {
    const Seg sg = bt.s[b];
    const int tid = fresh_v(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = bt.W, pitch = W | 1;
    lds_u64* s_row = (lds_u64*)s_raw;                            // [64 W][pitch]
    lds_f64* s_rho = (lds_f64*)(s_row + (size_t)W * 64 * pitch); // [64 W]
    lds_f32* s_rho32 = (lds_f32*)(s_rho + (size_t)W * 64);       // [64 W]
    pact_report* rep = a.rep + b;
    uint64_t* adj = (uint64_t*)a.adj + (size_t)b * bt.n_max * W;
    double* rho = a.rho + (size_t)b * bt.n_max;
    const int32_t* ix = a.idx + sg.base;
    const double* nnb = a.nn + sg.base;
    constexpr int U = 2;                                         // pairs in flight per group of lanes
    const bool settle = first && sa.near_list != nullptr;
    const int nchunk = a.dk * Elem<DT>::BYTES / 16;              // (settle: SMALL_SETTLE_CHUNKS at most)
    const int lpp = nchunk <= 16 ? 16 : 32, ng = 1024 / lpp, g = tid / lpp, gl = tid & (lpp - 1);
    const uint2* pairs = (const uint2*)(sa.near_list + (size_t)b * NEAR_CAP * 2);
    // ---- everything whose address depends on the thread's position only goes out before the first count is read
    const int pc = min(tid, sg.n - 1), r0 = tid >> 4, w0 = tid & 15;
    int tok = a.idx_ahead[sg.base + pc];
    double r = rho[pc];
    const bool split = settle && sg.d_n < EXACT_SUMS_D_N;         // densities that came in two parts (add_density)
    const double r_lo = split ? sa.rho_lo[(size_t)b * bt.n_max + pc] : 0.0;
    uint64_t word[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) word[k] = r0 + 64 * k < sg.n && w0 < W ? adj[(size_t)(r0 + 64 * k) * W + w0] : 0ull;
    uint2 pr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) pr[u] = settle ? pairs[u * ng + g] : make_uint2(0, 0);      // (garbage beyond the count, never used)
    static_assert(SMALL_TOKENS <= 1024, "one part (near_parts)");
    const uint32_t raw = settle ? (uint32_t)sa.near_cnt[b * NEAR_PARTS * NEAR_COUNTER] : 0u;
    const int checked = settle ? sa.near_cnt[b * NEAR_PARTS * NEAR_COUNTER + 1] : 0;
    const int q = clamp_count(rep->n_kept, sg.n), Wq = (q + 63) >> 6;
    const int cnt = (int)min(raw, (uint32_t)NEAR_CAP);
    if (a.idx_ahead != a.idx && tid < q) tok = ix[tid];
    if (settle && sa.far_words > 0) {
        uint32_t fb = 0u;                                        // (see settle_kernel)
        for (int k = tid; k < sa.far_words; k += 1024) fb = max(fb, sa.far_bits[(size_t)b * sa.far_words + k]);
#pragma unroll
        for (int sft = 32; sft >= 1; sft >>= 1) fb = max(fb, (uint32_t)__shfl_xor((int)fb, sft, 64));
        if (lane == 0) sh.far[wave] = fb;
    }
    if (split) {
        r += r_lo;
        if (tid < q) rho[tid] = r;
    }
    __syncthreads();                                             // (again: the LDS of before is free)
    if (tid == 0) { sh.looks = 0; sh.near_ties = 0; }
    if (tid < 16) sh.odd[tid] = 0ull;
    sh.tok[tid] = (uint16_t)tok;
    if (tid < 64 * W) { s_rho[tid] = r; s_rho32[tid] = (float)r; }
    const uint64_t last = q & 63 ? (1ull << (q & 63)) - 1ull : ~0ull;
    auto put = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int row = r0 + 64 * (k0 + k);
            if (row < q && w0 < Wq) s_row[row * pitch + w0] = w0 == Wq - 1 ? word[k] & last : word[k];
        }
    };
    put(0);
    if (q > 512) {
#pragma unroll
        for (int k = 0; k < 8; ++k) word[k] = r0 + 64 * (k + 8) < q && w0 < W ? adj[(size_t)(r0 + 64 * (k + 8)) * W + w0] : 0ull;
        put(8);
    }
    __syncthreads();
    // ---- 1. the pairs that fp32 could not decide (the order of operations of wave_dot64)
    if (cnt > 0) {
        constexpr int EPL = Elem<DT>::EPL;
        const char* kb = a.keys + (size_t)sg.base * ((size_t)nchunk * 16);
        const double d_c = (double)sg.d_c;
        auto clear = [&](int i, int j) __attribute__((always_inline)) {
            __hip_atomic_fetch_and((lds_u32*)(s_row + i * pitch) + (j >> 5), ~(1u << (j & 31)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            atomicAnd((unsigned long long*)&adj[(size_t)i * W + (j >> 6)], ~(1ull << (j & 63)));
        };
#pragma unroll 1
        for (int e0 = 0; e0 < cnt; e0 += ng * U) {               // (uniform)
            const char *ri[U], *rj[U];
            double acc[U], ni[U], nj[U];
            const bool two = e0 + ng < cnt;                      // (uniform) whether any group has a second pair
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * ng + g;
                if (e0 > 0) pr[u] = pairs[min(e, cnt - 1)];
                if (e >= cnt) pr[u] = make_uint2(0, 0);
                const int ti = sh.tok[min((int)(pr[u].x & ~NEAR_MIRROR), q - 1)], tj = sh.tok[min((int)pr[u].y, q - 1)];
                ri[u] = kb + (size_t)ti * nchunk * 16;
                rj[u] = kb + (size_t)tj * nchunk * 16;
                ni[u] = nnb[ti];
                nj[u] = nnb[tj];
                acc[u] = 0.0;
            }
            uint4 va[U], vb[U];
            const size_t o = (size_t)min(gl, nchunk - 1) * 16;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u > 0 && !two) break;
                va[u] = *(const uint4*)(ri[u] + o);
                vb[u] = *(const uint4*)(rj[u] + o);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u > 0 && !two) break;
                if (gl < nchunk) {
                    double x[8], y[8];
                    Elem<DT>::widen(va[u], x);
                    Elem<DT>::widen(vb[u], y);
#pragma unroll
                    for (int i = 0; i < EPL; ++i) acc[u] = fma(x[i], y[i], acc[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u > 0 && !two) break;
                const int pi = (int)(pr[u].x & ~NEAR_MIRROR), pj = (int)pr[u].y;
                const bool both = (pr[u].x & NEAR_MIRROR) != 0;
                const double dot = group_sum_f64(acc[u], lpp);
                const double d = pi != pj ? cos_dist64(dot, ni[u], nj[u]) : 0.0;
                if (gl == 0 && e0 + u * ng + g < cnt && pi < q && pj < q) {
                    if (beyond_cutoff(d, d_c)) {
                        clear(pi, pj);
                        if (both) clear(pj, pi);
                    }
                    if (const int ties = near_ties_of(d, d_c, both)) atomicAdd(&sh.near_ties, ties);
                }
            }
        }
        __syncthreads();
    }
    // ---- 2. the bits of preceding neighbours, in the place of the row's.  GL threads per token, every GL-th half word each
    {
        const int gsh = q <= 128 ? 3 : q <= 256 ? 2 : q <= 512 ? 1 : 0;
        const int p = tid >> gsh;
        if (p < q) {
            lds_u32* half = (lds_u32*)(s_row + p * pitch);
            const float fp = s_rho32[p];
            // a difference of the fp32 densities beyond `far` is one of the fp64 ones, and beyond the band c sqrt(rj) of the larger
            // density rj (inside it sqrt(rj) <= sqrt(rp) + c); the roundings to fp32 are 2^-23 of the larger density
            const float c = 0x1p-20f * (1.0f + 4.0f * 1.4426950f / sg.d_n), w = c * __builtin_amdgcn_sqrtf(fp) + c * c;
            const float far = 1.001f * (w + 0x1p-21f * (fp + w));
            bool odd = false;
#pragma unroll 1
            for (int h = tid & ((1 << gsh) - 1); h < 2 * Wq; h += 1 << gsh) {
                const uint32_t has = half[h], others = h == p >> 5 ? has & ~(1u << (p & 31)) : has;
                uint32_t pre = 0u;
                bool near = false;
#pragma unroll 1
                for (uint32_t bits = others; bits; bits &= bits - 1) {
                    const int k = __builtin_ctz(bits);
                    const float d = s_rho32[32 * h + k] - fp;
                    pre |= (d > far ? 1u : 0u) << k;
                    near |= !(fabsf(d) > far);
                }
                if (near) {                                      // again, in fp64
                    const double rp = s_rho[p], band2 = recheck_band2(sg.d_n);
                    pre = 0u;
#pragma unroll 1
                    for (uint32_t bits = others; bits; bits &= bits - 1) {
                        const int k = __builtin_ctz(bits), j = 32 * h + k;
                        const double x = s_rho[j], d = x - rp;
                        pre |= (precedes(x, j, rp, p) ? 1u : 0u) << k;
                        odd |= d * d <= band2 * fmax(x, rp);
                    }
                }
                if (has) half[h] = pre;
            }
            if (first && odd) atomicOr((unsigned long long*)&sh.odd[p >> 6], 1ull << (p & 63));
        }
    }
    __syncthreads();
    const bool on = tid < q;
    int listed = 0;
    if (first) {
        if (on && a.rho_opt) a.rho_opt[sg.base + tid] = r;
        const int pop = lane < 16 ? __popcll(sh.odd[lane]) : 0, inc = wave_scan_incl_i32(pop);
        listed = __builtin_amdgcn_readlane(inc, 15);
        const int at = __builtin_amdgcn_readlane(inc - pop, wave);           // (ahead of the branch: all lanes have to take part)
        if (listed) {
            static_assert(SMALL_TOKENS <= RHO_RECHECK_MAX && PACT_MAX_TOKENS <= 32768, "all may be listed; two 15-bit numbers per entry");
            const uint64_t odd = sh.odd[wave];
            if ((odd >> lane) & 1ull)
                a.tie_list[(size_t)b * RHO_RECHECK_MAX + at + lanes_below(odd, lane)] = tid | (tok << 16);
            stores_done();                                       // (the list, the bits and the densities are to be where the workers look for them)
        }
        if (tid == 1023) {                                       // (of the wavefront that has a selection of its own least often)
            __hip_atomic_fetch_add(&a.tie_cnt[4 * b + 3], SMALL_READY | (listed << 16), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            if (settle) {
                rep->dc_near_ties = sh.near_ties;
                uint32_t fb = 0u;
                if (sa.far_words > 0)
                    for (int k = 0; k < 16; ++k) fb = max(fb, sh.far[k]);
                report_settled(rep, raw > (uint32_t)NEAR_CAP, checked, fb, sg.d_n);
            }
        }
    }
    // ---- 3. the selection.  Two words of predecessors in registers, others from LDS
    const lds_u64* mine = s_row + tid * pitch;
    uint32_t left = 0u;
    if (on) {
#pragma unroll 4
        for (int w = 0; w < Wq; ++w) left |= (mine[w] != 0ull ? 1u : 0u) << w;
    }
    uint64_t m[2];
    int wn[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        wn[k] = left ? __builtin_ctz(left) : 0;
        m[k] = left ? mine[wn[k]] : 0ull;
        left &= left - 1 + (left == 0u);
    }
    lds_vu64* s_centre = (lds_vu64*)sh.centre;
    lds_vu64* s_open = (lds_vu64*)sh.open;
    uint64_t open = __ballot(on), centre = 0ull;
    if (lane == 0) { s_open[wave] = open; s_centre[wave] = 0ull; }
    __syncthreads();
    bool todo = on;
    int looks = 0;
    while (open) {                                               // (the same in all lanes)
        ++looks;
        bool blocked = false, pending = false;
        if (todo) {
            uint64_t o = 0ull, c = 0ull;
#pragma unroll
            for (int k = 0; k < 2; ++k) o |= s_open[wn[k]] & m[k];
            for (uint32_t rest = left; rest; rest &= rest - 1) { const int w = __builtin_ctz(rest); o |= s_open[w] & mine[w]; }
#pragma unroll
            for (int k = 0; k < 2; ++k) c |= s_centre[wn[k]] & m[k];
            for (uint32_t rest = left; rest; rest &= rest - 1) { const int w = __builtin_ctz(rest); c |= s_centre[w] & mine[w]; }
            blocked = c != 0ull;
            pending = o != 0ull;
        }
        const uint64_t up = __ballot(todo && !blocked && !pending), down = __ballot(todo && blocked);
        if (up | down) {
            centre |= up;
            open &= ~(up | down);
            if (lane == 0) { s_centre[wave] = centre; s_open[wave] = open; }     // (in this order)
            todo = todo && !blocked && pending;
        }
    }
    if (lane == 0) atomicMax(&sh.looks, looks);
    __syncthreads();
    // ---- the centres, numbered in ascending token order
    const int pop = lane < 16 ? __popcll(s_centre[lane]) : 0, inc = wave_scan_incl_i32(pop);
    const int before = __builtin_amdgcn_readlane(inc - pop, wave), n_centres = __builtin_amdgcn_readlane(inc, 15);
    if (lane == 0 && wave < Wq) a.cmask[(size_t)b * W + wave] = centre;
    if (on) {
        const bool isc = (centre >> lane) & 1ull;
        const int c = before + lanes_below(centre, lane);
        a.status[(size_t)b * bt.n_max + tid] = isc ? ST_CENTER : ST_NOT;
        a.cnum[(size_t)b * bt.n_max + tid] = isc ? c : -1;
        if (isc) a.center_idx[sg.base + c] = tok;
    }
    if (tid == 0) {
        rep->n_centers = n_centres;
        rep->rounds = sh.looks;
    }
    return listed;
}

// grid (B + workers), block 1024, dynamic LDS: small_lds, at least RECHECK_LDS.
template <int DT>
__global__ __launch_bounds__(1024) void select_small_kernel(Batch bt, CentresArgs a, SmallArgs sa) {
    touch_args<sizeof(CentresArgs) + sizeof(SmallArgs)>(min((int)blockIdx.x, PACT_MAX_BATCH - 1));
    extern __shared__ double s_dyn[];
    __shared__ SmallShared sh;
    auto meet = [&](int* counter, int add) __attribute__((always_inline)) { return count_in(counter, add, sh.got); };
    const bool resolver = (int)blockIdx.x < bt.B;
    const int workers = gridDim.x - bt.B, b = resolver ? blockIdx.x : ((int)blockIdx.x - bt.B) % bt.B;
    int T = 0, ticket = -1, changed = 0;
    bool select = resolver, first = true;
    if (!resolver) {
        if (threadIdx.x == 0) {
            int v = 0;
            for (int k = 0; k < SMALL_POLLS; ++k) {              // (some milliseconds at most)
                v = __hip_atomic_load(&a.tie_cnt[4 * b + 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (v & SMALL_READY) break;
                __builtin_amdgcn_s_sleep(8);
            }
            if (v & SMALL_READY && (v >> 16) & 0x7FF) v = __hip_atomic_fetch_add(&a.tie_cnt[4 * b + 3], 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
            sh.got = v;
        }
        __syncthreads();
        const int v = lane0_of(sh.got);
        T = v & SMALL_READY ? (v >> 16) & 0x7FF : 0;
        ticket = v & 0xFFFF;
        if (T == 0) return;
    }
    while (true) {
        if (select) {
            const int listed = select_sample<DT>(bt, a, sa, fresh_s(b), first, (unsigned char*)s_dyn, sh);
            if (!first || listed == 0) return;
            T = listed;
        }
        const int q = clamp_count(a.rep[b].n_kept, bt.s[b].n);
        const int nchunk = a.dk * Elem<DT>::BYTES / 16, rows = (T + 15) >> 4;
        int tiles = 4;                                           // (see centres_kernel)
        while (tiles > 1 && nchunk * tiles > 2 * 64) {
            const int half = 8 * tiles;
            if (rows * ((q + half - 1) / half) > items_wanted(workers / bt.B, nchunk, tiles) || T * (64 / half) > rho_fix_tokens(bt.n_max)) break;
            tiles >>= 1;
        }
        const int total = rows * ((q + 16 * tiles - 1) / (16 * tiles)), per = total < 128 ? 1 : 4;       // items; of a ticket
        bool again = false;
        if (select) {
            const int seen = meet(&a.tie_cnt[4 * b + 2], 4);
            if (seen & 1) {                                      // all items are done
                changed = seen & (ORDER_PAIRS | ORDER_BAND);
                again = changed || a.write_rho;
                if (!again) return;
            }
        }
        while (!again) {
            if (ticket < 0) {
                __syncthreads();
                if (threadIdx.x == 0) sh.got = __hip_atomic_fetch_add(&a.tie_cnt[4 * b + 3], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xFFFF;
                __syncthreads();
                ticket = lane0_of(sh.got);
            }
            const int item = ticket * per, mine = min(per, total - item);
            ticket = -1;
            if (mine <= 0) return;
            recheck_items<DT>(bt, a, fresh_s(b), fresh_s(T), fresh_s(q), fresh_s(item), fresh_s(item + mine), tiles, s_dyn);
            if (meet(&a.tie_cnt[4 * b + 1], mine) != total - mine) continue;
            changed = order_changed(bt, a, fresh_s(b), fresh_s(T), fresh_s(q), tiles, (unsigned char*)s_dyn, sh.flag);
            if (!(meet(&a.tie_cnt[4 * b + 2], changed | 1) & 4)) return;          // the selection still runs
            if (!changed && !a.write_rho) return;
            again = true;
        }
        // the fp64 densities take their places
        const int32_t* list = a.tie_list + (size_t)b * RHO_RECHECK_MAX;
        const double* part_b = a.rho_fix + (size_t)b * 2 * rho_fix_tokens(bt.n_max) * rho_fix_chunks(bt.n_max);
        const int t = fresh_v(threadIdx.x);
        if (t < T) a.rho[(size_t)b * bt.n_max + min(list[t] & 0xFFFF, q - 1)] = part_b[t];
        stores_done();                                           // (read back by this workgroup only)
        if (!changed) return;
        select = true;
        first = false;
    }
}

// ------------------------------------------------------------------------------------------
constexpr int CAND_BUF = 128;

// The two nearest-centre searches share one kernel (below): the assignment of the kept tokens
// needs only the centres, so in the fused path it runs beside the recovery of the pruned tokens
// (whose slowest wavefronts leave most of the chip idle) instead of before the candidate pass.
struct NearArgs {
    pact_report* rep;
    const char* keys; int dk;
    const double* nn;
    const uint64_t* adj;
    float margin;
    int32_t* cluster_id; int32_t* cluster_counts;
    int32_t* slots; int32_t* big;           // (optional) first members per cluster and the list of large clusters
    // assignment of kept tokens (Alg. 2 last loop); assign_blocks == 0: not in this launch
    const int32_t* idx; const uint64_t* cmask; const uint32_t* status; const int32_t* cnum; int assign_blocks;
    // recovery of pruned tokens (Eq. 8/9): the blocks before the assignment ones
    const int32_t* pruned_idx; const int32_t* center_idx; const float* cbest;
    // small samples, which look for their candidates here: reciprocal norms, fp32 keys' byte planes
    const float* rinv; const char* planes;
};

// Token `tok` joins cluster c (both local to the sample): the cluster's size goes up and, where
// the caller keeps them, the token takes the next of the cluster's member slots; the member that
// makes a cluster a large one puts it on the list of those.  counts/slots/big: the sample's.
__device__ __forceinline__ void join_cluster(const NearArgs& a, pact_report* rp, int base, int c, int tok) {
    const int s = atomicAdd(&a.cluster_counts[base + c], 1);
    if (a.slots) {
        if (s < MERGE_SLOTS) a.slots[(size_t)(base + c) * MERGE_SLOTS + s] = tok;
        if (s == MERGE_BIG - 1) a.big[base + atomicAdd(&rp->reserved[0], 1)] = c;
    }
}

// Dot product in fp64 of the rows `mine` and `other` by the 16 lanes part = 0..15 of a group
// (lane `part` takes the 16-byte chunks part, part + 16, ...; four chunks of either row in
// flight per lane).  Every lane of the group gets the sum.
template <int DT>
__device__ __forceinline__ double group_dot64(const char* mine, const char* other, int nchunk, int part) {
    constexpr int EPL = Elem<DT>::EPL;
    double acc = 0.0;
#pragma unroll 1
    for (int k0 = part; k0 < nchunk; k0 += 64) {
        uint4 va[4], vb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t o = (size_t)(k0 + 16 * u < nchunk ? k0 + 16 * u : k0) * 16;
            va[u] = *(const uint4*)(mine + o);
            vb[u] = *(const uint4*)(other + o);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (k0 + 16 * u < nchunk) {
                // (each word is tied to the running sum, so that conversions are not hoisted ahead of the
                //  additions: registers decide this kernel's occupancy)
                asm volatile("" : "+v"(va[u].x), "+v"(vb[u].x) : "v"(acc));
                if constexpr (DT == PACT_BF16) {
                    const uint32_t wa[4] = {va[u].x, va[u].y, va[u].z, va[u].w}, wb[4] = {vb[u].x, vb[u].y, vb[u].z, vb[u].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        uint32_t p = wa[i], r = wb[i];
                        asm volatile("" : "+v"(p), "+v"(r) : "v"(acc));
                        acc = fma((double)__uint_as_float(p << 16), (double)__uint_as_float(r << 16), acc);
                        acc = fma((double)__uint_as_float(p & 0xFFFF0000u), (double)__uint_as_float(r & 0xFFFF0000u), acc);
                    }
                } else {
                    double a[8], x[8];
                    Elem<DT>::widen(va[u], a);
                    Elem<DT>::widen(vb[u], x);
#pragma unroll
                    for (int i = 0; i < EPL; ++i) acc = fma(a[i], x[i], acc);
                }
            }
        }
    }
    return group_sum_f64(acc, 16);
}

// 16 lanes per token.  The set bits of words wb + part + 16 u (lane `part` of the group holds word[u]) as numbers from 64 wb on: those
// from the skip-th to the LIST_TURN - 1 after it into the token's list in LDS, n of them; ntot counts all.
constexpr int LIST_TURN = 16;
__device__ __forceinline__ void list_bits(const uint64_t (&word)[4], int wb, int lane, int skip, lds_i32* list, int& n, int& ntot) {
    const int part = lane & 15, gbase = lane & ~15;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        uint32_t who = (uint32_t)(__ballot(word[u] != 0) >> gbase) & 0xFFFFu;
        while (who) {
            const int src = __builtin_ctz(who);
            who &= who - 1;
            uint64_t bits = __shfl(word[u], gbase + src, 64);
            const int cbase = (wb + src + 16 * u) << 6;
            while (bits) {
                const int c = cbase + __builtin_ctzll(bits);
                bits &= bits - 1;
                if (ntot >= skip && n < LIST_TURN) {
                    if (part == 0) list[n] = c;
                    ++n;
                }
                ++ntot;
            }
        }
    }
}
// fp64 for the n listed candidates (token_of[c]: a candidate's token): their tokens and norms in one trip, then row by row.
template <int DT>
__device__ __forceinline__ void nearest_listed(const lds_i32* list, int n, int lane, const char* mine, double nnp, const char* kb,
                                               size_t row_bytes, const double* nnb, const int32_t* token_of, double thr,
                                               double& best, int& bestc) {
    const int part = lane & 15, gbase = lane & ~15, nchunk = (int)(row_bytes / 16);
    int ctk = 0, cid = 0;
    double cnn = 0.0;
    if (part < n) {
        cid = list[part];
        ctk = token_of[cid];
        cnn = nnb[ctk];
    }
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
        const int c = __shfl(cid, gbase + k, 64);
        const int tc = __shfl(ctk, gbase + k, 64);
        const double nc = __shfl(cnn, gbase + k, 64);
        const double d = cos_dist64(group_dot64<DT>(mine, kb + (size_t)tc * row_bytes, nchunk, part), nnp, nc);
        if (d < thr && (d < best || (d == best && c < bestc))) { best = d; bestc = c; }
    }
}

// The candidates of one token, listed by a wavefront from words of bits (a word per lane) and compared as the buffer fills.
template <int DT> struct CandidateList {
    lds_i32 *cand, *ctok;
    lds_f32* ccos;
    const char* mine; double nnp;
    const char* kb; size_t row_bytes; const double* nnb;
    const int32_t* ix;
    int dk, lane; float margin;
    int nbuf = 0, ntot = 0;
    __device__ __forceinline__ void compare(bool complete, double& best, int& bestj) {
        const int32_t* ixl = ix;
        nearest_candidate<DT>(cand, ctok, ccos, nbuf, complete, mine, nnp, kb, row_bytes, nnb, dk, lane, INFINITY, margin,
                              [ixl](int j) { return ixl[j]; }, best, bestj);
    }
    __device__ __forceinline__ void add(uint64_t word, int w, double& best, int& bestj) {      // bits of word w
        BitPop bp{word};
        while (bp.any()) {
            int bit;
            const bool ok = bp.pop(bit);
            const uint64_t m = __ballot(ok);
            if (ok) cand[nbuf + lanes_below(m, lane)] = (w << 6) + bit;
            nbuf += __popcll(m);
            ntot += __popcll(m);
            if (nbuf > CAND_BUF - 64) {
                compare(false, best, bestj);
                nbuf = 0;
            }
        }
    }
    __device__ __forceinline__ void finish(double& best, int& bestj) {
        if (nbuf) compare(nbuf == ntot, best, bestj);
    }
};

// Alg. 2 last loop: every kept token joins the nearest centre.  Candidates are the centres
// its bitmap row reaches (the nearest centre is within d_c, hence one of them; it need not
// precede the token); with one candidate no distance is needed, otherwise Eq. 5 is
// evaluated (fp32 screen, fp64 where it matters).
// TPW tokens per wavefront, 64 / TPW lanes each, as long as they look for their candidates: one while the chip holds a wavefront for
// each token, four beyond that.  Up to four candidates of a token are then compared in fp64 by its 16 lanes, row by row; more take
// the whole wavefront, token by token (fp32 cosines of eight candidates at a time, fp64 for those that are left).
// Event brackets: 27 600 kept tokens of 8 videos 29 -> 19 us, 18 200 of 16 ragged images 27 -> 24 us, 12 800 of 32 crops 17 us either way.
template <int DT, int TPW>
__device__ __forceinline__ void assign_body(const Batch& bt, const NearArgs& a, int blk, lds_i32* cand,
                                            lds_i32* ctok, lds_f32* ccos, lds_i32* s_c) {
    constexpr int GL = 64 / TPW, WPL = 64 / GL;            // lanes per token, bitmap words per lane and turn
    pact_report* rep = a.rep;
    const int dk = a.dk;
    const double* nn = a.nn;
    const uint64_t* cmask = a.cmask;
    const int b = blockIdx.y;
    const Seg sg = bt.s[b];
    const int lane = threadIdx.x & 63, gl = lane & (GL - 1);
    const int wave = threadIdx.x >> 6;
    const int pw = (blk * 4 + wave) * TPW;
    const int q = clamp_count(rep[b].n_kept, sg.n);
    if (pw >= q) return;
    const int p = pw + lane / GL;
    const bool on = p < q;
    const int32_t* ix = a.idx + sg.base;
    const int32_t* cn = a.cnum + (size_t)b * bt.n_max;
    const uint32_t* st = a.status + (size_t)b * bt.n_max;
    const double* nnb = nn + sg.base;
    const uint64_t* row = a.adj + ((size_t)b * bt.n_max + min(p, q - 1)) * bt.W;
    const uint64_t* cm = cmask + (size_t)b * bt.W;
    const int tok = ix[min(p, q - 1)];
    const uint32_t stp = st[min(p, q - 1)];
    const int cnp = cn[min(p, q - 1)];
    // (the first 64 words of the row and of the centre mask go out with them, before the status
    //  is looked at: a trip less for the tokens that are not centres)
    uint64_t first[WPL];
#pragma unroll
    for (int u = 0; u < WPL; ++u) {
        const int w = gl + GL * u;
        first[u] = w < bt.W ? row[w] & cm[w] : 0ull;
    }
    const int Wq = (q + 63) >> 6;
    const bool centre = stp == ST_CENTER;
    // the number of candidates (at most one per lane counts), and the first lane's that has one
    int cid = cnp, some = 0, j1 = -1;
    if (!centre) {
#pragma unroll
        for (int u = 0; u < WPL; ++u) {
            const int w = gl + GL * u;
            if (w == Wq - 1 && (q & 63)) first[u] &= (1ull << (q & 63)) - 1ull;
            if (w >= Wq) first[u] = 0ull;
            if (first[u] && j1 < 0) j1 = (w << 6) + __builtin_ctzll(first[u]);
            some += __popcll(first[u]);
        }
        for (int w = 64 + gl; w < Wq; w += GL) {
            uint64_t word = row[w] & cm[w];
            if (w == Wq - 1 && (q & 63)) word &= (1ull << (q & 63)) - 1ull;
            if (word && j1 < 0) j1 = (w << 6) + __builtin_ctzll(word);
            some += __popcll(word);
        }
    }
    const uint64_t gmask = GL == 64 ? ~0ull : ((1ull << (GL & 63)) - 1ull) << (lane & ~(GL - 1));
    const uint64_t have = __ballot(some > 0) & gmask, many = __ballot(some > 1) & gmask;
    const bool several = !centre && (many != 0 || (have & (have - 1)) != 0);
    if (!centre) {
        const int j = __shfl(j1, have ? __builtin_ctzll(have) : lane, 64);
        cid = have && !several ? cn[j] : -1;               // a single centre in reach: no distance needed
    }
    const size_t row_bytes = (size_t)dk * Elem<DT>::BYTES;
    const char* kb = a.keys + (size_t)sg.base * row_bytes;
    const bool few = TPW > 1 && group_sum_f32<16>((float)min(some, 1024)) <= 4.0f;
    if constexpr (TPW == 4) {
        if (several && few && on) {                        // (the same for a token's lanes)
            lds_i32* list = s_c + (threadIdx.x >> 4) * LIST_TURN;
            double best = INFINITY;
            int bestj = 0x7FFFFFFF;
            int n = 0, ntot = 0;
            list_bits(first, 0, lane, 0, list, n, ntot);
#pragma unroll 1
            for (int wb = 64; wb < Wq; wb += 64) {
                uint64_t word[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int w = wb + gl + 16 * u;
                    word[u] = w < Wq ? row[w] & cm[w] : 0ull;
                    if (w == Wq - 1 && (q & 63)) word[u] &= (1ull << (q & 63)) - 1ull;
                }
                list_bits(word, wb, lane, 0, list, n, ntot);
            }
            nearest_listed<DT>(list, n, lane, kb + (size_t)tok * row_bytes, nnb[tok], kb, row_bytes, nnb, ix, INFINITY, best, bestj);
            cid = bestj;
        }
    }
    uint64_t todo = __ballot(several && on && gl == 0 && !(TPW > 1 && few));
    while (todo) {
        const int l0 = __builtin_ctzll(todo);
        todo &= todo - 1;
        const bool mine_g = (lane & ~(GL - 1)) == l0;
        const int pa = pw + l0 / GL, toka = __builtin_amdgcn_readlane(tok, l0);
        const uint64_t* rowa = a.adj + ((size_t)b * bt.n_max + pa) * bt.W;
        const char* mine = kb + (size_t)toka * row_bytes;
        const double nnp = nnb[toka];
        double best = INFINITY;
        int bestj = 0x7FFFFFFF;
        CandidateList<DT> list{cand, ctok, ccos, mine, nnp, kb, row_bytes, nnb, ix, dk, lane, a.margin};
#pragma unroll 1
        for (int u = 0; u < WPL; ++u) {
            list.add(mine_g ? first[0] : 0ull, gl + GL * u, best, bestj);
#pragma unroll
            for (int v = 0; v + 1 < WPL; ++v) if (mine_g) first[v] = first[v + 1];
        }
#pragma unroll 1
        for (int w0 = 64; w0 < Wq; w0 += 64) {
            const int w = w0 + lane;
            uint64_t word = w < Wq ? rowa[w] & cm[w] : 0ull;
            if (w == Wq - 1 && (q & 63)) word &= (1ull << (q & 63)) - 1ull;
            list.add(word, w, best, bestj);
        }
        list.finish(best, bestj);
        if (mine_g) cid = bestj;                           // (a position; its cluster below, for all tokens at once)
    }
    if (several && on) cid = cid >= 0 && cid != 0x7FFFFFFF ? cn[cid] : -1;
    if (gl == 0 && on) {
        a.cluster_id[sg.base + tok] = cid;
        if (cid >= 0 && a.cluster_counts) join_cluster(a, rep + b, sg.base, cid, tok);
        note_odd_norm(rep + b, nnb[tok]);
    }
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4;
// The assignment for wide bf16 rows: 16 kept tokens per workgroup, all centres that any of them reaches (the neighbours of tokens that are close in the
// sequence are mostly the same) as 16 x 16 products on v_mfma_f32_16x16x32_bf16, 32 of them a turn, an eighth of the row's width per wavefront,
// straight from the rows.  A token per wavefront (assign_body) reads every candidate's row for every token, eight candidates in 14 dependent trips.
// 7290 rows of 7 KB with five centres each in reach: bracket 63 us -> 31, 20 to 24 of a workgroup's, of which 5 to the words of its tokens, 3 the list, 6 to 14
// the rows (72 MB in all, at the rate of the last-level cache), 5 fp64 where it is needed.
// Products are summed in chains of 224 elements, so the margin of the screen is a twelfth of the long chain's and few tokens
// are left with more than one candidate; those take fp64, a wavefront per token.  A token of which more than ASSIGN_KEEP candidates stay, or all tokens
// where more than ASSIGN_LIST centres are reached, are compared as assign_body does it.
// grid (16 tokens each, rounded up to a multiple of 8; an eighth of the sequence per XCD, whose L2 then holds the rows that are read again; B), block 512.
constexpr int ASSIGN_LIST = 1024, ASSIGN_KEEP = 8, ASSIGN_CHAIN = 7;
// (on the same rows the products of all 16 x 16 pairs are off by at most 2.5% of the margin's first term)
static float assign_tile_margin(int dk) { return (float)((ASSIGN_CHAIN * 32 + dk / 1024 + 24.0) * (1.0 / 8388608.0) + 2.5e-6); }
__global__ __launch_bounds__(512, 4) void assign_tile_kernel(Batch bt, NearArgs a, float tile_margin) {
    constexpr int DT = PACT_BF16, WAVES = 8;
    __shared__ uint64_t s_union[PACT_MAX_TOKENS / 64];
    __shared__ uint16_t s_j[ASSIGN_LIST];
    __shared__ int s_ct[ASSIGN_LIST];
    __shared__ float s_rc[ASSIGN_LIST], s_part[2][WAVES][16][17], s_keepc[16][ASSIGN_KEEP];
    __shared__ int s_keepj[16][ASSIGN_KEEP], s_keept[16][ASSIGN_KEEP], s_tok[16], s_count, s_best[16], s_todo[16], s_ntodo;
    __shared__ int s_cand[WAVES][CAND_BUF], s_ctok[WAVES][CAND_BUF];
    __shared__ float s_ccos[WAVES][CAND_BUF];
    const int b = blockIdx.y;
    const Seg sg = bt.s[b];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), t = (tid >> 4) & 15, gl = tid & 15;
    const bool owner = tid < 256;                                            // 16 lanes per token; the other wavefronts help with the products and in fp64
    const int p0 = (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * 16;
    if (p0 >= sg.n) return;
    // (the first 64 words of the token's row and of the mask of centres, and its status, go out ahead of the number of kept tokens: they lie inside the workspace)
    const uint64_t* cm = a.cmask + (size_t)b * bt.W;
    uint64_t ahead[4];
    {
        const uint64_t* r = a.adj + ((size_t)b * bt.n_max + min(p0 + t, sg.n - 1)) * bt.W;
#pragma unroll
        for (int u = 0; u < 4; ++u) ahead[u] = gl + 16 * u < bt.W ? r[gl + 16 * u] & cm[gl + 16 * u] : 0ull;
    }
    const int q = clamp_count(a.rep[b].n_kept, sg.n);
    if (p0 >= q) return;
    const int p = min(p0 + t, q - 1), Wq = (q + 63) >> 6;
    const bool on = owner && p0 + t < q;
    const int32_t* ix = a.idx + sg.base;
    const int32_t* cn = a.cnum + (size_t)b * bt.n_max;
    const double* nnb = a.nn + sg.base;
    const float* rinv = a.rinv + sg.base;
    const uint64_t* row = a.adj + ((size_t)b * bt.n_max + p) * bt.W;
    const int tok = ix[p];
    const bool centre = (a.status + (size_t)b * bt.n_max)[p] == ST_CENTER;
    const float rt = rinv[tok];
    for (int w = tid; w < Wq; w += 512) s_union[w] = 0ull;
    if (tid == 0) s_ntodo = 0;
    // the lane's part of the centres in reach: how many, and the first
    auto inside = [&](uint64_t word, int w) __attribute__((always_inline)) {
        if (w == Wq - 1 && (q & 63)) word &= (1ull << (q & 63)) - 1ull;
        return w < Wq && on && !centre ? word : 0ull;
    };
    auto reached = [&](int w) __attribute__((always_inline)) { return inside(w < Wq ? row[w] & cm[w] : 0ull, w); };
    int some = 0, j1 = -1;
    auto note = [&](uint64_t word, int w) __attribute__((always_inline)) {
        if (word && j1 < 0) j1 = (w << 6) + __builtin_ctzll(word);
        some += __popcll(word);
    };
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        ahead[u] = inside(ahead[u], gl + 16 * u);
        note(ahead[u], gl + 16 * u);
    }
#pragma unroll 4
    for (int w = 64 + gl; w < Wq; w += 16) note(reached(w), w);
    const int gbase = lane & 48;
    auto group_bits = [&](bool v) __attribute__((always_inline)) { return (uint32_t)(__ballot(v) >> gbase) & 0xFFFFu; };
    const uint32_t have = group_bits(some > 0), many = group_bits(some > 1);
    const bool several = on && !centre && (many != 0 || (have & (have - 1)) != 0);
    int bestj = have ? __shfl(j1, gbase + __builtin_ctz(have), 64) : -1;      // (a single centre in reach: no distance needed)
    if (gl == 0 && owner) s_tok[t] = several ? tok : -1;
    const size_t row_bytes = (size_t)a.dk * 2;
    const char* kb = a.keys + (size_t)sg.base * row_bytes;
    if (__syncthreads_or(several)) {
        if (several) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (ahead[u]) atomicOr((unsigned long long*)&s_union[gl + 16 * u], (unsigned long long)ahead[u]);
            for (int w = 64 + gl; w < Wq; w += 16) {
                const uint64_t word = reached(w);
                if (word) atomicOr((unsigned long long*)&s_union[w], (unsigned long long)word);
            }
        }
        __syncthreads();
        if (wave == 0) {
            int run = 0;
            for (int w0 = 0; w0 < Wq; w0 += 64) {
                uint64_t word = w0 + lane < Wq ? s_union[w0 + lane] : 0ull;
                const int cnt = __popcll(word), inc = wave_scan_incl_i32(cnt);
                for (int at = run + inc - cnt; word && at < ASSIGN_LIST; ++at) {
                    s_j[at] = (uint16_t)(((w0 + lane) << 6) + __builtin_ctzll(word));
                    word &= word - 1;
                }
                run += lane63_of(inc);
            }
            if (lane == 0) s_count = run;
        }
        __syncthreads();
        const int U = lane0_of(s_count);
        bool over = U > ASSIGN_LIST;
        int kept = 0;
        if (!over) {
            for (int k = tid; k < U; k += 512) {
                const int c = ix[s_j[k]];
                s_ct[k] = c;
                s_rc[k] = rinv[c];
            }
            __syncthreads();
            const int l16 = lane & 15, kg = lane >> 4, nchunk = a.dk / 8, steps = (nchunk + 3) / 4;
            const int from = steps * wave / WAVES, to = steps * (wave + 1) / WAVES;
            // (a token that needs no distance stands in with the row of one that does; the exchange is outside the choice, for all lanes)
            const int own = s_tok[l16], other = __shfl(own, __builtin_ctz((uint32_t)__ballot(own >= 0) | 0x10000u) & 15, 64);
            const char* rowA = kb + (size_t)max(own >= 0 ? own : other, 0) * row_bytes;
            float top = -INFINITY;
#pragma unroll 1
            for (int k0 = 0; k0 < U; k0 += 32) {
                const char* rowB[2];
                bool reach[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    rowB[i] = kb + (size_t)s_ct[min(k0 + 16 * i + l16, U - 1)] * row_bytes;
                    const int k = k0 + 16 * i + gl, j = s_j[min(k, U - 1)];
                    reach[i] = several && k < U && ((row[j >> 6] >> (j & 63)) & 1ull);
                }
                f32x4_t sum[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
                // (two loops and no branch around the second sixteen's products: across such a branch the compiler left three of the eight wait states between the last
                //  product and the addition that reads it out, and every fourth token had a stale sum.  A test follows all products of all kernels to their readers)
                auto products = [&](auto tiles) __attribute__((always_inline)) {
                    constexpr int NT = decltype(tiles)::value;
#pragma unroll 1
                    for (int s0 = from; s0 < to; s0 += ASSIGN_CHAIN) {
                        uint4 va[ASSIGN_CHAIN], vb[NT][ASSIGN_CHAIN];
#pragma unroll
                        for (int u = 0; u < ASSIGN_CHAIN; ++u) {
                            const int e = min(s0 + u, to - 1) * 4 + kg;
                            const size_t o = e < nchunk ? (size_t)e * 16 : 0;
                            va[u] = *(const uint4*)(rowA + o);
#pragma unroll
                            for (int i = 0; i < NT; ++i) vb[i][u] = *(const uint4*)(rowB[i] + o);
                        }
                        f32x4_t acc[NT];
#pragma unroll
                        for (int i = 0; i < NT; ++i) acc[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                        for (int u = 0; u < ASSIGN_CHAIN; ++u) {
                            const bool in = s0 + u < to && (s0 + u) * 4 + kg < nchunk;
                            const uint4 none = make_uint4(0, 0, 0, 0);
                            const bf16x8_t x = __builtin_bit_cast(bf16x8_t, in ? va[u] : none);
#pragma unroll
                            for (int i = 0; i < NT; ++i)
                                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, __builtin_bit_cast(bf16x8_t, in ? vb[i][u] : none), acc[i], 0, 0, 0);
                        }
#pragma unroll
                        for (int i = 0; i < NT; ++i) sum[i] += acc[i];
                    }
                };
                if (k0 + 16 < U) products(std::integral_constant<int, 2>{});
                else products(std::integral_constant<int, 1>{});
                // sum[i][r]: token 4 kg + r of the sixteen, candidate k0 + 16 i + l16; this wavefront's part of the row
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) s_part[i][wave][4 * kg + r][l16] = sum[i][r];
                __syncthreads();
                float v[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int k = min(k0 + 16 * i + gl, U - 1);
                    float dot = 0.0f;
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) dot += s_part[i][w][t][gl];
                    v[i] = dot * rt * s_rc[k];
                }
                __syncthreads();
                // the candidates that can still be the nearest: those before, then this turn's, by the token's 16 lanes
                top = fmaxf(top, group_max_f32<16>(fmaxf(reach[0] ? v[0] : -INFINITY, reach[1] ? v[1] : -INFINITY)));
                const float floor32 = top - 2.0f * tile_margin;
                const float oldc = gl < kept ? s_keepc[t][gl & (ASSIGN_KEEP - 1)] : 0.0f;
                const int oldj = gl < kept ? s_keepj[t][gl & (ASSIGN_KEEP - 1)] : 0;
                uint32_t m = group_bits(gl < kept && !(oldc < floor32));
                __builtin_amdgcn_wave_barrier();
                auto keep = [&](uint32_t m, int base, float c, int j) __attribute__((always_inline)) {
                    const int at = base + __popc(m & ((1u << gl) - 1u));
                    if (((m >> gl) & 1u) && at < ASSIGN_KEEP) { s_keepc[t][at] = c; s_keepj[t][at] = j; }
                    return base + __popc(m);
                };
                kept = keep(m, 0, oldc, oldj);
#pragma unroll
                for (int i = 0; i < 2; ++i) kept = keep(group_bits(reach[i] && !(v[i] < floor32)), kept, v[i], s_j[min(k0 + 16 * i + gl, U - 1)]);
                over = over || kept > ASSIGN_KEEP;
                kept = min(kept, ASSIGN_KEEP);
                __builtin_amdgcn_wave_barrier();
            }
            if (several) {
                bestj = s_keepj[t][0];
                if (gl < kept) s_keept[t][gl & (ASSIGN_KEEP - 1)] = ix[s_keepj[t][gl & (ASSIGN_KEEP - 1)]];
            }
        }
        // what is left for fp64 (and for the long way), a wavefront per token
        const bool left = several && (over || kept > 1);
        if (left && gl == 0) s_todo[atomicAdd(&s_ntodo, 1)] = t | kept << 8 | (over ? 1 << 16 : 0);
        __syncthreads();
        const int n = lane0_of(s_ntodo);
        for (int k = wave; k < n; k += WAVES) {
            const int what = lane0_of(s_todo[k]), ta = what & 15, toka = lane0_of(s_tok[ta]);
            const char* mine = kb + (size_t)toka * row_bytes;
            double best = INFINITY;
            int bj = 0x7FFFFFFF;
            if (!(what >> 16)) {
                nearest_fp64<DT, 7>((lds_i32*)s_keepj[ta], (lds_i32*)s_keept[ta], what >> 8 & 0xFF, mine, nnb[toka], kb, row_bytes, nnb, a.dk, lane,
                                    INFINITY, best, bj);
            } else {
                const uint64_t* rowa = a.adj + ((size_t)b * bt.n_max + p0 + ta) * bt.W;
                CandidateList<DT> list{(lds_i32*)s_cand[wave], (lds_i32*)s_ctok[wave], (lds_f32*)s_ccos[wave], mine, nnb[toka], kb, row_bytes, nnb, ix, a.dk, lane, a.margin};
#pragma unroll 1
                for (int w0 = 0; w0 < Wq; w0 += 64) {
                    const int w = w0 + lane;
                    uint64_t word = w < Wq ? rowa[w] & cm[w] : 0ull;
                    if (w == Wq - 1 && (q & 63)) word &= (1ull << (q & 63)) - 1ull;
                    list.add(word, w, best, bj);
                }
                list.finish(best, bj);
            }
            if (lane == 0) s_best[ta] = bj;
        }
        __syncthreads();
        if (left) bestj = s_best[t];
    }
    if (gl == 0 && on) {
        const int cid = centre ? cn[p] : bestj >= 0 && bestj != 0x7FFFFFFF ? cn[bestj] : -1;
        a.cluster_id[sg.base + tok] = cid;
        if (cid >= 0 && a.cluster_counts) join_cluster(a, a.rep + b, sg.base, cid, tok);
        note_odd_norm(a.rep + b, nnb[tok]);
    }
}

// What the matrix-core pass over centres x pruned tokens leaves (MODE_CAND of gram_kernel: the same byte products, cut and margin), for 16
// pruned tokens and in LDS: a wavefront per group of 64 centres and turn, v_mfma 16x16 straight from the key rows, 16 (fp32 keys: 12)
// 16-byte chunks of centres in flight per lane.  Bound by its chain: lists, rows and norms, products, 100 instructions of one wavefront.  (The lists were
// requested once their lengths were known at first: 3 us longer.)
// tokB: this lane's token (lanes 16 apart the same), first: the centre 64 wavefront + lane, if there is such a one.
// s_cb, s_cw: [group][16]; s_rs: [4 wavefronts][64].
template <int DT>
__device__ __forceinline__ void candidates_16(const NearArgs& a, const Seg& sg, int tokB, int first, int C, lds_f32* s_cb, lds_u64* s_cw,
                                              lds_f32* s_rs) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kg = lane >> 4;
    const int32_t* co = a.center_idx + sg.base;
    const float* rinv = a.rinv + sg.base;
    const int groups = (a.dk + 63) / 64;
    const size_t row = DT == PACT_BF16 ? (size_t)a.dk * 2 : (size_t)groups * 256;
    const char* kb = (DT == PACT_BF16 ? a.keys : a.planes) + (size_t)sg.base * row;
    const float rj = rinv[tokB], t_lo = recovery_reach(sg, a.margin);
    const char* rowB = kb + (size_t)tokB * row;
    lds_f32* rs = s_rs + wave * 64;
    for (int c0 = wave * 64; c0 < C; c0 += 4 * 64) {
        const int tokA = c0 + lane >= C ? 0 : c0 == wave * 64 ? first : co[c0 + lane];
        rs[lane] = rinv[tokA];
        const char* rowA[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) rowA[k] = kb + (size_t)__shfl(tokA, 16 * k + l16, 64) * row;
        f32x4_t acc[4];
        if constexpr (DT == PACT_BF16) {
            const int nchunk = a.dk / 8;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            for (int s0 = 0; s0 < nchunk; s0 += 16) {                    // (four steps of 32 elements in flight)
                uint4 va[4][4], vb[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = s0 + 4 * u + kg;
                    const size_t o = e < nchunk ? (size_t)e * 16 : 0;
                    vb[u] = *(const uint4*)(rowB + o);
#pragma unroll
                    for (int k = 0; k < 4; ++k) va[k][u] = *(const uint4*)(rowA[k] + o);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = s0 + 4 * u + kg < nchunk;
                    const uint4 none = make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, in ? va[k][u] : none),
                                                                         __builtin_bit_cast(bf16x8_t, in ? vb[u] : none), acc[k], 0, 0, 0);
                }
            }
        } else {
            i32x4_t ord[3][4];
#pragma unroll
            for (int o = 0; o < 3; ++o)
#pragma unroll
                for (int k = 0; k < 4; ++k) ord[o][k] = i32x4_t{0, 0, 0, 0};
            for (int g = 0; g < groups; ++g) {
                i32x4_t va[4][3], vb[3];
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) {
                    const size_t o = (size_t)g * 192 + pl * 64 + kg * 16;
                    vb[pl] = *(const i32x4_t*)(rowB + o);
#pragma unroll
                    for (int k = 0; k < 4; ++k) va[k][pl] = *(const i32x4_t*)(rowA[k] + o);
                }
#pragma unroll
                for (int o = 0; o < 3; ++o)
#pragma unroll
                    for (int pl = 0; pl <= o; ++pl)
#pragma unroll
                        for (int k = 0; k < 4; ++k) ord[o][k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(va[k][pl], vb[o - pl], ord[o][k], 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[k][r] = fmaf((float)ord[0][k][r], 16777216.0f, fmaf((float)ord[1][k][r], 65536.0f, (float)ord[2][k][r] * 256.0f));
        }
        // acc[k][r]: centre c0 + 16 k + 4 kg + r, token t0 + l16
        __builtin_amdgcn_wave_barrier();                                 // (the wavefront's own part of LDS)
        float top = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const f32x4_t f = *(const lds_f32x4*)(rs + 16 * k + 4 * kg);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc[k][r] = c0 + 16 * k + 4 * kg + r < C ? acc[k][r] * f[r] : __builtin_nanf("");
                top = fmaxf(top, acc[k][r]);
            }
        }
        top = fmaxf(top, __shfl_xor(top, 16, 64));
        top = fmaxf(top, __shfl_xor(top, 32, 64));
        const float cutv = candidate_cut(top, rj, a.margin, t_lo);
        uint32_t lo = 0u, hi = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            lo |= (acc[0][r] >= cutv ? 1u : 0u) << r | (acc[1][r] >= cutv ? 1u : 0u) << (16 + r);
            hi |= (acc[2][r] >= cutv ? 1u : 0u) << r | (acc[3][r] >= cutv ? 1u : 0u) << (16 + r);
        }
        uint64_t word = ((uint64_t)hi << 32 | lo) << (4 * kg);
        word |= __shfl_xor(word, 16, 64);
        word |= __shfl_xor(word, 32, 64);
        if (kg == 0) {
            s_cb[(c0 >> 6) * 16 + l16] = top;
            s_cw[(c0 >> 6) * 16 + l16] = word;
        }
    }
}

// Eq. 8/9: every pruned token joins the nearest centre iff its fp64 distance is below
// alpha*d_c.  The matrix-core pass left, per pruned token t and group w of 64 centres, the
// group's largest fp32 cosine cbest[w][t] and a word of candidates (bits of the centres within
// reach whose cosine is at most 2 * margin below it), laid out [w][t].  With gm the largest of
// a token's cbest values, the nearest centre in exact arithmetic is a candidate of a group
// whose cbest >= gm - 2 * margin (margin bounds the error of an fp32 cosine).  Usually that is
// one centre, clear of the threshold: decided without touching a key.  Otherwise (several
// candidates, or one too close to alpha*d_c) Eq. 5 is evaluated in fp64 for each of them.
// What a token costs is its chain of dependent memory accesses, so 16 lanes work on one token
// (16 tokens per block and turn): the values and words of 64 groups arrive in one trip and are
// kept for the listing, a candidate row in another.  Blocks blk = 0 .. nblk-1, 256 threads.
// s_c: [16][LIST_TURN] candidate ids per token slot.
// HERE: the candidates are found by candidates_16 (SMALL_TOKENS at most).  BESIDE: in one kernel with the assignment.
template <int DT, bool HERE, bool BESIDE>
__device__ __forceinline__ void recover_body(const Batch& bt, const NearArgs& a, int blk, int nblk, lds_i32* s_c, lds_f32* s_cb = nullptr,
                                             lds_u64* s_cw = nullptr, lds_f32* s_rs = nullptr) {
    pact_report* rep = a.rep;
    const int b = blockIdx.y;
    const Seg sg = bt.s[b];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int t_first = blk * 16 + (tid >> 4);
    // (in a full reduction the lists have room for n: they go out before their lengths are known)
    int tokB = 0, first = 0;
    if (HERE && a.idx) {
        tokB = a.pruned_idx[sg.base + min(blk * 16 + (tid & 15), sg.n - 1)];
        first = a.center_idx[sg.base + min(tid, sg.n - 1)];
    }
    const int q = clamp_count(rep[b].n_kept, sg.n), np = clamp_count(rep[b].n_pruned, sg.n - q),
              C = clamp_count(rep[b].n_centers, q);
    const size_t row_bytes = (size_t)a.dk * Elem<DT>::BYTES;
    const char* kb = a.keys + (size_t)sg.base * row_bytes;
    const double* nnb = a.nn + sg.base;
    const int32_t* co = a.center_idx + sg.base;
    const int32_t* pruned = a.pruned_idx + sg.base;
    int32_t* cluster_id = a.cluster_id + sg.base;
    int32_t* cluster_counts = a.cluster_counts ? a.cluster_counts + sg.base : nullptr;
    const double thr = (double)sg.alpha * (double)sg.d_c;
    const float margin = a.margin;
    const float t_lo = recovery_reach(sg, margin);
    const int Wc = (C + 63) >> 6;
    const float* cb = a.cbest + (size_t)b * bt.W * bt.n_max;        // [W][n_max]
    const uint64_t* cw = a.adj + ((size_t)b * bt.n_max + q) * bt.W; // [Wc][np]
    const int part = tid & 15, ts = tid >> 4;
    lds_i32* list = s_c + ts * LIST_TURN;
    for (int t = t_first; HERE ? t - ts < np : t < np; t += nblk * 16) {
        if constexpr (HERE) {
            if (!a.idx || t != t_first) {
                tokB = pruned[min(t - ts + part, np - 1)];
                if (C > 0) first = co[min(tid, C - 1)];
            }
            if (t - ts + part >= np) tokB = 0;
            __syncthreads();                                        // (the values of the turn before have been read)
            if (thr > 0.0 && C > 0) candidates_16<DT>(a, sg, tokB, first, C, s_cb, s_cw, s_rs);
            __syncthreads();
            if (t >= np) continue;
        }
        const int tok = HERE ? __shfl(tokB, (lane & 48) + ts, 64) : pruned[t];
        int res = -1;                                               // -1: no centre in reach
        if (thr > 0.0 && C > 0) {
            // groups part, part + 16, .. of the first 64 with their candidate words (a word is
            // only meaningful where the group's largest cosine is within reach); further
            // groups, if any, for the maximum only
            float v[4];
            uint64_t word[4];
            auto load_batch = [&](int wb) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int w = wb + part + 16 * u;
                    if constexpr (HERE) {
                        v[u] = w < Wc ? s_cb[w * 16 + ts] : -INFINITY;
                        word[u] = w < Wc ? s_cw[w * 16 + ts] : 0ull;
                    } else {
                        v[u] = w < Wc ? cb[(size_t)w * bt.n_max + t] : -INFINITY;
                        word[u] = w < Wc ? cw[(size_t)w * np + t] : 0ull;
                    }
                }
            };
            load_batch(0);
            float gm = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
            for (int w = 64 + part; w < Wc; w += 16) gm = fmaxf(gm, cb[(size_t)w * bt.n_max + t]);
            gm = group_max_f32<16>(gm);
            if (gm >= t_lo) {
                const float floor32 = fmaxf(gm - 2.0f * margin, t_lo);
                double thr_here = thr;                                   // (BESIDE: what follows of it and of the margin stays here; kept since the start it was spilled)
                float margin_here = margin;
                if constexpr (BESIDE && HERE) asm volatile("" : "+v"(thr_here), "+v"(margin_here));
                const bool clear = (double)gm - (1.0 - thr_here) > (double)margin_here;   // d < thr  <=>  cosine > 1 - thr: the nearest is certainly within alpha*d_c
                const char* mine = kb + (size_t)tok * row_bytes;
                double best = INFINITY;
                int bestc = 0x7FFFFFFF;
                bool first_batch_loaded = true;
                // The candidates are listed in the token's LDS slots, LIST_TURN per turn (one
                // turn unless the token is degenerate); all control flow from here on is uniform
                // within the 16 lanes of a token.
#pragma unroll 1
                for (int skip = 0;; skip += LIST_TURN) {
                    int n = 0, ntot = 0;
#pragma unroll 1
                    for (int wb = 0; wb < Wc; wb += 64) {
                        if (!first_batch_loaded) load_batch(wb);     // (the first turn starts with the values already here)
                        first_batch_loaded = false;
                        uint64_t within[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) within[u] = (v[u] >= floor32) ? word[u] : 0ull;
                        list_bits(within, wb, lane, skip, list, n, ntot);
                    }
                    if (ntot == 1 && clear) {                          // decided by the fp32 screen alone
                        bestc = list[0];
                        break;
                    }
                    nearest_listed<DT>(list, n, lane, mine, nnb[tok], kb, row_bytes, nnb, co, thr, best, bestc);
                    if (skip + LIST_TURN >= ntot) break;
                }
                res = bestc != 0x7FFFFFFF ? bestc : -1;
            }
        }
        if (part == 0) {
            cluster_id[tok] = res;
            // (recovered / dropped totals are derived from the cluster sizes by the merge: a
            //  counter that every wavefront hits would serialise at one L2 address)
            if (res >= 0 && cluster_counts) join_cluster(a, rep + b, sg.base, res, tok);
            note_odd_norm(rep + b, nnb[tok]);
        }
    }
}

// grid (recovery blocks + assign_blocks, B), block 256: the recovery blocks first - their chain of
// dependent accesses is the longest, and behind the assignment blocks (two turns of what the
// chip holds, the last ones idle: their number is sized by n, not by the kept tokens) they
// started 3 us late.
// PART: NEAREST_BOTH, or a build that holds one of the two searches only (the assignment alone
// needs fewer registers and runs four wavefronts per SIMD instead of three).  _HERE: the recovery finds its candidates itself (three per SIMD).
enum { NEAREST_BOTH = 0, NEAREST_ASSIGN = 1, NEAREST_RECOVER = 2, NEAREST_BOTH_HERE = 3, NEAREST_RECOVER_HERE = 4 };
template <int DT, int PART, int TPW>
__global__ __launch_bounds__(256, PART >= NEAREST_BOTH_HERE ? 3 : 4) void nearest_centre_kernel(Batch bt, NearArgs a) {
    __shared__ int s_cand[4][CAND_BUF], s_ctok[4][CAND_BUF];
    __shared__ float s_ccos[4][CAND_BUF];
    __shared__ int s_list[16 * LIST_TURN];
    const int wave = threadIdx.x >> 6;
    lds_i32* cand = (lds_i32*)s_cand[wave];
    lds_i32* ctok = (lds_i32*)s_ctok[wave];
    lds_f32* ccos = (lds_f32*)s_ccos[wave];
    constexpr bool HERE = PART == NEAREST_BOTH_HERE || PART == NEAREST_RECOVER_HERE;
    int block = blockIdx.x;
    if constexpr (HERE) asm("" : "+s"(block) : "s"(args_asked_for<sizeof(NearArgs)>(blockIdx.y)));       // (not volatile: see there)
    __shared__ uint64_t s_cw[HERE ? SMALL_TOKENS / 4 : 1];
    __shared__ float s_cb[HERE ? SMALL_TOKENS / 4 : 1];
    __shared__ f32x4_t s_rs[HERE ? 64 : 1];
    if constexpr (PART == NEAREST_ASSIGN) assign_body<DT, TPW>(bt, a, block, cand, ctok, ccos, (lds_i32*)s_list);
    else if constexpr (PART == NEAREST_RECOVER || PART == NEAREST_RECOVER_HERE)
        recover_body<DT, HERE, false>(bt, a, block, gridDim.x, (lds_i32*)s_list, (lds_f32*)s_cb, (lds_u64*)s_cw, (lds_f32*)s_rs);
    else if (block >= (int)gridDim.x - a.assign_blocks)
        assign_body<DT, TPW>(bt, a, block - (gridDim.x - a.assign_blocks), cand, ctok, ccos, (lds_i32*)s_list);
    else recover_body<DT, HERE, true>(bt, a, block, gridDim.x - a.assign_blocks, (lds_i32*)s_list, (lds_f32*)s_cb, (lds_u64*)s_cw, (lds_f32*)s_rs);
}

template <int PART, int TPW>
static int launch_nearest_part(const Batch& bt, const NearArgs& a, int blocks, pact_dtype k_dt, const char* name,
                               hipStream_t st) {
    dim3 grid(blocks, bt.B);
    if (k_dt == PACT_BF16) PACT_LAUNCH(name, (nearest_centre_kernel<PACT_BF16, PART, TPW>), grid, dim3(256), st, bt, a);
    else PACT_LAUNCH(name, (nearest_centre_kernel<PACT_F32, PART, TPW>), grid, dim3(256), st, bt, a);
    return PACT_OK;
}
// a.assign_blocks: whether the assignment takes part.  Four tokens per wavefront in it from 8192 kept ones on (see assign_body), beside the recovery
// from 20 000: its wavefronts then start behind the recovery's and one each is the shorter way up to that.  Both searches are always one launch.
// Batches as two launches (with their gap left out) / one / one with four tokens per wavefront, us: width 128, 32 of 729 (12 800 kept) 21.2 / 17.3 / 18.3, 5 of
// 5000 (13 700) 23.3 / 18.7 / 21.7, 2 of 16384 at lambda 0.5 (16 400) 30.2 / 26.5 / 31.9, 16 ragged images (21 500) 33.0 / 34.7 / 29.1, 8 of 6272 (27 600)
// 35.1 / 34.5 / 31.0, 40 of 2915 (64 000) 57.9 / 70.0 / 54.5; width 512: 29.1 / 22.1 / 23.1, 29.2 / 23.4 / 23.2, 36.0 / 32.5 / 36.1, 46.5 / 41.2 / 40.5,
// 46.1 / 43.3 / 40.1, 75.0 / 90.6 / 69.1; fp32 keys 33.5 / 24.4 / 25.3 to 97.7 / 102.8 / 88.2.
static int launch_nearest(const Batch& bt, NearArgs a, int recover_blocks, pact_dtype k_dt, const char* name,
                          hipStream_t st) {
    if (a.assign_blocks == 0)
        return a.rinv ? launch_nearest_part<NEAREST_RECOVER_HERE, 1>(bt, a, recover_blocks, k_dt, name, st)
                      : launch_nearest_part<NEAREST_RECOVER, 1>(bt, a, recover_blocks, k_dt, name, st);
    const bool four = !a.rinv && kept_estimate(bt) > (recover_blocks == 0 ? 8192 : 20000);
    a.assign_blocks = (bt.n_max + (four ? 15 : 3)) / (four ? 16 : 4);
    if (recover_blocks == 0)
        return four ? launch_nearest_part<NEAREST_ASSIGN, 4>(bt, a, a.assign_blocks, k_dt, name, st)
                    : launch_nearest_part<NEAREST_ASSIGN, 1>(bt, a, a.assign_blocks, k_dt, name, st);
    const int blocks = a.assign_blocks + recover_blocks;
    if (a.rinv) return launch_nearest_part<NEAREST_BOTH_HERE, 1>(bt, a, blocks, k_dt, name, st);
    return four ? launch_nearest_part<NEAREST_BOTH, 4>(bt, a, blocks, k_dt, name, st)
                : launch_nearest_part<NEAREST_BOTH, 1>(bt, a, blocks, k_dt, name, st);
}

// Which rows: event brackets of the assignment, a token per wavefront -> tiles, clustering alone, 300 / 1000 / 2000 / 4000 / 7290 tokens: 3584 wide 26 -> 19, 39 -> 19, 54 -> 27,
// 70 -> 26, 63 -> 31; 2048: 14 -> 12, 21 -> 16, 21 -> 15, 27 -> 17, 22 -> 20; 1024: 6.5 -> 6.6, 7.8 -> 9.2, 7.9 -> 9.2, 9.2 -> 9.6, 11.2 -> 12.8; 512: 10 -> 16 to 17 -> 24.
// Between 2 and 3.5 KB only where all rows together are 1.5 times what an XCD's L2 holds: a token per wavefront reads them again from there.  200 / 729 / 2000 / 3000 / 6000 tokens: 1032 wide
// 12.0 -> 14.6, 13.6 -> 14.0, 14.0 -> 16.0, 20.2 -> 20.2, 25.0 -> 21.9; 1280: 14.8 -> 15.3, 16.2 -> 18.1, 19.4 -> 21.2, 23.0 -> 20.4, 27.4 -> 26.2; 1536: 13.1 -> 14.7, 15.3 -> 17.3,
// 21.7 -> 20.1, 23.9 -> 20.7, 33.2 -> 25.7; 1792: 18.4 -> 15.6, 18.5 -> 15.4, 27.0 -> 22.2, 25.0 -> 20.0, 37.6 -> 26.4.
static bool assigns_by_tiles(const Batch& bt, int dk, int k_dt) {
    return k_dt == PACT_BF16 && dk * 2 > 2048 && (dk * 2 >= 3584 || (long)bt.n_max * dk * 2 >= 6000000);
}
static int launch_assign_tiles(const Batch& bt, NearArgs a, const float* rinv, hipStream_t st) {
    a.rinv = rinv;
    PACT_LAUNCH("assign", assign_tile_kernel, dim3((bt.n_max + 127) / 128 * 8, bt.B), dim3(512), st, bt, a, assign_tile_margin(a.dk));
    return PACT_OK;
}

// Stand-alone pact_reincorporate: totals of recovered / dropped tokens (the fused path gets
// them from the cluster sizes).  grid (B), block 1024.
__global__ __launch_bounds__(1024) void count_recovered_kernel(Batch bt, pact_report* rep,
                                                               const int32_t* __restrict__ pruned_idx,
                                                               const int32_t* __restrict__ cluster_id) {
    __shared__ int s_tot;
    const int b = blockIdx.x;
    const Seg sg = bt.s[b];
    const int q = clamp_count(rep[b].n_kept, sg.n), np = clamp_count(rep[b].n_pruned, sg.n - q);
    if (threadIdx.x == 0) s_tot = 0;
    __syncthreads();
    int loc = 0;
    for (int t = threadIdx.x; t < np; t += 1024) loc += cluster_id[sg.base + pruned_idx[sg.base + t]] >= 0;
    loc = (int)wave_sum_f64((double)loc);
    if ((threadIdx.x & 63) == 0 && loc) atomicAdd(&s_tot, loc);
    __syncthreads();
    if (threadIdx.x == 0) { rep[b].n_reincorporated = s_tot; rep[b].n_dropped = np - s_tot; }
}

// ------------------------------------------------------------------------------------------
int launch_centres(const Batch& bt, const Ws& w, const void* keys, pact_dtype k_dt, int32_t dk,
                   const int32_t* idx, int32_t* center_idx, int32_t* cluster_id,
                   int32_t* cluster_counts, pact_report* rep, double* rho_opt, int32_t* rank_opt,
                   int stat_words, bool assign_now, hipStream_t st) {
    const char* k = (const char*)keys;
    CentresArgs ca;
    std::memset(&ca, 0, sizeof(ca));
    ca.keys = k; ca.dk = dk; ca.idx = idx; ca.nn = w.nn; ca.rep = rep; ca.adj = w.adj; ca.rho = w.rho; ca.rho_opt = rho_opt;
    ca.preds = w.preds; ca.heads = w.heads; ca.tie_list = w.tie_list; ca.tie_cnt = w.tie_cnt; ca.rho_fix = w.rho_fix;
    ca.status = w.status; ca.cnum = w.cnum; ca.cmask = w.cmask; ca.center_idx = center_idx;
    ca.write_rho = rank_opt ? 1 : 0;
    ca.idx_ahead = assign_now ? w.ident : idx;               // (assign_now: a stand-alone call, on a caller's list or on w.ident)
    // at most a workgroup per CU in all
    auto launch_selection = [&](const char* name, auto kernel, size_t& raised, size_t lds, long workers, auto... more) -> int {
        if (workers > 256 - bt.B) workers = 256 - bt.B;
        if (lds < RECHECK_LDS) lds = RECHECK_LDS;
        if (lds > 48 * 1024 && lds > raised) {
            if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
                return PACT_ERR_HIP;
            raised = lds;
        }
        PACT_LAUNCH_SHMEM(name, kernel, dim3(bt.B + workers), dim3(1024), lds, st, bt, ca, more...);
        return PACT_OK;
    };
    static size_t raised[4] = {};
    const bool narrow = dk * (k_dt == PACT_BF16 ? 2 : 4) <= SMALL_SETTLE_CHUNKS * 16, small = selects_in_one(bt, narrow);
    if (!small || !narrow) {
        const bool wide = (size_t)dk * (k_dt == PACT_BF16 ? 2 : 4) > 2048;
        dim3 gset(settle_blocks(bt.n_max, wide), bt.B);
        const bool one = near_parts(bt.n_max, bt.B) == 1;
#define PACT_SETTLE(DT, CH)                                                                                           \
        PACT_LAUNCH("settle", (one ? settle_kernel<DT, CH, 1> : settle_kernel<DT, CH, NEAR_PARTS>), gset, dim3(256), st, bt, k, dk, idx, \
                    w.nn, w.near_list, w.near_cnt, w.stat, stat_words, w.rho, w.rho_lo, w.adj, rep)
        if (k_dt == PACT_BF16) { if (wide) PACT_SETTLE(PACT_BF16, 8); else PACT_SETTLE(PACT_BF16, 2); }
        else { if (wide) PACT_SETTLE(PACT_F32, 8); else PACT_SETTLE(PACT_F32, 2); }
#undef PACT_SETTLE
    }
    if (small) {
        // (see there)
        long workers = 0, one_turn = 0;
        for (int b = 0; b < bt.B; ++b) {
            workers += (bt.s[b].n + 31) / 32;
            one_turn += (kept_estimate(bt.s[b]) + 63) / 64;
        }
        if (workers > SMALL_WORKERS) workers = one_turn > SMALL_WORKERS ? one_turn : SMALL_WORKERS;
        SmallArgs sa{narrow ? w.near_list : nullptr, w.near_cnt, w.stat, stat_words, w.rho_lo};
        const int rc = k_dt == PACT_BF16 ? launch_selection("centres", select_small_kernel<PACT_BF16>, raised[0], small_lds(bt.W), workers, sa)
                                         : launch_selection("centres", select_small_kernel<PACT_F32>, raised[1], small_lds(bt.W), workers, sa);
        if (rc) return rc;
    } else {
        // One wavefront per kept token while the chip holds them all at once (32 per CU); beyond that four
        // tokens per wavefront (one image: 7.3 us against 9.5 us; 8 videos: 14.2 against 9.9 us).
        if (kept_estimate(bt) <= 256 * 32)
            PACT_LAUNCH("build_preds", build_preds_kernel<64>, dim3((bt.n_max + 3) / 4, bt.B), dim3(256), st, bt, rep, w.adj, w.rho,
                        rho_opt, w.preds, w.heads, idx, w.tie_list, w.tie_cnt);
        else
            PACT_LAUNCH("build_preds", build_preds_kernel<16>, dim3((bt.n_max + 15) / 16, bt.B), dim3(256), st, bt, rep, w.adj, w.rho,
                        rho_opt, w.preds, w.heads, idx, w.tie_list, w.tie_cnt);
        // (without a second turn up to four tiles of 16 listed tokens in each sample)
        long workers = 0;
        for (int b = 0; b < bt.B; ++b) workers += (bt.s[b].n + 15) / 16;
        const size_t lds = rounds_lds(bt.n_max, bt.W);
        const int rc = k_dt == PACT_BF16 ? launch_selection("centres", centres_kernel<PACT_BF16>, raised[2], lds, workers)
                                         : launch_selection("centres", centres_kernel<PACT_F32>, raised[3], lds, workers);
        if (rc) return rc;
    }
    if (rank_opt)          // (after the fp64 densities are in place)
        PACT_LAUNCH("density_rank", rank_kernel, dim3((bt.n_max + 63) / 64, bt.B), dim3(1024), st, bt, rep,
                    w.rho, rank_opt);
    if (!assign_now) return PACT_OK;          // the caller runs it with the recovery (launch_reincorporate)
    NearArgs a;
    std::memset(&a, 0, sizeof(a));
    a.rep = rep; a.keys = k; a.dk = dk; a.nn = w.nn; a.adj = w.adj; a.margin = (float)cos_margin(dk, k_dt);
    a.cluster_id = cluster_id; a.cluster_counts = cluster_counts;
    a.idx = idx; a.cmask = w.cmask; a.status = w.status; a.cnum = w.cnum;
    if (assigns_by_tiles(bt, dk, k_dt)) return launch_assign_tiles(bt, a, w.rinv, st);
    a.assign_blocks = 1;
    return launch_nearest(bt, a, 0, k_dt, "assign", st);
}

int launch_gram_candidates(const Batch& bt, const Ws& w, const void* keys, pact_dtype k_dt, int32_t dk,
                           const int32_t* pruned_idx, const int32_t* center_idx, pact_report* rep,
                           hipStream_t st);

// Where the recovery finds its candidates itself (candidates_16).  That saves a launch, 5 to 6 us; a turn of 256 centres - half of the kept tokens and
// more are centres - costs 3, the rows of all of them by one compute unit 2 to 4.  So up to 512 kept tokens and 256 KB of rows, with fp32 keys 320
// and 96 KB, and 12 MB over all workgroups.  Calls, us won by it, by kept tokens, lambda = 0.3 / 0.45:
//   width 128: 300 to 500: 2.0, 0.4, 0.3 to 1.3 / 1.3 to 3.4; 511: 0.3 / 1.6 to 2.4; 560: -1.0 / 1.5; 600 to 717: -0.6, 0.1, -0.5, -1.8; 2 samples of 416 to 511: 1.3 to
//   2.6 / 0.9 to 3.2, 4: 2.0 to 2.6 / 1.4, -1.6, 3.1; fp32 keys 300: 1.7 / 1.9, 330 (2, 4 samples): 1.1, 1.9 / 1.1, 1.6, 350: -0.7 / 2.2, 400: -0.8 / 1.9;
//   width 512, lambda = 0.45: 140 to 220 kept: 2.0 to 3.3, 256 (256 KB): 0.9, 2 samples 6.8, 300: 0.8; fp32 keys 60 (92 KB): 0.6, 66 to 80: 1.3 to 1.6, 4 to 16 samples of 64
//   to 80: -0.6 to 1.0, 100: -0.1, 128: -0.5;
//   the two passes alone, 16 of 729 17.3 -> 19.6, 64 of 300 22.1 -> 24.2, 64 of 200 19.0 -> 18.3 (10 MB), with fp32 keys 18.4 -> 21.0 (15 MB).
static bool finds_candidates_there(const Batch& bt, int dk, int k_dt) {
    if (bt.n_max > SMALL_TOKENS) return false;
    const bool f32 = k_dt == PACT_F32;
    const long row = f32 ? (dk + 63) / 64 * 192l : dk * 2l;
    long all = 0;
    for (int b = 0; b < bt.B; ++b) {
        const long pruned = prune_rank(bt.s[b].lambda, bt.s[b].n), kept = bt.s[b].n - pruned;
        if (kept > (f32 ? 320 : 512) || kept * row > (f32 ? 96 : 256) * 1024) return false;
        all += (pruned + 15) / 16 * kept * row;
    }
    return all <= 12 * 1024 * 1024;
}

// kept_idx != nullptr: the assignment of the kept tokens (deferred by launch_centres) runs in the
// same launch as the recovery.
int launch_reincorporate(const Batch& bt, const Ws& w, const void* keys, pact_dtype k_dt, int32_t dk,
                         const int32_t* pruned_idx, const int32_t* center_idx, int32_t* cluster_id,
                         int32_t* cluster_counts, pact_report* rep, bool count_totals,
                         const int32_t* kept_idx, hipStream_t st) {
    const bool here = finds_candidates_there(bt, dk, k_dt);
    int rc = here ? PACT_OK : launch_gram_candidates(bt, w, keys, k_dt, dk, pruned_idx, center_idx, rep, st);
    if (rc != PACT_OK) return rc;
    NearArgs a;
    std::memset(&a, 0, sizeof(a));
    a.rep = rep; a.keys = (const char*)keys; a.dk = dk; a.nn = w.nn; a.adj = w.adj;
    a.margin = (float)cos_margin(dk, k_dt);
    a.cluster_id = cluster_id; a.cluster_counts = cluster_counts;
    a.pruned_idx = pruned_idx; a.center_idx = center_idx; a.cbest = w.cbest;
    if (here) { a.rinv = w.rinv; a.planes = w.ksplit; }
    if (kept_idx) {
        a.idx = kept_idx; a.cmask = w.cmask; a.status = w.status; a.cnum = w.cnum;
        a.assign_blocks = 1;
        a.slots = w.slots; a.big = w.big;     // (a full reduction: the merge follows)
    }
    if ((rc = launch_nearest(bt, a, (bt.n_max + 15) / 16, k_dt, "reinc_assign", st))) return rc;
    if (count_totals)
        PACT_LAUNCH("count_recovered", count_recovered_kernel, dim3(bt.B), dim3(1024), st, bt, rep,
                    pruned_idx, cluster_id);
    return PACT_OK;
}

}  // namespace pact
