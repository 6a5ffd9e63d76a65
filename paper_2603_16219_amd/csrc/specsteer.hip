// SpecSteer verify-and-recover block for MI355X (gfx950): HIP kernels and the C ABI.
//
// What is computed (Algorithm 1 phases 2-3, Eq. 7, Eq. 8) is stated in
// include/specsteer.h.  How it is computed here:
//
//   row_lse        the dominant, HBM-bound pass.  Every valid row of G and S_noctx is
//                  cut into slices; one 64-lane wavefront streams one slice with
//                  non-temporal 16-byte loads and keeps a per-lane running (E, s) with
//                  sum_v 2^(h_v*c - E) = s,  c = log2(e)/T,  E an integer >= max(h*c).
//                  An integer reference makes every rescale an exact ldexp and costs
//                  no extra exponential: one v_exp_f32 per logit.  Waves never
//                  synchronise with each other (no barrier in the loop); a persistent
//                  grid strides over the slice list.  A ragged batch's row list is an
//                  exclusive scan of the draft lengths that every workgroup rebuilds in
//                  LDS at kernel start (prep_rows does it once in global memory for
//                  batches too large for LDS).
//   accept_recover one workgroup per sequence, or several.  Each (position, tensor) pair
//                  gets 16 lanes that merge the row's slice partials and take the draft
//                  token's logit, left there by the row pass; wave 0 applies the ratio test and finds the first
//                  rejection with a ballot.  All waves then stream the three logit rows
//                  of the rejected (or bonus) position once, forming the recovery
//                  exponent in double (in fp32, as the row pass does, when beta == 0 leaves
//                  no steering term), and record one (E, s) mass per 2048-logit chunk
//                  in LDS.  A double-precision scan over the chunk masses locates the
//                  chunk holding u*Z; only that chunk is read again, by four waves, to pick the
//                  token.
//                  Batches of at most 128 sequences share each recovery row between
//                  several workgroups; the one that delivers its chunk masses last
//                  draws the token (see accept_recover_kernel; hand-over by write-through
//                  stores and an arrival counter, without cache-wide fences).
//   block_once     small blocks in one launch: the row pass's partials and the recovery masses of every position, and the rest by the
//                  workgroup that delivers last
//   row_mass, row_draw  accept_recover without drafts, for rows too long for one workgroup each: the chunk masses, and the draw;
//                  row_draw also writes the full log-prob rows beside the draw, on request
//   recovery_logprob  the full log-prob rows where no workgroup shares a recovery row, a second sweep over the rows at n_b
//
// Precision: logits are widened exactly; sums of exponentials are accumulated in
// fp32 (one rounding per term, pairwise across lanes), every per-row scalar
// (log-sum-exp combine, log-probs, alpha, CDF walk across chunks) is double.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "device_common.h"
#include "plan.h"
#include "specsteer.h"
#include "unbound.h"
#include "words.h"

namespace {

constexpr int kLseThreads = 256;            // 4 independent waves per workgroup
constexpr int kEInit = -(1 << 29);          // "no logit seen yet" exponent reference
constexpr float kEClamp = 5.0e8f;           // keeps (int)ceil(h*c) inside int32 for any finite h
constexpr double kLn2 = 0.693147180559945309417232121458;
constexpr double kLog2e = 1.442695040888963407359924681002;

// every memory operation this wave has issued so far has completed: s_waitcnt vmcnt(0) lgkmcnt(0)
__device__ __forceinline__ void wait_stores() { __builtin_amdgcn_s_waitcnt(0x0070); }

// ------------------------------------------------------------------ online sum of exponentials

struct Acc {
    int E;
    float s;
};

__device__ __forceinline__ int exp_ref(float scaled_max) {
    return (int)ceilf(fminf(fmaxf(scaled_max, -kEClamp), kEClamp));
}

// fp32 path of the row pass: term = 2^(h*c_hi - E), c_hi = fl32(c).  The rounding of c would cost
// |h/T| * 2^-24 in the log-sum; it is repaid when the partials are merged: with z = h*c_hi - E
// the missing factor is 2^((z + E)*rho), rho = (c - c_hi)/c_hi ~ 2^-25, and the terms that carry
// the sum have |z| of a few units, so adding E*rho to the row's log2-sum leaves ~|z|*rho < 1e-6.
template <int N>
__device__ __forceinline__ void acc_add_f32(Acc& a, const float (&h)[N], float c_hi) {
    float m = h[0];
#pragma unroll
    for (int i = 1; i < N; ++i) m = fmaxf(m, h[i]);
    const int En = max(a.E, exp_ref(m * c_hi));
    a.s = ldexpf(a.s, a.E - En);
    a.E = En;
    const float nE = -(float)En;
    float t0 = 0.f, t1 = 0.f;
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        t0 += __builtin_amdgcn_exp2f(fmaf(h[i], c_hi, nE));
        if (i + 1 < N) t1 += __builtin_amdgcn_exp2f(fmaf(h[i + 1], c_hi, nE));
    }
    a.s += t0 + t1;
}

// The steering difference h_SLM^+ - h_SLM^- of Eq. 8.  A token masked (-inf) in both specialist rows
// carries no steering -- 0, not inf - inf; for equal finite logits the result is the same 0 as before.
__device__ __forceinline__ float steer_diff(float sp, float sm) { return sp == sm ? 0.f : sp - sm; }
__device__ __forceinline__ double steer_diff_d(float sp, float sm) { return sp == sm ? 0.0 : (double)sp - (double)sm; }

// recovery logit in the base-2 exponent domain: y = (G + beta*(S_ctx - S_noctx)) * log2(e)/T, in double.
__device__ __forceinline__ double rec_y(float g, float sp, float sm, double c, double bc) {
    return fma((double)g, c, steer_diff_d(sp, sm) * bc);
}

// Recovery pass accumulate.  The exponent reference is advanced from a cheap fp32 estimate of
// this vector's maximum; the term exponents themselves are formed in double,
//     z = g*c + (sp - sm)*beta*c - E   (two fused multiply-adds, E folded into the first),
// so the only roundings are the final conversion of the small number z to fp32 and the
// exponential.  sp - sm is taken in fp32: exact for bf16 inputs whose exponents differ by
// less than 16 (otherwise the smaller one is below 2^-16 of the larger and the difference
// rounds by at most 2^-25 of it); fp32 inputs widen first.
// Greedy decoding needs argmax of Eq. 8 itself: h_LLM + beta*(h_SLM^+ - h_SLM^-) as one exact
// difference, one rounded product and one rounded sum in double -- the same three operations
// the definition spells out, so the winner is reproducible bit for bit.  Strict '>' keeps the
// lowest index, because a lane meets its logits in increasing vocabulary order.
struct Best {
    double v;
    int idx;
};
constexpr int kNoBest = 0x7FFFFFFF;

// Running maximum over the N logits of one vector of a lane, then against the lane's best: with the place in the vector as
// what is carried, a logit costs a compare and three selects (and one of each without a steering term, where the logits are
// compared as they are), where a 64-bit row index carried from logit to logit took two selects and an addition more.  Bound by
// the vector ALU where rows are many: 1500 greedy rows of V = 128256 bf16 without a steering term 80.3 -> 67.0 us, steered
// 196.5 -> 190.0, 200 without 19.2 -> 15.9; a step of 512 sequences of V = 256000 295.9 -> 293.9, of 32 in fp32 41.1 -> 40.9.
template <int N, typename T>
__device__ __forceinline__ void best_of(Best& best, const T (&h)[N], int first) {
    T v = -__builtin_huge_valf();
    int at = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (h[i] > v) {
            v = h[i];
            at = i;
        }
    if ((double)v > best.v) {
        best.v = (double)v;
        best.idx = first + at;
    }
}

template <int DT, int N, bool GREEDY>
__device__ __forceinline__ void acc_add_rec(Acc& a, const float (&hg)[N], const float (&hp)[N], const float (&hm)[N],
                                            double c, double bc, float cf, float bcf, double beta, int first,
                                            Best& best) {
    if (GREEDY) {
        double hr[N];
#pragma unroll
        for (int i = 0; i < N; ++i) hr[i] = __dadd_rn((double)hg[i], __dmul_rn(beta, steer_diff_d(hp[i], hm[i])));
        best_of<N>(best, hr, first);
    }
    float d[N];
    float m = -3.0e38f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        d[i] = steer_diff(hp[i], hm[i]);
        m = fmaxf(m, fmaf(hg[i], cf, d[i] * bcf));
    }
    // the estimate is within a few 1e-5 of the exact exponent: half a unit of slack keeps z <= ~0.5
    const int En = max(a.E, exp_ref(m));
    a.s = ldexpf(a.s, a.E - En);
    a.E = En;
    const double nE = -(double)En;
    float t0 = 0.f, t1 = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double dd = (DT == SS_BF16) ? (double)d[i] : steer_diff_d(hp[i], hm[i]);
        const float z = (float)fma((double)hg[i], c, fma(dd, bc, nE));
        if (i & 1) t1 += __builtin_amdgcn_exp2f(z); else t0 += __builtin_amdgcn_exp2f(z);
    }
    a.s += t0 + t1;
}

__device__ __forceinline__ Partial wave_combine(Acc a) {
    const int Em = wave_max_i32(a.E);
    const float S = wave_sum_f32(ldexpf(a.s, a.E - Em));
    return Partial{Em, S};
}

// ------------------------------------------------------------------ row lists

// Which rows a row pass covers: positions [t_lo, t_hi) of every sequence that is still in play.
// The block is verified in one or more such windows (see the host side): Algorithm 1 stops at the
// first rejection, so the later positions of a sequence rejected early never need their rows.
struct RowWindow {
    const int32_t* draft_len;  // NULL => K_b = k_max
    const int32_t* state;      // NULL => every sequence; else rows only where state[b] == kInPlay
    int kmax, t_lo, t_hi;
};

// In the place of a draft token's logit: its id is outside the vocabulary.  A NaN that no bf16 logit is widened to.
constexpr unsigned kNoToken = 0x7FC0BAD1u;

// What the verdict kernel leaves per sequence: its first-rejection index (>= 0; final, Algorithm 1 has left its
// loop), or one of
constexpr int kInPlay = -1;   // nothing rejected so far and positions left to test
constexpr int kFlagged = -2;  // length or a draft id out of range

// Rows of sequence b inside the window.  A length outside [0, k_max] contributes none
// (the sequence is flagged elsewhere).
__device__ __forceinline__ int window_rows(const RowWindow& w, int b) {
    const int K = w.draft_len ? w.draft_len[b] : w.kmax;
    if (K < 0 || K > w.kmax) return 0;
    if (w.state && w.state[b] != kInPlay) return 0;
    return max(0, min(K, w.t_hi) - w.t_lo);
}

// off[b] = number of window rows before sequence b; off[B] = total.
// Called by every thread of a workgroup of NT threads (NT a multiple of 64, at most 1024);
// `off` may be LDS or global memory.  Ends with a barrier, so `off` is readable on return.
__device__ __forceinline__ void block_scan_rows(const RowWindow& win, int B, int* off, int NT) {
    __shared__ int wave_tot[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, NW = NT >> 6;
    int carry = 0;
    for (int b0 = 0; b0 < B; b0 += NT) {
        const int b = b0 + tid;
        const int k = b < B ? window_rows(win, b) : 0;
        int incl = k;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int y = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += y;
        }
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        int before = carry, all = 0;
        for (int w = 0; w < NW; ++w) {
            const int wt = wave_tot[w];
            if (w < wave) before += wt;
            all += wt;
        }
        if (b < B) off[b] = before + incl - k;
        carry += all;
        __syncthreads();
    }
    if (tid == 0) off[B] = carry;
    __syncthreads();
}

// Only for batches too large for the in-kernel LDS row list.
__global__ __launch_bounds__(1024) void prep_rows_kernel(const RowWindow win, int B, int32_t* __restrict__ row_off) {
    block_scan_rows(win, B, row_off, 1024);
}

// ------------------------------------------------------------------ kernel: row log-sum-exp partials

struct LseArgs {
    const void* G;
    const void* Sm;
    RowWindow win;             // the rows this launch covers
    int uniform_rows;          // > 0: every sequence has exactly this many window rows, no list needed
    const int32_t* row_off;    // else: the row list, [B+1], of a batch too large for the one in LDS
    Partial* partial;          // [B][win.t_hi - win.t_lo][2][NS]
    const int32_t* draft;
    float* draft_logit;        // [B][kmax][2] the draft token's logit in each tensor, or kNoToken; NULL: gathered by who needs it
    long sb, st;               // element strides
    int B, kmax, V, NS;
    int slice_vecs;            // 16-byte vectors per slice
    int list_in_lds;           // build the row list in LDS (else row_off was filled by prep_rows)
    float c_hi;                // fl32(log2(e)/T)
    uint32_t* zero_ptr;        // arrival counters of a split recovery: workgroup 0 clears zero_n of them
    int zero_n;
};

// Work item = (row, tensor, slice), flattened so that consecutive items are consecutive slices
// of one row.  One wave per item, no communication between waves; the grid is persistent and
// strides over the item list.  Ragged batches build the row list in LDS at kernel start
// (every workgroup repeats the same small scan), so no separate launch is needed.
// The wave that meets the draft token's vector leaves its logit beside the partials: it is in registers here, while the
// ratio test would gather it from HBM behind the load of the draft id, a round trip that every sequence of that launch
// waits for.  The id itself is looked at behind the item's first loads: before them it cost 300 ragged sequences 2 us.
// For an id outside the vocabulary the first slice leaves kNoToken, so that the ratio test needs no ids at all.
// Loads and stores of the vector memory are counted together, so that an item which begins with a wait for a load begins with one for
// the stores of the item before: with the id as a vector load, or the row list behind one pointer to LDS or global memory, all did.
// Slices of one group of loads are done sooner without it (64 sequences of 8 drafts, V = 32000 28.0 -> 26.8 us a step, 128 45.1 ->
// 42.9, 13 of 16 in fp32, V = 38784 24.7 -> 23.2, 64 ragged ones of 16, V = 32000 30.6 -> 29.4), and where a wave has few items (8 of V =
// 151936 19.0 -> 18.7).  Else rows stream faster with it, in the order that it keeps the waves in (without -> with: 64 of V = 151936
// 67.8 -> 66.8, of 100000 50.5 -> 49.8, 256 ragged ones of V = 50257 63.8 -> 63.4, 512 of 256000 601.5 -> 596.8), and wait as a rule.
template <int DT, int VEC, int kUnroll>
__global__ __launch_bounds__(kLseThreads) void row_lse_kernel(const LseArgs a) {
    extern __shared__ int lds_off[];
    const int lane = threadIdx.x & 63;
    const int wave_global = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kLseThreads / kWave) + (threadIdx.x >> 6)));
    const int waves_total = gridDim.x * (kLseThreads / kWave);
    const bool ragged = a.uniform_rows <= 0;
    if (ragged && a.list_in_lds) block_scan_rows(a.win, a.B, lds_off, kLseThreads);
    const auto* const lds_list = (const __attribute__((address_space(3))) int*)lds_off;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < a.zero_n; i += kLseThreads) a.zero_ptr[(long)i * kArriveStride] = 0u;
    const int R = ragged ? __builtin_amdgcn_readfirstlane(a.list_in_lds ? lds_off[a.B] : a.row_off[a.B]) : a.B * a.uniform_rows;
    const long slice_units = a.slice_vecs;
    constexpr long kGroup = (long)kWave * kUnroll;

    // The wave's items are waves_total apart: slice and row go on from those before without a division, and the sequence of
    // a ragged batch's row is looked up from the last one on, first among the next 64, then among 64 places that part all
    // that are left.  Divisions in 64 bits and a search by halves, eight
    // dependent reads of LDS, stood before the first load of every item, which counts where items are short: 16 sequences of up to
    // 8 positions 26.2 -> 25.1 us a step, 40 ragged ones 31.6 -> 30.4, 300 131.5 -> 129.5, 256 of V = 128256 164.2 -> 162.7.  64 at a
    // time to the end lost to halves where the rows of a wave lie thousands of sequences apart (the list in global memory; by halves,
    // 64 at a time, now): 58940 sequences of up to 16 positions, V = 2398 2658, 3146 and 2204 us, 27250 of 2, V = 7168 647, 717, 604,
    // 8000 of 16, V = 8000 625, 629, 599.
    const unsigned NS = (unsigned)a.NS;
    unsigned k_ = (unsigned)wave_global % NS, rx = (unsigned)wave_global / NS;
    const unsigned dk = (unsigned)waves_total % NS, drx = (unsigned)waves_total / NS;
    const bool in_order = slice_units > kGroup && 2u * (unsigned)R >= 4u * drx;  // more than one group of loads, four items a wave
    int b = 0, off_b = 0;  // ragged: the sequence of the row before, and its first row
    for (; rx < 2u * (unsigned)R; k_ += dk, rx += drx) {
        if (k_ >= NS) {
            k_ -= NS;
            if (++rx >= 2u * (unsigned)R) break;
        }
        const int k = (int)k_, x = (int)(rx & 1u), r = (int)(rx >> 1);
        if (in_order) wait_stores();
        int t;
        if (ragged) {
            // the largest b with off[b] <= r; off[B] = R > r.  Beyond the next 64, the 64 places that part what is left evenly
            int hi = a.B, step = 1;
            for (;;) {
                int n;
                const auto look = [&](const auto* list) {
                    const int o = list[min(b + step * (1 + lane), hi)];
                    n = __popcll(__ballot(o <= r));
                    if (n) off_b = __builtin_amdgcn_readlane(o, n - 1);
                };
                if (a.list_in_lds) look(lds_list); else look(a.row_off);
                b += n * step;
                if (n < kWave) {
                    if (step == 1) break;
                    hi = min(b + step, hi);
                }
                step = (hi - b + kWave - 1) / kWave;
            }
            t = a.win.t_lo + (r - off_b);
        } else {
            b = r / a.uniform_rows;
            t = a.win.t_lo + (r - b * a.uniform_rows);
        }
        const long elem_off = (long)b * a.sb + (long)t * a.st;
        const int y = a.draft_logit ? ld_uniform(a.draft + ((long)b * a.kmax + t)) : -1;  // looked at behind the first loads of the row
        float* const y_out = a.draft_logit + ((long)b * a.kmax + t) * 2 + x;
        const void* row = row_ptr<DT>(x ? a.Sm : a.G, elem_off);
        const int head = __builtin_amdgcn_readfirstlane(odd_head<DT>(row, elem_off));
        row = row_ptr<DT>(row, -(long)head);
        const long nvec = (a.V + head) / VEC;
        const int tailc = a.V + head - (int)(nvec * VEC);
        const bool masked = head && k == 0;  // this slice starts with the element before the row
        const long v0 = (long)k * slice_units;
        const long v1 = min(nvec, v0 + slice_units);
        const long nfull = v1 > v0 ? (v1 - v0) / kGroup : 0;  // wave-uniform trip count
        // the draft token's element in the row as it is read, and its vector counted from the slice's start, < 0 if none of this slice
        int ye = -1, yv = -1;
        const auto find_y = [&]() {
            ye = y >= 0 && y < a.V ? y + head : -1;
            if (ye < 0 && a.draft_logit && k == 0 && lane == 0) *y_out = __uint_as_float(kNoToken);
            yv = ye >= 0 && ye / VEC < v1 ? ye / VEC - (int)v0 : -1;
        };

        Acc acc{kEInit, 0.f};
        long v = v0 + lane;
        for (long g = 0; g < nfull; ++g, v += kGroup) {
            typename RawT<DT, VEC>::type raw[kUnroll];
#pragma unroll
            for (int j = 0; j < kUnroll; ++j) raw[j] = ld_raw<DT, VEC>(row, v + (long)kWave * j);
            if (g == 0) find_y();
            if (yv >= 0 && yv / (int)kGroup == (int)g) {
                float hy = 0.f;
#pragma unroll
                for (int j = 0; j < kUnroll; ++j) {
                    const float hj = elem_of(raw[j], ye % VEC);
                    hy = yv % (int)kGroup / kWave == j ? hj : hy;
                }
                if (yv % kWave == lane) *y_out = hy;
            }
            if (masked && g == 0 && lane == 0) raw[0] = set_first(raw[0], kBf16NegInf);
            float h[kUnroll * VEC];
#pragma unroll
            for (int j = 0; j < kUnroll; ++j) {
                float hj[VEC];
                unpack(raw[j], hj);
#pragma unroll
                for (int i = 0; i < VEC; ++i) h[j * VEC + i] = hj[i];
            }
            acc_add_f32<kUnroll * VEC>(acc, h, a.c_hi);
        }
        if (nfull == 0) find_y();
        // Less than a group, the end of a row, where slices are one group or two: all its loads in flight at once, those past it -inf.  A vector
        // at a time they were up to three round trips behind each other in one item of eight or sixteen (96 sequences of 8 drafts, V = 32000
        // 35.0 -> 30.9 us a step, 64 of 4 19.7 -> 18.2, 500 of 4 69.3 -> 64.7, 160 ragged of 8 32.6 -> 31.0, 20 of 8, V = 50257 18.7 -> 18.3).  Behind
        // the groups of longer slices other waves cover them, and the sums over logits that are not there cost more (256 ragged of V = 50257
        // 61.7 -> 62.6), as they do for a single load a lane.  Two loads a lane are a group of two: as one of four, half of
        // it not there, they took many short rows longer than a vector at a time did (us a step a vector at a time, as a group of four, of two:
        // 296 sequences of 34 drafts, V = 545 26.1, 28.0, 25.4, 397 of 63, V = 976 48.6, 50.9, 44.9, 211 of 32, V = 4648 37.7, 39.1, 37.2).
        const auto take_end = [&](auto loads) {
            constexpr int N = decltype(loads)::value;
            typename RawT<DT, VEC>::type raw[N];
            float h[N * VEC];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                raw[j] = neg_inf_raw<DT, VEC>();
                if (v + (long)kWave * j < v1) raw[j] = ld_raw<DT, VEC>(row, v + (long)kWave * j);
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (yv >= 0 && v + (long)kWave * j == v0 + yv) *y_out = elem_of(raw[j], ye % VEC);
                if (j == 0 && masked && v == 0) raw[0] = set_first(raw[0], kBf16NegInf);
                float hj[VEC];
                unpack(raw[j], hj);
#pragma unroll
                for (int i = 0; i < VEC; ++i) h[j * VEC + i] = hj[i];
            }
            acc_add_f32<N * VEC>(acc, h, a.c_hi);
            v = v1;
        };
        const long rest = v1 - v0 - nfull * kGroup;
        if (slice_units <= 2 * kGroup && rest > kWave) {
            if (rest <= 2 * kWave) take_end(std::integral_constant<int, 2>{});
            else take_end(std::integral_constant<int, kUnroll>{});
        }
        for (; v < v1; v += kWave) {
            typename RawT<DT, VEC>::type raw = ld_raw<DT, VEC>(row, v);
            if (yv >= 0 && v == v0 + yv) *y_out = elem_of(raw, ye % VEC);
            if (masked && v == 0) raw = set_first(raw, kBf16NegInf);
            float hj[VEC];
            unpack(raw, hj);
            acc_add_f32<VEC>(acc, hj, a.c_hi);
        }
        if (k == a.NS - 1 && lane < tailc && !(head && nvec == 0 && lane == 0)) {  // logits past the last full vector
            float hj[1] = {ld_elem<DT>(row, nvec * VEC + lane)};
            if (ye == nvec * VEC + lane) *y_out = hj[0];
            acc_add_f32<1>(acc, hj, a.c_hi);
        }
        const Partial p = wave_combine(acc);
        if (lane == 0) a.partial[(((long)b * (a.win.t_hi - a.win.t_lo) + (t - a.win.t_lo)) * 2 + x) * a.NS + k] = p;
    }
}

// ------------------------------------------------------------------ kernel: accept + recover

struct RecArgs {
    const void* G;
    const void* Sm;          // S_noctx, for the ratio test
    const void* recSp;       // S_ctx and S_noctx as the recovery sweep reads them: both alias G when
    const void* recSm;       //   beta == 0, so that the steering term is an exact zero and costs no HBM traffic
    const int32_t* draft;
    const int32_t* draft_len;
    const float* uniforms;
    const Partial* partial;  // slice partials of the window this launch tests, [B][t_hi - t_lo][2][NS]
    const float* draft_logit;  // [B][kmax][2] the draft tokens' logits (kNoToken: not in the vocabulary), or NULL: gathered from the rows
    int NS;                  // slices per row
    int t_lo, t_hi;          // the window; t_hi == k_max for the last one
    int32_t* state;          // several windows: what the verdicts so far have found; else NULL
    int32_t* accepted_len;
    int32_t* next_token;
    float* next_token_logprob;
    double* log2z;           // [B] log2 of the recovery row's normaliser, for a launch that writes the log-prob rows; else NULL
    float* recovery_logprobs;  // [B, V] log-prob rows if this launch writes them itself; else NULL
    float* draft_logprobs;
    long sb, st;
    int B, kmax, V;
    int NC;          // most chunks of a row (full chunks + one pseudo-chunk for the logits past the last vector)
    double c;        // log2(e) / T
    double bc;       // beta * log2(e) / T
    double beta;     // beta itself, for the greedy argmax of Eq. 8
    double lambda;
    double rho;      // (c - fl32(c)) / fl32(c): first-order repair of sums formed with the rounded scale
    float c_hi;      // fl32(c)
    int greedy;      // SS_FLAG_GREEDY
    int plain;       // beta == 0: no steering term, the specialist rows are not read by the recovery sweep
    // Small batches: `parts` workgroups share the recovery row of one sequence.
    int parts, part_chunks;  // part i takes chunks [i * part_chunks, (i+1) * part_chunks)
    int defer;            // the parts only deliver: row_draw_kernel draws, and writes the log-prob rows in segs workgroups a row
    int segs;
    Partial* chunk_tab;   // [B][NC] chunk masses, filled by the parts
    double* best_v;       // [B][NC] greedy candidates of the parts: value ...
    int32_t* best_i;      // [B][NC] ... and token
    uint32_t* arrive;     // [B][kArriveStride] parts that have delivered; cleared by the first row pass
};

// Hand-over between workgroups that may run on different XCDs, whose L2 caches are not coherent with each
// other, without a cache-wide write-back (a device-scope release fence writes the whole L2 back and costs about
// 40 ns of a serialised resource per fence): the producer writes with device-scope atomic stores, which go
// through to memory, waits for them to complete, and only then bumps the arrival counter; the workgroup that
// sees the counter complete reads with device-scope atomic loads.  Nobody ever waits for anybody.
template <typename T>
__device__ __forceinline__ void st_dev(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T ld_dev(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_dev_partial(Partial* p, Partial v) {
    st_dev(reinterpret_cast<unsigned long long*>(p),
           ((unsigned long long)__float_as_uint(v.s) << 32) | (unsigned long long)(unsigned)v.E);
}
__device__ __forceinline__ Partial ld_dev_partial(const Partial* p) {
    const unsigned long long w = ld_dev(reinterpret_cast<const unsigned long long*>(p));
    return Partial{(int)(unsigned)(w & 0xFFFFFFFFull), __uint_as_float((unsigned)(w >> 32))};
}

// The slice partials of one row merged by the 16 lanes of one DPP row (`l` is the lane's index in it, every lane
// returns the pair): lane l takes slices l, l+16, ..., four loads in flight, and the 16
// running pairs are merged by a fixed pattern, so the result does not depend on who computes it.  One lane per row
// (all slices in turn) spends a round trip per 16 slices and some 60 clocks per merge: with the 38
// slices of V = 151936 that was a third of the 4.5 us before the first rejection was known.
__device__ __forceinline__ Partial merge_partials_row16(const Partial* p, int ns, int l) {
    int Em = kEInit;
    float S = 0.f;
    for (int k0 = l; k0 < ns; k0 += 64) {
        Partial pv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pv[i] = k0 + 16 * i < ns ? p[k0 + 16 * i] : Partial{kEInit, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int En = max(Em, pv[i].E);
            S = ldexpf(S, Em - En) + ldexpf(pv[i].s, pv[i].E - En);
            Em = En;
        }
    }
    const int Er = row_max_i32(Em);
    return Partial{Er, row_sum_f32(ldexpf(S, Em - Er))};
}

// log2 of sum_v 2^(h_v * c) for one row from its merged partials
__device__ __forceinline__ double row_log2(Partial p, double rho) {
    return (double)p.E * (1.0 + rho) + log2((double)p.s);  // E*rho: see acc_add_f32
}

// PLAIN (beta == 0): the recovery distribution is Softmax(h_LLM / T); the two specialist rows are
// neither loaded nor unpacked, their logits read as 0 so that the steering term is an exact zero.
template <int DT, int VEC, bool PLAIN>
__device__ __forceinline__ void unpack_steer(const typename RawT<DT, VEC>::type& rp, const typename RawT<DT, VEC>::type& rm,
                                             float (&hp)[VEC], float (&hm)[VEC]) {
    if (PLAIN) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) hp[i] = hm[i] = 0.f;
    } else {
        unpack(rp, hp);
        unpack(rm, hm);
    }
}

template <int DT, bool PLAIN>
__device__ __forceinline__ float ld_steer(const void* row, long e) {
    return PLAIN ? 0.f : ld_elem<DT>(row, e);
}

// The three rows of sequence b at position n as the recovery sweep reads them.
template <int DT, int VEC>
struct RecRow {
    const void *g, *sp, *sm;
    int head;        // 1: read from one element before the row
    long nvec, nch;  // full vectors and the chunks they make
    int tailc, NC;   // logits past them, and chunks with those: a.NC or one less
    __device__ __forceinline__ RecRow(const RecArgs& a, int b, int n) {
        const long off = (long)b * a.sb + (long)n * a.st;
        g = row_ptr<DT>(a.G, off);
        sp = row_ptr<DT>(a.recSp, off);
        sm = row_ptr<DT>(a.recSm, off);
        // Rows off 4-byte boundaries are read from one element before, if all three are and a vector is there to mask it in
        head = a.V + 1 >= VEC ? odd_head<DT>(g, off) & odd_head<DT>(sp, off) & odd_head<DT>(sm, off) : 0;
        g = row_ptr<DT>(g, -(long)head);
        sp = row_ptr<DT>(sp, -(long)head);
        sm = row_ptr<DT>(sm, -(long)head);
        nvec = (a.V + head) / VEC;
        tailc = a.V + head - (int)(nvec * VEC);
        nch = (nvec + kWave * kChunkSteps - 1) / (kWave * kChunkSteps);
        NC = (int)nch + (tailc ? 1 : 0);
    }
};

// (E, s) mass of recovery chunk c, or of STEPS of its steps from step0 on, by one wave: sum over the chunk of 2^(y - E).  With a steering term the
// exponent is formed in double (acc_add_rec); PLAIN (beta == 0) has only h_LLM * c to form and takes the
// row pass's route, one fp32 fma per logit with the rounded scale c_hi, repaired to first order by the caller.
template <int DT, int VEC, bool GREEDY, bool PLAIN, int STEPS = kChunkSteps>
__device__ __forceinline__ Partial chunk_mass(const RecRow<DT, VEC>& row, long c, int lane, double cc, double bc, double beta,
                                              float c_hi, Best& best, int step0 = 0) {
    const void *g = row.g, *sp = row.sp, *sm = row.sm;
    const long nvec = row.nvec, nch = row.nch;
    const int tailc = row.tailc, head = row.head;
    const float cf = (float)cc, bcf = (float)bc;
    Acc acc{kEInit, 0.f};
    if (c < nch) {
        const long vbase = (c * kChunkSteps + step0) * kWave + lane;
        typename RawT<DT, VEC>::type rg[STEPS], rp[STEPS], rm[STEPS];
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            const long v = vbase + (long)j * kWave;
            if (v < nvec) {
                rg[j] = ld_raw<DT, VEC>(g, v);
                if (!PLAIN) {
                    rp[j] = ld_raw<DT, VEC>(sp, v);
                    rm[j] = ld_raw<DT, VEC>(sm, v);
                }
            }
        }
        if (head && vbase == 0) {  // the element before the row: masked, no steering
            rg[0] = set_first(rg[0], kBf16NegInf);
            if (!PLAIN) {
                rp[0] = set_first(rp[0], 0u);
                rm[0] = set_first(rm[0], 0u);
            }
        }
        if (PLAIN && vbase + (long)(STEPS - 1) * kWave < nvec) {  // all of it there: one accumulate over its vectors
            float h[STEPS * VEC];
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                float hj[VEC];
                unpack(rg[j], hj);
                if (GREEDY) best_of<VEC>(best, hj, (int)(vbase + (long)j * kWave) * VEC);
#pragma unroll
                for (int i = 0; i < VEC; ++i) h[j * VEC + i] = hj[i];
            }
            acc_add_f32<STEPS * VEC>(acc, h, c_hi);
        } else {
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                const long v = vbase + (long)j * kWave;
                if (v < nvec) {
                    float hg[VEC], hp[VEC], hm[VEC];
                    unpack(rg[j], hg);
                    unpack_steer<DT, VEC, PLAIN>(rp[j], rm[j], hp, hm);
                    if (PLAIN) {
                        if (GREEDY) best_of<VEC>(best, hg, (int)v * VEC);
                        acc_add_f32<VEC>(acc, hg, c_hi);
                    } else {
                        acc_add_rec<DT, VEC, GREEDY>(acc, hg, hp, hm, cc, bc, cf, bcf, beta, (int)v * VEC, best);
                    }
                }
            }
        }
    } else if (lane < tailc && step0 == 0) {
        const long e = nvec * VEC + lane;
        const float hg[1] = {ld_elem<DT>(g, e)}, hp[1] = {ld_steer<DT, PLAIN>(sp, e)}, hm[1] = {ld_steer<DT, PLAIN>(sm, e)};
        if (PLAIN) {
            if (GREEDY) best_of<1>(best, hg, (int)e);
            acc_add_f32<1>(acc, hg, c_hi);
        } else {
            acc_add_rec<DT, 1, GREEDY>(acc, hg, hp, hm, cc, bc, cf, bcf, beta, (int)e, best);
        }
    }
    return wave_combine(acc);
}

// The masses of two chunks of a bf16 row without steering, with the loads of both on their way at once; the first is whole, the second
// with WHOLE, else as far as the row goes.  Bound by latency: a wave with
// one chunk has 4 loads in flight, and sixteen such waves draw 33 GB/s through a compute unit.  64 rows of V = 151936 in
// one 16-wave workgroup each: 14.3 us a call with single chunks, 13.4 with pairs, V = 131072 13.3 -> 12.2.  A wave left with the row's last,
// partial chunk for a round of its own is the last of its workgroup (256 rows of V = 50256 8.52 us on the GPU, 8.12 with that chunk
// paired too, of V = 128256 14.9 -> 14.5).  Not with 8 waves, two workgroups to a unit (512 rows: 28.8 -> 29.3), and not in fp32, whose
// chunks are half the logits: the arithmetic of the others covers their latency (64 rows of V = 50257 9.63 us in pairs, 9.01 without, 256 of V =
// 32768 9.04, 8.54).
template <int DT, int VEC, bool GREEDY, bool WHOLE>
__device__ __forceinline__ void chunk_pair_mass(const RecRow<DT, VEC>& row, const long (&c)[2], int lane, float c_hi, Best& best, Partial (&out)[2]) {
    typename RawT<DT, VEC>::type r[2][kChunkSteps];
    const long end = WHOLE ? 0 : row.nvec;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < kChunkSteps; ++j) {
            const long v = (c[q] * kChunkSteps + j) * kWave + lane;
            if (WHOLE || q == 0 || v < end) r[q][j] = ld_raw<DT, VEC>(row.g, v);
        }
    if (row.head && c[0] == 0 && lane == 0) r[0][0] = set_first(r[0][0], kBf16NegInf);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        Acc acc{kEInit, 0.f};
        const long v0 = c[q] * kChunkSteps * kWave + lane;
        if (WHOLE || q == 0 || v0 + (kChunkSteps - 1) * kWave < end) {
            float h[kChunkSteps * VEC];
#pragma unroll
            for (int j = 0; j < kChunkSteps; ++j) {
                float hj[VEC];
                unpack(r[q][j], hj);
                if (GREEDY) best_of<VEC>(best, hj, (int)((c[q] * kChunkSteps + j) * kWave + lane) * VEC);
#pragma unroll
                for (int i = 0; i < VEC; ++i) h[j * VEC + i] = hj[i];
            }
            acc_add_f32<kChunkSteps * VEC>(acc, h, c_hi);
        } else {
#pragma unroll
            for (int j = 0; j < kChunkSteps; ++j) {
                if (v0 + j * kWave < end) {
                    float hj[VEC];
                    unpack(r[q][j], hj);
                    if (GREEDY) best_of<VEC>(best, hj, (int)(v0 + j * kWave) * VEC);
                    acc_add_f32<VEC>(acc, hj, c_hi);
                }
            }
        }
        out[q] = wave_combine(acc);
    }
}

// log2 of the recovery row's normaliser from the base-2 scale and the sum of the chunk masses on it.  PLAIN sums were
// formed with the rounded scale c_hi: an exponent comes back as y_hi = h * c_hi, the true one is y_hi * (1 + rho), and the
// row's log2-sum moves by rho * E* to first order (see acc_add_f32).
template <bool PLAIN>
__device__ __forceinline__ double mass_log2(const RecArgs& a, int Estar, double total) {
    return (double)Estar + log2(total) + (PLAIN ? a.rho : 0.0) * (double)Estar;
}

// The chunk masses of a recovery row (`tab`, LDS) as one wave sees them: lane l owns a run of `per` consecutive chunks,
// the first HELD of them in registers.
template <int HELD>
struct ChunkScan {
    int lo, hi, Estar;
    double held[HELD];       // masses of chunks lo, lo + 1, ... on the scale 2^Estar; 0 past the run
    double incl, total;      // mass up to the end of this lane's run, and of the row
    const Partial* tab;

    __device__ __forceinline__ double mass(int c) const { return ldexp((double)tab[c].s, tab[c].E - Estar); }
    __device__ __forceinline__ ChunkScan(const Partial* t, int NC, int lane) : tab(t) {
        const int per = (NC + kWave - 1) / kWave;
        lo = min(lane * per, NC);
        hi = min(lo + per, NC);
        Partial p[HELD];
        int Em = kEInit;
#pragma unroll
        for (int i = 0; i < HELD; ++i) {
            p[i] = lo + i < hi ? tab[lo + i] : Partial{kEInit, 0.f};
            Em = max(Em, p[i].E);
        }
        for (int c = lo + HELD; c < hi; ++c) Em = max(Em, tab[c].E);
        Estar = wave_max_i32(Em);
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < HELD; ++i) {
            held[i] = ldexp((double)p[i].s, p[i].E - Estar);
            sum += held[i];
        }
        for (int c = lo + HELD; c < hi; ++c) sum += mass(c);
        incl = wave_incl_scan_f64(sum);
        total = wave_last_f64(incl);
    }
};

// The chunk that holds the share u of a row's mass.
struct Found {
    int c, Estar, last;          // last: u is not below the total (u >= 1 or not a number); c is then the last chunk with any mass
    double base, target, total;  // mass before the chunk, u's share and all of it, on the scale 2^Estar
};
template <int HELD>
__device__ __forceinline__ Found find_chunk_held(const Partial* tab, int NC, int lane, double us) {
    const ChunkScan<HELD> cs(tab, NC, lane);
    Found f;
    f.Estar = cs.Estar;
    f.total = cs.total;
    f.target = us * cs.total;
    f.last = 0;
    f.base = 0.0;
    int cfound = -1, clast = -1;
    double cbase = 0.0, cum = wave_shift_up_f64(cs.incl);
    const auto meet = [&](int c, double m) {
        if (m > 0.0) clast = c;
        const double cum2 = cum + m;
        if (cfound < 0 && cum2 > f.target) {
            cfound = c;
            cbase = cum;
        }
        cum = cum2;
    };
#pragma unroll
    for (int i = 0; i < HELD; ++i)
        if (cs.lo + i < cs.hi) meet(cs.lo + i, cs.held[i]);
    for (int c = cs.lo + HELD; c < cs.hi; ++c) meet(c, cs.mass(c));
    const unsigned long long fmask = __ballot(cfound >= 0);
    if (fmask) {
        const int L = first_lane(fmask);
        f.c = __builtin_amdgcn_readlane(cfound, L);
        f.base = wave_readlane_f64(cbase, L);
    } else {
        f.c = max(wave_max_i32(clast), 0);
        f.last = 1;
    }
    return f;
}

// Two chunks a lane are all there are up to V = 262144 bf16; two more that are not there took the scan 0.15 us (8 sequences of V = 151936 18.4 -> 18.2 us a
// step on the GPU, 16 25.9 -> 25.65, 200 steered rows of V = 128256 30.3 -> 30.0).  Beyond, four: with two held and the rest from LDS 8 sampled rows of
// V = 250000 fp32 took 6.4 us instead of 6.2.
__device__ __forceinline__ Found find_chunk(const Partial* tab, int NC, int lane, double us) {
    return NC <= 2 * kWave ? find_chunk_held<2>(tab, NC, lane, us) : find_chunk_held<4>(tab, NC, lane, us);
}

constexpr int kMassWaves = 4;
constexpr int kDrawWaves = 4;  // a chunk is one vector of each of the first 4 waves' lanes

// Inverse-CDF draw for one sequence by a workgroup, from the chunk masses `tab` (LDS) of its recovery row: a
// double-precision scan over the masses finds the chunk holding u*Z, and only that chunk is read again to pick the token,
// a vector a lane of the first four waves.  Every one of them scans the masses for itself, so that they meet only once, over the sums
// of their quarters; with ONE_SCAN, in the workgroups of many rows that share a unit's vector ALUs, one does it for all
// (1290 sampled rows of V = 42298 24.4 -> 23.7 us, 1224 of V = 56960 27.7 -> 27.1).  The normaliser's logarithm is taken with the token's by the wave
// that picks it; by all four while the chunk was on its way, it took longer than the chunk (32 sampled rows of V = 24576 6.07 -> 5.92 us
// on the GPU, of V = 32768 6.63 -> 6.45, 8 sequences of V = 151936 18.75 -> 18.62 a step).
// What bounds it is the chain of dependent steps, in which the chip is idle: by one wave, with four vectors a lane, the part
// behind the table took 3.6 us (8 sequences of V = 151936), now 2.9.  512 steered rows of V = 128256 67.0 -> 66.1 us.
// Returns log2 Z to wave 0 where a.log2z or a.recovery_logprobs asks for it; one lane writes the per-sequence outputs.
template <int DT, int VEC, bool PLAIN, bool ONE_SCAN>
__device__ __forceinline__ double draw_token(const RecArgs& a, int b, int n, double us, int wave, int lane, const Partial* tab,
                                             const RecRow<DT, VEC>& row, double* sh_sum, int* sh_any, Found* sh_found) {
    const void *g = row.g, *sp = row.sp, *sm = row.sm;
    const long nvec = row.nvec, nch = row.nch;
    const int tailc = row.tailc, head = row.head, NC = row.NC;
    double incl_l = 0.0, base = 0.0, target = 0.0, dE = 0.0, sc = 0.0, ls = 0.0, log2Z = 0.0;
    float p[VEC];
    long first = 0;          // vocabulary index of this lane's first logit, counted from the row as it is read
    bool take_last = false;  // the uniform is not below the total mass (u >= 1 or not a number)
    Found at;
    if (ONE_SCAN ? wave == 0 : wave < kDrawWaves) at = find_chunk(tab, NC, lane, us);
    if (ONE_SCAN) {
        if (wave == 0 && lane == 0) *sh_found = at;
        __syncthreads();
        at = *sh_found;
    }
    if (wave < kDrawWaves) {
        const int cstar = at.c;
        target = at.target;
        base = at.base;
        take_last = at.last;
        // The terms are taken relative to the chunk's own exponent reference, 2^(y - Ec), so that the logits that carry
        // the chunk are normal fp32 numbers however far the chunk sits below the row's maximum; `sc` brings them to the
        // scale of the chunk table in double, exactly.
        const int Ec = tab[cstar].E;
        dE = (double)Ec;
        const float nE = -(float)Ec;
        sc = ldexp(1.0, Ec - at.Estar);
#pragma unroll
        for (int i = 0; i < VEC; ++i) p[i] = 0.f;
        const long v = (long)cstar * (kWave * kChunkSteps) + wave * kWave + lane;
        const bool full = cstar < nch && v < nvec;
        typename RawT<DT, VEC>::type rg{}, rp{}, rm{};
        if (full) {
            rg = ld_raw<DT, VEC>(g, v);
            if (!PLAIN) {
                rp = ld_raw<DT, VEC>(sp, v);
                rm = ld_raw<DT, VEC>(sm, v);
            }
        }
        float hg[VEC], hp[VEC], hm[VEC];
        int have = full ? VEC : 0;  // logits this lane holds
        first = v * VEC;
        unpack(rg, hg);
        unpack_steer<DT, VEC, PLAIN>(rp, rm, hp, hm);
        if (cstar >= nch) {         // the logits past the last full vector, one a lane
            first = nvec * VEC + lane;
            if (wave == 0 && lane < tailc) {
                have = 1;
                hg[0] = ld_elem<DT>(g, first);
                hp[0] = ld_steer<DT, PLAIN>(sp, first);
                hm[0] = ld_steer<DT, PLAIN>(sm, first);
            }
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float term = PLAIN ? __builtin_amdgcn_exp2f(fmaf(hg[i], a.c_hi, nE))
                                     : __builtin_amdgcn_exp2f((float)(rec_y(hg[i], hp[i], hm[i], a.c, a.bc) - dE));
            p[i] = i < have ? term : 0.f;
        }
        if (head && first == 0) p[0] = 0.f;  // the element before the row
#pragma unroll
        for (int i = 0; i < VEC; i += 2) ls += (double)p[i] + (double)p[i + 1];
        incl_l = wave_incl_scan_f64(ls * sc);
        const unsigned long long pm = __ballot(ls > 0.0);
        if (lane == 63) {
            sh_sum[wave] = incl_l;
            sh_any[wave] = pm != 0ull;
        }
    }
    __syncthreads();
    if (wave >= kDrawWaves) return 0.0;
    // The wave whose quarter reaches the target.  If none does (rounding between the chunk table and the re-read, or
    // take_last): the last logit of the chunk that still carries probability.
    int wsel = -1, wlast = 0;
    double start = base;
#pragma unroll
    for (int w = 0; w < kDrawWaves; ++w) {
        const double sum = sh_sum[w];
        if (sh_any[w]) wlast = w;
        if (wsel < 0) {
            if (!take_last && start + sum > target) wsel = w; else start += sum;
        }
    }
    const bool found = wsel >= 0;
    if (wave == (found ? wsel : wlast)) {
        const unsigned long long over = __ballot(found && start + incl_l > target), pm = __ballot(ls > 0.0);
        const int L = over ? first_lane(over) : (pm ? 63 - __clzll((long long)pm) : 0);
        // Lane L's last term with any mass stands if none reaches the target (the chunk's largest logit is within one unit of Ec, so one
        // exists unless the row holds something that is not a number; the index is valid then too).
        double cum = wave_shift_up_f64(incl_l) + start;
        int at_i = 0;
        float term = 0.f;
        bool done = false;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            cum += (double)p[i] * sc;
            if (!done && p[i] > 0.f) {
                at_i = i;
                term = p[i];
                done = found && cum > target;
            }
        }
        // The token's exponent is taken back from its term, whose rounding the masses hold too: where one token carries the row it
        // drops out of the difference, which the logits' own exponent would leave in the log-prob (1e-7).
        // One logarithm for both, in lane L and beside it
        const double lg = log2(lane == L ? (term > 0.f ? (double)term : 1.0) : at.total);
        log2Z = (double)at.Estar + wave_readlane_f64(lg, L ^ 1) + (PLAIN ? a.rho : 0.0) * (double)at.Estar;
        if (lane == L) {
            const double y_hi = dE + lg, y = PLAIN ? y_hi + a.rho * y_hi : y_hi;
            a.accepted_len[b] = n;
            a.next_token[b] = (int32_t)min(max(first + at_i - head, 0l), (long)a.V - 1);
            if (a.next_token_logprob) a.next_token_logprob[b] = (float)(kLn2 * (y - log2Z));
        }
    }
    return wave == 0 && (a.log2z || a.recovery_logprobs) ? mass_log2<PLAIN>(a, at.Estar, at.total) : log2Z;
}

// The same for greedy decoding, by one wave: the token is known, only the normaliser is needed.
template <bool PLAIN>
__device__ __forceinline__ double greedy_token(const RecArgs& a, int b, int n, int lane, const Partial* tab, int NC, Best pick) {
    const ChunkScan<4> cs(tab, NC, lane);
    const double log2Z = mass_log2<PLAIN>(a, cs.Estar, cs.total);
    if (lane == 0) {
        a.accepted_len[b] = n;
        a.next_token[b] = min(max(pick.idx, 0), a.V - 1);
        if (a.next_token_logprob) a.next_token_logprob[b] = (float)(kLn2 * (pick.v * a.c - log2Z));
    }
    return log2Z;
}

// Slice partials of (sequence b, position t, tensor x), t in the window.
__device__ __forceinline__ const Partial* partials_of(const RecArgs& a, int b, int t, int x) {
    return a.partial + (((long)b * (a.t_hi - a.t_lo) + (t - a.t_lo)) * 2 + x) * a.NS;
}

// What the ratio test knows of a (position, tensor) pair, in LDS: the row's merged partials and the draft token's logit (kNoToken: none).
struct Pairs {
    Partial* row;  // [2 * kmax], pair 2 * t + x
    float* h;
    // log P(y_t), for who asks for it
    __device__ __forceinline__ double logprob(const RecArgs& a, int q) const { return kLn2 * ((double)h[q] * a.c - row_log2(row[q], a.rho)); }
    __device__ __forceinline__ bool unknown(int t) const { return __float_as_uint(h[2 * t]) == kNoToken || __float_as_uint(h[2 * t + 1]) == kNoToken; }
    // Eq. 7 at position t against the uniform u: P_LLM / (lambda * P_SLM^-) is 2^((h_LLM - h_SLM^-) * c) times the rows' sums the other way
    // round, so that one exponential decides.  By the two log-probs a logarithm, and a division by the acceptance probability's form, stood
    // in the chain before the first rejection, where nothing else runs (one sequence of 64 drafts, V = 40000 17.4 -> 16.5 us a step, of 4,
    // V = 32000 fp32 8.4 -> 7.95 in one launch; 64 of 8, V = 151936 66.5 -> 66.2).  Not a number on the right accepts, as a minimum with 1 does.
    __device__ __forceinline__ bool rejects(const RecArgs& a, int t, double u) const {
        const Partial g = row[2 * t], m = row[2 * t + 1];
        const double d = ((double)h[2 * t] - (double)h[2 * t + 1]) * a.c - ((double)g.E - (double)m.E) * (1.0 + a.rho);
        return !(u <= 1.0) || u * ((double)g.s * a.lambda) > exp2(d) * (double)m.s;
    }
};

// Phase 2 for one sequence by a workgroup of NT threads, on the positions [T0, Kt) of the window (those before T0
// are known to have been accepted):
//   2a  every (position, tensor) pair gets 16 lanes: merge the row's slice partials, take the draft
//       token's logit, leave both in LDS
//   2b  wave 0: Eq. 7 on every position, first rejection by ballot
// Returns the first rejected position, Kt if none, to every thread; kFlagged if a draft id among those positions is outside
// the vocabulary or `bad` is set in any thread.  sh: kRatioWords<NT> words of LDS.
//
// What bounds it is its chain of memory round trips, while nothing else runs on the compute unit: everything in the workspace is
// loaded before the length is known (past it there are leftovers, which are not used), the draft tokens' logits among it, which
// lie beside the partials.  Draft slots and rows past the length belong to the caller and are never read.  With the logits gathered behind the ids behind the length the first rejection of a block was known
// 2.6 us after the launch's first workgroup; the recovery kernel of 8 sequences of V = 151936 took 10.7 us and 9.7 since.
template <int NT>
constexpr int kRatioWords = NT / kWave + 1;
template <int DT, int NT>
__device__ __forceinline__ int ratio_test_block(const RecArgs& a, int b, int T0, int Kt, bool bad, const Pairs& pairs, int* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l = tid & 15;
    const int kmax = a.kmax, V = a.V, Tend = a.t_hi;
    const float* un = a.uniforms + (long)b * (kmax + 1);
    const float u0 = T0 + lane < Tend ? un[T0 + lane] : 0.f;  // wave 0's first block, on its way while the rows are merged
    const int* draft = a.draft + (long)b * kmax;
    const auto gather = [&](int q) {  // the draft token's logit at (position, tensor) pair q < 2 * Kt, or kNoToken
        const int y = draft[q >> 1];
        const long off = (long)b * a.sb + (long)(q >> 1) * a.st;
        return y >= 0 && y < V ? ld_elem<DT>(row_ptr<DT>(q & 1 ? a.Sm : a.G, off), y) : __uint_as_float(kNoToken);
    };
    const float* left = a.draft_logit ? a.draft_logit + (long)b * kmax * 2 : nullptr;
    const int q0 = 2 * T0 + (tid >> 4);
    // One round for the whole window, loaded ahead of the length, or where the length makes it one (2 ragged sequences of up to 9 drafts,
    // V = 55616, in rounds by the window 14.8 us a step, by the length 14.4; longer ones within 1 % either way).
    const int top = 2 * (Tend - T0) <= NT / 16 ? Tend : Kt;
    if (2 * (top - T0) <= NT / 16) {
        float h = 0.f;
        Partial m{0, 0.f};
        if (q0 < 2 * top) {
            if (left) h = left[q0]; else if (q0 < 2 * Kt) h = gather(q0);
            m = merge_partials_row16(partials_of(a, b, q0 >> 1, q0 & 1), a.NS, l);
        }
        if (q0 < 2 * Kt && l == 0) {
            pairs.row[q0] = m;
            pairs.h[q0] = h;
        }
    } else {
        // More pairs than groups of sixteen lanes: only the merging goes in rounds, and the logits come meanwhile, a lane to every
        // pair.  With all of it in the rounds each of them cost 0.9 us of dependent loads: 27 positions tested by 4 waves took 4, and one
        // sequence of 128 positions, V = 40000, 24.1 us a step where it took 20.6 (20.8 with the logits asked for behind the merging).
        const int qa = 2 * T0 + tid;
        const float ha = left && qa < 2 * Tend ? left[qa] : 0.f;
        for (int q = q0; q < 2 * Kt; q += NT / 16) {
            const Partial m = merge_partials_row16(partials_of(a, b, q >> 1, q & 1), a.NS, l);
            if (l == 0) pairs.row[q] = m;
        }
        for (int q = qa; q < 2 * Kt; q += NT) pairs.h[q] = !left ? gather(q) : q == qa ? ha : left[q];
    }
    const bool any = __ballot(bad) != 0ull;
    if (lane == 0) sh[1 + wave] = any;
    __syncthreads();
    if (wave == 0) {
        int first_rej = Kt;
        bool unknown = lane < NT / kWave && sh[1 + (lane < NT / kWave ? lane : 0)] != 0;
        for (int t0 = T0; t0 < Kt; t0 += kWave) {
            const int t = t0 + lane;
            bool rej = false;
            if (t < Kt) {
                rej = pairs.rejects(a, t, (double)(t0 == T0 ? u0 : un[t]));
                unknown = unknown || pairs.unknown(t);
            }
            const unsigned long long rmask = __ballot(rej);
            if (rmask && first_rej == Kt) first_rej = t0 + first_lane(rmask);
        }
        const bool flagged = __ballot(unknown) != 0ull;
        if (lane == 0) sh[0] = flagged ? kFlagged : first_rej;
    }
    __syncthreads();
    return sh[0];
}

// Between two row passes: the ratio test on the positions of the window just scored, [t_lo, min(K_b, t_hi)), of
// every sequence still in play, with exactly the arithmetic of the final kernel.  A sequence rejected there is
// finished as far as verification goes (Algorithm 1 breaks out of the loop at the first
// rejection): its later rows are never scored and its first-rejection index is final.  After the first window
// every draft id of the sequence is range-checked, so a sequence is flagged exactly as in the
// one-pass schedule.
//
// NT = 128, two waves, test a window of up to 8 positions (4 without rounds); 512 a longer one (of 32 positions: 20 sequences of 128
// drafts, V = 65536, 50.4 -> 47.3 us a step).
template <int DT, int NT>
__global__ __launch_bounds__(NT) void verdict_kernel(const RecArgs a) {
    extern __shared__ double smem_d[];
    __shared__ int sh_ratio[kRatioWords<NT>];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int kmax = a.kmax, V = a.V;
    const bool first = a.t_lo == 0;
    if (!first && a.state[b] != kInPlay) return;
    const int K = a.draft_len ? a.draft_len[b] : kmax;
    bool bad = K < 0 || K > kmax;
    const int Kt = bad ? 0 : min(K, a.t_hi);
    if (first && !bad) {  // ids behind the window; those inside it are checked with their rows
        for (int t = Kt + tid; t < K; t += NT) {
            const int y = a.draft[(long)b * kmax + t];
            bad = bad || y < 0 || y >= V;
        }
    }
    const Pairs pairs{reinterpret_cast<Partial*>(smem_d), reinterpret_cast<float*>(smem_d + 2 * kmax)};
    const int n = ratio_test_block<DT, NT>(a, b, a.t_lo, Kt, bad, pairs, sh_ratio);
    if (tid == 0) a.state[b] = n == Kt && K > a.t_hi ? kInPlay : n;
}

// Best candidate of the wave, left in every lane: larger value, then lower index.
__device__ __forceinline__ void wave_best(Best& best) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const double ov = __shfl_xor(best.v, d, kWave);
        const int oi = __shfl_xor(best.idx, d, kWave);
        if (ov > best.v || (ov == best.v && oi < best.idx)) {
            best.v = ov;
            best.idx = oi;
        }
    }
}

// ------------------------------------------------------------------ log-prob rows

constexpr int kLogprobThreads = 256;
constexpr int kLogprobUnroll = 2;  // vectors per tensor a thread has in flight

// fp32 pair or quad stored at any element boundary (an odd vocabulary size starts its rows anywhere)
__device__ __forceinline__ void st_f32x4(float* p, float x, float y, float z, float w) {
    const f32x4 v = {x, y, z, w};
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}

constexpr int kNoTail = 0x7FFFFFFF;

// log Softmax(h_rec / T) of kLogprobUnroll vectors of a row, v and those `step` behind it, and of logit `tail` past the last
// full vector, where there is one.  log2_z() gives the row's normaliser, asked for while the vectors are on their way.
template <int DT, int VEC, bool PLAIN, typename F>
__device__ __forceinline__ void write_logprobs(const void* g, const void* sp, const void* sm, float* out, int V, long v0,
                                               int step, int tail, double c, double bc, F log2_z) {
    const long nvec = V / VEC;
    typename RawT<DT, VEC>::type rg[kLogprobUnroll], rp[kLogprobUnroll], rm[kLogprobUnroll];
#pragma unroll
    for (int j = 0; j < kLogprobUnroll; ++j) {
        const long v = v0 + j * step;
        if (v < nvec) {
            rg[j] = ld_raw<DT, VEC>(g, v);
            if (!PLAIN) {
                rp[j] = ld_raw<DT, VEC>(sp, v);
                rm[j] = ld_raw<DT, VEC>(sm, v);
            }
        }
    }
    const double log2Z = log2_z();
#pragma unroll
    for (int j = 0; j < kLogprobUnroll; ++j) {
        const long v = v0 + j * step;
        if (v >= nvec) break;
        float hg[VEC], hp[VEC], hm[VEC], o[VEC];
        unpack(rg[j], hg);
        unpack_steer<DT, VEC, PLAIN>(rp[j], rm[j], hp, hm);
#pragma unroll
        for (int i = 0; i < VEC; ++i) o[i] = (float)(kLn2 * (rec_y(hg[i], hp[i], hm[i], c, bc) - log2Z));
#pragma unroll
        for (int i = 0; i < VEC; i += 4) st_f32x4(out + v * VEC + i, o[i], o[i + 1], o[i + 2], o[i + 3]);
    }
    if (tail < V - nvec * VEC) {
        const long e = nvec * VEC + tail;
        out[e] = (float)(kLn2 * (rec_y(ld_elem<DT>(g, e), ld_steer<DT, PLAIN>(sp, e), ld_steer<DT, PLAIN>(sm, e), c, bc) - log2Z));
    }
}

// Everything after the row pass in one launch, a workgroup of NT threads per sequence:
//   2a  every (position, tensor) pair gets 16 lanes: merge its slice partials, take the draft token's
//       logit that the row pass left, log P(y_t) into LDS  (one memory round trip, see ratio_test_block)
//   2b  wave 0: Eq. 7 on every position, first rejection by ballot
//   3   all waves stream the three rows at the rejected (or bonus) position once, one (E, s)
//       mass per 2048-logit chunk into LDS
//   4   the first four waves draw the token (greedy: wave 0)
//   5   all waves write the log-prob row, where it is short enough (logprobs_in_recovery)
// a.defer: steps 4 and 5 are row_draw_kernel's.
// Only workgroup barriers separate the steps; nothing crosses workgroups.
//
// a.parts > 1: that many workgroups share a sequence.  Each repeats steps 2a-2b, takes a.part_chunks
// consecutive chunks in step 3 and delivers its chunk masses to a table in global memory; the part that
// arrives last (an atomic counter per sequence, no workgroup ever waits for another) runs step 4
// from the complete table.  The deliveries are made and counted by one wave with write-through stores
// (st_dev, wait_stores), and the last part reads them with device-scope loads: no cache-wide fence.
template <int DT, int VEC, bool GREEDY, bool PLAIN, int NT>
__global__ __launch_bounds__(NT) void accept_recover_kernel(const RecArgs a) {
    extern __shared__ double smem_d[];
    __shared__ int sh_ratio[kRatioWords<NT>];
    __shared__ Partial sh_part[NT == 1024 ? NT / kWave : 1];
    __shared__ double sh_sum[kDrawWaves];
    __shared__ int sh_any[kDrawWaves], sh_last;
    __shared__ Found sh_found;
    __shared__ double sh_best_v[NT / kWave];
    __shared__ int sh_best_i[NT / kWave];
    __shared__ double sh_log2z;

    const int S = a.parts;
    const int b = (int)blockIdx.x / S, part = (int)blockIdx.x - b * S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NW = NT / kWave;
    const int kmax = a.kmax, V = a.V;
    const Pairs pairs{reinterpret_cast<Partial*>(smem_d), reinterpret_cast<float*>(smem_d + 2 * kmax)};
    Partial* tab = reinterpret_cast<Partial*>(smem_d + 3 * kmax);   // [NC] chunk masses

    const double us = GREEDY ? 0.0 : (double)a.uniforms[(long)b * (kmax + 1) + kmax];  // read here, where nothing waits for it
    // Several windows: a sequence a verdict kernel saw rejected (or at its end) keeps that first-rejection
    // index; a sequence still in play is tested here on the positions of the last window.  One window: every
    // sequence is tested here over all K positions.
    const int state = a.state ? a.state[b] : kInPlay;
    int n = state, Kt = 0;
    if (state == kInPlay) {
        const int K = a.draft_len ? a.draft_len[b] : kmax;
        const bool bad_len = K < 0 || K > kmax;
        Kt = bad_len ? 0 : K;
        n = kmax > 0 ? ratio_test_block<DT, NT>(a, b, a.t_lo, Kt, bad_len, pairs, sh_ratio) : bad_len ? kFlagged : 0;
    }
    const bool bad = n < 0;
    // Valid positions' log-probs, padded slots 0, a flagged sequence NaN throughout; up to 32 drafts by the wave that has the fewest chunks
    const bool one_wave = 2 * kmax <= kWave;
    if (a.draft_logprobs && part == S - 1 && (!one_wave || wave == NW - 1)) {
        const float nanv = __int_as_float(0x7FC00000);
        for (int i = one_wave ? lane : tid; i < kmax * 2; i += one_wave ? kWave : NT)
            a.draft_logprobs[(long)b * kmax * 2 + i] = bad ? nanv : (i < 2 * Kt ? (float)pairs.logprob(a, i) : 0.f);
    }
    if (bad) {
        if (tid == 0 && part == 0) {
            a.accepted_len[b] = -1;
            a.next_token[b] = -1;
            if (a.next_token_logprob) a.next_token_logprob[b] = __int_as_float(0x7FC00000);
        }
        return;
    }

    // ---- 3
    const RecRow<DT, VEC> row(a, b, n);
    Best best{-__builtin_huge_val(), kNoBest};
    const int c0 = part * a.part_chunks, c1 = min(row.NC, c0 + a.part_chunks);
    // Shared rows: chunks left over for a last round of at most half the waves are dealt out in halves or quarters, so that the round
    // takes as much less.  64 sequences of V = 151936, 75 chunks, in 4 parts of 16 whole chunks and 3 in quarters: 67.7 us a step, with the
    // 3 whole 68.2, in the 3 parts of 25 that leave a quarter of the units idle 68.9; 80 of V = 100000 36.2, 36.9 and 38.5; 100 of V =
    // 151936 in 2 parts of 32 and 6 in halves 63.9, whole 64.6.
    const int over = NT == 1024 && S > 1 && c1 > c0 ? (c1 - c0) % NW : 0;
    const int ways = over == 0 || 2 * over > NW ? 1 : 4 * over > NW ? 2 : 4;
    const int cw = ways > 1 ? c1 - over : c1;  // whole chunks end here
    int c = c0 + wave;
    if (PLAIN && DT == SS_BF16 && NT == 1024) {
        Partial p[2];
        for (; c + NW < cw && (long)(c + NW + 1) * (kWave * kChunkSteps) <= row.nvec; c += 2 * NW) {
            chunk_pair_mass<DT, VEC, GREEDY, true>(row, {c, c + NW}, lane, a.c_hi, best, p);
            if (lane == 0) tab[c] = p[0], tab[c + NW] = p[1];
        }
        if (c + NW < cw && c + NW < row.nch) {
            chunk_pair_mass<DT, VEC, GREEDY, false>(row, {c, c + NW}, lane, a.c_hi, best, p);
            if (lane == 0) tab[c] = p[0], tab[c + NW] = p[1];
            c += 2 * NW;
        }
    }
    for (; c < cw; c += NW) {
        const Partial p = chunk_mass<DT, VEC, GREEDY, PLAIN>(row, c, lane, a.c, a.bc, a.beta, a.c_hi, best);
        if (lane == 0) tab[c] = p;
    }
    if (NT == 1024 && ways > 1 && wave < over * ways) {
        const int cs = cw + wave / ways, step0 = wave % ways * (kChunkSteps / ways);
        const Partial p = ways == 2
            ? chunk_mass<DT, VEC, GREEDY, PLAIN, kChunkSteps / 2>(row, cs, lane, a.c, a.bc, a.beta, a.c_hi, best, step0)
            : chunk_mass<DT, VEC, GREEDY, PLAIN, kChunkSteps / 4>(row, cs, lane, a.c, a.bc, a.beta, a.c_hi, best, step0);
        if (lane == 0) sh_part[wave] = p;
    }
    const auto mass = [&](int c) {  // of a chunk of this part
        if (NT != 1024 || c < cw) return tab[c];
        Partial m = sh_part[(c - cw) * ways];
        for (int i = 1; i < ways; ++i) {
            const Partial q = sh_part[(c - cw) * ways + i];
            const int E = max(m.E, q.E);
            m = Partial{E, ldexpf(m.s, m.E - E) + ldexpf(q.s, q.E - E)};
        }
        return m;
    };
    if (GREEDY) {
        wave_best(best);
        if (lane == 0) {
            sh_best_v[wave] = best.v;
            sh_best_i[wave] = best.idx;
        }
    }
    __syncthreads();
    if (GREEDY && wave == 0) {
        best.v = lane < NW ? sh_best_v[lane] : -__builtin_huge_val();
        best.idx = lane < NW ? sh_best_i[lane] : kNoBest;
        wave_best(best);
        if (best.idx <= V) best.idx -= row.head;
    }
    if (a.defer) {
        for (int c = c0 + tid; c < c1; c += NT) a.chunk_tab[(long)b * a.NC + c] = mass(c);
        if (tid == 0) {
            if (GREEDY) {
                a.best_v[(long)b * a.NC + part] = best.v;
                a.best_i[(long)b * a.NC + part] = min(best.idx, V);
            }
            if (part == 0) a.accepted_len[b] = n;
        }
        return;
    }
    if (S > 1) {  // deliver this part; only the last part to arrive goes on
        Partial* gtab = a.chunk_tab + (long)b * a.NC;
        if (wave == 0) {
            for (int c = c0 + lane; c < c1; c += kWave) st_dev_partial(gtab + c, mass(c));
            if (GREEDY && lane == 0) {
                st_dev(reinterpret_cast<unsigned long long*>(a.best_v + (long)b * a.NC + part),
                       (unsigned long long)__double_as_longlong(best.v));
                st_dev(a.best_i + (long)b * a.NC + part, min(best.idx, V));
            }
            wait_stores();  // this wave's deliveries have reached memory before it is counted
            if (lane == 0)
                sh_last = __hip_atomic_fetch_add(a.arrive + (long)b * kArriveStride, 1u, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT) == (unsigned)S - 1u;
        }
        __syncthreads();
        if (!sh_last) return;
        for (int c = tid; c < row.NC; c += NT) tab[c] = ld_dev_partial(gtab + c);
        if (GREEDY && wave == 0) {
            best = Best{-__builtin_huge_val(), kNoBest};
            for (int i = lane; i < S; i += kWave) {
                const double v = __longlong_as_double((long long)ld_dev(
                    reinterpret_cast<const unsigned long long*>(a.best_v + (long)b * a.NC + i)));
                const int idx = ld_dev(a.best_i + (long)b * a.NC + i);
                if (v > best.v || (v == best.v && idx < best.idx)) best = Best{v, idx};
            }
            wave_best(best);
        }
        __syncthreads();
    }

    // ---- 4
    // The waves that do not draw end here where nothing is left for them (a barrier waits for the surviving waves only), so that the
    // next workgroup can start (1290 sampled rows of V = 42298 24.4 -> 24.3 us).
    if (wave >= kDrawWaves && !a.recovery_logprobs) return;
    if (!GREEDY || wave == 0) {
        const double log2Z = GREEDY ? greedy_token<PLAIN>(a, b, n, lane, tab, row.NC, best)
                                    : draw_token<DT, VEC, PLAIN, NT == 512>(a, b, n, us, wave, lane, tab, row, sh_sum, sh_any, &sh_found);
        if (tid == 0) {
            if (a.log2z) a.log2z[b] = log2Z;
            sh_log2z = log2Z;
        }
    }
    if (!a.recovery_logprobs) return;

    // ---- 5 (only with the row in one part)
    __syncthreads();
    const long nv = V / VEC, off = (long)b * a.sb + (long)n * a.st;
    const void *g = row_ptr<DT>(a.G, off), *sp = row_ptr<DT>(a.recSp, off), *sm = row_ptr<DT>(a.recSm, off);
    for (long v = tid; v < nv || v == tid; v += NT * kLogprobUnroll)
        write_logprobs<DT, VEC, PLAIN>(g, sp, sm, a.recovery_logprobs + (long)b * V, V, v, NT, v == tid ? tid : kNoTail, a.c, a.bc, [&] { return sh_log2z; });
}

// ------------------------------------------------------------------ kernel: small blocks in one launch

// The words of words.h in memory, written and read with device-scope atomics: whoever finds every word of a sequence has all that was
// delivered, without a counter that someone would have had to clear before.
struct Words {
    unsigned long long* w;
    CallTag tag;
    __device__ __forceinline__ void put(int i, unsigned v) const { st_dev(w + i, (unsigned long long)value_word(tag, i, v)); }
    __device__ __forceinline__ void arrive(int i) const { st_dev(w + i, (unsigned long long)arrival_word(tag, i)); }
    __device__ __forceinline__ unsigned long long load(int i) const { return ld_dev(w + i); }
    __device__ __forceinline__ void put_best(int i, double v, int idx) const {
        const unsigned long long x = (unsigned long long)__double_as_longlong(v);
        st_dev(w + i, (unsigned long long)best_word(tag, i, x));
        st_dev(w + i + 1, (unsigned long long)best_word2(tag, i, x, (unsigned)idx));
    }
    __device__ __forceinline__ bool get_best(int i, double& v, int& idx) const {
        const unsigned long long x = ld_dev(w + i), y = ld_dev(w + i + 1);
        v = __longlong_as_double((long long)best_value(x, y));
        idx = (int)best_token(y);
        return are_best_words(tag, i, x, y);
    }
    __device__ __forceinline__ void clear(int i) const { st_dev(w + i, 0ull); }
};

struct OnceArgs {
    RecArgs rec;
    unsigned long long* words;  // [B][word_stride], see once_space
    long word_stride;
    CallTag tag;                // of this call's words
    OnceSpace once;
};

// The row pass's sum over a chunk of full vectors, those that are not there -inf.
template <int DT, int VEC>
__device__ __forceinline__ void lse_chunk(Acc& acc, const typename RawT<DT, VEC>::type (&r)[kChunkSteps], float c_hi) {
    float h[kChunkSteps * VEC];
#pragma unroll
    for (int j = 0; j < kChunkSteps; ++j) {
        float hj[VEC];
        unpack(r[j], hj);
#pragma unroll
        for (int i = 0; i < VEC; ++i) h[j * VEC + i] = hj[i];
    }
    acc_add_f32<kChunkSteps * VEC>(acc, h, c_hi);
}

// The whole block for small batches, without log-prob rows: a workgroup for kOnceWaves chunks of one position of one sequence, a chunk a wave.
//   1  the chunk's slice partials in G and S_noctx (a draft's position) and its recovery mass, from one reading of the three rows;
//      the workgroup's partials merged
//   2  hand-over: the masses, and behind them, as words that say that they are there, the partials (the bonus position: only that)
//   3  the part that finds the words of all parts: ratio test, first rejection, draw from the masses of that position
// What bounds such a block is its chain of memory round trips and launches.  By a row pass, and a recovery whose parts each test, sweep the
// rows of one position and hand over, there were eight round trips and a launch between; the masses of every position, formed beside
// the partials on units that are idle, leave five: logits, hand-over (two), the other parts' masses, and the chunk that the token is in.  One
// sequence of 4 drafts, V = 32000 fp32 10.55 -> 7.9 us a step (a launch less of host time, and 7.7 on the GPU instead of 10.1), 1 of 8
// drafts, V = 128256 bf16 13.5 -> 10.4, 4 of 8, V = 50257 14.3 -> 10.5.
// Nothing waits that need not: the masses go to memory while the partials are formed, and Eq. 7 is evaluated by every wave while the other
// parts' masses come (behind them it was 7.95 us on the GPU for the first of those, 7.65 now, 11.4 for the third, 10.5 now).
// Parts end together, so that several find all words; the claim, an exchange on its way beside the masses, leaves one of them (should another
// come behind its clearing, both draw, from the same words, the same token).  Nobody waits for anybody.
template <int DT, int VEC, bool GREEDY, bool PLAIN>
__global__ __launch_bounds__(kOnceWaves * kWave) void block_once_kernel(const OnceArgs o) {
    const RecArgs& a = o.rec;
    static_assert(kOnceWaves == kDrawWaves, "a vector a lane of the drawing waves");
    extern __shared__ double smem_d[];
    __shared__ Partial sh_lse[kOnceWaves][2];
    __shared__ double sh_best_v[kOnceWaves], sh_sum[kDrawWaves];
    __shared__ int sh_best_i[kOnceWaves], sh_any[kDrawWaves], sh_missing[kOnceWaves], sh_mine;
    __shared__ float sh_h[2 * kOnceMaxDrafts];
    const int kmax = a.kmax, V = a.V, NC = a.NC, PP = o.once.parts;
    const int per = (kmax + 1) * PP, b = (int)blockIdx.x / per, part = (int)blockIdx.x - b * per, t = part / PP, pp = part - t * PP;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Partial* const mass = reinterpret_cast<Partial*>(smem_d);                                     // [kmax + 1][NC]
    const Pairs pairs{mass + (kmax + 1) * NC, sh_h};                                              // [kmax][2]
    unsigned* const parts = reinterpret_cast<unsigned*>(pairs.row + 2 * kmax);                   // [kmax][PP][2][E, s]
    double* const cand_v = smem_d + (kmax + 1) * NC + 2 * kmax + 2 * kmax * PP;                  // [kmax + 1][PP]
    int* const cand_i = reinterpret_cast<int*>(cand_v + (GREEDY ? (kmax + 1) * PP : 0));

    const int K = a.draft_len ? a.draft_len[b] : kmax;
    const float u = lane <= kmax ? a.uniforms[(long)b * (kmax + 1) + lane] : 0.f;  // of the tests and, in lane kmax, of the draw
    const auto flag = [&]() {
        const float nanv = __int_as_float(0x7FC00000);
        if (a.draft_logprobs && tid < 2 * kmax) a.draft_logprobs[(long)b * kmax * 2 + tid] = nanv;
        if (tid == 0) {
            a.accepted_len[b] = -1;
            a.next_token[b] = -1;
            if (a.next_token_logprob) a.next_token_logprob[b] = nanv;
        }
    };
    if (K < 0 || K > kmax) {
        if (part == 0) flag();
        return;
    }
    if (t > K) return;
    unsigned long long* const w = o.words + (long)b * o.word_stride;
    const Words words{w, o.tag};
    unsigned long long* const gmass = w + o.once.masses;

    // ---- one chunk of this position
    const int y = tid < 2 * K ? a.draft[(long)b * kmax + (tid >> 1)] : 0;
    const int c = pp * kOnceWaves + wave;
    const RecRow<DT, VEC> row(a, b, t);
    const void* const sm = row_ptr<DT>(a.Sm, (long)b * a.sb + (long)t * a.st - row.head);  // row.sm, but with PLAIN
    const bool with_m = !PLAIN || t < K;  // without steering nothing asks for S_noctx at the bonus position
    const long vbase = (long)c * (kChunkSteps * kWave) + lane;
    const bool whole = c < row.nch, last = c == row.nch && lane < row.tailc;  // full vectors, or one logit past them
    typename RawT<DT, VEC>::type rg[kChunkSteps], rp[kChunkSteps], rm[kChunkSteps];
    float tg[1] = {0.f}, tp[1] = {0.f}, tm[1] = {0.f};
    if (whole) {
#pragma unroll
        for (int j = 0; j < kChunkSteps; ++j) {
            const long v = vbase + (long)j * kWave;
            rg[j] = rp[j] = rm[j] = neg_inf_raw<DT, VEC>();  // past the row: adds nothing, and has no steering
            if (v < row.nvec) {
                rg[j] = ld_raw<DT, VEC>(row.g, v);
                if (!PLAIN) rp[j] = ld_raw<DT, VEC>(row.sp, v);
                if (with_m) rm[j] = ld_raw<DT, VEC>(sm, v);
            }
        }
    } else if (last) {
        const long e = row.nvec * VEC + lane;
        tg[0] = ld_elem<DT>(row.g, e);
        tp[0] = ld_steer<DT, PLAIN>(row.sp, e);
        if (with_m) tm[0] = ld_elem<DT>(sm, e);
    }
    float hy = 0.f;
    if (tid < 2 * K) {  // the draft tokens' logits, on their way beside the rows
        const long off = (long)b * a.sb + (long)(tid >> 1) * a.st;
        hy = y >= 0 && y < V ? ld_elem<DT>(row_ptr<DT>(tid & 1 ? a.Sm : a.G, off), y) : __uint_as_float(kNoToken);
    }
    Acc g{kEInit, 0.f}, m{kEInit, 0.f}, rec{kEInit, 0.f};
    Best best{-__builtin_huge_val(), kNoBest};
    const bool first = row.head && vbase == 0;  // this lane's first vector starts with the element before the row
    if (first) {
        rg[0] = set_first(rg[0], kBf16NegInf);
        rm[0] = set_first(rm[0], kBf16NegInf);
    }
    // the recovery mass, as chunk_mass has it, on its way to memory while the partials are formed
    const auto take_g = [&]() {
        if (whole) lse_chunk<DT, VEC>(g, rg, a.c_hi);
        else if (last) acc_add_f32<1>(g, tg, a.c_hi);
    };
    if (PLAIN) take_g();
    if (whole) {
        if (first) rp[0] = set_first(rp[0], 0u);
        const auto m0 = first ? set_first(rm[0], 0u) : rm[0];
#pragma unroll
        for (int j = 0; j < kChunkSteps; ++j) {
            const int at = (int)(vbase + (long)j * kWave) * VEC;
            float hg[VEC], hp[VEC], hm[VEC];
            unpack(rg[j], hg);
            unpack_steer<DT, VEC, PLAIN>(rp[j], j == 0 ? m0 : rm[j], hp, hm);
            if (!PLAIN) acc_add_rec<DT, VEC, GREEDY>(rec, hg, hp, hm, a.c, a.bc, (float)a.c, (float)a.bc, a.beta, at, best);
            if (PLAIN && GREEDY) best_of<VEC>(best, hg, at);
            if (PLAIN && vbase + (long)j * kWave < row.nvec) acc_add_f32<VEC>(rec, hg, a.c_hi);
        }
        if (PLAIN && vbase + (long)(kChunkSteps - 1) * kWave < row.nvec) rec = g;
    } else if (last) {
        const int at = (int)(row.nvec * VEC) + lane;
        if (!PLAIN) acc_add_rec<DT, 1, GREEDY>(rec, tg, tp, tm, a.c, a.bc, (float)a.c, (float)a.bc, a.beta, at, best);
        if (PLAIN && GREEDY) best_of<1>(best, tg, at);
        if (PLAIN) rec = g;
    }
    const Partial p = wave_combine(rec);
    if (c < row.NC && lane == 0) st_dev_partial(reinterpret_cast<Partial*>(gmass) + (long)t * NC + c, p);
    if (t < K) {
        if (!PLAIN) take_g();
        if (whole) lse_chunk<DT, VEC>(m, rm, a.c_hi);
        else if (last) acc_add_f32<1>(m, tm, a.c_hi);
        const Partial pg = wave_combine(g), pm = wave_combine(m);
        if (lane == 0) {
            sh_lse[wave][0] = pg;
            sh_lse[wave][1] = pm;
        }
    }
    if (GREEDY) {
        wave_best(best);
        if (lane == 0) {
            sh_best_v[wave] = best.v;
            sh_best_i[wave] = best.idx <= V ? best.idx - row.head : best.idx;
        }
    }
    if (tid < 2 * K) sh_h[tid] = hy;
    wait_stores();  // the masses have reached memory before the words that tell of them
    __syncthreads();
    if (wave == 0) {
        if (t < K) {
            const int x = lane >> 1 & 1;
            int E = sh_lse[0][x].E;
#pragma unroll
            for (int i = 1; i < kOnceWaves; ++i) E = max(E, sh_lse[i][x].E);
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < kOnceWaves; ++i) s += ldexpf(sh_lse[i][x].s, sh_lse[i][x].E - E);
            if (lane < 4) words.put(2 + 4 * part + lane, lane & 1 ? __float_as_uint(s) : (unsigned)E);
        } else if (lane == 0) {
            words.arrive((int)o.once.flags + pp);
        }
        if (GREEDY) {
            best.v = lane < kOnceWaves ? sh_best_v[lane] : -__builtin_huge_val();
            best.idx = lane < kOnceWaves ? sh_best_i[lane] : kNoBest;
            wave_best(best);
            if (lane == 0) words.put_best((int)o.once.best + 2 * part, best.v, min(best.idx, V));
        }
        wait_stores();
    }
    __syncthreads();

    // ---- whether all parts have delivered.  One that ends a moment before the last may find so too: the claim leaves one of them.
    bool all = true;
    const int nlse = 4 * K * PP, nflag = nlse + PP, ncand = GREEDY ? (K + 1) * PP : 0;
    const auto word = [&](int i) { return i < nlse ? 2 + i : (int)o.once.flags + (i - nlse); };
    for (int i = tid; i < nflag; i += kOnceWaves * kWave) {
        const unsigned long long x = words.load(word(i));
        all = is_word(o.tag, word(i), i < nlse, x) && all;
        if (i < nlse) parts[i] = (unsigned)x;
    }
    if (GREEDY)
        for (int i = tid; i < ncand; i += kOnceWaves * kWave) all = words.get_best((int)o.once.best + 2 * i, cand_v[i], cand_i[i]) && all;
    const unsigned long long missing = __ballot(!all);
    if (lane == 0) sh_missing[wave] = missing != 0ull;
    __syncthreads();
    if (sh_missing[0] | sh_missing[1] | sh_missing[2] | sh_missing[3]) return;
    const unsigned long long claim = (unsigned long long)claim_word(o.tag);
    unsigned long long before = 0ull;
    if (tid == 0) before = __hip_atomic_exchange(w, claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- the ratio test, by every wave, while the masses and the claim are on their way
    constexpr int kHeld = 5;
    unsigned long long held[kHeld];
    const int nmass = (K + 1) * NC;
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
        const int at = tid + i * kOnceWaves * kWave;
        held[i] = at < nmass ? ld_dev(gmass + at) : 0ull;
    }
    const int l = tid & 15;
    for (int q = tid >> 4; q < 2 * K; q += kOnceWaves * kWave / 16) {
        const unsigned* const e = parts + (((q >> 1) * PP + l) * 2 + (q & 1)) * 2;
        const Partial p = l < PP ? Partial{(int)e[0], __uint_as_float(e[1])} : Partial{kEInit, 0.f};
        const int E = row_max_i32(p.E);
        const Partial m{E, row_sum_f32(ldexpf(p.s, p.E - E))};
        if (l == 0) pairs.row[q] = m;
    }
    __syncthreads();
    bool rej = false, none = false;
    if (lane < K) {
        rej = pairs.rejects(a, lane, (double)u);
        none = pairs.unknown(lane);
    }
    const unsigned long long rmask = __ballot(rej), nmask = __ballot(none);
    const int n = rmask ? first_lane(rmask) : K;
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
        const int at = tid + i * kOnceWaves * kWave;
        if (at < nmass) mass[at] = Partial{(int)(unsigned)held[i], __uint_as_float((unsigned)(held[i] >> 32))};
    }
    for (int at = tid + kHeld * kOnceWaves * kWave; at < nmass; at += kOnceWaves * kWave) mass[at] = ld_dev_partial(reinterpret_cast<Partial*>(gmass) + at);
    if (tid == 0) sh_mine = before != claim;
    __syncthreads();
    if (!sh_mine) return;
    for (int i = tid; i < nflag; i += kOnceWaves * kWave) words.clear(word(i));
    for (int i = tid; i < 2 * ncand; i += kOnceWaves * kWave) words.clear((int)o.once.best + i);
    if (tid == 0) words.clear(0);
    if (nmask) {
        flag();
        return;
    }
    if (a.draft_logprobs && tid < 2 * kmax) a.draft_logprobs[(long)b * kmax * 2 + tid] = tid < 2 * K ? (float)pairs.logprob(a, tid) : 0.f;

    // ---- the draw
    const RecRow<DT, VEC> at(a, b, n);
    const Partial* const tab = mass + n * NC;
    if (GREEDY) {
        if (wave > 0) return;
        best.v = lane < PP ? cand_v[n * PP + lane] : -__builtin_huge_val();
        best.idx = lane < PP ? cand_i[n * PP + lane] : kNoBest;
        wave_best(best);
        greedy_token<PLAIN>(a, b, n, lane, tab, at.NC, best);
    } else {
        const double us = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(u), kmax));
        draw_token<DT, VEC, PLAIN, false>(a, b, n, us, wave, lane, tab, at, sh_sum, sh_any, nullptr);
    }
}

// ------------------------------------------------------------------ kernels: few rows without drafts

// k_max == 0 and the row in several parts: with no row pass to clear arrival counters, the masses and the draw are two
// launches instead of a fill, a sweep with a hand-over and a draw by the last part, whose chain of round trips was what
// bound it (64 steered rows of V = 131072 17.1 -> 15.1 us a call, of V = 196608 22.0 -> 18.6; 101 sampled rows of V = 151552 17.9
// -> 14.4, which is the host's time).
//
// The masses of kMassWaves chunks of a row, one a wave, and greedy candidates with them: as many workgroups as there are
// chunks for, without a serial part, so that all loads are on their way at once.
template <int DT, int VEC, bool GREEDY, bool PLAIN>
__global__ __launch_bounds__(kMassWaves * kWave) void row_mass_kernel(const RecArgs a) {
    const int b = (int)blockIdx.x / a.parts, part = (int)blockIdx.x - b * a.parts;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const RecRow<DT, VEC> row(a, b, 0);
    const int c = part * kMassWaves + wave;
    if (c >= row.NC) return;
    Best best{-__builtin_huge_val(), kNoBest};
    const Partial p = chunk_mass<DT, VEC, GREEDY, PLAIN>(row, c, lane, a.c, a.bc, a.beta, a.c_hi, best);
    const long at = (long)b * a.NC + c;  // greedy candidates: one a chunk
    if (GREEDY) wave_best(best);
    if (lane == 0) {
        a.chunk_tab[at] = p;
        if (GREEDY) {
            a.best_v[at] = best.v;
            a.best_i[at] = min(best.idx - (best.idx <= a.V ? row.head : 0), a.V);
        }
    }
}

// The token of a row from its masses, and with a.segs > 0 its log-prob row: one workgroup draws, the others write a segment each, so
// that the draw's chain of steps and the sweep over the row run side by side.  Each of them forms the row's
// normaliser from the masses itself, while its logits are on their way.  Behind a draw by the last part, a launch of its own for
// the rows took 16 sequences of V = 151936 to 33.8 us a call, 31.9 now (two launches of 7 and 12 us became 9 and 8); 32 of
// V = 128256 47.6 -> 44.8, 64 of V = 151936 89.8 -> 87.1.
template <int DT, int VEC, bool GREEDY, bool PLAIN>
__global__ __launch_bounds__(kLogprobThreads) void row_draw_kernel(const RecArgs a) {
    static_assert(kLogprobThreads == kDrawWaves * kWave, "a vector a lane of the drawing waves");
    extern __shared__ double smem_d[];
    __shared__ double sh_sum[kDrawWaves];
    __shared__ int sh_any[kDrawWaves];
    const int b = (int)blockIdx.x / (a.segs + 1), seg = (int)blockIdx.x - b * (a.segs + 1) - 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kmax = a.kmax;
    const double us = GREEDY || seg >= 0 ? 0.0 : (double)a.uniforms[(long)b * (kmax + 1) + kmax];
    // the row: what the ratio test has found, or the only one there is (no draft can have a length)
    const int n = kmax > 0 ? a.accepted_len[b] : a.draft_len && a.draft_len[b] != 0 ? -1 : 0;
    if (n < 0) {  // flagged: the log-prob row is left unwritten
        if (kmax == 0 && seg < 0 && tid == 0) {
            a.accepted_len[b] = -1;
            a.next_token[b] = -1;
            if (a.next_token_logprob) a.next_token_logprob[b] = __int_as_float(0x7FC00000);
        }
        return;
    }
    const RecRow<DT, VEC> row(a, b, n);
    const long at = (long)b * a.NC;
    if (seg >= 0) {
        const long off = (long)b * a.sb + (long)n * a.st;
        write_logprobs<DT, VEC, PLAIN>(row_ptr<DT>(a.G, off), row_ptr<DT>(a.recSp, off), row_ptr<DT>(a.recSm, off),
                                       a.recovery_logprobs + (long)b * a.V, a.V, (long)seg * (kLogprobThreads * kLogprobUnroll) + tid,
                                       kLogprobThreads, seg == a.segs - 1 ? tid : kNoTail, a.c, a.bc, [&] {
                                           const ChunkScan<4> cs(a.chunk_tab + at, row.NC, lane);
                                           return mass_log2<PLAIN>(a, cs.Estar, cs.total);
                                       });
        return;
    }
    Partial* tab = reinterpret_cast<Partial*>(smem_d);
    for (int c = tid; c < row.NC; c += kLogprobThreads) tab[c] = a.chunk_tab[at + c];
    Best best{-__builtin_huge_val(), kNoBest};
    if (GREEDY && wave == 0) {
        const int cands = kmax > 0 ? a.parts : row.NC;  // one a part, or one a chunk
        for (int i = lane; i < cands; i += kWave) {
            const double v = a.best_v[at + i];
            const int idx = a.best_i[at + i];
            if (v > best.v || (v == best.v && idx < best.idx)) best = Best{v, idx};
        }
        wave_best(best);
    }
    __syncthreads();
    if (GREEDY && wave > 0) return;
    if (GREEDY) greedy_token<PLAIN>(a, b, n, lane, tab, row.NC, best);
    else draw_token<DT, VEC, PLAIN, false>(a, b, n, us, wave, lane, tab, row, sh_sum, sh_any, nullptr);
}

// ------------------------------------------------------------------ kernel: log-prob rows

struct LogprobArgs {
    const void* G;
    const void* recSp;
    const void* recSm;
    const int32_t* accepted_len;  // the row n_b of every sequence, -1 for a flagged one
    const double* log2z;
    float* out;                   // [B, V]
    long sb, st;
    int V;
    int segs;                     // workgroups per row
    double c, bc;
};

// log Softmax(h_rec / T) at row n_b, after accept_recover has left n_b and the row's log2-normaliser.
// HBM-bound: three rows read and one fp32 row written per sequence.  A launch of its own but for short rows, because the
// workgroup that draws a sequence's token is one of at most a few hundred, each tied to the rate of one
// compute unit; cut into segments of two vectors a thread, the sweep covers the chip (16 sequences of
// V = 151936 bf16: 40 us of a 57 us recovery kernel before, 7 us as a launch of its own).
template <int DT, int VEC, bool PLAIN>
__global__ __launch_bounds__(kLogprobThreads) void recovery_logprob_kernel(const LogprobArgs a) {
    const int b = (int)blockIdx.x / a.segs, seg = (int)blockIdx.x - b * a.segs;
    const int n = a.accepted_len[b];
    if (n < 0) return;  // a flagged sequence's row is left unwritten
    const long off = (long)b * a.sb + (long)n * a.st;
    write_logprobs<DT, VEC, PLAIN>(row_ptr<DT>(a.G, off), row_ptr<DT>(a.recSp, off), row_ptr<DT>(a.recSm, off),
                                   a.out + (long)b * a.V, a.V, (long)seg * (kLogprobThreads * kLogprobUnroll) + threadIdx.x,
                                   kLogprobThreads, seg == a.segs - 1 ? (int)threadIdx.x : kNoTail, a.c, a.bc, [&] { return a.log2z[b]; });
}

// ------------------------------------------------------------------ host side

// One row pass over window `win`.  `uniform_rows` > 0 when every sequence has that many rows.
template <int DT, int VEC>
void launch_row_pass(LseArgs la, const Window& w, const RowWindow& win, int uniform_rows, int32_t* row_off, Partial* partial,
                     hipStream_t stream) {
    const int B = la.B;
    const int cus = device_cu_count();
    la.win = win;
    la.NS = w.NS;
    la.slice_vecs = w.slice_vecs;
    la.uniform_rows = uniform_rows;
    la.row_off = row_off;
    la.partial = partial;
    const bool listed = uniform_rows <= 0;
    // the row list is built in LDS by the row pass unless the batch is too large for it
    const bool global_list = listed && B > kMaxLdsBatch;
    la.list_in_lds = (listed && !global_list) ? 1 : 0;
    if (global_list) launch(prep_rows_kernel, dim3(1), dim3(1024), 0, stream, win, B, row_off);
    const long items = (long)B * (w.t_hi - w.t_lo) * 2 * la.NS;
    if (items <= 0) return;
    const long per_wg = kLseThreads / kWave;
    long wgs = (items + per_wg - 1) / per_wg;
    const long cap = (long)cus * kLseWgPerCu;
    if (wgs > cap) wgs = cap;
    const size_t lds = la.list_in_lds ? (size_t)(B + 1) * sizeof(int) : 0;
    launch(row_lse_kernel<DT, VEC, kLseUnroll>, dim3((unsigned)wgs), dim3(kLseThreads), lds,
                       stream, la);
}

// Whether what is enqueued on the stream goes into a graph.
bool being_captured(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
        (void)hipGetLastError();  // the launches will tell
        return false;
    }
    return status == hipStreamCaptureStatusActive;
}

template <int DT>
unsigned elem_parity(const void* p) { return (unsigned)(reinterpret_cast<uintptr_t>(p) / (DT == SS_BF16 ? 2 : 4)) & 1u; }

template <int DT, int VEC>
hipError_t launch_all(LseArgs la, RecArgs ra, const Plan& pl, char* ws, float* recovery_logprobs, bool unbound, hipStream_t stream,
                      hipEvent_t* ev) {
    const int B = ra.B, kmax = ra.kmax, V = ra.V;
    int32_t* lists[2] = {reinterpret_cast<int32_t*>(ws), reinterpret_cast<int32_t*>(ws + pl.off_list2)};
    int32_t* state = reinterpret_cast<int32_t*>(ws + pl.off_state);
    Partial* partial = reinterpret_cast<Partial*>(ws + pl.off_partial);
    // the verdicts' position-by-position log-probs are only complete in the one-pass schedule
    const bool one_pass = ra.draft_logprobs != nullptr || pl.windows == 1;
    const Window* wins = one_pass ? &pl.all : pl.win;
    const int windows = one_pass ? 1 : pl.windows;
    hipError_t ev_err = hipSuccess;
    auto mark = [&](int i) {  // stage boundary of the timed entry point
        if (!ev) return;
        const hipError_t e = hipEventRecord(ev[i], stream);
        if (e != hipSuccess && ev_err == hipSuccess) ev_err = e;
    };
    const bool ragged = ra.draft_len != nullptr && kmax > 0;
    ra.partial = partial;
    la.draft = ra.draft;
    la.draft_logit = pl.draft_logit ? reinterpret_cast<float*>(ws + pl.off_draft_logit) : nullptr;
    ra.draft_logit = la.draft_logit;
    ra.state = windows > 1 ? state : nullptr;
    const unsigned bases[3] = {elem_parity<DT>(ra.G), elem_parity<DT>(ra.recSp), elem_parity<DT>(ra.recSm)};
    ra.NC = chunks_per_row(V, VEC, odd_rows_possible(VEC, bases, B, kmax, ra.sb, ra.st));
    RecShape shape = recovery_shape(B, ra.NC, kmax, device_cu_count(), pl.split);
    if (kmax == 0 && shape.part_chunks < ra.NC && rows_in_one_launch(B, ra.NC, DT, ra.plain != 0, ra.greedy != 0, unbound || being_captured(stream)))
        shape = RecShape{1024, ra.NC};
    const bool rows_inside = recovery_logprobs && logprobs_in_recovery(B, kmax, V, DT == SS_BF16 ? 2 : 4);
    // Log-prob rows that lie on the logits (fp32 rows without drafts, in place): the token is drawn before any of them is written
    const size_t esz = DT == SS_BF16 ? 2 : 4, span = ((size_t)(B - 1) * ra.sb + (size_t)kmax * ra.st + V) * esz;
    const auto on_rows = [&](const void* t) {
        const uintptr_t in = reinterpret_cast<uintptr_t>(t), out = reinterpret_cast<uintptr_t>(recovery_logprobs);
        return out < in + span && in < out + (size_t)B * V * sizeof(float);
    };
    const bool in_place = recovery_logprobs && (on_rows(ra.G) || on_rows(ra.recSp) || on_rows(ra.recSm));
    if ((rows_inside || in_place) && shape.part_chunks < ra.NC) shape = RecShape{1024, ra.NC};
    ra.recovery_logprobs = rows_inside ? recovery_logprobs : nullptr;
    ra.log2z = recovery_logprobs && !rows_inside ? reinterpret_cast<double*>(ws + pl.off_log2z) : nullptr;
    ra.part_chunks = shape.part_chunks;
    ra.parts = (ra.NC + ra.part_chunks - 1) / ra.part_chunks;
    const bool split = ra.parts > 1;
    ra.arrive = reinterpret_cast<uint32_t*>(ws + pl.off_arrive);
    ra.best_v = reinterpret_cast<double*>(ws + pl.off_best_v);
    ra.best_i = reinterpret_cast<int32_t*>(ws + pl.off_best_i);
    ra.chunk_tab = reinterpret_cast<Partial*>(ws + pl.off_chunk_tab);
    la.zero_ptr = ra.arrive;
    la.zero_n = split ? B : 0;
    const size_t ratio = (size_t)2 * kmax * (sizeof(Partial) + sizeof(float)), smem = ratio + (size_t)ra.NC * sizeof(Partial);

    const int kind = (ra.greedy ? 1 : 0) | (ra.plain ? 2 : 0);
    // The call whose stages are timed has them one behind the other.
    const OncePlan once = once_plan(pl, B, kmax, V, ra.NC, DT, ra.plain != 0, ra.greedy != 0, ragged, device_cu_count());
    if (once.taken && !ev && windows == 1 && !recovery_logprobs) {
        static void (*const kernels[4])(OnceArgs) = {block_once_kernel<DT, VEC, false, false>, block_once_kernel<DT, VEC, true, false>,
                                                     block_once_kernel<DT, VEC, false, true>, block_once_kernel<DT, VEC, true, true>};
        const OnceArgs oa{ra, reinterpret_cast<unsigned long long*>(ws + pl.off_partial), once.stride, next_call_tag(), once.space};
        launch(kernels[kind], dim3((unsigned)(B * (kmax + 1) * once.space.parts)), dim3(kOnceWaves * kWave),
               once_lds(kmax, ra.NC, ra.greedy != 0), stream, oa);
        return hipGetLastError();
    }

    mark(0);
    for (int i = 0; i < windows; ++i) {
        const Window& w = wins[i];
        const bool listed = ragged || i > 0;
        ra.NS = w.NS;
        ra.t_lo = w.t_lo;
        ra.t_hi = w.t_hi;
        if (kmax > 0)
            launch_row_pass<DT, VEC>(la, w, RowWindow{listed ? ra.draft_len : nullptr, i > 0 ? state : nullptr, kmax, w.t_lo, w.t_hi},
                                     listed ? 0 : w.t_hi, lists[i > 0], partial, stream);
        la.zero_n = 0;
        if (i == 0) mark(1);
        if (i + 1 < windows) {
            const bool few = w.t_hi - w.t_lo <= 8;
            launch(few ? verdict_kernel<DT, 128> : verdict_kernel<DT, 512>, dim3((unsigned)B), dim3(few ? 128 : 512),
                               ratio, stream, ra);
        }
        if (i == 0) mark(2);
    }
    mark(3);
    // accept + recover: LDS holds the per-position log-probs and one mass per recovery chunk
    const dim3 rec_grid((unsigned)(B * ra.parts));
    using RecKernel = void (*)(RecArgs);
    static const RecKernel rec_kernels[3][4] = {  // [256, 512, 1024 threads][greedy | plain << 1]
        {accept_recover_kernel<DT, VEC, false, false, 256>, accept_recover_kernel<DT, VEC, true, false, 256>,
         accept_recover_kernel<DT, VEC, false, true, 256>, accept_recover_kernel<DT, VEC, true, true, 256>},
        {accept_recover_kernel<DT, VEC, false, false, 512>, accept_recover_kernel<DT, VEC, true, false, 512>,
         accept_recover_kernel<DT, VEC, false, true, 512>, accept_recover_kernel<DT, VEC, true, true, 512>},
        {accept_recover_kernel<DT, VEC, false, false, 1024>, accept_recover_kernel<DT, VEC, true, false, 1024>,
         accept_recover_kernel<DT, VEC, false, true, 1024>, accept_recover_kernel<DT, VEC, true, true, 1024>}};
    const long per = kLogprobThreads * kLogprobUnroll;  // vectors of a segment of a log-prob row
    const int segs = V / VEC > per ? (int)((V / VEC + per - 1) / per) : 1;
    const bool rows_apart = recovery_logprobs && !rows_inside;
    ra.defer = split && (kmax == 0 || rows_apart) ? 1 : 0;
    if (ra.defer) {
        static const RecKernel mass[4] = {row_mass_kernel<DT, VEC, false, false>, row_mass_kernel<DT, VEC, true, false>,
                                          row_mass_kernel<DT, VEC, false, true>, row_mass_kernel<DT, VEC, true, true>};
        static const RecKernel draw[4] = {row_draw_kernel<DT, VEC, false, false>, row_draw_kernel<DT, VEC, true, false>,
                                          row_draw_kernel<DT, VEC, false, true>, row_draw_kernel<DT, VEC, true, true>};
        if (kmax == 0) {
            ra.parts = (ra.NC + kMassWaves - 1) / kMassWaves;
            launch(mass[kind], dim3((unsigned)(B * ra.parts)), dim3(kMassWaves * kWave), 0, stream, ra);
        } else {
            launch(rec_kernels[shape.threads >> 9][kind], rec_grid, dim3((unsigned)shape.threads), smem, stream, ra);
        }
        ra.segs = rows_apart ? segs : 0;
        ra.recovery_logprobs = recovery_logprobs;
        launch(draw[kind], dim3((unsigned)(B * (ra.segs + 1))), dim3(kLogprobThreads), smem, stream, ra);
    } else {
        launch(rec_kernels[shape.threads >> 9][kind], rec_grid, dim3((unsigned)shape.threads), smem, stream, ra);
        if (rows_apart) {
            const LogprobArgs pa{ra.G, ra.recSp, ra.recSm, ra.accepted_len, ra.log2z, recovery_logprobs, ra.sb, ra.st, V,
                                 segs, ra.c, ra.bc};
            launch(ra.plain ? recovery_logprob_kernel<DT, VEC, true> : recovery_logprob_kernel<DT, VEC, false>,
                               dim3((unsigned)(B * segs)), dim3(kLogprobThreads), 0, stream, pa);
        }
    }
    mark(4);
    const hipError_t launch_err = hipGetLastError();
    return launch_err != hipSuccess ? launch_err : ev_err;
}

ss_status verify_block_impl(const void* G, const void* S_ctx, const void* S_noctx, const int32_t* draft,
                            const int32_t* draft_len, const float* uniforms, const ss_params* params,
                            int32_t* accepted_len, int32_t* next_token, float* next_token_logprob,
                            float* recovery_logprobs, float* draft_logprobs, void* workspace,
                            size_t workspace_bytes, void* stream, hipEvent_t* ev, bool unbound = false) {
    if (!params) return SS_ERR_NULL;
    if (params->dtype != SS_F32 && params->dtype != SS_BF16) return SS_ERR_DTYPE;
    if (!shape_ok(params)) return SS_ERR_SHAPE;
    if (!G || !S_ctx || !S_noctx || !uniforms || !accepted_len || !next_token) return SS_ERR_NULL;
    if (params->k_max > 0 && !draft) return SS_ERR_NULL;
    if (!(params->lambda > 0.f) || !std::isfinite(params->lambda)) return SS_ERR_PARAM;
    if (!(params->temperature > 0.f) || !std::isfinite(params->temperature)) return SS_ERR_PARAM;
    if (!std::isfinite(params->beta)) return SS_ERR_PARAM;
    if ((params->flags & ~(uint32_t)(SS_FLAG_GREEDY | SS_FLAG_FULL_ROWS)) != 0) return SS_ERR_PARAM;
    const long V = params->vocab;
    if (params->stride_t < 0 || params->stride_b < 0) return SS_ERR_STRIDE;
    const long st = params->stride_t ? params->stride_t : V;
    const long sb = params->stride_b ? params->stride_b : (long)(params->k_max + 1) * st;
    if (st < V || sb < (long)params->k_max * st + V) return SS_ERR_STRIDE;
    // logits must sit on element boundaries; the 16-byte loads themselves need no more than that
    const uintptr_t esz = params->dtype == SS_BF16 ? 2 : 4;
    if (((reinterpret_cast<uintptr_t>(G) | reinterpret_cast<uintptr_t>(S_ctx) | reinterpret_cast<uintptr_t>(S_noctx)) &
         (esz - 1)) != 0)
        return SS_ERR_STRIDE;
    const Plan pl = make_plan(params, workspace_bytes);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 || workspace_bytes < pl.bytes)
        return SS_ERR_WORKSPACE;
    if (params->batch == 0) return SS_OK;

    char* ws = static_cast<char*>(workspace);

    const double T = (double)params->temperature;
    const double c = kLog2e / T;
    const float c_hi = (float)c;  // the row pass scales by this; the merge repairs the difference

    LseArgs la;
    la.G = G; la.Sm = S_noctx; la.row_off = nullptr; la.partial = nullptr; la.draft = nullptr; la.draft_logit = nullptr; la.uniform_rows = 0;
    la.win = RowWindow{nullptr, nullptr, params->k_max, 0, params->k_max};
    la.sb = sb; la.st = st; la.B = params->batch; la.kmax = params->k_max; la.V = params->vocab;
    la.NS = 0; la.slice_vecs = 0; la.list_in_lds = 0; la.c_hi = c_hi;
    la.zero_ptr = nullptr; la.zero_n = 0;

    RecArgs ra;
    const bool steer = params->beta != 0.f;
    ra.G = G; ra.Sm = S_noctx; ra.recSp = steer ? S_ctx : G; ra.recSm = steer ? S_noctx : G; ra.draft = draft; ra.draft_len = draft_len; ra.uniforms = uniforms;
    ra.accepted_len = accepted_len; ra.next_token = next_token;
    ra.next_token_logprob = next_token_logprob;
    ra.draft_logprobs = draft_logprobs; ra.sb = sb; ra.st = st; ra.B = params->batch; ra.kmax = params->k_max;
    ra.V = params->vocab; ra.NS = 0; ra.NC = 0; ra.c = c;
    ra.bc = (double)params->beta * c; ra.lambda = (double)params->lambda;
    ra.rho = (c - (double)c_hi) / (double)c_hi;
    ra.beta = (double)params->beta;
    ra.greedy = (params->flags & SS_FLAG_GREEDY) ? 1 : 0;
    ra.plain = steer ? 0 : 1;
    ra.c_hi = c_hi;
    ra.defer = 0; ra.segs = 0;
    ra.parts = 1; ra.part_chunks = 0; ra.chunk_tab = nullptr; ra.best_v = nullptr; ra.best_i = nullptr; ra.arrive = nullptr;

    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t err;
    if (params->dtype == SS_BF16) {
        err = launch_all<SS_BF16, 8>(la, ra, pl, ws, recovery_logprobs, unbound, s, ev);
    } else {
        err = launch_all<SS_F32, 4>(la, ra, pl, ws, recovery_logprobs, unbound, s, ev);
    }
    return err == hipSuccess ? SS_OK : SS_ERR_DEVICE;
}

// ------------------------------------------------------------------ library-owned scratch for callers that cannot allocate

// specsteer_verify_block_static runs the block with this array as its workspace.  Every GPU the library runs
// on holds its own copy until the process ends.  In host code the array's name is only a handle for the lookup
// below, never an address to hand to a kernel: the device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[SS_STATIC_SCRATCH_BYTES];

// Device address of `scratch` on the current device (looked up with that device current, on the first call
// there); NULL if the lookup fails.  Host threads may race to fill an entry, all with the same value.
void* static_scratch_ptr() {
    static std::atomic<void*> ptrs[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    void* p = ptrs[dev].load(std::memory_order_acquire);
    if (!p) {
        void* q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) return nullptr;
        ptrs[dev].store(q, std::memory_order_release);
        p = q;
    }
    return p;
}

}  // namespace

extern "C" {

size_t specsteer_workspace_bytes(const ss_params* params) {
    if (!shape_ok(params)) return 0;
    return make_plan(params).bytes;
}

ss_status specsteer_verify_block(const void* G, const void* S_ctx, const void* S_noctx, const int32_t* draft,
                                 const int32_t* draft_len, const float* uniforms, const ss_params* params,
                                 int32_t* accepted_len, int32_t* next_token, float* next_token_logprob,
                                 float* recovery_logprobs, float* draft_logprobs, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    return verify_block_impl(G, S_ctx, S_noctx, draft, draft_len, uniforms, params, accepted_len, next_token,
                             next_token_logprob, recovery_logprobs, draft_logprobs, workspace, workspace_bytes,
                             stream, nullptr);
}

ss_status specsteer_verify_block_unbound(const void* G, const void* S_ctx, const void* S_noctx, const int32_t* draft,
                                         const int32_t* draft_len, const float* uniforms, const ss_params* params,
                                         int32_t* accepted_len, int32_t* next_token, float* next_token_logprob,
                                         float* recovery_logprobs, float* draft_logprobs, void* workspace,
                                         size_t workspace_bytes, void* stream) {
    return verify_block_impl(G, S_ctx, S_noctx, draft, draft_len, uniforms, params, accepted_len, next_token,
                             next_token_logprob, recovery_logprobs, draft_logprobs, workspace, workspace_bytes,
                             stream, nullptr, true);
}

ss_status specsteer_verify_block_timed(const void* G, const void* S_ctx, const void* S_noctx, const int32_t* draft,
                                       const int32_t* draft_len, const float* uniforms, const ss_params* params,
                                       int32_t* accepted_len, int32_t* next_token, float* next_token_logprob,
                                       float* recovery_logprobs, float* draft_logprobs, void* workspace,
                                       size_t workspace_bytes, void* stream, float* stage_ms) {
    if (!stage_ms) return SS_ERR_NULL;
    for (int i = 0; i < SS_NUM_STAGES; ++i) stage_ms[i] = 0.f;
    hipEvent_t ev[SS_NUM_STAGES + 1];
    int made = 0;
    for (; made <= SS_NUM_STAGES; ++made)
        if (hipEventCreate(&ev[made]) != hipSuccess) break;
    ss_status st = SS_ERR_DEVICE;
    if (made == SS_NUM_STAGES + 1) {
        st = verify_block_impl(G, S_ctx, S_noctx, draft, draft_len, uniforms, params, accepted_len, next_token,
                               next_token_logprob, recovery_logprobs, draft_logprobs, workspace, workspace_bytes,
                               stream, ev);
        if (st == SS_OK && params->batch > 0) {
            if (hipEventSynchronize(ev[SS_NUM_STAGES]) != hipSuccess) st = SS_ERR_DEVICE;
            for (int i = 0; st == SS_OK && i < SS_NUM_STAGES; ++i)
                if (hipEventElapsedTime(&stage_ms[i], ev[i], ev[i + 1]) != hipSuccess) st = SS_ERR_DEVICE;
        }
    }
    for (int i = 0; i < made; ++i) (void)hipEventDestroy(ev[i]);
    return st;
}

ss_status specsteer_verify_block_static(const void* G, const void* S_ctx, const void* S_noctx, const int32_t* draft,
                                        const int32_t* draft_len, const float* uniforms, const ss_params* params,
                                        int32_t* accepted_len, int32_t* next_token, float* next_token_logprob,
                                        float* recovery_logprobs, float* draft_logprobs, void* stream) {
    if (!params) return SS_ERR_NULL;
    if (params->dtype != SS_F32 && params->dtype != SS_BF16) return SS_ERR_DTYPE;
    if (!shape_ok(params)) return SS_ERR_SHAPE;
    if (make_plan(params).bytes > (size_t)SS_STATIC_SCRATCH_BYTES) return SS_ERR_WORKSPACE;  // block too large for the static scratch
    void* ws = static_scratch_ptr();
    if (!ws) return SS_ERR_DEVICE;
    return verify_block_impl(G, S_ctx, S_noctx, draft, draft_len, uniforms, params, accepted_len, next_token,
                             next_token_logprob, recovery_logprobs, draft_logprobs, ws, (size_t)SS_STATIC_SCRATCH_BYTES,
                             stream, nullptr);
}

int specsteer_first_window(const ss_params* params) {
    if (!shape_ok(params)) return -1;
    return first_window(params);
}

const char* specsteer_status_string(int status) {
    switch (status) {
        case SS_OK: return "ok";
        case SS_ERR_NULL: return "a required pointer is NULL";
        case SS_ERR_SHAPE: return "batch, k_max or vocab out of range";
        case SS_ERR_DTYPE: return "unknown logits dtype";
        case SS_ERR_PARAM: return "lambda, beta, temperature or flags out of range";
        case SS_ERR_STRIDE: return "strides negative or rows overlap";
        case SS_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case SS_ERR_DEVICE: return "HIP launch failed";
        default: return "unknown status";
    }
}

int specsteer_version(void) { return 100; }

}  // extern "C"
