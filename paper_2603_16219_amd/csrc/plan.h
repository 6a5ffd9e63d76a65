// Host-side planning of the block: row windows, slices, the shape of the recovery launch and the layout of the
// workspace.  Plain C++ with no device code, so that the rules can be checked without a GPU.
#pragma once

#include <cstddef>
#include <cstdint>

#include "specsteer.h"

namespace {

constexpr int kWave = 64;  // lanes of a wavefront

// Launch-shape constants of the row pass; the defaults are the measured optimum on MI355X for
// the B=256, V=128256 bf16 workload and can be overridden at build time for other sweeps.
#ifndef SS_LSE_UNROLL
#define SS_LSE_UNROLL 4
#endif
#ifndef SS_LSE_WG_PER_CU
#define SS_LSE_WG_PER_CU 4
#endif
#ifndef SS_LSE_MAX_SLICE_VECS
#define SS_LSE_MAX_SLICE_VECS 4096
#endif
constexpr int kLseUnroll = SS_LSE_UNROLL;   // 16-byte loads in flight per lane
constexpr int kLseWgPerCu = SS_LSE_WG_PER_CU;  // persistent workgroups per CU
constexpr int kMinSliceVecs = kWave * kLseUnroll;  // smallest slice: one unrolled group
constexpr int kMaxSliceVecs = SS_LSE_MAX_SLICE_VECS;  // 64 KiB of logits per slice
constexpr int kMaxSlices = 64;
constexpr int kMaxLdsBatch = 8192;          // ragged batches up to this size keep their row list in LDS
// Arrival counters of different sequences lie 256 bytes apart: atomics on one cache line are served one after the
// other, 7.4 ns each (4800 arrivals on 64 neighbouring counters: 36 us; 256 or 64 bytes apart: no queue).
constexpr int kArriveStride = 64;
constexpr int kChunkSteps = 4;              // recovery chunk = 4 wave-steps (2048 bf16 logits)

struct Partial {
    int E;    // integer exponent reference of this slice
    float s;  // sum over the slice of 2^(h*c - E)
};

constexpr int kMaxWindows = 12;  // first window of one position, each next one as long as all before it: 1024 positions

struct Window {
    int t_lo, t_hi;
    int NS, slice_vecs;  // slices per row, vectors per slice
};

struct Plan {
    int vec;         // logits per 16-byte vector
    int windows;
    Window win[kMaxWindows];
    Window all;      // one pass over all k_max positions (taken when draft_logprobs is requested)
    size_t off_list2, off_log2z, off_state, off_partial;
    bool draft_logit;  // there is space for the draft tokens' logits
    size_t off_draft_logit;
    bool split;      // the tables of a shared recovery row are there
    size_t off_arrive, off_best_v, off_best_i, off_chunk_tab;
    size_t bytes;
};

constexpr int kSplitMaxBatch = 128;  // workspace is reserved for shared recovery rows up to this batch (half of MI355X's 256 units)

// Shape of the recovery launch: threads per workgroup, and chunks per part of a recovery row.
//   - So few chunks that 4-wave workgroups with one chunk a wave leave at most 8 waves per compute unit: spread
//     them like that, since a chunk's arithmetic (some 1.5 us alone on a SIMD) takes as long as four of them
//     sharing one.  With 8 sequences of V = 151936 (75 chunks) the recovery kernel goes from 17.2 us (40
//     workgroups of 16 waves) to 11.5; beyond that line the parts' repeated ratio tests weigh more than the
//     spread gains (64 such sequences: 69.4 us a step in 19 parts,
//     68.0 in 4).
//     Not where one 16-wave workgroup takes the row in a round and the hand-over between parts, or the ratio test by
//     fewer waves, costs more (us a step of 8 sequences, 16 waves -> spread): from 5 to 8 chunks (4 drafts, V = 6166
//     11.4 -> 12.7, V = 14400 12.8 -> 13.4; 10 chunks 14.5 -> 14.1); up to 16 with no draft, where parts cost a
//     launch of their own (rows of V = 6166, 14400 or 32768 11.4 -> 14.5, the host's time), or with more than 16 drafts (V = 20000, 20
//     drafts: 17.0 -> 17.4, 32 18.4 -> 18.9); a single part of 4 waves with more than 8 drafts (V = 2000, 12 drafts: 12.1 ->
//     12.4).  Beyond 16 chunks up to 32 drafts (V = 151936: 24 drafts 27.1 -> 24.8, 32 30.8 -> 29.1; one sequence of V = 40000,
//     48 drafts: 17.1 -> 17.9).
//     The blocks of up to 16 drafts in these figures take one launch now, but for calls that want log-prob rows. What still comes here,
//     spread instead of 16 waves, as multiples of the time in the middle of some 200 calls each: 17 to 32 drafts up to 4 chunks 1.09, 5 to 8
//     1.08 to 1.14, 9 to 12 1.03 to 1.07, 13 to 16 1.00; 9 to 16 drafts with log-prob rows up to 4 chunks 1.08.
//   - At least two compute units per sequence: as many 16-wave parts as there are units per sequence, and no more than rounds of
//     16 chunks (80 sequences of V = 100000, 49 chunks: 38.5 us a step in 2 equal parts of two rounds, 36.9 in 3 of 17, 36.2 with
//     the chunk over dealt out in quarters).
//   - Up to one sequence per unit: one 16-wave workgroup each.  More: 8-wave workgroups, two to a unit, so that the
//     serial ends of one sequence (ratio test, token pick) overlap the sweep of another (300 sequences of
//     V = 100000: 132 us a step against 137 in balanced parts and 140 with 16 waves).
struct RecShape {
    int threads, part_chunks;
};

inline RecShape recovery_shape(int B, int NC, int kmax, int cus, bool split) {
    const bool spread = NC <= 4 ? kmax <= 8 : NC <= 16 ? NC > 8 && kmax > 0 && kmax <= 16 : kmax <= 32;
    if (split && spread && (long)B * NC <= 8l * cus) return {256, 4};
    if (split && B <= cus / 2) {
        const int rows = (NC + 15) / 16;  // rounds of 16 chunks
        const int most = cus / B < rows ? cus / B : rows;
        return {1024, (NC + most - 1) / most};
    }
    return {B <= cus ? 1024 : 512, NC};
}

// Whether rows without a draft that recovery_shape would cut into parts are taken whole by one 16-wave workgroup each.  Parts
// cost a second launch, 2.3 us of the host's time, and spread a row over the chip.
//   In a captured graph launches cost the host nothing, and the GPU's time decides (us on the GPU in two launches -> in one, bf16 rows
// without a steering term: 1 of 17 chunks 6.2 -> 6.6, of 76 6.0 -> 11.9; 32 of 20 7.3 -> 7.1, of 24 7.5 -> 7.8; 64 of 20 7.8 -> 7.6, of 75 9.8 ->
// 13.0; 96 of 28 8.5 -> 8.4, of 36 8.9 -> 9.2; 128 of 36 9.5 -> 9.2, of 44 10.2 -> 10.2; fp32: 1 of 24 5.3 -> 5.2, of 32 5.4 -> 5.7; 64 of 32
// 7.6 -> 7.6, of 40 7.8 -> 8.2; 128 of 40 9.2 -> 8.6, of 64 10.9 -> 11.4; with one, fp32: 96 of 17 9.6 -> 10.3, 128 of 17 11.2 -> 10.7, of 24
// 12.7 -> 12.9; bf16: 128 of 17 12.3 -> 12.5).
//   Outside of one, but for the binding's native wrappers (csrc/calls.cpp), whose host time is less than the GPU's, the lines are where
// back-to-back calls with some 9 us of host time beside the launches (marshalling and three allocations in Python) are as fast either way:
// they are bound by the host, 14.3 us in
// two launches whatever the size, 11.4 in one until the rate of one compute unit (or, with a steering term, its
// arithmetic) takes over.  A caller with less host time of its own, or whose host runs ahead of the GPU, pays up to twice the GPU's
// time for it between these lines and those above; it gets the other shape by capturing the call.  Us a call in two launches -> in
// one, by chunks of a row:
//   - sampled rows, bf16: 32 rows of 64 chunks 14.2 -> 11.7, of 76 13.4 -> 13.3, of 80 14.2 -> 14.5; 64 of 75 (V = 151936) 14.6 ->
//     13.4; 128 of 76 14.1 -> 14.0, of 80 14.3 -> 15.1; 8 of 80 13.6 -> 13.4, of 88 14.3 -> 14.2.
//   - sampled rows, fp32: 8 of 112 14.2 -> 12.4, of 149 14.2 -> 15.2; 32 of 100 14.3 -> 12.9, of 112 14.2 -> 14.2; 64 of 100
//     14.4 -> 13.6, of 112 14.4 -> 14.9; 128 of 92 14.3 -> 14.2, of 100 14.3 -> 14.8.
//   - steered rows, bf16: 8 of 28 14.3 -> 12.9, of 30 14.3 -> 14.4; 32 of 25 14.3 -> 13.5, of 32 14.5 -> 15.6; 128 of 24
//     14.3 -> 13.7, of 26 14.4 -> 14.7.
//   - steered rows, fp32: 8 of 36 14.3 -> 12.5; 32 of 33 14.2 -> 13.6, of 36 14.2 -> 14.4; 128 of 28 14.4 -> 13.6, of 30 14.4 -> 14.6.
//   - greedy, where every logit is compared too: bf16 rows without a steering term 8 of 52 13.4 -> 12.2, 128 of 52 14.2 -> 13.1,
//     32 of 60 13.5 -> 13.8; fp32 64 of 92 14.3 -> 13.9, of 104 14.2 -> 14.8; steered bf16 128 of 20 14.3 -> 13.9, 32 of 22 14.2 ->
//     14.5; steered fp32 as sampled.
inline bool rows_in_one_launch(int B, int NC, int dtype, bool plain, bool greedy, bool captured) {
    if (captured) return plain ? NC <= (dtype == SS_BF16 ? 11 + B / 5 : 24 + B / 8) : dtype == SS_F32 && B > 112 && NC <= 20;
    if (greedy && plain) return NC <= (dtype == SS_BF16 ? 56 : B <= 64 ? 92 : 84);
    if (greedy) return NC <= (dtype == SS_BF16 ? 20 : B <= 32 ? 32 : 28);
    if (plain) return NC <= (dtype == SS_BF16 ? (B <= 8 ? 84 : 76) : B <= 8 ? 120 : B <= 64 ? 104 : 92);
    return NC <= (dtype == SS_BF16 ? (B <= 8 ? 28 : 24) : B <= 32 ? 34 : 28);
}

// Whether the recovery launch writes the requested log-prob rows itself, its row in one part, or a launch of their own does.
// A launch costs 2.5 us of host time, which is what such small calls take; the workgroup that drew the token takes longer
// over its row than the chip does, which counts the sooner, the more drafted rows the call has.  By the bytes of a row, three
// read and one written (us a call, a launch of its own -> inside; bf16, 4 drafts): one sequence of V = 1000 20.1 -> 17.8, of
// V = 32000 20.4 -> 18.7, of V = 40000 20.5 -> 20.9; 2 of V = 32000 22.2 -> 19.8, of V = 40000 20.7 -> 23.0; 4 of V = 32000
// 20.4 -> 21.0; 8 of V = 24000 20.7 -> 19.1 (16 drafts 21.7 -> 21.7); 16 of V = 20000 22.0 -> 20.7 (16 drafts 22.1 -> 23.2);
// 100 of V = 16384 23.9 -> 23.2, 600 of them 72.6 -> 67.4.
inline bool logprobs_in_recovery(int B, int kmax, int V, int esz) {
    const long drafts = (long)B * kmax, row = (long)V * (3 * esz + 4);
    return row <= (B <= 16 && drafts <= 128 ? (drafts <= 4 ? 384l : drafts <= 8 ? 320l : 256l) : 164l) << 10;
}

// Several row passes pay off when the batch is large enough to be bandwidth-bound and long enough for
// a first rejection to cut rows: a first window is scored for everyone, what follows only for the sequences that
// are still in play.  A further window costs some 10 us (a verdict launch, and the ends of a row pass), the time of
// 66 MB of rows.
//   - From kEarlyExitMinBytes of rows: a first window of a quarter of the positions and one of the rest (256 ragged
//     sequences of up to 16 positions, V = 128256: 4 and 12; cut into 4, 4 and 8 it gains 2 us of 168 at
//     acceptance 0.8 and loses 10 where nearly everything is accepted).  Below it a second window pays or not by what is
//     accepted, which the host does not know: 64 sequences of 8 positions, V = 151936 (311 MB), 69.1 us a step in one window,
//     67.4 in 4 and 4, 70.5 in 2 and 6 at acceptance 0.8; 69.9, 52.5 and 46.6 at 0.4; 69.1, 78.1 and 79.7 where nearly
//     everything is accepted.
//   - From doubling_min_bytes of rows a position, the rows behind one position are already worth a launch: windows of
//     1, 1, 2, 4, ... positions.  512 sequences of 8 positions, V = 256000 bf16 (500 MiB a position): 362 -> 298 us a step
//     at acceptance 0.4, 603 -> 525 at 0.8.
constexpr long kEarlyExitMinBytes = 512l << 20;

// What doubling windows gain falls with the rows of a position, with the positions behind the first ones (fewer of
// them in ragged drafts) and with the share that is accepted, of which the threshold lambda is what the host knows.
// Microseconds a step in two windows -> in doubling ones (ragged drafts in brackets), 495 or 512 sequences, bf16, a recipe
// of acceptance 0.8 at lambda 0.5:
//   - 6 positions and more, from 240 MiB.  At 242 MiB 16 of them 408 -> 329 (297 -> 281), 8 294 -> 276 (213 -> 220), 6
//     270 -> 250 (197 -> 205); at 280 MiB 8 of them 346 -> 307 (247 -> 243).  At 140 MB (273 sequences, V = 128256)
//     184 -> 190.
//   - 4 and 5 positions, from 280 MiB: 4 of them 244 -> 237 (194 -> 199), 5 270 -> 255 (204 -> 205); at 242 MiB 211 -> 214
//     (168 -> 178) and 237 -> 237 (181 -> 191).
//   - lambda below 0.4, from 280 MiB: at 0.3 8 positions 357 -> 339 (250 -> 258); at 242 MiB 313 -> 307 (222 -> 237).
//   - lambda below 0.2, from 480 MiB: at 0.1 8 positions of 500 MiB 722 -> 676 (480 -> 468), of 375 MiB 528 -> 517 (356 -> 369),
//     of 242 MiB 358 -> 368 (237 -> 262); at 0.01, where nearly everything is accepted, 794 -> 794 (514 -> 517), 585 -> 602
//     (382 -> 406) and 386 -> 419 (251 -> 283), though a poorer specialist gains there too (500 MiB: 516 -> 425).
inline long doubling_min_bytes(const ss_params* p) {
    if (!(p->lambda >= 0.2f)) return 480l << 20;
    return (p->lambda < 0.4f || p->k_max < 6 ? 280l : 240l) << 20;
}

inline long position_bytes(const ss_params* p) {  // both tensors' rows of one position, all sequences
    return 2l * p->batch * p->vocab * (p->dtype == SS_BF16 ? 2 : 4);
}

inline int first_window(const ss_params* p) {
    if (p->flags & SS_FLAG_FULL_ROWS) return p->k_max;
    if (p->k_max < 4) return p->k_max;
    if (position_bytes(p) * p->k_max < kEarlyExitMinBytes) return p->k_max;
    return position_bytes(p) >= doubling_min_bytes(p) ? 1 : p->k_max / 4;
}

inline bool shape_ok(const ss_params* p) {
    if (!p) return false;
    if (p->batch < 0 || p->k_max < 0 || p->k_max > SS_MAX_K) return false;
    if (p->vocab < 1 || p->vocab > SS_MAX_VOCAB) return false;
    if (p->dtype != SS_F32 && p->dtype != SS_BF16) return false;
    if ((long)p->batch * (p->k_max + 1) > (1l << 30)) return false;
    return true;
}

// Small blocks in one launch (block_once_kernel): a wave forms the slice partials and the recovery mass of one chunk of one position, so
// that nothing is left behind the ratio test but the draw.  Parts of kOnceWaves chunks.  In the workspace, per sequence and in 8-byte
// words: the claim, then for each part its partials (four words, a draft's position) or that it has arrived (one, the bonus
// position), its greedy candidate (two), and a mass for each chunk of every position.
constexpr int kOnceWaves = 4;
constexpr int kOnceMaxDrafts = 16;
constexpr int kOnceMaxParts = 16;  // of a position: a lane each of the sixteen that merge it
struct OnceSpace {
    int parts;  // of a position
    long flags, best, masses, words;
};
inline OnceSpace once_space(int kmax, int NC, bool greedy) {
    OnceSpace s;
    s.parts = (NC + kOnceWaves - 1) / kOnceWaves;
    const long positions = (long)kmax + 1;
    s.flags = 2 + 4l * kmax * s.parts;  // the partials lie before them, from word 2 on
    s.best = s.flags + s.parts;
    s.masses = s.best + (greedy ? 2 * positions * s.parts : 0);
    s.words = s.masses + positions * NC;
    return s;
}

// Its LDS: the masses, the rows' merged partials, what the parts delivered of them, and the candidates of a sequence.
inline size_t once_lds(int kmax, int NC, bool greedy) {
    const size_t positions = (size_t)kmax + 1, parts = (size_t)(NC + kOnceWaves - 1) / kOnceWaves;
    return positions * NC * sizeof(Partial) + 2 * kmax * sizeof(double) + 4 * kmax * parts * sizeof(unsigned) +
           (greedy ? positions * parts * (sizeof(double) + sizeof(int)) : 0);
}

// Which blocks, by workgroups a compute unit.  The third rows of all positions are read and summed for one of them, which costs nothing while
// units are idle; beyond, a row pass and a recovery that share the chip's arithmetic take less.  Us a step by graph replays, two
// launches -> one, by workgroups on 256 units:
//   - bf16, up to 2 1/8: 144 (1 sequence of 8 drafts, V = 128256) 13.5 -> 10.4, 252 (4 of 8, V = 50257) 14.3 -> 10.5, 504 (8 of 8, V = 50257) 15.4 ->
//     13.3, 544 (2 of 16, V = 128256) 15.6 -> 14.6; 576 (16 of 8, V = 32000) 14.7 -> 15.1, 640 (8 of 4, V = 128256) 14.8 -> 15.3, 864 16.1 -> 17.6.
//   - bf16 with lengths, of whose workgroups some have nothing to do, or without a steering term, up to 3: lengths 576 14.8 -> 13.1, 768 15.4
//     -> 14.3 (all of full length 768 15.9 -> 15.95, 702 15.3 -> 15.5); without 576 12.6 -> 11.9, 768 13.5 -> 12.1.
//   - fp32, whose chunks are half the logits, up to 4: 40 (1 of 4, V = 32000) 10.1 -> 7.7, 512 (16 of 1, V = 65536) 13.4 -> 11.7, 624 (6 of 12, V = 32000)
//     14.3 -> 12.9, 768 13.8 -> 13.2, 832 (4 of 12, V = 65536) 15.8 -> 15.0, 1024 15.75 -> 15.6.
//   - Greedy with a steering term compares every logit in double: bf16 up to 1 (224 15.0 -> 12.7; 336 14.8 -> 15.5), fp32 up to 1 1/2 (384 13.4
//     -> 12.75); without one up to 2 (512 14.2 -> 12.6).
// Rows of up to 8 chunks, which a recovery takes in one workgroup a sequence without a hand-over, gain less:
//   - Greedy ones of less than 5 whole chunks nothing, but for fp32 without a steering term: one wave forms all the sums of its chunk, those in double and
//     those past the row's end among them. bf16, 160 (32 of 4, V = 40) 9.2 -> 11.4, 15 (3 of 4, V = 1000) 9.2 -> 11.2, 95 (19 of 4, V = 8192) 11.6
//     -> 12.5, without a steering term 255 (51 of 4, V = 1000) 9.2 -> 9.8; fp32, 255 (51 of 4, V = 40) 8.4 -> 9.6, 45 (9 of 4, V = 4096) 9.7 -> 10.1.
//   - Other greedy ones gain up to 1, bf16 without a steering term (250, V = 16384 11.2 -> 10.6; 380 11.8 -> 12.3) and fp32 with one (250, V = 8192 11.7 ->
//     10.9; 380 12.4 -> 12.6).
//   - Sampled bf16 up to 2 (480, V = 10240 13.4 -> 12.9; 540 13.7 -> 14.4, V = 9000 13.2 -> 14.6, V = 8192 13.6 -> 15.1), and no further with lengths or
//     without a steering term either from 4 chunks on (lengths 510, V = 9000 13.5 -> 12.9; 640 13.8 -> 15.1).
//   - Sampled fp32 up to 3 (760, V = 8192 14.4 -> 13.1, V = 6166 13.4 -> 13.3; 890 13.7 -> 14.4, 1020 14.3 -> 15.4), with lengths or without a steering term as
//     far as longer rows.
//   - Sampled ones of 4 whole chunks and less than half of a fifth, where every second workgroup has little to do: fp32 up to 2 (552, V = 4344
//     12.1 -> 12.4; 700, V = 4211 11.9 -> 12.7; 742, V = 4242 12.4 -> 13.4, 720, V = 4410 12.6 -> 13.1), with lengths or without a steering term up to 3 (750, V = 4171 11.2 -> 10.8;
//     928, V = 4130 13.3 -> 14.3, 976, V = 4316 13.0 -> 13.9), bf16 up to 1 1/2 (408, V = 8484 12.4 -> 13.1).
inline bool block_in_one_launch(int B, int kmax, int V, int NC, int dtype, bool plain, bool greedy, bool ragged, int cus) {
    if (kmax < 1 || kmax > kOnceMaxDrafts || NC > kOnceMaxParts * kOnceWaves) return false;
    const int chunk = kChunkSteps * kWave * (dtype == SS_BF16 ? 8 : 4);
    const bool bf16 = dtype == SS_BF16, brief = NC <= 8, reduced = plain || ragged, barely = V > 4 * chunk && 2l * V < 9l * chunk;
    if (greedy && (bf16 || !plain) && V < 5 * chunk) return false;
    const int eighths = greedy ? (bf16 ? (plain && !brief ? 16 : 8) : plain ? 16 : brief ? 8 : 12)
                        : bf16 ? (brief ? (reduced ? (NC < 4 ? 24 : 16) : barely ? 12 : 16) : reduced ? 24 : 17)
                               : (barely ? (reduced ? 24 : 16) : brief && !reduced ? 24 : 32);
    return 8l * B * (kmax + 1) * ((NC + kOnceWaves - 1) / kOnceWaves) <= (long)eighths * cus;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

inline int chunks_of(int elems, int vec) {
    const long nvec = elems / vec;
    const long nch = (nvec + kWave * kChunkSteps - 1) / (kWave * kChunkSteps);
    return (int)nch + ((elems % vec) ? 1 : 0);
}

// Whether the recovery sweep can meet a row that it reads from one element before its start: a bf16 row behind the
// tensor's first, at an odd element in all three tensors (`bases`: bit 0 of each tensor's element address).
inline bool odd_rows_possible(int vec, const unsigned (&bases)[3], int B, int kmax, long sb, long st) {
    if (vec != 8 || (bases[0] & 1) != (bases[1] & 1) || (bases[0] & 1) != (bases[2] & 1)) return false;
    return (bases[0] & 1) || (B > 1 && (sb & 1)) || (kmax > 0 && (st & 1));
}

// Most recovery chunks of a row; a row read from one element before its start has those of V + 1.  The launch is shaped
// by what its rows really have: with V a multiple of 2048 the element more is a chunk more, and that chunk may start
// another round of 16.  Counting it where no row is odd gave 64 sequences of V = 131072 3 parts of 22 chunks instead of 4 of
// 16 (a step of 4 drafts 44.3 us, 43.3 without it; steering rows 18.1, 16.8), and 128 of V = 65536 two rounds instead of
// one (43.8, 42.9; rows 17.9, 16.9).  The other way round once in ten sizes: 64 rows of V = 196608 21.9 in 4 parts of 25,
// 22.4 in 3 of 32.  The workspace is laid out for either.
inline int chunks_per_row(int V, int vec, bool odd_rows) {
    const int n = chunks_of(V, vec), m = odd_rows ? chunks_of(V + 1, vec) : n;
    return n > m ? n : m;
}

// Slices per row for a pass expected to cover `row_tensors` (row, tensor) pairs: 64 KiB slices for
// big passes, smaller ones (down to one unrolled group) when there are too few rows to give every
// resident wave several slices -- a wave that gets one or two long slices cannot balance.
inline void slice_plan(long nvec, long row_tensors, int most, Window& w) {
    long ns_lo = (nvec + kMaxSliceVecs - 1) / kMaxSliceVecs;
    long ns_hi = (nvec + kMinSliceVecs - 1) / kMinSliceVecs;
    long want = row_tensors > 0 ? (32768 + row_tensors - 1) / row_tensors : 1;
    long ns = want < ns_lo ? ns_lo : (want > ns_hi ? ns_hi : want);
    if (ns > most) ns = most;
    if (ns < 1) ns = 1;
    long sv = (nvec + ns - 1) / ns;
    sv = (sv + kMinSliceVecs - 1) / kMinSliceVecs * kMinSliceVecs;
    ns = (nvec + sv - 1) / sv;
    if (ns < 1) ns = 1;
    w.NS = (int)ns;
    w.slice_vecs = (int)sv;
}

// Bytes up to the tables of a shared recovery row, the tables themselves when `split` is set, and the draft tokens' logits when
// `logits` is.
inline Plan lay_out(const ss_params* p, bool split, bool logits) {
    Plan pl;
    pl.vec = p->dtype == SS_BF16 ? 8 : 4;
    const long nvec = (p->vocab + pl.vec - 1) / pl.vec;
    // The space of the slice partials: that of one window of all positions and of two, the first a quarter of the
    // positions, at the finest of their slicings.  The windows use it one after the other.
    const int quarter = first_window(p) < p->k_max ? p->k_max / 4 : p->k_max;
    const long rows1 = (long)p->batch * quarter, rows2 = (long)p->batch * (p->k_max - quarter);
    Window two[2];
    slice_plan(nvec, rows1 * 2, kMaxSlices, two[0]);
    // a later window covers only the sequences still in play: typically a third of the padded rows
    slice_plan(nvec, rows2 * 2 / 3, kMaxSlices, two[1]);
    slice_plan(nvec, (long)p->batch * p->k_max * 2, kMaxSlices, pl.all);
    pl.all.t_lo = 0;
    pl.all.t_hi = p->k_max;
    int ns_max = two[0].NS > two[1].NS ? two[0].NS : two[1].NS;
    if (pl.all.NS > ns_max) ns_max = pl.all.NS;
    pl.windows = 0;
    for (int t = 0, hi = first_window(p);; hi = 2 * t) {
        if (t > 0 && (position_bytes(p) < doubling_min_bytes(p) || hi + t / 2 >= p->k_max)) hi = p->k_max;  // no last window shorter than half the one before
        Window& w = pl.win[pl.windows++];
        const long rows = (long)p->batch * (hi - t);
        const long most = hi > t ? (long)p->k_max * ns_max / (hi - t) : kMaxSlices;
        slice_plan(nvec, t == 0 ? rows * 2 : rows * 2 / 3, most < kMaxSlices ? (int)most : kMaxSlices, w);
        w.t_lo = t;
        w.t_hi = hi;
        if (hi >= p->k_max) break;
        t = hi;
    }
    const size_t B = (size_t)p->batch;
    size_t o = align_up((B + 1) * sizeof(int32_t), 256);  // row list of the first pass
    pl.off_list2 = o;    o += align_up((B + 1) * sizeof(int32_t), 256);      // row list of the second pass
    pl.off_log2z = o;    o += 2 * align_up((B ? B : 1) * sizeof(int32_t), 256);  // one double per sequence
    pl.off_state = o;    o += align_up((B ? B : 1) * sizeof(int32_t), 256);
    pl.off_partial = o;
    o += align_up(((size_t)p->batch * p->k_max * 2 + 1) * (size_t)ns_max * sizeof(Partial), 256);
    const size_t NC = (size_t)chunks_per_row(p->vocab, pl.vec, pl.vec == 8);
    pl.split = split && p->batch >= 1 && p->batch <= kSplitMaxBatch;
    pl.off_arrive = pl.off_best_v = pl.off_best_i = pl.off_chunk_tab = o;
    if (pl.split) {
        pl.off_arrive = o;     o += align_up(B * kArriveStride * sizeof(uint32_t), 256);
        pl.off_best_v = o;     o += align_up(B * (NC < 32 ? 32 : NC) * sizeof(double), 256);
        pl.off_best_i = o;     o += align_up(B * NC * sizeof(int32_t), 256);
        pl.off_chunk_tab = o;  o += align_up(B * NC * sizeof(Partial), 256);
    } else if (p->batch >= 1 && p->batch <= kSplitMaxBatch) {
        // not used, and never more than the tables: which blocks fit the static scratch stays what it is
        o += align_up(B * sizeof(uint32_t), 256) + align_up(B * 256, 256) +
             align_up(B * (size_t)chunks_of(p->vocab, pl.vec) * sizeof(Partial), 256);
    }
    pl.draft_logit = logits;
    pl.off_draft_logit = o;
    if (logits) o += align_up((size_t)p->batch * p->k_max * 2 * sizeof(float), 256);
    pl.bytes = o;
    return pl;
}

// The plan with the shared recovery row and the draft tokens' logits, unless only a plan without them fits the static scratch:
// which blocks that entry point takes does not depend on either.
inline Plan make_plan(const ss_params* p) {
    const Plan whole = lay_out(p, true, true);
    if (whole.bytes <= (size_t)SS_STATIC_SCRATCH_BYTES) return whole;
    const Plan split = lay_out(p, true, false);
    if (split.bytes <= (size_t)SS_STATIC_SCRATCH_BYTES) return split;
    const Plan small = lay_out(p, false, false);
    return small.bytes <= (size_t)SS_STATIC_SCRATCH_BYTES ? small : whole;
}

// Whether a block takes one launch, in the workspace of a plan: its words begin where the slice partials would, `stride` of them for each
// sequence.  The workspace's size is that of two launches, which is what callers hold, so space is a second gate behind the lines above.
// From V = 32000 on sampled blocks always fit.  Greedy ones, whose candidates take two words a part, do not from 3 to 6 drafts on in
// fp32 (4 sequences of 3, V = 62209: 586 words, 584 there; 8 of 4, V = 32000: 378, 376) and 4 to 7 in bf16 (3 of 4, V = 100352: 598, 597).  Short rows of more than 128
// sequences, where there are no tables of shared rows, do not.
struct OncePlan {
    bool taken;
    long stride;
    OnceSpace space;
};
inline OncePlan once_plan(const Plan& pl, int B, int kmax, int V, int NC, int dtype, bool plain, bool greedy, bool ragged, int cus) {
    OncePlan o;
    o.space = once_space(kmax, NC, greedy);
    o.stride = B > 0 ? (long)((pl.bytes - pl.off_partial) / sizeof(uint64_t)) / B : 0;
    o.taken = block_in_one_launch(B, kmax, V, NC, dtype, plain, greedy, ragged, cus) && o.space.words <= o.stride;
    return o;
}

// The plan for a workspace of `bytes`, the richest that fits it; make_plan's, which the caller has to refuse, if none does.  Where
// only a plan without the draft tokens' logits fits the static scratch a larger block asks for less than a smaller one (349
// sequences of 1000 drafts, V = 40: 8.0 MiB, 350: 5.3), and a caller that holds what the larger needs can run the smaller without them too.
// Up to kDraftLogitsAsked positions a block lies too far below the static scratch's limit (at most 3.1 MiB) for that, and
// what make_plan says is what it takes.
constexpr long kDraftLogitsAsked = 512;
inline Plan make_plan(const ss_params* p, size_t bytes) {
    const Plan pl = make_plan(p);
    if (bytes >= pl.bytes || !pl.draft_logit || (long)p->batch * p->k_max <= kDraftLogitsAsked) return pl;
    const Plan lean = lay_out(p, true, false);
    return lean.bytes <= bytes ? lean : pl;
}

}  // namespace
