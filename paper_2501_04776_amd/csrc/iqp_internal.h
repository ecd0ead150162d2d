// Internal interface between the host runtime (iqp_api.cpp) and the gfx950
// kernels (iqp_kernels.hip). Not installed; the public ABI is include/iqp.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace iqp {

// Every extent the kernels tile over is padded to a multiple of this.
constexpr int64_t kPad = 128;
// IQP_SPLIT3_BF16: the third theta limb is E4M3(rest * 2^kLo8Exp)
constexpr int kLo8Exp = 20;

// Work slots of one MI355X at one wave per SIMD: 256 CUs x 4 SIMDs.
constexpr int64_t kWaveSlots = 1024;

// Samples per block of the epilogue reduction (fixed: part of the
// deterministic summation order).
constexpr int64_t kEpiChunk = 1024;

__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
__host__ __device__ inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// Tile configuration of the two contractions (wave tile = 32*fm x 32*fn).
struct TileCfg {
    int fm = 4, fn = 4;      // forward: observables x samples
    bool fixed_fwd = false;  // the forward tile was asked for
    int bfm = 2, bfn = 2;    // backward: observables x gates
    int64_t splits = 0;      // forward split over gate words; 0 = choose
    int64_t bsplits = 0;     // backward split over sample words; 0 = choose
    int64_t obgroup = 8;     // backward unit order: observable blocks per group
};

// Kernel-family ids for the optional per-kernel timing.
enum KernelFamily {
    KF_PARITY = 0, KF_THETA, KF_FWD, KF_EPI, KF_FIN, KF_WEIGHTS, KF_BWD, KF_GRAD, KF_MMD,
    KF_COUNT
};

// A launch records (family, start, stop) events when timing is on.
struct LaunchCtx {
    hipStream_t stream;
    bool timing;
};

void timed_begin(const LaunchCtx &lc, int family, hipEvent_t *ev);
void timed_end(const LaunchCtx &lc, int family, hipEvent_t ev);

// Fixed-point backward weights (IQP_SPLIT3_BF16): |S_ki| <= sigma_k maps to
// integers N with |N| <= kI8Max = 127 * 256 + 127, the largest magnitude two
// signed 8-bit limbs hold as N = 256 hi + lo with hi = floor((N + 128) / 256)
// in [-127, 127] and lo in [-128, 127]. Over at most 2^16 samples per work
// unit the INT32 sums of each limb, and 256 hi_sum + lo_sum, stay exact
// (|256 * 127 K + 128 K| < 2^31 for K <= 2^16).
constexpr double kI8Max = 32639.0;
constexpr int64_t kI8MaxSamplesPerUnit = (int64_t)1 << 16;

// Support-list capacity: the qubits of a generator of weight <= kSupCap are
// listed; heavier generators are read from their bit rows.
constexpr int kSupCap = 8;

// The FP32 passes have two ways to the same bits (the FP32 matrix product adds
// one term at a time, in gate or sample order, and adding a zero term changes
// nothing): the matrix cores over all entries of C, or one addition per non-zero
// one. nnz counts C's entries on the device; at most `limit` of them take the
// second way. NULL: always the matrix cores. All kernels of a pass read nnz, so
// none of them may write where it lives.
struct ChainGate {
    const unsigned long long *nnz = nullptr;
    unsigned long long limit = 0;
};

// Observables of weight 0 (most operators of a wide kernel bandwidth) leave the
// dense forward: the others, in any order, are rows 0 .. *nrows - 1 of C and E;
// perm[row] = observable, pos[observable] = row or -1. NULL: all rows, in order.
struct RowPerm {
    const int32_t *perm = nullptr, *pos = nullptr, *nrows = nullptr;
};

// ---- per-step arguments -----------------------------------------------------
// Each step's kernel body takes one of these and a block (or work-unit)
// index. A single-problem launch passes the struct as the kernel argument; a
// batched launch reads one struct per problem from a device array and maps
// its flat block index to (problem, local block) through a prefix sum of the
// per-problem block counts.

// prec: IQP_FP32 (t32 split by gate parity), IQP_SPLIT_BF16 and
// IQP_SPLIT_BF16_FP8 (hi, lo), IQP_SPARSE_FP32 (t32 plain), IQP_SPLIT3_BF16
// (hi, mid, lo).
struct ThetaArgs {
    const double *theta;
    int64_t m, m_pad;
    int prec;
    uint16_t *hi, *lo, *mid;
    float *t32;
    unsigned long long *nnz;  // zeroed when not NULL (ChainGate)
};
inline int64_t blocks_of(const ThetaArgs &a) { return ceil_div(a.m_pad, 256); }

// Bit columns of `rows`: Xt[q * ldx + rw], q < 64 W, rw < ldx (>= ceil(R/64)),
// and a zero column q = 64 W (Xt holds 64 W + 1 columns).
struct BitsliceArgs {
    const uint64_t *rows;
    int64_t R;
    int W;
    int64_t ldx;
    uint64_t *Xt;
};
inline int64_t blocks_of(const BitsliceArgs &a) { return ceil_div(a.ldx * a.W, 4); }

// Finds the observables of weight > 0 (RowPerm; *nrows must read 0).
struct RowPermArgs {
    const uint64_t *ops;
    int64_t l;
    int W;
    int32_t *perm, *pos, *nrows;
};
inline int64_t blocks_of(const RowPermArgs &a) { return ceil_div(a.l, 256); }

// Support lists of `rows` generators (m real ones, W words each; rows >= m
// are written as weight 0): sup[j * kSupCap + k] = qubit of the k-th set bit
// of generator j, -1 past its weight, and sup[j * kSupCap] = -2 for a
// generator heavier than kSupCap.
struct SupportArgs {
    const uint64_t *gens;
    int64_t m;
    int W;
    int64_t rows;
    int32_t *sup;
};
inline int64_t blocks_of(const SupportArgs &a) { return ceil_div(a.rows, 256); }

// Parity of each generator (m of them, W words each, support lists `sup`
// covering 64 Gw rows) against `rows` (R of them, those past R read as 0; Rw
// words of 64 rows), in layout 0 (row-major), 1 (tiled32), 2 (transposed
// tiled32), 3 (transposed row-major) or 4 (transposed word-major); Gw = output
// words per row in layouts 0/1, generator words in the others.
// A block of the kernel takes rw row words and 64 gpb generators; from
// kColumnWords words per row on, and where kColumnWaves says so, rw is 0 and the
// kernel reads the bit columns Xt (ldx words each) that launch_parity makes first.
constexpr int kBitsWordMajor = 4;
constexpr int kColumnWords = 128;
struct ParityArgs {
    const uint64_t *rows;
    int64_t R;
    const uint64_t *gens;
    const int32_t *sup;
    int64_t m;
    int W;
    uint64_t *Xt;
    int64_t ldx;
    int64_t Rw, R_out, Gw;
    uint64_t *out;
    int rw;
    int64_t gpb;
    RowPerm perm = {};  // rows: the first *nrows of them, row i being perm[i]
    ChainGate gate = {};
    int when = 0;  // 1: only for the matrix cores, 2: only for the other way
};
// Row words per block, the most that leave room for two blocks in a CU's LDS,
// and the stride of a qubit's words there: an odd stride (or one of 1 or 2)
// spreads the gathers over the banks.
inline int parity_rw(int W) {
    return W <= 7 ? 16 : W <= 17 ? 8 : W <= 31 ? 4 : W <= 63 ? 2 : W < kColumnWords ? 1 : 0;
}
__host__ __device__ constexpr int parity_stride(int rw) { return rw >= 4 ? rw + 1 : rw; }
// Generators per block so that about three blocks run per CU: the transposes
// that stage a block's rows are paid once for all of them.
inline int64_t parity_gpb(int64_t Gw, int64_t Rw, int rw) {
    const int64_t want = ceil_div(Gw * ceil_div(Rw, rw), 768);
    return want < 4 ? 4 : want > 64 ? 64 : round_up(want, 4);
}
// The parities of rows of 64 words and more (one row word a block, stored a word at
// a time) lose to the bit columns in memory once these kernels' waves, one for 64
// generators and 64 row words, fill the SIMDs: at 10^4 rows, 10^5 generators and 4100
// to 8100 qubits C and B^T row-major at mean weight 3 take 430 us from LDS and 360
// from columns, layouts 0 to 2 at mean weight 20 1.0 to 3.8 times as long (at 3 0.7 to
// 0.9 times). With 939 waves and fewer LDS takes 0.05 to 0.9 times at most weights.
constexpr int64_t kColumnWaves = 1024;
inline ParityArgs parity_args(const uint64_t *rows, int64_t R, const uint64_t *gens,
                              const int32_t *sup, int64_t m, int W, uint64_t *Xt, int64_t ldx,
                              int64_t Rw, int64_t R_out, int64_t Gw, uint64_t *out) {
    ParityArgs a{rows, R, gens, sup, m, W, Xt, ldx, Rw, R_out, Gw, out, parity_rw(W), 4};
    if (W >= 64 && Gw * ceil_div(Rw, 64) >= kColumnWaves) a.rw = 0;
    if (a.rw) a.gpb = parity_gpb(Gw, Rw, a.rw);
    return a;
}
// The same from LDS at any number of waves (bitflip circuits, and forwards that leave
// rows out).
inline ParityArgs parity_from_rows(ParityArgs a) {
    a.rw = parity_rw(a.W);
    if (a.rw) a.gpb = parity_gpb(a.Gw, a.Rw, a.rw);
    return a;
}
inline int64_t blocks_of(const ParityArgs &a) {
    return a.rw ? ceil_div(a.Rw, a.rw) * ceil_div(a.Gw, a.gpb)
                : ceil_div(a.Gw * ceil_div(a.Rw, 64), 4);
}
inline size_t lds_of(const ParityArgs &a) {
    return a.rw ? (size_t)(64 * a.W + 1) * parity_stride(a.rw) * 8 : 0;
}
inline BitsliceArgs columns_of(const ParityArgs &a) {
    return BitsliceArgs{a.rows, a.R, a.W, a.ldx, a.Xt};
}

// E = C Theta B^T, tiled over observables x samples, gate words split
// `splits` ways (partials E[split][l_pad][s_pad]).
struct FwdArgs {
    const uint64_t *cbits, *bbits;
    const uint16_t *thh, *thl, *thm;  // thm: third limb (IQP_SPLIT3_BF16 only)
    const float *t32;
    int64_t m_pad, l_pad, s_pad, splits;
    float *E;
    const int32_t *nrows = nullptr;  // rows that are there (RowPerm)
    ChainGate gate = {};             // FP32 only
};
inline int64_t fwd_units(const FwdArgs &a, int fm, int fn) {
    return (a.l_pad / (32 * fm)) * ceil_div(a.s_pad / (32 * fn), 4) * a.splits;
}

// With one chunk per observable (s <= kEpiChunk) the kernel that has the sums
// writes the results itself.
struct FinArgs {
    const double *part;
    int64_t l, s;
    double *mean, *stderr_, *rowsum;
};

struct EpiArgs {
    const float *E;
    int64_t splits, l, s, l_pad, s_pad;
    float *phase_out;
    double *part;
    FinArgs fin = {};
    const int32_t *pos = nullptr;  // RowPerm
    ChainGate gate = {};
};

// Non-zero entries of C (tiled32 bits of l_pad rows, mw gate words) added to *nnz.
struct CountArgs {
    const uint64_t *cbits;
    int64_t l_pad, mw;
    unsigned long long *nnz;
};
constexpr int64_t kCountWords = 2048;  // words per block
inline int64_t blocks_of(const CountArgs &a) { return ceil_div(a.l_pad * a.mw, kCountWords); }

// The FP32 forward over the non-zero entries of C: cbits tiled32, t32 split by
// gate parity, btrm B^T row-major (Rw words per gate), the gate words split
// `splits` ways as the matrix-core kernel splits them.
struct ChainFwdArgs {
    const uint64_t *cbits;
    int64_t mw;
    const float *t32;
    int64_t m_pad;
    const uint64_t *btrm;
    int64_t Rw, l, s, splits;
    float *phase_out;
    double *part;
    FinArgs fin;
    ChainGate gate;
};
// The FP32 backward over the non-zero entries: crm C row-major (mw words per
// row), rank[k][w] = entries of row k before word w; *nnz counts all, or stays
// past any limit when a row holds more than cap entries.
struct RankArgs {
    const uint64_t *crm;
    int64_t l, mw, cap;
    uint32_t *rank;
    unsigned long long *nnz;
};
// (a wave per row; the counter takes one atomic add per block)
__host__ __device__ inline int64_t blocks_of(const RankArgs &a) {
    return a.l < 4096 ? ceil_div(a.l, 4) : 1024;
}
// T[(ks l + k) cap + position of gate j in row k] = the sum over the samples of
// split ks of S_ki (-1)^{b_ij}.
struct ChainBwdArgs {
    const uint64_t *crm;
    int64_t mw, m_pad;
    const uint64_t *btbits;  // word-major
    int64_t l, s, s_pad, ksplits, cap;
    const float *phase;
    const double *coef;
    float *T;
    ChainGate gate;
};
inline int64_t blocks_of(const ChainBwdArgs &a) { return a.l * a.ksplits; }
struct ChainGradArgs {
    const uint64_t *ctbits;  // word-major
    const uint32_t *rank;
    const float *T;
    int64_t l, lw, m, m_pad, mw, ksplits, cap;
    double *grad;
    ChainGate gate;
};
constexpr int64_t kChainMaxSplits = 8;
inline int64_t blocks_of(const ChainGradArgs &a) { return a.mw; }
constexpr int64_t kChainChunk = 2 * kEpiChunk;  // samples per block
inline int64_t blocks_of(const ChainFwdArgs &a) { return a.l * ceil_div(a.s, kChainChunk); }
// A wave per (observable, chunk) unit where that makes several rounds of eight
// waves per SIMD, a block per unit before (10^4 units: 45 us by wave, 38 by
// block; 10^5: 195 and 224).
__host__ __device__ inline bool epilogue_by_wave(const EpiArgs &a) {
    return a.l * ceil_div(a.s, kEpiChunk) >= 64 * kWaveSlots;
}
// (more units than 2^24 - 1 blocks were never accepted, and a unit's number
// fits 32 bits)
inline int64_t blocks_of(const EpiArgs &a) {
    const int64_t units = a.l * ceil_div(a.s, kEpiChunk);
    return epilogue_by_wave(a) && units < ((int64_t)1 << 24) ? ceil_div(units, 4) : units;
}

inline int64_t blocks_of(const FinArgs &a) {
    return a.s <= kEpiChunk ? 0 : ceil_div(a.l, 256);
}

// coef[2k], coef[2k+1] = alpha_k, beta_k of the backward weights. For the
// fixed-point weights (IQP_SPLIT3_BF16) also the row scale
// sq[k] = (|alpha_k| + |beta_k|) / kI8Max and a zeroed non-finite flag nf[k];
// both pointers are NULL for the other forms. gcnt (NULL in the sparse form):
// n_gcnt counters of the gate lists, zeroed.
struct CoefArgs {
    const double *grad_mean;
    int64_t l, s;
    double *coef;
    double *sq;
    int32_t *nf;
    int32_t *gcnt;
    int64_t n_gcnt;
};
inline int64_t blocks_of(const CoefArgs &a) { return ceil_div(a.l, 256); }

// IQP_SPLIT3_BF16: shi / slo hold the high / low signed 8-bit limbs of
// N_ki = rint(S_ki / sq[k]) (|N| <= kI8Max), and nf[k] is set to 1 where a
// weight of row k is not finite. IQP_SPLIT_BF16_FP8: shi holds the FP16 limb
// and slo (one byte per weight) the FP8 E4M3 limb of S_ki 2^e_k, and sq[k] is
// set to 2^-e_k.
struct WeightsArgs {
    const float *phase;
    const double *coef;
    int64_t l, s, l_pad, s_pad;
    int prec;
    uint16_t *shi, *slo;
    float *s32;
    int32_t *nf;
    double *sq;
    ChainGate gate = {};  // FP32 only, as in the steps below
};
inline int64_t blocks_of(const WeightsArgs &a) { return (a.s_pad / 64) * (a.l_pad / 64); }

// Gate lists of the backward. A block of 32 cf observables contributes to the
// gradient of gate j only if some observable of the block anticommutes with
// j, so the contraction runs over the listed gates of each block. A gate is
// listed by the halves of the block (cf / 2 fragments of 32 rows each) that
// hold such an observable: both (class 0), the lower only (class 1), the
// upper only (class 2). gcnt[ob * 4 + class] counts; with one class array
// (`split` 0) every listed gate is in class 0. Entries of class 0 at
// glist[(ob * 2) * m_pad + i], of class 1 at glist[(ob * 2 + 1) * m_pad + i],
// of class 2 at the end of that array, glist[(ob * 2 + 2) * m_pad - 1 - i].
// The order of a list varies from run to run; no result depends on it, since
// every gate is a column of its own in the product.
struct GateListArgs {
    const uint64_t *ctbits;
    int64_t m, m_pad, lw;
    int cw;     // 64-row words per block: cf / 2
    int split;  // classes by half (1) or one class (0)
    int32_t *gcnt, *glist;
    ChainGate gate = {};
};
constexpr int64_t kListSeg = 1024;  // gates per block of the list kernel
inline int64_t blocks_of(const GateListArgs &a) {
    return (a.lw / a.cw) * ceil_div(a.m_pad, kListSeg);
}

// T = S B (observables x listed gates, K = samples, split `ksplits` ways over
// the sample words) and the gradient partials gpart[ksplits][n_ob][m_pad],
// n_ob = l_pad / (32 cf), written for the listed gates of each block only;
// btbits / ctbits are the transposed word-major parities of the samples /
// observables against the generators (word w of gate j at [w * m_pad + j]). Every
// split must hold >= 1 sample word.
struct BwdArgs {
    const uint16_t *shi, *slo;
    const float *s32;
    const uint64_t *btbits, *ctbits;
    int64_t m_pad, l_pad, s_pad, ksplits;
    float *gpart;
    const double *sq;   // row scales (IQP_SPLIT3_BF16, IQP_SPLIT_BF16_FP8) and
                        // non-finite flags (IQP_SPLIT3_BF16)
    const int32_t *nf;
    int64_t obgroup;    // observable blocks per unit group (unit order only)
    const int32_t *gcnt, *glist;
    ChainGate gate = {};
};
// How the backward of a form runs its tile configuration bfm x bfn: gates of a
// wave in column blocks of 32 (fn), and whether the lists are split by the
// halves of a block of 32 bfm observables.
struct BwdShape {
    int fn;
    bool split;
};
BwdShape bwd_shape(int prec, int bfm, int bfn);
// Workgroup tiles over one block's gate lists: room for every gate, and for
// the partly filled last tile of each further class (gates that fit one tile
// never take more).
__host__ __device__ inline int64_t bwd_list_tiles(int64_t m_pad, int fn, bool split) {
    return ceil_div(m_pad, 128 * fn) + (split && m_pad > 128 * fn ? 2 : 0);
}
inline int64_t bwd_units(const BwdArgs &a, int prec, int bfm, int bfn) {
    const BwdShape sh = bwd_shape(prec, bfm, bfn);
    return bwd_list_tiles(a.m_pad, sh.fn, sh.split) * (a.l_pad / (32 * bfm)) * a.ksplits;
}

// n_parts = ksplits n_ob partials per gate, block ob of 64 cw rows present
// only where one of its C^T words is non-zero.
struct GradArgs {
    const float *gpart;
    int64_t n_ob, ksplits, m, m_pad;
    double *grad;
    const uint64_t *ctbits;
    int cw;
    ChainGate gate = {};
};
inline int64_t blocks_of(const GradArgs &a) { return ceil_div(a.m, 64); }

// Stochastic bitflip circuits (exact product form).
struct BitflipPrepArgs {
    const double *theta;
    int64_t m;
    double *enc;  // [m] copysign(-log|cos 2 theta|, cos 2 theta)
};
inline int64_t blocks_of(const BitflipPrepArgs &a) { return ceil_div(a.m, 256); }

struct BitflipFwdArgs {
    const uint64_t *cbits;  // tiled32 C bits, mw gate words per observable row
    const double *enc;
    int64_t l, mw;
    double *mean, *stderr_;  // stderr_ may be NULL (written 0: the value is exact)
    double *stat;            // [l][2]
};
inline int64_t blocks_of(const BitflipFwdArgs &a) { return ceil_div(a.l, 4); }

struct BitflipGradArgs {
    const uint64_t *ctbits;  // transposed tiled32 C^T bits, lw observable words per gate row
    const double *enc, *theta, *stat, *grad_mean;
    int64_t m, lw;
    double *grad;
};
inline int64_t blocks_of(const BitflipGradArgs &a) { return ceil_div(a.m, 256); }

// The same from the parities in registers (rows of fewer than kColumnWords
// words): par names the observables' rows and the blocking; sums per gate
// chunk psum / pcode [ngc][l_pad], dot products per observable chunk part
// [nrc][m_pad].
// Their blocks walk over the set bits of each row word in turn, so where the
// rows are few a block takes fewer words of them: no word past the rows, and as
// few as it takes for a block per CU. Forward and gradient call, 10 qubits, 50
// gates, 1000 observables (one block at 16 words): 36 and 77 -> 15 and 20 us; 1000
// qubits, 10^5 gates, 300 observables 134 and 159 -> 36 and 58 us, with the
// finishing step's share below.
inline ParityArgs bitflip_blocking(ParityArgs a) {
    a = parity_from_rows(a);
    while (a.rw > 1 && (a.rw >= 2 * a.Rw || blocks_of(a) < 256)) {
        a.rw /= 2;
        a.gpb = parity_gpb(a.Gw, a.Rw, a.rw);
    }
    return a;
}
struct BitflipSumArgs {
    ParityArgs par;
    const double *enc;
    int64_t l_pad;
    double *psum;
    int32_t *pcode;
};
inline size_t lds_of(const BitflipSumArgs &a) {
    const size_t sums = (size_t)64 * a.par.rw * 20, bits = lds_of(a.par);
    return sums > bits ? sums : bits;
}
struct BitflipFinishArgs {
    const double *psum;
    const int32_t *pcode;
    int64_t ngc, l, l_pad;
    double *mean;
    const double *grad_mean;  // NULL: forward only
    double *stat, *val;       // [l][2] each
};
struct BitflipDotArgs {
    ParityArgs par;
    const double *enc, *stat, *val;
    int64_t l, m_pad;
    double *part;
};
inline size_t lds_of(const BitflipDotArgs &a) { return lds_of(a.par) + (size_t)a.par.rw * 65 * 8; }
struct BitflipChainArgs {
    const double *part, *theta;
    int64_t nrc, m, m_pad;
    double *grad;
};

// Where the sparse kernels read the sample parities b_ij of generator j
// (bit i % 64 of word i / 64):
//   shared samples:       btrm, B^T row-major, Rwb sample words per generator
//   independent samples:  xt, the bit columns of each observable's own
//                         samples (xt + k * xstride, column q at q * Rwb),
//                         combined over the support list sup (or the bit row
//                         of gens for a generator heavier than kSupCap)
struct SampleParity {
    const uint64_t *btrm;
    const uint64_t *xt;  // NULL for shared samples
    int64_t Rwb, xstride;
    const int32_t *sup;
    const uint64_t *gens;
    int W;
    const uint64_t *ops;  // the observables (W words each)
};

// Sparse-C contraction (FP32 on the vector units): the phases summed over
// each observable's anticommuting generators only.
//   crm   C row-major: Gw gate words per observable row
//   t32   2 theta' per generator (plain FP32)
struct SparseFwdArgs {
    const uint64_t *crm;
    int64_t Gw;
    const float *t32;
    SampleParity bsrc;
    int64_t l, s;
    float *phase_out;  // [l][s] or NULL
    double *part;      // [l][ceil(s / kEpiChunk)][2] as the dense epilogue writes it
    FinArgs fin;
};

// acc[m_pad + 1] int64 (the last slot flags a non-finite contribution) and
// *scale: the fixed-point scale of the gradient sums, from the bound
// sum_k s (|alpha_k| + |beta_k|) on every partial sum.
struct SparseBoundArgs {
    const double *coef;
    int64_t l, s, m_pad;
    long long *acc;
    double *scale;
};
inline int64_t blocks_of(const SparseBoundArgs &a) { return ceil_div(a.m_pad + 1, 256); }

struct SparseBwdArgs {
    const uint64_t *crm;
    int64_t Gw;
    SampleParity bsrc;
    int64_t l, s, m_pad;  // j < m_pad; acc[m_pad] is the non-finite flag
    const float *phase;
    const double *coef, *scale;
    long long *acc;
};

// Bit columns of l sample sets of s rows each ([l][s][W], row i of set k at
// samples + (k s + i) W): xt[k * 64 W * ldx + q * ldx + rw], bit r = qubit q
// of row 64 rw + r of set k (rows >= s read as 0), q < 64 W, rw < ldx (a
// multiple of 16; one block per set and 16 row words).
struct IndepSliceArgs {
    const uint64_t *samples;
    int64_t l, s;
    int W;
    int64_t ldx;
    uint64_t *xt;
};

struct SparseFinishArgs {
    const long long *acc;
    const double *scale;
    int64_t m, m_pad;
    double *grad;
};
inline int64_t blocks_of(const SparseFinishArgs &a) { return ceil_div(a.m, 256); }

// ---- launchers (iqp_kernels.hip, iqp_sparse_kernels.hip); each returns
// hipGetLastError() ----
hipError_t launch_prep(const LaunchCtx &lc, const ThetaArgs &a, const SupportArgs &b);
hipError_t launch_prep(const LaunchCtx &lc, const CoefArgs &a, const SupportArgs &b);
hipError_t launch_prep(const LaunchCtx &lc, const BitflipPrepArgs &a, const SupportArgs &b);
hipError_t launch_support(const LaunchCtx &lc, const SupportArgs &a);
hipError_t launch_row_perm(const LaunchCtx &lc, const RowPermArgs &a);
// Parities in one layout, or of two row sets: (la, lb) one of (1, 1), (4, 4),
// (0, 3).
hipError_t launch_parity(const LaunchCtx &lc, int layout, const ParityArgs &a);
hipError_t launch_parity2(const LaunchCtx &lc, int la, const ParityArgs &a, int lb,
                          const ParityArgs &b);
hipError_t launch_phase_fwd(const LaunchCtx &lc, int prec, int fm, int fn, const FwdArgs &a);
hipError_t launch_epilogue(const LaunchCtx &lc, const EpiArgs &a);
hipError_t launch_finalize(const LaunchCtx &lc, const FinArgs &a);
hipError_t launch_weights(const LaunchCtx &lc, const WeightsArgs &a);
hipError_t launch_gate_list(const LaunchCtx &lc, const GateListArgs &a);
hipError_t launch_phase_bwd(const LaunchCtx &lc, int prec, int fm, int fn, const BwdArgs &a);
hipError_t launch_grad_reduce(const LaunchCtx &lc, const GradArgs &a);
hipError_t launch_count(const LaunchCtx &lc, const CountArgs &a);
hipError_t launch_chain_fwd(const LaunchCtx &lc, const ChainFwdArgs &a);
hipError_t launch_rank(const LaunchCtx &lc, const RankArgs &a);
hipError_t launch_chain_bwd(const LaunchCtx &lc, const ChainBwdArgs &a);
hipError_t launch_chain_grad(const LaunchCtx &lc, const ChainGradArgs &a);
hipError_t launch_sparse_fwd(const LaunchCtx &lc, const SparseFwdArgs &a);
hipError_t launch_sparse_bound(const LaunchCtx &lc, const SparseBoundArgs &a);
hipError_t launch_sparse_bwd(const LaunchCtx &lc, const SparseBwdArgs &a);
hipError_t launch_sparse_finish(const LaunchCtx &lc, const SparseFinishArgs &a);
hipError_t launch_indep_slice(const LaunchCtx &lc, const IndepSliceArgs &a);
hipError_t launch_bitflip_fwd(const LaunchCtx &lc, const BitflipFwdArgs &a);
hipError_t launch_bitflip_grad(const LaunchCtx &lc, const BitflipGradArgs &a);
hipError_t launch_bitflip_sum(const LaunchCtx &lc, const BitflipSumArgs &a);
hipError_t launch_bitflip_finish(const LaunchCtx &lc, const BitflipFinishArgs &a);
hipError_t launch_bitflip_dot(const LaunchCtx &lc, const BitflipDotArgs &a);
hipError_t launch_bitflip_chain(const LaunchCtx &lc, const BitflipChainArgs &a);

// Batched launches: `args` is a device array of np argument structs of the
// step's type and `off` a device array of np + 1 prefix sums of their block
// counts (off[0] = 0, off[np] = total > 0).
enum StepKind {
    SK_THETA = 0, SK_BITSLICE, SK_PARITY1, SK_PARITY4, SK_EPI, SK_FIN, SK_COEF,
    SK_WEIGHTS, SK_GRAD, SK_SUPPORT, SK_GATELIST, SK_COLPARITY1, SK_COLPARITY4, SK_COUNT
};
hipError_t launch_batched(const LaunchCtx &lc, int kind, const void *args, const int64_t *off,
                          int np, int64_t total, size_t lds);

// Persistent contractions over a work queue: `grid` workgroups take work
// units 0 .. off[np]-1 in order from `counter` (which must read 0 at launch);
// unit u belongs to problem p with off[p] <= u < off[p+1] and is that
// problem's local unit u - off[p].
hipError_t launch_phase_fwd_persistent(const LaunchCtx &lc, int prec, int fm, int fn,
                                       const FwdArgs *args, const int64_t *off, int np,
                                       unsigned long long *counter, int grid);
hipError_t launch_phase_bwd_persistent(const LaunchCtx &lc, int prec, int fm, int fn,
                                       const BwdArgs *args, const int64_t *off, int np,
                                       unsigned long long *counter, int grid);
// Workgroups of the persistent contraction that fit on the device at once.
int persistent_grid(bool fwd, int prec, int fm, int fn);
// Zero n work-queue counters (a kernel, so it can be captured in a graph).
hipError_t launch_reset_counters(const LaunchCtx &lc, unsigned long long *c, int n);

// pstat[2k] = sum_n (-1)^{a_k . x_n}, pstat[2k+1] = that sum / N, for the
// observables ops [l][W] against the training strings data [N][W].
hipError_t launch_data_stats(const LaunchCtx &lc, const uint64_t *ops, int64_t l,
                             const uint64_t *data, int64_t N, int W, double *pstat);

hipError_t launch_mmd_loss(const LaunchCtx &lc, const double *pstat, const double *rowsum,
                           const double *op_weight, int64_t l, int64_t s, int64_t N, int unbiased,
                           double *loss);

hipError_t launch_coef_mmd(const LaunchCtx &lc, const double *pstat, const double *rowsum,
                           const double *op_weight, int64_t l, int64_t s, int unbiased,
                           double *coef, double *sq, int32_t *nf, int32_t *gcnt, int64_t n_gcnt);

}  // namespace iqp
