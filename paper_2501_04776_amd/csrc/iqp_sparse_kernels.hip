// gfx950 kernels of the sparse-C contraction and of independent estimates.
//
// Sparse-C: E_ki = sum_{j in J_k} t_j (-1)^{b_ij}, t_j = 2 theta'_j, over the
// generators J_k that anticommute with observable k (the set bits of row k of
// C), on the vector units in FP32: the dense contraction's result with
// |J_k| / m of its work.
//
// Independent estimates (the l x s x n sample tensor of Sec. 2.3): observable
// k averages over its own s samples, so its sample parities come from the bit
// columns of its own sample set instead of one B^T shared by all observables.
// Nothing else changes, so both forms run the same bodies over a different
// source of sample-parity words. Both directions read tables: 16-entry sums
// over 4 generators (forward) or 4 samples (backward) in LDS, indexed by
// nibbles of parity bits.
#include <cstdlib>

#include "iqp_device.h"

namespace iqp {

// ---------------------------------------------------------------------------
// Sample-parity words: word w of generator j holds b_ij of samples 64 w ..
// 64 w + 63 (bit i % 64). A block covers one chunk of kSpWords words; the
// sample-parity rows hold whole chunks (a multiple of kSpWords words, the
// words of samples >= s being 0), so every load of a chunk's words is
// unconditional.
constexpr int kSpWords = kEpiChunk / 64;
// the float nearest pi and a float near 1 / pi: the forward's FP32 sums are
// folded by whole multiples q of the former (any q is exact bookkeeping)
constexpr float kPiF = 3.14159274f;
constexpr float kInvPiF = 0.318309873f;

// ---------------------------------------------------------------------------
// Gradient: for every (k, j in J_k) the partial T_kj = sum_i S_ki (-1)^{b_ij}
// of a sample chunk is added into an int64 fixed-point accumulator of gate
// j. Integer addition is associative, so the result does not depend on the
// order in which the lanes add, and no per-pair storage is needed. The scale keeps every sum below 2^62: |T_kj| <= s
// (|alpha_k| + |beta_k|) summed over k.
__device__ __forceinline__ void sparse_bound_body(const SparseBoundArgs &a, int64_t blk) {
    const int64_t j = blk * 256 + threadIdx.x;
    if (j <= a.m_pad) gptr(a.acc)[j] = 0;
    if (blk != 0) return;
    __shared__ double sh[256];
    double g = 0.0;
    for (int64_t k = threadIdx.x; k < a.l; k += 256)
        g += (double)a.s * (fabs(gptr(a.coef)[2 * k]) + fabs(gptr(a.coef)[2 * k + 1]));
    g = block_sum_256(g, sh);
    if (threadIdx.x == 0) {
        const double G = (g > 0.0 && isfinite(g)) ? g : 1.0;
        gptr(a.scale)[0] = ldexp(1.0, 61 - ilogb(G));
    }
}

hipError_t launch_sparse_bound(const LaunchCtx &lc, const SparseBoundArgs &a) {
    return plain_launch<SparseBoundArgs, sparse_bound_body>(lc, KF_WEIGHTS, a, blocks_of(a));
}

// Gradient by table lookup. A block takes observable k and kC (1 or 2) chunks
// of kEpiChunk samples, each with tables of its own. Thread t computes S_ki for
// the four samples 4t .. 4t + 3 of the chunk and writes their 16 signed sums
//   L_t[v] = sum_{b < 4} (-1)^{v_b} S_{k, c + 4t + b},  v = 0 .. 15,
// so that, with v_t(j) the nibble of generator j's parity bits over those
// four samples (bits 4t .. 4t + 3 of the chunk's parity words), the chunk's
// partial T_kj = sum_i S_ki (-1)^{b_ij} is the sum over t of L_t[v_t(j)]:
// 256 table reads per generator and chunk in place of 1024 masked adds. The
// generators J_k (the set bits of row k of C) are compacted into a list in
// LDS; each lane takes one generator of the list, forms its 16 parity words
// of the chunk (one 128-byte line of B^T for shared samples; for
// independent sets the XOR of the line of each support column of k's own
// samples), sums its 256 table entries and adds the total into the
// generator's fixed-point accumulator. The lanes of a wave read one table
// at a time, a 64-byte row of 16 entries in distinct banks, so the reads
// never conflict.
constexpr int kLutTables = (int)(kEpiChunk / 4);  // one per thread of the block
constexpr int kLutList = 1024;                    // generators per list fill
// Over shared samples, gradient blocks take two chunks once that leaves
// kPairBlocks of them: half the atomics into the gates' sums, which bound the
// kernel once the parity rows outgrow an L2, and half the compactions. Whole
// gradients with two and with one chunk a block: n = 300, 40000 gates, 10^4 samples
// 0.301 and 0.420 ms at 1600 observables; n = 1000, 10^5 gates 1.16 and 1.99 ms.
// With few blocks the longer ones are the time, and where the chunks are odd in
// number half of the blocks are half as long, so the line is twice as high there.
// Over 230 shapes of 50 to 7000 observables and 2 to 10 chunks, two chunks took
// 0.57 to 1.10 of the time of one past the line (0.82 in the mean; over 1.03 in
// eight shapes, whose rows of C have some ten entries), 0.81 to 1.23 from 320
// blocks to the line and 0.94 to 1.50 below. Three chunks a block (tables of 48
// KB) took 0.90 to 1.06 of the time of two, four 1.00 to 1.27.
//
// Independent sets read every observable's own bit columns, wait for them more
// than for anything else, and lose waves to the larger tables: two chunks took
// more time than one, up to 1.4 and more, in 164 of 214 shapes, so they take one.
constexpr int64_t kPairBlocks = 640;

static_assert(kLutTables == 256, "one table per thread of a 256-thread block");

// Exclusive prefix over the block of per-thread counts c (the block's total
// in *tot); wsum holds the 4 wave totals and is reused only after the next
// barrier of the caller's loop.
__device__ __forceinline__ int block_excl_scan(int c, int *wsum, int *tot) {
    const int lane = threadIdx.x & 63, w = wave_id();
    int x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = wsum[i];
        before += i < w ? v : 0;
        all += v;
    }
    *tot = all;
    return before + x - c;
}


// The set bits of words w0 .. w1 - 1 of a row of C (word w: word(w)), in gate
// order, into the LDS list lst, 256 row words at a time (a block prefix sum of
// their popcounts places each word's bits); fill(n) runs on every full list (n = kLutList) and on
// the last, partial one (n may be 0), between barriers, so fill may read
// lst and the block's other shared data freely.
template <typename R, typename F>
__device__ __forceinline__ void compact_words(R word, int64_t w0, int64_t w1, int32_t *lst,
                                              int (*wsum)[4], F fill) {
    const int tid = threadIdx.x;
    int n = 0, it = 0;
    for (int64_t base = w0; base < w1; base += 256) {
        uint64_t v = base + tid < w1 ? word(base + tid) : 0ull;
        for (;;) {
            int tot;
            const int off = block_excl_scan(__popcll(v), wsum[it & 1], &tot);
            ++it;
            const int room = kLutList - n;
            for (int pos = off; v != 0ull && pos < room; ++pos) {
                lst[n + pos] = (int32_t)((base + tid) * 64 + __builtin_ctzll(v));
                v &= v - 1;
            }
            const int take = tot < room ? tot : room;
            n += take;
            if (n == kLutList) {  // uniform over the block
                __syncthreads();
                fill(n);
                __syncthreads();
                n = 0;
            }
            if (tot <= room) break;
        }
    }
    __syncthreads();
    fill(n);
}

template <typename F>
__device__ __forceinline__ void compact_row(glb<const uint64_t> crow, int64_t Gw, int32_t *lst,
                                            int (*wsum)[4], F fill) {
    compact_words([&](int64_t w) { return crow[w]; }, 0, Gw, lst, wsum, fill);
}

// The 16 parity words of generator j over chunk ch (lane-varying j).
template <bool kIndep>
__device__ __forceinline__ void lut_row(const SparseBwdArgs &a, int64_t k, int64_t ch, int64_t j,
                                        u32x4 (&wv)[8]);
template <>
__device__ __forceinline__ void lut_row<false>(const SparseBwdArgs &a, int64_t, int64_t ch,
                                               int64_t j, u32x4 (&wv)[8]) {
    const glb<const u32x4> src =
        (glb<const u32x4>)(gptr(a.bsrc.btrm) + j * a.bsrc.Rwb + ch * kSpWords);
#pragma unroll
    for (int q = 0; q < 8; ++q) wv[q] = src[q];
}
template <>
__device__ __forceinline__ void lut_row<true>(const SparseBwdArgs &a, int64_t k, int64_t ch,
                                              int64_t j, u32x4 (&wv)[8]) {
    const glb<const uint64_t> cols = gptr(a.bsrc.xt) + k * a.bsrc.xstride + ch * kSpWords;
    auto add_col = [&](int64_t q) {
        const glb<const u32x4> src = (glb<const u32x4>)(cols + q * a.bsrc.Rwb);
#pragma unroll
        for (int i = 0; i < 8; ++i) wv[i] ^= src[i];
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) wv[i] = u32x4{0, 0, 0, 0};
    const glb<const int32_t> sj = gptr(a.bsrc.sup) + j * kSupCap;
    if (sj[0] == -2) {  // heavier than kSupCap: its bit row
        for (int w = 0; w < a.bsrc.W; ++w) {
            uint64_t g = gptr(a.bsrc.gens)[j * a.bsrc.W + w];
            while (g) {
                add_col(w * 64 + __builtin_ctzll(g));
                g &= g - 1;
            }
        }
        return;
    }
    for (int e = 0; e < kSupCap; ++e) {
        const int32_t q = sj[e];
        if (q < 0) break;
        add_col(q);
    }
}

// An observable of weight 0 commutes with every generator (most operators of a
// wide kernel bandwidth): its blocks need no row of C. (Uniform over the block.) A
// lane per word, one load's latency: a scalar loop, which waited for word after word,
// cost more than a short row of C does. 5000 qubits, 1000 gates, 10^4 observables and
// samples: forward 0.77 -> 0.47 ms, gradient 0.76 -> 0.54 ms.
__device__ __forceinline__ bool weight_zero(const SampleParity &b, int64_t k) {
    uint64_t any = 0ull;
    for (int w = threadIdx.x & 63; w < b.W; w += 64) any |= gptr(b.ops)[k * b.W + w];
    return __ballot(any != 0ull) == 0ull;
}

template <bool kIndep, int kC>
__device__ __forceinline__ void sparse_bwd_lut_body(const SparseBwdArgs &a, int64_t blk) {
    // chunk-major: the blocks that run together read the same 128-byte columns
    // of the parity rows (fewer HBM fetches than observable-major order)
    const int64_t cg = blk / a.l, k = blk - cg * a.l, ch0 = cg * kC;
    const int64_t left = ceil_div(a.s, kEpiChunk) - ch0;
    const int nc = left < kC ? (int)left : kC;
    const int tid = threadIdx.x, lane = tid & 63;
    __shared__ __attribute__((aligned(16))) float tab[kC * kLutTables * 16];
    __shared__ int32_t lst[kLutList];
    __shared__ int wsum[2][4];

    // all phases in flight at once, before anything waits: with two chunks a block
    // four waves run per SIMD, too few for one load after the other (1000 qubits and
    // gates, 10^4 observables and samples: gradient 549 -> 495 us, one chunk 502)
    float ph[kC][4];
#pragma unroll
    for (int c = 0; c < kC; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int64_t i = (ch0 + c) * kEpiChunk + 4 * tid + b;
            ph[c][b] = gptr(a.phase)[k * a.s + (i < a.s ? i : a.s - 1)];
        }
    if (weight_zero(a.bsrc, k)) return;

    // the tables of these chunks
    const double al = gptr(a.coef)[2 * k], be = gptr(a.coef)[2 * k + 1];
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {
        float S[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int64_t i = (ch0 + c) * kEpiChunk + 4 * tid + b;
            float v = 0.0f;
            if (i < a.s) {
                float sn, cs;
                sincosf(kC > 1 && c > 0 ? ph[kC - 1][b] : ph[0][b], &sn, &cs);
                v = (float)((al + be * (double)cs) * (double)sn);
            }
            S[b] = v;
        }
        // x[u] over samples 0, 1 and y[u] over samples 2, 3, bit set = minus
        const float x[4] = {S[0] + S[1], S[1] - S[0], S[0] - S[1], -S[0] - S[1]};
        const float y[4] = {S[2] + S[3], S[3] - S[2], S[2] - S[3], -S[2] - S[3]};
        float4 *row = reinterpret_cast<float4 *>(tab + (c * kLutTables + tid) * 16);
#pragma unroll
        for (int h = 0; h < 4; ++h)
            row[h] = make_float4(x[0] + y[h], x[1] + y[h], x[2] + y[h], x[3] + y[h]);
    }

    const glb<const uint64_t> crow = gptr(a.crm) + k * a.Gw;
    const double scale = gptr(a.scale)[0];
    // each wave takes list entries wave_id() * 64 + lane, + 256, ...
    auto process = [&](int n) {
        for (int g = wave_id() * 64 + lane; g - lane < n; g += 256) {
            if (g >= n) continue;
            const int64_t j = lst[g];
            long long add = 0;
#pragma unroll 1
            for (int c = 0; c < nc; ++c) {
                u32x4 wv[8];
                lut_row<kIndep>(a, k, ch0 + c, j, wv);
                float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
                const char *tb = reinterpret_cast<const char *>(tab + c * kLutTables * 16);
#pragma unroll
                for (int r = 0; r < kSpWords; ++r) {
                    // word r holds nibbles t = 16 r + e (bits 4e .. 4e + 3): byte
                    // e' of x[2h] is 4 times nibble 8h + 2e', of x[2h + 1] 4 times
                    // nibble 8h + 2e' + 1 (kept opaque so that each byte costs one
                    // extract instead of a shift and a mask)
                    uint32_t x[4];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t d = wv[r / 2][2 * (r % 2) + h];
                        x[2 * h] = (d << 2) & 0x3C3C3C3Cu;
                        x[2 * h + 1] = (d >> 2) & 0x3C3C3C3Cu;
                        asm volatile("" : "+v"(x[2 * h]), "+v"(x[2 * h + 1]));
                    }
                    float v[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const uint32_t o = (x[e / 4 % 2 + 2 * (e / 8)] >> (8 * (e % 4))) & 0xFFu;
                        const int t = 16 * r + 8 * (e / 8) + 2 * (e % 4) + e / 4 % 2;
                        v[e] = *reinterpret_cast<const float *>(tb + t * 64 + o);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] += v[e] + v[e + 8];
                }
                const float tot = ((acc[0] + acc[1]) + (acc[2] + acc[3])) +
                                  ((acc[4] + acc[5]) + (acc[6] + acc[7]));
                if (isfinite(tot))
                    add += llrint((double)tot * scale);
                else
                    atomicOr((unsigned long long *)&gptr(a.acc)[a.m_pad], 1ull);
            }
            atomicAdd((unsigned long long *)&gptr(a.acc)[j], (unsigned long long)add);
        }
    };

    __syncthreads();  // tables written
    compact_row(crow, a.Gw, lst, wsum, process);
}

// Forward by table lookup. A block takes observable k and one chunk of
// kEpiChunk samples; its waves take 4 of the chunk's 16 sample words each,
// 4 samples a lane (lut_sample). The generators J_k are compacted into
// the LDS list as in the backward, and every 4 consecutive entries get a
// 16-entry table of their angle sums,
//   G_e[v] = sum_{b < 4, v_b = 1} t_{lst[4e + b]},  t_j = 2 theta'_j (FP32),
// so that a sample's sum over the 64 entries 64g .. 64g + 63 is the sum of
// 16 table reads indexed by its parity bits for those generators, 4 at a
// time. Those bits come from an exchange over the wave: lane L loads the
// parity words of entry 64g + L for the wave's samples, and lut_transpose
// gives each lane all 64 entries' bits of its own 4. The nibble offsets are
// formed as in the backward ((x << 2) and
// (x >> 2) masked to 0x3C per byte) and a byte permute places each one
// under the group's table base (g * 1024 bytes; the table within the group
// is the LDS instruction's immediate offset). All lanes read one 16-entry
// table at a time, so the reads never conflict. Per sample,
//   E_ki = T_k - 2 sum_{j in J_k, b_ij = 1} t_j,  T_k = sum_{j in J_k} t_j (FP64),
// with the FP32 sum folded modulo the float nearest pi every 32 generators
// (the whole multiples kept in an exact count), then reduced modulo 2 pi in
// FP64 as the dense epilogue does. Bound by the vector units, which issue on every
// cycle (five waves per SIMD over the run): per sample and 64 entries 20
// instructions for the exchange, 24 for the offsets, 24 for the sums and the fold
// (85 with a full 64x64 transpose per word, when n = 300, 1000 observables, 10^4
// samples took 0.309 ms and now 0.294; n = 1000, 10^5 gates, 2000 observables
// 1.02 and 0.92 ms).
template <bool kIndep>
__device__ __forceinline__ void lut_fwd_words(const SparseFwdArgs &a, int64_t k, int64_t sw,
                                              int64_t j, u32x4 (&wv)[2]);
template <>
__device__ __forceinline__ void lut_fwd_words<false>(const SparseFwdArgs &a, int64_t, int64_t sw,
                                                     int64_t j, u32x4 (&wv)[2]) {
    const glb<const u32x4> src = (glb<const u32x4>)(gptr(a.bsrc.btrm) + j * a.bsrc.Rwb + sw);
    wv[0] = src[0];
    wv[1] = src[1];
}
template <>
__device__ __forceinline__ void lut_fwd_words<true>(const SparseFwdArgs &a, int64_t k, int64_t sw,
                                                    int64_t j, u32x4 (&wv)[2]) {
    const glb<const uint64_t> cols = gptr(a.bsrc.xt) + k * a.bsrc.xstride + sw;
    auto add_col = [&](int64_t q) {
        const glb<const u32x4> src = (glb<const u32x4>)(cols + q * a.bsrc.Rwb);
        wv[0] ^= src[0];
        wv[1] ^= src[1];
    };
    const glb<const int32_t> sj = gptr(a.bsrc.sup) + j * kSupCap;
    if (sj[0] == -2) {  // heavier than kSupCap: its bit row
        for (int w = 0; w < a.bsrc.W; ++w) {
            uint64_t g = gptr(a.bsrc.gens)[j * a.bsrc.W + w];
            while (g) {
                add_col(w * 64 + __builtin_ctzll(g));
                g &= g - 1;
            }
        }
        return;
    }
    for (int e = 0; e < kSupCap; ++e) {
        const int32_t q = sj[e];
        if (q < 0) break;
        add_col(q);
    }
}

// The exchange before the forward's lookups. On entry lane e holds the parity
// words of generator e (of 64) for 256 samples, dword q the samples 32 q ..
// 32 q + 31; on return each lane holds all 64 generators' bits of 4 samples,
// as nibbles of 4 generators, one table each. A lane's index bit is swapped
// with a dword's (lane bits 5 and 4 by gfx950's register swaps, bit 2 by masked
// DPP moves: no bit work) or with a bit's place inside the dword (lane bit 3
// with bit 4, a DPP move and a byte select; lane bits 1 and 0 with bits 1 and
// 0, so that the 4 generators of a table sit side by side). The samples' bits 2
// and 3 stay inside the dword: which sample comes to which lane does not
// matter, and 4 full 64x64 transposes would take 35 vector instructions and 2
// swizzles a word where this takes 20. Table t (bits t3 t2 t1 t0) of sample r
// (bits r1 r0) is the nibble r0 of byte 2 t1 + r1 of dword t3 t2 t0.
__device__ __forceinline__ void lut_transpose(uint32_t (&d)[8], int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // lane bit 5 with dword bit 2
        const auto r = __builtin_amdgcn_permlane32_swap(d[q], d[q + 4], false, false);
        d[q] = r[0];
        d[q + 4] = r[1];
    }
#pragma unroll
    for (int q = 0; q < 8; q += (q & 1) ? 3 : 1) {  // lane bit 4 with dword bit 1
        const auto r = __builtin_amdgcn_permlane16_swap(d[q], d[q + 2], false, false);
        d[q] = r[0];
        d[q + 2] = r[1];
    }
#pragma unroll
    for (int q = 0; q < 8; q += 2) {  // lane bit 2 with dword bit 0
        const uint32_t x = d[q], y = d[q + 1];
        d[q] = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)y, 0x114, 0xF, 0xA, false);
        d[q + 1] = (uint32_t)__builtin_amdgcn_update_dpp((int)y, (int)x, 0x104, 0xF, 0x5, false);
    }
    const uint32_t sel = (lane & 8) ? 0x03020706u : 0x05040100u;
#pragma unroll
    for (int q = 0; q < 8; ++q)  // lane bit 3 with bit 4
        d[q] = __builtin_amdgcn_perm(lane_xor<8>(d[q]), d[q], sel);
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
        small_stage<2, 1, 0x33333333u>(d[q], d[q + 1], lane);
        small_stage<1, 0, 0x55555555u>(d[q], d[q + 1], lane);
    }
}

// The sample (of the wave's 256) that lane holds as its r-th after
// lut_transpose.
__device__ __forceinline__ int lut_sample(int lane, int r) {
    return (lane & 3) | (r << 2) | ((lane & 8) << 1) | ((lane & 4) << 3) | ((lane & 48) << 2);
}

template <bool kIndep>
__device__ __forceinline__ void sparse_fwd_lut_body(const SparseFwdArgs &a, int64_t blk) {
    const int64_t nchunk = ceil_div(a.s, kEpiChunk);
    const int64_t ch = blk / a.l, k = blk - ch * a.l;  // chunk-major, as the backward
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    __shared__ __attribute__((aligned(16))) float tab[kLutTables * 16];
    __shared__ int32_t lst[kLutList];
    __shared__ int wsum[2][4];
    __shared__ double red[3][4];
    const int64_t sw = ch * kSpWords + 4 * wave;  // the wave's first sample word
    const glb<const float> t32 = gptr(a.t32);
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, kpi[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    double Tp = 0.0;  // this thread's share of T_k
    auto fill = [&](int n) {
        {  // table tid: entries 4 tid .. 4 tid + 3 (0 past the list)
            float t[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int e = 4 * tid + b;
                t[b] = e < n ? t32[lst[e]] : 0.0f;
                Tp += (double)t[b];
            }
            const float x[4] = {0.0f, t[0], t[1], t[0] + t[1]};
            const float y[4] = {0.0f, t[2], t[3], t[2] + t[3]};
            float4 *row = reinterpret_cast<float4 *>(tab + tid * 16);
#pragma unroll
            for (int h = 0; h < 4; ++h)
                row[h] = make_float4(x[0] + y[h], x[1] + y[h], x[2] + y[h], x[3] + y[h]);
        }
        __syncthreads();
        const char *tb = reinterpret_cast<const char *>(tab);
        for (int g = 0; 64 * g < n; ++g) {
            const int e = 64 * g + lane;
            u32x4 wv[2] = {u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}};
            if (e < n) lut_fwd_words<kIndep>(a, k, sw, lst[e], wv);
            uint32_t d[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) d[q] = wv[q / 4][q % 4];
            lut_transpose(d, lane);
            const uint32_t gb = (uint32_t)g * 1024u;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                uint32_t m[8];  // byte i: 4 * its low (c = 0) or high nibble
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    m[q] = (c == 0 ? d[q] << 2 : d[q] >> 2) & 0x3C3C3C3Cu;
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int r = 2 * o + c;
                    float v[16];
#pragma unroll
                    for (int t = 0; t < 16; ++t) {
                        const uint32_t at = __builtin_amdgcn_perm(
                            gb, m[(t & 1) | ((t >> 1) & 6)],
                            0x07060500u | (uint32_t)(2 * ((t >> 1) & 1) + o));
                        v[t] = *reinterpret_cast<const float *>(tb + t * 64 + at);
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float p =
                            ((v[8 * h] + v[8 * h + 1]) + (v[8 * h + 2] + v[8 * h + 3])) +
                            ((v[8 * h + 4] + v[8 * h + 5]) + (v[8 * h + 6] + v[8 * h + 7]));
                        acc[r] += p;
                        const float qq = rintf(acc[r] * kInvPiF);
                        acc[r] = fmaf(-qq, kPiF, acc[r]);
                        kpi[r] += qq;
                    }
                }
            }
        }
    };
    if (!weight_zero(a.bsrc, k)) compact_row(gptr(a.crm) + k * a.Gw, a.Gw, lst, wsum, fill);

    // T_k = the sum of the threads' shares (waves, then the 4 wave sums in order)
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) Tp += __shfl_xor(Tp, st, 64);
    if (lane == 0) red[0][wave] = Tp;
    __syncthreads();
    const double T = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    double sc = 0.0, sc2 = 0.0;
    float IQP_GLOBAL *ph = a.phase_out ? gptr(a.phase_out) + k * a.s : nullptr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t i = sw * 64 + lut_sample(lane, r);
        if (i < a.s) {
            const double e = T - 2.0 * ((double)acc[r] + (double)kpi[r] * (double)kPiF);
            const double kk = rint(e * IQP_INV_TWO_PI);
            double rr = fma(-kk, IQP_TWO_PI_HI, e);
            rr = fma(-kk, IQP_TWO_PI_LO, rr);
            const float rf = (float)rr;
            const float c = cosf(rf);
            if (ph) ph[i] = rf;
            sc += (double)c;
            sc2 += (double)c * (double)c;
        }
    }
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) {
        sc += __shfl_xor(sc, st, 64);
        sc2 += __shfl_xor(sc2, st, 64);
    }
    if (lane == 0) {
        red[1][wave] = sc;
        red[2][wave] = sc2;
    }
    __syncthreads();
    if (tid == 0) {
        sc = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
        sc2 = (red[2][0] + red[2][1]) + (red[2][2] + red[2][3]);
        if (nchunk == 1) {
            finalize_store(a.fin, k, sc, sc2);
        } else {
            double IQP_GLOBAL *part = gptr(a.part) + (k * nchunk + ch) * 2;
            part[0] = sc;
            part[1] = sc2;
        }
    }
}

// One block per (observable, chunk) unit. When the units outnumber the grid
// (at most kMaxBlocks blocks), the strided form takes them in steps of the
// grid's size, with a barrier before a block's next unit rewrites its LDS;
// it is a separate instantiation because the loop costs the body registers
// (98 and 99 instead of 77 and 80 VGPRs: two waves per SIMD).
template <bool kIndep, bool kStrided>
__global__ __launch_bounds__(256) void sparse_fwd_lut_kernel(SparseFwdArgs a, int64_t units) {
    if (!kStrided) {
        sparse_fwd_lut_body<kIndep>(a, (int64_t)blockIdx.x);
        return;
    }
    for (int64_t b = blockIdx.x; b < units; b += gridDim.x) {
        sparse_fwd_lut_body<kIndep>(a, b);
        __syncthreads();
    }
}

template <bool kIndep, bool kStrided, int kC>
__global__ __launch_bounds__(256) void sparse_bwd_lut_kernel(SparseBwdArgs a, int64_t units) {
    if (!kStrided) {
        sparse_bwd_lut_body<kIndep, kC>(a, (int64_t)blockIdx.x);
        return;
    }
    for (int64_t b = blockIdx.x; b < units; b += gridDim.x) {
        sparse_bwd_lut_body<kIndep, kC>(a, b);
        __syncthreads();
    }
}

// Blocks of a table-lookup launch: one per unit up to kMaxBlocks, or fewer
// when IQP_SPARSE_GRID_CAP is set, so that tests can take the strided path
// at small sizes.
static int64_t lut_grid(int64_t units) {
    const char *c = getenv("IQP_SPARSE_GRID_CAP");
    const long long v = c ? atoll(c) : 0;
    const int64_t cap = v > 0 ? (int64_t)v : (int64_t)kMaxBlocks;
    const int64_t g = units < cap ? units : cap;
    return g < kMaxBlocks ? g : kMaxBlocks;
}

hipError_t launch_sparse_fwd(const LaunchCtx &lc, const SparseFwdArgs &a) {
    const int64_t units = a.l * ceil_div(a.s, kEpiChunk);
    if (units <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)lut_grid(units);
    hipEvent_t ev;
    timed_begin(lc, KF_FWD, &ev);
    const bool strided = (int64_t)blocks < units;
    if (a.bsrc.xt && strided)
        hipLaunchKernelGGL((sparse_fwd_lut_kernel<true, true>), dim3(blocks), dim3(256), 0,
                           lc.stream, a, units);
    else if (a.bsrc.xt)
        hipLaunchKernelGGL((sparse_fwd_lut_kernel<true, false>), dim3(blocks), dim3(256), 0,
                           lc.stream, a, units);
    else if (strided)
        hipLaunchKernelGGL((sparse_fwd_lut_kernel<false, true>), dim3(blocks), dim3(256), 0,
                           lc.stream, a, units);
    else
        hipLaunchKernelGGL((sparse_fwd_lut_kernel<false, false>), dim3(blocks), dim3(256), 0,
                           lc.stream, a, units);
    hipError_t e = hipGetLastError();
    timed_end(lc, KF_FWD, ev);
    return e;
}

template <bool kIndep, int kC>
static void launch_bwd_lut(const LaunchCtx &lc, const SparseBwdArgs &a) {
    const int64_t units = a.l * ceil_div(a.s, kC * kEpiChunk);
    const unsigned blocks = (unsigned)lut_grid(units);
    if ((int64_t)blocks < units)
        hipLaunchKernelGGL((sparse_bwd_lut_kernel<kIndep, true, kC>), dim3(blocks), dim3(256), 0,
                           lc.stream, a, units);
    else
        hipLaunchKernelGGL((sparse_bwd_lut_kernel<kIndep, false, kC>), dim3(blocks), dim3(256), 0,
                           lc.stream, a, units);
}

hipError_t launch_sparse_bwd(const LaunchCtx &lc, const SparseBwdArgs &a) {
    if (a.l <= 0 || a.s <= 0) return hipSuccess;
    hipEvent_t ev;
    timed_begin(lc, KF_BWD, &ev);
    const int64_t chunks = ceil_div(a.s, kEpiChunk);
    if (a.bsrc.xt)
        launch_bwd_lut<true, 1>(lc, a);
    else if (chunks > 1 && a.l * ceil_div(chunks, 2) >= kPairBlocks * (1 + chunks % 2))
        launch_bwd_lut<false, 2>(lc, a);
    else
        launch_bwd_lut<false, 1>(lc, a);
    hipError_t e = hipGetLastError();
    timed_end(lc, KF_BWD, ev);
    return e;
}

__device__ __forceinline__ void sparse_finish_body(const SparseFinishArgs &a, int64_t blk) {
    const int64_t j = blk * 256 + threadIdx.x;
    if (j >= a.m) return;
    const bool bad = gptr(a.acc)[a.m_pad] != 0;
    gptr(a.grad)[j] = bad ? (double)NAN : -2.0 * (double)gptr(a.acc)[j] / gptr(a.scale)[0];
}

hipError_t launch_sparse_finish(const LaunchCtx &lc, const SparseFinishArgs &a) {
    return plain_launch<SparseFinishArgs, sparse_finish_body>(lc, KF_GRAD, a, blocks_of(a));
}

// ---------------------------------------------------------------------------
// FP32 forward over the non-zero entries of C (ChainGate). The 32x32x2 FP32
// matrix product is a chain of fused multiply-adds in K order (checked against
// fmaf, zeros left out, over random operands), so E of one gate split is the
// running FP32 sum of +-2 theta'_j over the anticommuting gates in gate order,
// and this kernel, which adds just those terms in that order, gives the same
// bits. A block takes observable k and 2048 samples, a lane 8 consecutive
// samples; the row of C is compacted into an LDS list as in the table-lookup
// kernels, and per entry a wave loads one parity byte per lane (64 contiguous
// bytes of B^T) and adds under its bits: a shift, a sign insert and an add per
// term, against a matrix-core term for every entry of C, zero or not. n = 300,
// 517 observables, 2501 samples, C 1.3 % full (7.7e8 non-zero terms): 0.148 ms, 5.2e12
// terms/s; the matrix-core kernel 1.95 ms, 3.0e13 of all terms. The vector units
// issue on 62 % of the cycles, 4.7 instructions a term; the rest is waiting for
// the parity bytes with too little else to run, 2.6 waves per SIMD over the run:
// the second block of an observable has 453 samples, one busy wave in four.
__device__ __forceinline__ void count_body(const CountArgs &a, int64_t blk) {
    __shared__ double sh[256];
    const int64_t total = a.l_pad * a.mw;
    int n = 0;
#pragma unroll
    for (int64_t q = 0; q < kCountWords / 256; ++q) {
        const int64_t i = blk * kCountWords + q * 256 + threadIdx.x;
        n += i < total ? __popcll(gptr(a.cbits)[i]) : 0;
    }
    const double s = block_sum_256((double)n, sh);
    if (threadIdx.x == 0) atomicAdd(a.nnz, (unsigned long long)s);
}

hipError_t launch_count(const LaunchCtx &lc, const CountArgs &a) {
    return plain_launch<CountArgs, count_body>(lc, KF_PARITY, a, blocks_of(a));
}

__device__ __forceinline__ void chain_fwd_body(const ChainFwdArgs &a, int64_t blk) {
    if (!chain_on(a.gate)) return;
    __shared__ int32_t lst[kLutList];
    __shared__ float tl[kLutList];
    __shared__ int wsum[2][4];
    __shared__ double red[2][4];
    const int64_t nchunk = ceil_div(a.s, kEpiChunk);
    const int64_t ch = blk / a.l, k = blk - ch * a.l;  // chunk-major
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int64_t i0 = ch * kChainChunk + wave * 512 + lane * 8;  // the lane's first sample
    const bool active = ch * kChainChunk + wave * 512 < a.s;      // uniform over the wave
    const glb<const uint64_t> crow = gptr(a.cbits) + (k >> 5) * a.mw * 32 + (k & 31);
    // samples past s: any byte of the row
    const glb<const uint8_t> bytes = (glb<const uint8_t>)gptr(a.btrm);
    const uint32_t boff = i0 < a.s ? (uint32_t)(i0 >> 3) : 0u;
    const int64_t stride = a.Rw * 8;
    const int64_t half = a.m_pad >> 1;
    float acc[8];
    double E[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        acc[b] = 0.0f;
        E[b] = 0.0;
    }
    auto fill = [&](int n) {
        // pad to whole groups of 8 with zero terms
        const int np = (n + 7) & ~7;
        for (int e = tid; e < np; e += 256) {
            if (e >= n) lst[e] = 0;
            const int64_t j = e < n ? lst[e] : 0;
            tl[e] = e < n ? gptr(a.t32)[(j & 1) * half + (j >> 1)] : 0.0f;
        }
        __syncthreads();
        if (!active) return;
        uint32_t nx[8], cu[8];
        auto load = [&](int e) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                nx[q] = (bytes + (int64_t)__builtin_amdgcn_readfirstlane(lst[e + q]) * stride)[boff];
        };
        if (np > 0) load(0);
        for (int e = 0; e < np; e += 8) {
#pragma unroll
            for (int q = 0; q < 8; ++q) cu[q] = nx[q];
            if (e + 8 < np) load(e + 8);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(tl[e + q]));
                const uint32_t y = cu[q] ^ (uint32_t)((int32_t)t >> 31);
                const float mag = __uint_as_float(t & 0x7FFFFFFFu);
#pragma unroll
                for (int b = 0; b < 8; ++b)
                    acc[b] += __builtin_copysignf(mag, __uint_as_float(y << (31 - b)));
            }
        }
    };
    const int64_t wps = ceil_div(a.mw, a.splits);
    for (int64_t sp = 0; sp < a.splits; ++sp) {
        const int64_t w0 = sp * wps, w1 = w0 + wps < a.mw ? w0 + wps : a.mw;
        compact_words([&](int64_t w) { return crow[w * 32]; }, w0, w1, lst, wsum, fill);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            E[b] += (double)acc[b];
            acc[b] = 0.0f;
        }
        __syncthreads();  // the list is filled anew
    }
    double sc = 0.0, sc2 = 0.0;
    float IQP_GLOBAL *ph = a.phase_out ? gptr(a.phase_out) + k * a.s : nullptr;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        if (i0 + b < a.s) {
            const double kk = rint(E[b] * IQP_INV_TWO_PI);
            double rr = fma(-kk, IQP_TWO_PI_HI, E[b]);
            rr = fma(-kk, IQP_TWO_PI_LO, rr);
            const float rf = (float)rr;
            const float c = cosf(rf);
            if (ph) ph[i0 + b] = rf;
            sc += (double)c;
            sc2 += (double)c * (double)c;
        }
    }
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) {
        sc += __shfl_xor(sc, st, 64);
        sc2 += __shfl_xor(sc2, st, 64);
    }
    if (lane == 0) {
        red[0][wave] = sc;
        red[1][wave] = sc2;
    }
    __syncthreads();
    const int64_t c2 = ch * 2 + tid;  // the block's two epilogue chunks
    if (tid < 2 && c2 < nchunk) {
        sc = red[0][2 * tid] + red[0][2 * tid + 1];
        sc2 = red[1][2 * tid] + red[1][2 * tid + 1];
        if (nchunk == 1) {
            finalize_store(a.fin, k, sc, sc2);
        } else {
            double IQP_GLOBAL *part = gptr(a.part) + (k * nchunk + c2) * 2;
            part[0] = sc;
            part[1] = sc2;
        }
    }
}

hipError_t launch_chain_fwd(const LaunchCtx &lc, const ChainFwdArgs &a) {
    return plain_launch<ChainFwdArgs, chain_fwd_body>(lc, KF_FWD, a, blocks_of(a));
}

// FP32 backward over the non-zero entries of C, by the same argument: T_kj of a
// sample split is the running FP32 sum of +-S_ki in sample order, and only
// entries with c_kj = 1 reach the gradient, where the matrix-core kernel adds
// them row by row, alternate groups of four rows in two sums. A block takes
// observable k and a split: its gates are listed in LDS, a lane holds up to
// four of them, and walks the samples with |S_ki| and the signs of 64 samples
// read from LDS by all lanes at once. The T go to memory in row order; the
// second kernel gives a lane a gate, finds each T by the row's entries before
// the wave's 64 gates and a ballot, and adds them in the order above. At the
// sizes above 0.099 ms, 7.8e12 terms/s, bound by the vector units, which issue on
// 80 % of the cycles, 4 instructions a term (three for the term, the rest for
// the weights, which every block of a row computes), and 0.033 ms for the sums
// (vector instructions on 30 % of the cycles: the scalar work per row and the
// latency of the loads).
// Ranks: a wave takes the rows 4 b + v, 4 b + v + 4 (blocks), ..., 256 words at a
// time. At most 1024 blocks, whose additions to the one counter follow one
// another: a block per row took 221 us for 20000 rows of 80 words.
__device__ __forceinline__ void rank_body(const RankArgs &a, int64_t blk) {
    __shared__ unsigned long long cnt[4];
    const int lane = threadIdx.x & 63, wv = wave_id();
    const int64_t step = blocks_of(a) * 4;
    unsigned long long total = 0ull;
    for (int64_t k = blk * 4 + wv; k < a.l; k += step) {
        const glb<const uint64_t> row = gptr(a.crm) + k * a.mw;
        int n = 0;
        for (int64_t base = 0; base < a.mw; base += 256) {
            int c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t w = base + 64 * q + lane;
                c[q] = w < a.mw ? __popcll(row[w]) : 0;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t w = base + 64 * q + lane;
                int x = c[q];
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int y = __shfl_up(x, d, 64);
                    if (lane >= d) x += y;
                }
                if (w < a.mw) gptr(a.rank)[k * a.mw + w] = (uint32_t)(n + x - c[q]);
                n += __builtin_amdgcn_readlane(x, 63);
            }
        }
        // a row without room: the top bit, which no number of entries reaches
        if (n > a.cap) total |= 1ull << 63;
        total += (unsigned long long)n;
    }
    if (lane == 0) cnt[wv] = total;
    __syncthreads();
    if (threadIdx.x != 0) return;
    const unsigned long long top = (cnt[0] | cnt[1] | cnt[2] | cnt[3]) & (1ull << 63);
    const unsigned long long all = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    if (top) atomicOr(a.nnz, top);
    else if (all) atomicAdd(a.nnz, all);
}

hipError_t launch_rank(const LaunchCtx &lc, const RankArgs &a) {
    return plain_launch<RankArgs, rank_body>(lc, KF_PARITY, a, blocks_of(a));
}

// NQ gates per lane over one word of 64 samples: acc[q] += +-|S| in order.
template <int NQ>
__device__ __forceinline__ void chain_word(float (&acc)[4], const uint64_t (&y)[4],
                                           const float *mag) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const float4 m = *reinterpret_cast<const float4 *>(mag + 32 * h + 4 * g);
            const float mv[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    acc[q] += __builtin_copysignf(
                        mv[b], __uint_as_float((uint32_t)(y[q] >> (32 * h)) << (31 - 4 * g - b)));
        }
    }
}

__device__ __forceinline__ void chain_bwd_body(const ChainBwdArgs &a, int64_t blk) {
    if (!chain_on(a.gate)) return;
    __shared__ int32_t lst[kLutList];
    __shared__ __attribute__((aligned(16))) float mag[kEpiChunk];
    __shared__ uint64_t sgn[kSpWords];
    __shared__ int wsum[2][4];
    const int64_t ks = blk / a.l, k = blk - ks * a.l;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int64_t sw = a.s_pad / 64, wps = ceil_div(sw, a.ksplits);
    const int64_t w0 = ks * wps, w1 = w0 + wps < sw ? w0 + wps : sw;
    const double al = gptr(a.coef)[2 * k], be = gptr(a.coef)[2 * k + 1];
    const glb<const uint64_t> bt = gptr(a.btbits);
    float IQP_GLOBAL *T = gptr(a.T) + (ks * a.l + k) * a.cap;
    auto fill = [&](int n) {
        // no entry (an observable of weight 0, or a row of whole lists): no pass
        // over the samples (uniform over the block)
        if (n == 0) return;
        // gates of this wave: entries q 256 + 64 wave + lane
        const int left = n - wave * 64;
        const int nq = __builtin_amdgcn_readfirstlane(left <= 0 ? 0 : (left + 255) / 256);
        int32_t j[4];
        float acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = q * 256 + tid;
            j[q] = e < n ? lst[e] : 0;
            acc[q] = 0.0f;
        }
        for (int64_t c0 = w0; c0 < w1; c0 += kSpWords) {
            __syncthreads();  // mag and sgn of the chunk before are read
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = c0 * 64 + q * 256 + tid;
                float v = 0.0f;
                if (i < a.s) {
                    float sn, cs;
                    sincosf(gptr(a.phase)[k * a.s + i], &sn, &cs);
                    v = (float)((al + be * (double)cs) * (double)sn);
                }
                mag[q * 256 + tid] = fabsf(v);
                const uint64_t m = __ballot(__float_as_int(v) < 0);
                if (lane == 0) sgn[q * 4 + wave] = m;
            }
            __syncthreads();
            if (!nq) continue;
            const int nw = (int)(w1 - c0 < kSpWords ? w1 - c0 : kSpWords);
            uint64_t nx[4], y[4];
            auto load = [&](int w) {
                const glb<const uint64_t> row = bt + (c0 + w) * a.m_pad;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < nq) nx[q] = row[(uint32_t)j[q]];
            };
            load(0);
            for (int w = 0; w < nw; ++w) {
                const uint64_t sg = sgn[w];
#pragma unroll
                for (int q = 0; q < 4; ++q) y[q] = nx[q] ^ sg;
                if (w + 1 < nw) load(w + 1);
                const float *mw = mag + w * 64;
                if (nq == 4) chain_word<4>(acc, y, mw);
                else if (nq == 3) chain_word<3>(acc, y, mw);
                else if (nq == 2) chain_word<2>(acc, y, mw);
                else chain_word<1>(acc, y, mw);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q * 256 + tid < n) T[q * 256 + tid] = acc[q];
        T += n;
    };
    compact_row(gptr(a.crm) + k * a.mw, a.mw, lst, wsum, fill);
}

hipError_t launch_chain_bwd(const LaunchCtx &lc, const ChainBwdArgs &a) {
    return plain_launch<ChainBwdArgs, chain_bwd_body>(lc, KF_BWD, a, blocks_of(a));
}

// One block per 64 gates; wave v takes the 64-row words v, v + 4, ... of C^T.
__device__ __forceinline__ void chain_grad_body(const ChainGradArgs &a, int64_t gw) {
    if (!chain_on(a.gate)) return;
    __shared__ double sh[4][64];
    const int lane = threadIdx.x & 63, wv = wave_id();
    const int64_t j = gw * 64 + lane;
    double acc = 0.0;
    for (int64_t ob = wv; ob < a.lw; ob += 4) {
        const uint64_t word = gptr(a.ctbits)[ob * a.m_pad + j];
        if (__ballot(word != 0ull) == 0ull) continue;
        float gs[kChainMaxSplits][2];
#pragma unroll
        for (int q = 0; q < (int)kChainMaxSplits; ++q) gs[q][0] = gs[q][1] = 0.0f;
        // the entries of this word's rows before the wave's gates, lane r: row r
        const int64_t kr = ob * 64 + lane;
        const uint32_t mine = kr < a.l ? gptr(a.rank)[kr * a.mw + gw] : 0u;
#pragma unroll
        for (int r0 = 0; r0 < 64; r0 += 4) {
            uint32_t slot[4];
            bool bit[4];
            bool any = false;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bit[i] = (word >> (r0 + i)) & 1ull;
                const uint64_t b = __ballot(bit[i]);
                any |= b != 0ull;
                slot[i] = (uint32_t)__builtin_amdgcn_readlane((int)mine, r0 + i) +
                          (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
            }
            if (!any) continue;  // uniform over the wave
#pragma unroll
            for (int q = 0; q < (int)kChainMaxSplits; ++q) {
                if (q >= a.ksplits) break;
                float t[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    t[i] = bit[i] ? gptr(a.T)[((q * a.l) + ob * 64 + r0 + i) * a.cap + slot[i]] : 0.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) gs[q][(r0 >> 2) & 1] += t[i];
            }
        }
#pragma unroll
        for (int q = 0; q < (int)kChainMaxSplits; ++q)
            if (q < a.ksplits) acc += (double)(gs[q][0] + gs[q][1]);
    }
    sh[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && j < a.m)
        gptr(a.grad)[j] = -2.0 * (((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane]);
}

hipError_t launch_chain_grad(const LaunchCtx &lc, const ChainGradArgs &a) {
    return plain_launch<ChainGradArgs, chain_grad_body>(lc, KF_GRAD, a, blocks_of(a));
}

// ---------------------------------------------------------------------------
// Bit columns of every observable's own sample set. A step is (set k, group g
// of 16 row words = 1024 rows, chunk c of 8 qubit words); ldx is a multiple
// of 16. Persistent blocks (two per CU: LDS and registers allow two) take
// steps b, b + grid, ...: the block reads words [8c, 8c + 8) of its 1024 rows
// with coalesced loads (8 lanes cover one row's run) into registers, moves
// them to LDS (row stride 9 words, so the column reads below hit distinct
// banks) and issues the loads of its next step, which stay in flight while
// wave v transposes words v and v + 4: for each of the 16 64-row blocks lane
// r takes row r's word from LDS and the 64 x 64 bit transpose leaves lane q
// with column 64 w + q, so lane q writes that column's 16 row words as one
// 128-byte run, a whole cache line. Every sample word is read once and every
// output line written by one lane. Rows past s read as 0.
constexpr int kSliceWords = 16;  // row words per step: 1024 rows
constexpr int kSliceChunk = 8;   // qubit words per step
constexpr int kSliceStride = kSliceChunk + 1;
constexpr int64_t kSliceBlocks = 512;

struct SliceStep {
    int64_t k, g;
    int w0, cw;
};

__device__ __forceinline__ SliceStep slice_step(const IndepSliceArgs &a, int64_t q) {
    const int64_t ngrp = a.ldx / kSliceWords;
    const int nch = (a.W + kSliceChunk - 1) / kSliceChunk;
    const int64_t u = q / nch;
    SliceStep st;
    st.w0 = (int)(q - u * nch) * kSliceChunk;
    st.cw = a.W - st.w0 < kSliceChunk ? a.W - st.w0 : kSliceChunk;
    st.k = u / ngrp;
    st.g = u - st.k * ngrp;
    return st;
}

// this thread's 32 words of a step: word j of rows r0 + 32 it (rows past s
// read row s - 1 here and are zeroed when stored to LDS, so that nothing
// waits on these loads before then)
__device__ __forceinline__ void slice_load(const IndepSliceArgs &a, const SliceStep &st, int j,
                                           int r0, uint64_t (&v)[32]) {
    if (j >= st.cw) return;
    const uint64_t IQP_GLOBAL *rows = gptr(a.samples) + st.k * a.s * a.W + st.w0 + j;
    const int64_t base = st.g * (kSliceWords * 64) + r0;
#pragma unroll
    for (int it = 0; it < 32; ++it) {
        const int64_t row = base + 32 * it;
        v[it] = rows[(row < a.s ? row : a.s - 1) * a.W];
    }
}

__device__ __forceinline__ void indep_slice_body(const IndepSliceArgs &a, int64_t blk) {
    __shared__ uint64_t stage[kSliceWords * 64 * kSliceStride];
    const int64_t total = a.l * (a.ldx / kSliceWords) * ((a.W + kSliceChunk - 1) / kSliceChunk);
    const int64_t grid = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = tid & (kSliceChunk - 1);  // word within the chunk this thread loads
    const int r0 = tid / kSliceChunk;       // first of its rows; the rest step by 32
    uint64_t v[32];
    SliceStep st = slice_step(a, blk);
    if (blk < total) slice_load(a, st, j, r0, v);
    for (int64_t q = blk; q < total; q += grid) {
        __syncthreads();  // the previous step's LDS reads are done
        if (j < st.cw) {
            const int64_t base = st.g * (kSliceWords * 64) + r0;
#pragma unroll
            for (int it = 0; it < 32; ++it)
                stage[(r0 + 32 * it) * kSliceStride + j] = base + 32 * it < a.s ? v[it] : 0ull;
        }
        __syncthreads();
        const SliceStep cur = st;
        if (q + grid < total) {
            st = slice_step(a, q + grid);
            slice_load(a, st, j, r0, v);
        }
        uint64_t IQP_GLOBAL *set = gptr(a.xt) + cur.k * 64 * a.W * a.ldx + cur.g * kSliceWords;
        for (int jw = wave; jw < cur.cw; jw += 4) {
            uint64_t y[kSliceWords];
#pragma unroll
            for (int t = 0; t < kSliceWords; ++t)
                y[t] = transpose64(stage[(t * 64 + lane) * kSliceStride + jw], lane);
            uint64_t IQP_GLOBAL *dst = set + (int64_t)((cur.w0 + jw) * 64 + lane) * a.ldx;
#pragma unroll
            for (int t = 0; t < kSliceWords; ++t) dst[t] = y[t];
        }
    }
}

hipError_t launch_indep_slice(const LaunchCtx &lc, const IndepSliceArgs &a) {
    if (a.ldx % kSliceWords != 0 || a.s < 1) return hipErrorInvalidValue;
    const int64_t steps = a.l * (a.ldx / kSliceWords) * ((a.W + kSliceChunk - 1) / kSliceChunk);
    return plain_launch<IndepSliceArgs, indep_slice_body>(lc, KF_PARITY, a,
                                                          steps < kSliceBlocks ? steps : kSliceBlocks);
}

}  // namespace iqp
