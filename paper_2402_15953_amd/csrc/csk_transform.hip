// Power-of-two transforms over the sketches: the fp64 complex FFT used by the estimate
// (Alg. 3 evaluates cross-correlations through FFT / IFFT) and the number-theoretic
// transform (same structure, Montgomery arithmetic modulo a 31-bit prime) used for the
// exact modular evaluation.
//
// Lengths up to 4096 are done in one pass inside LDS.  Longer lengths m = N1 * N2 (N2 =
// 2^S, from 1024 to 4096, default_split_bits() or the tuned split) use the four-step decomposition
// (Bailey): element n = N2 n1 + n2.
//   forward: pass 1 transforms each column n2 over n1 (stride N2) and multiplies output
//            f1 by w_m^(f1 n2); pass 2 transforms each row over n2.  Position N2 f1 + f2
//            then holds frequency f = f1 + N1 f2 (no final transpose).
//   inverse: takes that permuted order back to natural order: row pass over f2 with
//            w_m^(-n2 f1) applied to output n2, then the column pass over f1.
// Inside LDS each tile is loaded in bit-reversed order and finished by radix-2
// decimation-in-time stages; twiddles come from host-computed tables.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "csk_internal.h"
#include "csk_rings.h"
#include "csk_transform.h"

namespace csk {

namespace {

// A block transforms one tile of TILE elements: the fp64 FFT with TILE / 4 threads (two
// butterflies per thread per stage; the pass is bound by memory and wants the loads of
// many wavefronts), the NTT with TILE / 8 (four per thread: its passes wait on their
// barriers, and two independent butterfly groups per thread between two barriers
// measured 13-20% faster than one; four per thread were slower again).  Two-pass lengths use the smallest tile that keeps the column
// pass's reads in runs of at least 8 elements: a 2^16-point transform is 64 blocks of
// 1024 elements per vector (24 KB of LDS each, several blocks per CU) rather than 16
// blocks of 4096 (96 KB, one per CU), so its passes fill the chip.
constexpr int kSingleTile = 4096;

// LDS position of tile element i: one padding word after every 32, so that the
// bit-reversed loads (whose first 64 positions are multiples of the tile length / 64)
// and the butterflies at small strides spread over the banks instead of meeting on a
// few of them.
__device__ __forceinline__ int lp(int i) { return i + (i >> 5); }
template <int TILE>
constexpr int lds_len() { return TILE + TILE / 32; }

__device__ __forceinline__ uint32_t bitrev(uint32_t x, int bits)
{
    return bits ? (__brev(x) >> (32 - bits)) : 0u;
}

// Copies w_L^j (j < L / 2, L = 2^log2L) from the table tw[k] = w_T^k, T = 2^log2T, into
// LDS; every stage of a length-L transform takes its twiddles from there.
template <int NT, class T>
__device__ __forceinline__ void load_stage_twiddles(T *stw, int log2L, const T *__restrict__ tw, int log2T)
{
    for (int j = threadIdx.x; j < (1 << (log2L - 1)); j += NT) stw[j] = tw[(size_t)j << (log2T - log2L)];
}

// Radix-2 DIT stages on C interleaved transforms of length 2^log2L held in LDS as
// s[lp(n * C + c)] (bit-reversed input, natural output); stw from load_stage_twiddles.
// Stages go in pairs: a thread takes the four elements two consecutive stages combine,
// applies both stages' radix-2 butterflies in registers (the same operations as two
// separate stages, so the same rounding), and writes them back once.
//
// Addressing: with D = half * C the tile distance between a group's elements, group b
// starts at idx0 = ((b >> log2 D) << (log2 D + 2)) + (b & (D - 1)), and its block of 4D
// tile positions starts at a multiple of 4D.  A power-of-two block of at most 32
// positions then lies inside one 32-position stretch, and larger ones start on one, so
// element j sits jD + (jD >> 5) padded positions after element 0 for every group: one
// padded address per group, the other three at offsets uniform over the stage.
template <int NT, class Ring>
__device__ __forceinline__ void lds_stages(typename Ring::T *s, int log2L, int log2C, const Ring &R,
                                           const typename Ring::T *stw)
{
    using T = typename Ring::T;
    int lh = 0;
    for (; lh + 1 < log2L; lh += 2) {
        const int sD = lh + log2C;
        const int D = 1 << sD;
        const int o1 = D + (D >> 5), o2 = 2 * D + ((2 * D) >> 5), o3 = 3 * D + ((3 * D) >> 5);
        const int sh2 = log2L - lh - 2;           // twiddle index shift of the second stage
        const int quarter = 1 << (log2L - 2);     // (k + half) << sh2 = (k << sh2) + quarter
        const int kmask = (1 << lh) - 1;
        const int ngr = (1 << (log2L - 2)) << log2C;
        for (int b = threadIdx.x; b < ngr; b += NT) {
            T *e = s + lp(((b >> sD) << (sD + 2)) + (b & (D - 1)));
            const int w2i = ((b >> log2C) & kmask) << sh2;
            const T x0 = e[0], x1 = e[o1], x2 = e[o2], x3 = e[o3];
            // stage lh: pairs (0, 1) and (2, 3), twiddle w_{2 half}^k
            const T w1 = stw[w2i << 1];
            T v = R.mul(x1, w1);
            const T y0 = R.add(x0, v), y1 = R.sub(x0, v);
            v = R.mul(x3, w1);
            const T y2 = R.add(x2, v), y3 = R.sub(x2, v);
            // stage lh + 1: pairs (0, 2) with w_{4 half}^k and (1, 3) with w_{4 half}^(k + half)
            const T w2 = stw[w2i];
            const T w3 = stw[w2i + quarter];
            v = R.mul(y2, w2);
            e[0] = R.add(y0, v);
            e[o2] = R.sub(y0, v);
            v = R.mul(y3, w3);
            e[o1] = R.add(y1, v);
            e[o3] = R.sub(y1, v);
        }
        __syncthreads();
    }
    for (; lh < log2L; ++lh) {  // the last stage when their number is odd
        const int sD = lh + log2C;
        const int D = 1 << sD;
        const int o1 = D + (D >> 5);
        const int sh = log2L - lh - 1;
        const int kmask = (1 << lh) - 1;
        const int nbf = (1 << (log2L - 1)) << log2C;
        for (int b = threadIdx.x; b < nbf; b += NT) {
            T *e = s + lp(((b >> sD) << (sD + 1)) + (b & (D - 1)));
            const T u = e[0];
            const T v = R.mul(e[o1], stw[((b >> log2C) & kmask) << sh]);
            e[0] = R.add(u, v);
            e[o1] = R.sub(u, v);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- fp64 complex FFT pass

// Source of a pass: either the complex work buffer, or (first pass) the int64 sketches
// of the (relation, repetition) pair packed into one complex vector: re + i * im.
struct F64Src {
    const int64_t *const *re;  // [n_vec] sketch loaded as the real part (null: in place)
    const int64_t *const *im;  // [n_vec] sketch loaded as the imaginary part (entry null: 0)
};

template <int TILE>
__global__ __launch_bounds__(TILE / 4) void k_fft_f64(F64Src src, double2 *buf, PassGeom g,
                                                     const double2 *__restrict__ tw, int log2T,
                                                     const double2 *__restrict__ stage, int log2S)
{
    constexpr int NT = TILE / 4;
    __shared__ double2 s[lds_len<TILE>()];
    __shared__ double2 stw[TILE / 2];
    const int v = blockIdx.x;
    const int blk = blockIdx.y;
    const int C = 1 << g.log2C;
    const int L = 1 << g.log2L;
    const int64_t m = (int64_t)1 << g.log2m;
    const int64_t base = (int64_t)blk * g.block_stride;
    double2 *vec = buf + (size_t)v * m;
    const int total = L << g.log2C;
    if (src.re) {
        const int64_t *re = src.re[v];
        const int64_t *im = src.im[v];
        for (int idx = threadIdx.x; idx < total; idx += NT) {
            const int n = idx >> g.log2C, c = idx & (C - 1);
            const int64_t pos = base + (int64_t)c * g.col_stride + (int64_t)n * g.elem_stride;
            s[lp((bitrev(n, g.log2L) << g.log2C) + c)] =
                make_double2((double)re[pos], im ? (double)im[pos] : 0.0);
        }
    } else {
        for (int idx = threadIdx.x; idx < total; idx += NT) {
            const int n = idx >> g.log2C, c = idx & (C - 1);
            const int64_t pos = base + (int64_t)c * g.col_stride + (int64_t)n * g.elem_stride;
            s[lp((bitrev(n, g.log2L) << g.log2C) + c)] = vec[pos];
        }
    }
    load_stage_twiddles<NT>(stw, g.log2L, stage, log2S);
    __syncthreads();
    RingC R;
    lds_stages<NT, RingC>(s, g.log2L, g.log2C, R, stw);
    for (int idx = threadIdx.x; idx < total; idx += NT) {
        const int n = idx >> g.log2C, c = idx & (C - 1);
        const int64_t pos = base + (int64_t)c * g.col_stride + (int64_t)n * g.elem_stride;
        double2 val = s[lp((n << g.log2C) + c)];
        if (g.twiddle) {
            const int64_t colid = (int64_t)blk * C + c;
            const int64_t e = ((int64_t)n * colid) & (m - 1);
            val = R.mul(val, tw[(size_t)e << (log2T - g.log2m)]);
        }
        vec[pos] = val;
    }
}

// ---------------------------------------------------------------- NTT pass

struct ModSrc {
    const int64_t *const *ptr;  // [vec_per_prime] sketch of vector v % vec_per_prime (null: in place)
};

// The NTT holds sixteen elements per thread and takes up to four stages between two trips
// through LDS: a transform of length 2^LG is one to three rounds of decimation in frequency
// with radices 2^rbits(LG, round), each round's DFTs in registers.  Element s of the tile
// after a round is block b (the digits of the frequency found so far, first digit most
// significant) times the remaining length plus the index within it, so a round reads and
// writes the same places and the last one's outputs sit at digit-reversed frequencies.
constexpr int kNttE = 16;  // elements per thread
constexpr int ntt_rounds(int lg) { return lg <= 4 ? 1 : lg <= 8 ? 2 : 3; }
constexpr int ntt_rbits(int lg, int round)
{
    return ntt_rounds(lg) == 1   ? lg
           : ntt_rounds(lg) == 2 ? (round == 0 ? (lg + 1) / 2 : lg / 2)
                                 : (round == 0 ? (lg + 2) / 3 : round == 1 ? (lg + 1) / 3 : lg / 3);
}
constexpr int ntt_threads(int lg, int lc) { return (1 << (lg + lc)) / kNttE < 64 ? 64 : (1 << (lg + lc)) / kNttE; }

// DFT of length 2^RB in registers, decimation in frequency: x[k] in, frequency bitrev(k)
// in x[k] out.  w[j] = w_R^j, j < R / 2.  Inputs below p.  The last stage's results are
// below 2p when `lazy` (a twiddle multiplies them next), else below p.
template <int RB, bool LAZY>
__device__ __forceinline__ void dft_regs(uint32_t (&x)[1 << RB], const RingM &R, const uint32_t *w)
{
    constexpr int N = 1 << RB;
#pragma unroll
    for (int st = 0; st < RB; ++st) {
        const int half = N >> (st + 1);
        const bool last = st == RB - 1;
#pragma unroll
        for (int b = 0; b < N; b += 2 * half)
#pragma unroll
            for (int k = 0; k < half; ++k) {
                const uint32_t a = x[b + k], c = x[b + k + half];
                const uint32_t u = a + c, v = a - c + R.p;  // both below 2p
                x[b + k] = LAZY && last ? u : min(u, u - R.p);
                // w_{2 half}^k = w_N^(k N / (2 half))
                x[b + k + half] = k == 0 ? (LAZY && last ? v : min(v, v - R.p)) : R.mul(v, w[k << st]);
            }
    }
}

constexpr int brev_bits(int x, int bits)
{
    int r = 0;
    for (int i = 0; i < bits; ++i) r |= ((x >> i) & 1) << (bits - 1 - i);
    return r;
}

// One round of the tile's transforms (see above).  src(n, c) supplies the first round's
// inputs, dst(f, c, value) takes the last one's outputs; s is the tile in LDS, stw the
// powers of w_L.  Every thread of the block calls it.
template <int LG, int LC, int ROUND, class Src, class Dst>
__device__ __forceinline__ void ntt_round(uint32_t *s, const uint32_t *stw, const RingM &R, const uint32_t *wr,
                                          Src &&src, Dst &&dst)
{
    constexpr int NR = ntt_rounds(LG), RB = ntt_rbits(LG, ROUND), N = 1 << RB;
    constexpr int done = ROUND == 0 ? 0 : ROUND == 1 ? ntt_rbits(LG, 0) : ntt_rbits(LG, 0) + ntt_rbits(LG, 1);
    constexpr int LJ = LG - done, LN = LJ - RB;  // log2 of the length before and after the round
    constexpr bool first = ROUND == 0, last = ROUND == NR - 1;
    constexpr int NT = ntt_threads(LG, LC);
    constexpr int groups = 1 << (LG + LC - RB);
#pragma unroll
    for (int g0 = 0; g0 < groups; g0 += NT) {
        const int g = g0 + threadIdx.x;
        if (groups < NT && g >= groups) break;
        const int c = g & ((1 << LC) - 1), h = g >> LC;
        // middle rounds: h = block * 2^LN + index; last round: h counts the blocks by their
        // frequency, first digit fastest, so that neighbouring lanes store neighbours
        int blk = h >> LN, i = h & ((1 << LN) - 1);
        if (last && NR == 3) {
            constexpr int r0 = ntt_rbits(LG, 0), r1 = ntt_rbits(LG, 1);
            blk = ((h & ((1 << r0) - 1)) << r1) | (h >> r0);
        }
        const int at = (((blk << LJ) + i) << LC) + c;  // element k at at + k 2^(LN + LC)
        uint32_t x[N];
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = first ? src(i + (k << LN), c) : s[lp(at + (k << (LN + LC)))];
        dft_regs<RB, !last>(x, R, wr);
        if (last) {
#pragma unroll
            for (int k = 0; k < N; ++k) dst(h + (k << done), c, k, x[brev_bits(k, RB)]);
        } else {
            // frequency digit k of index i: times w_(2^LJ)^(i k)
#pragma unroll
            for (int k = 0; k < N; ++k) {
                uint32_t v = x[brev_bits(k, RB)];
                v = k == 0 ? min(v, v - R.p) : R.mul(v, stw[(i * k) << (LG - LJ)]);
                s[lp(at + (k << (LN + LC)))] = v;
            }
        }
    }
}

// One pass: a block transforms 2^LC interleaved columns of length 2^LG.  Bound by the vector
// unit and memory about equally.  Two stages per trip through LDS with four elements per
// thread cost as much address arithmetic, LDS instructions and barriers as butterflies:
// 15 vectors of 2^21 at 3 primes took 213 us (columns) and 144 us (rows), 97 and 103 us in
// registers.
template <int LG, int LC>
__global__ __launch_bounds__(ntt_threads(LG, LC)) void k_ntt(ModSrc src, uint32_t *buf, PassGeom g, int vec_per_prime,
                                                             const PrimeDev *__restrict__ primes,
                                                             const uint32_t *__restrict__ roots, int log2T,
                                                             const uint32_t *__restrict__ stage, int log2S, int inverse)
{
    constexpr int TILE = 1 << (LG + LC), NT = ntt_threads(LG, LC), NR = ntt_rounds(LG);
    __shared__ uint32_t s[NR > 1 ? lds_len<TILE>() + 1 : 1];
    __shared__ uint32_t stw[NR > 1 ? 1 << LG : 1];
    const int v = blockIdx.x;
    const int pi = v / vec_per_prime;
    const PrimeDev &P = primes[pi];  // by reference: a copy with minv[] indexed would live in scratch
    const RingM R{P.p, P.pinv_neg};
    const uint32_t *tw = roots + ((size_t)(2 * pi + inverse) << log2T);
    const uint32_t *st = stage + ((size_t)(2 * pi + inverse) << log2S);
    const int blk = blockIdx.y;
    const int64_t m = (int64_t)1 << g.log2m;
    const int64_t base = (int64_t)blk * g.block_stride;
    uint32_t *vec = buf + (size_t)v * m;
    if (NR > 1)
        for (int e = threadIdx.x; e < (1 << LG); e += NT) stw[e] = st[(size_t)e << (log2S - LG)];
    // roots of the register DFTs: w_R^j from the table's quarter-length entries (uniform)
    constexpr int RB0 = ntt_rbits(LG, 0), RB1 = NR > 1 ? ntt_rbits(LG, 1) : 1, RB2 = NR > 2 ? ntt_rbits(LG, 2) : 1;
    auto small_roots = [&](uint32_t *w, int rb) {
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = j < (1 << rb) / 2 ? st[(size_t)j << (log2S - rb)] : 0u;
    };
    const int64_t *in = src.ptr ? src.ptr[v % vec_per_prime] : nullptr;
    auto load = [&](int n, int c) {
        const int64_t pos = base + (int64_t)c * g.col_stride + (int64_t)n * g.elem_stride;
        return in ? mont_from_i64(R, in[pos], P.r2, P.r3, P.neg2_64) : vec[pos];
    };
    // Output n of column c is multiplied by w_m^(n colid): a thread's outputs are an
    // arithmetic progression in n (frequencies f0 + k step), so two entries of the long
    // table, w^(f0 colid) and w^(step colid), give them all by one product each.  Exact
    // arithmetic: the same residues as one lookup per element.
    const int sh = log2T - g.log2m;
    uint32_t t_cur = 0, t_step = 0;
    auto store = [&](int f, int c, int k, uint32_t val) {
        if (g.twiddle) {
            if (k == 0) {
                constexpr int step = 1 << (LG - (NR == 1 ? RB0 : NR == 2 ? RB1 : RB2));
                const int64_t col = ((int64_t)blk << LC) + c;
                t_cur = tw[(size_t)((f * col) & (m - 1)) << sh];
                t_step = tw[(size_t)((step * col) & (m - 1)) << sh];
            } else {
                t_cur = R.mul(t_cur, t_step);
            }
            val = R.mul(val, t_cur);
        }
        if (g.scale) val = R.mul(val, P.minv[g.log2m]);
        vec[base + (int64_t)c * g.col_stride + (int64_t)f * g.elem_stride] = val;
    };
    uint32_t w[8];
    small_roots(w, RB0);
    if constexpr (NR > 1) __syncthreads();  // stw
    ntt_round<LG, LC, 0>(s, stw, R, w, load, store);
    if constexpr (NR > 1) {
        __syncthreads();
        if constexpr (RB1 != RB0) small_roots(w, RB1);
        ntt_round<LG, LC, 1>(s, stw, R, w, load, store);
    }
    if constexpr (NR > 2) {
        __syncthreads();
        if constexpr (RB2 != RB1) small_roots(w, RB2);
        ntt_round<LG, LC, 2>(s, stw, R, w, load, store);
    }
}

// Two-pass lengths: tiles of N2 = 2^S elements, columns of N1 = 2^(log2m - S) <= N2.
PassGeom column_pass(int log2m, int S, bool twiddle)
{
    PassGeom g{};
    g.log2m = log2m;
    g.log2L = log2m - S;
    g.log2C = S - g.log2L;
    g.elem_stride = (int64_t)1 << S;
    g.col_stride = 1;
    g.block_stride = (int64_t)1 << g.log2C;
    g.blocks = (1 << S) >> g.log2C;
    g.twiddle = twiddle;
    return g;
}

PassGeom row_pass(int log2m, int S, bool twiddle)
{
    PassGeom g{};
    g.log2m = log2m;
    g.log2L = S;
    g.log2C = 0;
    g.elem_stride = 1;
    g.col_stride = 0;
    g.block_stride = (int64_t)1 << S;
    g.blocks = 1 << (log2m - S);
    g.twiddle = twiddle;
    return g;
}

// Launch of one pass with the tile its geometry needs (single pass: the whole vector in
// one 4096-element tile; two-pass lengths: 2^S elements).
template <class F>
void with_tile(const PassGeom &g, bool single, F &&f)
{
    const int tile_bits = g.log2L + g.log2C;  // = S for both passes
    if (single || tile_bits == 12) f(std::integral_constant<int, kSingleTile>{});
    else if (tile_bits == 10) f(std::integral_constant<int, 1024>{});
    else f(std::integral_constant<int, 2048>{});
}

PassGeom single_pass(int log2m)
{
    PassGeom g{};
    g.log2m = log2m;
    g.log2L = log2m;
    g.log2C = 0;
    g.elem_stride = 1;
    g.block_stride = 0;
    g.blocks = 1;
    return g;
}

}  // namespace

int split_for(int device, int log2m)
{
    const int t = tune_split(device, log2m);
    return t && split_ok(log2m, t) ? t : default_split_bits(log2m);
}

cs_status fft_f64_forward(const int64_t *const *re, const int64_t *const *im, int n_vec, double2 *buf, int log2m,
                          int S, const TwiddleTables &tw, hipStream_t s)
{
    if (n_vec == 0) return CS_OK;
    F64Src first{re, im};
    F64Src self{nullptr, nullptr};
    auto pass = [&](const PassGeom &g, bool single, const F64Src &src) {
        with_tile(g, single, [&](auto tile) {
            constexpr int T = decltype(tile)::value;
            hipLaunchKernelGGL(k_fft_f64<T>, dim3(n_vec, g.blocks), dim3(T / 4), 0, s, src, buf, g, tw.full, tw.log2T,
                               tw.stage, tw.log2S);
        });
        return hipGetLastError();
    };
    if (log2m <= 12) {
        CSK_HIP(pass(single_pass(log2m), true, first));
        return CS_OK;
    }
    CSK_HIP(pass(column_pass(log2m, S, true), false, first));
    CSK_HIP(pass(row_pass(log2m, S, false), false, self));
    return CS_OK;
}

namespace {
// The column pass of the NTT reads its columns in runs of C 4-byte residues (8 bytes from
// the sketches): 32 columns per block up to length 2^8, 16 beyond (tiles of at most 2^14
// residues, 64 KB of LDS).  The decomposition, and with it the output order, is the
// same as with the fp64 FFT's narrower blocks.
constexpr int ntt_log2c(int lg) { return lg <= 8 ? 5 : 4; }
PassGeom widen_columns(PassGeom g)
{
    const int c = ntt_log2c(g.log2L);
    g.blocks = (g.blocks << g.log2C) >> c;
    g.log2C = c;
    g.block_stride = (int64_t)1 << c;
    return g;
}

template <int LG, bool ROW>
void ntt_launch(const PassGeom &g, const ModSrc &src, int n_vec, uint32_t *buf, int vec_per_prime,
                const PrimeDev *primes, const ModTables &roots, int inverse, hipStream_t s)
{
    constexpr int LC = ROW ? 0 : ntt_log2c(LG);
    hipLaunchKernelGGL((k_ntt<LG, LC>), dim3(n_vec, g.blocks), dim3(ntt_threads(LG, LC)), 0, s, src, buf, g,
                       vec_per_prime, primes, roots.full, roots.log2T, roots.stage, roots.log2S, inverse);
}

// Row (and single) passes have one column; two-pass rows are 2^10 to 2^12 long, the columns
// of lengths up to 2^21 at most 2^10.
hipError_t ntt_pass(const PassGeom &g, const ModSrc &src, int n_vec, uint32_t *buf, int vec_per_prime,
                    const PrimeDev *primes, const ModTables &roots, int inverse, hipStream_t s)
{
    auto go = [&](auto lg, auto row) {
        ntt_launch<decltype(lg)::value, decltype(row)::value>(g, src, n_vec, buf, vec_per_prime, primes, roots, inverse,
                                                              s);
    };
    auto pick = [&](auto row) {
        switch (g.log2L) {
#define CSK_NTT_CASE(LG) \
    case LG: go(std::integral_constant<int, LG>{}, row); break;
            CSK_NTT_CASE(1)
            CSK_NTT_CASE(2)
            CSK_NTT_CASE(3)
            CSK_NTT_CASE(4)
            CSK_NTT_CASE(5)
            CSK_NTT_CASE(6)
            CSK_NTT_CASE(7)
            CSK_NTT_CASE(8)
            CSK_NTT_CASE(9)
            CSK_NTT_CASE(10)
            default:
                if constexpr (decltype(row)::value) {
                    if (g.log2L == 11) go(std::integral_constant<int, 11>{}, row);
                    else if (g.log2L == 12) go(std::integral_constant<int, 12>{}, row);
                    else return hipErrorInvalidValue;
                } else {
                    return hipErrorInvalidValue;
                }
#undef CSK_NTT_CASE
        }
        return hipGetLastError();
    };
    return g.log2C == 0 ? pick(std::true_type{}) : pick(std::false_type{});
}
}  // namespace

cs_status ntt_forward(const int64_t *const *ptrs, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s)
{
    const int n_vec = vec_per_prime * n_primes;
    if (n_vec == 0) return CS_OK;
    ModSrc first{ptrs};
    ModSrc self{nullptr};
    const ModSrc &in = ptrs ? first : self;
    if (log2m <= 12) {
        CSK_HIP(ntt_pass(single_pass(log2m), in, n_vec, buf, vec_per_prime, primes, roots, 0, s));
        return CS_OK;
    }
    CSK_HIP(ntt_pass(widen_columns(column_pass(log2m, S, true)), in, n_vec, buf, vec_per_prime, primes,
                     roots, 0, s));
    CSK_HIP(ntt_pass(row_pass(log2m, S, false), self, n_vec, buf, vec_per_prime, primes, roots, 0, s));
    return CS_OK;
}

cs_status ntt_inverse(int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S, const PrimeDev *primes,
                      const ModTables &roots, hipStream_t s)
{
    const int n_vec = vec_per_prime * n_primes;
    if (n_vec == 0) return CS_OK;
    ModSrc self{nullptr};
    if (log2m <= 12) {
        PassGeom g = single_pass(log2m);
        g.scale = 1;
        CSK_HIP(ntt_pass(g, self, n_vec, buf, vec_per_prime, primes, roots, 1, s));
        return CS_OK;
    }
    CSK_HIP(ntt_pass(row_pass(log2m, S, true), self, n_vec, buf, vec_per_prime, primes, roots, 1, s));
    PassGeom g2 = widen_columns(column_pass(log2m, S, false));
    g2.scale = 1;
    CSK_HIP(ntt_pass(g2, self, n_vec, buf, vec_per_prime, primes, roots, 1, s));
    return CS_OK;
}

}  // namespace csk
