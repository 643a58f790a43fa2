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
// Inside a pass, rounds of register DFTs exchange their elements through LDS; twiddles
// come from host-computed tables.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "csk_internal.h"
#include "csk_rings.h"
#include "csk_transform.h"

namespace csk {

namespace {

// LDS position of tile element i: one padding element after every 32, so that accesses at
// strides of powers of two spread over the banks.
__device__ __forceinline__ int lp(int i) { return i + (i >> 5); }
template <int TILE>
constexpr int lds_len() { return TILE + TILE / 32; }

// A thread holds 2^EB elements and takes up to EB stages between two trips through LDS: a
// transform of length 2^LG is a few rounds of decimation in frequency with radices
// 2^round_bits(LG, EB, round), each round's DFTs in registers.  Element s of the tile
// after a round is block b (the digits of the frequency found so far, first digit most
// significant) times the remaining length plus the index within it, so a round reads and
// writes the same places and the last one's outputs sit at digit-reversed frequencies.
constexpr int n_rounds(int lg, int eb) { return (lg + eb - 1) / eb; }
constexpr int round_bits(int lg, int eb, int round)
{
    return lg / n_rounds(lg, eb) + (round < lg % n_rounds(lg, eb) ? 1 : 0);
}
constexpr int bits_before(int lg, int eb, int round)
{
    int b = 0;
    for (int i = 0; i < round; ++i) b += round_bits(lg, eb, i);
    return b;
}
constexpr int pass_threads(int lg, int lc, int eb) { return (1 << (lg + lc)) >> eb < 64 ? 64 : (1 << (lg + lc)) >> eb; }

constexpr int brev_bits(int x, int bits)
{
    int r = 0;
    for (int i = 0; i < bits; ++i) r |= ((x >> i) & 1) << (bits - 1 - i);
    return r;
}

// One round of the tile's transforms (see above).  src(n, c, e) supplies the first round's
// inputs (e counts the thread's), dst(f, c, k, it, value) takes the last one's outputs (k counts a DFT's, whose
// frequencies f are an arithmetic progression, it the thread's DFTs); s is the tile in LDS, root(e) the power
// w_L^e, Dft the ring's register DFTs and the thread's index.
template <int LG, int LC, int EB, int ROUND, class Dft, class T, class Root, class Src, class Dst>
__device__ __forceinline__ void pass_round(T *s, const Dft &D, Root &&root, Src &&src, Dst &&dst)
{
    constexpr int NR = n_rounds(LG, EB), RB = round_bits(LG, EB, ROUND), N = 1 << RB;
    constexpr int done = bits_before(LG, EB, ROUND);
    constexpr int LJ = LG - done, LN = LJ - RB;  // log2 of the length before and after the round
    constexpr bool first = ROUND == 0, last = ROUND == NR - 1;
    constexpr int NT = pass_threads(LG, LC, EB);
    constexpr int groups = 1 << (LG + LC - RB);
#pragma unroll
    for (int g0 = 0; g0 < groups; g0 += NT) {
        const int g = g0 + D.tid;
        if (groups < NT && g >= groups) break;
        const int c = g & ((1 << LC) - 1), h = g >> LC;
        // middle rounds: h = block * 2^LN + index; last round: h counts the blocks by their
        // frequency, first digit fastest, so that neighbouring lanes store neighbours
        int blk = h >> LN, i = h & ((1 << LN) - 1);
        if (last && NR > 2) {
            blk = 0;
#pragma unroll
            for (int q = 0; q < NR - 1; ++q) {
                const int digit = (h >> bits_before(LG, EB, q)) & ((1 << round_bits(LG, EB, q)) - 1);
                blk = (blk << round_bits(LG, EB, q)) | digit;
            }
        }
        const int at = (((blk << LJ) + i) << LC) + c;  // element k at at + k 2^(LN + LC)
        T x[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if constexpr (first) x[k] = src(i + (k << LN), c, (g0 / NT) * N + k);
            else x[k] = s[lp(at + (k << (LN + LC)))];
        }
        D.template dft<RB, !last>(x);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const T v = x[brev_bits(k, RB)];  // frequency digit k
            if constexpr (last) dst(h + (k << done), c, k, g0 / NT, v);
            else s[lp(at + (k << (LN + LC)))] = k == 0 ? D.settle(v) : D.mul(v, root((i * k) << (LG - LJ)));
        }
    }
}

// Every round of a pass from ROUND on.
template <int LG, int LC, int EB, int ROUND = 0, class Dft, class T, class Root, class Src, class Dst>
__device__ __forceinline__ void pass_rounds(T *s, Dft &D, Root &&root, Src &&src, Dst &&dst)
{
    if constexpr (ROUND > 0) __syncthreads();
    D.template load_roots<round_bits(LG, EB, ROUND)>();
    pass_round<LG, LC, EB, ROUND>(s, D, root, src, dst);
    if constexpr (ROUND + 1 < n_rounds(LG, EB)) pass_rounds<LG, LC, EB, ROUND + 1>(s, D, root, src, dst);
}

// ---------------------------------------------------------------- fp64 complex FFT pass

// Source of a pass: either the complex work buffer, or (first pass) the int64 sketches
// of the (relation, repetition) pair packed into one complex vector: re + i * im.
struct F64Src {
    const int64_t *const *re;  // [n_vec] sketch loaded as the real part (null: in place)
    const int64_t *const *im;  // [n_vec] sketch loaded as the imaginary part (entry null: 0)
    // first pass: where the norm partials (sum of squares, of absolute values) of either
    // sketch go, one pair per block of the pass
    const int64_t *re_norm, *im_norm;
    double *norms;
};

// v[0..N) summed over the wavefront (lane 0 holds them).
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N])
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += __shfl_down(v[i], o, 64);
}

// Sums of squares and absolute values of the real and the imaginary parts.
template <int E>
__device__ __forceinline__ void add_norms(const double2 (&x)[E], double (&n)[4])
{
    double q[E][4];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        q[e][0] = x[e].x * x[e].x;
        q[e][1] = fabs(x[e].x);
        q[e][2] = x[e].y * x[e].y;
        q[e][3] = fabs(x[e].y);
    }
#pragma unroll
    for (int h = E / 2; h > 0; h >>= 1)  // a tree: log2 E additions deep
#pragma unroll
        for (int e = 0; e < h; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) q[e][i] += q[e + h][i];
#pragma unroll
    for (int i = 0; i < 4; ++i) n[i] = q[0][i];
}

// Register DFTs of complex doubles, decimation in frequency: x[k] in, frequency
// brev_bits(k) in x[k] out.  Along any path of a round of RB stages there are at most RB
// complex products, the round's twiddle among them (the last stage's is by 1), as in RB
// radix-2 stages: the error bound of the estimate counts one per stage.
struct DftC {
    const double2 *stage;  // w_(2^log2S) powers
    int log2S;
    int tid;
    double2 w[8];
    RingC R;
    template <int RB>
    __device__ __forceinline__ void load_roots()
    {
#pragma unroll
        for (int j = 0; j < (1 << RB) / 2; ++j) w[j] = stage[(size_t)j << (log2S - RB)];
    }
    __device__ __forceinline__ double2 settle(double2 v) const { return v; }
    __device__ __forceinline__ double2 mul(double2 v, double2 t) const { return R.mul(v, t); }
    template <int RB, bool LAZY>
    __device__ __forceinline__ void dft(double2 (&x)[1 << RB]) const
    {
        constexpr int N = 1 << RB;
#pragma unroll
        for (int st = 0; st < RB; ++st) {
            const int half = N >> (st + 1);
#pragma unroll
            for (int b = 0; b < N; b += 2 * half)
#pragma unroll
                for (int k = 0; k < half; ++k) {
                    const double2 a = x[b + k], c = x[b + k + half];
                    x[b + k] = R.add(a, c);
                    const double2 v = R.sub(a, c);
                    // w_4 = -i exactly
                    x[b + k + half] = k == 0          ? v
                                      : 2 * k == half ? make_double2(v.y, -v.x)
                                                      : R.mul(v, w[k << st]);
                }
        }
    }
};

// One pass: a block transforms 2^LC interleaved columns of length 2^LG.  Bound by memory
// (16 bytes read and written per element: the row pass at 5 TB/s, the column pass, whose
// sources are runs of 128 bytes, at 3.6; 38 vectors of 2^18 take 64 and 88 us, 106 each
// with two stages per trip through LDS).  FIRST: from the sketches, whose norms are summed on
// the way (a pass of their own over the int64 counters took 81 us of that estimate).  The stage roots are read through the cache: in LDS
// they would take as much of it as the tile and halve the blocks per CU.
template <int LG, int LC, int EB, bool FIRST>
__global__ __launch_bounds__(pass_threads(LG, LC, EB)) void k_fft_f64(F64Src src, double2 *buf, PassGeom g,
                                                                  const double2 *__restrict__ columns,
                                                                  const double2 *__restrict__ stage, int log2S)
{
    __shared__ double2 s[n_rounds(LG, EB) > 1 ? lds_len<(1 << (LG + LC))>() : 1];
    const int v = blockIdx.x;
    const int blk = blockIdx.y;
    const int64_t m = (int64_t)1 << g.log2m;
    const int64_t base = (int64_t)blk * g.block_stride;
    double2 *vec = buf + (size_t)v * m;
    constexpr int E = 1 << EB;
    double2 x[FIRST ? E : 1];
    if constexpr (FIRST) {
        // this thread's inputs, and their norms
        constexpr int RB = round_bits(LG, EB, 0), NT = pass_threads(LG, LC, EB), groups = 1 << (LG + LC - RB);
        const int64_t *re = src.re[v], *im = src.im[v];
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = make_double2(0.0, 0.0);
#pragma unroll
        for (int g0 = 0; g0 < groups; g0 += NT) {
            const int h = g0 + (int)threadIdx.x;
            if (groups < NT && h >= groups) break;
            const int64_t at = base + (int64_t)(h & ((1 << LC) - 1)) * g.col_stride + (int64_t)(h >> LC) * g.elem_stride;
#pragma unroll
            for (int k = 0; k < (1 << RB); ++k) {
                const int64_t pos = at + ((int64_t)k << (LG - RB)) * g.elem_stride;
                x[(g0 / NT) * (1 << RB) + k] = make_double2((double)re[pos], im ? (double)im[pos] : 0.0);
            }
        }
        double nr[4];
        add_norms<E>(x, nr);
        wave_sums(nr);
        __shared__ double s_nr[NT / 64][4];
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s_nr[threadIdx.x >> 6][i] = nr[i];
        }
        __syncthreads();
        if (threadIdx.x < 4 && (threadIdx.x < 2 || im)) {
            double a = 0.0;
            for (int w = 0; w < NT / 64; ++w) a += s_nr[w][threadIdx.x];
            src.norms[((threadIdx.x < 2 ? src.re_norm : src.im_norm)[v] + blk) * 2 + (threadIdx.x & 1)] = a;
        }
    }
    auto load = [&](int n, int c, int e) {
        if constexpr (FIRST) return x[e];
        else return vec[base + (int64_t)c * g.col_stride + (int64_t)n * g.elem_stride];
    };
    DftC D{stage, log2S, (int)threadIdx.x};
    auto store = [&](int f, int c, int k, int it, double2 val) {
        // w_m^(f column), from the table in tile order: looked up in the table of powers, a
        // tile's 2^11 twiddles lie in as many cache lines
        if (g.twiddle) val = D.R.mul(val, columns[((size_t)blk << (LG + LC)) + ((size_t)f << LC) + c]);
        vec[base + (int64_t)c * g.col_stride + (int64_t)f * g.elem_stride] = val;
    };
    auto root = [&](int e) { return stage[(size_t)e << (log2S - LG)]; };
    pass_rounds<LG, LC, EB>(s, D, root, load, store);
}

// ---------------------------------------------------------------- NTT pass

// Register DFTs of residues.  Inputs below p; the last stage's results are below 2p when
// LAZY (a twiddle multiplies them next), else below p.
struct DftM {
    RingM R;
    const uint32_t *stage;  // w_(2^log2S) powers
    int log2S;
    int tid;
    uint32_t w[8];
    template <int RB>
    __device__ __forceinline__ void load_roots()
    {
#pragma unroll
        for (int j = 0; j < (1 << RB) / 2; ++j) w[j] = stage[(size_t)j << (log2S - RB)];
    }
    __device__ __forceinline__ uint32_t settle(uint32_t v) const { return min(v, v - R.p); }
    __device__ __forceinline__ uint32_t mul(uint32_t v, uint32_t t) const { return R.mul(v, t); }
    template <int RB, bool LAZY>
    __device__ __forceinline__ void dft(uint32_t (&x)[1 << RB]) const
    {
        constexpr int N = 1 << RB;
#pragma unroll
        for (int st = 0; st < RB; ++st) {
            const int half = N >> (st + 1);
            const bool lazy = LAZY && st == RB - 1;
#pragma unroll
            for (int b = 0; b < N; b += 2 * half)
#pragma unroll
                for (int k = 0; k < half; ++k) {
                    const uint32_t a = x[b + k], c = x[b + k + half];
                    const uint32_t u = a + c, v = a - c + R.p;  // both below 2p
                    x[b + k] = lazy ? u : settle(u);
                    // w_(2 half)^k = w_N^(k 2^st)
                    x[b + k + half] = k == 0 ? (lazy ? v : settle(v)) : R.mul(v, w[k << st]);
                }
        }
    }
};

// One pass: a block transforms 2^LC interleaved columns of length 2^LG.  Bound by the vector
// unit and memory about equally.  Two stages per trip through LDS with four elements per
// thread cost as much address arithmetic, LDS instructions and barriers as butterflies:
// 15 vectors of 2^21 at 3 primes took 213 us (columns) and 144 us (rows), 97 and 103 us in
// registers.
// MODE: the source's where it is kInPlace or kTable, so that their loads carry no branch (one
// per element cost the 5-chain's estimate 3%); kGeneric for the others.
constexpr int kGeneric = -1;
template <int LG, int LC, int EB, int MODE>
__global__ __launch_bounds__(pass_threads(LG, LC, EB)) void k_ntt(ModSrc src, uint32_t *buf, PassGeom g, int vec_per_prime, int n_primes,
                                                              const PrimeDev *__restrict__ primes,
                                                              const uint32_t *__restrict__ roots, int log2T,
                                                              const uint32_t *__restrict__ stage, int log2S, int inverse)
{
    constexpr int TILE = 1 << (LG + LC), NT = pass_threads(LG, LC, EB), NR = n_rounds(LG, EB);
    __shared__ uint32_t s[NR > 1 ? lds_len<TILE>() : 1];
    __shared__ uint32_t stw[NR > 1 ? 1 << LG : 1];  // w_L^e
    // Workgroups go to the 8 XCDs round-robin.  When the sketches are read, the primes of
    // one tile follow each other on one XCD, whose L2 then fetches its int64 values once.
    // Tiles of fewer than 32 columns write runs shorter than a cache line: an XCD takes
    // neighbouring ones, so that one L2 gathers a line (16 columns, 10 vectors of 2^21: 68 ->
    // 65 us; from 32 on neighbours are spread, 451 us against 456 for the 5-chain's estimate).
    int pi, j, blk;
    {
        const uint32_t tiles = (uint32_t)vec_per_prime * g.blocks, id = blockIdx.x;
        uint32_t tile;
        if ((src.mode == ModSrc::kTable || src.mode == ModSrc::kPadSketch) && (tiles & 7) == 0) {
            const uint32_t w = id >> 3, K = n_primes;
            pi = (int)(w % K);
            tile = LC < 5 ? (id & 7) * (tiles >> 3) + w / K : (w / K) * 8 + (id & 7);
        } else {
            pi = (int)(id / tiles);
            tile = id % tiles;
        }
        j = (int)(tile / g.blocks);
        blk = (int)(tile % g.blocks);
    }
    const int v = pi * vec_per_prime + j;
    const PrimeDev &P = primes[pi];  // by reference: a copy with minv[] indexed would live in scratch
    const RingM R{P.p, P.pinv_neg};
    const uint32_t *tw = roots + ((size_t)(2 * pi + inverse) << log2T);
    DftM D{R, stage + ((size_t)(2 * pi + inverse) << log2S), log2S, (int)threadIdx.x};
    const int64_t m = (int64_t)1 << g.log2m;
    const int64_t base = (int64_t)blk * g.block_stride;
    uint32_t *vec = buf + (size_t)v * m;
    const int64_t *in = src.mode == ModSrc::kTable ? src.table[j] : src.sketch + (size_t)j * src.m;
    const uint32_t *reg = src.reg + (size_t)v * (src.mode == ModSrc::kMul ? m : (int64_t)src.m);
    auto load = [&](int n, int c, int) -> uint32_t {
        const int64_t pos = base + (int64_t)c * g.col_stride + (int64_t)n * g.elem_stride;
        if constexpr (MODE == ModSrc::kInPlace) return vec[pos];
        if constexpr (MODE == ModSrc::kTable) return mont_from_i64(R, in[pos], P.r2, P.r3, P.neg2_64);
        if (src.periodic) {
            const int64_t q = (m - pos) & (m - 1);
            if (q >= 2 * (int64_t)src.m - 1) return 0u;
            const int64_t at = q < src.m ? q : q - src.m;
            return src.mode == ModSrc::kPadReg ? reg[at] : mont_from_i64(R, in[at], P.r2, P.r3, P.neg2_64);
        }
        const bool pad = src.mode == ModSrc::kPadSketch || src.mode == ModSrc::kPadReg;
        if (pad && pos >= src.m) return 0u;
        const int64_t at = pad && src.reverse && pos > 0 ? src.m - pos : pos;
        switch (src.mode) {
            case ModSrc::kInPlace: return vec[pos];
            case ModSrc::kMul: return R.mul(vec[pos], reg[pos]);
            case ModSrc::kPadReg: return reg[at];
            default: return mont_from_i64(R, in[at], P.r2, P.r3, P.neg2_64);
        }
    };
    // Output n of column c is multiplied by w_m^(n colid): a thread's outputs are an
    // arithmetic progression in n, so two entries of the long table, w^(f0 colid) and
    // w^(step colid), give them all by one product each.  Exact arithmetic: the same
    // residues as one lookup per element.
    const int sh = log2T - g.log2m;
    uint32_t t_cur = 0, t_step = 0;
    auto store = [&](int f, int c, int k, int it, uint32_t val) {
        if (g.twiddle) {
            if (k == 0) {
                constexpr int step = 1 << (LG - round_bits(LG, EB, NR - 1));
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
    if constexpr (NR > 1) {
        for (int e = threadIdx.x; e < (1 << LG); e += NT) stw[e] = D.stage[(size_t)e << (log2S - LG)];
        __syncthreads();
    }
    pass_rounds<LG, LC, EB>(s, D, [&](int e) { return stw[e]; }, load, store);
}

// The last pass of the factors' transforms and the sum over the frequencies of their product
// (ProductItem): a workgroup transforms its rows of one factor after another and multiplies
// in registers, so the spectra are never written.  Factor k conjugated is its spectrum at
// -f: row r of it comes from row N1 - r read backwards, whose output N2 - 1 - f2 a factor
// w_N2^n on input n moves to f2 (row 0: from itself, without it).  MODE kTable: lengths of
// one pass, straight from the sketches.  Bound by memory (4 bytes read per element) and the
// vector unit.
template <int LG, int EB, int MODE>
__global__ __launch_bounds__(pass_threads(LG, 0, EB)) void k_ntt_product(
    const int64_t *const *__restrict__ table, const uint32_t *__restrict__ buf, int log2m, int vec_per_prime,
    const ProductItem *__restrict__ items, const int64_t *__restrict__ prefix, int n_items,
    const PrimeDev *__restrict__ primes, const uint32_t *__restrict__ stage, int log2S, uint32_t *partials,
    int64_t plane, int scale)
{
    constexpr int L = 1 << LG, NT = pass_threads(LG, 0, EB), NR = n_rounds(LG, EB);
    constexpr int N = 1 << round_bits(LG, EB, NR - 1);  // outputs of a DFT of the last round
    __shared__ uint32_t s[NR > 1 ? lds_len<L>() : 1];
    __shared__ uint32_t stw[L];  // w_L^e
    __shared__ uint32_t s_sum[NT / 64];
    const int pi = blockIdx.y;
    const int item = find_item(prefix, n_items, blockIdx.x);
    const ProductItem &I = items[item];
    const int within = (int)(blockIdx.x - prefix[item]), t = within / I.nb, blk = within - t * I.nb;
    const PrimeDev &P = primes[pi];
    const RingM R{P.p, P.pinv_neg};
    DftM D{R, stage + ((size_t)(2 * pi) << log2S), log2S, (int)threadIdx.x};
    for (int e = threadIdx.x; e < L; e += NT) stw[e] = D.stage[(size_t)e << (log2S - LG)];
    __syncthreads();
    auto root = [&](int e) { return stw[e]; };
    const int rows = 1 << (log2m - LG), per = rows / I.nb;
    // this thread's first-round inputs of factor k of a row; the next factor's are on their
    // way while one is transformed
    using In = std::conditional_t<MODE == ModSrc::kTable, int64_t, uint32_t>;
    auto fetch = [&](int row, int k, In (&x)[1 << EB]) {
        constexpr int RB0 = round_bits(LG, EB, 0), LN = LG - RB0;
        const int back = (int)((I.conj >> k) & 1u), flip = -back;
        const int64_t v = I.vec[k] + t;
        const In *in;
        if constexpr (MODE == ModSrc::kTable) in = table[v];
        else in = buf + (((size_t)pi * vec_per_prime + v) << log2m) + ((size_t)(back && row ? rows - row : row) << LG);
#pragma unroll
        for (int g0 = 0; g0 < (1 << LN); g0 += NT) {
            const int h = g0 + (int)threadIdx.x;
            if ((1 << LN) < NT && h >= (1 << LN)) break;
#pragma unroll
            for (int e = 0; e < (1 << RB0); ++e)
                x[(g0 / NT) * (1 << RB0) + e] = in[(((h + (e << LN)) ^ flip) + back) & (L - 1)];
        }
    };
    uint32_t acc = 0;
    In cur[1 << EB];
    fetch(blk * per, 0, cur);
    for (int row = blk * per; row < (blk + 1) * per; ++row) {
        uint32_t prod[1 << EB];
#pragma unroll
        for (int e = 0; e < (1 << EB); ++e) prod[e] = 0u;  // a lane without outputs adds nothing
        for (int k = 0; k < I.r; ++k) {
            In next[1 << EB];
            const bool last = k + 1 == I.r && row + 1 == (blk + 1) * per;  // fetches itself again
            fetch(k + 1 == I.r && !last ? row + 1 : row, last ? k : k + 1 == I.r ? 0 : k + 1, next);
            if (k || row > blk * per) __syncthreads();  // the tile's readers are done
            const bool twist = MODE != ModSrc::kTable && row && ((I.conj >> k) & 1u);
            {
                int id = threadIdx.x;  // opaque: addresses are not kept in registers between factors
                asm volatile("" : "+v"(id));
                D.tid = id;
            }
            auto value = [&](int e) -> uint32_t {
                if constexpr (MODE == ModSrc::kTable) return mont_from_i64(R, cur[e], P.r2, P.r3, P.neg2_64);
                else return cur[e];
            };
            auto store = [&](int, int, int kk, int it, uint32_t val) {
                uint32_t &x = prod[it * N + kk];
                x = k ? R.mul(x, val) : val;
            };
            if (twist) pass_rounds<LG, 0, EB>(s, D, root, [&](int n, int, int e) { return R.mul(value(e), stw[n]); }, store);
            else pass_rounds<LG, 0, EB>(s, D, root, [&](int, int, int e) { return value(e); }, store);
#pragma unroll
            for (int e = 0; e < (1 << EB); ++e) cur[e] = next[e];
        }
#pragma unroll
        for (int e = 0; e < (1 << EB); ++e) acc = R.add(acc, prod[e]);
    }
    for (int o = 32; o > 0; o >>= 1) acc = R.add(acc, __shfl_down(acc, o, 64));
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NT / 64; ++w) acc = R.add(acc, s_sum[w]);
        if (scale) acc = R.mul(acc, P.minv[log2m]);
        uint32_t *o = partials + (size_t)pi * plane + I.out + (int64_t)t * I.stride;
        o[blk] = acc;
        if (blk == 0)
            for (int b = I.nb; b < I.stride; ++b) o[b] = 0u;
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

namespace {
// Columns per block: the NTT reads runs of 4-byte residues (8 bytes from the sketches), 32
// columns up to length 2^8 and 16 beyond (tiles of at most 2^14 residues, 64 KB of LDS);
// the FFT runs of 16-byte elements, 16 columns down to 4 (tiles of 2^11 or 2^12, at most
// 66 KB).  The decomposition, and with it the output order, is the same for both.
constexpr int ntt_log2c(int lg) { return lg <= 8 ? 5 : 4; }
constexpr int fft_log2c(int lg) { return lg <= 7 ? 4 : lg <= 9 ? 3 : 2; }

// log2 of the elements per thread, measured (microseconds; 38 complex vectors, 76 x 3
// residue vectors):                    2^18          2^16 (15, 30)   2^10 (2, 4 x 3)
//   fft columns  4 / 8 / 16            87 / 102 / 148   9 / 12 / 17
//   fft rows                           74 / 64 / 59     9.8 / 8.3 / 8.8   4.5 / 5.3 / 8.2
//   ntt columns                        273 / 200 / 175  21 / 19.5 / 19.2
//   ntt rows                           193 / 136 / 153  19.4 / 19 / 22    4.5 / 5.8 / 8.9
// Single passes up to 2^10 run on few workgroups, where a thread's chain counts, and the
// int64 sources of the fp64 columns want the loads of many wavefronts.
constexpr int fft_elems(int lg, int lc, bool single) { return lc > 0 || (single && lg <= 10) ? 2 : 3; }
constexpr int ntt_elems(int lg, int lc, bool single) { return lc > 0 && lg >= 7 ? 4 : single && lg <= 10 ? 2 : 3; }
PassGeom with_columns(PassGeom g, int log2c)
{
    g.blocks = (g.blocks << g.log2C) >> log2c;
    g.log2C = log2c;
    g.block_stride = (int64_t)1 << log2c;
    return g;
}

// f(log2L, row, single) as integral constants.  Row and single passes have one column; two-pass
// rows are 2^10 to 2^12 long, the columns of lengths up to 2^21 at most 2^10.
template <class F>
hipError_t with_length(const PassGeom &g, F &&f)
{
    using T_ = std::true_type;
    using F_ = std::false_type;
    if (g.log2C > 0) {
        switch (g.log2L) {
#define CSK_LENGTH(LG, ROW, SINGLE) \
    case LG: f(std::integral_constant<int, LG>{}, ROW{}, SINGLE{}); break;
            CSK_LENGTH(1, F_, F_)
            CSK_LENGTH(2, F_, F_)
            CSK_LENGTH(3, F_, F_)
            CSK_LENGTH(4, F_, F_)
            CSK_LENGTH(5, F_, F_)
            CSK_LENGTH(6, F_, F_)
            CSK_LENGTH(7, F_, F_)
            CSK_LENGTH(8, F_, F_)
            CSK_LENGTH(9, F_, F_)
            CSK_LENGTH(10, F_, F_)
            default: return hipErrorInvalidValue;
        }
    } else if (g.blocks == 1) {
        switch (g.log2L) {
            CSK_LENGTH(1, T_, T_)
            CSK_LENGTH(2, T_, T_)
            CSK_LENGTH(3, T_, T_)
            CSK_LENGTH(4, T_, T_)
            CSK_LENGTH(5, T_, T_)
            CSK_LENGTH(6, T_, T_)
            CSK_LENGTH(7, T_, T_)
            CSK_LENGTH(8, T_, T_)
            CSK_LENGTH(9, T_, T_)
            CSK_LENGTH(10, T_, T_)
            CSK_LENGTH(11, T_, T_)
            CSK_LENGTH(12, T_, T_)
            default: return hipErrorInvalidValue;
        }
    } else {
        switch (g.log2L) {
            CSK_LENGTH(10, T_, F_)
            CSK_LENGTH(11, T_, F_)
            CSK_LENGTH(12, T_, F_)
            default: return hipErrorInvalidValue;
        }
    }
#undef CSK_LENGTH
    return hipGetLastError();
}

hipError_t fft_pass(const PassGeom &g, const F64Src &src, int n_vec, double2 *buf, const TwiddleTables &tw,
                    hipStream_t s)
{
    return with_length(g, [&](auto lg, auto row, auto single) {
        constexpr int LG = decltype(lg)::value, LC = decltype(row)::value ? 0 : fft_log2c(LG);
        constexpr int EB = fft_elems(LG, LC, decltype(single)::value);
        auto go = [&](auto first) {
            hipLaunchKernelGGL((k_fft_f64<LG, LC, EB, decltype(first)::value>), dim3(n_vec, g.blocks),
                               dim3(pass_threads(LG, LC, EB)), 0, s, src, buf, g, tw.columns, tw.stage, tw.log2S);
        };
        // the first pass is the column one, or the only one
        if constexpr (LC > 0 || decltype(single)::value) go(std::true_type{});
        else go(std::false_type{});
    });
}

__global__ void k_column_twiddles(double2 *out, const double2 *__restrict__ tw, int log2m, int log2L, int log2C)
{
    const uint32_t m = 1u << log2m;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x) {
        const uint32_t c = j & ((1u << log2C) - 1), f = (j >> log2C) & ((1u << log2L) - 1);
        const uint32_t col = ((j >> (log2C + log2L)) << log2C) + c;
        out[j] = tw[(uint32_t)(((uint64_t)f * col) & (m - 1))];
    }
}

hipError_t ntt_pass(const PassGeom &g, const ModSrc &src, int n_vec, uint32_t *buf, int vec_per_prime,
                    const PrimeDev *primes, const ModTables &roots, int inverse, hipStream_t s)
{
    return with_length(g, [&](auto lg, auto row, auto single) {
        constexpr int LG = decltype(lg)::value, LC = decltype(row)::value ? 0 : ntt_log2c(LG);
        constexpr int EB = ntt_elems(LG, LC, decltype(single)::value);
        auto go = [&](auto mode) {
            hipLaunchKernelGGL((k_ntt<LG, LC, EB, decltype(mode)::value>), dim3((unsigned)n_vec * g.blocks),
                               dim3(pass_threads(LG, LC, EB)), 0, s, src, buf, g, vec_per_prime, n_vec / vec_per_prime,
                               primes, roots.full, roots.log2T, roots.stage, roots.log2S, inverse);
        };
        if (src.mode == ModSrc::kInPlace) go(std::integral_constant<int, ModSrc::kInPlace>{});
        else if (src.mode == ModSrc::kTable) go(std::integral_constant<int, ModSrc::kTable>{});
        else go(std::integral_constant<int, kGeneric>{});
    });
}
}  // namespace

cs_status column_twiddles(double2 *out, const double2 *tw, int log2m, int S, hipStream_t s)
{
    hipLaunchKernelGGL(k_column_twiddles, dim3(1024), dim3(256), 0, s, out, tw, log2m, log2m - S, fft_log2c(log2m - S));
    CSK_HIP(hipGetLastError());
    return CS_OK;
}

int fft_norm_blocks(int log2m, int S) { return log2m <= 12 ? 1 : (1 << S) >> fft_log2c(log2m - S); }

int fft_norm_adds(int log2m, int S)
{
    if (log2m <= 12) {
        const int EB = fft_elems(log2m, 0, true);
        return EB + 6 + pass_threads(log2m, 0, EB) / 64;
    }
    const int lg = log2m - S, lc = fft_log2c(lg), EB = fft_elems(lg, lc, false);
    return EB + 6 + pass_threads(lg, lc, EB) / 64 + (fft_norm_blocks(log2m, S) + 63) / 64 + 6;
}

cs_status fft_f64_forward(const SketchVectors &v, int n_vec, double2 *buf, int log2m, int S, const TwiddleTables &tw,
                          hipStream_t s)
{
    if (n_vec == 0) return CS_OK;
    const F64Src first{v.re, v.im, v.re_norm, v.im_norm, v.norms};
    if (log2m <= 12) {
        CSK_HIP(fft_pass(single_pass(log2m), first, n_vec, buf, tw, s));
        return CS_OK;
    }
    CSK_HIP(fft_pass(with_columns(column_pass(log2m, S, true), fft_log2c(log2m - S)), first, n_vec, buf, tw, s));
    CSK_HIP(fft_pass(row_pass(log2m, S, false), F64Src{}, n_vec, buf, tw, s));
    return CS_OK;
}

cs_status ntt_forward(const ModSrc &src, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s)
{
    const int n_vec = vec_per_prime * n_primes;
    if (n_vec == 0) return CS_OK;
    if (log2m <= 12) {
        CSK_HIP(ntt_pass(single_pass(log2m), src, n_vec, buf, vec_per_prime, primes, roots, 0, s));
        return CS_OK;
    }
    CSK_HIP(ntt_pass(with_columns(column_pass(log2m, S, true), ntt_log2c(log2m - S)), src, n_vec, buf, vec_per_prime,
                     primes, roots, 0, s));
    CSK_HIP(ntt_pass(row_pass(log2m, S, false), ModSrc{}, n_vec, buf, vec_per_prime, primes, roots, 0, s));
    return CS_OK;
}

cs_status ntt_columns(const ModSrc &src, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s)
{
    CSK_HIP(ntt_pass(with_columns(column_pass(log2m, S, true), ntt_log2c(log2m - S)), src, vec_per_prime * n_primes, buf,
                     vec_per_prime, primes, roots, 0, s));
    return CS_OK;
}

cs_status ntt_products(const int64_t *const *table, const uint32_t *buf, int vec_per_prime, int n_primes,
                       const ProductItem *items, const int64_t *prefix, int n_items, int64_t blocks, int log2m, int S,
                       const PrimeDev *primes, const ModTables &roots, uint32_t *partials, int64_t plane, bool scale,
                       hipStream_t s)
{
    const bool single = log2m <= 12;
    CSK_HIP(with_length(single ? single_pass(log2m) : row_pass(log2m, S, false), [&](auto lg, auto row, auto sgl) {
        constexpr int LG = decltype(lg)::value;
        constexpr bool kSingle = decltype(sgl)::value;
        if constexpr (decltype(row)::value) {
            constexpr int EB = ntt_elems(LG, 0, kSingle), MODE = kSingle ? ModSrc::kTable : ModSrc::kInPlace;
            hipLaunchKernelGGL((k_ntt_product<LG, EB, MODE>), dim3((unsigned)blocks, n_primes),
                               dim3(pass_threads(LG, 0, EB)), 0, s, table, buf, log2m, vec_per_prime, items, prefix,
                               n_items, primes, roots.stage, roots.log2S, partials, plane, scale ? 1 : 0);
        }
    }));
    return CS_OK;
}

cs_status ntt_inverse(const ModSrc &src, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s)
{
    const int n_vec = vec_per_prime * n_primes;
    if (n_vec == 0) return CS_OK;
    if (log2m <= 12) {
        PassGeom g = single_pass(log2m);
        g.scale = 1;
        CSK_HIP(ntt_pass(g, src, n_vec, buf, vec_per_prime, primes, roots, 1, s));
        return CS_OK;
    }
    CSK_HIP(ntt_pass(row_pass(log2m, S, true), src, n_vec, buf, vec_per_prime, primes, roots, 1, s));
    PassGeom g2 = with_columns(column_pass(log2m, S, false), ntt_log2c(log2m - S));
    g2.scale = 1;
    CSK_HIP(ntt_pass(g2, ModSrc{}, n_vec, buf, vec_per_prime, primes, roots, 1, s));
    return CS_OK;
}

}  // namespace csk
