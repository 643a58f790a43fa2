// Transform launchers (fp64 FFT and NTT) and the per-prime constants they use.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "csk_internal.h"

namespace csk {

// Geometry of one transform pass: each block transforms 2^log2C interleaved transforms
// of length 2^log2L whose element n of column c sits at
// block_base + c * col_stride + n * elem_stride, block_base = blockIdx.x * block_stride.
struct PassGeom {
    int32_t log2m;
    int32_t log2L;
    int32_t log2C;
    int32_t blocks;
    int64_t elem_stride;
    int64_t col_stride;
    int64_t block_stride;
    int32_t twiddle;   // multiply output n of column c by w_m^(n * (blockIdx.x * C + c))
    int32_t scale;     // multiply by m^-1 (inverse NTT, last pass)
};

// Constants of one NTT prime, as the device reads them.
struct PrimeDev {
    uint32_t p;
    uint32_t pinv_neg;   // -p^-1 mod 2^32
    uint32_t r2;         // 2^64 mod p
    uint32_t r3;         // 2^96 mod p
    uint32_t neg2_64;    // Montgomery form of -2^64 mod p
    uint32_t one;        // Montgomery form of 1 (2^32 mod p)
    uint32_t minv[kMaxLog2N + 1];  // Montgomery form of 2^-L mod p
};

// Row length 2^S of the two-pass transforms (lengths above 4096), which is also their
// tile.  Default: the smallest S >= 10 that leaves the column pass at least 8
// interleaved columns (128 contiguous bytes of fp64 complex per row read): 1024 for
// 2^13..2^17, 2048 for 2^18..2^19, 4096 for 2^20..2^21.  The autotuner may pick another
// S with split_ok(); every transform of one estimate uses the same S for one length.
__host__ __device__ inline int default_split_bits(int log2m) { return (log2m + 4) / 2 > 10 ? (log2m + 4) / 2 : 10; }
// The split an estimate uses for length 2^log2m on `device` (tuned, else the default).
int split_for(int device, int log2m);

// Position of frequency f in the output of the forward transform of length 2^log2m
// with row length 2^S.
__host__ __device__ inline uint32_t freq_pos(uint32_t f, int log2m, int S)
{
    if (log2m <= 12) return f;
    const uint32_t n1 = 1u << (log2m - S);
    return ((f & (n1 - 1)) << S) | (f >> (log2m - S));
}
// Frequency held at position pos of the forward transform's output.
__host__ __device__ inline uint32_t pos_freq(uint32_t pos, int log2m, int S)
{
    if (log2m <= 12) return pos;
    return (pos >> S) | ((pos & ((1u << S) - 1)) << (log2m - S));
}

// A transform's root table (the powers of a primitive 2^log2T-th root) and the one its
// stages read: 2^12 entries, or the same table for shorter transforms.  A tile of length L
// takes every 2^(12 - log2 L)-th entry of it; from the table of a long transform it took
// entries a kilobyte apart, many times the tile's own bytes in cache lines.
constexpr int kStageLog2 = 12;
template <class T>
struct RootTables {
    const T *full;
    const T *stage;
    int log2T, log2S;
    // the fp64 column pass's twiddles in the order it uses them (column_twiddles; null for
    // lengths of one pass)
    const T *columns;
};
using TwiddleTables = RootTables<double2>;
using ModTables = RootTables<uint32_t>;
// Both tables of length 2^log2m on `device`, built on first use (full = null on failure);
// S is the row length's logarithm of the transforms that will use them.
TwiddleTables twiddle_tables(int device, int log2m, int S, hipStream_t s, cs_status *st);
ModTables mod_tables(int device, int log2m, hipStream_t s, cs_status *st);

// out[j] = tw[...], the m twiddles of the fp64 column pass at row length 2^S: a block's
// outputs in tile order, blocks one after another.
cs_status column_twiddles(double2 *out, const double2 *tw, int log2m, int S, hipStream_t s);

// Complex vectors re[v] + i im[v] (device pointer tables of int64 sketches; im[v] may be
// null).  Their first pass leaves the sketches' norm partials (sum of squares, sum of
// absolute values), fft_norm_blocks() pairs a sketch from pair re_norm[v] and im_norm[v] of
// `norms` on.
struct SketchVectors {
    const int64_t *const *re, *const *im;
    const int64_t *re_norm, *im_norm;
    double *norms;
};
int fft_norm_blocks(int log2m, int S);
// Most additions on a term's path to a norm, a wavefront's sum of the partials included.
int fft_norm_adds(int log2m, int S);

// Their forward fp64 FFTs into buf [n_vec][m].
cs_status fft_f64_forward(const SketchVectors &v, int n_vec, double2 *buf, int log2m, int S, const TwiddleTables &tw,
                          hipStream_t s);

// Where the first pass of a modular transform takes element `pos` of vector v = (prime, j)
// from: the sketch's int64 value or a residue, converted, padded or multiplied on the way
// instead of by passes of their own.
struct ModSrc {
    enum Mode : int32_t {
        kInPlace,    // the buffer itself
        kTable,      // sketch table[j]
        kPadSketch,  // sketch base + j m, zero beyond m; reversed (i -> (m - i) mod m) when asked
        kPadReg,     // the same of residue vector reg + v m
        kMul,        // the buffer's element times mul's at the same place
    } mode = kInPlace;
    const int64_t *const *table = nullptr;
    const int64_t *sketch = nullptr;
    const uint32_t *reg = nullptr;  // kPadReg, kMul
    uint32_t m = 0;
    int32_t reverse = 0;
    // kPadSketch, kPadReg: element i is the value (2^log2m - i) mod 2^log2m of the vector
    // repeated twice, zero beyond (its transform at f is the repetition's at -f)
    int32_t periodic = 0;
    static ModSrc from_table(const int64_t *const *t)
    {
        ModSrc s;
        s.mode = kTable;
        s.table = t;
        return s;
    }
    static ModSrc padded_sketch(const int64_t *p, uint32_t m, bool reverse)
    {
        ModSrc s;
        s.mode = kPadSketch;
        s.sketch = p;
        s.m = m;
        s.reverse = reverse;
        return s;
    }
    static ModSrc padded_reg(const uint32_t *p, uint32_t m, bool reverse)
    {
        ModSrc s;
        s.mode = kPadReg;
        s.reg = p;
        s.m = m;
        s.reverse = reverse;
        return s;
    }
    static ModSrc times(const uint32_t *p)
    {
        ModSrc s;
        s.mode = kMul;
        s.reg = p;
        return s;
    }
};
cs_status ntt_forward(const ModSrc &src, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s);
// The column pass alone (lengths above 4096): ntt_products takes the rows.
cs_status ntt_columns(const ModSrc &src, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s);

// d products of r factors, each summed over its frequencies: factor k of product t is vector
// vec[k] + t, at -f where conj has bit k.  Partial sums of product t go to out + t stride of
// each prime's plane: nb of them, the rest of the stride is set to zero.
struct ProductItem {
    int32_t r, nb, stride;
    uint32_t conj;
    int64_t out;
    int32_t vec[kMaxRel];
};
// Partial sums of one product: a workgroup's rows, up to four per lane of the wavefront that
// adds them (64 workgroups a product left a second round of them nearly empty).
inline int product_blocks(int log2m, int S) { return log2m <= 12 ? 1 : std::min(256, 1 << (log2m - S)); }
// Lengths up to 4096 are transformed from the sketches in `table`, longer ones from their
// column pass in buf [primes][vec_per_prime][2^log2m].  prefix: workgroups before each item
// (d nb of them an item), `blocks` in all.  scale: partial sums times 2^-log2m.
cs_status ntt_products(const int64_t *const *table, const uint32_t *buf, int vec_per_prime, int n_primes,
                       const ProductItem *items, const int64_t *prefix, int n_items, int64_t blocks, int log2m, int S,
                       const PrimeDev *primes, const ModTables &roots, uint32_t *partials, int64_t plane, bool scale,
                       hipStream_t s);

// Flattened launches: block b belongs to item i with prefix[i] <= b < prefix[i + 1].
__device__ __forceinline__ int find_item(const int64_t *__restrict__ prefix, int n, int64_t b)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

cs_status ntt_inverse(const ModSrc &src, int vec_per_prime, int n_primes, uint32_t *buf, int log2m, int S,
                      const PrimeDev *primes, const ModTables &roots, hipStream_t s);

}  // namespace csk
