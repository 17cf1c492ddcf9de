// Scaling and residue split: the two HBM-bound passes over A and B that
// precede the INT8 products (Section III-B; Algorithm 1 Steps III, IV, V-i/ii).
//
// Operands are handled as "rows": the rows of op(A) and the columns of op(B),
// each a vector of k complex numbers (rows i and i+m of A-hat share one
// exponent, Section III-B).  Two memory orders occur: rows whose k elements
// are contiguous (contig_h) and rows that are contiguous with each other
// (consecutive rows adjacent, stride_r == 1).  Every kernel has a variant for
// each so that global loads stay coalesced.
#include <algorithm>

#include "internal.h"

namespace ozc {
namespace {

constexpr uint64_t kAbsMask = 0x7fffffffffffffffull;
constexpr uint64_t kInfBits = 0x7ff0000000000000ull;

typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec2 __attribute__((ext_vector_type(2)));

// One element of kind EK (ElemKind) at index idx; real elements have im = 0.
template <int EK>
__device__ __forceinline__ void load_elem(const void *base, int64_t idx, double &re, double &im) {
    if constexpr (EK == kElemC) {
        const fvec2 v = global_ptr(reinterpret_cast<const fvec2 *>(base))[idx];
        re = (double)v.x;
        im = (double)v.y;
    } else if constexpr (EK == kElemZ) {
        const dvec2 v = global_ptr(reinterpret_cast<const dvec2 *>(base))[idx];
        re = v.x;
        im = v.y;
    } else if constexpr (EK == kElemD) {
        re = global_ptr(reinterpret_cast<const double *>(base))[idx];
        im = 0.0;
    } else {
        re = (double)global_ptr(reinterpret_cast<const float *>(base))[idx];
        im = 0.0;
    }
}

__device__ __forceinline__ uint64_t abs_bits(double x) {
    return (uint64_t)__double_as_longlong(x) & kAbsMask;
}

// floor(log2 v) for the positive finite double whose bit pattern is `bits`.
__device__ __forceinline__ int ilogb_bits(uint64_t bits) {
    int ef = (int)(bits >> 52);
    if (ef == 0) return -1074 + 63 - __clzll((long long)bits);
    return ef - 1023;
}

// |x| = M * 2^E, M < 2^53 integer (x finite).
__device__ __forceinline__ void decompose(double x, uint64_t &M, int &E) {
    uint64_t b = abs_bits(x);
    int ef = (int)(b >> 52);
    uint64_t mant = b & ((1ull << 52) - 1);
    if (ef == 0) {
        M = mant;
        E = -1074;
    } else {
        M = mant | (1ull << 52);
        E = ef - 1075;
    }
}

// ceil(|x| * 2^sh) for finite x when the result is below 2^63.
__device__ __forceinline__ uint64_t ceil_scaled(double x, int sh) {
    uint64_t M;
    int E;
    decompose(x, M, E);
    if (M == 0) return 0;
    int s = E + sh;
    if (s >= 0) return M << s;
    if (s <= -64) return 1;
    int r = -s;
    return (M + ((1ull << r) - 1)) >> r;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        uint64_t o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

constexpr int kHChunk = 2048;  // k-elements per block along a row

__global__ void fill_u64_kernel(uint64_t *p, int64_t n, uint64_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------- row max |x|

// Block (bx, by) of the scan grids: contig rows take 4 rows x kHChunk elements
// (a wave per row), strided rows 256 rows x kHChunk / 8 elements.
template <int EK>
__device__ __forceinline__ void maxabs_contig_body(const OperandView &v, uint64_t *maxbits,
                                                   int64_t bx, int64_t by) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t r = bx * 4 + wave;
    if (r >= v.rows) return;
    const int64_t h0 = by * kHChunk;
    const int64_t h1 = min(v.k, h0 + kHChunk);
    uint64_t m = 0;
    for (int64_t h = h0 + lane; h < h1; h += 64) {
        double re, im;
        load_elem<EK>(v.base, r * v.stride_r + h, re, im);
        uint64_t a = abs_bits(re), b = abs_bits(im);
        m = max(m, max(a, b));
    }
    m = wave_max_u64(m);
    if (lane == 0 && m) atomicMax((unsigned long long *)&maxbits[r], (unsigned long long)m);
}

template <int EK>
__device__ __forceinline__ void maxabs_strided_body(const OperandView &v, uint64_t *maxbits,
                                                    int64_t bx, int64_t by, int hc) {
    const int64_t r = bx * 256 + threadIdx.x;
    if (r >= v.rows) return;
    const int64_t h0 = by * hc;
    const int64_t h1 = min(v.k, h0 + hc);
    uint64_t m = 0;
    for (int64_t h = h0; h < h1; ++h) {
        double re, im;
        load_elem<EK>(v.base, r + h * v.stride_h, re, im);
        m = max(m, max(abs_bits(re), abs_bits(im)));
    }
    if (m) atomicMax((unsigned long long *)&maxbits[r], (unsigned long long)m);
}

// ---------------------------------------------------------------- fast-mode sum of squares
// sigma_r = sum over the 2k reals of ceil(|x| 2^(F - e_r))^2, e_r = floor(log2 max|x|):
// an integer upper bound of 2^(2F) ||row / 2^e_r||_2^2, independent of summation order.
// The moduli-count predictor takes it with its statistics in one pass:
// tau_r = sum ceil(|x| 2^(F - e_r)) (an upper bound of 2^F ||row / 2^e_r||_1) and the
// number of zero reals of the operand, added to *zeros (all rows, finite or not).
// Real operands have k reals per row (the imaginary parts do not exist).

template <int EK>
__device__ __forceinline__ void sigma_contig_body(const OperandView &v, const uint64_t *maxbits,
                                                  uint64_t *sigma, uint64_t *tau, uint64_t *zeros,
                                                  int64_t bx, int64_t by) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t r = bx * 4 + wave;
    if (r >= v.rows) return;
    const uint64_t mb = maxbits[r];
    const bool live = mb != 0 && mb < kInfBits;
    const int sh = live ? kSigmaFracBits - ilogb_bits(mb) : 0;
    const int64_t h0 = by * kHChunk;
    const int64_t h1 = min(v.k, h0 + kHChunk);
    uint64_t s = 0, t = 0, z = 0;
    for (int64_t h = h0 + lane; h < h1; h += 64) {
        double re, im;
        load_elem<EK>(v.base, r * v.stride_r + h, re, im);
        z += (re == 0.0) + (!elem_real(EK) && im == 0.0);
        if (!live) continue;
        uint64_t a = ceil_scaled(re, sh), b = ceil_scaled(im, sh);
        s += a * a + b * b;
        t += a + b;
    }
    s = wave_sum_u64(s);
    if (lane == 0 && s) atomicAdd((unsigned long long *)&sigma[r], (unsigned long long)s);
    t = wave_sum_u64(t);
    z = wave_sum_u64(z);
    if (lane == 0 && t) atomicAdd((unsigned long long *)&tau[r], (unsigned long long)t);
    if (lane == 0 && z) atomicAdd((unsigned long long *)zeros, (unsigned long long)z);
}

template <int EK>
__device__ __forceinline__ void sigma_strided_body(const OperandView &v, const uint64_t *maxbits,
                                                   uint64_t *sigma, uint64_t *tau, uint64_t *zeros,
                                                   int64_t bx, int64_t by, int hc) {
    const int64_t r = bx * 256 + threadIdx.x;
    if (r >= v.rows) return;
    const uint64_t mb = maxbits[r];
    const bool live = mb != 0 && mb < kInfBits;
    const int sh = live ? kSigmaFracBits - ilogb_bits(mb) : 0;
    const int64_t h0 = by * hc;
    const int64_t h1 = min(v.k, h0 + hc);
    uint64_t s = 0, t = 0, z = 0;
    for (int64_t h = h0; h < h1; ++h) {
        double re, im;
        load_elem<EK>(v.base, r + h * v.stride_h, re, im);
        z += (re == 0.0) + (!elem_real(EK) && im == 0.0);
        if (!live) continue;
        uint64_t a = ceil_scaled(re, sh), b = ceil_scaled(im, sh);
        s += a * a + b * b;
        t += a + b;
    }
    if (s) atomicAdd((unsigned long long *)&sigma[r], (unsigned long long)s);
    if (t) atomicAdd((unsigned long long *)&tau[r], (unsigned long long)t);
    if (z) atomicAdd((unsigned long long *)zeros, (unsigned long long)z);
}

// ---------------------------------------------------------------- exponents
// Fast mode: mu_r = t - e_r with t the largest integer <= P'_fast - 1 such that
// 8 sigma 4^t <= (P - 1) 2^(2F)  (the Cauchy-Schwarz rule of Section III-B in
// exact integer form).  Accurate mode: mu_r = (5 - e_r) + t with t the largest
// integer such that 2 X_r 4^t <= P - 1, X_r the row maximum of the bound product.

// Smallest d with s <= fast_thr[d] (at most kThr - 1).  fast_thr[d] = floor(X 4^d) for one
// X, so its bit length is that of fast_thr[0] plus 2 d: the bit length of s leaves one
// entry to compare with.  (Entries clamped to 2^64 - 1 are met by every s.)
__device__ __forceinline__ int fast_index(uint64_t s, const OZC_AS_CONST NTable *ct) {
    const int b0 = 64 - __clzll((long long)ct->fast_thr[0]), bs = 64 - __clzll((long long)s);
    const int d = bs > b0 ? (bs - b0 + 1) >> 1 : 0;
    if (d >= kThr - 1) return kThr - 1;
    return bs == b0 + 2 * d && ct->fast_thr[d] < s ? d + 1 : d;
}

// The exponent of a fast-mode row from its maximum (bit pattern mb, finite, nonzero) and
// the FP64 sum S of its squares alone, where these decide it.  sigma enters the rule only
// through the index above, a step function with steps of a factor 4, and with
// y = |x| 2^(F - e) and n reals in the row
//   S 2^(2F - 2e) <= sigma < sum (y + 1)^2 <= S' + 2 sqrt(n S') + n,  S' = S 2^(2F - 2e)
// (Cauchy-Schwarz; the rounding of S, at most n 2^-53 <= 2^-35 relative, is covered by
// factors 1 -+ 2^-30).  When both ends have the same index, it is sigma's.  They differ
// for about one row in 10^3..10^4 (S' >= 2^40, so the interval is 4e-4 wide at k = 16384),
// and for exponents so large or small that the squares may leave the FP64 range: then
// the exact integer sum is needed (returns false).
__device__ __forceinline__ bool exponent_from_squares(uint64_t mb, double S, double n,
                                                      const OZC_AS_CONST NTable *ct, int &mu) {
    const int e = ilogb_bits(mb);
    if (e < -450 || e > 450) return false;
    const double Sp = __builtin_ldexp(S, 2 * (kSigmaFracBits - e));
    const double hi = Sp * (1.0 + 0x1p-30);
    const double up = (hi + 2.0 * __builtin_sqrt(n * hi) + n) * (1.0 + 0x1p-30) + 1.0;
    // index of x >= 2^39: thresholds are X 4^d, so the smallest d >= 0 with x / X <= 4^d, from the
    // exponent of x / X.  (At an exact power of four one too many; the factors above make that
    // right for the lower end, whose true value is larger, and safe for the upper one.)
    auto index = [&](double x) {
        const int e2 = __builtin_amdgcn_frexp_exp(x * ct->inv_fast_thr0) - 1;  // floor(log2)
        return e2 >= 0 ? (e2 + 2) >> 1 : 0;
    };
    const int dl = index(Sp * (1.0 - 0x1p-30)), du = index(up);
    mu = ct->fast_tmax - dl - e;
    return dl == du;
}

__device__ __forceinline__ void fast_exponents_body(const uint64_t *maxbits, const uint64_t *sigma,
                                                    int64_t rows, int64_t rows_pad,
                                                    const NTable *tab, int16_t *mu,
                                                    uint32_t *status, int64_t bx) {
    const int64_t r = bx * 256 + threadIdx.x;
    if (r >= rows_pad) return;
    int16_t out = kExpZero;
    if (r < rows) {
        const uint64_t mb = maxbits[r];
        if (mb >= kInfBits) {
            out = kExpNonfinite;
            atomicOr(status, 1u);
        } else if (mb != 0) {
            const OZC_AS_CONST NTable *ct = const_ptr(tab);
            out = (int16_t)(ct->fast_tmax - fast_index(sigma[r], ct) - ilogb_bits(mb));
        }
    }
    mu[r] = out;
}

__device__ __forceinline__ void accu_exponents_body(const uint64_t *maxbits, const int32_t *X,
                                                    int64_t rows, int64_t rows_pad,
                                                    const NTable *tab, int16_t *mu,
                                                    uint32_t *status, int64_t bx) {
    const int64_t r = bx * 256 + threadIdx.x;
    if (r >= rows_pad) return;
    int16_t out = kExpZero;
    if (r < rows) {
        const uint64_t mb = maxbits[r];
        if (mb >= kInfBits) {
            out = kExpNonfinite;
            atomicOr(status, 1u);
        } else if (mb != 0 && X[r] > 0) {
            const uint64_t x = (uint64_t)X[r];
            int d = 0;
            const OZC_AS_CONST NTable *ct = const_ptr(tab);
            while (d < kThr - 1 && ct->accu_thr[d] < x) ++d;
            out = (int16_t)((kAccuIntBits - 1) - ilogb_bits(mb) + ct->accu_thi - d);
        }
    }
    mu[r] = out;
}

// Both operands of a single call: A's blocks, then B's.
__global__ __launch_bounds__(256) void pair_accu_exponents_kernel(AccuSide a, AccuSide b, uint32_t blocks_a,
                                                                  const NTable *tab, uint32_t *status) {
    const bool second = blockIdx.x >= blocks_a;
    const AccuSide &o = second ? b : a;
    accu_exponents_body(o.maxbits, o.X, o.v.rows, o.rows_pad, tab, o.mu, status,
                        second ? blockIdx.x - blocks_a : blockIdx.x);
}

// ---------------------------------------------------------------- one-read scaling scan
// Maximum and FP64 sum of squares of every row in ONE read of the operand, and the
// exponents from them (exponent_from_squares); the integer sums are formed only for the
// rows that need them, by a second read of these rows (exact_sums).
// Bound by HBM: 16 rows x `chunk` k-elements per block of 1024 threads, eight loads in
// flight per thread.  Rows with contiguous k take a wave each; rows contiguous with each
// other take 16 rows (256-byte runs of complex128) x 64 k per load.
// With one part per row (chunk >= k) the block finishes its rows, exponents included: one
// launch, no atomics and nothing to clear.  With several parts they go to part_max and
// part_sq ([part][row]) and scan_finish_kernel combines them: a block per group and part, each
// with the whole of its rows' parts, so that all of them see which rows need their integer sums;
// each block then forms its own part of these and the last one to arrive has the total.
// Accurate mode takes the maxima only, and clears the rows' bound-product maxima X.
// Whole calls against the two-read scans with their fill and exponent launches: ZGEMM 64^3
// 46.1 -> 29.0 us (9 launches -> 4, one split launch among them), 384 x 320 x 40000
// 1237 -> 1111 us, CGEMM 4096^3 at N = 6 1481 -> 1402 us, ZGEMM 4096^3 3305 -> 3204 us.
constexpr int kScanRows = 16, kScanThreads = 1024, kScanLanes = kScanThreads / kScanRows;
constexpr int kScanUnroll = 8;

struct RowScan {
    // places the parts' results in `scratch` (row_scan_scratch bytes)
    __host__ __device__ __forceinline__ void use(void *scratch) {
        part_max = (uint64_t *)scratch;
        part_sq = (double *)(part_max + parts * rows_pad);
        part_sum = (uint64_t *)(part_sq + parts * rows_pad);
        arrived = (uint32_t *)(part_sum + rows_pad);
    }
    OperandView v;
    int64_t rows_pad, chunk;
    int32_t parts, groups;   // parts per row, groups of kScanRows rows (rows_pad / 16)
    uint64_t *part_max;      // parts > 1: [parts][rows_pad]
    double *part_sq;
    uint64_t *part_sum;      // [rows_pad]: integer sums ...
    uint32_t *arrived;       // [groups]: ... and the blocks that have added to them
    int16_t *mu;             // fast mode: exponents
    uint64_t *maxbits;       // accurate mode: row maxima ...
    int32_t *X;              // ... and bound maxima to clear
};

// Integer sums over the k-elements h0 .. h1 - 1 of the block's rows from r0 on with need[i] != 0
// (the rows' maxima; `rows` of them), added to exact[i] (cleared).  All threads of the block
// call this.  Up to four rows are taken one by one by all threads (rows next to a threshold,
// one in 10^3..10^4), more of them together in the scan's access pattern, one more read of the
// operand: operands beyond the range of FP64 squares need every row.  One by one, a load at a
// time and by the few blocks that combine the parts, whole operands took ZGEMM 384 x 320 x 40000
// 2250 us (now 1007; 781 within the range), DGEMM 8000 x 64 x 9000 2041 (821; 715), ZGEMM
// 2048^3 (A as it is, B transposed) 668 (549; 530).
constexpr int kExactByRow = 4, kExactUnroll = 4;
template <int EK>
__device__ __forceinline__ void exact_sums(const OperandView &v, int64_t r0, int64_t h0, int64_t h1,
                                           const uint64_t *need, int rows, unsigned long long *exact) {
    int tid = threadIdx.x;  // not shared with the scan's loop, which has no register to spare
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const bool each = rows <= kExactByRow, together = !each && !v.contig_h;
    // this thread's rows i, i + di, ... and elements `first`, first + step, ... of them
    const int threads = blockDim.x;
    int i = each ? 0 : (together ? lane % kScanRows : tid >> 6);
    const int di = each ? 1 : (together ? kScanRows : threads / 64);
    const int first = each ? tid : (together ? tid / kScanRows : lane);
    const int step = each ? threads : (together ? threads / kScanRows : 64);
    uint64_t s = 0;
    for (; i < kScanRows; i += di) {
        if (need[i] == 0) continue;
        const int sh = kSigmaFracBits - ilogb_bits(need[i]);
        const int64_t base = (r0 + i) * v.stride_r;
        s = 0;
#pragma unroll 1
        for (int64_t h = h0 + first; h < h1; h += step * kExactUnroll) {
            double re[kExactUnroll], im[kExactUnroll];
#pragma unroll
            for (int u = 0; u < kExactUnroll; ++u)
                load_elem<EK>(v.base, base + min(h + u * step, h1 - 1) * v.stride_h, re[u], im[u]);
#pragma unroll
            for (int u = 0; u < kExactUnroll; ++u) {
                const uint64_t a = ceil_scaled(re[u], sh), b = ceil_scaled(im[u], sh);
                if (h + u * step < h1) s += a * a + b * b;
            }
        }
        if (together) break;
        s = wave_sum_u64(s);
        if (lane == 0) atomicAdd(&exact[i], (unsigned long long)s);
    }
    if (!together) return;
#pragma unroll
    for (int off = 32; off >= kScanRows; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane < kScanRows && s) atomicAdd(&exact[lane], (unsigned long long)s);
}

// Exponents (or, accurate mode, maxima) of the block's kScanRows rows from r0 on: m and q
// hold row r0 + tid's maximum and sum of squares in threads tid < kScanRows.  `part` of
// a.parts blocks on the same rows; each has the same m and q.  All threads of the block call
// this (it synchronises).
template <int EK, bool ACCU>
__device__ __forceinline__ void scan_finish(const RowScan &a, int64_t r0, int part, uint64_t m, double q,
                                            const NTable *tab) {
    __shared__ uint64_t need[kScanRows];
    __shared__ unsigned long long exact[kScanRows];
    const int tid = threadIdx.x;
    const int64_t row = r0 + tid;
    const bool mine = tid < kScanRows && row < a.rows_pad;
    if constexpr (ACCU) {
        if (mine && row < a.v.rows) {
            a.maxbits[row] = m;
            a.X[row] = 0;
        }
        return;
    }
    const OZC_AS_CONST NTable *ct = const_ptr(tab);
    int mu = kExpZero;
    bool open = false;
    if (mine && row < a.v.rows) {
        if (m >= kInfBits) mu = kExpNonfinite;
        else if (m != 0)
            open = !exponent_from_squares(m, q, (double)(elem_real(EK) ? a.v.k : 2 * a.v.k), ct, mu);
    }
    if (tid < kScanRows) {
        need[tid] = open ? m : 0;
        exact[tid] = 0;
    }
    if (mine && !open && part == 0) a.mu[row] = (int16_t)mu;
    if (!__syncthreads_or(open)) return;
    int rows = 0;
    for (int i = 0; i < kScanRows; ++i) rows += need[i] != 0;
    const int64_t h0 = part * a.chunk;
    exact_sums<EK>(a.v, r0, h0, min(a.v.k, h0 + a.chunk), need, rows, exact);
    __syncthreads();
    // (everything a thread keeps across the sums costs the scan a register: from LDS again)
    const uint64_t top = threadIdx.x < kScanRows ? need[threadIdx.x] : 0;
    uint64_t s = top ? exact[threadIdx.x] : 0;
    if (a.parts > 1) {  // the parts meet: the last block to arrive has the sums
        __shared__ bool last;
        uint64_t *sum = a.part_sum + r0 + threadIdx.x;
        if (top) atomicAdd((unsigned long long *)sum, (unsigned long long)s);
        __threadfence();
        if (threadIdx.x == 0) last = atomicAdd(&a.arrived[r0 / kScanRows], 1u) == (uint32_t)a.parts - 1;
        __syncthreads();
        if (!last) return;
        __threadfence();
        if (top) s = atomicAdd((unsigned long long *)sum, 0ull);
    }
    if (top) a.mu[r0 + threadIdx.x] = (int16_t)(ct->fast_tmax - fast_index(s, ct) - ilogb_bits(top));
}

template <int EK, bool ACCU>
__device__ __forceinline__ void row_scan_body(const RowScan &a, int group, int part, const NTable *tab) {
    __shared__ uint64_t lm[kScanThreads / 64][kScanRows];
    __shared__ double lq[kScanThreads / 64][kScanRows];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r0 = (int64_t)group * kScanRows;
    const bool contig = a.v.contig_h != 0;
    const int64_t r = r0 + (contig ? wave : lane % kScanRows);
    const int hl = contig ? lane : tid / kScanRows;
    const int64_t h0 = part * a.chunk, h1 = min(a.v.k, h0 + a.chunk);
    uint64_t m = 0;
    double q = 0.0;
    if (r < a.v.rows && h0 < h1) {
        const int64_t base = r * a.v.stride_r;
        for (int64_t h = h0 + hl; h < h1; h += kScanLanes * kScanUnroll) {
            double re[kScanUnroll], im[kScanUnroll];
            // clamped addresses: the loads are unconditional, so all of them are in flight
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u)
                load_elem<EK>(a.v.base, base + min(h + u * kScanLanes, h1 - 1) * a.v.stride_h, re[u], im[u]);
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) {
                const bool in = h + u * kScanLanes < h1;  // past the end: the last element again
                m = max(m, max(abs_bits(re[u]), abs_bits(im[u])));
                if constexpr (!ACCU) {
                    const double x = in ? re[u] : 0.0, y = in ? im[u] : 0.0;
                    q = fma(x, x, q);
                    if constexpr (!elem_real(EK)) q = fma(y, y, q);
                }
            }
        }
    }
    // rows contiguous with each other: the lanes of a row are 16 apart
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        if (!contig && off < kScanRows) break;
        m = max(m, __shfl_xor(m, off, 64));
        if constexpr (!ACCU) q += __shfl_xor(q, off, 64);
    }
    if (contig) {
        if (lane == 0) {
            lm[0][wave] = m;
            if constexpr (!ACCU) lq[0][wave] = q;
        }
    } else if (lane < kScanRows) {
        lm[wave][lane] = m;
        if constexpr (!ACCU) lq[wave][lane] = q;
    }
    __syncthreads();
    if (tid < kScanRows) {
        m = lm[0][tid];
        if constexpr (!ACCU) q = lq[0][tid];
        if (!contig) {
            for (int w = 1; w < kScanThreads / 64; ++w) {
                m = max(m, lm[w][tid]);
                if constexpr (!ACCU) q += lq[w][tid];
            }
        }
        if (a.parts > 1 && r0 + tid < a.rows_pad) {
            a.part_max[part * a.rows_pad + r0 + tid] = m;
            if constexpr (!ACCU) {
                a.part_sq[part * a.rows_pad + r0 + tid] = q;
                if (part == 0) a.part_sum[r0 + tid] = 0;
                if (part == 0 && tid == 0) a.arrived[group] = 0;
            }
        }
    }
    if (a.parts == 1) scan_finish<EK, ACCU>(a, r0, 0, m, q, tab);
}

// Rows scanned in several parts: group and part of block `blk` (accurate mode: one block per
// group), 16 threads per row over the parts.
template <bool ACCU>
__host__ __device__ __forceinline__ int64_t scan_finish_blocks(int64_t groups, int64_t parts) {
    return parts > 1 ? (ACCU ? groups : groups * parts) : 0;
}
template <int EK, bool ACCU>
__device__ __forceinline__ void scan_combine(const RowScan &w, int blk, const NTable *tab) {
    const int part = blk / w.groups;
    const int64_t r0 = (int64_t)(blk - part * w.groups) * kScanRows;
    __shared__ uint64_t lm[16][kScanRows];
    __shared__ double lq[16][kScanRows];
    const int tid = threadIdx.x, rl = tid % kScanRows, pl = tid / kScanRows;
    uint64_t m = 0;
    double q = 0.0;
    if (r0 + rl < w.v.rows) {
        for (int p = pl; p < w.parts; p += 16) {
            m = max(m, w.part_max[p * w.rows_pad + r0 + rl]);
            if constexpr (!ACCU) q += w.part_sq[p * w.rows_pad + r0 + rl];
        }
    }
    lm[pl][rl] = m;
    lq[pl][rl] = q;
    __syncthreads();
    if (tid < kScanRows) {
        for (int p = 1; p < 16; ++p) {
            m = max(m, lm[p][tid]);
            q += lq[p][tid];
        }
    }
    scan_finish<EK, ACCU>(w, r0, part, m, q, tab);
}

// ---------------------------------------------------------------- accurate-mode magnitudes
// Tile of 32 rows x 64 k-elements per block.  Each thread takes 8 elements
// and writes the 7-bit magnitudes ceil(|x| 2^(5 - e)) of the real and
// imaginary parts and their difference (the three INT8 operands of the bound
// product, Section III-B), staged in LDS and stored zero-padded to
// rows_pad x k_pad in slab-major order: the 64-wide k-slab kb of a plane is a
// contiguous rows_pad x 64-byte block (row r at byte 64 r), so that the
// product kernels stream whole cache lines.

constexpr int kTileR = 32, kTileH = 64, kLdsPitch = 80;

template <int EK, bool CONTIG_H>
__device__ __forceinline__ void ceil7_body(const OperandView &v, const uint64_t *maxbits,
                                           int8_t *dst, int64_t rows_pad, int64_t k_pad,
                                           int64_t bx, int64_t by) {
    constexpr int NPLANES = elem_real(EK) ? 1 : 3;  // real: Abar only; complex: Abar_R, Abar_I, Abar_R - Abar_I
    __shared__ __align__(16) int8_t lds[NPLANES][kTileR][kLdsPitch];
    const int tid = threadIdx.x;
    const int64_t h0 = bx * kTileH;
    const int64_t r0 = by * kTileR;
    const int64_t plane_pitch = rows_pad * k_pad;

#pragma unroll
    for (int e = 0; e < 8; ++e) {
        // element coordinates: consecutive lanes follow the contiguous direction
        const int hl = CONTIG_H ? (tid & 63) : (tid >> 5) + 8 * e;
        const int rl = CONTIG_H ? (tid >> 6) + 4 * e : (tid & 31);
        const int64_t r = r0 + rl, h = h0 + hl;
        int a = 0, b = 0;
        if (r < v.rows && h < v.k) {
            const uint64_t mb = maxbits[r];
            if (mb != 0 && mb < kInfBits) {
                const int ex = ilogb_bits(mb);
                double re, im;
                load_elem<EK>(v.base, r * v.stride_r + h * v.stride_h, re, im);
                if (v.conj) im = -im;
                a = (int)ceil_scaled(re, (kAccuIntBits - 1) - ex);
                b = (int)ceil_scaled(im, (kAccuIntBits - 1) - ex);
            }
        }
        lds[0][rl][hl] = (int8_t)a;
        if constexpr (NPLANES == 3) {
            lds[1][rl][hl] = (int8_t)b;
            lds[2][rl][hl] = (int8_t)(a - b);
        }
    }
    __syncthreads();
    for (int t = tid; t < NPLANES * kTileR * 4; t += 256) {
        const int pl = t >> 7, row = (t >> 2) & 31, seg = t & 3;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 val = *reinterpret_cast<const u32x4 *>(&lds[pl][row][seg * 16]);
        int8_t *out = dst + (int64_t)pl * plane_pitch + (bx * rows_pad + r0 + row) * kTileH + seg * 16;
        *global_ptr(reinterpret_cast<u32x4 *>(out)) = val;
    }
}

// ---------------------------------------------------------------- residue split
// Truncation a' = trunc(x 2^mu) and symmetric residues modulo every p_l (and,
// for Karatsuba, the reduced sum of the real and imaginary residues), written
// with zero k-padding to k_pad in the slab-major order of the product kernels
// (rows up to rows_pad; the padding rows are left as they are).  No LDS staging: a block of 256 threads covers 16 rows and one
// 64-wide k-slab; each thread holds 4 consecutive k of one row and writes
// their residues as one 4-byte word per plane and modulus.  Sixteen
// consecutive lanes share a row, so each wave writes 4 whole 64-byte rows
// (256 contiguous bytes) per plane and modulus.  Loads: for rows contiguous
// with each other one load instruction reads 4 rows at 16 k (64-byte runs);
// for rows with contiguous k each lane reads its own 64-byte run.
//
// Residues through byte dot products: the signed a' is written as the W-word integer
// u = a' + 2^(32 W - 1) (0 <= u < 2^(32 W), W the smallest word count with
// |a'| < 2^(32 W - 1)), and per modulus x' = sum_j u_j w_j + 128 - (2^(32 W - 1) mod p),
// with u_j the bytes of u and w_j = 2^(8 j) mod p in [0, p - 1]: one unsigned 4-byte
// dot product per word (the offsets enter as the accumulator's start), so that
// x = x' - 128 is congruent to a' modulo p and |x| <= 16 * 255 * 255 + 255 < 2^20.
// Its symmetric residue s comes in FP32 as the byte s + 128 = x' - p q with
// q = floor(fl(x' fl(1/p) + (0.5 - 128 fl(1/p)))) = floor(fl(x fl(1/p) + 0.5)), one fma
// (the offset is exact): the computed value is within |x / p| 2^-24 + ulp / 2 < 1 / (2p)
// of x / p + 1/2, which for odd p lies at least 1 / (2p) from every integer, so q is
// x / p rounded to the nearest integer; for p = 256 everything is exact and a tie
// rounds up, giving s = -128.  So s + 128 is an exact integer in [0, 255]: one
// conversion-and-insert per byte, and flipping bit 7 of each byte gives the signed
// residue.  The reduced sum of the real and imaginary residues takes the same rule.
constexpr int kEPT = 4;                   // k-consecutive elements per thread
constexpr int kDirectRows = 4 * kEPT;     // 256 threads, 64 / kEPT threads per row

__device__ __forceinline__ uint32_t pack_bytes(int a, int b, int c, int d) {
    return (uint32_t)(a & 0xff) | ((uint32_t)(b & 0xff) << 8) | ((uint32_t)(c & 0xff) << 16) |
           ((uint32_t)(d & 0xff) << 24);
}

// Four residues (one byte each, k ascending) as one store.
__device__ __forceinline__ void store_word(int8_t *p, uint32_t w) {
    *global_ptr(reinterpret_cast<uint32_t *>(p)) = w;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// The residues r[0..kEPT-1] as one store.
static_assert(kEPT == 2 || kEPT == 4 || kEPT == 8, "2, 4 or 8 elements per thread");
template <int E>
__device__ __forceinline__ void store_res(int8_t *p, const int (&r)[E]) {
    if constexpr (E == 8) {
        const u32x2 w{pack_bytes(r[0], r[1], r[2], r[3]), pack_bytes(r[4], r[5], r[6], r[7])};
        *global_ptr(reinterpret_cast<u32x2 *>(p)) = w;
    } else if constexpr (E == 4) {
        *global_ptr(reinterpret_cast<uint32_t *>(p)) = pack_bytes(r[0], r[1], r[2], r[3]);
    } else {
        *global_ptr(reinterpret_cast<uint16_t *>(p)) = (uint16_t)((r[0] & 0xff) | ((r[1] & 0xff) << 8));
    }
}

// u = a' + 2^(32 W - 1) for a' = trunc(|x| 2^mu) signed like x (|a'| < 2^(32 W - 1)),
// as W little-endian 32-bit words, in FP64: a' is exact as a double (|x| 2^mu is a
// power-of-two scaling of x, and anything below 1 truncates to 0), and the words come
// off from the bottom, q_{i+1} = floor(q_i 2^-32), word_i = q_i - 2^32 q_{i+1} in
// [0, 2^32) (exact: an integer below 2^32); the top q is signed, and adding the bias
// 2^31 to it flips its sign bit.
template <int W>
__device__ __forceinline__ void biased_words(double x, int mu, uint32_t (&u)[W]) {
    double q = __builtin_trunc(__builtin_ldexp(x, mu));
#pragma unroll
    for (int i = 0; i < W - 1; ++i) {
        const double hi = __builtin_floor(q * 0x1p-32);
        u[i] = (uint32_t)__builtin_fma(hi, -0x1p32, q);
        q = hi;
    }
    u[W - 1] = (uint32_t)(int32_t)q ^ 0x80000000u;
}

// x' = sum_j u_j w_j + 128 - (2^(32 W - 1) mod p) as a float (an exact integer).
template <int W>
__device__ __forceinline__ float byte_dot(const uint32_t (&u)[W], const uint32_t (&wb)[W],
                                          uint32_t bias) {
    uint32_t acc = bias;
#pragma unroll
    for (int i = 0; i < W; ++i) acc = __builtin_amdgcn_udot4(u[i], wb[i], acc, false);
    return (float)(int32_t)acc;
}

// s + 128 for the symmetric residue s of x = x' - 128 (x' an exact integer, |x| < 2^20).
__device__ __forceinline__ float smod_u8(float xs, float p, float ip, float rbias) {
    return __builtin_fmaf(-__builtin_floorf(__builtin_fmaf(xs, ip, rbias)), p, xs);
}

// kEPT consecutive elements of row r from h0 on, conjugated where the view says so; zeros past k.
template <int EK>
__device__ __forceinline__ void load_quad(const OperandView &v, int64_t r, int64_t h0, double *re, double *im) {
#pragma unroll
    for (int j = 0; j < kEPT; ++j) {
        re[j] = im[j] = 0.0;
        const int64_t h = h0 + j;
        if (h < v.k) {
            load_elem<EK>(v.base, r * v.stride_r + h * v.stride_h, re[j], im[j]);
            if (v.conj) im[j] = -im[j];
        }
    }
}

// The residues of kEPT consecutive elements (exponent ex) to out, one word per plane and
// modulus; elements past k are zeros, whose residues are 0.
template <int EK, int NPLANES, int W>
__device__ __forceinline__ void split_quad(const double *re, const double *im, int ex,
                                           const NTable *__restrict__ tab, int nmod,
                                           int8_t *__restrict__ out, int64_t plane_pitch) {
    static_assert(NPLANES != 1 || elem_real(EK), "one residue plane for real operands only");
    static_assert(kEPT == 4, "one 4-byte word of residues per plane and modulus");
    uint32_t uR[kEPT][W], uI[kEPT][W];
#pragma unroll
    for (int j = 0; j < kEPT; ++j) {
        biased_words<W>(re[j], ex, uR[j]);
        if constexpr (NPLANES > 1) biased_words<W>(im[j], ex, uI[j]);
    }
    // a modulus' constants are loaded while the one before is worked on: with few waves
    // (short calls) the scalar loads' latency would show once per modulus
    struct Rule {
        float p, ip, rb;
        uint32_t wb[W], bias;
    };
    auto rule_of = [&](int l) {
        const OZC_AS_CONST ModConst &mc = const_ptr(tab)->mod[l];
        Rule r{mc.pf, mc.ipf, mc.rbias, {}, mc.wbias[W - 1]};
#pragma unroll
        for (int i = 0; i < W; ++i) r.wb[i] = mc.wbyte[i];
        return r;
    };
    Rule next = rule_of(0);
    for (int l = 0; l < nmod; ++l) {
        const Rule cur = next;
        next = rule_of(min(l + 1, nmod - 1));
        const float p = cur.p, ip = cur.ip, rb = cur.rb;
        const uint32_t(&wb)[W] = cur.wb;
        const uint32_t bias = cur.bias;
        uint32_t wa = 0, wbi = 0, wc = 0;  // residues + 128 as bytes, k ascending
#pragma unroll
        for (int j = 0; j < kEPT; ++j) {
            const float sa = smod_u8(byte_dot<W>(uR[j], wb, bias), p, ip, rb);
            wa = __builtin_amdgcn_cvt_pk_u8_f32(sa, j, wa);
            if constexpr (NPLANES > 1) {
                const float sb = smod_u8(byte_dot<W>(uI[j], wb, bias), p, ip, rb);
                wbi = __builtin_amdgcn_cvt_pk_u8_f32(sb, j, wbi);
                if constexpr (NPLANES == 3) {  // (s_a + s_b) + 128 = (sa - 128) + sb
                    const float sc = smod_u8((sa - 128.0f) + sb, p, ip, rb);
                    wc = __builtin_amdgcn_cvt_pk_u8_f32(sc, j, wc);
                }
            }
        }
        int8_t *o = out + (int64_t)l * NPLANES * plane_pitch;
        store_word(o, wa ^ 0x80808080u);
        if constexpr (NPLANES > 1) store_word(o + plane_pitch, wbi ^ 0x80808080u);
        if constexpr (NPLANES == 3) store_word(o + 2 * plane_pitch, wc ^ 0x80808080u);
    }
}

// k padding, or a row without scaling: every residue is 0.
template <int NPLANES>
__device__ __forceinline__ void split_zeros(int nmod, int8_t *__restrict__ out, int64_t plane_pitch) {
    const int z[kEPT] = {};
    for (int q = 0; q < nmod * NPLANES; ++q) store_res(out + (int64_t)q * plane_pitch, z);
}

// status (may be null): bit 0 is set when a row holds inf or NaN.
template <int EK, int NPLANES, int W>
__device__ __forceinline__ void split_body(const OperandView &v, const int16_t *__restrict__ mu,
                                           const NTable *__restrict__ tab, int nmod,
                                           int8_t *__restrict__ dst, int64_t rows_pad,
                                           int64_t k_pad, int64_t bx, int64_t by, uint32_t *status) {
    const int tid = threadIdx.x;
    constexpr int TPR = kTileH / kEPT;  // threads per row
    const int rl = tid / TPR;
    const int oc = tid % TPR;
    const int64_t r = by * kDirectRows + rl;
    const int64_t h0 = bx * kTileH + kEPT * oc;

    // Rows past the operand (row padding) are not written: they meet only output rows or
    // columns past the product, which nothing reads.  Padding along k must be zero.
    if (r >= v.rows) return;
    const int ex = global_ptr(mu)[r];
    if (status && ex == kExpNonfinite && h0 == 0) atomicOr(status, 1u);
    int8_t *out = dst + (bx * rows_pad + r) * kTileH + kEPT * oc;
    if (ex == kExpZero || ex == kExpNonfinite || h0 >= v.k) {
        split_zeros<NPLANES>(nmod, out, rows_pad * k_pad);
        return;
    }
    double re[kEPT], im[kEPT];
    load_quad<EK>(v, r, h0, re, im);
    split_quad<EK, NPLANES, W>(re, im, ex, tab, nmod, out, rows_pad * k_pad);
}

// One operand of a single call's split, or of its scan and split in one.
struct SplitSide {
    OperandView v;
    const int16_t *mu;
    int8_t *dst;
    int64_t rows_pad;
    uint32_t blocks;  // split: (k_pad / 64) x (rows_pad / kDirectRows); in one: rows_pad / RB
    int16_t *mu_out;  // in one: exponents
};

// ---------------------------------------------------------------- scan and split in one
// Rows of at most kPrepMaxK elements: a block reads RB rows into registers, decides their
// exponents and splits them, one launch for both operands.  64 threads per row, each with two
// runs of 4 consecutive k, one in each half of up to eight 64-wide k-slabs; RB is blockDim / 64.
// Calls this short are chains of launches that the chip waits for: what bounds them is the
// latency of each, about 7 us a launch.  ZGEMM 64^3 24.4 -> 20.7 us, 256^3 29.9 -> 26.3 us
// against the scan and the split in two launches; from 16 rows x 256 blocks on 16 rows share a
// block (CGEMM 4096 x 4096 x 512 at N = 6: 352 us with 4 rows, 341 with 16, 344 in two launches);
// longer rows are no faster in one launch (1000^3 113 against 107 us: too few waves per block).
constexpr int kPrepMaxK = 512;

// sigma of one row by `lanes` threads (thread `lane` of them): the partial sum.
template <int EK>
__device__ __forceinline__ uint64_t exact_sigma_part(const OperandView &v, int64_t r, uint64_t mb,
                                                     int lane, int lanes) {
    const int sh = kSigmaFracBits - ilogb_bits(mb);
    uint64_t s = 0;
    for (int64_t h = lane; h < v.k; h += lanes) {
        double re, im;
        load_elem<EK>(v.base, r * v.stride_r + h * v.stride_h, re, im);
        const uint64_t a = ceil_scaled(re, sh), b = ceil_scaled(im, sh);
        s += a * a + b * b;
    }
    return s;
}

template <int EK, int NPLANES, int W>
__device__ __forceinline__ void prep_rows_body(const SplitSide &w, int64_t r0, int64_t k_pad,
                                               const NTable *__restrict__ tab, int nmod) {
    constexpr int kMaxRB = 16;
    __shared__ uint64_t lm[4][kMaxRB], lx[4][kMaxRB];
    __shared__ double lq[4][kMaxRB];
    const OperandView &v = w.v;
    const int RB = blockDim.x / 64, tid = threadIdx.x;
    const int oc = tid % 16, rl = tid / 16 % RB, part = tid / 16 / RB;  // part: every fourth slab
    const int64_t r = r0 + rl;
    const int slabs = (int)(k_pad / kTileH);
    const bool inside = r < v.rows;
    uint64_t m = 0;
    double q = 0.0;
    double re[2][kEPT], im[2][kEPT];  // slabs part and part + 4
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int64_t h0 = (int64_t)(part + 4 * t) * kTileH + kEPT * oc;
        load_quad<EK>(v, r, inside ? h0 : v.k, re[t], im[t]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int j = 0; j < kEPT; ++j) {
            m = max(m, max(abs_bits(re[t][j]), abs_bits(im[t][j])));
            q = fma(re[t][j], re[t][j], q);
            if constexpr (!elem_real(EK)) q = fma(im[t][j], im[t][j], q);
        }
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        m = max(m, __shfl_xor(m, off, 64));
        q += __shfl_xor(q, off, 64);
    }
    if (oc == 0) {
        lm[part][rl] = m;
        lq[part][rl] = q;
    }
    __syncthreads();
    m = max(max(lm[0][rl], lm[1][rl]), max(lm[2][rl], lm[3][rl]));
    q = (lq[0][rl] + lq[1][rl]) + (lq[2][rl] + lq[3][rl]);
    const OZC_AS_CONST NTable *ct = const_ptr(tab);
    int ex = kExpZero;
    bool open = false;
    if (inside) {
        if (m >= kInfBits) ex = kExpNonfinite;
        else if (m != 0)
            open = !exponent_from_squares(m, q, (double)(elem_real(EK) ? v.k : 2 * v.k), ct, ex);
    }
    if (__syncthreads_or(open)) {  // rows that need their integer sum
        uint64_t x = open ? exact_sigma_part<EK>(v, r, m, part * 16 + oc, 64) : 0;
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
        if (oc == 0) lx[part][rl] = x;
        __syncthreads();
        if (open) {
            x = (lx[0][rl] + lx[1][rl]) + (lx[2][rl] + lx[3][rl]);
            ex = ct->fast_tmax - fast_index(x, ct) - ilogb_bits(m);
        }
    }
    if (r >= w.rows_pad) return;
    if (oc == 0 && part == 0) w.mu_out[r] = (int16_t)ex;
    if (!inside) return;
    const bool live = ex != kExpZero && ex != kExpNonfinite;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int sl = part + 4 * t;
        if (sl >= slabs) break;
        int8_t *out = w.dst + (sl * w.rows_pad + r) * kTileH + kEPT * oc;
        if (live && sl * kTileH + kEPT * oc < v.k)
            split_quad<EK, NPLANES, W>(re[t], im[t], ex, tab, nmod, out, w.rows_pad * k_pad);
        else
            split_zeros<NPLANES>(nmod, out, w.rows_pad * k_pad);
    }
}

// ---------------------------------------------------------------- kernels (one problem)

// Both operands of one call in one launch, the blocks of A first.
template <int EK, bool ACCU>
__global__ __launch_bounds__(kScanThreads) void pair_row_scan_kernel(RowScan a, RowScan b,
                                                                     const NTable *tab,
                                                                     uint32_t *status) {
    if (status && blockIdx.x == 0 && threadIdx.x == 0) *status = 0;  // set again by the split
    const int nA = a.groups * a.parts;
    int blk = (int)blockIdx.x;
    const bool second = blk >= nA;
    if (second) blk -= nA;
    const RowScan &w = second ? b : a;
    row_scan_body<EK, ACCU>(w, blk % w.groups, blk / w.groups, tab);
}

// (a side with one part has no blocks here)
template <int EK, bool ACCU>
__global__ __launch_bounds__(256) void scan_finish_kernel(RowScan a, RowScan b, int blocksA,
                                                          const NTable *tab) {
    const int blk = (int)blockIdx.x;
    const bool second = blk >= blocksA;
    scan_combine<EK, ACCU>(second ? b : a, second ? blk - blocksA : blk, tab);
}
// The predictor's scans (maxima, then integer sums with its statistics) of both operands
// of one call in one launch per pass, blocks of A first, then those of B, each on the grid its own launch would have: one ramp-up and tail per pass
// instead of two, which shows where an operand takes tens of microseconds.  The
// maxima and the integer sums of squares are combined by atomics, so the result does
// not depend on the order of the blocks.
struct ScanSide {
    OperandView v;
    uint64_t *maxbits, *sigma;
    uint64_t *tau, *zeros;  // with the sums: the predictor's statistics
    int64_t gx, blocks;     // grid columns and blocks of this operand
    int hc;                 // strided layout: k-elements per thread
};
// Row maxima, or (SUMS) sums of squares and the statistics
template <int EK, bool SUMS>
__device__ __forceinline__ void scan_side(const ScanSide &sd, int64_t lb) {
    const int64_t bx = lb % sd.gx, by = lb / sd.gx;
    if (sd.v.contig_h) {
        if constexpr (SUMS) sigma_contig_body<EK>(sd.v, sd.maxbits, sd.sigma, sd.tau, sd.zeros, bx, by);
        else maxabs_contig_body<EK>(sd.v, sd.maxbits, bx, by);
    } else {
        if constexpr (SUMS)
            sigma_strided_body<EK>(sd.v, sd.maxbits, sd.sigma, sd.tau, sd.zeros, bx, by, sd.hc);
        else maxabs_strided_body<EK>(sd.v, sd.maxbits, bx, by, sd.hc);
    }
}
template <int EK, bool SUMS>
__global__ __launch_bounds__(256) void pair_scan_kernel(ScanSide a, ScanSide b) {
    const int64_t blk = blockIdx.x;
    if (blk < a.blocks) scan_side<EK, SUMS>(a, blk);
    else scan_side<EK, SUMS>(b, blk - a.blocks);
}
// The exponents of both operands of one call in one launch (the blocks of A first).
struct ExpSide {
    const uint64_t *maxbits, *sigma;
    int64_t rows, rows_pad, blocks;
    int16_t *mu;
};
__global__ __launch_bounds__(256) void pair_fast_exponents_kernel(ExpSide a, ExpSide b,
                                                                  const NTable *tab, uint32_t *status) {
    const int64_t blk = blockIdx.x;
    if (blk < a.blocks) fast_exponents_body(a.maxbits, a.sigma, a.rows, a.rows_pad, tab, a.mu, status, blk);
    else fast_exponents_body(b.maxbits, b.sigma, b.rows, b.rows_pad, tab, b.mu, status, blk - a.blocks);
}
// The residues of both operands of one call in one launch (the blocks of A first).
template <int EK, int NPLANES, int W>
__global__ __launch_bounds__(256) void pair_split_kernel(SplitSide a, SplitSide b,
                                                         const NTable *__restrict__ tab, int nmod,
                                                         int64_t k_pad, uint32_t *status) {
    uint32_t blk = blockIdx.x;
    const bool second = blk >= a.blocks;
    if (second) blk -= a.blocks;
    const SplitSide &w = second ? b : a;
    const uint32_t gx = (uint32_t)(k_pad / kTileH);
    split_body<EK, NPLANES, W>(w.v, w.mu, tab, nmod, w.dst, w.rows_pad, k_pad, blk % gx, blk / gx,
                               status);
}

template <int EK, int NPLANES, int W>
__global__ __launch_bounds__(1024) void pair_prep_kernel(SplitSide a, SplitSide b,
                                                         const NTable *__restrict__ tab, int nmod,
                                                         int64_t k_pad, uint32_t *status) {
    uint32_t blk = blockIdx.x;
    if (status && blk == 0 && threadIdx.x == 0) *status = 0;  // set again by the reconstruction
    const bool second = blk >= a.blocks;
    if (second) blk -= a.blocks;
    prep_rows_body<EK, NPLANES, W>(second ? b : a, (int64_t)blk * (blockDim.x / 64), k_pad, tab, nmod);
}

// Both operands of a single call: A's blocks, then B's.  Small accurate calls are chains of
// launches: this one and the exponents' one took two each (scaling with the bound product,
// ZGEMM 100 x 100 x 300 37.5 -> 30.8 us, CGEMM 500 x 700 x 1000 50.5 -> 39.9 us, ZGEMM 2048^3 113.1 ->
// 111.3 us).
template <int EK>
__global__ __launch_bounds__(256) void pair_ceil7_kernel(AccuSide a, AccuSide b, uint32_t blocks_a,
                                                         int64_t k_pad) {
    const bool second = blockIdx.x >= blocks_a;
    const AccuSide &o = second ? b : a;
    const uint32_t lb = second ? blockIdx.x - blocks_a : blockIdx.x, gx = (uint32_t)(k_pad / kTileH);
    const uint32_t by = lb / gx, bx = lb - by * gx;
    if (o.v.contig_h) ceil7_body<EK, true>(o.v, o.maxbits, o.bar, o.rows_pad, k_pad, bx, by);
    else ceil7_body<EK, false>(o.v, o.maxbits, o.bar, o.rows_pad, k_pad, bx, by);
}

// ---------------------------------------------------------------- kernels (batched)

// Last segment whose first block is <= b (first blocks ascending).
template <typename F>
__device__ __forceinline__ int find_seg(int n, int64_t b, F first) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first(mid) <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__host__ __device__ __forceinline__ int64_t scan_grid_x(const OperandView &v) {
    return v.contig_h ? (v.rows + 3) / 4 : (v.rows + 255) / 256;
}
__host__ __device__ __forceinline__ int64_t scan_grid_y(const OperandView &v) {
    const int64_t hc = v.contig_h ? kHChunk : kHChunk / 8;
    return (v.k + hc - 1) / hc;
}

// The predictor's scans: row maxima, or (SUMS) integer sums and statistics
// (BatchOperand::sigma, tau, zeros)
template <int EK, bool SUMS>
__global__ __launch_bounds__(256) void batch_scan_kernel(const BatchOperand *ops, int nops) {
    const int64_t b = blockIdx.x;
    const int o = find_seg(nops, b, [&](int i) { return ops[i].blk_scan; });
    const OperandView v = ops[o].v;
    const int64_t lb = b - ops[o].blk_scan, gx = scan_grid_x(v);
    const int64_t bx = lb % gx, by = lb / gx;
    const BatchOperand &op = ops[o];
    if (v.contig_h) {
        if constexpr (SUMS) sigma_contig_body<EK>(v, op.maxbits, op.sigma, op.tau, op.zeros, bx, by);
        else maxabs_contig_body<EK>(v, op.maxbits, bx, by);
    } else {
        if constexpr (SUMS)
            sigma_strided_body<EK>(v, op.maxbits, op.sigma, op.tau, op.zeros, bx, by, kHChunk / 8);
        else maxabs_strided_body<EK>(v, op.maxbits, bx, by, kHChunk / 8);
    }
}

__device__ __forceinline__ RowScan row_scan_of(const BatchOperand &op) {
    RowScan w;
    w.v = op.v;
    w.rows_pad = op.rows_pad;
    w.chunk = op.scan_chunk;
    w.parts = op.scan_parts;
    w.groups = (int32_t)(op.rows_pad / kScanRows);
    w.use(op.res);  // free until the split
    w.mu = op.mu;
    w.maxbits = op.maxbits;
    w.X = op.X;
    return w;
}
// Also clears the status word (null: not) and `ncounters` work-queue counters of the
// kernels that follow.
template <int EK, bool ACCU>
__global__ __launch_bounds__(kScanThreads) void batch_row_scan_kernel(const BatchOperand *ops, int nops,
                                                                      uint32_t *status, uint32_t *counters,
                                                                      int ncounters) {
    if (blockIdx.x == 0) {
        if (status && threadIdx.x == 0) *status = 0;
        if ((int)threadIdx.x < ncounters) counters[threadIdx.x] = 0;
    }
    const int64_t b = blockIdx.x;
    const int o = find_seg(nops, b, [&](int i) { return ops[i].blk_rows; });
    const RowScan w = row_scan_of(ops[o]);
    const int lb = (int)(b - ops[o].blk_rows);
    row_scan_body<EK, ACCU>(w, lb % w.groups, lb / w.groups, ops[o].tab);
}
template <int EK, bool ACCU>
__global__ __launch_bounds__(256) void batch_scan_finish_kernel(const BatchOperand *ops, int nops) {
    const int64_t b = blockIdx.x;  // an operand scanned in one part has no blocks here
    const int o = find_seg(nops, b, [&](int i) { return ops[i].blk_finish; });
    scan_combine<EK, ACCU>(row_scan_of(ops[o]), (int)(b - ops[o].blk_finish), ops[o].tab);
}

__global__ __launch_bounds__(256) void batch_accu_exponents_kernel(const BatchOperand *ops, int nops,
                                                                   uint32_t *status) {
    const int64_t b = blockIdx.x;
    const int o = find_seg(nops, b, [&](int i) { return ops[i].blk_exp; });
    const BatchOperand &op = ops[o];
    accu_exponents_body(op.maxbits, op.X, op.v.rows, op.rows_pad, op.tab, op.mu, status,
                        b - op.blk_exp);
}

template <int EK>
__global__ __launch_bounds__(256) void batch_ceil7_kernel(const BatchOperand *ops, int nops) {
    const int64_t b = blockIdx.x;
    const int o = find_seg(nops, b, [&](int i) { return ops[i].blk_ceil7; });
    const BatchOperand &op = ops[o];
    const int64_t lb = b - op.blk_ceil7, gx = op.k_pad / kTileH;
    const int64_t bx = lb % gx, by = lb / gx;
    if (op.v.contig_h) ceil7_body<EK, true>(op.v, op.maxbits, op.bar, op.rows_pad, op.k_pad, bx, by);
    else ceil7_body<EK, false>(op.v, op.maxbits, op.bar, op.rows_pad, op.k_pad, bx, by);
}

// Operands of one launch may have different moduli counts; W covers the largest |a'|.
template <int EK, int NPLANES, int W>
__global__ __launch_bounds__(256) void batch_split_kernel(const BatchOperand *ops, int nops,
                                                          uint32_t *status) {
    const int64_t b = blockIdx.x;
    const int o = find_seg(nops, b, [&](int i) { return ops[i].blk_split; });
    const BatchOperand &op = ops[o];
    const int64_t lb = b - op.blk_split, gx = op.k_pad / kTileH;
    const int64_t bx = lb % gx, by = lb / gx;
    split_body<EK, NPLANES, W>(op.v, op.mu, op.tab, op.nmod, op.res, op.rows_pad, op.k_pad, bx, by,
                               status);
}

__global__ void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

#define OZC_W_CASES(CASE) CASE(1) CASE(2) CASE(3) CASE(4)

template <int EK, int NPLANES>
hipError_t batch_split_w(const BatchOperand *ops, int nops, int64_t blocks, int nw, uint32_t *status,
                         hipStream_t s) {
    dim3 grid((unsigned)blocks);
#define OZC_BSPLIT_CASE(W)                                                                   \
    case W:                                                                                  \
        hipLaunchKernelGGL((batch_split_kernel<EK, NPLANES, W>), grid, dim3(256), 0, s,  \
                           ops, nops, status);                                               \
        break;
    switch (nw) {
        OZC_W_CASES(OZC_BSPLIT_CASE)
        default:
            return hipErrorInvalidValue;
    }
#undef OZC_BSPLIT_CASE
    return hipGetLastError();
}

// threads: 256 for the split, 64 RB for scan and split in one
template <int EK, int NPLANES>
hipError_t pair_split_w(const SplitSide &a, const SplitSide &b, bool scan, int threads, const NTable *tab,
                        int nmod, int nw, int64_t k_pad, uint32_t *status, hipStream_t s) {
    const dim3 grid(a.blocks + b.blocks), block((unsigned)threads);
#define OZC_SPLIT_CASE(W)                                                                              \
    case W:                                                                                            \
        if (scan)                                                                                      \
            hipLaunchKernelGGL((pair_prep_kernel<EK, NPLANES, W>), grid, block, 0, s, a, b, tab, nmod, \
                               k_pad, status);                                                         \
        else                                                                                           \
            hipLaunchKernelGGL((pair_split_kernel<EK, NPLANES, W>), grid, block, 0, s, a, b, tab,      \
                               nmod, k_pad, status);                                                   \
        break;
    switch (nw) {
        OZC_W_CASES(OZC_SPLIT_CASE)
        default:
            return hipErrorInvalidValue;
    }
#undef OZC_SPLIT_CASE
    return hipGetLastError();
}
#undef OZC_W_CASES


}  // namespace

hipError_t launch_fill_u64(uint64_t *p, int64_t n, uint64_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// k-elements per thread of the strided scans: 256, halved (down to 16) while the grid
// would have fewer than 1024 blocks, so that small operands still spread over the chip.
static int strided_chunk(const OperandView &v) {
    const int64_t bx = (v.rows + 255) / 256;
    int hc = kHChunk / 8;
    while (hc > 16 && bx * ((v.k + hc - 1) / hc) < 1024) hc /= 2;
    return hc;
}

static ScanSide scan_side_of(const OperandView &v, uint64_t *maxbits, uint64_t *sigma,
                             uint64_t *tau, uint64_t *zeros) {
    ScanSide sd{v, maxbits, sigma, tau, zeros, 0, 0, 0};
    if (v.rows <= 0 || v.k <= 0) return sd;  // no blocks
    if (v.contig_h) {
        sd.gx = (v.rows + 3) / 4;
        sd.blocks = sd.gx * ((v.k + kHChunk - 1) / kHChunk);
    } else {
        sd.hc = strided_chunk(v);
        sd.gx = (v.rows + 255) / 256;
        sd.blocks = sd.gx * ((v.k + sd.hc - 1) / sd.hc);
    }
    return sd;
}

template <int EK>
hipError_t pair_scans_ek(const ScanSide &a, const ScanSide &b, bool sums, hipStream_t s) {
    const int64_t blocks = a.blocks + b.blocks;
    if (blocks == 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    if (sums) hipLaunchKernelGGL((pair_scan_kernel<EK, true>), grid, dim3(256), 0, s, a, b);
    else hipLaunchKernelGGL((pair_scan_kernel<EK, false>), grid, dim3(256), 0, s, a, b);
    return hipGetLastError();
}

hipError_t launch_pair_scans(const OperandView &va, const OperandView &vb, bool single,
                             uint64_t *maxA, uint64_t *maxB, hipStream_t s, uint64_t *sigA,
                             uint64_t *sigB, uint64_t *tauA, uint64_t *tauB, uint64_t *zeros) {
    const bool stats = tauA != nullptr;
    if (stats != (tauB != nullptr) || stats != (zeros != nullptr) || stats != (sigA != nullptr) ||
        stats != (sigB != nullptr))
        return hipErrorInvalidValue;
    const ScanSide a = scan_side_of(va, maxA, sigA, tauA, zeros);
    const ScanSide b = scan_side_of(vb, maxB, sigB, tauB, zeros);
    return single ? pair_scans_ek<kElemC>(a, b, stats, s) : pair_scans_ek<kElemZ>(a, b, stats, s);
}

// Parts of a row: one while a thread's share of it is at most 64 loads or both operands'
// row groups give every CU a block of 1024 threads (one launch does the whole phase then);
// otherwise parts of 1024 k and more that bring the grid to about 1024 blocks.  A batch
// (groups_all = 0) has other blocks to fill the chip with: only the serial chain of a long row is cut.
int64_t row_scan_parts(int64_t k, int64_t groups_all) {
    if (k <= 64 * kScanLanes || groups_all >= 512) return 1;
    const int64_t parts = (k + 2047) / 2048;
    return groups_all > 0 ? std::max<int64_t>(1, std::min(parts, (1023 + groups_all) / groups_all)) : parts;
}
int64_t row_scan_scratch(int64_t rows_pad, int64_t parts) {
    return parts > 1 ? 16 * parts * rows_pad + 8 * rows_pad + 4 * (rows_pad / kScanRows) : 0;
}

static RowScan row_scan_of(const OperandView &v, int64_t rows_pad, int64_t groups_all, void *scratch) {
    RowScan w{};
    w.v = v;
    w.rows_pad = rows_pad;
    w.groups = (int32_t)(rows_pad / kScanRows);
    const int64_t parts = row_scan_parts(v.k, groups_all);
    w.chunk = (v.k + parts - 1) / parts;
    w.parts = (int32_t)parts;
    w.use(scratch);
    return w;
}

template <int EK>
static hipError_t row_scans_ek(const RowScan &a, const RowScan &b, bool accurate, const NTable *tab,
                               uint32_t *status, hipStream_t s) {
    const int64_t blocks = (int64_t)a.groups * a.parts + (int64_t)b.groups * b.parts;
    const int fa = (int)(accurate ? scan_finish_blocks<true>(a.groups, a.parts) : scan_finish_blocks<false>(a.groups, a.parts));
    const int fb = (int)(accurate ? scan_finish_blocks<true>(b.groups, b.parts) : scan_finish_blocks<false>(b.groups, b.parts));
    if (blocks > INT32_MAX) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks), block(kScanThreads);
    if (accurate) hipLaunchKernelGGL((pair_row_scan_kernel<EK, true>), grid, block, 0, s, a, b, tab, status);
    else hipLaunchKernelGGL((pair_row_scan_kernel<EK, false>), grid, block, 0, s, a, b, tab, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || fa + fb == 0) return e;
    const dim3 fgrid((unsigned)(fa + fb));
    if (accurate) hipLaunchKernelGGL((scan_finish_kernel<EK, true>), fgrid, dim3(256), 0, s, a, b, fa, tab);
    else hipLaunchKernelGGL((scan_finish_kernel<EK, false>), fgrid, dim3(256), 0, s, a, b, fa, tab);
    return hipGetLastError();
}

static hipError_t row_scans(RowScan &a, RowScan &b, int ek, bool accurate, const NTable *tab,
                            uint32_t *status, hipStream_t s) {
    switch (ek) {
        case kElemZ: return row_scans_ek<kElemZ>(a, b, accurate, tab, status, s);
        case kElemC: return row_scans_ek<kElemC>(a, b, accurate, tab, status, s);
        case kElemD: return row_scans_ek<kElemD>(a, b, accurate, tab, status, s);
        case kElemS: return row_scans_ek<kElemS>(a, b, accurate, tab, status, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_row_exponents(const OperandView &va, const OperandView &vb, int ek, int64_t m_pad,
                                int64_t n_pad, int16_t *mu, int16_t *nu, const ScanScratch &sc,
                                const NTable *tab, uint32_t *status, hipStream_t s) {
    if (va.rows <= 0 || vb.rows <= 0 || va.k <= 0 || m_pad % kScanRows || n_pad % kScanRows)
        return hipErrorInvalidValue;
    const int64_t groups = (m_pad + n_pad) / kScanRows;
    RowScan a = row_scan_of(va, m_pad, groups, sc.A), b = row_scan_of(vb, n_pad, groups, sc.B);
    if (row_scan_scratch(m_pad, a.parts) > sc.bytesA || row_scan_scratch(n_pad, b.parts) > sc.bytesB)
        return hipErrorInvalidValue;
    a.mu = mu;
    b.mu = nu;
    return row_scans(a, b, ek, false, tab, status, s);
}

hipError_t launch_row_maxima(const OperandView &va, const OperandView &vb, int ek, int64_t m_pad,
                             int64_t n_pad, uint64_t *maxA, uint64_t *maxB, int32_t *X, int32_t *Y,
                             const ScanScratch &sc, uint32_t *status, hipStream_t s) {
    if (va.rows <= 0 || vb.rows <= 0 || va.k <= 0 || m_pad % kScanRows || n_pad % kScanRows)
        return hipErrorInvalidValue;
    const int64_t groups = (m_pad + n_pad) / kScanRows;
    RowScan a = row_scan_of(va, m_pad, groups, sc.A), b = row_scan_of(vb, n_pad, groups, sc.B);
    if (row_scan_scratch(m_pad, a.parts) > sc.bytesA || row_scan_scratch(n_pad, b.parts) > sc.bytesB)
        return hipErrorInvalidValue;
    a.maxbits = maxA;
    b.maxbits = maxB;
    a.X = X;
    b.X = Y;
    return row_scans(a, b, ek, true, nullptr, status, s);
}

hipError_t launch_pair_fast_exponents(const uint64_t *maxA, const uint64_t *sigA, int64_t m,
                                      int64_t m_pad, int16_t *mu, const uint64_t *maxB,
                                      const uint64_t *sigB, int64_t n, int64_t n_pad, int16_t *nu,
                                      const NTable *tab, uint32_t *status, hipStream_t s) {
    const ExpSide a{maxA, sigA, m, m_pad, m_pad > 0 ? (m_pad + 255) / 256 : 0, mu};
    const ExpSide b{maxB, sigB, n, n_pad, n_pad > 0 ? (n_pad + 255) / 256 : 0, nu};
    const int64_t blocks = a.blocks + b.blocks;
    if (blocks == 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(pair_fast_exponents_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, b, tab,
                       status);
    return hipGetLastError();
}

hipError_t launch_pair_accu_exponents(const AccuSide &a, const AccuSide &b, const NTable *tab,
                                      uint32_t *status, hipStream_t s) {
    const int64_t blkA = (a.rows_pad + 255) / 256, blkB = (b.rows_pad + 255) / 256;
    if (blkA + blkB <= 0) return hipSuccess;
    if (blkA + blkB > INT32_MAX) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(pair_accu_exponents_kernel, dim3((unsigned)(blkA + blkB)), dim3(256), 0, s, a, b,
                       (uint32_t)blkA, tab, status);
    return hipGetLastError();
}

static hipError_t pair_split_ek(const SplitSide &a, const SplitSide &b, bool scan, int threads, int ek,
                                const NTable *tab, int nmod, int nplanes, int abits, int64_t k_pad,
                                uint32_t *status, hipStream_t s) {
    if (abits > kMaxSplitBits) return hipErrorInvalidValue;
    const int nw = split_words(abits);
    if ((nplanes == 1) != elem_real(ek)) return hipErrorInvalidValue;
#define OZC_SPLIT_ARGS a, b, scan, threads, tab, nmod, nw, k_pad, status, s
    switch (ek) {
        case kElemZ: return nplanes == 3 ? pair_split_w<kElemZ, 3>(OZC_SPLIT_ARGS) : pair_split_w<kElemZ, 2>(OZC_SPLIT_ARGS);
        case kElemC: return nplanes == 3 ? pair_split_w<kElemC, 3>(OZC_SPLIT_ARGS) : pair_split_w<kElemC, 2>(OZC_SPLIT_ARGS);
        case kElemD: return pair_split_w<kElemD, 1>(OZC_SPLIT_ARGS);
        case kElemS: return pair_split_w<kElemS, 1>(OZC_SPLIT_ARGS);
        default: return hipErrorInvalidValue;
    }
#undef OZC_SPLIT_ARGS
}

hipError_t launch_pair_split(const OperandView &va, const OperandView &vb, int ek, const int16_t *mu,
                             const int16_t *nu, const NTable *tab, int nmod, int nplanes, int abits,
                             int8_t *resA, int64_t m_pad, int8_t *resB, int64_t n_pad, int64_t k_pad,
                             uint32_t *status, hipStream_t s) {
    if (m_pad % kDirectRows || n_pad % kDirectRows || k_pad % kTileH) return hipErrorInvalidValue;
    const int64_t blkA = batch_split_blocks(m_pad, k_pad), blkB = batch_split_blocks(n_pad, k_pad);
    if (blkA + blkB > INT32_MAX) return hipErrorInvalidConfiguration;
    const SplitSide a{va, mu, resA, m_pad, (uint32_t)blkA, nullptr}, b{vb, nu, resB, n_pad, (uint32_t)blkB, nullptr};
    return pair_split_ek(a, b, false, 256, ek, tab, nmod, nplanes, abits, k_pad, status, s);
}

bool prep_in_one(int64_t k) { return k <= kPrepMaxK; }
hipError_t launch_pair_prep(const OperandView &va, const OperandView &vb, int ek, int16_t *mu, int16_t *nu,
                            const NTable *tab, int nmod, int nplanes, int abits, int8_t *resA,
                            int64_t m_pad, int8_t *resB, int64_t n_pad, int64_t k_pad, uint32_t *status,
                            hipStream_t s) {
    if (va.rows <= 0 || vb.rows <= 0 || va.k <= 0 || va.k > kPrepMaxK || m_pad % kScanRows ||
        n_pad % kScanRows || k_pad % kTileH)
        return hipErrorInvalidValue;
    // 4 rows per block until 16 fill every CU
    const int RB = va.rows + vb.rows >= 16 * 256 ? 16 : 4;
    const int64_t blkA = m_pad / RB, blkB = n_pad / RB;
    if (blkA + blkB > INT32_MAX) return hipErrorInvalidConfiguration;
    const SplitSide a{va, mu, resA, m_pad, (uint32_t)blkA, mu}, b{vb, nu, resB, n_pad, (uint32_t)blkB, nu};
    return pair_split_ek(a, b, true, 64 * RB, ek, tab, nmod, nplanes, abits, k_pad, status, s);
}

hipError_t launch_pair_ceil7(const AccuSide &a, const AccuSide &b, int ek, int64_t k_pad, hipStream_t s) {
    if (a.rows_pad % kTileR || b.rows_pad % kTileR || k_pad % kTileH) return hipErrorInvalidValue;
    const int64_t blkA = batch_ceil7_blocks(a.rows_pad, k_pad), blkB = batch_ceil7_blocks(b.rows_pad, k_pad);
    if (blkA + blkB <= 0) return hipSuccess;
    if (blkA + blkB > INT32_MAX) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(blkA + blkB));
    switch (ek) {
        case kElemZ: hipLaunchKernelGGL(pair_ceil7_kernel<kElemZ>, grid, dim3(256), 0, s, a, b, (uint32_t)blkA, k_pad); break;
        case kElemC: hipLaunchKernelGGL(pair_ceil7_kernel<kElemC>, grid, dim3(256), 0, s, a, b, (uint32_t)blkA, k_pad); break;
        case kElemD: hipLaunchKernelGGL(pair_ceil7_kernel<kElemD>, grid, dim3(256), 0, s, a, b, (uint32_t)blkA, k_pad); break;
        case kElemS: hipLaunchKernelGGL(pair_ceil7_kernel<kElemS>, grid, dim3(256), 0, s, a, b, (uint32_t)blkA, k_pad); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int64_t batch_scan_blocks(const OperandView &v) {
    if (v.rows <= 0 || v.k <= 0) return 0;
    return scan_grid_x(v) * scan_grid_y(v);
}
int64_t batch_exp_blocks(int64_t rows_pad) { return (rows_pad + 255) / 256; }
int64_t batch_split_blocks(int64_t rows_pad, int64_t k_pad) {
    return (k_pad / kTileH) * (rows_pad / kDirectRows);
}

hipError_t launch_batch_scan(const BatchOperand *ops, int nops, int64_t blocks, bool single,
                             bool stats, hipStream_t s) {
    if (blocks <= 0 || nops <= 0) return hipSuccess;
    dim3 grid((unsigned)blocks);
#define OZC_SCAN(EKV, PV) hipLaunchKernelGGL((batch_scan_kernel<EKV, PV>), grid, dim3(256), 0, s, ops, nops)
    if (single) {
        if (stats) OZC_SCAN(kElemC, true);
        else OZC_SCAN(kElemC, false);
    } else {
        if (stats) OZC_SCAN(kElemZ, true);
        else OZC_SCAN(kElemZ, false);
    }
#undef OZC_SCAN
    return hipGetLastError();
}

bool batch_row_scan_plan(BatchOperand &op, int64_t res_bytes) {
    const int64_t parts = row_scan_parts(op.v.k, 0);
    op.scan_parts = (int32_t)parts;
    op.scan_chunk = (op.v.k + parts - 1) / parts;
    return row_scan_scratch(op.rows_pad, parts) <= res_bytes;
}
int64_t batch_row_scan_blocks(const BatchOperand &op) { return op.rows_pad / kScanRows * op.scan_parts; }
int64_t batch_scan_finish_blocks(const BatchOperand &op, bool accurate) {
    const int64_t groups = op.rows_pad / kScanRows;
    return accurate ? scan_finish_blocks<true>(groups, op.scan_parts) : scan_finish_blocks<false>(groups, op.scan_parts);
}

template <int EK, bool ACCU>
static hipError_t batch_row_scan_ek(const BatchOperand *ops, int nops, int64_t blocks, int64_t finish,
                                    uint32_t *status, uint32_t *counters, int ncounters, hipStream_t s) {
    hipLaunchKernelGGL((batch_row_scan_kernel<EK, ACCU>), dim3((unsigned)blocks), dim3(kScanThreads), 0, s,
                       ops, nops, status, counters, ncounters);
    if (finish > 0)
        hipLaunchKernelGGL((batch_scan_finish_kernel<EK, ACCU>), dim3((unsigned)finish), dim3(256), 0, s,
                           ops, nops);
    return hipGetLastError();
}
hipError_t launch_batch_row_scan(const BatchOperand *ops, int nops, int64_t blocks, int64_t finish,
                                 bool single, bool accurate, uint32_t *status, uint32_t *counters,
                                 int ncounters, hipStream_t s) {
    if (blocks <= 0 || nops <= 0 || ncounters > kScanThreads) return hipErrorInvalidValue;
#define OZC_ARGS ops, nops, blocks, finish, status, counters, ncounters, s
    if (single) return accurate ? batch_row_scan_ek<kElemC, true>(OZC_ARGS) : batch_row_scan_ek<kElemC, false>(OZC_ARGS);
    return accurate ? batch_row_scan_ek<kElemZ, true>(OZC_ARGS) : batch_row_scan_ek<kElemZ, false>(OZC_ARGS);
#undef OZC_ARGS
}

hipError_t launch_batch_accu_exponents(const BatchOperand *ops, int nops, int64_t blocks,
                                       uint32_t *status, hipStream_t s) {
    if (blocks <= 0 || nops <= 0) return hipSuccess;
    hipLaunchKernelGGL(batch_accu_exponents_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ops, nops,
                       status);
    return hipGetLastError();
}

int64_t batch_ceil7_blocks(int64_t rows_pad, int64_t k_pad) {
    return (k_pad / kTileH) * (rows_pad / kTileR);
}

hipError_t launch_batch_ceil7(const BatchOperand *ops, int nops, int64_t blocks, bool single,
                              hipStream_t s) {
    if (blocks <= 0 || nops <= 0) return hipSuccess;
    if (single) hipLaunchKernelGGL((batch_ceil7_kernel<true>), dim3((unsigned)blocks), dim3(256), 0, s, ops, nops);
    else hipLaunchKernelGGL((batch_ceil7_kernel<false>), dim3((unsigned)blocks), dim3(256), 0, s, ops, nops);
    return hipGetLastError();
}

hipError_t launch_batch_split(const BatchOperand *ops, int nops, int64_t blocks, bool single,
                              int nplanes, int abits, uint32_t *status, hipStream_t s) {
    if (blocks <= 0 || nops <= 0) return hipSuccess;
    if (abits > kMaxSplitBits) return hipErrorInvalidValue;
    const int nw = split_words(abits);
    if (single)
        return nplanes == 3 ? batch_split_w<kElemC, 3>(ops, nops, blocks, nw, status, s)
                            : batch_split_w<kElemC, 2>(ops, nops, blocks, nw, status, s);
    return nplanes == 3 ? batch_split_w<kElemZ, 3>(ops, nops, blocks, nw, status, s)
                        : batch_split_w<kElemZ, 2>(ops, nops, blocks, nw, status, s);
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

}  // namespace ozc
