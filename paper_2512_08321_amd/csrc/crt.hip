// CRT reconstruction, inverse scaling and alpha/beta (Algorithm 1 Steps
// V-v, V-vi and VI).
//
// For every output entry and each of the real and imaginary parts the kernel
// forms S = sum_l s_l E'_l with s_l = (P/p_l) q_l, reduces C' = mod(S, P)
// into [-P/2, P/2) and rounds C' to the nearest double (ties to even), then
// scales by 2^-(mu_i + nu_j).  The paper evaluates S as an unevaluated sum
// of two doubles and reduces it in double-double arithmetic (Section II,
// equation (5); Section IV-A); here S is accumulated exactly as 38-bit chunks
// in FP64 (s_l split into 38-bit chunks, every partial sum an integer below
// kMaxPartSum * 2^38 * 2^7 < 2^52), and reduced mod P on the same chunks, which removes
// the reconstruction error altogether and makes the output bit-reproducible
// against an exact reference; C' is rounded once, by error-free sums of its chunks (the
// double-double output and rare values: as a 256-bit integer).
#include "internal.h"

namespace ozc {
namespace {

using ConstTab = const OZC_AS_CONST NTable *;

// The reduction works on the 38-bit chunks of S held in FP64: every value it
// forms is an integer below 2^53, so every operation below is exact.  Bounds, with
// E = kMaxPartSum = 96 terms s_l E'_l at most (one per modulus and part, |E'_l| <= 2^7):
// |S| < 2^7 E P, |r_c| < 2^7 E 2^38 < 2^52 for a chunk of S, |q| <= 2^7 E + 1 < 2^14 for
// the quotient, so |q P_c| < (2^7 E + 1) 2^38 and |r_c - q P_c| < (2^8 E + 1) 2^38 < 2^53.
constexpr double kChunk = (double)(1ull << kChunkBits);   // 2^38
static_assert(kMaxModuli <= kMaxPartSum, "one term per modulus at least");
static_assert(((256ull * kMaxPartSum + 2) << kChunkBits) < (1ull << 53), "exact in FP64, a carry included");
constexpr double kInvChunk = 1.0 / kChunk;                 // 2^-38, exact

// Chunks 0 .. C-2 into [0, 2^38), the carries into the top chunk (which keeps the sign).
template <int C>
__device__ __forceinline__ void normalize(double (&r)[C]) {
#pragma unroll
    for (int c = 0; c < C - 1; ++c) {
        const double f = floor(r[c] * kInvChunk);
        r[c] = fma(-f, kChunk, r[c]);
        r[c + 1] += f;
    }
}

// After normalize(): value >= 0  <=>  top chunk >= 0.  Brings R into [-P/2, P/2)
// when the quotient estimate was one off.
template <int C>
__device__ __forceinline__ void settle_range(double (&r)[C], ConstTab tab) {
    double t[C];
#pragma unroll
    for (int c = 0; c < C; ++c) t[c] = 2.0 * r[c] - tab->Pchunk[c];
    normalize<C>(t);
    if (t[C - 1] >= 0.0) {  // 2R >= P
#pragma unroll
        for (int c = 0; c < C; ++c) r[c] -= tab->Pchunk[c];
        normalize<C>(r);
        return;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) t[c] = 2.0 * r[c] + tab->Pchunk[c];
    normalize<C>(t);
    if (t[C - 1] < 0.0) {  // 2R < -P
#pragma unroll
        for (int c = 0; c < C; ++c) r[c] += tab->Pchunk[c];
        normalize<C>(r);
    }
}

// A 256-bit magnitude w (little-endian words) rounded to nearest-even as d * 2^sh.
__device__ __forceinline__ double round_w4(const uint64_t (&w)[4], int &sh) {
    if ((w[1] | w[2] | w[3]) == 0) {
        sh = 0;
        return (double)w[0];  // exact when < 2^53, otherwise one correct rounding
    }
    const int wi = w[3] ? 3 : (w[2] ? 2 : 1);
    const uint64_t top = wi == 3 ? w[3] : (wi == 2 ? w[2] : w[1]);
    const uint64_t below = wi == 3 ? w[2] : (wi == 2 ? w[1] : w[0]);
    uint64_t rest = wi == 3 ? (w[1] | w[0]) : (wi == 2 ? w[0] : 0);
    const int nb = 64 - __clzll((long long)top);  // 1..64
    uint64_t W;
    if (nb == 64) {
        W = top;
        rest |= below;
    } else {
        W = (top << (64 - nb)) | (below >> nb);
        rest |= below << (64 - nb);
    }
    W |= (rest != 0) ? 1ull : 0ull;  // sticky bit below the rounding position
    sh = 64 * (wi - 1) + nb;
    return (double)W;
}

// w - d 2^sh for the rounded value d 2^sh of w (|difference| <= half an ulp of d):
// the magnitude of the difference into r, its sign as the return value (true: negative).
__device__ __forceinline__ bool rounding_residual(const uint64_t (&w)[4], double d, int sh,
                                                  uint64_t (&r)[4]) {
    const uint64_t bits = (uint64_t)__double_as_longlong(d);
    const uint64_t M = (bits & ((1ull << 52) - 1)) | (1ull << 52);
    const int s = (int)(bits >> 52) - 1075 + sh;  // d 2^sh = M 2^s, s >= 0 when d is inexact
    uint64_t h[4] = {0, 0, 0, 0};
    const int q = s >> 6, o = s & 63;
    if (q < 4) h[q] = M << o;
    if (o && q + 1 < 4) h[q + 1] = M >> (64 - o);
    uint64_t borrow = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint64_t x = w[j], y = h[j];
        const uint64_t t = x - y;
        const uint64_t b2 = (x < y) ? 1ull : 0ull;
        r[j] = t - borrow;
        borrow = b2 | ((t < borrow) ? 1ull : 0ull);
    }
    if (!borrow) return false;
    uint64_t c = 1;  // negate the two's complement
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        r[j] = ~r[j] + c;
        c = (c && r[j] == 0) ? 1ull : 0ull;
    }
    return true;
}

// mod(S, P) rounded to nearest-even as d * 2^sh; S given as C unnormalised 38-bit
// chunks in FP64 (|r_c| < 2^52).  With low (and shl) non-null, also the rounding
// residual mod(S, P) - d 2^sh rounded to nearest-even as *low * 2^shl (0 when d is
// exact), for double-double outputs.
// The quotient q = rint(S / P) comes from the chunks' Horner sum times fl(1/P) (error
// far below 2^-20, since |S| < 2^7 E P); R = S - q P chunk by chunk (|q P_c| < 2^52,
// exact); a quotient within 2^-20 of a tie is checked exactly (settle_range).  |R| then
// goes to a 256-bit integer for the rounding.
template <int C>
__device__ __forceinline__ double reconstruct(double (&r)[C], ConstTab tab, int &sh,
                                              double *low = nullptr, int *shl = nullptr) {
    double sa = r[C - 1];
#pragma unroll
    for (int c = C - 2; c >= 0; --c) sa = fma(sa, kChunk, r[c]);
    const double x = sa * tab->inv_P;  // ~ S / P
    const double qd = rint(x);         // |q| < 2^14
#pragma unroll
    for (int c = 0; c < C; ++c) r[c] = fma(-qd, tab->Pchunk[c], r[c]);
    normalize<C>(r);
    if (fabs(x - qd) > 0.5 - 1.0 / 1048576.0) settle_range<C>(r, tab);

    const bool neg = r[C - 1] < 0.0;
    if (neg) {
#pragma unroll
        for (int c = 0; c < C; ++c) r[c] = -r[c];
        normalize<C>(r);
    }
    // chunk c (in [0, 2^38), the top one too since |R| < P / 2) at bit 38 c
    uint64_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double hi = floor(r[c] * 0x1p-32);
        const uint32_t lo32 = (uint32_t)fma(-hi, 0x1p32, r[c]);
        const uint64_t v = ((uint64_t)(uint32_t)hi << 32) | lo32;
        const int o = kChunkBits * c;
        w[o >> 6] |= v << (o & 63);
        if ((o & 63) + kChunkBits > 64) w[(o >> 6) + 1] |= v >> (64 - (o & 63));
    }
    const double d = round_w4(w, sh);
    if (low) {
        *low = 0.0;
        *shl = 0;
        const bool exact = (w[1] | w[2] | w[3]) == 0 && w[0] < (1ull << 53);
        if (!exact) {
            uint64_t rr[4];
            const bool rneg = rounding_residual(w, d, sh, rr);
            const double e = round_w4(rr, *shl);
            *low = e == 0.0 ? 0.0 : ((rneg != neg) ? -e : e);  // a zero residual is +0
        }
    }
    return neg ? -d : d;
}

// a + b = s + e exactly (Knuth).
__device__ __forceinline__ double two_sum(double a, double b, double &e) {
    const double s = a + b, t = s - a;
    e = (a - (s - t)) + (b - t);
    return s;
}

// a + b + c rounded once to nearest-even (Boldo and Melquiond, "Emulation of a FMA and
// correctly rounded sums: proved algorithms using rounding to odd", 2008): the low parts of
// two error-free sums are added with rounding to odd, which the last addition cannot mistake
// for a tie.
__device__ __forceinline__ double sum3(double a, double b, double c) {
    double ul, tl, ve;
    const double uh = two_sum(b, c, ul);
    const double th = two_sum(a, uh, tl);
    const double v = two_sum(tl, ul, ve);
    int64_t vb = __double_as_longlong(v);
    // inexact and even: one step towards the error, to the odd neighbour
    if (ve != 0.0 && (vb & 1) == 0) vb += (ve > 0.0) == (v > 0.0) ? 1 : -1;
    return th + __longlong_as_double(vb);
}

// reconstruct() without the residual, straight from the chunks: the quotient as there, then
// the chunks' sum rounded once.  Two chunks: a fused multiply-add.  Three: sum3.  More: the
// low chunks are normalised and all below the third from the top only set its last bit
// (rounding to odd), which is far below the rounding position unless the top two nearly
// cancel; those rare values take reconstruct().  The 256-bit integer rounding takes about
// 80 instructions per value, sum3 about 25, the fused multiply-add one.  Reconstructions of
// 4096^2 outputs with it and the loads ahead: CGEMM at N = 6 104 -> 86 us (3.9 TB/s), DGEMM
// at N = 14 131 -> 99 us (3.7 TB/s), ZGEMM at N = 14 206 -> 186..198, at N = 24 326 -> 290 us.
template <int C>
__device__ __forceinline__ double reconstruct_fast(double (&r)[C], ConstTab tab, int &sh) {
    double sa = r[C - 1];
#pragma unroll
    for (int c = C - 2; c >= 0; --c) sa = fma(sa, kChunk, r[c]);
    const double x = sa * tab->inv_P;
    const double qd = rint(x);
    if (fabs(x - qd) > 0.5 - 1.0 / 1048576.0) return reconstruct<C>(r, tab, sh);
    double t[C];
#pragma unroll
    for (int c = 0; c < C; ++c) t[c] = fma(-qd, tab->Pchunk[c], r[c]);
    if constexpr (C == 1) {
        sh = 0;
        return t[0];
    } else if constexpr (C == 2) {
        sh = 0;
        return fma(t[1], kChunk, t[0]);
    } else if constexpr (C == 3) {
        sh = kChunkBits;
        return sum3(t[2] * kChunk, t[1], t[0] * kInvChunk);
    } else {
        bool rest = false;
#pragma unroll
        for (int c = 0; c < C - 2; ++c) {
            const double f = floor(t[c] * kInvChunk);
            t[c] = fma(-f, kChunk, t[c]);  // in [0, 2^38)
            t[c + 1] += f;
            if (c < C - 3) rest = rest || t[c] != 0.0;
        }
        // t[C-3] + (something in (0, 1)) to odd
        if (rest) t[C - 3] = fma(2.0, floor(t[C - 3] * 0.5), 1.0);
        const double a = t[C - 1] * kChunk;
        if (fabs(a + t[C - 2]) < 0x1p20) return reconstruct<C>(r, tab, sh);
        sh = kChunkBits * (C - 2);
        return sum3(a, t[C - 2], t[C - 3] * kInvChunk);
    }
}

__device__ __forceinline__ void alpha_beta(double cr, double ci, double ar, double ai, double br,
                                           double bi, bool beta_zero, double Cr, double Ci,
                                           double &orr, double &oi) {
    const double xr = fma(ar, cr, -(ai * ci));
    const double xi = fma(ar, ci, ai * cr);
    if (beta_zero) {
        orr = xr;
        oi = xi;
    } else {
        orr = fma(br, Cr, fma(-bi, Ci, xr));
        oi = fma(br, Ci, fma(bi, Cr, xi));
    }
}

// C elements of kind EK (ElemKind); real elements carry no imaginary part.
typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec2 __attribute__((ext_vector_type(2)));

template <int EK>
__device__ __forceinline__ void load_c(const void *C, int64_t idx, double &re, double &im) {
    if constexpr (EK == kElemC) {
        const fvec2 v = global_ptr(reinterpret_cast<const fvec2 *>(C))[idx];
        re = v.x;
        im = v.y;
    } else if constexpr (EK == kElemZ) {
        const dvec2 v = global_ptr(reinterpret_cast<const dvec2 *>(C))[idx];
        re = v.x;
        im = v.y;
    } else if constexpr (EK == kElemD) {
        re = global_ptr(reinterpret_cast<const double *>(C))[idx];
        im = 0.0;
    } else {
        re = global_ptr(reinterpret_cast<const float *>(C))[idx];
        im = 0.0;
    }
}

template <int EK>
__device__ __forceinline__ void store_c(void *C, int64_t idx, double re, double im) {
    if constexpr (EK == kElemC) global_ptr(reinterpret_cast<fvec2 *>(C))[idx] = fvec2{(float)re, (float)im};
    else if constexpr (EK == kElemZ) global_ptr(reinterpret_cast<dvec2 *>(C))[idx] = dvec2{re, im};
    else if constexpr (EK == kElemD) global_ptr(reinterpret_cast<double *>(C))[idx] = re;
    else global_ptr(reinterpret_cast<float *>(C))[idx] = (float)re;
}

constexpr int kCrtBatch = 4;
static_assert(kMaxModuli % kCrtBatch == 0, "the last batch's weights stay inside the table");

// One thread: 4 consecutive rows i of one column j; block bx covers threads
// 256 bx ... 256 bx + 255 of the ceil(m / 4) x n grid (padding rows get no thread).
// Real outputs (EK real) reconstruct the one E' plane of each modulus; alpha and beta
// are real then (imaginary parts zero), so the fused multiply-add order below reduces
// to x = alpha c, out = fma(beta, C, x).
template <int C, int EK, bool DD = false, bool PARTS = false>
__device__ __forceinline__ void crt_output_body(const CrtArgs &a, int64_t bx) {
    constexpr bool REAL = elem_real(EK);
    constexpr int EPL = REAL ? 1 : 2;  // E' planes per modulus
    // below 2^32 threads unless the output has 2^34 elements
    const int64_t m4 = (a.m + 3) >> 2;
    const int64_t t = bx * 256 + threadIdx.x;
    const int64_t j = (uint64_t)(m4 | (bx * 256 + 255)) >> 32 ? t / m4 : (int64_t)((uint32_t)t / (uint32_t)m4);
    const int64_t ib = (t - j * m4) * 4;
    if (j >= a.n || ib >= a.m) return;

    const int64_t planeC = a.n_pad * a.m_pad;
    // S = sum_l s_l E'_l in 38-bit chunks: |partial sums| < kMaxPartSum 2^38 2^7 < 2^52,
    // every fused multiply-add exact
    double accR[4][C], accI[4][C];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) accR[u][c] = accI[u][c] = 0.0;

    ConstTab tab = const_ptr(a.tab);
    const OZC_AS_GLOBAL int8_t *E = global_ptr(a.eprime) + j * a.m_pad + ib;
    auto add = [&](const double (&sc)[C], const double (&er)[4], const double (&ei)[4]) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                accR[u][c] = fma(sc[c], er[u], accR[u][c]);
                if constexpr (!REAL) accI[u][c] = fma(sc[c], ei[u], accI[u][c]);
            }
        }
    };
    // The E' of every modulus, then the further parts of the moduli from l_split on (their
    // products were cut along k: the parts' residues add up).  In batches: the next batch's
    // words and this one's weights are loaded before the sums.  A batch that runs past the
    // last entry reads that one again and adds nothing.
    const int entries = a.nmod + (PARTS ? (a.nmod - a.l_split) * (a.parts - 1) : 0);
    const OZC_AS_GLOBAL int8_t *E2 = PARTS ? global_ptr(a.eprime_parts) + j * a.m_pad + ib : nullptr;
    uint32_t wr[kCrtBatch], wi[kCrtBatch];
    auto load = [&](int e0) {
#pragma unroll
        for (int q = 0; q < kCrtBatch; ++q) {
            const int e = min(e0 + q, entries - 1);
            const OZC_AS_GLOBAL int8_t *p = !PARTS || e < a.nmod ? E + (int64_t)(EPL * e) * planeC
                                                                 : E2 + (int64_t)(EPL * (e - a.nmod)) * planeC;
            wr[q] = *reinterpret_cast<const OZC_AS_GLOBAL uint32_t *>(p);
            wi[q] = REAL ? 0u : *reinterpret_cast<const OZC_AS_GLOBAL uint32_t *>(p + planeC);
        }
    };
    // The exponents: with the first loads, except at five chunks, where their registers cost a
    // wave of occupancy (267 against 260 us at N = 20); before any store of C in any case.
    const bool beta_zero = a.beta_r == 0.0 && a.beta_i == 0.0;
    int nuj, mus[4];
    auto exponents = [&]() {
        nuj = global_ptr(a.nu)[j];
#pragma unroll
        for (int u = 0; u < 4; ++u) mus[u] = ib + u < a.m ? global_ptr(a.mu)[ib + u] : 0;
        if (a.status && nuj == kExpNonfinite && ib == 0) atomicOr(a.status, 1u);
    };
    if constexpr (C < 5) exponents();
    load(0);
    int l = 0;  // PARTS: modulus of the entry
    for (int e0 = 0; e0 < entries; e0 += kCrtBatch) {
        uint32_t cr[kCrtBatch], ci[kCrtBatch];
        double sc[kCrtBatch][C];
#pragma unroll
        for (int q = 0; q < kCrtBatch; ++q) {
            cr[q] = wr[q];
            ci[q] = wi[q];
#pragma unroll
            for (int c = 0; c < C; ++c) sc[q][c] = tab->mod[PARTS ? l : e0 + q].schunk[c];
            if constexpr (PARTS) l = l + 1 < a.nmod ? l + 1 : a.l_split;
        }
        if (e0 + kCrtBatch < entries) load(e0 + kCrtBatch);
#pragma unroll
        for (int q = 0; q < kCrtBatch; ++q) {
            if (e0 + q >= entries) break;
            double er[4], ei[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                er[u] = (double)(int)(int8_t)(cr[q] >> (8 * u));
                ei[u] = (double)(int)(int8_t)(ci[q] >> (8 * u));
            }
            add(sc[q], er, ei);
        }
    }

    if constexpr (C >= 5) exponents();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = ib + u;
        if (i >= a.m) continue;
        const int mui = mus[u];
        if (a.status && mui == kExpNonfinite && j == 0) atomicOr(a.status, 1u);
        double cr, ci;
        double lr = 0.0, li = 0.0;  // double-double outputs: the low parts
        if (mui == kExpNonfinite || nuj == kExpNonfinite) {
            cr = ci = __builtin_nan("");
            lr = li = cr;
        } else if (mui == kExpZero || nuj == kExpZero) {
            cr = ci = 0.0;
        } else if constexpr (DD) {
            int shr, shi, slr, sli;
            double er, ei;
            const double dr = reconstruct<C>(accR[u], tab, shr, &er, &slr);
            const double di = reconstruct<C>(accI[u], tab, shi, &ei, &sli);
            cr = ldexp(dr, shr - (mui + nuj));
            ci = ldexp(di, shi - (mui + nuj));
            lr = ldexp(er, slr - (mui + nuj));
            li = ldexp(ei, sli - (mui + nuj));
        } else {
            int shr, shi = 0;
            const double dr = reconstruct_fast<C>(accR[u], tab, shr);
            const double di = REAL ? 0.0 : reconstruct_fast<C>(accI[u], tab, shi);
            cr = ldexp(dr, shr - (mui + nuj));
            ci = REAL ? 0.0 : ldexp(di, shi - (mui + nuj));
        }
        const int64_t idx = j * a.ldc + i;
        if constexpr (DD) {  // alpha = 1, beta = 0: the two parts as they are
            global_ptr(reinterpret_cast<dvec2 *>(a.C))[idx] = dvec2{cr, ci};
            global_ptr(reinterpret_cast<dvec2 *>(a.C_lo))[idx] = dvec2{lr, li};
            continue;
        }
        double Cr = 0.0, Ci = 0.0;
        if (!beta_zero) load_c<EK>(a.C, idx, Cr, Ci);
        double orr, oi;
        alpha_beta(cr, ci, a.alpha_r, a.alpha_i, a.beta_r, a.beta_i, beta_zero, Cr, Ci, orr, oi);
        store_c<EK>(a.C, idx, orr, oi);
    }
}

template <int C, int EK, bool PARTS>
__global__ __launch_bounds__(256) void crt_output_kernel(CrtArgs a) {
    crt_output_body<C, EK, false, PARTS>(a, blockIdx.x);
}

template <int C>
__global__ __launch_bounds__(256) void crt_dd_kernel(CrtArgs a) {
    crt_output_body<C, kElemZ, true>(a, blockIdx.x);
}

template <int C, bool SINGLE>
__global__ __launch_bounds__(256) void batch_crt_kernel(const BatchCrt *probs, int nprob) {
    const int64_t b = blockIdx.x;
    int lo = 0, hi = nprob - 1;  // last problem whose first block is <= b
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (probs[mid].blk0 <= b) lo = mid;
        else hi = mid - 1;
    }
    // The problem's arguments are copied out of the list first: read through a reference
    // into global memory, every field would be loaded again after each store of C (the
    // compiler cannot rule out that the stores overwrite the list).
    const CrtArgs a = probs[lo].a;
    crt_output_body<C, SINGLE>(a, b - probs[lo].blk0);
}

template <int C>
hipError_t launch_batch_C(const BatchCrt *probs, int nprob, int64_t blocks, bool single, hipStream_t s) {
    dim3 grid((unsigned)blocks);
    if (single) hipLaunchKernelGGL((batch_crt_kernel<C, true>), grid, dim3(256), 0, s, probs, nprob);
    else hipLaunchKernelGGL((batch_crt_kernel<C, false>), grid, dim3(256), 0, s, probs, nprob);
    return hipGetLastError();
}

// C := alpha * 0 + beta * C (alpha == 0 or k == 0), with the same operation order.
template <int EK>
__global__ void scale_c_kernel(void *C, int64_t m, int64_t n, int64_t ldc, double ar, double ai,
                               double br, double bi) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m * n) return;
    const int64_t i = t % m, j = t / m;
    const bool beta_zero = br == 0.0 && bi == 0.0;
    double Cr = 0.0, Ci = 0.0;
    if (!beta_zero) load_c<EK>(C, j * ldc + i, Cr, Ci);
    double orr, oi;
    alpha_beta(0.0, 0.0, ar, ai, br, bi, beta_zero, Cr, Ci, orr, oi);
    store_c<EK>(C, j * ldc + i, orr, oi);
}

template <int C>
hipError_t launch_C(const CrtArgs &a, hipStream_t s) {
    const int64_t threads = ((a.m + 3) / 4) * a.n;
    dim3 grid((unsigned)((threads + 255) / 256));
    const bool parts = a.parts > 1 && a.l_split < a.nmod;
    if (a.C_lo) {
        if (a.ek != kElemZ || parts) return hipErrorInvalidValue;
        hipLaunchKernelGGL((crt_dd_kernel<C>), grid, dim3(256), 0, s, a);
        return hipGetLastError();
    }
#define OZC_CRT(EKV)                                                                                     \
    case EKV:                                                                                            \
        if (parts) hipLaunchKernelGGL((crt_output_kernel<C, EKV, true>), grid, dim3(256), 0, s, a);      \
        else hipLaunchKernelGGL((crt_output_kernel<C, EKV, false>), grid, dim3(256), 0, s, a);           \
        break;
    switch (a.ek) {
        OZC_CRT(kElemZ)
        OZC_CRT(kElemC)
        OZC_CRT(kElemD)
        OZC_CRT(kElemS)
        default: return hipErrorInvalidValue;
    }
#undef OZC_CRT
    return hipGetLastError();
}

}  // namespace

hipError_t launch_crt_output(const CrtArgs &a, hipStream_t s) {
    if (a.m <= 0 || a.n <= 0) return hipSuccess;
    if (a.m_pad % 4 || a.nmod < 1 || a.l_split < 0 || a.l_split > a.nmod || a.parts < 1 ||
        a.l_split + (a.nmod - a.l_split) * a.parts > kMaxPartSum)
        return hipErrorInvalidValue;
    switch (a.nchunks) {
        case 1: return launch_C<1>(a, s);
        case 2: return launch_C<2>(a, s);
        case 3: return launch_C<3>(a, s);
        case 4: return launch_C<4>(a, s);
        case 5: return launch_C<5>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_scale_c(void *C, int64_t m, int64_t n, int64_t ldc, int ek, double ar,
                          double ai, double br, double bi, hipStream_t s) {
    if (m <= 0 || n <= 0) return hipSuccess;
    dim3 grid((unsigned)((m * n + 255) / 256));
    switch (ek) {
        case kElemZ: hipLaunchKernelGGL(scale_c_kernel<kElemZ>, grid, dim3(256), 0, s, C, m, n, ldc, ar, ai, br, bi); break;
        case kElemC: hipLaunchKernelGGL(scale_c_kernel<kElemC>, grid, dim3(256), 0, s, C, m, n, ldc, ar, ai, br, bi); break;
        case kElemD: hipLaunchKernelGGL(scale_c_kernel<kElemD>, grid, dim3(256), 0, s, C, m, n, ldc, ar, ai, br, bi); break;
        case kElemS: hipLaunchKernelGGL(scale_c_kernel<kElemS>, grid, dim3(256), 0, s, C, m, n, ldc, ar, ai, br, bi); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int64_t batch_crt_blocks(int64_t m, int64_t n) { return (((m + 3) / 4) * n + 255) / 256; }

hipError_t launch_batch_crt(const BatchCrt *probs, int nprob, int64_t blocks, int nchunks,
                            bool single, hipStream_t s) {
    if (blocks <= 0 || nprob <= 0) return hipSuccess;
    switch (nchunks) {
        case 1: return launch_batch_C<1>(probs, nprob, blocks, single, s);
        case 2: return launch_batch_C<2>(probs, nprob, blocks, single, s);
        case 3: return launch_batch_C<3>(probs, nprob, blocks, single, s);
        case 4: return launch_batch_C<4>(probs, nprob, blocks, single, s);
        case 5: return launch_batch_C<5>(probs, nprob, blocks, single, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ozc
