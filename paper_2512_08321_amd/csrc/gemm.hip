// Per-modulus complex INT8 products on the gfx950 matrix cores with INT32
// accumulation (Section III-A; Algorithm 1 Step V-iii/iv).
//
// One block computes a TM x TN output tile of one modulus l with WM x WN
// waves; each wave owns (BM*16) x (BN*16) outputs as BM x BN blocks of
// v_mfma_i32_16x16x64_i8 (large problems: 256 x 256 tiles, 8 waves of
// 128 x 64, two waves per SIMD; small problems: 128 x 128, 4 waves of
// 64 x 64; calls that leave CUs idle: 64 x 64, 4 waves of 64 x 16).  The products of the chosen algorithm run one after another over
// the same tile, each as a k-loop over a ring of LDS buffers that the load
// units fill straight from global memory a few 64-wide k-slabs ahead of the
// matrix cores (one barrier per k-slab).  Between products
// the INT32 accumulators are reduced to symmetric residues in registers; one
// packed INT8 carry per output survives to the next product, and E'_R, E'_I
// are stored as soon as they are final, so only INT8 data leaves the chip:
//   Karatsuba (eq. (10)): D = R.R, E = I.I, F = S.S (S = reduced R + I):
//                         E'_R = mod(D - E), E'_I = mod(F - mod(D + E))
//   expanded  (eq. (7)):  E'_R = mod(RR - II), E'_I = mod(RI + IR)
// A third plan computes the accurate-mode bound product (Section III-B):
//   Cbar_I = Abar_I Bbar_R + Abar_R Bbar_I, Cbar_R = Cbar_I + (Abar_R - Abar_I)(Bbar_R - Bbar_I),
// folded on the fly into row and column maxima (Cbar is never stored).
// Real matrices (Algorithm 1 as stated for real A, B) take one product per
// modulus, E' = mod(A'_l B'_l), and one real bound product Abar Bbar.
//
// Block order: block ids are dealt round-robin to the 8 XCDs; ids are
// remapped so that each XCD walks its own contiguous part of the
// (modulus, tile) sequence, tiles grouped 4 rows at a time, so that the
// blocks resident on one XCD share A and B panels in that XCD's L2.
//
// MFMA operand layout: lane l of a 16x16x64 instruction supplies 16 bytes of
// row (l mod 16) of the A block and of column (l mod 16) of the B block, at
// k-offset 16 * (l / 16); both operands use the same k assignment, so the
// product does not depend on how the hardware orders k inside the 64-wide
// step.  Accumulator register r of lane l holds row 4(l/16) + r, column
// (l mod 16).
#include <algorithm>
#include <cmath>
#include <utility>

#include "acc_math.h"
#include "internal.h"

namespace ozc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int BK = 64;

enum { KIND_KARATSUBA = 0, KIND_4M = 1, KIND_BOUND = 2, KIND_REAL = 3, KIND_BOUND_REAL = 4 };

// Products of each plan as (A plane, B plane) pairs, in execution order.
template <int KIND>
struct Plan {
    static constexpr bool real = KIND == KIND_REAL || KIND == KIND_BOUND_REAL;
    static constexpr bool bound = KIND == KIND_BOUND || KIND == KIND_BOUND_REAL;
    static constexpr int nseg = real ? 1 : (KIND == KIND_4M ? 4 : 3);
    static constexpr int nplanes = real ? 1 : (KIND == KIND_4M ? 2 : 3);
    static constexpr int eplanes = real ? 1 : 2;  // E' planes per modulus
    // Karatsuba: RR, II, SS.  Expanded: RR, II, RI, IR.  Bound: I.R, R.I, D.D (D = R - I).
    // Real products and the real bound: the one product R.R.
    __device__ static constexpr int pa(int s) {
        return KIND == KIND_BOUND ? (s == 0 ? 1 : (s == 1 ? 0 : 2)) : (KIND == KIND_4M ? (s & 1) : s);
    }
    __device__ static constexpr int pb(int s) {
        return KIND == KIND_4M ? (s == 2 ? 1 : (s == 3 ? 0 : s)) : s;
    }
};

// s + 128 of the symmetric residue s of an INT32 value x, an accumulator or an accumulator
// plus or minus residues, given as v = x + 2^31 modulo 2^32 (accumulators start at 2^31).
// As in the residue split, one byte dot product gives x' = sum_j v_j (2^(8 j) mod p) + 128 -
// (2^31 mod p), congruent to x + 128 and below 2^20 in magnitude, and the rest is exact in
// FP32: s + 128 = x' - p floor(fl(x' fl(1/p) + 0.5 - 128 fl(1/p))).  x stays in INT32: an
// accumulator is bounded by k 127^2 (odd p; k <= 2^17) and the residues added to it (at
// most three times 127) keep it below 2^31 - p; for p = 256 the wrap-around modulo 2^32
// leaves the byte unchanged.
// Six instructions per output with the packing of four residues into a word; the epilogue
// is bound by them where k is short.  The rule before, rint(x (1/p)) in FP64, took five FP64
// ones and two more to pack, and E' went out in 4-byte stores; products then and now, same
// card: ZGEMM 4096^3 at N = 14 2505 -> 2377 us, 4096 x 4096 x 128 435 -> 301 us, DGEMM 1536 x
// 2048 x 1000 75 -> 57 us, SGEMM 3000 x 3000 x 700 at N = 8 102 -> 70 us.
struct ModRule {
    uint32_t wb, bias;
    float p, ip, rb;
};
__device__ __forceinline__ ModRule mod_rule(const NTable *tab, int l) {
    const OZC_AS_CONST ModConst &mc = const_ptr(tab)->mod[l];
    return ModRule{mc.wbyte[0], mc.wbias[0], mc.pf, mc.ipf, mc.rbias};
}
template <int U>
__device__ __forceinline__ uint32_t put_residue(uint32_t v, const ModRule &r, uint32_t w) {
    const float x = (float)(int32_t)__builtin_amdgcn_udot4(v, r.wb, r.bias, false);
    const float s = __builtin_fmaf(-__builtin_floorf(__builtin_fmaf(x, r.ip, r.rb)), r.p, x);
    return __builtin_amdgcn_cvt_pk_u8_f32(s, U, w);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int byte_of(uint32_t w, int u) { return (int)(int8_t)(w >> (8 * u)); }

// The 64 rows (or columns) of a group of four 16 x 16 blocks are dealt to the blocks so that a
// lane ends up with 16 consecutive rows of its column: matrix row x of block t is row
// 16 (x / 4) + 4 t + x mod 4 of the group.  A lane's accumulators of the four blocks (rows
// 4 (lane / 16) + 0..3 of each) are then rows 16 (lane / 16) + 0..15, in order, and E' moves in
// 16-byte accesses without any exchange between lanes.
__device__ __forceinline__ int group_row(int x) { return 16 * (x >> 2) + (x & 3); }

// LDS tile layout: 64-byte rows of four 16-byte granules; granule g of row r is stored at
// position g ^ sw(r), sw(r) = r5 | (r4 ^ r5 ^ r1) << 1 (ri = bit i of r).  A fragment read takes
// granule lane / 16 of row group_row(lane mod 16) + 4 t.  128-bit reads are served sixteen
// lanes at a time, lanes 0-3, 12-15, 20-23 and 24-27 together, then 4-7, 8-11, 16-19 and 28-31,
// and the same 32 lanes up: each sixteen hit distinct groups of banks (counters: no conflicts;
// r4 | (r5 ^ r1) << 1, which only tells consecutive lanes apart, has four cycles per read).
__device__ __forceinline__ int swz_bits(int row) {
    const int b = row >> 5;
    return (b & 1) | (((b ^ (row >> 4) ^ (row >> 1)) & 1) << 1);
}

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0..N-1, so that
// register arrays are only ever indexed by constants.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// A wave-uniform value into a scalar register: integer divisions leave theirs in vector
// registers, and with it every address computed from it.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ void map_tile(uint32_t L, uint32_t TR, uint32_t TC, uint32_t total, int &l,
                                         int64_t &ti, int64_t &tj) {
    // XCD x (blocks x, x + 8, ...) -> contiguous part x of total / 8 tiles, one more in the
    // first total % 8 parts.  Block counts are below 2^31: 32-bit divisions.
    const uint32_t x = L & 7, rem8 = total & 7;
    const uint32_t q = x * (total >> 3) + min(x, rem8) + (L >> 3);
    const uint32_t T = TR * TC, mod = uniform(q / T);
    l = (int)mod;
    const uint32_t t = q - mod * T;
    constexpr uint32_t G = 4;
    const uint32_t grp = t / (G * TC);
    const uint32_t rem = t - grp * (G * TC);
    const uint32_t rows = min(G, TR - grp * G);
    const uint32_t col = rem / rows;
    ti = uniform(grp * G + (rem - col * rows));
    tj = uniform(col);
}

// WM x WN waves of BM x BN blocks of 16 x 16 outputs; one 64-wide k-slab per pipeline stage.
// k-slabs are copied global -> LDS by the load units directly (gfx950
// global_load_lds_dwordx4) into a ring of NSTAGE buffers, NSTAGE - 1 slabs
// ahead of the matrix cores.  REG_CARRY: the residue carried between the
// products of a modulus stays in registers; otherwise it is parked in the
// thread's own E'_I words.  PREFETCH: the next product's first stages are
// queued before the current product's epilogue; otherwise each product
// starts its own ring after the epilogue.  Both pay where k is short (4096^3:
// 15% faster products); for long k the plain schedule keeps the tiles of an
// XCD in step (16384^3: L2 hit rate 84% against 65%, 148 against 152 ms; 8192^3 17.75 against
// 17.35 ms, 4096^3 2459 against 2360 us).
template <int WM_, int WN_, int BM_, int BN_, int NSTAGE_, bool REG_CARRY_, bool PREFETCH_>
struct TileCfg {
    static constexpr int WM = WM_, WN = WN_, BM = BM_, BN = BN_;
    static constexpr int NSTAGE = NSTAGE_;
    static constexpr bool REG_CARRY = REG_CARRY_, PREFETCH = PREFETCH_;
    static constexpr int TM = WM * BM * 16, TN = WN * BN * 16;
    static constexpr int THREADS = 64 * WM * WN;
    static constexpr int STAGE = (TM + TN) * 4;   // uint4 per k-slab in LDS
};
using CfgLarge = TileCfg<2, 4, 8, 4, 4, false, false>;  // 256 x 256 output tiles, 512 threads, 128 KB LDS
using CfgSmall = TileCfg<2, 2, 4, 4, 4, true, true>;    // 128 x 128, 256 threads, 64 KB LDS
// 256 x 256 tiles with the short-k schedule: single calls with k_pad < kLongK and batches.
using CfgLargeShortK = TileCfg<2, 4, 8, 4, 4, true, true>;
static_assert(CfgLargeShortK::TM == CfgLarge::TM && CfgLargeShortK::TN == CfgLarge::TN,
              "both large-tile schedules share the operand padding");
constexpr int64_t kLongK = 16384;  // short-k faster up to 8192^3, plain at 16384^3 (above)

// One wave copies 64 x 16 bytes from global memory straight into 1 KB of LDS:
// lane i reads sbase + voff_i + OFF and writes lds_base + OFF + 16 i (the
// instruction offset applies to both addresses).  The base address and the
// LDS base are wave-uniform scalars and the per-lane offset is fixed for the
// whole kernel, so a copy costs no vector instructions.  Issued as inline
// assembly so that the compiler does not serialise later LDS reads behind it;
// completion is tracked explicitly with vmcnt_wait() before the barrier.
// M0 is written only here in these kernels (checked in the generated code); the
// clobber entry documents it although the compiler treats M0 as reserved.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF>
__device__ __forceinline__ void dma16(const int8_t *sbase, uint32_t voff, uint32_t lds_base) {
    static_assert(OFF >= 0 && OFF < 4096, "instruction offset range");
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(voff),
                 "s"(sbase), "s"(lds_base), "n"(OFF)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
// A wave-uniform pointer forced into scalar registers.
__device__ __forceinline__ const int8_t *uniform_ptr(const int8_t *p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const int8_t *)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
template <int N>
__device__ __forceinline__ void vmcnt_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void block_barrier() { __builtin_amdgcn_s_barrier(); }

// Copies of one k-slab into a ring stage: each wave fills whole 1 KB chunks (16 rows) of the
// A and B parts.  Lane i of a chunk writes LDS granule i, i.e. row 16 c + i / 4 at position
// i mod 4, which holds the swizzled global granule (i mod 4) ^ swz_bits(row).
template <int TM, int TN, int NW>
struct SlabCopy {
    static constexpr int QA = TM / 16 / NW, QB = TN / 16 / NW, NLOAD = QA + QB;  // loads per wave
    static_assert(TM / 16 % NW == 0 && TN / 16 % NW == 0 && QA <= 4 && QB <= 4, "chunks per wave");
    uint32_t va[QA], vb[QB];  // per-lane global offsets (without the instruction offset), fixed
    uint32_t la, lb;          // the wave's first chunk in a stage
    __device__ __forceinline__ SlabCopy(int wv, int lane) {
        const int crow = lane >> 2;
        static_for<QA>([&](auto q) {
            const int row = (wv * QA + q) * 16 + crow;
            va[q] = (uint32_t)(wv * QA * 1024 + crow * BK + ((lane & 3) ^ swz_bits(row)) * 16);
        });
        static_for<QB>([&](auto q) {
            const int row = (wv * QB + q) * 16 + crow;
            vb[q] = (uint32_t)(wv * QB * 1024 + crow * BK + ((lane & 3) ^ swz_bits(row)) * 16);
        });
        la = (uint32_t)(wv * QA * 1024);
        lb = (uint32_t)(TM * 64 + wv * QB * 1024);
    }
    __device__ __forceinline__ void issue(const int8_t *sa, const int8_t *sb, uint32_t stage) const {
        static_for<QA>([&](auto q) { dma16<q * 1024>(sa, va[q], stage + la); });
        static_for<QB>([&](auto q) { dma16<q * 1024>(sb, vb[q], stage + lb); });
    }
};

// A wave's share of a product, BM x BN blocks of v_mfma_i32_16x16x64_i8 per k-slab, one
// instruction's k.  That instruction at random operands reaches 4060 TOP/s on registers where
// the 32 x 32 x 32 one reaches 3460 (both 4.85 POP/s on zeros): the chip runs at its power limit
// here, and half as many accumulator updates per multiply-add toggle less.
// Fragments are single-buffered: a block row's A fragment is read again, for the next slab,
// right behind its last use, and the B fragments behind theirs in the last two block rows,
// so each has most of a slab to arrive and no copy of it is held.
// Against 32 x 32 x 32 instructions on the same tiles (fragments of half slabs in two sets,
// the barrier between the halves), products, same card: ZGEMM N = 14 2048^3 361 -> 348 us, 4096^3
// 2430 -> 2310 us, 8192^3 19260 -> 17780 us, 16384^3 151.0 -> 138.8 ms (2660 TOP/s); N = 13
// 2048^3 336 -> 320 us; 128 x 128 tiles, 1000 x 900 x 1100 65.7 -> 62.0 us, DGEMM 900 x 900 x 4096
// 70.6 -> 66.2 us.  With the barrier ahead of the slab's first matrix instruction 16384^3 takes
// 148 ms, with a fifth buffer 140 ms (4096^3 2410 us).
template <int BM, int BN>
struct WaveTile {
    static_assert(BM % 4 == 0 && BM >= 4 && (BN == 4 || BN == 1), "groups of four blocks");
    v4i fa[BM], fb[BN];
    const int loff;  // the lane's granule of block 0: the others are at fixed distances, since
                     // their rows differ in bits that the swizzle does not use
    __device__ __forceinline__ explicit WaveTile(int lane)
        : loff(group_row(lane & 15) * 4 + ((lane >> 4) ^ swz_bits(group_row(lane & 15)))) {}
    // fragment b of the wave's rows (columns) in the stage part at `base`
    __device__ __forceinline__ v4i frag(const uint4 *base, int b) const {
        const uint4 t = base[loff + (64 * (b >> 2) + 4 * (b & 3)) * 4];
        return v4i{(int)t.x, (int)t.y, (int)t.z, (int)t.w};
    }
    __device__ __forceinline__ void read_all(const uint4 *A, const uint4 *B) {
        static_for<BN>([&](auto j) { fb[j] = frag(B, j); });
        static_for<BM>([&](auto i) { fa[i] = frag(A, i); });
    }
    // acc += this slab; the fragments of the next slab from A, B (behind the last slab the
    // ring's next buffer: unused).  meet() waits until that
    // slab is there for all waves: behind the first block row, so that the waves meet with
    // matrix instructions queued.
    template <typename Meet>
    __device__ __forceinline__ void slab(v4i (&acc)[BM][BN], const uint4 *A, const uint4 *B, Meet meet) {
        auto mfma = [&](auto i, auto j) {
            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        };
        static_for<BM - 2>([&](auto i) {
            static_for<BN>([&](auto j0) {
                constexpr int j = (i & 1) ? BN - 1 - j0 : (int)j0;
                mfma(i, std::integral_constant<int, j>{});
            });
            if constexpr (i == 0) {
                __builtin_amdgcn_sched_barrier(0);
                meet();
            }
            fa[i] = frag(A, i);
        });
        static_for<BN>([&](auto j) {
            mfma(std::integral_constant<int, BM - 2>{}, j);
            mfma(std::integral_constant<int, BM - 1>{}, j);
            fb[j] = frag(B, j);
        });
        fa[BM - 2] = frag(A, BM - 2);
        fa[BM - 1] = frag(A, BM - 1);
        // the order written above: the scheduler would gather the reads
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        static_for<BM - 3>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, BN, 0);  // matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // an LDS read
        });
        static_for<BN>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        });
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
};

// One output tile (ti, tj) of modulus l over the k-slabs s0 .. s0 + nk - 1: all products of
// the plan and their epilogues, E' to the modulus' planes at ep.
// Ends with a block barrier, so a caller may run the next tile right away.
template <int KIND, typename C, bool DUMP>
__device__ __forceinline__ void gemm_tile(const GemmArgs &a, const BoundArgs &b, int8_t *ep, int l,
                                          int64_t ti, int64_t tj, int s0, int nk) {
    using P = Plan<KIND>;
    constexpr int TM = C::TM, TN = C::TN, BM = C::BM, BN = C::BN;
    constexpr int WTM = BM * 16, WTN = BN * 16;  // wave tile
    __shared__ uint4 lds[C::NSTAGE][C::STAGE];   // [buffer][A rows, B rows]

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv % C::WM, wn = wv / C::WM;

    constexpr bool bound = P::bound;
    const int64_t m_pad = bound ? b.m_pad : a.m_pad;
    const int64_t n_pad = bound ? b.n_pad : a.n_pad;
    const int64_t k_pad = bound ? b.k_pad : a.k_pad;
    const int64_t i0 = ti * TM, j0 = tj * TN;

    // planes are slab-major: k-slab s (64 wide) of a plane is m_pad x 64 bytes at s * slabA
    const int64_t planeA = m_pad * k_pad, planeB = n_pad * k_pad;
    const int64_t slabA = m_pad * BK, slabB = n_pad * BK;
    const int8_t *baseA =
        uniform_ptr((bound ? b.A : a.A) + (int64_t)l * P::nplanes * planeA + i0 * BK + s0 * slabA);
    const int8_t *baseB =
        uniform_ptr((bound ? b.B : a.B) + (int64_t)l * P::nplanes * planeB + j0 * BK + s0 * slabB);

    ModRule rule{};
    if constexpr (!bound) rule = mod_rule(a.tab, l);
    constexpr int bias = bound || DUMP ? 0 : kAccBias;  // accumulators' start
    const int64_t planeC = bound ? 0 : a.n_pad * a.m_pad;

    using Copy = SlabCopy<TM, TN, C::WM * C::WN>;
    const Copy copy(wv, lane);
    constexpr int NLOAD = Copy::NLOAD;
    // a slab is waited for one slab before it is used, while the one before it is computed and
    // its fragments are read, and queued AHEAD slabs ahead of its use
    static_assert(C::NSTAGE >= 3, "DMA ring needs at least three buffers");
    constexpr int AHEAD = C::NSTAGE - 1;
    const uint32_t lbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)(&lds[0][0]);
    // plane bases of product g (wave-uniform)
    auto pa_of = [&](int g) { return uniform_ptr(baseA + (int64_t)P::pa(g) * planeA); };
    auto pb_of = [&](int g) { return uniform_ptr(baseB + (int64_t)P::pb(g) * planeB); };
    auto issue_from = [&](const int8_t *sa, const int8_t *sb_, int st) {  // slab st -> buffer st % NSTAGE
        copy.issue(sa + st * slabA, sb_ + st * slabB, lbase + (uint32_t)((st % C::NSTAGE) * C::STAGE * 16));
    };
    // The first AHEAD slabs of a product.  Those of product g + 1 are issued right
    // after product g's last barrier, so they load while g's epilogue runs.
    auto issue_first = [&](int g) {
        const int8_t *sa = pa_of(g), *sb_ = pb_of(g);
        static_for<AHEAD>([&](auto st) {
            if (st < nk) issue_from(sa, sb_, st);
        });
    };
    auto partA = [&](int st) { return lds[st % C::NSTAGE] + wm * WTM * 4; };
    auto partB = [&](int st) { return lds[st % C::NSTAGE] + (TM + wn * WTN) * 4; };

    v4i acc[BM][BN];
    uint32_t cw[BM][BN];  // packed carry residues (kept here, or reloaded from E'_I)
    if constexpr (C::PREFETCH) issue_first(0);

#pragma unroll 1
    for (int sgi = 0; sgi < P::nseg; ++sgi) {
        if (!bound || sgi == 0) {
            static_for<BM>([&](auto bi) { static_for<BN>([&](auto bj) { acc[bi][bj] = (v4i)bias; }); });
        }
        {
            const int8_t *sa = pa_of(sgi), *sb_ = pb_of(sgi);
            // slabs 1 .. AHEAD-1 may stay in flight, except when this product's first
            // slabs were queued before the previous epilogue's stores: then wait for all
            if constexpr (!C::PREFETCH) issue_first(sgi);
            const bool fresh = !C::PREFETCH || sgi == 0;
            if (fresh && nk > 2 && AHEAD >= 3) vmcnt_wait<2 * NLOAD>();
            else if (fresh && nk > 1 && AHEAD >= 2) vmcnt_wait<NLOAD>();
            else vmcnt_wait<0>();
            block_barrier();
            WaveTile<BM, BN> wt(lane);
            wt.read_all(partA(0), partB(0));
            // At the last slab the fragments read ahead are not used.
            constexpr int LATER = AHEAD >= 2 ? AHEAD - 2 : 0;
            const int main_end = max(nk - AHEAD, 0);
#pragma unroll 1
            for (int s = 0; s < main_end; ++s) {
                wt.slab(acc, partA(s + 1), partB(s + 1), [&]() {
                    vmcnt_wait<LATER * NLOAD>();
                    block_barrier();  // slab s+1 visible; slab s-1's buffer free
                    issue_from(sa, sb_, s + AHEAD);
                });
            }
#pragma unroll 1
            for (int s = main_end; s < nk; ++s) {
                wt.slab(acc, partA(s + 1), partB(s + 1), [&]() {
                    if (s + 1 + LATER < nk) vmcnt_wait<LATER * NLOAD>();
                    else vmcnt_wait<0>();
                    block_barrier();
                });
            }
            block_barrier();  // all waves done with the ring before it is refilled
        }

        // ------------------------------------------------ per-product epilogue
        // (compile-time loops only: the accumulators must stay in registers)
        // The residue carried from one product to the next (mod(D) then mod(D + E) for
        // Karatsuba, mod(RR) and mod(RI) for the expanded form) stays in registers, or
        // is parked in this thread's own E'_I words, which receive the final E'_I last
        // (each lane re-reads only what it wrote, so no synchronisation is needed).
        // Parked carries are loaded and awaited first; then the next product's first
        // stages are queued, so that their copies overlap the rest of this epilogue.
        constexpr bool karatsuba = KIND == KIND_KARATSUBA;
        // 16 rows of a column: the lane's outputs of group q's four blocks in block column bj
        int el = lane;  // not hoisted: the addresses would live (in scratch) through the k-loops
        asm volatile("" : "+v"(el));
        const int64_t col0 = j0 + wn * WTN + group_row(el & 15);
        const int64_t row0 = i0 + wm * WTM + 16 * (el >> 4);
        auto e16 = [&](int8_t *E, int q, int bj) {
            return reinterpret_cast<u32x4 *>(E + (col0 + 4 * bj) * a.m_pad + row0 + 64 * q);
        };
        // the group's residues, four to a word: value(block, accumulator register)
        auto residues = [&](auto value) {
            u32x4 w;
            static_for<4>([&](auto t) {
                uint32_t x = 0;
                static_for<4>([&](auto u) {
                    x = put_residue<u>(value(t, (int)u) ^ (DUMP ? (uint32_t)kAccBias : 0u), rule, x);
                });
                w[(int)t] = x ^ 0x80808080u;
            });
            return w;
        };
        int8_t *ER = ep, *EI = ep + planeC;  // EI: not used by real products
        if constexpr (C::PREFETCH) {
            if (sgi + 1 < P::nseg) issue_first(sgi + 1);
        }
        if constexpr (DUMP) {
            int32_t *D = a.prods + ((int64_t)l * P::nseg + sgi) * planeC;
            static_for<BM>([&](auto bi) {
                static_for<BN>([&](auto bj) {
                    static_for<4>([&](auto r) {
                        D[(col0 + 4 * bj) * a.m_pad + row0 + 64 * (bi / 4) + 4 * (bi % 4) + r] = acc[bi][bj][(int)r];
                    });
                });
            });
        }
        if constexpr (bound) {
            // complex: acc holds Cbar_I after the second product, Cbar_R after the third;
            // real: Abar Bbar after the one product
            if (P::real || sgi >= 1) {
                static_for<BM>([&](auto bi) {
                    static_for<4>([&](auto r) {
                        int x = acc[bi][0][(int)r];
                        static_for<BN>([&](auto bj) { x = max(x, acc[bi][bj][(int)r]); });
#pragma unroll
                        for (int off = 8; off >= 1; off >>= 1) x = max(x, __shfl_xor(x, off, 64));
                        if ((lane & 15) == 0 && x > 0)
                            atomicMax(&b.X[row0 + 64 * (bi / 4) + 4 * (bi % 4) + r], x);
                    });
                });
                static_for<BN>([&](auto bj) {
                    int y = 0;
                    static_for<BM>([&](auto bi) { static_for<4>([&](auto r) { y = max(y, acc[bi][bj][(int)r]); }); });
                    y = max(y, __shfl_xor(y, 16, 64));
                    y = max(y, __shfl_xor(y, 32, 64));
                    if (lane < 16 && y > 0) atomicMax(&b.Y[col0 + 4 * bj], y);
                });
            }
        } else if constexpr (P::real) {
            // E' = mod(A'_l B'_l): one reduction per output (Algorithm 1 Step V-iv)
            static_for<BM / 4>([&](auto q) {
                static_for<BN>([&](auto bj) {
                    *e16(ER, q, bj) = residues([&](int t, int r) { return (uint32_t)acc[4 * (int)q + t][bj][r]; });
                });
            });
        } else {
            static_for<BM / 4>([&](auto q) {
                // A parked carry is read back one row of blocks at a time before that row's
                // stores: a load after a store is not moved above it (they might alias), so
                // word-by-word read-back waited for a memory round trip per word.
                if (!C::REG_CARRY && sgi >= 1 && (karatsuba || sgi != 2)) {
                    u32x4 back[BN];
                    static_for<BN>([&](auto bj) { back[bj] = *e16(EI, q, bj); });
                    static_for<BN>([&](auto bj) {
                        static_for<4>([&](auto t) { cw[4 * q + t][bj] = back[bj][(int)t]; });
                    });
                }
                static_for<BN>([&](auto bj) {
                    u32x4 *er = e16(ER, q, bj), *ei = e16(EI, q, bj);
                    // The first product of a pair is reduced and carried; the second
                    // enters the reduction unreduced (accumulator +- carried residue
                    // stays in range, see put_residue): 4 reductions per output and
                    // modulus in both forms.
                    auto x = [&](int t, int r) { return acc[4 * (int)q + t][bj][r]; };
                    auto d = [&](int t, int r) { return byte_of(cw[4 * (int)q + t][bj], r); };
                    auto carry = [&](const u32x4 &o) {
                        if constexpr (C::REG_CARRY) static_for<4>([&](auto t) { cw[4 * q + t][bj] = o[(int)t]; });
                        else *ei = o;
                    };
                    if (sgi == 0 || (!karatsuba && sgi == 2)) {
                        carry(residues([&](int t, int r) { return (uint32_t)x(t, r); }));
                    } else if (sgi == 1) {
                        // Karatsuba: E'_R = mod(D - E), carry mod(D + E); expanded: E'_R = mod(RR - II)
                        *er = residues([&](int t, int r) { return acc_sub(d(t, r), x(t, r)); });
                        if constexpr (karatsuba) carry(residues([&](int t, int r) { return acc_add(d(t, r), x(t, r)); }));
                    } else {
                        // Karatsuba: E'_I = mod(F - mod(D + E)); expanded: E'_I = mod(RI + IR)
                        *ei = residues([&](int t, int r) { return karatsuba ? acc_sub(x(t, r), d(t, r)) : acc_add(d(t, r), x(t, r)); });
                    }
                });
            });
        }
    }
}

// ---------------------------------------------------------------- products held to the end
// Waves of 64 x 64 outputs that hold every product of the plan in INT32 accumulators of
// its own until the end (192 registers for complex products), so the ring of LDS buffers
// runs through the products without a break and each output is reduced twice (once per
// part) instead of three or four times with residues carried in between:
//   Karatsuba: E'_R = mod(D - E), E'_I = mod(F - D - E)
//   expanded:  E'_R = mod(RR - II), E'_I = mod(RI + IR) (one accumulator for RI + IR)
// |F - D - E| <= 3 k 127^2 stays below 2^31 for kOnceChunk k-elements (p = 256 may wrap:
// harmless modulo 2^32); longer k runs in chunks, the accumulators replaced by their
// symmetric residues in between.
// The first accumulator starts at the bias 2^31 that put_residue expects: it carries over
// to both results (X - Y and Z - X - Y modulo 2^32).
// Against the 128 x 128 tiles with carried residues, same card, products (32 x 32 x 32
// instructions): ZGEMM 64^3 10.8 -> 8.5 us, 256^3 expanded 15.5 -> 12.4 us, 1000 x 900 x 1100
// 70 -> 65 us.  On 256 x 256-tile shapes it loses from k = 1024 on (2048^3 at N = 13: 390
// against 354 us, 4096^3 3200 against 2377 us): a 64 x 64 wave reads a third more LDS per
// matrix instruction and a 128 x 128 block copies twice the bytes into it.
// Waves of 64 x 16 (BN = 1, four to a 64 x 64 tile): see choose_64_tiles.
constexpr int kOnceChunk = 32768 / BK;  // k-slabs
template <int WM_, int WN_, int BN_, int NSTAGE_, int NACC_, int WAVES_>
struct OnceCfg {
    static constexpr int WM = WM_, WN = WN_, BM = 4, BN = BN_, NSTAGE = NSTAGE_, NACC = NACC_;
    static constexpr int TM = WM * 64, TN = WN * BN * 16, THREADS = 64 * WM * WN;
    static constexpr int WAVES = WAVES_;         // per SIMD: bounds the registers
    static constexpr int STAGE = (TM + TN) * 4;  // uint4 per 64-wide k-slab in LDS
};

// As gemm_tile: one output tile (ti, tj) of modulus l over the k-slabs s0 .. s0 + slabs - 1,
// E' to the modulus' planes at ep.  AGAIN: a block barrier stands behind the last slab, so that
// the caller may run the next tile right away: the last barrier of the slabs themselves does not
// wait for the other waves' reads of the slab behind it, and the next tile's copies go to
// the same buffers.
template <int KIND, typename C, bool AGAIN>
__device__ __forceinline__ void once_tile(const GemmArgs &a, int8_t *ep, int l, int64_t ti, int64_t tj,
                                          int s0, int slabs) {
    using P = Plan<KIND>;
    static_assert(!P::bound, "bound products fold maxima, they have no E'");
    constexpr int TM = C::TM, TN = C::TN, BM = C::BM, BN = C::BN, NSTAGE = C::NSTAGE;
    constexpr int NACC = C::NACC;
    static_assert(NACC == (P::real ? 1 : 3), "one accumulator per held product");
    __shared__ uint4 lds[NSTAGE][C::STAGE];  // [buffer][A rows, B rows]
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv % C::WM, wn = wv / C::WM;
    const int64_t i0 = ti * TM, j0 = tj * TN;
    const int64_t planeA = a.m_pad * a.k_pad, planeB = a.n_pad * a.k_pad;
    const int64_t slabA = a.m_pad * BK, slabB = a.n_pad * BK;
    const int8_t *baseA = uniform_ptr(a.A + (int64_t)l * P::nplanes * planeA + i0 * BK + s0 * slabA);
    const int8_t *baseB = uniform_ptr(a.B + (int64_t)l * P::nplanes * planeB + j0 * BK + s0 * slabB);
    const ModRule rule = mod_rule(a.tab, l);

    // ring of NSTAGE one-slab buffers, filled AHEAD slabs ahead (see gemm_tile)
    using Copy = SlabCopy<TM, TN, C::WM * C::WN>;
    const Copy copy(wv, lane);
    constexpr int NLOAD = Copy::NLOAD;
    static_assert(NSTAGE >= 3, "DMA ring needs at least three buffers");
    constexpr int AHEAD = NSTAGE - 1, LATER = AHEAD - 2 > 0 ? AHEAD - 2 : 0;
    const uint32_t lbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)(&lds[0][0]);
    v4i acc[NACC][BM][BN];
    static_for<NACC>([&](auto z) {
        static_for<BM>([&](auto bi) {
            static_for<BN>([&](auto bj) { acc[z][bi][bj] = (v4i)(z == 0 ? kAccBias : 0); });
        });
    });
    auto partA = [&](int buf) { return lds[buf] + wm * 64 * 4; };
    const int wcol = wn * BN / 4 * 64 + wn * BN % 4 * 4;  // the wave's first column
    auto partB = [&](int buf) { return lds[buf] + (TM + wcol) * 4; };
    for (int c0 = 0;;) {
        const int nk = min(slabs - c0, kOnceChunk);
        const int8_t *sa = baseA, *sb = baseB;  // the next slab to queue
        int iseg = 0, ist = 0, ibuf = 0;        // its product, slab and buffer
        auto issue = [&]() {
            copy.issue(sa, sb, lbase + (uint32_t)(ibuf * C::STAGE * 16));
            ibuf = ibuf + 1 == NSTAGE ? 0 : ibuf + 1;
            sa += slabA;
            sb += slabB;
            if (++ist == nk) {  // first slab of the next product's planes
                ist = 0;
                ++iseg;
                const int pa = KIND == KIND_4M ? iseg & 1 : iseg;
                const int pb = KIND == KIND_4M ? (iseg ^ (iseg >> 1)) & 1 : iseg;
                sa = uniform_ptr(baseA + pa * planeA);
                sb = uniform_ptr(baseB + pb * planeB);
            }
        };
        const int T = P::nseg * nk;
        static_for<AHEAD>([&](auto t) {
            if (t < T) issue();
        });

        if (T > 2 && AHEAD >= 3) vmcnt_wait<2 * NLOAD>();
        else if (T > 1) vmcnt_wait<NLOAD>();
        else vmcnt_wait<0>();
        block_barrier();
        WaveTile<BM, BN> wt(lane);
        wt.read_all(partA(0), partB(0));
        int t = 0, cur = 0;
        static_for<P::nseg>([&](auto seg) {
            constexpr int z = seg < NACC ? (int)seg : NACC - 1;
#pragma unroll 1
            for (int s = 0; s < nk; ++s, ++t) {
                // at the last slab of all the wait and the barrier close the ring, and the
                // fragments read ahead are not used: one path, so that the accumulators
                // stay in place
                cur = cur + 1 == NSTAGE ? 0 : cur + 1;
                wt.slab(acc[z], partA(cur), partB(cur), [&]() {
                    if (t + 1 + LATER < T) vmcnt_wait<LATER * NLOAD>();
                    else vmcnt_wait<0>();
                    block_barrier();  // slab t+1 visible; slab t-1's buffer free
                    if (t + AHEAD < T) issue();
                });
            }
        });
        c0 += nk;
        if (AGAIN || c0 < slabs) block_barrier();  // all waves done with the ring before it is refilled
        if (c0 >= slabs) break;
        baseA += nk * slabA;
        baseB += nk * slabB;
        static_for<NACC>([&](auto z) {
            static_for<BM>([&](auto bi) {
                static_for<BN>([&](auto bj) {
                    static_for<4>([&](auto r) {
                        const int v = acc[z][bi][bj][(int)r];
                        const uint32_t u = put_residue<0>(z == 0 ? (uint32_t)v : acc_flip(v), rule, 0u);
                        acc[z][bi][bj][(int)r] = acc_refill(u, z == 0);
                    });
                });
            });
        });
    }

    const int64_t planeC = a.n_pad * a.m_pad;
    const int64_t col0 = j0 + wcol + group_row(lane & 15);
    int8_t *E = ep + i0 + wm * 64 + 16 * (lane >> 4);
    auto store = [&](auto bj, int plane, auto value) {
        u32x4 w;
        static_for<4>([&](auto t) {
            uint32_t x = 0;
            static_for<4>([&](auto u) { x = put_residue<u>(value(t, (int)u), rule, x); });
            w[(int)t] = x ^ 0x80808080u;
        });
        *global_ptr(reinterpret_cast<u32x4 *>(E + plane * planeC + (col0 + 4 * bj) * a.m_pad)) = w;
    };
    static_for<BN>([&](auto bj) {
        if constexpr (P::real) {
            store(bj, 0, [&](int t, int r) { return (uint32_t)acc[0][t][bj][r]; });
        } else {
            store(bj, 0, [&](int t, int r) { return acc_sub(acc[0][t][bj][r], acc[1][t][bj][r]); });
            store(bj, 1, [&](int t, int r) {
                if constexpr (KIND == KIND_4M) return acc_flip(acc[2][t][bj][r]);
                else return acc_sub(acc[2][t][bj][r], acc[0][t][bj][r]) - (uint32_t)acc[1][t][bj][r];
            });
        }
    });
}

// E' planes of modulus l in a.eprime.
template <int KIND>
__device__ __forceinline__ int8_t *eprime_of(const GemmArgs &a, int l) {
    return a.eprime + (int64_t)l * Plan<KIND>::eplanes * a.n_pad * a.m_pad;
}

// The work of block `blk` of a single call: modulus, tile, k-slabs and E' planes.  The
// first l_split moduli take one block per tile; each tile of the others takes a.parts
// blocks, which cut its k-slabs evenly and write E' planes of their own (congruent sums:
// the reconstruction adds the parts' residues).
struct BlockWork {
    int l, s0, nk;
    int64_t ti, tj;
    int8_t *ep;
};
template <int KIND, typename C>
__device__ __forceinline__ BlockWork block_work(const GemmArgs &a, uint32_t blk) {
    const uint32_t TR = C::TM == 64 ? (uint32_t)a.rows64 : (uint32_t)(a.m_pad / C::TM);
    const uint32_t TC = C::TN == 64 ? (uint32_t)a.cols64 : (uint32_t)(a.n_pad / C::TN);
    const uint32_t whole = (uint32_t)a.l_split * TR * TC;
    const int slabs = (int)(a.k_pad / BK);
    BlockWork w;
    if (blk < whole) {
        map_tile(blk, TR, TC, whole, w.l, w.ti, w.tj);
        w.s0 = 0;
        w.nk = slabs;
        w.ep = eprime_of<KIND>(a, w.l);
        return w;
    }
    const int ns = a.nmod - a.l_split;  // split moduli
    int lp;
    map_tile(blk - whole, TR, TC, (uint32_t)(ns * a.parts) * TR * TC, lp, w.ti, w.tj);
    const int part = (int)uniform((uint32_t)lp / (uint32_t)ns), ls = lp - part * ns;
    w.l = a.l_split + ls;
    w.s0 = (int)uniform((uint32_t)(slabs * part) / (uint32_t)a.parts);
    w.nk = (int)uniform((uint32_t)(slabs * (part + 1)) / (uint32_t)a.parts) - w.s0;
    w.ep = part == 0 ? eprime_of<KIND>(a, w.l)
                     : a.eprime_parts + (int64_t)((part - 1) * ns + ls) * Plan<KIND>::eplanes * a.n_pad * a.m_pad;
    return w;
}

// Two waves per SIMD at least: with 512 registers allowed the compiler keeps accumulators in
// the accumulation half and copies them from slab to slab (real bound of 576 x 960 x 23655:
// 328 against 294 us with the scan).
template <int KIND, typename C, bool DUMP>
__global__ __launch_bounds__(C::THREADS, 2) void residue_gemm_kernel(GemmArgs a) {
    const BlockWork w = block_work<KIND, C>(a, blockIdx.x);
    gemm_tile<KIND, C, DUMP>(a, BoundArgs{}, w.ep, w.l, w.ti, w.tj, w.s0, w.nk);
}

template <int KIND, typename C>
__global__ __launch_bounds__(C::THREADS, C::WAVES) void once_gemm_kernel(GemmArgs a) {
    const BlockWork w = block_work<KIND, C>(a, blockIdx.x);
    once_tile<KIND, C, false>(a, w.ep, w.l, w.ti, w.tj, w.s0, w.nk);
}

template <int KIND, typename C>
__global__ __launch_bounds__(C::THREADS, 2) void bound_gemm_kernel(BoundArgs b) {
    const uint32_t TR = (uint32_t)(b.m_pad / C::TM), TC = (uint32_t)(b.n_pad / C::TN);
    int l;
    int64_t ti, tj;
    map_tile(blockIdx.x, TR, TC, TR * TC, l, ti, tj);
    gemm_tile<KIND, C, false>(GemmArgs{}, b, nullptr, 0, ti, tj, 0, (int)(b.k_pad / BK));
}

// A batch's tile of either class.
template <int KIND, typename C>
struct BatchTile {
    __device__ static __forceinline__ void run(const GemmArgs &a, int l, int64_t ti, int64_t tj) {
        gemm_tile<KIND, C, false>(a, BoundArgs{}, eprime_of<KIND>(a, l), l, ti, tj, 0, (int)(a.k_pad / BK));
    }
};
template <int KIND, int WM, int WN, int BN, int NSTAGE, int NACC, int WAVES>
struct BatchTile<KIND, OnceCfg<WM, WN, BN, NSTAGE, NACC, WAVES>> {
    __device__ static __forceinline__ void run(const GemmArgs &a, int l, int64_t ti, int64_t tj) {
        once_tile<KIND, OnceCfg<WM, WN, BN, NSTAGE, NACC, WAVES>, true>(a, eprime_of<KIND>(a, l), l, ti, tj, 0,
                                                                       (int)(a.k_pad / BK));
    }
};

// Persistent kernel over the work queue of a batch: each block takes the next
// item from the counter until the queue is empty.  Items of one problem are
// numbered (modulus group, tile row, tile column); problems are ordered by the
// host (largest k first).
template <int KIND, typename C>
__global__ __launch_bounds__(C::THREADS, 2) void batch_gemm_kernel(const BatchGemm *probs, int nprob,
                                                                int64_t items, int group,
                                                                uint32_t *counters, int64_t chunk) {
    __shared__ int64_t item_s;
    // Work-groups are dispatched to the XCDs in turn (block b on XCD b mod 8).  The
    // item sequence is cut into chunks of `chunk` items (the blocks one XCD holds at a
    // time), dealt to the XCDs in turn, each XCD with its own counter: the tiles that
    // run together on an XCD are neighbours of one product and share their operand
    // panels in that XCD's L2.  A block whose queue is empty takes items from the
    // other queues.  Any dispatch order gives the same results.
    // Per item the block needs the queue's counter and its problem's record, each a
    // round trip to L2: the next item is claimed as soon as the current one is known
    // (the atomic returns while this item computes), and the problem is looked up
    // first where the previous item was (a block's items rise within a queue, and a
    // problem has many items), with a binary search only when that misses.  Item
    // numbers are below 2^32 (the counters are 32-bit), so the index arithmetic is
    // 32-bit.  The counter address is offset by a zero the compiler cannot see through:
    // for a uniform address it combines the lanes' atomics into one and reads the
    // result back at once, which would wait for the round trip right there.
    const int64_t nchunks = items / chunk, rem = items - nchunks * chunk;
    const uint32_t ch = (uint32_t)chunk;
    const int home = (int)(blockIdx.x % kBatchQueues);
    int lo = 0;          // problem of the previous item
    uint32_t ahead = 0;  // thread 0: the item claimed for the next round
    uint32_t zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    for (int qs = 0; qs < kBatchQueues; ++qs) {
        const int q = (home + qs) % kBatchQueues;
        const int64_t nq = (nchunks / kBatchQueues + (q < nchunks % kBatchQueues ? 1 : 0)) * chunk +
                           (nchunks % kBatchQueues == q ? rem : 0);
        if (threadIdx.x == 0) ahead = atomicAdd(&counters[q], 1u);
        for (;;) {
            if (threadIdx.x == 0) item_s = (int64_t)ahead;
            __syncthreads();
            // item numbers are block-uniform: in a scalar register, so that everything
            // derived from them (the problem's record, the copies' addresses) is scalar
            const uint32_t j32 = __builtin_amdgcn_readfirstlane((uint32_t)item_s);
            __syncthreads();
            if (j32 >= nq) break;
            if (threadIdx.x == 0) ahead = atomicAdd(&counters[q] + zero, 1u);
            const uint32_t jc = uniform(j32 / ch);
            const int64_t w = ((int64_t)jc * kBatchQueues + q) * ch + (j32 - jc * ch);
            const OZC_AS_CONST BatchGemm *pl = const_ptr(probs);
            const int64_t f0 = pl[lo].item0;
            const int64_t f1 = lo + 1 < nprob ? pl[lo + 1].item0 : items;
            if (w < f0 || w >= f1) {  // last problem whose first item is <= w
                int hi = w < f0 ? lo - 1 : nprob - 1;
                lo = w < f0 ? 0 : lo + 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (pl[mid].item0 <= w) lo = mid;
                    else hi = mid - 1;
                }
            }
            const OZC_AS_CONST BatchGemm &pb = pl[lo];
            const uint32_t T = (uint32_t)pb.TR * (uint32_t)pb.TC, local = (uint32_t)(w - pb.item0);
            const int lg = (int)uniform(local / T);
            const uint32_t t = local - (uint32_t)lg * T;
            const int64_t ti = uniform(t / (uint32_t)pb.TC), tj = t - (uint32_t)ti * (uint32_t)pb.TC;
            GemmArgs a{pb.A, pb.B, pb.m_pad, pb.n_pad, pb.k_pad, pb.nmod, KIND == KIND_4M ? 1 : 0,
                       pb.tab, pb.eprime, nullptr, C::TM, pb.nmod, 1, nullptr};
            const int l1 = min(pb.nmod, (lg + 1) * group);
            for (int l = lg * group; l < l1; ++l) BatchTile<KIND, C>::run(a, l, ti, tj);
        }
    }
}

// Persistent kernel over the tiles of a batch's bound products (accurate mode).
template <typename C>
__global__ __launch_bounds__(C::THREADS, 2) void batch_bound_kernel(const BatchBound *probs, int nprob,
                                                                int64_t items, uint32_t *counter) {
    __shared__ int64_t item_s;
    for (;;) {
        if (threadIdx.x == 0) item_s = (int64_t)atomicAdd(counter, 1u);
        __syncthreads();
        const int64_t w = item_s;
        __syncthreads();
        if (w >= items) break;
        int lo = 0, hi = nprob - 1;  // last problem whose first item is <= w
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (probs[mid].item0 <= w) lo = mid;
            else hi = mid - 1;
        }
        const BatchBound &pb = probs[lo];
        const int64_t t = w - pb.item0;
        const int64_t ti = t / pb.TC, tj = t - ti * pb.TC;
        gemm_tile<KIND_BOUND, C, false>(GemmArgs{}, pb.b, nullptr, 0, ti, tj, 0, (int)(pb.b.k_pad / BK));
    }
}

template <int KIND, typename C>
void launch_batch_kind(const BatchGemm *probs, int nprob, int64_t items, int group,
                       uint32_t *counters, int grid, hipStream_t s) {
    const int64_t chunk = grid >= kBatchQueues ? grid / kBatchQueues : 1;  // resident blocks per XCD
    hipLaunchKernelGGL((batch_gemm_kernel<KIND, C>), dim3((unsigned)grid), dim3(C::THREADS), 0, s,
                       probs, nprob, items, group, counters, chunk);
}

template <int KIND, typename C>
int blocks_per_cu() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_gemm_kernel<KIND, C>, C::THREADS, 0) !=
        hipSuccess)
        n = 1;
    return n > 0 ? n : 1;
}

template <int KIND, typename C>
void launch_kind(const GemmArgs &a, bool dump, int64_t blocks, hipStream_t s) {
    if (dump) hipLaunchKernelGGL((residue_gemm_kernel<KIND, C, true>), dim3((unsigned)blocks), dim3(C::THREADS), 0, s, a);
    else hipLaunchKernelGGL((residue_gemm_kernel<KIND, C, false>), dim3((unsigned)blocks), dim3(C::THREADS), 0, s, a);
}

// 128 x 128 output tiles, 256 threads, 64 KB LDS: two blocks per CU, two waves per SIMD
using Once128 = OnceCfg<2, 2, 4, 4, 3, 2>;
using Once128Real = OnceCfg<2, 2, 4, 4, 1, 2>;
using Once64 = OnceCfg<1, 4, 1, 4, 3, 4>;
using Once64Real = OnceCfg<1, 4, 1, 4, 1, 4>;

template <int KIND, typename C>
hipError_t launch_once(const GemmArgs &a, int64_t blocks, hipStream_t s) {
    hipLaunchKernelGGL((once_gemm_kernel<KIND, C>), dim3((unsigned)blocks), dim3(C::THREADS), 0, s, a);
    return hipGetLastError();
}

template <int KIND, typename C>
void launch_dump(const GemmArgs &a, int64_t blocks, hipStream_t s) {
    hipLaunchKernelGGL((residue_gemm_kernel<KIND, C, true>), dim3((unsigned)blocks), dim3(C::THREADS), 0,
                       s, a);
}

}  // namespace

int gemm_tile_for(int64_t m, int64_t n) { return (m >= 1024 && n >= 1024) ? 256 : 128; }
int gemm_kstep_for(int) { return BK; }
int gemm_tile_rows(int tile) { return tile == 256 ? CfgLarge::TM : CfgSmall::TM; }
int gemm_tile_cols(int tile) { return tile == 256 ? CfgLarge::TN : CfgSmall::TN; }

// Whether a single call's products run on 64 x 64 tiles.  Where a call's 128 x 128 tiles leave
// CUs idle, its time is one block's: the reductions of 64 x 64 outputs per wave (some 320 x 8
// vector instructions, 4 us for complex products) behind a chain of slabs.  A quarter of that
// on four times the CUs is shorter; once the CUs are full, the smaller tile's operand reads
// (five LDS reads per four matrix instructions, against two per four) cost more than that.
// Products in us, 128 x 128 against 64 x 64, blocks of the latter on 256 CUs:
//   ZGEMM N = 14, 64 x 64 (14 blocks)   k = 64   8.5 -> 6.8,   k = 256  11.0 -> 8.2
//   ZGEMM N = 14, 256 x 256 (224)       k = 64   9.0 -> 7.1,   k = 512  14.3 -> 10.8,  k = 1024 20.3 -> 15.2
//   ZGEMM N = 14, 256 x 512 (448)       k = 64   9.8 -> 8.4,   k = 512  14.9 -> 12.4,  k = 1024 20.3 -> 16.4
//   ZGEMM N = 14, 320 x 576 (630)       k = 64   11.0 -> 9.6,  k = 512  14.9 -> 14.1,  k = 1024 20.9 -> 20.7
//   ZGEMM N = 14, 384 x 512 (672)       k = 64   10.4 -> 9.6,  k = 512  14.9 -> 14.2,  k = 1024 20.6 -> 21.0
//   ZGEMM N = 14, 448 x 512 (784)       k = 64   11.3 -> 11.4, k = 512  15.0 -> 16.4,  k = 1024 20.9 -> 25.9
//   ZGEMM N = 14, 320 x 576 (630)       k = 1088 21.3 -> 21.3, k = 2048 32.3 -> 33.2
//   DGEMM N = 14, 256 x 512 (448)       k = 64   7.3 -> 6.8,   k = 1024 11.1 -> 9.8
//   DGEMM N = 14, 320 x 576 (630)       k = 64   7.8 -> 7.3,   k = 1024 11.6 -> 11.0
//   DGEMM N = 14, 448 x 512 (784)       k = 64   8.1 -> 8.3,   k = 1024 11.7 -> 12.7
// Products that are cut along k keep 128 x 128 tiles (the cut's parts are sized for them).
bool choose_64_tiles(int tile, int nmod, int64_t m, int64_t n, int64_t k_pad, int cus) {
    if (tile != 128 || m > (int64_t)64 * 1024 || n > (int64_t)64 * 1024) return false;
    const int64_t blocks = (int64_t)nmod * ((m + 63) / 64) * ((n + 63) / 64);
    return blocks <= cus || (2 * blocks <= 5 * (int64_t)cus && k_pad <= 1024);
}

// How a single call's products are cut along k.  A launch whose tiles leave CUs idle, or
// whose last round of blocks is short, gains from more and shorter blocks; every part pays
// an epilogue, and E' planes of its own that the reconstruction reads too.  The choice is
// the least of these times in us, fitted to whole calls (1010 of 16 .. 4000 rows and columns and
// k of 128 .. 60000, all four types, each timed whole and in every number of parts):
//   one slab (64 k) of one product: 64 x 64 tiles 0.2; 128 x 128 tiles 0.26 alone on a CU, 0.43
//   for two of them; 256 x 256 tiles 0.9; where the residues pass the Infinity Cache (300 MB) 0.28,
//   0.34 and 0.5;
//   the rest of a block: 3, 5 and 11.5 (one real product: 2, 3 and 5);
//   a further entry of the reconstruction's sums: 0.165 (real 0.125), its share of a load's
//   latency in a chain of loads four entries apart, or its bytes at 4.2 TB/s; and 0.5 for the call.
// Over those calls the choice is 0.3% from the best of them (geometric mean; 1.9% with constants
// from older kernels and no term for the entries' latency, which took 77 of them slower than whole,
// by up to 25%; now 8, by up to 7%).  384 x 320 x 40000 at N = 14 (126 tiles): 4 parts, products
// 685 -> 346 us; 2048^3 at N = 13 (832 tiles of 256 x 256 on 256 CUs): the last modulus in 3 parts instead
// of a fourth round that is a quarter full, 345 -> 323 us.  Calls, whole against 8, 4 and 6 parts:
// ZGEMM 47 x 110 x 791 at N = 11 30.4 and 40.7 us, 256 x 256 x 512 expanded at N = 14 29.6 and 37.4, DGEMM
// 80 x 136 x 2022 at N = 14 31.3 and 37.3.
KSplit choose_k_split(int tile, int algo, int nmod, int64_t m, int64_t n, int64_t k_pad, int cus) {
    const bool real = algo == 2, small = tile == 128;
    const int nseg = real ? 1 : (algo == 1 ? 4 : 3), nplanes = real ? 1 : (algo == 1 ? 2 : 3);
    const int64_t TR = (m + tile - 1) / tile, TC = (n + tile - 1) / tile;
    const double T = (double)TR * (double)TC;
    const int64_t slabs = k_pad / BK;
    const bool far = (double)nmod * nplanes * (double)((TR + TC) * tile) * (double)k_pad > 3e8;
    const double rest = small ? (real ? 3.0 : 5.0) : (real ? 5.0 : 11.5);
    const double slots = small ? 2.0 * cus : cus;
    const double alone = small ? (far ? 0.34 : 0.26) : 0.9, full = small ? (far ? 0.5 : 0.43) : 0.9;
    // a block of n slabs with this many on the chip, and a launch of them
    auto block_us = [&](int64_t n, double blocks) {
        return nseg * (double)n * (blocks <= cus ? alone : full) + rest;
    };
    auto launch_us = [&](int64_t n, double blocks) {
        const double rounds = std::floor(blocks / slots), more = blocks - rounds * slots;
        return rounds * block_us(n, slots) + (more > 0.0 ? block_us(n, more) : 0.0);
    };
    KSplit best{nmod, 1};
    const double whole = choose_64_tiles(tile, nmod, m, n, k_pad, cus)
                             ? nseg * (double)slabs * (far ? 0.28 : 0.2) + (real ? 2.0 : 3.0)
                             : launch_us(slabs, nmod * T);
    double best_us = 0.97 * whole;
    // what an even spread of the blocks over the slots would take, epilogues included: no
    // split does better
    if (nmod * T >= slots && nmod * T / slots * block_us(slabs, nmod * T) + 0.5 >= best_us) return best;
    const double entry_us = std::max(real ? 0.125 : 0.165, (real ? 1.0 : 2.0) * T * tile * tile / 4.2e6);
    for (int parts : {2, 3, 4, 6, 8}) {
        if (parts > slabs) break;
        for (int ls = 0; ls < nmod; ++ls) {
            if (ls + (nmod - ls) * parts > kMaxPartSum) continue;
            const double n1 = ls * T, n2 = (nmod - ls) * T * parts;
            const int64_t part_slabs = (slabs + parts - 1) / parts;
            const double b1 = block_us(slabs, n1 + n2), b2 = block_us(part_slabs, n1 + n2);
            double us = ls == 0 ? launch_us(part_slabs, n2)
                                : std::max(std::ceil(n1 / slots) * b1, (n1 * b1 + n2 * b2) / slots + 0.5 * b2);
            us += (nmod - ls) * (parts - 1) * entry_us + 0.5;
            if (us < best_us) {
                best_us = us;
                best = KSplit{ls, parts};
            }
        }
    }
    return best;
}

hipError_t launch_residue_gemm(const GemmArgs &a, hipStream_t s) {
    const int tile = a.tile;
    if (tile != 128 && tile != 256) return hipErrorInvalidValue;
    const int tr = gemm_tile_rows(tile), tc = gemm_tile_cols(tile);
    if (a.m_pad % tr || a.n_pad % tc || a.k_pad % gemm_kstep_for(tile) || a.nmod < 1)
        return hipErrorInvalidValue;
    if (a.l_split < 0 || a.l_split > a.nmod || a.parts < 1 || a.parts > kMaxParts || a.parts > a.k_pad / BK ||
        (a.parts > 1 && a.l_split < a.nmod && !a.eprime_parts))
        return hipErrorInvalidValue;
    const int64_t blocks = (a.l_split + (int64_t)(a.nmod - a.l_split) * a.parts) * (a.m_pad / tr) * (a.n_pad / tc);
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    const bool dump = a.prods != nullptr;
    if (a.algo < 0 || a.algo > 2) return hipErrorInvalidValue;
    if (a.rows64 > 0) {
        if (tile != 128 || dump || a.l_split < a.nmod || a.rows64 * 64 > a.m_pad || a.cols64 < 1 || a.cols64 * 64 > a.n_pad)
            return hipErrorInvalidValue;
        const int64_t small = (int64_t)a.nmod * a.rows64 * a.cols64;
        if (small >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
        if (a.algo == 2) return launch_once<KIND_REAL, Once64Real>(a, small, s);
        if (a.algo == 1) return launch_once<KIND_4M, Once64>(a, small, s);
        return launch_once<KIND_KARATSUBA, Once64>(a, small, s);
    }
    if (tile == 128 && !dump) {
        if (a.algo == 2) return launch_once<KIND_REAL, Once128Real>(a, blocks, s);
        if (a.algo == 1) return launch_once<KIND_4M, Once128>(a, blocks, s);
        return launch_once<KIND_KARATSUBA, Once128>(a, blocks, s);
    }
    if (tile == 128) {  // with the raw products written out
        if (a.algo == 2) launch_dump<KIND_REAL, CfgSmall>(a, blocks, s);
        else if (a.algo == 1) launch_dump<KIND_4M, CfgSmall>(a, blocks, s);
        else launch_dump<KIND_KARATSUBA, CfgSmall>(a, blocks, s);
        return hipGetLastError();
    }
    // one product per modulus: the long-k schedule keeps no carry, so it serves every k
    if (a.algo == 2) launch_kind<KIND_REAL, CfgLarge>(a, dump, blocks, s);
    else if (a.k_pad >= kLongK) {
        if (a.algo == 0) launch_kind<KIND_KARATSUBA, CfgLarge>(a, dump, blocks, s);
        else launch_kind<KIND_4M, CfgLarge>(a, dump, blocks, s);
    } else {
        if (a.algo == 0) launch_kind<KIND_KARATSUBA, CfgLargeShortK>(a, dump, blocks, s);
        else launch_kind<KIND_4M, CfgLargeShortK>(a, dump, blocks, s);
    }
    return hipGetLastError();
}

// The bound product is 1/N of the work; it always runs on 128 x 128 tiles
// (valid for buffers padded to 128 or 256).
hipError_t launch_bound_gemm(const BoundArgs &b, hipStream_t s) {
    constexpr int tile = 128;
    if (b.m_pad % tile || b.n_pad % tile || b.k_pad % BK) return hipErrorInvalidValue;
    const int64_t blocks = (b.m_pad / tile) * (b.n_pad / tile);
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(CfgSmall::THREADS);
    if (b.real) hipLaunchKernelGGL((bound_gemm_kernel<KIND_BOUND_REAL, CfgSmall>), grid, block, 0, s, b);
    else hipLaunchKernelGGL((bound_gemm_kernel<KIND_BOUND, CfgSmall>), grid, block, 0, s, b);
    return hipGetLastError();
}

hipError_t launch_batch_bound(const BatchBound *probs, int nprob, int64_t items,
                              uint32_t *counter, hipStream_t s) {
    if (items <= 0 || nprob <= 0) return hipSuccess;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batch_bound_kernel<CfgSmall>,
                                                     CfgSmall::THREADS, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    int64_t grid = (int64_t)cus * per_cu;
    if (grid > items) grid = items;
    hipLaunchKernelGGL((batch_bound_kernel<CfgSmall>), dim3((unsigned)grid), dim3(CfgSmall::THREADS), 0,
                       s, probs, nprob, items, counter);
    return hipGetLastError();
}

int batch_gemm_blocks_per_cu(int tile) {
    return tile == 256 ? blocks_per_cu<KIND_KARATSUBA, CfgLargeShortK>() : blocks_per_cu<KIND_KARATSUBA, Once128>();
}

hipError_t launch_batch_gemm(const BatchGemm *probs, int nprob, int64_t items, int tile, int group,
                             int algo, uint32_t *counters, int grid_blocks, hipStream_t s) {
    if (items <= 0 || nprob <= 0) return hipSuccess;
    if ((tile != 128 && tile != 256) || group < 1) return hipErrorInvalidValue;
    if (grid_blocks <= 0) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            cus = 256;
        grid_blocks = cus * batch_gemm_blocks_per_cu(tile);
    }
    if ((int64_t)grid_blocks > items) grid_blocks = (int)items;
    if (tile == 256) {
        if (algo == 0) launch_batch_kind<KIND_KARATSUBA, CfgLargeShortK>(probs, nprob, items, group, counters, grid_blocks, s);
        else launch_batch_kind<KIND_4M, CfgLargeShortK>(probs, nprob, items, group, counters, grid_blocks, s);
    } else {
        if (algo == 0) launch_batch_kind<KIND_KARATSUBA, Once128>(probs, nprob, items, group, counters, grid_blocks, s);
        else launch_batch_kind<KIND_4M, Once128>(probs, nprob, items, group, counters, grid_blocks, s);
    }
    return hipGetLastError();
}

}  // namespace ozc
