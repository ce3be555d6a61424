// Pair phase of the MCPT(2) sweep in FP64 on CDNA4 matrix cores.
//
// For a stored pair (X, Y) with V = V_XY (nX x nY, rows (i,a) of X, columns
// (j,b) of Y) and the spin-adapted monomer combinations M = 2T - S(T):
//
//   Tau  = D_XY * (V + M_X V + V M_Y^T)       Eq. 59: source + T_X and T_Y couplings
//   E_D2 = 4 <V, Tau>                          Eq. 55
//   G_X += Tau V^T,   G_Y += Tau^T V           Eq. 58: the pair term seen from X and from Y
//
// (the Eq. 58 pair term of monomer X is G_X + G_X^T, formed where G is read, so a contribution
// may be put on either side of the diagonal).  The four products are dense n x n x n
// contractions on the FP64 matrix instructions.
//
// Structure.  Persistent workgroups walk the pair list; workgroup b runs on
// XCD b % 8 and each XCD takes a contiguous range of the monomer-sorted pairs,
// so the M and G blocks it touches stay in its L2.  Two variants:
//  * LDS-resident V (pairs for which pair_fits_lds): eight wavefronts (two per SIMD), one workgroup
//    per CU, v_mfma_f64_4x4x4 on 8 x 8 blocks (pair_body_lds).  V is staged once per pair into LDS
//    and every product reads it from there: V is streamed from HBM once per pass, and the L2 is
//    asked for the next pair's V behind the Tau tasks.  M and Tau (a scratch slot per workgroup)
//    come from L2 in fragment order.
//  * V from L2 (larger pairs): four wavefronts, two workgroups per CU, v_mfma_f64_16x16x4 on 3 x 3
//    super-blocks of 16 x 16 tiles (accumulators in registers, each operand fragment reused three
//    times); whole super-blocks go round-robin to the wavefronts and the super-blocks left over
//    as 1 x 3 row strips.  Task shapes are compile-time (3 x 3, 1 x 3 or a single tile) so each MFMA
//    block is straight-line code.  A wave raises its issue priority while it runs an MFMA block.
//
// The rest of this comment is about the 16 x 16 tiles of the second variant.
// Operand layout of the instruction (measured): A lane l = (row l%16, k l/16),
// B lane l = (k l/16, column l%16), accumulator element t of lane l = (row
// l/16 + 4t, column l%16).  A 16-deep k chunk is loaded as 4 contiguous values
// per lane, so lane l covers k = k0 + 4*(l/16) + s at step s for both operands.
#include <algorithm>

#include "mcpt_internal.hpp"

namespace mcpt {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kThreadsL = 512;   // LDS-resident V: eight wavefronts, one workgroup per CU
constexpr int kThreadsG = 256;   // V from L2: four wavefronts, two workgroups per CU
constexpr int kSB = 3;           // super-block edge in tiles
constexpr int kXcds = 8;
constexpr int kLdsPair = 20408;  // LDS doubles (163,264 B) for V (nx8 rows of ldv) and the energy differences
constexpr int kEnergySlots = 64; // LDS doubles for the parts of E_D2

template <int R, int C>
struct Shape {
    static constexpr int NR = R, NC = C;
};

__device__ inline d4 mfma(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ inline d4 load4(const double* p) { return *reinterpret_cast<const d4*>(p); }

// M[r][k .. k+3] (k a multiple of 4) in fragment order
__device__ inline d4 load4_frag(const double* m, int np, int r, int k) {
    const double* p = m + frag_at(np, r, k);
    const d2 lo = *reinterpret_cast<const d2*>(p);
    const d2 hi = *reinterpret_cast<const d2*>(p + 16);
    return d4{lo.x, lo.y, hi.x, hi.y};
}

__device__ inline void split(const d4& v, double (&o)[4]) {
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
}

__device__ inline int acc_row(int lane, int t) { return (lane >> 4) + 4 * t; }
__device__ inline int acc_col(int lane) { return lane & 15; }

template <int NR, int NC>
__device__ inline void zero(d4 (&acc)[NR][NC]) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[i][j] = d4(0.0);
}

template <int NR, int NC>
__device__ inline void mma_block(d4 (&acc)[NR][NC], const double (&a)[NR][4], const double (&b)[NC][4]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[i][j] = mfma(a[i][s], b[j][s], acc[i][j]);
    __builtin_amdgcn_s_setprio(0);
}

struct PairView {
    const double* V;      // nX x nY, row-major, global
    const double* MX;     // npX x npX
    const double* MY;     // npY x npY
    const double* dX;     // e_i - e_a over rows (i,a) of X
    const double* dY;     // e_j - e_b over columns (j,b) of Y
    double* GX;
    double* GY;
    int nX, npX;
    int nY, npY;
    int nx8, ny8;         // nX, nY rounded up to the 8 x 8 blocks of the LDS variant
    int ldv;              // LDS row stride of V when staged (ny8 + 4)
};

// ---------------------------------------------------------------------------
// V staged in LDS (sV: nx8 rows, row stride ldv, zero past nX and nY): products on
// v_mfma_f64_4x4x4, whose four independent 4 x 4 x 4 blocks q = 2 qr + qc are laid
// out as one 8 x 8 output block.  Lane 16 g + 4 q + r holds A[4 qr + r][k], B[k][4 qc + r]
// and D[4 qr + g][4 qc + r]; both operands are read twice (by the two qc or qr), which
// the LDS and the L1 serve as broadcasts.  An 8-deep k chunk is two steps, k = k0 + 2 g + s,
// so operands with k contiguous load two steps at once.
// ---------------------------------------------------------------------------
struct Lane8 {
    int k;      // 2 g: k of step 0 within a chunk
    int a, b;   // row of the A fragment, column of the B fragment
    int r, c;   // row and column of the accumulator
    int t, tT;  // place of the accumulator in its block in fragment order, and in the transposed block
    int t2, tT2; // place of the pair of columns (rows) that pair_cols (pair_rows) gives this lane
    bool second; // ... which belongs to the second block: for pair_cols; for pair_rows: secondT
    bool secondT;
};

__device__ __forceinline__ Lane8 lane8(int lane) {
    const int g = lane >> 4, qr = (lane >> 3) & 1, qc = (lane >> 2) & 1, r = lane & 3;
    const int row = 4 * qr + g, col = 4 * qc + r;
    return {2 * g, 4 * qr + r, 4 * qc + r, row, col, (col >> 1) * 16 + row * 2 + (col & 1),
            (row >> 1) * 16 + col * 2 + (row & 1), (col >> 1) * 16 + row * 2, (2 * qr + (g >> 1)) * 16 + col * 2,
            (r & 1) != 0, (g & 1) != 0};
}

typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// Accumulators x, y of two blocks, one value per lane each, to two values of one block per lane, so that they
// leave as one 16-byte store: two columns (lanes with odd columns take y's) ...
__device__ __forceinline__ d2 pair_cols(double x, double y, bool odd) {
    const double send = odd ? x : y;
    const u2 w = __builtin_bit_cast(u2, send);
    u2 v;
    v.x = __builtin_amdgcn_mov_dpp(w.x, 0xB1, 0xf, 0xf, false)   /* quad_perm 1,0,3,2 */;
    v.y = __builtin_amdgcn_mov_dpp(w.y, 0xB1, 0xf, 0xf, false);
    const double got = __builtin_bit_cast(double, v);
    return odd ? d2{got, y} : d2{x, got};
}

// ... or two rows (the odd 16-lane rows, which hold the odd rows, take y's)
__device__ __forceinline__ d2 pair_rows(double x, double y) {
    const u2 a = __builtin_bit_cast(u2, x), b = __builtin_bit_cast(u2, y);
    const auto lo = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
    return d2{__builtin_bit_cast(double, u2{lo[0], hi[0]}), __builtin_bit_cast(double, u2{lo[1], hi[1]})};
}

__device__ __forceinline__ d2 load2(const double* p) { return *reinterpret_cast<const d2*>(p); }

// A task's output: N or (X = 1, hr or hc) N + 1 rows and columns of blocks.  The product loops exist for each of
// the sizes, the epilogues, which run once per task, for all: with a copy for each, a pair's phases no longer fit
// the instruction cache, and the epilogues took as long as the products.
struct Extra {
    int hr, hc;   // 0 or 1
};

// Nothing but matrix instructions between the fences, then eight wait states, and the operands live until
// behind those: a v_mfma_f64_4x4x4 still reads its A and B registers when the instructions behind it issue, and a
// vector instruction that wrote one of them right behind it (an address formed in the last fragment's
// registers) spoiled the product.  The compiler keeps no distance there and no published table names one, so
// the eight states are what s_nop takes in one instruction, not a derived bound; the operands of the empty
// statements keep the register allocator from giving those registers away inside the fences.  The
// disassembly of the built library is tested for it.
template <int NR, int NC, int A>
__device__ __forceinline__ void mma8(double (&acc)[A][A], const double (&a)[NR][2], const double (&b)[NC][2]) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7");
#pragma unroll
    for (int i = 0; i < NR; ++i) asm volatile("" ::"v"(a[i][0]), "v"(a[i][1]));
#pragma unroll
    for (int j = 0; j < NC; ++j) asm volatile("" ::"v"(b[j][0]), "v"(b[j][1]));
    __builtin_amdgcn_sched_barrier(0);
}

// acc += A B over K chunks of 8, A's and B's fragments from la(k, a) and lb(k, b): two sets of
// fragments, the next chunk's reads in flight while this one is multiplied
template <int NR, int NC, int A, class LA, class LB>
__device__ __forceinline__ void product8(double (&acc)[A][A], int K, LA&& la, LB&& lb) {
    double a0[NR][2], b0[NC][2], a1[NR][2], b1[NC][2];
    auto step = [&](int k, const double (&a)[NR][2], const double (&b)[NC][2], double (&an)[NR][2],
                    double (&bn)[NC][2]) __attribute__((always_inline)) {
        const int kn = min(k + 1, K - 1);
        la(kn, an);
        lb(kn, bn);
        mma8<NR, NC, A>(acc, a, b);
    };
    la(0, a0);
    lb(0, b0);
    int k = 0;
#pragma unroll 1
    for (; k + 1 < K; k += 2) {
        step(k, a0, b0, a1, b1);
        step(k + 1, a1, b1, a0, b0);
    }
    if (k < K) mma8<NR, NC, A>(acc, a0, b0);
}

// fragments of N row blocks (from block rb) of a global matrix in fragment order, kb blocks per row
template <int N>
struct GlbFrags {
    const char* base;
    uint32_t off, step;
    __device__ __forceinline__ GlbFrags(const double* m, int kb, int rb, const Lane8& l, int row)
        : base(reinterpret_cast<const char*>(m) + (int64_t)rb * kb * 512), off((8 * l.k + 2 * row) * 8),
          step(kb * 512) {}
    __device__ __forceinline__ void operator()(int k, double (&f)[N][2]) const {
        const char* q = base + k * 512;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uint32_t o = off;
            asm("" : "+v"(o));   // keeps the lane's part a 32-bit offset beside the uniform address
            const d2 v = *reinterpret_cast<const d2*>(q + (int64_t)i * step + o);
            f[i][0] = v.x;
            f[i][1] = v.y;
        }
    }
};

// fragments of N row blocks (from row r) of V in LDS, k contiguous
template <int N>
struct LdsRows {
    const double* row;
    int step;
    __device__ __forceinline__ LdsRows(const double* sV, int ld, int r, int lk) : row(sV + r * ld + lk), step(8 * ld) {}
    __device__ __forceinline__ void operator()(int k, double (&f)[N][2]) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const d2 v = load2(row + i * step + 8 * k);
            f[i][0] = v.x;
            f[i][1] = v.y;
        }
    }
};

// fragments of N column blocks (from column c) of V in LDS, k along the rows
template <int N>
struct LdsCols {
    const double* col;
    int ld;
    __device__ __forceinline__ LdsCols(const double* sV, int ld_, int c, int lk) : col(sV + lk * ld_ + c), ld(ld_) {}
    __device__ __forceinline__ void operator()(int k, double (&f)[N][2]) const {
        const double *v0 = col + 8 * k * ld, *v1 = v0 + ld;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            f[j][0] = v0[8 * j];
            f[j][1] = v1[8 * j];
        }
    }
};

// B blocks of 8 cut into m segments of s or s + 1 blocks (s = 1: of one), `longer` of the longer ones first
struct Cut {
    int s, m, longer;
    __device__ __forceinline__ int start(int i) const { return i * s + min(i, longer); }
    __device__ __forceinline__ int more(int i) const { return i < longer ? 1 : 0; }
};

__device__ __forceinline__ Cut cut(int B, int s) {
    Cut c;
    c.s = s;
    c.m = s == 1 ? B : (B + s) / (s + 1);
    c.longer = B - s * c.m;
    return c;
}

// Segments of 4 or 5 blocks (17 blocks, n = 135: 5+4+4+4), 2 or 3, or single ones: the longest that R and C can
// be cut into, and not 4 or 5 where that leaves too few tasks for eight waves.  2,372 pairs, us a launch with the
// line at 20, 40 and 64 blocks (Tau: R C, G: R^2 + C^2): n = 32 (16 and 32 blocks) 108, 103, 103; n = 40 (25 and
// 50) 166, 133, 123; n = 64 (64 and 128) 218 below each, 242 with Tau in shorter ones; n = 72 (81 and 162) 282,
// and 310.  Single blocks in place of 2 or 3 gain nothing at n = 16 and lose from n = 27 on (103, 125).
// Sides of 6, 7 and 11 blocks cannot be cut into 4 and 5.
__device__ __forceinline__ int seg_len(int R, int C, int blocks) {
    auto cuts = [](int B, int s) { return B >= s * ((B + s) / (s + 1)); };
    if (blocks >= 64 && cuts(R, 4) && cuts(C, 4)) return 4;
    return R >= 2 && C >= 2 ? 2 : 1;
}

// Task t of the rectangles of two cuts, the larger ones first; but the fifth is a small one: waves 0 and 4
// share a SIMD, and wave 0 has the largest (17 x 17 blocks: 25 + 16 against 20 + 20 on the other SIMDs).
__device__ __forceinline__ void rect_task(const Cut& r, const Cut& c, int t, int& i, int& j) {
    const int lr = r.longer, lc = c.longer, sr = r.m - lr, sc = c.m - lc, n = r.m * c.m;
    int u = t;
    if (sr * sc > 0 && n > 8 && t >= 4) u = t == 4 ? n - 1 : t - 1;
    if (u < lr * lc) {
        i = u / lc;
        j = u - i * lc;
        return;
    }
    u -= lr * lc;
    if (u < lr * sc) {
        i = u / sc;
        j = lc + u - i * sc;
        return;
    }
    u -= lr * sc;
    if (u < sr * lc) {
        i = u / lc;
        j = u - i * lc;
        i += lr;
        return;
    }
    u -= sr * lc;
    i = u / sc;
    j = lc + u - i * sc;
    i += lr;
}

template <int S, int E>
struct Seg8 {
    static constexpr int N = S, X = E;
};

template <class F>
__device__ __forceinline__ void with_seg(int s, F&& f) {
    if (s == 4) f(Seg8<4, 1>{});
    else if (s == 2) f(Seg8<2, 1>{});
    else f(Seg8<1, 0>{});
}

// ---------------------------------------------------------------------------
// V read from global memory (pairs too large for LDS)
// ---------------------------------------------------------------------------
template <int NR, int NC>
__device__ void tau_sb_glb(const PairView& p, int r0, int c0, int lane, d4 (&acc)[NR][NC]) {
    const int lr = lane & 15, lk = (lane >> 4) * 4;
    for (int k0 = 0; k0 < p.npX; k0 += 16) {
        double a[NR][4], b[NC][4];
#pragma unroll
        for (int i = 0; i < NR; ++i) split(load4_frag(p.MX, p.npX, (r0 + i) * 16 + lr, k0 + lk), a[i]);
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = (c0 + j) * 16 + lr;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kk = k0 + lk + s;
                b[j][s] = (kk < p.nX && c < p.nY) ? p.V[(int64_t)kk * p.nY + c] : 0.0;
            }
        }
        mma_block(acc, a, b);
    }
    for (int k0 = 0; k0 < p.npY; k0 += 16) {
        double a[NR][4], b[NC][4];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int r = (r0 + i) * 16 + lr;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kk = k0 + lk + s;
                a[i][s] = (r < p.nX && kk < p.nY) ? p.V[(int64_t)r * p.nY + kk] : 0.0;
            }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) split(load4_frag(p.MY, p.npY, (c0 + j) * 16 + lr, k0 + lk), b[j]);
        mma_block(acc, a, b);
    }
}

template <int NR, int NC>
__device__ void gx_sb_glb(const PairView& p, const double* tau, int r0, int q0, int lane, d4 (&acc)[NR][NC]) {
    const int lr = lane & 15, lk = (lane >> 4) * 4;
    for (int k0 = 0; k0 < p.npY; k0 += 16) {
        double a[NR][4], b[NC][4];
#pragma unroll
        for (int i = 0; i < NR; ++i) split(load4(tau + (int64_t)((r0 + i) * 16 + lr) * p.npY + k0 + lk), a[i]);
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int q = (q0 + j) * 16 + lr;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kk = k0 + lk + s;
                b[j][s] = (q < p.nX && kk < p.nY) ? p.V[(int64_t)q * p.nY + kk] : 0.0;
            }
        }
        mma_block(acc, a, b);
    }
}

template <int NR, int NC>
__device__ void gy_sb_glb(const PairView& p, const double* tau, int c0, int q0, int lane, d4 (&acc)[NR][NC]) {
    const int lr = lane & 15, lk = (lane >> 4) * 4;
    for (int k0 = 0; k0 < p.npX; k0 += 16) {
        double a[NR][4], b[NC][4];
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int s = 0; s < 4; ++s) a[i][s] = tau[(int64_t)(k0 + lk + s) * p.npY + (c0 + i) * 16 + lr];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int q = (q0 + j) * 16 + lr;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kk = k0 + lk + s;
                b[j][s] = (kk < p.nX && q < p.nY) ? p.V[(int64_t)kk * p.nY + q] : 0.0;
            }
        }
        mma_block(acc, a, b);
    }
}

// ---------------------------------------------------------------------------
// task lists: full super-blocks round-robin over the waves (partial edge
// super-blocks as single tiles of the same wave), the remainder tile by tile
// ---------------------------------------------------------------------------
struct Grid {
    int RT, CT, SR, SC, n;    // tiles, super-blocks per dimension, super-block count
};

__device__ inline Grid make_grid(int RT, int CT) {
    Grid g;
    g.RT = RT;
    g.CT = CT;
    g.SR = (RT + kSB - 1) / kSB;
    g.SC = (CT + kSB - 1) / kSB;
    g.n = g.SR * g.SC;
    return g;
}

// Visit the tasks of `wave` over the concatenation of grids g0 and g1 (g1 may be
// empty): f(which, r0, c0, shape) in tile coordinates, shape Shape<3,3>,
// Shape<1,3> or Shape<1,1>.  Full super-blocks go round-robin to the waves; the
// super-blocks left over after the last full round are cut into 1 x 3 row
// strips (three independent accumulators keep the MFMA pipe busy, where single
// tiles would wait on each k chunk) and dealt out one by one.  Edge super-blocks
// narrower than three tiles run as single tiles.
template <class F>
__device__ inline void for_tasks(const Grid& g0, const Grid& g1, int wave, int nwaves, F&& f) {
    const int total = g0.n + g1.n;
    const int full = total - total % nwaves;
    for (int sb = wave; sb < full; sb += nwaves) {
        const int which = sb >= g0.n ? 1 : 0;
        const Grid& g = which ? g1 : g0;
        const int s = which ? sb - g0.n : sb;
        const int r0 = (s / g.SC) * kSB, c0 = (s % g.SC) * kSB;
        const int nr = min(kSB, g.RT - r0), nc = min(kSB, g.CT - c0);
        if (nr == kSB && nc == kSB) {
            f(which, r0, c0, Shape<kSB, kSB>{});
        } else {
            for (int i = 0; i < nr; ++i) {
                if (nc == kSB) f(which, r0 + i, c0, Shape<1, kSB>{});
                else
                    for (int j = 0; j < nc; ++j) f(which, r0 + i, c0 + j, Shape<1, 1>{});
            }
        }
    }
    int idx = 0;
    for (int sb = full; sb < total; ++sb) {
        const int which = sb >= g0.n ? 1 : 0;
        const Grid& g = which ? g1 : g0;
        const int s = which ? sb - g0.n : sb;
        const int r0 = (s / g.SC) * kSB, c0 = (s % g.SC) * kSB;
        const int nr = min(kSB, g.RT - r0), nc = min(kSB, g.CT - c0);
        for (int i = 0; i < nr; ++i) {
            if (nc == kSB) {
                if (idx++ % nwaves == wave) f(which, r0 + i, c0, Shape<1, kSB>{});
            } else {
                for (int j = 0; j < nc; ++j, ++idx)
                    if (idx % nwaves == wave) f(which, r0 + i, c0 + j, Shape<1, 1>{});
            }
        }
    }
}

// G block contributions: FP64 atomics into G, or (deterministic mode) plain
// stores of the whole padded block into the pair's partial slot
template <int NR, int NC>
__device__ inline void atomic_flush(double* G, double* part, int ld, int n, int r0, int q0, int lane,
                                    const d4 (&acc)[NR][NC]) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = (q0 + j) * 16 + acc_col(lane);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int r = (r0 + i) * 16 + acc_row(lane, t);
                if (part) part[(int64_t)r * ld + c] = acc[i][j][t];
                else if (r < n && c < n) unsafeAtomicAdd(G + (int64_t)r * ld + c, acc[i][j][t]);
            }
        }
}

// the same for the 8 x 8 blocks of the LDS variant; a stored block off the diagonal holds its mirror
// image's part too, so that one is set to zero
template <int NR, int NC, int X>
__device__ __forceinline__ void flush8(double* G, double* part, int ld, int n, int r0, int q0, Extra e, const Lane8& l,
                                       const double (&acc)[NR + X][NC + X]) {
    double* dst = (part ? part : G) + (int64_t)(r0 + l.r) * ld + q0 + l.c;
    double* mirror = part + (int64_t)(q0 + l.r) * ld + r0 + l.c;
#pragma unroll
    for (int i = 0; i < NR + X; ++i) {
        if (i == NR && !e.hr) break;
        const bool row = r0 + 8 * i + l.r < n;
#pragma unroll
        for (int j = 0; j < NC + X; ++j) {
            if (j == NC && !e.hc) break;
            if (part) {
                dst[8 * j] = acc[i][j];
                if (r0 != q0) mirror[(int64_t)8 * j * ld + 8 * i] = 0.0;
            } else if (row && q0 + 8 * j + l.c < n) {
                unsafeAtomicAdd(dst + 8 * j, acc[i][j]);
            }
        }
        dst += 8 * ld;
    }
}

__device__ inline double wave_sum(double x) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

__device__ inline int64_t pair_for(int64_t it, int64_t n_pair) {
    const int g = gridDim.x;
    if (g % kXcds != 0) return (int64_t)blockIdx.x + it * g;
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds, per = g / kXcds;
    const int64_t begin = n_pair * xcd / kXcds, end = n_pair * (xcd + 1) / kXcds;
    const int64_t p = begin + local + it * per;
    return p < end ? p : INT64_MAX;
}

__device__ inline PairView make_view(const PairDesc& pd, const MonoDesc* monos, const double* dif,
                                     const double* V, const double* M, double* G) {
    const MonoDesc dx = monos[pd.x], dy = monos[pd.y];
    PairView p;
    p.V = V + pd.v_off;
    p.MX = M + dx.mat_off;
    p.MY = M + dy.mat_off;
    p.dX = dif + dx.dif_off;
    p.dY = dif + dy.dif_off;
    p.GX = G + dx.mat_off;
    p.GY = G + dy.mat_off;
    p.nX = dx.n;
    p.npX = dx.np;
    p.nY = dy.n;
    p.npY = dy.np;
    p.nx8 = (dx.n + 7) & ~7;
    p.ny8 = (dy.n + 7) & ~7;
    p.ldv = p.ny8 + 4;
    return p;
}

// Pairs read from L2, one pair per workgroup.  DIMER (1: every monomer of one size, 2: any
// sizes, from the pair's descriptor) adds the dimer-internal source of po to the numerator of
// Tau and keeps Tau.
template <int NT, int DIMER>
__device__ inline void pair_body_glb(const PairDesc* __restrict__ pairs, int64_t n_pair,
                                 const MonoDesc* __restrict__ monos, const double* __restrict__ dif,
                                 const double* __restrict__ V, const double* __restrict__ M,
                                 double* __restrict__ G, double* __restrict__ scratch, int64_t slot_elems,
                                 double* __restrict__ ed2, int couple, const ClState* __restrict__ cl,
                                 PartOut po, double* red) {
    constexpr int NW = NT / 64;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double* tau = scratch + (int64_t)blockIdx.x * slot_elems;
    for (int64_t it = 0;; ++it) {
        const int64_t pi = pair_for(it, n_pair);
        if (pi >= n_pair) break;
        const PairDesc pd = pairs[pi];
        if (cl && cl[pd.cluster].done) continue;   // cluster stopped: uniform over the workgroup
        const PairView p = make_view(pd, monos, dif, V, M, G);
        const int RB = p.npX / 16, CB = p.npY / 16;

        // ---- Tau = D_XY * (V + M_X V + V M_Y^T), E_D2 = 4 <V, Tau> ----
        double epart = 0.0;
        // the pair's dimer-internal source and Tau (sizes and offsets from its descriptor)
        int dvx = 1, dvy = 1, dm1 = 0, dm2 = 0;
        const double *Sp = nullptr, *Y1p = nullptr, *Y2p = nullptr;
        double* Tp = nullptr;
        if (DIMER == 1) {   // one size: every pair's matrices np x np at orig * mat_stride
            dvx = dvy = po.v;
            dm1 = dm2 = p.npY;
            Sp = po.S + pd.orig * po.mat_stride;
            Y1p = po.Y1 + pd.orig * po.mat_stride;
            Y2p = po.Y2 + pd.orig * po.mat_stride;
            Tp = po.tau_out + pd.orig * po.mat_stride;
        } else if (DIMER == 2) {
            const DimerDesc& e = po.dd[pd.orig];
            dvx = e.vx;
            dvy = e.vy;
            dm1 = e.m1;
            dm2 = e.m2;
            Sp = po.S + e.tau_off;
            Y1p = po.Y1 + e.y1_off;
            Y2p = po.Y2 + e.y2_off;
            Tp = po.tau_out + e.tau_off;
        }
        for_tasks(make_grid(RB, CB), make_grid(0, 0), wave, NW, [&](int, int r0, int c0, auto shape) {
            constexpr int NR = decltype(shape)::NR, NC = decltype(shape)::NC;
            d4 acc[NR][NC];
            zero(acc);
            tau_sb_glb(p, r0, c0, lane, acc);
            // Epilogue, one tile column at a time: its inputs are gathered before its stores to
            // the Tau slot (a global store orders later global loads behind it), indices are
            // clamped into the valid block and the padding is masked by selects, so the loads
            // issue back to back with one wait instead of a branch and a round trip per element.
            // dX and dY are read at the padded indices directly (zero beyond n; masked).
            const double *dXs = p.dX, *dYs = p.dY;
            double dxr[NR][4];
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t) dxr[i][t] = dXs[(r0 + i) * 16 + acc_row(lane, t)];
            if constexpr (DIMER == 0) {
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int c = (c0 + j) * 16 + acc_col(lane);
                    const int cc = min(c, p.nY - 1);
                    const double dyc = dYs[c];
                    double vv[NR][4];
#pragma unroll
                    for (int i = 0; i < NR; ++i)
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int rr = min((r0 + i) * 16 + acc_row(lane, t), p.nX - 1);
                            vv[i][t] = p.V[(int64_t)rr * p.nY + cc];
                        }
#pragma unroll
                    for (int i = 0; i < NR; ++i)
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int r = (r0 + i) * 16 + acc_row(lane, t);
                            const bool ok = r < p.nX && c < p.nY;
                            const double dinv = recip(dxr[i][t] + dyc);
                            const double tv = ok ? dinv * (vv[i][t] + acc[i][j][t]) : 0.0;
                            epart += ok ? vv[i][t] * tv : 0.0;
                            if (couple) tau[(int64_t)r * p.npY + c] = tv;
                        }
                }
            } else {
                // with the dimer source, four reads per element (V, S and the two cross-ring
                // products at the clamped element rr = (ii,a), cc = (jj,b)): one tile at a time,
                // or the gathered values of a whole tile column spill
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int c = (c0 + j) * 16 + acc_col(lane);
                    const int cc = min(c, p.nY - 1);
                    const double dyc = dYs[c];
#pragma unroll
                    for (int i = 0; i < NR; ++i) {
                        double vv[4], dsrc[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int rr = min((r0 + i) * 16 + acc_row(lane, t), p.nX - 1);
                            const int r = (r0 + i) * 16 + acc_row(lane, t);
                            vv[t] = p.V[(int64_t)rr * p.nY + cc];
                            if (DIMER == 1) {
                                const int ii = rr / dvx, a = rr - ii * dvx, jj = cc / dvx, b = cc - jj * dvx;
                                dsrc[t] = Sp[(int64_t)r * p.npY + c] -
                                          Y1p[(int64_t)(ii * dvx + b) * dm1 + jj * dvx + a] -
                                          Y2p[(int64_t)(jj * dvx + a) * dm1 + ii * dvx + b];
                            } else {
                                const int ii = rr / dvx, a = rr - ii * dvx, jj = cc / dvy, b = cc - jj * dvy;
                                dsrc[t] = Sp[(int64_t)r * p.npY + c] -
                                          Y1p[(int64_t)(ii * dvy + b) * dm2 + jj * dvx + a] -
                                          Y2p[(int64_t)(jj * dvx + a) * dm1 + ii * dvy + b];
                            }
                        }
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int r = (r0 + i) * 16 + acc_row(lane, t);
                            const bool ok = r < p.nX && c < p.nY;
                            const double dinv = recip(dxr[i][t] + dyc);
                            const double tv = ok ? dinv * (vv[t] + dsrc[t] + acc[i][j][t]) : 0.0;
                            epart += ok ? vv[t] * tv : 0.0;
                            if (couple) tau[(int64_t)r * p.npY + c] = tv;
                            Tp[(int64_t)r * p.npY + c] = tv;
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        });
        epart = wave_sum(epart);
        if (lane == 0) red[wave] = epart;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int w = 0; w < NW; ++w) s += red[w];
            ed2[pd.orig] = 4.0 * s;
        }
        if (couple) {
            // ---- G_X += Tau V^T (RB x RB tiles), G_Y += Tau^T V (CB x CB tiles) ----
            for_tasks(make_grid(RB, RB), make_grid(CB, CB), wave, NW, [&](int which, int r0, int c0, auto shape) {
                constexpr int NR = decltype(shape)::NR, NC = decltype(shape)::NC;
                d4 acc[NR][NC];
                zero(acc);
                if (which == 0) {
                    gx_sb_glb(p, tau, r0, c0, lane, acc);
                    atomic_flush(p.GX, po.part ? po.part + po.off[pi] : nullptr, p.npX, p.nX, r0, c0, lane, acc);
                } else {
                    gy_sb_glb(p, tau, r0, c0, lane, acc);
                    atomic_flush(p.GY, po.part ? po.part + po.off[pi] + (int64_t)p.npX * p.npX : nullptr, p.npY,
                                 p.nY, r0, c0, lane, acc);
                }
            });
        }
        __syncthreads();
    }
}

// V resident in LDS (the pair list given to it holds only pairs that fit).
//
// What bounds it: the FP64 matrix pipe, and what does not overlap with it.  v_mfma_f64_16x16x4 sustains
// 47 TFLOP/s on this device, v_mfma_f64_4x4x4 76 (both as mcpt_device_rates streams them), and its blocks pad n = 135
// to 136 instead of 144.
// On the 1000-monomer crystal the mean of four coupled launches and the energy pass is 16.2 ms (46.0 TFLOP/s;
// 19.9 ms with 16 x 16 x 4 tiles).  Of the 258,000 cycles of a coupled pair (n = 135) the products take 180,000 (157,000 at the
// pipe's 16 cycles each), staging V 14,000, the stores of Tau and Tau^T 27,000 and the atomics behind the last products most of
// the rest: a store or an atomic instruction occupies a CU's memory path for 90 to 200 cycles, whatever its width.
// ldv = ny8 + 4 puts 8 consecutive rows on distinct 8-bank groups (row reads) and the 4 row pairs of a column read on
// distinct 16-bank groups.  Tried: tasks of (4-5) x (8-9) blocks, one per wave (17.3 ms: all waves store at
// once); one code for the four task sizes with the odd row and column behind branches (17.6); twelve waves (27.5:
// spills); reading LDS fragments without a chunk's lead (18.7).
template <int DIMER>
__device__ __forceinline__ void pair_body_lds(const PairDesc* __restrict__ pairs, int64_t n_pair,
                                     const MonoDesc* __restrict__ monos, const double* __restrict__ dif,
                                     const double* __restrict__ V, const double* __restrict__ M,
                                     double* __restrict__ G, double* __restrict__ scratch, int64_t slot_elems,
                                     double* __restrict__ ed2, int couple, const ClState* __restrict__ cl,
                                     PartOut po, double* sV, double* red, int* next) {
    constexpr int NT = kThreadsL, NW = NT / 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int first = wave;
    // one wave of each SIMD goes first, the other fills its gaps
    if (wave < 4) __builtin_amdgcn_s_setprio(1);
    const Lane8 l = lane8(lane);
    double* tau = scratch + (int64_t)blockIdx.x * slot_elems;
    double sink = 0.0;
    for (int64_t it = 0;; ++it) {
        const int64_t pi = pair_for(it, n_pair);
        if (pi >= n_pair) break;
        const PairDesc pd = pairs[pi];
        if (cl && cl[pd.cluster].done) continue;   // cluster stopped: uniform over the workgroup
        const PairView p = make_view(pd, monos, dif, V, M, G);
        const int RB = p.nx8 / 8, CB = p.ny8 / 8;
        double* sD = sV + p.nx8 * p.ldv;
        double* tauT = tau + (int64_t)p.nx8 * p.ny8;   // Tau (rows of X) and Tau^T in fragment order
        {   // Stage V, zero-padded to nx8 rows of ldv; loads batched, nine rows per wave of three times 64 columns, or
            // three of one for rows of at most 64, where most of those would be empty: 2,372 pairs of n = 16 took
            // 80 us a launch with 9 x 3 throughout, 73 with 9 x 1 and take 64; of n = 51, 195, 188 and 185.
            auto stage = [&](auto cols) __attribute__((always_inline)) {
                constexpr int kCols = decltype(cols)::N, kRows = kCols == 1 ? 3 : 9;
                for (int rb = wave; rb < p.nx8; rb += NW * kRows)
                    for (int cb = 0; cb < p.ldv; cb += 64 * kCols) {
                        double tmp[kRows][kCols];
#pragma unroll
                        for (int k = 0; k < kRows; ++k)
#pragma unroll
                            for (int m = 0; m < kCols; ++m) {
                                const int r = rb + NW * k, c = cb + lane + 64 * m;
                                tmp[k][m] = (r < p.nX && c < p.nY) ? p.V[(int64_t)r * p.nY + c] : 0.0;
                            }
#pragma unroll
                        for (int k = 0; k < kRows; ++k)
#pragma unroll
                            for (int m = 0; m < kCols; ++m) {
                                const int r = rb + NW * k, c = cb + lane + 64 * m;
                                if (r < p.nx8 && c < p.ldv) sV[r * p.ldv + c] = tmp[k][m];
                            }
                    }
            };
            if (p.ldv <= 64) stage(Seg8<1, 0>{});
            else stage(Seg8<3, 0>{});
            // the energy differences of X's rows and Y's columns (zero in the padding) for the epilogue
            for (int k = threadIdx.x; k < p.nx8 + p.ny8; k += NT) sD[k] = k < p.nx8 ? p.dX[k] : p.dY[k - p.nx8];
            if (threadIdx.x < kEnergySlots) red[threadIdx.x] = 0.0;
            if (threadIdx.x < 2) next[threadIdx.x] = NW;
            __syncthreads();
        }

        // the pair's dimer-internal source and Tau (sizes and offsets from its descriptor)
        int dvx = 1, dvy = 1, dm1 = 0, dm2 = 0;
        const double *Sp = nullptr, *Y1p = nullptr, *Y2p = nullptr;
        double* Tp = nullptr;
        if (DIMER == 1) {   // one size: every pair's matrices np x np at orig * mat_stride
            dvx = dvy = po.v;
            dm1 = dm2 = p.npY;
            Sp = po.S + pd.orig * po.mat_stride;
            Y1p = po.Y1 + pd.orig * po.mat_stride;
            Y2p = po.Y2 + pd.orig * po.mat_stride;
            Tp = po.tau_out + pd.orig * po.mat_stride;
        } else if (DIMER == 2) {
            const DimerDesc& e = po.dd[pd.orig];
            dvx = e.vx;
            dvy = e.vy;
            dm1 = e.m1;
            dm2 = e.m2;
            Sp = po.S + e.tau_off;
            Y1p = po.Y1 + e.y1_off;
            Y2p = po.Y2 + e.y2_off;
            Tp = po.tau_out + e.tau_off;
        }
        // Two phases of tasks, one code.  Tau = D_XY * (V + M_X V + V M_Y^T) and E_D2 by rectangles; then
        // (couple) what G_X = Tau V^T and G_Y = Tau^T V add to G + G^T, the only form G is used in: for two
        // segments i > j the sum G_ij + G_ji^T = Tau_i V_j^T + V_i Tau_j^T goes to block (i, j) alone, for
        // i = j the plain product.  As many multiplications as both full products, and 181 instead of 289
        // blocks of atomics at n = 135: FP64 atomics, 206 cycles for 64 lanes with every compute unit
        // adding, took as long as the products of this phase.  The first task of each wave is fixed, the others
        // go to the waves as they come free; E_D2 is summed by task, and repeats bitwise.
        double* px = po.part ? po.part + po.off[pi] : nullptr;
        double* py = px ? px + (int64_t)p.npX * p.npX : nullptr;
        const int st = seg_len(RB, CB, RB * CB), sx = seg_len(RB, RB, RB * RB + CB * CB),
                  sy = seg_len(CB, CB, RB * RB + CB * CB);
        const Cut tr = cut(RB, st), tc = cut(CB, st), cx = cut(RB, sx), cy = cut(CB, sy);
        const int nt = tr.m * tc.m, ox = cx.m * (cx.m - 1) / 2, oy = cy.m * (cy.m - 1) / 2;
        const bool by_task = nt <= kEnergySlots;   // otherwise E_D2 is summed by wave, the tasks dealt in turn
#pragma unroll 1
        for (int phase = 0; phase < (couple ? 2 : 1); ++phase) {
            const int total = phase == 0 ? nt : ox + oy + cx.m + cy.m;
#pragma unroll 1
            for (int t = first; t < total;) {
                // 0: Tau, 1: G_X, 2: G_Y; segment i of the rows and j of the columns
                const int u0 = phase == 0 ? t : t < ox + oy ? (t < ox ? t : t - ox) : t - ox - oy;
                const bool off = t < ox + oy;   // of the G tasks: i > j (two products each) before i = j
                const int kind = phase == 0 ? 0 : (off ? t < ox : u0 < cx.m) ? 1 : 2;
                const Cut cr = kind == 0 ? tr : kind == 1 ? cx : cy, cc = kind == 0 ? tc : cr;
                int i, j;
                if (kind == 0) {
                    rect_task(cr, cc, t, i, j);
                } else if (off) {
                    int u = u0;
                    i = 1;
                    while (u >= i) u -= i++;
                    j = u;
                } else {
                    i = j = kind == 1 ? u0 : u0 - cx.m;
                }
                const int rb = cr.start(i), cb = cc.start(j), r0 = 8 * rb, c0 = 8 * cb;
                const Extra e{__builtin_amdgcn_readfirstlane(cr.more(i)), __builtin_amdgcn_readfirstlane(cc.more(j))};
                double epart = 0.0;
                with_seg(cr.s, [&](auto seg) __attribute__((always_inline)) {
                    constexpr int N = decltype(seg)::N, X = decltype(seg)::X, NR = N, NC = N;
                    double acc[N + X][N + X] = {};
                    // the operand from global memory: M_X and M_Y, Tau, or Tau^T
                    const double* ga = kind == 0 ? p.MX : kind == 1 ? tau : tauT;
                    const double* gb = kind == 0 ? p.MY : ga;
                    const int ka = kind == 0 ? p.npX / 8 : kind == 1 ? CB : RB, kb = kind == 0 ? p.npY / 8 : ka;
                    // V by rows or by columns in LDS: a loop of its own for each, so that no wait is shared
                    auto products = [&](auto nr, auto nc) __attribute__((always_inline)) {
                        constexpr int NR = decltype(nr)::N, NC = decltype(nc)::N, A = N + X;
                        const GlbFrags<NR> fa(ga, ka, rb, l, l.a);
                        const GlbFrags<NC> fb(gb, kb, cb, l, l.b);
                        if (kind == 1) product8<NR, NC, A>(acc, CB, fa, LdsRows<NC>(sV, p.ldv, c0 + l.b, l.k));
                        else product8<NR, NC, A>(acc, RB, fa, LdsCols<NC>(sV, p.ldv, c0 + l.b, l.k));
                        if (kind != 0 && i == j) return;
                        if (kind == 2) product8<NR, NC, A>(acc, RB, LdsCols<NR>(sV, p.ldv, r0 + l.a, l.k), fb);
                        else product8<NR, NC, A>(acc, CB, LdsRows<NR>(sV, p.ldv, r0 + l.a, l.k), fb);
                    };
                    if (e.hr && e.hc) products(Seg8<N + X, 0>{}, Seg8<N + X, 0>{});
                    else if (e.hr) products(Seg8<N + X, 0>{}, Seg8<N, 0>{});
                    else if (e.hc) products(Seg8<N, 0>{}, Seg8<N + X, 0>{});
                    else products(Seg8<N, 0>{}, Seg8<N, 0>{});
                    if (kind) {
                        flush8<N, N, X>(kind == 1 ? p.GX : p.GY, kind == 1 ? px : py, kind == 1 ? p.npX : p.npY,
                                        kind == 1 ? p.nX : p.nY, r0, c0, e, l, acc);
                        return;
                    }
                    // Epilogue, two block columns at a time; the padding is masked by selects, so the
                    // reads issue back to back.  dX and dY are zero beyond n (masked).
                    double dxr[NR + X];
                    int vr[NR + X];
#pragma unroll
                    for (int i = 0; i < NR + X; ++i) {
                        const int r = r0 + 8 * (i == NR && !e.hr ? NR - 1 : i) + l.r;
                        dxr[i] = sD[r];
                        vr[i] = r * p.ldv;
                    }
#pragma unroll
                    for (int j0 = 0; j0 < NC + X; j0 += 2) {
                        if (j0 == NC && !e.hc) break;
                        const bool two = j0 + 1 < NC;   // NC is even, or 1
                        double tv[NR + X][2];
#pragma unroll
                        for (int jj = 0; jj < 2; ++jj) {
                            if (jj && !two) continue;
                            const int j = j0 + jj;
                            const int c = c0 + 8 * j + l.c;
                            const double dyc = sD[p.nx8 + c];
                            double vv[NR + X], dsrc[NR + X];
#pragma unroll
                            for (int i = 0; i < NR + X; ++i) {
                                vv[i] = sV[vr[i] + c];
                                dsrc[i] = 0.0;
                                if (DIMER) {
                                    const int r = r0 + 8 * (i == NR && !e.hr ? NR - 1 : i) + l.r;
                                    const int rr = min(r, p.nX - 1), cc = min(c, p.nY - 1);
                                    const int ovx = dvx, ovy = DIMER == 1 ? dvx : dvy;
                                    const int ii = rr / ovx, a = rr - ii * ovx, j1 = cc / ovy, b = cc - j1 * ovy;
                                    dsrc[i] = Sp[(int64_t)r * p.npY + c] -
                                              Y1p[(int64_t)(ii * ovy + b) * dm2 + j1 * ovx + a] -
                                              Y2p[(int64_t)(j1 * ovx + a) * dm1 + ii * ovy + b];
                                }
                            }
#pragma unroll
                            for (int i = 0; i < NR + X; ++i) {
                                if (i == NR && !e.hr) break;
                                const int r = r0 + 8 * i + l.r;
                                const bool ok = r < p.nX && c < p.nY;
                                const double dinv = recip(dxr[i] + dyc);
                                const double num = DIMER ? vv[i] + dsrc[i] + acc[i][j] : vv[i] + acc[i][j];
                                tv[i][jj] = ok ? dinv * num : 0.0;
                                epart += ok ? vv[i] * tv[i][jj] : 0.0;
                                if (DIMER) Tp[(int64_t)r * p.npY + c] = tv[i][jj];
                            }
                            if (DIMER) __builtin_amdgcn_sched_barrier(0);
                        }
                        if (couple) {
                            double* t0 = tau + (rb * CB + cb + j0) * 64;
                            double* tT0 = tauT + ((cb + j0) * RB + rb) * 64;
                            if (two) {
                                t0 += l.t2 + (l.second ? 64 : 0);
                                tT0 += l.tT2 + (l.secondT ? RB * 64 : 0);
#pragma unroll
                                for (int i = 0; i < NR + X; ++i) {
                                    if (i == NR && !e.hr) break;
                                    *reinterpret_cast<d2*>(t0 + i * CB * 64) = pair_cols(tv[i][0], tv[i][1], l.second);
                                    *reinterpret_cast<d2*>(tT0 + i * 64) = pair_rows(tv[i][0], tv[i][1]);
                                }
                            } else {
#pragma unroll
                                for (int i = 0; i < NR + X; ++i) {
                                    if (i == NR && !e.hr) break;
                                    t0[i * CB * 64 + l.t] = tv[i][0];
                                    tT0[i * 64 + l.tT] = tv[i][0];
                                }
                            }
                        }
                    }
                });
                if (kind == 0) {
                    epart = wave_sum(epart);
                    if (lane == 0) red[by_task ? t : wave] += epart;
                }
                if (phase == 0 && !by_task) {
                    t += NW;
                } else {
                    int n = 0;
                    if (lane == 0) n = atomicAdd(next + phase, 1);
                    t = __builtin_amdgcn_readfirstlane(n);
                }
            }
            if (phase == 1) break;
            if (wave & 2) {
                // ask the L2 for the next pair's V (waves 2, 3, 6, 7: their SIMDs have the smaller tasks and
                // would wait at the barrier)
                const int64_t pn = pair_for(it + 1, n_pair);
                if (pn < n_pair) {
                    const PairDesc nd = pairs[pn];
                    const int64_t nv = (int64_t)monos[nd.x].n * monos[nd.y].n;
                    const double* vn = V + nd.v_off;
                    for (int64_t e = ((wave >> 2) * 128 + (wave & 1) * 64 + lane) * 16; e < nv; e += NT / 2 * 16) sink += vn[e];
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                const int n = by_task ? nt : NW;
                double s = 0.0;
                for (int w = 0; w < n; ++w) s += red[w];
                ed2[pd.orig] = 4.0 * s;
            }
        }
        __syncthreads();
    }
    if (sink == 1.2345e300) ed2[0] = sink;   // keeps the prefetch loads; never true for finite inputs
}

template <int DIMER>
__global__ __launch_bounds__(kThreadsL) void pair_fp64_lds_kernel(
    const PairDesc* __restrict__ pairs, int64_t n_pair, const MonoDesc* __restrict__ monos,
    const double* __restrict__ dif, const double* __restrict__ V, const double* __restrict__ M,
    double* __restrict__ G, double* __restrict__ scratch, int64_t slot_elems,
    double* __restrict__ ed2, int couple, const Ctrl* __restrict__ ctrl,
    const ClState* __restrict__ cl, PartOut po) {
    if (ctrl && ctrl->done) return;
    __shared__ __align__(16) double sV[kLdsPair];
    __shared__ double red[kEnergySlots];
    __shared__ int next[2];
    pair_body_lds<DIMER>(pairs, n_pair, monos, dif, V, M, G, scratch, slot_elems, ed2, couple, cl, po, sV, red, next);
}

template <int DIMER>
__global__ __launch_bounds__(kThreadsG, 2) void pair_fp64_glb_kernel(
    const PairDesc* __restrict__ pairs, int64_t n_pair, const MonoDesc* __restrict__ monos,
    const double* __restrict__ dif, const double* __restrict__ V, const double* __restrict__ M,
    double* __restrict__ G, double* __restrict__ scratch, int64_t slot_elems,
    double* __restrict__ ed2, int couple, const Ctrl* __restrict__ ctrl,
    const ClState* __restrict__ cl, PartOut po) {
    if (ctrl && ctrl->done) return;
    __shared__ double red[kThreadsG / 64];
    pair_body_glb<kThreadsG, DIMER>(pairs, n_pair, monos, dif, V, M, G, scratch, slot_elems, ed2, couple, cl, po, red);
}

// ---------------------------------------------------------------------------
// pairs from L2, split: Tau tasks, then G tasks, each a 3 x 3 block of tiles
// of one pair (edge blocks tile by tile), taken by the waves of the XCD the
// pair belongs to in pair order
// ---------------------------------------------------------------------------
__device__ inline int sb_count(int tiles) { return (tiles + kSB - 1) / kSB; }

// Operands of the two-launch form.  What bounds it is the matrix pipe (v_mfma_f64_16x16x4, 47 TFLOP/s), once a chunk's
// loads are in flight while the chunk before it is multiplied.  So the loads take no conditions: rows and columns
// past the pair's last read the last (their products are masked at the end), and only the last, partial chunk
// of 16 clamps k, where the other operand (M or Tau) is zero.  120 monomers of
// o5v27 and o8v56: 6.66 to 5.92 ms a sweep (0.21 TFLOP), with G's blocks above the diagonal left out, and
// 5.50 with the pairs dealt to the XCDs by weight.
// N tiles' values for the chunk at k0 into f (four k per lane from k0 + lk).
template <int N>
struct GlbM {   // rows of M (fragment order)
    const double* m;
    int np, r0, lr, lk;
    template <bool TAIL>
    __device__ __forceinline__ void load(int k0, double (&f)[N][4]) const {
#pragma unroll
        for (int i = 0; i < N; ++i) split(load4_frag(m, np, (r0 + i) * 16 + lr, k0 + lk), f[i]);
    }
};

template <int N>
struct GlbRows {   // rows of a row-major matrix, k along the row
    const double* row[N];
    int n, lk;   // length of a row
    __device__ __forceinline__ GlbRows(const double* m, int rows, int cols, int ld, int r0, int lane)
        : n(cols), lk((lane >> 4) * 4) {
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = m + (int64_t)min((r0 + i) * 16 + (lane & 15), rows - 1) * ld;
    }
    template <bool TAIL>
    __device__ __forceinline__ void load(int k0, double (&f)[N][4]) const {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int s = 0; s < 4; ++s) f[i][s] = row[i][TAIL ? min(k0 + lk + s, n - 1) : k0 + lk + s];
    }
};

template <int N>
struct GlbCols {   // columns of a row-major matrix, k down the rows
    const double* m;
    int n, ld, lk;   // rows
    int col[N];
    __device__ __forceinline__ GlbCols(const double* m_, int rows, int cols, int ld_, int c0, int lane)
        : m(m_), n(rows), ld(ld_), lk((lane >> 4) * 4) {
#pragma unroll
        for (int j = 0; j < N; ++j) col[j] = min((c0 + j) * 16 + (lane & 15), cols - 1);
    }
    template <bool TAIL>
    __device__ __forceinline__ void load(int k0, double (&f)[N][4]) const {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double* q = m + (int64_t)(TAIL ? min(k0 + lk + s, n - 1) : k0 + lk + s) * ld;
#pragma unroll
            for (int j = 0; j < N; ++j) f[j][s] = q[col[j]];
        }
    }
};

// acc += A B over k < K
template <int NR, int NC, class LA, class LB>
__device__ __forceinline__ void product_glb(const LA& A, const LB& B, int K, d4 (&acc)[NR][NC]) {
    const int full = K & ~15;
    double a[NR][4], b[NC][4], an[NR][4], bn[NC][4];
    if (full) {
        A.template load<false>(0, an);
        B.template load<false>(0, bn);
    }
    for (int k0 = 0; k0 < full; k0 += 16) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int i = 0; i < NR; ++i) a[i][s] = an[i][s];
#pragma unroll
            for (int j = 0; j < NC; ++j) b[j][s] = bn[j][s];
        }
        const int kn = k0 + 16 < full ? k0 + 16 : k0;   // the load past the last chunk repeats it
        A.template load<false>(kn, an);
        B.template load<false>(kn, bn);
        mma_block(acc, a, b);
    }
    if (full < K) {
        A.template load<true>(full, a);
        B.template load<true>(full, b);
        mma_block(acc, a, b);
    }
}

// Tau = D_XY * (V + M_X V + V M_Y^T) on tiles (r0.., c0..) into the pair's Tau slot; returns the
// lane's part of <V, Tau>
template <int NR, int NC>
__device__ inline double tau_block_glb(const PairView& p, double* tau, int r0, int c0, int lane, int couple) {
    d4 acc[NR][NC];
    zero(acc);
    const int lr = lane & 15, lk = (lane >> 4) * 4;
    product_glb(GlbM<NR>{p.MX, p.npX, r0, lr, lk}, GlbCols<NC>(p.V, p.nX, p.nY, p.nY, c0, lane), p.nX, acc);   // M_X V
    product_glb(GlbRows<NR>(p.V, p.nX, p.nY, p.nY, r0, lane), GlbM<NC>{p.MY, p.npY, c0, lr, lk}, p.nY, acc);   // V M_Y^T
    double dxr[NR][4];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) dxr[i][t] = p.dX[(r0 + i) * 16 + acc_row(lane, t)];
    double epart = 0.0;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int c = (c0 + j) * 16 + acc_col(lane);
        const int cc = min(c, p.nY - 1);
        const double dyc = p.dY[c];
        double vv[NR][4];
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int rr = min((r0 + i) * 16 + acc_row(lane, t), p.nX - 1);
                vv[i][t] = p.V[(int64_t)rr * p.nY + cc];
            }
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int r = (r0 + i) * 16 + acc_row(lane, t);
                const bool ok = r < p.nX && c < p.nY;
                const double tv = ok ? recip(dxr[i][t] + dyc) * (vv[i][t] + acc[i][j][t]) : 0.0;
                epart += ok ? vv[i][t] * tv : 0.0;
                if (couple) tau[(int64_t)r * p.npY + c] = tv;
            }
    }
    return epart;
}

__global__ __launch_bounds__(kThreadsG, 2) void pair_glb_tau_kernel(
    GlbTasks T, const PairDesc* __restrict__ pairs, const MonoDesc* __restrict__ monos,
    const double* __restrict__ dif, const double* __restrict__ V, const double* __restrict__ M,
    double* __restrict__ scratch, double* __restrict__ ed2, int couple, const Ctrl* __restrict__ ctrl,
    const ClState* __restrict__ cl) {
    if (ctrl && ctrl->done) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for_glb_tasks<kThreadsG / 64>(T, wave, [&](int j, int lt) {
        const PairDesc pd = pairs[T.xpair[j]];
        if (cl && cl[pd.cluster].done) return;   // uniform over the wave
        const PairView p = make_view(pd, monos, dif, V, M, nullptr);
        double* tau = scratch + T.tau_off[j];
        const int RB = p.npX / 16, CB = p.npY / 16, SC = (CB + T.sb - 1) / T.sb;
        const int r0 = (lt / SC) * T.sb, c0 = (lt % SC) * T.sb;
        const int nr = min(T.sb, RB - r0), nc = min(T.sb, CB - c0);
        double epart = 0.0;
        if (nr == kSB && nc == kSB) {
            epart = tau_block_glb<kSB, kSB>(p, tau, r0, c0, lane, couple);
        } else {
            for (int i = 0; i < nr; ++i)
                for (int k = 0; k < nc; ++k) epart += tau_block_glb<1, 1>(p, tau, r0 + i, c0 + k, lane, couple);
        }
        epart = wave_sum(epart);
        if (lane == 0) unsafeAtomicAdd(ed2 + pd.orig, 4.0 * epart);
    });
}

// Block (r0, c0) of G_X or G_Y: below the diagonal with the transpose of block (c0, r0) added, since G enters the
// monomer equation as G + G^T only (half the atomic additions, 206 cycles of the store path per 64 values)
template <int NR, int NC>
__device__ inline void g_block_glb(const PairView& p, const double* tau, int which, int r0, int c0, bool both, int lane) {
    d4 acc[NR][NC];
    zero(acc);
    if (which == 0) {
        product_glb(GlbRows<NR>(tau, p.npX, p.npY, p.npY, r0, lane), GlbRows<NC>(p.V, p.nX, p.nY, p.nY, c0, lane), p.nY, acc);
        if (both)
            product_glb(GlbRows<NR>(p.V, p.nX, p.nY, p.nY, r0, lane), GlbRows<NC>(tau, p.npX, p.npY, p.npY, c0, lane), p.nY, acc);
        atomic_flush(p.GX, nullptr, p.npX, p.nX, r0, c0, lane, acc);
    } else {
        product_glb(GlbCols<NR>(tau, p.npX, p.npY, p.npY, r0, lane), GlbCols<NC>(p.V, p.nX, p.nY, p.nY, c0, lane), p.nX, acc);
        if (both)
            product_glb(GlbCols<NR>(p.V, p.nX, p.nY, p.nY, r0, lane), GlbCols<NC>(tau, p.npX, p.npY, p.npY, c0, lane), p.nX, acc);
        atomic_flush(p.GY, nullptr, p.npY, p.nY, r0, c0, lane, acc);
    }
}

__global__ __launch_bounds__(kThreadsG, 2) void pair_glb_g_kernel(
    GlbTasks T, const PairDesc* __restrict__ pairs, const MonoDesc* __restrict__ monos,
    const double* __restrict__ dif, const double* __restrict__ V, const double* __restrict__ M,
    double* __restrict__ G, const double* __restrict__ scratch, const Ctrl* __restrict__ ctrl,
    const ClState* __restrict__ cl) {
    if (ctrl && ctrl->done) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for_glb_tasks<kThreadsG / 64>(T, wave, [&](int j, int lt) {
        const PairDesc pd = pairs[T.xpair[j]];
        if (cl && cl[pd.cluster].done) return;
        const PairView p = make_view(pd, monos, dif, V, M, G);
        const double* tau = scratch + T.tau_off[j];
        const int RB = p.npX / 16, CB = p.npY / 16, SR = (RB + T.sb - 1) / T.sb;
        const int nx = SR * (SR + 1) / 2, which = lt < nx ? 0 : 1;
        int u = which ? lt - nx : lt, i = 0;   // row i of the triangle: blocks (i, 0) .. (i, i)
        while (u > i) u -= ++i;
        const int n = which ? CB : RB, r0 = i * T.sb, c0 = u * T.sb;
        const int nr = min(T.sb, n - r0), nc = min(T.sb, n - c0);
        if (nr == kSB && nc == kSB) {
            g_block_glb<kSB, kSB>(p, tau, which, r0, c0, r0 != c0, lane);
        } else {
            for (int e = 0; e < nr; ++e)
                for (int k = 0; k < nc; ++k) g_block_glb<1, 1>(p, tau, which, r0 + e, c0 + k, r0 != c0, lane);
        }
    });
}

}  // namespace

int glb_tau_tasks(int npX, int npY, int sb) {
    const int sr = (npX / 16 + sb - 1) / sb, sc = (npY / 16 + sb - 1) / sb;
    return sr * sc;
}

int glb_g_tasks(int npX, int npY, int sb) {
    const int sr = (npX / 16 + sb - 1) / sb, sc = (npY / 16 + sb - 1) / sb;
    return sr * (sr + 1) / 2 + sc * (sc + 1) / 2;
}

void launch_pair_fp64_split(const GlbTasks& tau_tasks, const GlbTasks& g_tasks, int n_chunk_pairs,
                            const PairDesc* pairs, const MonoDesc* monos, const double* dif, const double* V,
                            const double* M, double* G, double* scratch, int grid, double* ed2, int couple,
                            const Ctrl* ctrl, const ClState* cl, hipStream_t s) {
    if (n_chunk_pairs <= 0) return;
    launch_zero_ed2(pairs, tau_tasks.xpair, n_chunk_pairs, ed2, ctrl, cl, s);
    hipLaunchKernelGGL(pair_glb_tau_kernel, dim3(grid), dim3(kThreadsG), 0, s, tau_tasks, pairs, monos, dif, V, M,
                       scratch, ed2, couple, ctrl, cl);
    if (couple)
        hipLaunchKernelGGL(pair_glb_g_kernel, dim3(grid), dim3(kThreadsG), 0, s, g_tasks, pairs, monos, dif, V, M,
                           G, scratch, ctrl, cl);
}

int pair_fp64_blocks_per_cu(int lds_variant) {
    int n = 0;
    hipError_t e = lds_variant
                       ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, pair_fp64_lds_kernel<0>, kThreadsL, 0)
                       : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, pair_fp64_glb_kernel<0>, kThreadsG, 0);
    if (e != hipSuccess || n < 1) n = 1;
    return n;
}

int64_t pair_tau_slot(int nX, int nY) {
    const int64_t x8 = (nX + 7) & ~7, y8 = (nY + 7) & ~7, x16 = (nX + 15) & ~15, y16 = (nY + 15) & ~15;
    return pair_fits_lds(nX, nY) ? std::max(2 * x8 * y8, x16 * y16) : x16 * y16;
}

bool pair_fits_lds(int nX, int nY) {
    const int64_t nx8 = (nX + 7) & ~7, ny8 = (nY + 7) & ~7;
    return nx8 * (ny8 + 4) + nx8 + ny8 <= kLdsPair;
}

void launch_pair_fp64(int lds_variant, PartOut po, const PairDesc* pairs, int64_t n_pair, const MonoDesc* monos,
                      const double* dif, const double* V, const double* M, double* G, double* scratch,
                      int64_t slot_elems, int grid, double* ed2, int couple, const Ctrl* ctrl, const ClState* cl,
                      hipStream_t s) {
    if (n_pair <= 0) return;
    const int dimer = po.S == nullptr ? 0 : po.dd ? 2 : 1;
    if (lds_variant) {
        if (dimer == 2)
            hipLaunchKernelGGL(pair_fp64_lds_kernel<2>, dim3(grid), dim3(kThreadsL), 0, s, pairs, n_pair, monos,
                               dif, V, M, G, scratch, slot_elems, ed2, couple, ctrl, cl, po);
        else if (dimer == 1)
            hipLaunchKernelGGL(pair_fp64_lds_kernel<1>, dim3(grid), dim3(kThreadsL), 0, s, pairs, n_pair, monos,
                               dif, V, M, G, scratch, slot_elems, ed2, couple, ctrl, cl, po);
        else
            hipLaunchKernelGGL(pair_fp64_lds_kernel<0>, dim3(grid), dim3(kThreadsL), 0, s, pairs, n_pair, monos,
                               dif, V, M, G, scratch, slot_elems, ed2, couple, ctrl, cl, po);
    } else {
        if (dimer == 2)
            hipLaunchKernelGGL(pair_fp64_glb_kernel<2>, dim3(grid), dim3(kThreadsG), 0, s, pairs, n_pair, monos,
                               dif, V, M, G, scratch, slot_elems, ed2, couple, ctrl, cl, po);
        else if (dimer == 1)
            hipLaunchKernelGGL(pair_fp64_glb_kernel<1>, dim3(grid), dim3(kThreadsG), 0, s, pairs, n_pair, monos,
                               dif, V, M, G, scratch, slot_elems, ed2, couple, ctrl, cl, po);
        else
            hipLaunchKernelGGL(pair_fp64_glb_kernel<0>, dim3(grid), dim3(kThreadsG), 0, s, pairs, n_pair, monos,
                               dif, V, M, G, scratch, slot_elems, ed2, couple, ctrl, cl, po);
    }
}

}  // namespace mcpt
