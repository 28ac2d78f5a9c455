// m2l_sym.hip -- M2L of whole sibling groups through the symmetry of the
// square (dense V lists, FP64, 64 padded coefficients).
//
// The four children of a box and the 32 boxes around them whose children the
// V lists draw on (the children of the parent's neighbours) form, about the
// parent's centre, a figure that the eight symmetries of the square (D4) map
// to itself, and every M2L operator obeys T(g d) = P_g T(d) P_g^-1 with P_g a
// signed permutation of the real coefficients: a rotation by 90 degrees
// multiplies coefficient n by i^-n, the reflection x <-> y by i^-n after
// conjugation.  In coordinates adapted to the group's irreducible
// representations the map from the 32 x 64 source coefficients to the 4 x 64
// local ones falls into blocks: 32 x 256 for each of the four one-dimensional
// representations (A1, A2, B1, B2) and 64 x 512, applied twice, for the
// two-dimensional one (E): 98,304 multiply-adds per parent where 4 x 27 dense
// 64 x 64 products take 442,368, with the same result up to rounding.
//
// Conventions.  r: rotation by 90 degrees, s: (x, y) -> (y, x); g = r^k s^e.
// For a source orbit {g s0} v_g = P_g^-1 M(g s0); u(X) = sum_g X(g) v_g for a
// one-dimensional representation X, u_ac = sum_g E_ac(g) v_g with E(r) =
// (0 -1; 1 0), E(s) = diag(1, -1).  With the target child t0 (the upper
// right), S_h = T(t0 - h s0) P_h (zero for adjacent boxes),
//   w(X) = [sum_h X(h) S_h] u(X),   w_ab = sum_c [sum_h E_bc(h) S_h] u_ac,
// summed over the orbits, and the local expansion of child g t0 is
//   L(g t0) = P_g (1/8) [sum_X X(g) w(X) + 2 sum_ab E_ab(g) w_ab].
// s fixes t0, so w(X) lies in the X(s) eigenspace of P_s, w_a1 in the +1 and
// w_a2 in the -1 one (32 coordinates each: V+ and V-), and the same holds for
// u on the two orbits on the diagonals, which have four boxes.
#include "fmm.h"

namespace yk {

namespace {

typedef double sym_d4 __attribute__((ext_vector_type(4)));
typedef double sym_d2 __attribute__((ext_vector_type(2)));

constexpr int kSymPP = 64;                // padded coefficients
constexpr int kSymChunk = 128;            // doubles of one operator fragment (64 lanes x 2)
constexpr int kSymChunks = 128;           // fragments per wavefront and level
constexpr int kSymRing = 8;               // fragments in flight
constexpr int kSymLevel = 4 * kSymChunks * kSymChunk;   // operator doubles per level
constexpr int kSymCols = 16;              // parents per workgroup

// source orbits about the parent's centre, in half child sides: three of
// eight boxes, two (on the diagonals) of four
__device__ constexpr int kOrbX[5] = {3, 5, 5, 3, 5}, kOrbY[5] = {1, 1, 3, 3, 5};

// (x, y) -> r^k s^e (x, y)
__device__ __forceinline__ void sym_apply(int k, int e, int &x, int &y) {
    if (e) {
        const int t = x;
        x = y;
        y = t;
    }
    for (int i = 0; i < k; ++i) {
        const int t = x;
        x = -y;
        y = t;
    }
}

// P_{r^k s^e} e_j = sign e_(returned index)
__device__ __forceinline__ int sym_perm(int k, int e, int j, double &sign) {
    sign = 1.0;
    if (j == 0 || j >= kSymPP - 1) return j;   // Re M_0, and the padding entry
    const int n = (j + 1) >> 1, c = (j + 1) & 1;   // M_n's real (c = 0) or imaginary part
    const int ex = ((e ? -c : c) - n * (k + e)) & 3;
    sign = ex >= 2 ? -1.0 : 1.0;
    return 2 * n - 1 + (ex & 1);
}

// the coordinate that stands for index n = 0..31 of V+ and of V-
__device__ __forceinline__ int sym_plus(int n) { return n == 0 ? 0 : (n & 3) == 2 ? 2 * n : 2 * n - 1; }
__device__ __forceinline__ int sym_minus(int n) {
    return n == 0 ? kSymPP - 1 : (n & 3) == 0 ? 2 * n : 2 * n - 1;
}

// Operator fragments of one level, in the order k_m2l_sym consumes them: per
// wavefront w eight phases of 16 fragments, for the coefficient indices n =
// 16 hf .. 16 hf + 15 the three orbits of eight and then the two of four
// together; per step two fragments of representation w (its two row tiles) and
// two of row tile w of E.  Lane l holds, for row l % 16, contraction indices
// 2 (l / 16) + {0, 1} of a fragment's eight.
// Built once per tree from the 40 dense operators (column-major).
__global__ void k_sym_ops(int level0, const double *__restrict__ m2l, double *__restrict__ op) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // one double
    const int level = level0 + (int)(t / kSymLevel);
    const int f = (int)(t % kSymLevel);
    const int e2 = f & 1, lane = (f >> 1) & 63, chunk = (f >> 7) % kSymChunks, w = (f >> 7) / kSymChunks;
    const int phase = chunk >> 4, hf = phase >> 2;
    const bool full = (phase & 3) < 3;
    // four fragments per step of 16 contraction indices of E (q = 2 c, 2 c + 1)
    // and eight of w
    const int c = full ? (chunk & 15) >> 2 : (chunk & 7) >> 2, f4 = chunk & 3;
    const int orb = full ? (phase & 3) : 3 + ((chunk & 15) >> 3);
    const bool isE = f4 >= 2;
    int row, k;   // output coordinate (0..31 of the representation, 0..63 of E), contraction index of the orbit
    if (!isE) {
        row = 16 * f4 + (lane & 15);
        k = 8 * c + 2 * (lane >> 4) + e2;          // within the half: 2 n + part, or n
        k += hf * (full ? 32 : 16);
    } else {
        row = 16 * w + (lane & 15);
        k = 8 * (2 * c + f4 - 2) + 2 * (lane >> 4) + e2;
        if (full) k = (k >> 5) * 64 + hf * 32 + (k & 31);   // u_a1, then u_a2
        else k += hf * 32;
    }
    // i: row of the dense operators; j: column; cc: second index of E
    int i, j, cc = 0, b = 0;
    if (!isE) {
        const bool plus = (w & 1) == 0;   // A1, B1
        i = plus ? sym_plus(row) : sym_minus(row);
        j = full ? (k < 2 ? (k == 0 ? 0 : kSymPP - 1) : k - 1) : plus ? sym_plus(k) : sym_minus(k);
    } else {
        b = row >> 5;
        i = b == 0 ? sym_plus(row & 31) : sym_minus(row & 31);
        if (full) {
            cc = k >> 6;
            const int kk = k & 63;
            j = kk < 2 ? (kk == 0 ? 0 : kSymPP - 1) : kk - 1;
        } else {
            cc = k & 1;
            j = cc == 0 ? sym_plus(k >> 1) : sym_minus(k >> 1);
        }
    }
    double v = 0.0;
    if (i < kSymPP - 1 && j < kSymPP - 1) {
        const double *Tl = m2l + (int64_t)level * kNumOff * kSymPP * kSymPP;
        for (int e = 0; e < 2; ++e)
            for (int r = 0; r < 4; ++r) {
                int x = kOrbX[orb], y = kOrbY[orb];
                sym_apply(r, e, x, y);
                const int dx = (x - 1) / 2, dy = (y - 1) / 2;   // source minus target child, in boxes (even differences)
                if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1) continue;
                double wt;
                if (!isE) {
                    wt = ((w >= 2 && (r & 1)) ? -1.0 : 1.0) * (((w & 1) && e) ? -1.0 : 1.0);
                } else {
                    // E(r^k s^e): cos, -sin; sin, cos, the second column negated by s
                    const int cs = r == 0 ? 1 : r == 2 ? -1 : 0, sn = r == 1 ? 1 : r == 3 ? -1 : 0;
                    wt = b == 0 ? (cc == 0 ? cs : -sn) : (cc == 0 ? sn : cs);
                    if (cc == 1 && e) wt = -wt;
                }
                if (wt == 0.0) continue;
                // offset id: (dy, dx) over [-3, 3]^2 without the 3 x 3 block
                int oid = (dy + 3) * 7 + dx + 3;
                oid -= (dy > 1 || (dy >= -1 && dy <= 1 && dx > 1) ? 3 : 0) +
                       (dy > 1 ? 6 : dy >= -1 ? 3 * (dy + 1) : 0);
                double sg;
                const int jj = sym_perm(r, e, j, sg);
                v += wt * sg * Tl[(int64_t)oid * kSymPP * kSymPP + (int64_t)jj * kSymPP + i];
            }
        // (1/8, and 2/8 for E, of the inverse transform; the diagonal orbits'
        // sum over h counts every box twice, which the two equal coordinates
        // of an eigenvector's u make up for)
        v *= isE ? 0.25 : 0.125;
    }
    op[t] = v;
}

// One workgroup: 16 parents (the columns), four wavefronts.  Eight phases, each
// eight boxes around every parent and 16 coefficient indices: a thread
// transforms the index n of one parent (u above, exact sums and differences)
// and stores the results to LDS as matrix-core B operands; wavefront w then
// multiplies representation w (two row tiles) and row tile w of E (both
// columns a), its operator fragments streaming from L2 through a ring of
// registers.  The next phase's sources are loaded meanwhile.  Bound by the
// FP64 matrix cores: 384 steps of 2,048 flops per wavefront, 24.6 k cycles per
// tile.  On 2^20 uniform points (21,844 parents, 1,365 tiles) the launch takes
// 116 us (413 us for the dense products by box it stands for), the matrix
// cores busy 49% of it; without its loads and transforms it would take 87 us,
// the last of 2.7 rounds of two workgroups per compute unit being partly
// filled.  Three workgroups (168 registers) and a second LDS buffer (one
// barrier per phase) measured the same.  On one tile it takes 22 us, so small
// trees gain too: 4,096 points 17 + 5 us before, 85 tiles 51 + 5 -> 25 us.
struct SymLane {
    double s, sgn, sx, sy, tx, ty;
    bool odd;
};

__device__ __forceinline__ int sym_slot(int kappa, int col) { return (kappa * 16 + ((col + kappa) & 15)) * 2; }

__device__ __forceinline__ void sym_put(double *Bs, int kappa, int col, double a, double b) {
    *reinterpret_cast<sym_d2 *>(Bs + sym_slot(kappa, col)) = sym_d2{a, b};
}

struct Cx {
    double re, im;
};

// A = sum_k X(r^k) z^k m_k for X(r) = 1, B for -1; C = sum_k cos z^k m_k,
// S = sum_k sin z^k m_k (angles k pi/2), z = i^n
__device__ __forceinline__ void sym_dft(const SymLane &q, const Cx *m, Cx &A, Cx &B, Cx &C, Cx &S) {
    const Cx p{__builtin_fma(q.s, m[2].re, m[0].re), __builtin_fma(q.s, m[2].im, m[0].im)};
    C = Cx{__builtin_fma(-q.s, m[2].re, m[0].re), __builtin_fma(-q.s, m[2].im, m[0].im)};
    const Cx f{__builtin_fma(q.s, m[3].re, m[1].re), __builtin_fma(q.s, m[3].im, m[1].im)};
    const Cx h{__builtin_fma(-q.s, m[3].re, m[1].re), __builtin_fma(-q.s, m[3].im, m[1].im)};
    const double fx = q.odd ? f.im : f.re, fy = q.odd ? f.re : f.im;
    const double hx = q.odd ? h.im : h.re, hy = q.odd ? h.re : h.im;
    A = Cx{__builtin_fma(q.sx, fx, p.re), __builtin_fma(q.sy, fy, p.im)};
    B = Cx{__builtin_fma(-q.sx, fx, p.re), __builtin_fma(-q.sy, fy, p.im)};
    S = Cx{q.sx * hx, q.sy * hy};
}

// X + P_s Y and X - P_s Y
__device__ __forceinline__ void sym_reflect(const SymLane &q, const Cx &X, const Cx &Y, Cx &plus, Cx &minus) {
    const double u = q.odd ? Y.im : Y.re, v = q.odd ? Y.re : Y.im;
    plus = Cx{__builtin_fma(q.tx, u, X.re), __builtin_fma(q.ty, v, X.im)};
    minus = Cx{__builtin_fma(-q.tx, u, X.re), __builtin_fma(-q.ty, v, X.im)};
}

// The loads are unconditional (row 0 stands in for an absent box) and the
// zeros of absent boxes selected when the values are taken, so that an orbit's
// loads all stay in flight during the multiplication before; a bit of valid
// per box.
__device__ __forceinline__ void sym_load(const int32_t *__restrict__ sp, int n, const double *__restrict__ X, Cx *m,
                                         unsigned &valid) {
    valid = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int32_t b = sp[k];
        const double *row = X + (int64_t)(b >= 0 ? b : 0) * kSymPP;
        m[k].re = row[n == 0 ? 0 : 2 * n - 1];
        m[k].im = row[2 * n];
        valid |= b >= 0 ? 1u << k : 0u;
    }
}

// the values of a phase into LDS: n1 = n % 16, col the parent
template <bool FULL>
__device__ __forceinline__ void sym_store(const SymLane &q, const Cx *raw, unsigned valid, int col, int n, int n1,
                                          double *Bs) {
    Cx m[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        m[k].re = (valid >> k) & 1 ? raw[k].re : 0.0;
        m[k].im = ((valid >> k) & 1) && n > 0 ? raw[k].im : 0.0;
    }
    if constexpr (FULL) {
        Cx A, B, C, S, A2, B2, C2, S2, x, y;
        sym_dft(q, m, A, B, C, S);
        sym_dft(q, m + 4, A2, B2, C2, S2);
        sym_reflect(q, A, A2, x, y);
        sym_put(Bs, n1, col, x.re, x.im);             // A1
        sym_put(Bs + 512, n1, col, y.re, y.im);       // A2
        sym_reflect(q, B, B2, x, y);
        sym_put(Bs + 1024, n1, col, x.re, x.im);      // B1
        sym_put(Bs + 1536, n1, col, y.re, y.im);      // B2
        sym_reflect(q, C, C2, x, y);
        sym_put(Bs + 2048, n1, col, x.re, x.im);            // u_11
        sym_put(Bs + 3072, n1 + 16, col, y.re, y.im);       // u_22
        sym_reflect(q, S, S2, x, y);
        sym_put(Bs + 3072, n1, col, x.re, x.im);            // u_21
        sym_put(Bs + 2048, n1 + 16, col, -y.re, -y.im);     // u_12
    } else {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            Cx A, B, C, S;
            sym_dft(q, m + 4 * o, A, B, C, S);
            // the V+ and V- coordinates
            auto split = [&](const Cx &z, double &p, double &v) {
                const double a = q.odd || q.sgn > 0 ? z.re : z.im, b = q.odd || q.sgn > 0 ? z.im : z.re;
                p = q.odd ? __builtin_fma(-q.sgn, b, a) : a;
                v = q.odd ? __builtin_fma(q.sgn, b, a) : b;
            };
            double ap, am, bp, bm, cp, cm, sp, sm;
            split(A, ap, am);
            split(B, bp, bm);
            split(C, cp, cm);
            split(S, sp, sm);
            double *D = Bs + 2048 * o;
            const int at = sym_slot(n1 >> 1, col) + (n1 & 1);
            D[at] = ap;
            D[256 + at] = am;
            D[512 + at] = bp;
            D[768 + at] = bm;
            sym_put(D + 1024, n1, col, cp, -sm);
            sym_put(D + 1536, n1, col, sp, cm);
        }
    }
}

// NQ steps, each eight contraction indices of representation w (at B1) and 16
// of E (at E0 and E1): twelve matrix-core steps on six independent sums (one
// sum's steps follow each other at six steps' distance)
template <int NQ>
__device__ __forceinline__ void sym_multiply(const double *B1, const double *E0, const double *E1, int lane,
                                             const sym_d2 *&Ap, sym_d2 *ring, sym_d4 *acc1, sym_d4 *accE) {
    const int g = lane >> 4, col = lane & 15;
    static_assert(4 * NQ % kSymRing == 0, "the ring starts every call at 0");
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const sym_d2 b = *reinterpret_cast<const sym_d2 *>(B1 + sym_slot(4 * q + g, col));
        sym_d2 e[2][2], a[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            e[h][0] = *reinterpret_cast<const sym_d2 *>(E0 + sym_slot(4 * (2 * q + h) + g, col));
            e[h][1] = *reinterpret_cast<const sym_d2 *>(E1 + sym_slot(4 * (2 * q + h) + g, col));
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int r = (4 * q + f) % kSymRing;
            a[f] = ring[r];
            ring[r] = Ap[(4 * q + f + kSymRing) * 64];
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            acc1[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][x], b[x], acc1[0], 0, 0, 0);
            acc1[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][x], b[x], acc1[1], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                accE[2 * h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2 + h][x], e[h][0][x], accE[2 * h], 0, 0, 0);
                accE[2 * h + 1] =
                    __builtin_amdgcn_mfma_f64_16x16x4f64(a[2 + h][x], e[h][1][x], accE[2 * h + 1], 0, 0, 0);
            }
        }
    }
    Ap += 4 * NQ * 64;
}

// One box of a level coarser than the sibling groups serve: its 27 dense
// products by one workgroup.  Wavefront w takes slots w, w + 4, ..; lane l rows
// 2 (l % 32) + {0, 1} and the columns of parity l / 32, so that one load
// covers two columns; half a slot's loads are issued together.
__device__ __forceinline__ void sym_coarse_box(int box, const int32_t *__restrict__ vl, const int32_t *__restrict__ oid,
                                               const double *__restrict__ Op, const double *__restrict__ X, double *sh,
                                               double *__restrict__ out) {
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    for (int f = tid; f < kNumV * kSymPP; f += 256) {
        const int32_t b = vl[f / kSymPP];
        const double v = X[(int64_t)(b >= 0 ? b : 0) * kSymPP + f % kSymPP];
        sh[f] = b >= 0 ? v : 0.0;
    }
    __syncthreads();
    sym_d2 acc{0.0, 0.0};
    for (int sl = w; sl < kNumV; sl += 4) {
        if (vl[sl] < 0) continue;
        const sym_d2 *A = reinterpret_cast<const sym_d2 *>(Op + (int64_t)oid[sl] * kSymPP * kSymPP) + lane;
        const double *x = sh + sl * kSymPP + (lane >> 5);
        for (int k0 = 0; k0 < kSymPP / 2; k0 += 16) {
            sym_d2 a[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) a[k] = A[(k0 + k) * 64];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double v = x[2 * (k0 + k)];
                acc.x = __builtin_fma(a[k].x, v, acc.x);
                acc.y = __builtin_fma(a[k].y, v, acc.y);
            }
        }
    }
    acc.x += __shfl_xor(acc.x, 32, 64);
    acc.y += __shfl_xor(acc.y, 32, 64);
    double *red = sh + kNumV * kSymPP;
    if (lane < 32) *reinterpret_cast<sym_d2 *>(red + w * kSymPP + 2 * lane) = acc;
    __syncthreads();
    if (tid < kSymPP)
        out[(int64_t)box * kSymPP + tid] =
            (red[tid] + red[kSymPP + tid]) + (red[2 * kSymPP + tid] + red[3 * kSymPP + tid]);
}

__global__ __launch_bounds__(256, 2) void k_m2l_sym(const int4 *__restrict__ tiles, int ntiles,
                                                    const int32_t *__restrict__ src,
                                                    const int32_t *__restrict__ tgt, const double *__restrict__ Op,
                                                    int level0, const int2 *__restrict__ coarse,
                                                    const int32_t *__restrict__ vlist,
                                                    const uint32_t *__restrict__ bcode,
                                                    const int32_t *__restrict__ slot_oid,
                                                    const double *__restrict__ dense, const double *__restrict__ X,
                                                    double *__restrict__ out) {
    __shared__ double Bs[4096];
    __shared__ int32_t s_src[kSymCols * 32];
    if ((int)blockIdx.x >= ntiles) {   // (whole workgroups)
        const int2 bl = coarse[blockIdx.x - ntiles];   // {box, level}
        sym_coarse_box(bl.x, vlist + (int64_t)bl.x * kNumV, slot_oid + (bcode[bl.x] & 3u) * kNumV,
                       dense + (int64_t)bl.y * kNumOff * kSymPP * kSymPP, X, Bs, out);
        return;
    }
    // consecutive tiles on one XCD (as in the other M2L kernels)
    const int nb = ntiles, xb = blockIdx.x % 8, ib = blockIdx.x / 8;
    const int bid = xb * (nb / 8) + min(xb, nb % 8) + ib;
    const int4 tl = tiles[bid];   // {level, first parent, parents}
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int n1 = tid & 15, col = tid >> 4;   // coefficient index modulo 16, parent
    for (int t = tid; t < kSymCols * 32; t += 256)
        s_src[t] = (t >> 5) < tl.z ? src[(int64_t)tl.y * 32 + t] : -1;
    const sym_d2 *Ap = reinterpret_cast<const sym_d2 *>(Op + (int64_t)(tl.x - level0) * kSymLevel +
                                                        (int64_t)w * kSymChunks * kSymChunk) + lane;
    SymLane q;
    q.odd = n1 & 1;   // (the same for n1 and n1 + 16)
    q.s = q.odd ? -1.0 : 1.0;
    q.sgn = (n1 & 2) ? -1.0 : 1.0;
    q.sx = q.odd ? -q.sgn : q.sgn;
    q.sy = q.sgn;
    q.tx = q.odd ? -q.sgn : q.sgn;
    q.ty = -q.sgn;
    sym_d4 acc1[2] = {sym_d4{0, 0, 0, 0}, sym_d4{0, 0, 0, 0}}, accE[4] = {acc1[0], acc1[0], acc1[0], acc1[0]};
    sym_d2 ring[kSymRing];
#pragma unroll
    for (int i = 0; i < kSymRing; ++i) ring[i] = Ap[i * 64];
    __syncthreads();
    Cx m[8];
    unsigned valid;
    const int32_t *sp = s_src + col * 32;
    sym_load(sp, n1, X, m, valid);
#pragma unroll 1
    for (int hf = 0; hf < 2; ++hf) {
        const int n = n1 + 16 * hf;
#pragma unroll
        for (int ph = 0; ph < 4; ++ph) {
            if (ph < 3) sym_store<true>(q, m, valid, col, n, n1, Bs);
            else sym_store<false>(q, m, valid, col, n, n1, Bs);
            __syncthreads();
            if (ph < 3) sym_load(sp + 8 * (ph + 1), n, X, m, valid);
            else if (hf == 0) sym_load(sp, n + 16, X, m, valid);
            if (ph < 3) {
                sym_multiply<4>(Bs + 512 * w, Bs + 2048, Bs + 3072, lane, Ap, ring, acc1, accE);
            } else {
                sym_multiply<2>(Bs + 256 * w, Bs + 1024, Bs + 1536, lane, Ap, ring, acc1, accE);
                sym_multiply<2>(Bs + 2048 + 256 * w, Bs + 3072, Bs + 3584, lane, Ap, ring, acc1, accE);
            }
            __syncthreads();
        }
    }
    // outputs [256 rows][16 parents]: 32 of each representation, then 64 of E
    // for each a
    auto at = [](int row, int col) { return row * 16 + ((col + row) & 15); };
    {
        const int g = lane >> 4, cc = lane & 15;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            Bs[at(32 * w + g + 4 * r, cc)] = acc1[0][r];
            Bs[at(32 * w + 16 + g + 4 * r, cc)] = acc1[1][r];
            Bs[at(128 + 16 * w + g + 4 * r, cc)] = accE[0][r] + accE[2][r];
            Bs[at(192 + 16 * w + g + 4 * r, cc)] = accE[1][r] + accE[3][r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int n = n1 + 16 * h;
        if (col >= tl.z) continue;
        const double a1 = Bs[at(n, col)], a2 = Bs[at(32 + n, col)], b1 = Bs[at(64 + n, col)], b2 = Bs[at(96 + n, col)];
        const double e0p = Bs[at(128 + n, col)], e0m = Bs[at(160 + n, col)];
        const double e1p = Bs[at(192 + n, col)], e1m = Bs[at(224 + n, col)];
        const int32_t *tg = tgt + (int64_t)(tl.y + col) * 4;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double vp = k == 0 ? a1 + b1 + e0p : k == 1 ? a1 - b1 + e1p : k == 2 ? a1 + b1 - e0p : a1 - b1 - e1p;
            const double vm = k == 0 ? a2 + b2 + e1m : k == 1 ? a2 - b2 - e0m : k == 2 ? a2 + b2 - e1m : a2 - b2 + e0m;
            double re, im;
            if (q.odd) {
                re = vp + vm;
                im = q.sgn > 0 ? vm - vp : vp - vm;
            } else {
                re = q.sgn > 0 ? vp : vm;
                im = q.sgn > 0 ? vm : vp;
            }
            // P_{r^k}: times i^(-n k)
            const int ex = (-n * k) & 3;
            const double x = ex == 0 ? re : ex == 1 ? -im : ex == 2 ? -re : im;
            const double y = ex == 0 ? im : ex == 1 ? re : ex == 2 ? -im : -re;
            const int32_t b = tg[k];
            if (b >= 0) {
                double *o = out + (int64_t)b * kSymPP;
                o[n == 0 ? 0 : 2 * n - 1] = x;
                o[n == 0 ? kSymPP - 1 : 2 * n] = n == 0 ? 0.0 : y;   // (n = 0: the padding entry)
            }
        }
    }
}

}  // namespace

// A target box receives its V list's contributions mixed with those of its
// siblings' sources, which cancel only up to rounding: a box at the shortest
// offset (two sides) leaves about 1e-16 of its contribution in targets whose
// own share of it (at up to 3 sqrt(2) sides) is smaller by
// exp(2.24 side / alpha).  At boxes of at most four alpha that is about 1e-12
// of the share itself; coarser levels keep the separate products.  Measured, one
// box's charges alone, its targets two and three boxes away against the same
// truncated sums, each relative to its own (worst, median): at sides of one
// alpha 4.6e-15, 1.7e-15 (by box 5.1e-15, 1.3e-15), of two 1.9e-14, 2.9e-15
// (6.0e-15, 3.1e-15), of 3.99 1.1e-12, 7.1e-15 (2.7e-14, 6.2e-15).  Order 31
// leaves up to 1.6e-10 of such a target's sum there: against exact sums the
// largest errors by either route are the same.
constexpr double kSymMaxSide = 4.0;

int sym_first_level(const FmmPlan &pl) {
    int l = std::max(pl.lmin, 2);
    while (l <= pl.L && pl.lev[l].side > kSymMaxSide * pl.alpha) ++l;
    return l;
}

void build_sym_ops(Context &ctx, FmmPlan &pl) {
    if (pl.Pp != kSymPP) {
        pl.symop.release();
        return;
    }
    const int l0 = sym_first_level(pl), nl = pl.L + 1 - l0;
    if (nl <= 0) return;
    // (a ring's worth of fragments beyond the end is read, never used)
    const size_t total = (size_t)nl * kSymLevel, pad = (size_t)kSymRing * kSymChunk;
    double *op = pl.symop.ensure(total + pad);
    hipLaunchKernelGGL(k_sym_ops, dim3((unsigned)(total / 256)), dim3(256), 0, ctx.stream, l0, pl.m2l.p, op);
    check_launch(ctx, "k_sym_ops");
    launch_fill(ctx, (int64_t)pad, 0.0, op + total);
}

void launch_m2l_sym(Context &ctx, FmmPlan &pl, ActiveSet &as) {
    hipLaunchKernelGGL(k_m2l_sym, dim3((unsigned)(as.n_sym_tiles + as.n_sym_coarse)), dim3(256), 0, ctx.stream,
                       as.sym_tiles.p, as.n_sym_tiles, as.sym_src.p, as.sym_tgt.p, pl.symop.p, as.sym_level,
                       as.sym_coarse.p, pl.vlist.p, pl.bcode.p, pl.slot_oid.p, pl.m2l.p, pl.M.p, pl.Lc.p);
    check_launch(ctx, "k_m2l_sym");
}

}  // namespace yk
