// fmm_kernels.hip -- upward pass, M2L, downward pass and near field of the
// modified-Helmholtz FMM (expansion conventions in fmm.h), FP64.
#include <climits>
#include <type_traits>

#include "fmm.h"
#include "yk_bessel.h"

namespace yk {

namespace {

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// Consecutive workgroups are dealt round-robin to the 8 XCDs, each with its
// own L2.  Remapping block b so that every XCD walks one contiguous range of
// the (Morton-ordered) work list keeps neighbouring boxes' data in one L2.
// The map is a bijection on [0, n).
__device__ __forceinline__ int xcd_remap(int b, int n) {
    constexpr int kXcd = 8;
    const int x = b % kXcd, i = b / kXcd;
    const int q = n / kXcd, r = n % kXcd;
    return x * q + min(x, r) + i;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---------------------------------------------------------------- gathers --
__global__ void k_gather_q(int64_t n, const int32_t *__restrict__ perm, const double *__restrict__ q,
                           double *__restrict__ qs) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) qs[k] = q[perm[k]];
}

__global__ void k_gather_dn(int64_t off, int64_t n, const int32_t *__restrict__ perm,
                            const double *__restrict__ dn, double *__restrict__ dns) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int32_t i = perm[off + k];
    dns[2 * k] = dn[2 * i];
    dns[2 * k + 1] = dn[2 * i + 1];
}

// the same with the dipole vectors formed on the way: dn_i = w_i sigma_i n_i
__global__ void k_gather_dn_form(int64_t off, int64_t n, const int32_t *__restrict__ perm,
                                 const double *__restrict__ w, const double *__restrict__ sigma,
                                 const double *__restrict__ normal, double *__restrict__ dns) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int32_t i = perm[off + k];
    const double s = 1.0 * (w ? w[i] : 1.0) * sigma[i];
    dns[2 * k] = s * normal[2 * i];
    dns[2 * k + 1] = s * normal[2 * i + 1];
}

__global__ void k_scatter_out(int64_t off, int64_t n, const int32_t *__restrict__ perm,
                              const double *__restrict__ outs, double *__restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[perm[off + k]] = outs[off + k];
}

// ------------------------------------------------------------ F_n helpers --
// F_n(y) = sum_k y^k/(k!(n+1)_k): the two starting values F_{p+1}, F_{p+2} by
// their series; below that, F_n = F_{n+1} + y F_{n+2} / ((n+1)(n+2)) (the
// three-term recurrence of I_n, stable downwards).
__device__ __forceinline__ void f_start(double y, const double *__restrict__ sc, int nser,
                                        double &Fn1, double &Fn2) {
    double a = sc[nser - 1], b = sc[2 * nser - 1];
    for (int k = nser - 2; k >= 0; --k) {
        a = a * y + sc[k];
        b = b * y + sc[nser + k];
    }
    Fn1 = a;   // F_{p+1}
    Fn2 = b;   // F_{p+2}
}

// ------------------------------------------------------------------- P2M ---
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// P2M of the adaptive tree with four lanes (a DPP quad) per leaf for a
// compile-time order PO: each lane takes every fourth point of its leaf and
// accumulates all 2p+1 outputs in registers; the lanes' partial sums are combined
// at the end.  tiles: {level, first entry of leaf_list, entries} per workgroup,
// each with its level's tables.  Per point: F_n downwards
// (G_n = F_n(y)/F_n(Y) in registers), then the terms with the powers of
// conj(z) upwards.
template <int PO>
__global__ __launch_bounds__(64) void k_p2m_quad(
    const int32_t *__restrict__ lrange, const double *__restrict__ bcx, const double *__restrict__ bcy,
    const double *__restrict__ px, const double *__restrict__ py, const double *__restrict__ qs,
    const double *__restrict__ dns, int64_t off1, int has_q, int has_d, double inv_alpha,
    const double *__restrict__ invFY, const double *__restrict__ da, const double *__restrict__ db,
    const double *__restrict__ cnn, const double *__restrict__ sc, int Pp, double *__restrict__ M,
    const int32_t *__restrict__ leaf_list, const int4 *__restrict__ tiles, const int32_t *__restrict__ nser_lv,
    const double *__restrict__ invR_lv, int sc_stride) {
    constexpr int p = PO, P = 2 * PO + 1;
    extern __shared__ double smem[];
    const int4 t = tiles[blockIdx.x];
    const int nser = nser_lv[t.x];
    const double invR = invR_lv[t.x];
    sc += (int64_t)t.x * sc_stride;
    invFY += (int64_t)t.x * (p + 2);
    da += (int64_t)t.x * (p + 2);
    db += (int64_t)t.x * (p + 2);
    double *t_sc = smem;                   // [2 nser] F_{p+1}, F_{p+2} series
    double *t_cnn = t_sc + 2 * nser;       // [p+2]
    double *t_ify = t_cnn + (p + 2);       // [p+2]
    double *t_da = t_ify + (p + 2);        // [p+1]
    double *t_db = t_da + (p + 1);         // [p+1]
    const int lane = threadIdx.x, q4 = lane & 3;
    const bool leaf_ok = (lane >> 2) < t.z;
    const int64_t b = leaf_ok ? leaf_list[t.y + (lane >> 2)] : 0;
    for (int k = lane; k < 2 * nser; k += 64) t_sc[k] = sc[k];
    for (int k = lane; k < p + 2; k += 64) {
        t_cnn[k] = cnn[k];
        t_ify[k] = invFY[k];
    }
    if (has_d)
        for (int k = lane; k < p + 1; k += 64) {
            t_da[k] = da[k];
            t_db[k] = db[k];
        }
    double acc[P];
#pragma unroll
    for (int o = 0; o < P; ++o) acc[o] = 0.0;
    double G[p + 2];
    __syncthreads();
    const double cx = bcx[b], cy = bcy[b];
    for (int set = 0; set < 2; ++set) {
        if ((set == 0 && !has_q) || (set == 1 && !has_d)) continue;
        const int s0 = leaf_ok ? lrange[b * 6 + 2 * set] : 0;
        const int e0 = leaf_ok ? lrange[b * 6 + 2 * set + 1] : 0;
        // a lane without a point reads a point of its own set (weight 0
        // below): the leaf's first, else the set's first (index 0 or off1)
        auto clamp_j = [&](int j) { return j < e0 ? j : (e0 > s0 ? s0 : (set == 0 ? 0 : (int)off1)); };
        // the next point's coordinates are loaded one iteration ahead
        int jn = clamp_j(s0 + q4);
        double nx = px[jn], ny = py[jn];
        for (int j0 = s0;; j0 += 4) {
            const int j = j0 + q4;
            const bool valid = j < e0;
            if (!__any(valid)) break;
            const int jc = jn;
            const double cxp = nx, cyp = ny;
            jn = clamp_j(j + 4);
            nx = px[jn];
            ny = py[jn];
            const double wx = (cxp - cx) * inv_alpha, wy = (cyp - cy) * inv_alpha;
            const double y = 0.25 * (wx * wx + wy * wy);
            const double zx = wx * invR, zy = -wy * invR;   // conj(w)/R
            double F1, F2;
            f_start(y, t_sc, nser, F1, F2);
            // G_n for n = 0..p+1 (n = p+1 only for the dipole window)
            G[p + 1] = F1 * t_ify[p + 1];
#pragma unroll
            for (int n = p; n >= 0; --n) {
                const double F0 = F1 + y * F2 * t_cnn[n];
                G[n] = F0 * t_ify[n];
                F2 = F1;
                F1 = F0;
            }
            if (set == 0) {
                const double qv = valid ? qs[jc] : 0.0;
                double pr = 1.0, pi = 0.0;     // conj(z)^n
#pragma unroll
                for (int n = 0; n <= p; ++n) {
                    const double g = qv * G[n];
                    if (n == 0) {
                        acc[0] += g;
                    } else {
                        acc[2 * n - 1] = __builtin_fma(g, pr, acc[2 * n - 1]);
                        acc[2 * n] = __builtin_fma(g, pi, acc[2 * n]);
                    }
                    const double nr = pr * zx - pi * zy;
                    pi = pr * zy + pi * zx;
                    pr = nr;
                }
            } else {
                const double h = valid ? 0.5 * inv_alpha : 0.0;
                const double Dx = h * dns[2 * (jc - off1)], Dy = h * dns[2 * (jc - off1) + 1];
                // window Psi_{n-1}, Psi_n, Psi_{n+1};  Psi_k = G_k conj(z)^k
                double pr = zx, pi = zy;                       // conj(z)^1
                double c_r = G[0], c_i = 0.0;                  // Psi_0
                double n_r = G[1] * pr, n_i = G[1] * pi;       // Psi_1
                double m_r = n_r, m_i = -n_i;                  // Psi_{-1} = conj(Psi_1)
#pragma unroll
                for (int n = 0; n <= p; ++n) {
                    // term_n = h [a_n D Psi_{n+1} + b_n conj(D) Psi_{n-1}]  (h folded into D)
                    const double an = t_da[n], bn = t_db[n];
                    const double t1r = Dx * n_r - Dy * n_i, t1i = Dx * n_i + Dy * n_r;
                    const double t2r = Dx * m_r + Dy * m_i, t2i = Dx * m_i - Dy * m_r;
                    if (n == 0) {
                        acc[0] += an * t1r + bn * t2r;
                    } else {
                        acc[2 * n - 1] += an * t1r + bn * t2r;
                        acc[2 * n] += an * t1i + bn * t2i;
                    }
                    m_r = c_r; m_i = c_i;
                    c_r = n_r; c_i = n_i;
                    const double nr = pr * zx - pi * zy;
                    pi = pr * zy + pi * zx;
                    pr = nr;
                    if (n + 2 <= p + 1) {
                        n_r = G[n + 2] * pr; n_i = G[n + 2] * pi;
                    } else {
                        n_r = 0.0; n_i = 0.0;
                    }
                }
            }
        }
    }
    // sums over the leaf's lanes; lane q4 writes outputs q4, q4 + 4, ...
#pragma unroll
    for (int o = 0; o < P; ++o) {
        double v = acc[o];
        v += dpp_d<0xB1>(v);    // quad_perm [1,0,3,2]
        v += dpp_d<0x4E>(v);    // quad_perm [2,3,0,1]
        if (leaf_ok && o % 4 == q4) M[b * Pp + o] = v;
    }
    if (leaf_ok)
        for (int o = P + q4; o < Pp; o += 4) M[b * Pp + o] = 0.0;
}

// Charges-only P2M in two halves of the orders: blockIdx.y = 0 takes orders
// 0..NS-1, blockIdx.y = 1 orders NS..p (NS = (p+1)/2), so each wavefront holds
// half the accumulators and half the G_n and more wavefronts fit a SIMD.  As
// in k_p2m_quad, four lanes per leaf over its points and DPP quad sums.  The
// upper half starts its powers at conj(z)^NS by repeated squaring and stops
// its downward F recurrence at NS.  Writes every entry of the leaves'
// multipoles (padding included); dipoles are added afterwards.  The blocks
// also clear zero[0..nzero) on the side (the local expansions, so that no
// launch of its own is needed).
constexpr int kP2MStage = 384;   // charges staged in LDS per block and round

template <int PO, int H>
__device__ __forceinline__ void p2m_half_body(
    int64_t leaf_base, int64_t nleaf, const int32_t *__restrict__ lrange,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ qs, int has_q, double inv_alpha,
    double invR, const double *t_ify, const double *t_cnn, const double *t_sc, int nser, int Pp,
    double *__restrict__ M, double *sx, double *sy, double *sq, int skip_d) {
    constexpr int p = PO, NS = (PO + 1) / 2;
    constexpr int N0 = H == 0 ? 0 : NS, N1 = H == 0 ? NS - 1 : p;   // orders of this half
    constexpr int O0 = H == 0 ? 0 : 2 * NS - 1;                      // its first output
    constexpr int NA = H == 0 ? 2 * NS - 1 : 2 * (p - NS + 1);       // its outputs
    constexpr int NG = N1 - N0 + 1;
    const int lane = threadIdx.x, q4 = lane & 3;
    const int64_t l0 = (int64_t)blockIdx.x * 16;
    const int64_t li = l0 + (lane >> 2);
    // (with skip_d, leaves that hold dipoles are left to the dipole pass)
    const bool leaf_ok = li < nleaf && !(skip_d && lrange[li * 6 + 3] > lrange[li * 6 + 2]);
    const int64_t b = leaf_base + (leaf_ok ? li : 0);
    double acc[NA];
#pragma unroll
    for (int o = 0; o < NA; ++o) acc[o] = 0.0;
    double G[NG];
    const double cx = bcx[b], cy = bcy[b];
    const int s0 = leaf_ok ? lrange[li * 6] : 0;
    const int e0 = (leaf_ok && has_q) ? lrange[li * 6 + 1] : s0;
    // the charges of the block's leaves (consecutive in Morton order, so one
    // run, up to the charges of leaves left to the dipole pass) are staged in
    // LDS in rounds of kP2MStage: one memory round trip per round, not per
    // point.  The run's ends come from the leaves that hold charges (an empty
    // range carries no position).
    int pbeg = e0 > s0 ? s0 : INT_MAX, pend = e0 > s0 ? e0 : 0;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        pbeg = min(pbeg, __shfl_xor(pbeg, m, 64));
        pend = max(pend, __shfl_xor(pend, m, 64));
    }
    for (int cs = pbeg; cs < pend; cs += kP2MStage) {
        const int cn = min(kP2MStage, pend - cs);
        __syncthreads();
        for (int k = lane; k < cn; k += 64) {
            sx[k] = px[cs + k];
            sy[k] = py[cs + k];
            sq[k] = qs[cs + k];
        }
        __syncthreads();
        // this lane's points j = s0 + q4 + 4k that fall in [cs, cs + cn)
        int j = s0 + q4;
        if (j < cs) j += (cs - j + 3) / 4 * 4;
        for (;; j += 4) {
            const bool valid = j < e0 && j < cs + cn;
            if (!__any(valid)) break;
            const int jl = valid ? j - cs : 0;
            const double qv = valid ? sq[jl] : 0.0;
            const double wx = (sx[jl] - cx) * inv_alpha, wy = (sy[jl] - cy) * inv_alpha;
            const double y = 0.25 * (wx * wx + wy * wy);
            const double zx = wx * invR, zy = -wy * invR;   // conj(w)/R
            double F1, F2;
            f_start(y, t_sc, nser, F1, F2);
#pragma unroll
            for (int n = p; n >= N0; --n) {
                const double F0 = F1 + y * F2 * t_cnn[n];
                if (n <= N1) G[n - N0] = F0 * t_ify[n];
                F2 = F1;
                F1 = F0;
            }
            // conj(z)^N0
            double pr = 1.0, pi = 0.0;
            {
                double br = zx, bi = zy;
#pragma unroll
                for (int bit = 0; bit < 6; ++bit) {
                    if ((N0 >> bit) & 1) {
                        const double nr = pr * br - pi * bi;
                        pi = pr * bi + pi * br;
                        pr = nr;
                    }
                    if ((N0 >> (bit + 1)) != 0) {
                        const double nr = br * br - bi * bi;
                        bi = 2.0 * br * bi;
                        br = nr;
                    }
                }
            }
#pragma unroll
            for (int n = N0; n <= N1; ++n) {
                const double g = qv * G[n - N0];
                if (n == 0) {
                    acc[0] += g;
                } else {
                    acc[2 * n - 1 - O0] = __builtin_fma(g, pr, acc[2 * n - 1 - O0]);
                    acc[2 * n - O0] = __builtin_fma(g, pi, acc[2 * n - O0]);
                }
                const double nr = pr * zx - pi * zy;
                pi = pr * zy + pi * zx;
                pr = nr;
            }
        }
    }
#pragma unroll
    for (int o = 0; o < NA; ++o) {
        double v = acc[o];
        v += dpp_d<0xB1>(v);    // quad_perm [1,0,3,2]
        v += dpp_d<0x4E>(v);    // quad_perm [2,3,0,1]
        if (leaf_ok && (o & 3) == q4) M[b * Pp + O0 + o] = v;
    }
    if (H == 1 && leaf_ok)
        for (int o = 2 * p + 1 + q4; o < Pp; o += 4) M[b * Pp + o] = 0.0;
}

template <int PO>
__global__ __launch_bounds__(64) void k_p2m_half(
    int64_t leaf_base, int64_t nleaf, const int32_t *__restrict__ lrange,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ qs, int has_q, double inv_alpha,
    double invR, const double *__restrict__ invFY, const double *__restrict__ cnn,
    const double *__restrict__ sc, int nser, int Pp, double *__restrict__ M, int skip_d,
    double *__restrict__ zero, int64_t nzero) {
    constexpr int p = PO;
    extern __shared__ double smem[];
    {
        const int64_t nthr = (int64_t)gridDim.x * gridDim.y * 64;
        for (int64_t e = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 64 + threadIdx.x; e < nzero; e += nthr)
            zero[e] = 0.0;
    }
    double *t_sc = smem;                   // [2 nser] F_{p+1}, F_{p+2} series
    double *t_cnn = t_sc + 2 * nser;       // [p+2]
    double *t_ify = t_cnn + (p + 2);       // [p+2]
    for (int k = threadIdx.x; k < 2 * nser; k += 64) t_sc[k] = sc[k];
    for (int k = threadIdx.x; k < p + 2; k += 64) {
        t_cnn[k] = cnn[k];
        t_ify[k] = invFY[k];
    }
    __syncthreads();
    __shared__ double sx[kP2MStage], sy[kP2MStage], sq[kP2MStage];
    if (blockIdx.y == 0)
        p2m_half_body<PO, 0>(leaf_base, nleaf, lrange, bcx, bcy, px, py, qs, has_q, inv_alpha, invR, t_ify,
                             t_cnn, t_sc, nser, Pp, M, sx, sy, sq, skip_d);
    else
        p2m_half_body<PO, 1>(leaf_base, nleaf, lrange, bcx, bcy, px, py, qs, has_q, inv_alpha, invR, t_ify,
                             t_cnn, t_sc, nser, Pp, M, sx, sy, sq, skip_d);
}

// Cached P2M: the map from a point's strength to its leaf's multipole depends
// on the point and the tree only.  k_p2m_rows writes, per sorted point, the
// Pp coefficients it contributes per unit charge (charges) or per unit dipole
// component (dipoles: one row for each of d.n's two components); k_p2m_apply
// then forms every leaf's multipole as a sum of rows (one wavefront per leaf,
// lane = coefficient, contiguous loads).  Padding entries are zero.
__global__ __launch_bounds__(256) void k_p2m_rows(
    int64_t n0, int64_t n1, int64_t off1, const int32_t *__restrict__ pleaf, int64_t leaf_base,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, double inv_alpha, double invR, const double *__restrict__ invFY,
    const double *__restrict__ da, const double *__restrict__ db, const double *__restrict__ cnn,
    const double *__restrict__ sc, int nser, int p, int Pp, double *__restrict__ rq,
    double *__restrict__ rd, double *__restrict__ Gs) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n0 + n1) return;
    const bool dip = i >= n0;
    const int64_t j = dip ? off1 + (i - n0) : i;   // sorted point index
    const int64_t b = leaf_base + pleaf[j];
    const double wx = (px[j] - bcx[b]) * inv_alpha, wy = (py[j] - bcy[b]) * inv_alpha;
    const double y = 0.25 * (wx * wx + wy * wy);
    const double zx = wx * invR, zy = -wy * invR;   // conj(w)/R
    // G_n = F_n(y)/F_n(Y), n = 0..p+1, in this thread's scratch row of Gs
    double *G = Gs + i * (int64_t)(p + 2);
    double F1, F2;
    f_start(y, sc, nser, F1, F2);
    G[p + 1] = F1 * invFY[p + 1];
    for (int n = p; n >= 0; --n) {
        const double F0 = F1 + y * F2 * cnn[n];
        G[n] = F0 * invFY[n];
        F2 = F1;
        F1 = F0;
    }
    if (!dip) {
        double *row = rq + i * (int64_t)Pp;
        double pr = 1.0, pi = 0.0;     // conj(z)^n
        for (int n = 0; n <= p; ++n) {
            if (n == 0) {
                row[0] = G[0];
            } else {
                row[2 * n - 1] = G[n] * pr;
                row[2 * n] = G[n] * pi;
            }
            const double nr = pr * zx - pi * zy;
            pi = pr * zy + pi * zx;
            pr = nr;
        }
        for (int o = 2 * p + 1; o < Pp; ++o) row[o] = 0.0;
    } else {
        // term_n = h [a_n D Psi_{n+1} + b_n conj(D) Psi_{n-1}], D = Dx + i Dy:
        // the rows hold the coefficients of Dx and of Dy
        double *rx = rd + (i - n0) * 2 * (int64_t)Pp, *ry = rx + Pp;
        const double h = 0.5 * inv_alpha;
        double pr = zx, pi = zy;                       // conj(z)^1
        double c_r = G[0], c_i = 0.0;                  // Psi_0
        double n_r = G[1] * pr, n_i = G[1] * pi;       // Psi_1
        double m_r = n_r, m_i = -n_i;                  // Psi_{-1} = conj(Psi_1)
        for (int n = 0; n <= p; ++n) {
            const double an = h * da[n], bn = h * db[n];
            const double xr = an * n_r + bn * m_r, yr = -an * n_i + bn * m_i;
            const double xi = an * n_i + bn * m_i, yi = an * n_r - bn * m_r;
            if (n == 0) {
                rx[0] = xr;
                ry[0] = yr;
            } else {
                rx[2 * n - 1] = xr; ry[2 * n - 1] = yr;
                rx[2 * n] = xi;     ry[2 * n] = yi;
            }
            m_r = c_r; m_i = c_i;
            c_r = n_r; c_i = n_i;
            const double nr = pr * zx - pi * zy;
            pi = pr * zy + pi * zx;
            pr = nr;
            if (n + 2 <= p + 1) {
                n_r = G[n + 2] * pr; n_i = G[n + 2] * pi;
            } else {
                n_r = 0.0; n_i = 0.0;
            }
        }
        for (int o = 2 * p + 1; o < Pp; ++o) rx[o] = ry[o] = 0.0;
    }
}

// The strengths of the sorted points: gathered arrays (qs, dns), or read
// through the permutation (perm) from the caller's q and either dipole vectors
// dn or the factors w sigma n of the double-layer operator.
struct Strengths {
    const double *qs = nullptr, *dns = nullptr;
    const int32_t *perm = nullptr;
    const double *q = nullptr, *dn = nullptr, *w = nullptr, *sigma = nullptr, *normal = nullptr;
    __device__ __forceinline__ double charge(int64_t j) const { return perm ? q[perm[j]] : qs[j]; }
    // dipole of sorted position j, off1 the first dipole's
    __device__ __forceinline__ double2 dipole(int64_t j, int64_t off1) const {
        if (!perm) return make_double2(dns[2 * (j - off1)], dns[2 * (j - off1) + 1]);
        const int32_t i = perm[j];
        if (dn) return make_double2(dn[2 * i], dn[2 * i + 1]);
        const double s = (w ? w[i] : 1.0) * sigma[i];
        return make_double2(s * normal[2 * i], s * normal[2 * i + 1]);
    }
};

// one block of four wavefronts per leaf, lanes over coefficients: wavefront w
// sums the leaf's points w, w + 4, ... (two chains per lane) and the four
// partial rows are added through LDS; the blocks also clear zero[0..nzero)
constexpr int kRowStage = 256;   // strengths staged at a time (a multiple of the 32 that the wavefronts take together)
struct P2MApply {
    int64_t leaf_base, nleaf;
    const int32_t *lrange;
    const double *rq, *rd;
    int P, Pp;
    double *M, *zero;
    int64_t nzero;
};
__device__ __forceinline__ void p2m_apply(int64_t li, const P2MApply &a, const Strengths &st, int64_t off1, int has_q,
                                          int has_d, double *lds) {
    double(*part)[64] = reinterpret_cast<double(*)[64]>(lds);
    double *sx = lds + 256, *sy = sx + kRowStage;
    const int Pp = a.Pp;
    // zero[0..nzero) = 0 on the side (the local expansions, cleared here
    // rather than by a launch of their own)
    for (int64_t e = li * 256 + threadIdx.x; e < a.nzero; e += a.nleaf * 256) a.zero[e] = 0.0;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t b = a.leaf_base + li;
    const int s0 = a.lrange[li * 6], e0 = has_q ? a.lrange[li * 6 + 1] : s0;
    const int s1 = a.lrange[li * 6 + 2], e1 = has_d ? a.lrange[li * 6 + 3] : s1;
    const int o = lane;   // (Pp <= 64)
    double acc = 0.0;
    // this wavefront's points w, w + 4, ... of the cn staged: up to eight at a
    // time, all their rows' loads in flight (beyond the end: the last row, times
    // the zero that the stage is padded with)
    auto sum_rows = [&](auto at, int cn) {
        for (int j = w; j < cn; j += 32) {
            if (j + 16 < cn) at(std::integral_constant<int, 8>(), j);
            else if (j + 4 < cn) at(std::integral_constant<int, 4>(), j);
            else at(std::integral_constant<int, 1>(), j);
        }
    };
    for (int c0 = s0; c0 < e0; c0 += kRowStage) {
        const int cn = min(kRowStage, e0 - c0);
        __syncthreads();
        sx[threadIdx.x] = (int)threadIdx.x < cn ? st.charge(c0 + threadIdx.x) : 0.0;
        __syncthreads();
        if (o < Pp) {
            const double *r = a.rq + (int64_t)c0 * Pp + o;
            sum_rows([&](auto N, int j) {
                double m[N];
#pragma unroll
                for (int u = 0; u < N; ++u) m[u] = r[(int64_t)min(j + 4 * u, cn - 1) * Pp];
#pragma unroll
                for (int u = 0; u < N; ++u) acc = __builtin_fma(m[u], sx[j + 4 * u], acc);
            }, cn);
        }
    }
    for (int c0 = s1; c0 < e1; c0 += kRowStage) {
        const int cn = min(kRowStage, e1 - c0);
        __syncthreads();
        double2 d = make_double2(0.0, 0.0);
        if ((int)threadIdx.x < cn) d = st.dipole(c0 + threadIdx.x, off1);
        sx[threadIdx.x] = d.x;
        sy[threadIdx.x] = d.y;
        __syncthreads();
        if (o < Pp) {
            const double *r = a.rd + (int64_t)(c0 - off1) * 2 * Pp + o;
            sum_rows([&](auto N, int j) {
                double mx[N], my[N];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const double *rj = r + (int64_t)min(j + 4 * u, cn - 1) * 2 * Pp;
                    mx[u] = rj[0];
                    my[u] = rj[Pp];
                }
#pragma unroll
                for (int u = 0; u < N; ++u)
                    acc = __builtin_fma(mx[u], sx[j + 4 * u], __builtin_fma(my[u], sy[j + 4 * u], acc));
            }, cn);
        }
    }
    part[w][lane] = acc;
    __syncthreads();
    if (w == 0 && o < Pp)
        a.M[b * Pp + o] = o < a.P ? (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]) : 0.0;
}
constexpr int kP2MApplyLds = 256 + 2 * kRowStage;   // doubles
__global__ __launch_bounds__(256) void k_p2m_apply(P2MApply a, Strengths st, int64_t off1, int has_q, int has_d) {
    __shared__ double lds[kP2MApplyLds];
    p2m_apply(blockIdx.x, a, st, off1, has_q, has_d, lds);
}

// ------------------------------------------------------------- M2L (MFMA) --
// Matrix-core version: one workgroup (4 wavefronts) per tile of up to 64
// target boxes of one level and parity class.  C (Pp x 64 local
// coefficients) stays in accumulation registers for all 27 offsets; for each
// offset the Pp x Pp operator is double-buffered in LDS (prefetched into
// registers during the previous offset's MFMAs) and the gathered multipoles
// of the 16 boxes of a wavefront are read straight into B fragments.
//   v_mfma_f64_16x16x4f64: lane l holds A[l%16][l/16], B[l/16][l%16] and
//                          C rows l/16 + 4r, column l%16 (r = 0..3);
//   v_mfma_f32_16x16x4f32: same A, B; C rows 4(l/16) + r.
typedef double yk_d4 __attribute__((ext_vector_type(4)));
typedef float yk_f4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<double> {
    using acc = yk_d4;
    static __device__ __forceinline__ acc step(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct Mfma<float> {
    using acc = yk_f4;
    static __device__ __forceinline__ acc step(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// M2L by box, over its 27 V-list slots or (sparse) one translation at a time:
//   out[box] += sum_s Op[level][slot_op[cls][s]] * X[src[box][s]]
// Every box of a tile has the same level and parity class (so the same
// operator per slot).  X is read in its own type TS and converted to T.
//
// A workgroup owns 64 boxes (4 wavefronts x 16 columns) and walks the slots;
// the slot's Pp x Pp operator is double-buffered in LDS and the gathered
// source coefficients of the next slot are loaded while the current slot runs.
// With P = 16 NB + 1 real coefficients (p a multiple of 8), the last index
// SP = 16 NB is split off: the matrix cores take the 16 NB x 16 NB block of
// indices 0..SP-1 and the vector units add row SP and column SP (a padded
// 16 (NB+1) product would spend 40% more matrix-core work on padding).
//
// Contraction order: lane group g (lane / 16) supplies, in the two matrix-core
// steps of pair kp, the contraction indices 8 kp + 2 g and 8 kp + 2 g + 1, so
// each lane loads its source coefficients as aligned pairs; the operator
// fragments read from LDS follow the same order.
typedef double yk_dpair __attribute__((ext_vector_type(2)));
typedef float yk_fpair __attribute__((ext_vector_type(2)));
template <typename TS> struct Pair2;
template <> struct Pair2<double> { using type = yk_dpair; };
template <> struct Pair2<float> { using type = yk_fpair; };

template <typename T, typename TS, int PP, bool SPLIT_REQ, int CB>
__global__ __launch_bounds__(256) void k_tile_gemm(const int4 *__restrict__ tiles, int tile0,
                                                   const int32_t *__restrict__ boxes, int nslot,
                                                   const int32_t *__restrict__ src,
                                                   const int32_t *__restrict__ slot_op,
                                                   const T *__restrict__ Op, int64_t op_stride,
                                                   const TS *__restrict__ X, int nparts,
                                                   double *__restrict__ out,
                                                   const int32_t *__restrict__ tgt, double *__restrict__ slab) {
    constexpr bool SPLIT = SPLIT_REQ && PP > 16;   // (the host never asks for PP = 16)
    constexpr int NB = SPLIT ? PP / 16 - 1 : PP / 16;   // 16-row blocks on the matrix cores
    constexpr int SP = 16 * NB;                         // split-off index (SPLIT only)
    constexpr int NKP = 2 * NB;                         // contraction pairs
    // LDS copy of the operator: the NCOL columns used, each LDA rows (with the
    // split, 49 x 52 instead of 64 x 64 for p = 24: less LDS, so three
    // workgroups fit a compute unit, and a column stride off the bank period)
    constexpr int NCOL = SPLIT ? SP + 1 : PP;
    constexpr int LDA = SPLIT ? ((SP + 1 + 3) & ~3) : PP;
    constexpr int kPairs = NCOL * LDA / 2;              // operator pairs per slot
    constexpr int NL2 = (kPairs + 255) / 256;           // pairs per thread
    constexpr int kMaxSlot = 27;
    constexpr int NC = 64 * CB;                         // boxes (columns) per workgroup
    using V2 = typename Pair2<TS>::type;
    using T2 = typename Pair2<T>::type;
    __shared__ T As[2][NCOL * LDA];
    __shared__ int32_t s_src[kMaxSlot * NC];
    using MF = Mfma<T>;
    // nparts > 1 (few tiles): the slots of a tile are shared among nparts
    // workgroups.  With tgt (sparse M2L) the tile's entries are translation
    // indices: the source is src[entry], the target is row tgt[entry].  In both
    // cases several workgroups contribute to one output row, so each stores its
    // result in a row of its own of slab
    // (translation `entry`, or column j of workgroup bid: row bid * NC + j),
    // which k_slab_reduce_* then add to the outputs in a fixed order: the
    // sums do not depend on the order the workgroups run in.
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int part = bid % nparts;
    const int4 tl = tiles[tile0 + bid / nparts];
    const int level = tl.x, cls = tl.y, start = tl.z, count = tl.w;
    const int sl0 = part * nslot / nparts, sl1 = (part + 1) * nslot / nparts;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4;
    // column block c of this wavefront: columns 16 (CB w + c) + lane % 16
    int jb[CB];
    bool colvalid[CB];
    int64_t boxj[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        jb[c] = 16 * (CB * w + c) + (lane & 15);
        colvalid[c] = jb[c] < count;
        boxj[c] = colvalid[c] ? (tgt ? tgt[boxes[start + jb[c]]] : boxes[start + jb[c]]) : -1;
    }
    // source box of every (slot, column) of the tile, -1 where empty
    for (int e = sl0 * NC + tid; e < sl1 * NC; e += 256) {
        const int sl = e / NC, j = e % NC;
        s_src[e] = j < count ? src[(int64_t)boxes[start + j] * nslot + sl] : -1;
    }
    typename MF::acc acc[CB][NB];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int r = 0; r < NB; ++r) acc[c][r] = typename MF::acc{0, 0, 0, 0};
    T rowacc[CB], colacc[CB][NB][4];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        rowacc[c] = T(0);
#pragma unroll
        for (int r = 0; r < NB; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) colacc[c][r][q] = T(0);
    }
    const T *Olev = Op + (int64_t)level * op_stride;
    auto op_of = [&](int sl) -> const T2 * {
        return reinterpret_cast<const T2 *>(Olev + (size_t)slot_op[cls * nslot + sl] * PP * PP);
    };
    // global pair of LDS pair e (column-major, PP rows per column in memory)
    auto gpair = [&](int e) { return (e / (LDA / 2)) * (PP / 2) + e % (LDA / 2); };
    // B fragment of a slot: unconditional loads (row 0 stands in for an empty
    // slot) and the empty slot's zeros selected when the fragment is consumed,
    // so the loads of the next slot stay in flight during the current one (a
    // select, not a product, so whatever row 0 holds never reaches the sums)
    V2 braw[CB][NKP];
    TS bsraw[CB];
    bool bvalid[CB];
    T bcur[CB][2 * NKP], bs[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        bsraw[c] = TS(0);
        bvalid[c] = false;
        bs[c] = T(0);
    }
    T2 pre[NL2];
    auto load_b = [&](int sl) {
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int32_t sj = s_src[sl * NC + jb[c]];
            const TS *row = X + (int64_t)(sj >= 0 ? sj : 0) * PP;
            const V2 *row2 = reinterpret_cast<const V2 *>(row) + g;
#pragma unroll
            for (int kp = 0; kp < NKP; ++kp) braw[c][kp] = row2[4 * kp];
            if constexpr (SPLIT) bsraw[c] = row[SP];
            bvalid[c] = sj >= 0;
        }
    };
    auto take_b = [&]() {
#pragma unroll
        for (int c = 0; c < CB; ++c) {
#pragma unroll
            for (int kp = 0; kp < NKP; ++kp) {
                bcur[c][2 * kp] = bvalid[c] ? (T)braw[c][kp].x : T(0);
                bcur[c][2 * kp + 1] = bvalid[c] ? (T)braw[c][kp].y : T(0);
            }
            if constexpr (SPLIT) bs[c] = bvalid[c] ? (T)bsraw[c] : T(0);
        }
    };
    __syncthreads();
    load_b(sl0);
    {
        const T2 *Tg = op_of(sl0);
        T2 *Ad = reinterpret_cast<T2 *>(As[0]);
#pragma unroll
        for (int e = 0; e < NL2; ++e)
            if (kPairs >= 256 * NL2 || tid + 256 * e < kPairs) Ad[tid + 256 * e] = Tg[gpair(tid + 256 * e)];
    }
    take_b();
    __syncthreads();
    for (int slot = sl0; slot < sl1; ++slot) {
        const int cur = (slot - sl0) & 1;
        const bool more = slot + 1 < sl1;
        if (more) {
            load_b(slot + 1);
            const T2 *Tg = op_of(slot + 1);
#pragma unroll
            for (int e = 0; e < NL2; ++e)
                if (kPairs >= 256 * NL2 || tid + 256 * e < kPairs) pre[e] = Tg[gpair(tid + 256 * e)];
        }
        // operator column-major: A[i][k] = As[k * LDA + i]; step (kp, e) takes
        // contraction index 8 kp + 2 g + e in lane group g; each operator
        // fragment read from LDS serves the CB column blocks
        // (the fragments of step s are read two steps ahead, into a ring of
        // three, so the matrix cores do not wait on LDS between steps)
        const T *Ac = As[cur] + 2 * g * LDA + (lane & 15);
        constexpr int NS = 2 * NKP;   // steps; step s = 2 kp + e
        T afr[3][NB];
        auto read_a = [&](int st, T *dst) {
#pragma unroll
            for (int rt = 0; rt < NB; ++rt) dst[rt] = Ac[(8 * (st >> 1) + (st & 1)) * LDA + 16 * rt];
        };
        read_a(0, afr[0]);
        if (NS > 1) read_a(1, afr[1]);
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            if (st + 2 < NS) read_a(st + 2, afr[(st + 2) % 3]);
#pragma unroll
            for (int rt = 0; rt < NB; ++rt)
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[c][rt] = MF::step(afr[st % 3][rt], bcur[c][st], acc[c][rt]);
        }
        if constexpr (SPLIT) {
            const T *A = As[cur];
            // row SP: this lane's share of sum_k A[SP][k] b[k]; column SP into
            // the rows this lane holds of the matrix-core result
#pragma unroll
            for (int kp = 0; kp < NKP; ++kp)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const T a = A[(8 * kp + 2 * g + e) * LDA + SP];
#pragma unroll
                    for (int c = 0; c < CB; ++c) rowacc[c] += a * bcur[c][2 * kp + e];
                }
            if (g == 0) {
                const T a = A[SP * LDA + SP];
#pragma unroll
                for (int c = 0; c < CB; ++c) rowacc[c] += a * bs[c];
            }
#pragma unroll
            for (int rt = 0; rt < NB; ++rt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const T a = A[SP * LDA + 16 * rt + MF::row(lane, q)];
#pragma unroll
                    for (int c = 0; c < CB; ++c) colacc[c][rt][q] += a * bs[c];
                }
        }
        if (more) {
            T2 *Ad = reinterpret_cast<T2 *>(As[cur ^ 1]);
#pragma unroll
            for (int e = 0; e < NL2; ++e)
                if (kPairs >= 256 * NL2 || tid + 256 * e < kPairs) Ad[tid + 256 * e] = pre[e];
            take_b();
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        if constexpr (SPLIT) {
            rowacc[c] += __shfl_xor(rowacc[c], 16, 64);
            rowacc[c] += __shfl_xor(rowacc[c], 32, 64);
        }
        if (colvalid[c]) {
            const bool store = slab != nullptr;
            double *o = store ? slab + (tgt ? (int64_t)boxes[start + jb[c]] : (int64_t)bid * NC + jb[c]) * PP
                                : out + boxj[c] * PP;
#pragma unroll
            for (int rt = 0; rt < NB; ++rt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 16 * rt + MF::row(lane, q);
                    const double v = SPLIT ? (double)acc[c][rt][q] + (double)colacc[c][rt][q] : (double)acc[c][rt][q];
                    o[i] = store ? v : o[i] + v;
                }
            if constexpr (SPLIT) {
                if (g == 0) o[SP] = store ? (double)rowacc[c] : o[SP] + (double)rowacc[c];
                // padding entries SP + 1 .. PP - 1: the sums over the rows take them too
                if (store)
                    for (int i = SP + 1 + g; i < PP; i += 4) o[i] = 0.0;
            }
        }
    }
}

// Persistent M2L for 64 padded coefficients without the split (p = 31), FP64,
// on trees with at least as many tiles as the launch has workgroups.  The
// launch is one resident round (three workgroups per compute unit: the slot's
// operator is staged in LDS in two halves of 32 contraction columns, double
// buffered at half-slot steps, 32 KB); workgroup b takes the contiguous run
// [U b / G, U (b + 1) / G) of the U = 54 ntiles (tile, slot, half) units in
// the tiles' order and keeps the tile's results in its accumulators across
// the slots, so no compute unit idles while another finishes a last round of
// whole tiles.  A run is at least 54 units long, so a tile is shared by at
// most two workgroups; those add into the local expansions, which are zero
// before M2L, with atomic adds, and with two addends into zero the sum does
// not depend on their order.  A tile that lies within one run is added
// without atomics.  The matrix-core steps and fragment layout are those of
// k_tile_gemm.
__global__ __launch_bounds__(256) void k_m2l_persist(const int4 *__restrict__ tiles, int ntiles,
                                                     const int32_t *__restrict__ boxes,
                                                     const int32_t *__restrict__ src,
                                                     const int32_t *__restrict__ slot_op,
                                                     const double *__restrict__ Op, int64_t op_stride,
                                                     const double *__restrict__ X, double *__restrict__ out) {
    constexpr int PP = 64, NB = 4, LDA = 64, NCOLH = 32, NSH = 8, kSlots = 27, NH = 2;
    constexpr int kPairs = NCOLH * LDA / 2;   // operator pairs per half
    constexpr int NL2 = kPairs / 256;         // pairs per thread
    __shared__ double As[2][NCOLH * LDA];
    using MF = Mfma<double>;
    const int G = gridDim.x;
    const int bid = xcd_remap(blockIdx.x, G);
    const int64_t U = (int64_t)ntiles * kSlots * NH;
    const int64_t u0 = U * bid / G, u1 = U * (bid + 1) / G;
    if (u0 >= u1) return;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4;
    const int jb = 16 * w + (lane & 15);
    // current tile
    int4 tl = tiles[(int)(u0 / (kSlots * NH))];
    bool colvalid = jb < tl.w;
    int64_t boxj = colvalid ? boxes[tl.z + jb] : -1;
    yk_d4 acc[NB];
#pragma unroll
    for (int r = 0; r < NB; ++r) acc[r] = yk_d4{0, 0, 0, 0};
    yk_dpair braw[8];
    bool bvalid = false;
    double bcur[16];
    yk_dpair pre[NL2];
    auto load_b = [&](const int4 &t, int sl) {
        int32_t sj = -1;
        if (jb < t.w) sj = src[(int64_t)boxes[t.z + jb] * kSlots + sl];
        const yk_dpair *row2 = reinterpret_cast<const yk_dpair *>(X + (int64_t)(sj >= 0 ? sj : 0) * PP) + g;
#pragma unroll
        for (int kp = 0; kp < 8; ++kp) braw[kp] = row2[4 * kp];
        bvalid = sj >= 0;
    };
    auto take_b = [&]() {
#pragma unroll
        for (int kp = 0; kp < 8; ++kp) {
            bcur[2 * kp] = bvalid ? braw[kp].x : 0.0;
            bcur[2 * kp + 1] = bvalid ? braw[kp].y : 0.0;
        }
    };
    auto op_half = [&](const int4 &t, int sl, int h) -> const yk_dpair * {
        return reinterpret_cast<const yk_dpair *>(Op + (int64_t)t.x * op_stride +
                                                  (size_t)slot_op[t.y * kSlots + sl] * PP * PP) +
               (size_t)h * NCOLH * (PP / 2);
    };
    {
        const int sl = (int)((u0 / NH) % kSlots), h = (int)(u0 % NH);
        load_b(tl, sl);
        const yk_dpair *Tg = op_half(tl, sl, h);
        yk_dpair *Ad = reinterpret_cast<yk_dpair *>(As[0]);
#pragma unroll
        for (int e = 0; e < NL2; ++e) Ad[tid + 256 * e] = Tg[tid + 256 * e];
        take_b();
    }
    __syncthreads();
    int64_t tile_first = (u0 / (kSlots * NH)) * (kSlots * NH);
    for (int64_t u = u0; u < u1; ++u) {
        const int cur = (int)((u - u0) & 1);
        const int h = (int)(u % NH), sl = (int)((u / NH) % kSlots);
        const bool more = u + 1 < u1;
        const int64_t un = u + 1;
        const int hn = (int)(un % NH), sln = (int)((un / NH) % kSlots);
        const bool new_tile = more && sln == 0 && hn == 0;
        int4 tn = tl;
        if (more) {
            if (new_tile) tn = tiles[(int)(un / (kSlots * NH))];
            if (hn == 0) load_b(tn, sln);
            const yk_dpair *Tg = op_half(tn, sln, hn);
#pragma unroll
            for (int e = 0; e < NL2; ++e) pre[e] = Tg[tid + 256 * e];
        }
        // this half's B values (a select: bcur is never indexed at run time)
        double bp[NSH];
#pragma unroll
        for (int st = 0; st < NSH; ++st) bp[st] = h ? bcur[NSH + st] : bcur[st];
        const double *Ac = As[cur] + 2 * g * LDA + (lane & 15);
        double afr[3][NB];
        auto read_a = [&](int st, double *dst) {
#pragma unroll
            for (int rt = 0; rt < NB; ++rt) dst[rt] = Ac[(8 * (st >> 1) + (st & 1)) * LDA + 16 * rt];
        };
        read_a(0, afr[0]);
        read_a(1, afr[1]);
#pragma unroll
        for (int st = 0; st < NSH; ++st) {
            if (st + 2 < NSH) read_a(st + 2, afr[(st + 2) % 3]);
#pragma unroll
            for (int rt = 0; rt < NB; ++rt) acc[rt] = MF::step(afr[st % 3][rt], bp[st], acc[rt]);
        }
        // the tile's last unit, or the run's: add the results (a run may end,
        // or start, between the two halves of a slot)
        if ((h == NH - 1 && sl == kSlots - 1) || !more) {
            const bool whole = tile_first >= u0 && tile_first + kSlots * NH <= u1;
            if (colvalid) {
                double *o = out + boxj * PP;
#pragma unroll
                for (int rt = 0; rt < NB; ++rt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int i = 16 * rt + MF::row(lane, q);
                        if (whole) o[i] += acc[rt][q];
                        else atomicAdd(o + i, acc[rt][q]);
                    }
            }
#pragma unroll
            for (int r = 0; r < NB; ++r) acc[r] = yk_d4{0, 0, 0, 0};
        }
        if (more) {
            yk_dpair *Ad = reinterpret_cast<yk_dpair *>(As[cur ^ 1]);
#pragma unroll
            for (int e = 0; e < NL2; ++e) Ad[tid + 256 * e] = pre[e];
            if (hn == 0) take_b();
            if (new_tile) {
                tl = tn;
                tile_first = un;
                colvalid = jb < tl.w;
                boxj = colvalid ? boxes[tl.z + jb] : -1;
            }
        }
        __syncthreads();
    }
}

// Fixed-order sums of the slab rows of k_tile_gemm into the outputs.
// Sparse M2L: target box t of the list gets rows[off[t] .. off[t+1]) (its
// translations in increasing index), one wavefront per target.  Bound by the
// latency of the row loads: the row indices are read by the lanes in one load
// and the rows' loads issued kCsrRows together (one row after the other: 11.5
// us on the 28,672-node boundary tree; a density solve there 2.27 -> 2.15 ms).
constexpr int kCsrRows = 8;
__global__ __launch_bounds__(256) void k_slab_reduce_csr(int64_t ntgt, const int32_t *__restrict__ tgt,
                                                         const int32_t *__restrict__ off,
                                                         const int32_t *__restrict__ rows,
                                                         const double *__restrict__ slab, int PP,
                                                         double *__restrict__ out) {
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (t >= ntgt) return;   // (whole wavefronts)
    const int i = lane < PP ? lane : PP - 1;
    const int k0 = off[t], k1 = off[t + 1];
    double *o = out + (int64_t)tgt[t] * PP + i;
    const double before = *o;
    double acc = 0.0;
    for (int kb = k0; kb < k1; kb += 64) {
        const int nk = min(64, k1 - kb);
        const int mine = rows[kb + min(lane, nk - 1)];
        for (int k = 0; k < nk; k += kCsrRows) {
            double v[kCsrRows];
#pragma unroll
            for (int u = 0; u < kCsrRows; ++u)
                v[u] = slab[(int64_t)__shfl(mine, min(k + u, nk - 1), 64) * PP + i];
#pragma unroll
            for (int u = 0; u < kCsrRows; ++u)
                if (k + u < nk) acc += v[u];
        }
    }
    if (lane < PP) *o = before + acc;
}

// Split slots: column j of tile t gets the rows of its nparts (<= kMaxParts)
// workgroups in part order.  A thread per element and all its parts' loads
// issued together (a workgroup per tile walking its elements one part after
// the other was a chain of 112 memory round trips: 35 us a launch whatever
// its size, now about 5: a pass over 4,096 + 1,536 points 112 -> 80 us).
constexpr int kMaxParts = 7;
__global__ __launch_bounds__(256) void k_slab_reduce_parts(const int4 *__restrict__ tiles, int tile0,
                                                           const int32_t *__restrict__ boxes, int nparts, int NC,
                                                           const double *__restrict__ slab, int PP,
                                                           double *__restrict__ out) {
    const int t = blockIdx.x;
    const int4 tl = tiles[tile0 + t];
    const int e = blockIdx.y * 256 + threadIdx.x;
    if (e >= tl.w * PP) return;
    const int j = e / PP, i = e - j * PP;
    const double *s = slab + ((int64_t)t * nparts * NC + j) * PP + i;
    double v[kMaxParts];
#pragma unroll
    for (int part = 0; part < kMaxParts; ++part) v[part] = s[(int64_t)min(part, nparts - 1) * NC * PP];
    double acc = 0.0;
#pragma unroll
    for (int part = 0; part < kMaxParts; ++part)
        if (part < nparts) acc += v[part];
    out[(int64_t)boxes[tl.z + j] * PP + i] += acc;
}

// Where the partial rows of a launch whose workgroups share output rows go,
// and (sparse M2L) the fixed order in which they are summed.
struct SlabPlan {
    DevBuf<double> *buf = nullptr;
    int64_t ntgt = 0;                           // sparse: targets with translations
    const int32_t *tgt = nullptr, *off = nullptr, *rows = nullptr;
};

template <typename T, typename TS, int CB = 1>
void launch_tile_gemm(Context &ctx, int P, int Pp, int ntiles, const int4 *tiles, int tile0,
                      const int32_t *boxes, int nslot, const int32_t *src, const int32_t *slot_op,
                      const T *Op, int64_t op_stride, const TS *X, double *out, const int32_t *tgt = nullptr,
                      const SlabPlan *slab = nullptr, int64_t ntrans = 0) {
    if (ntiles <= 0) return;
    if (nslot < 1 || nslot > 27) throw Error{YK_ERR_INTERNAL, "tile GEMM supports 1..27 slots"};
    const bool split = Pp >= 32 && P == Pp - 15;
    // fewer tiles than compute units: share each tile's slots among up to 7
    // workgroups (about 4 slots each), whose partial rows are summed after
    const int nparts = (slab && nslot >= 8 && ntiles < 256) ? std::min(kMaxParts, (512 + ntiles - 1) / ntiles) : 1;
    const unsigned grid = (unsigned)ntiles * (unsigned)nparts;
    if (tgt && !slab) throw Error{YK_ERR_INTERNAL, "sparse tile GEMM needs a slab"};
    constexpr int NC = 64 * CB;
    double *sl = nullptr;
    if (tgt) sl = slab->buf->ensure((size_t)std::max<int64_t>(ntrans, 1) * Pp);
    else if (nparts > 1) sl = slab->buf->ensure((size_t)grid * NC * Pp);
#define YK_TILE_CASE(PPV)                                                                          \
    case PPV:                                                                                      \
        if (split)                                                                                 \
            hipLaunchKernelGGL((k_tile_gemm<T, TS, PPV, true, CB>), dim3(grid), dim3(256), 0,     \
                               ctx.stream, tiles, tile0, boxes, nslot, src, slot_op, Op, op_stride, \
                               X, nparts, out, tgt, sl);                                          \
        else                                                                                       \
            hipLaunchKernelGGL((k_tile_gemm<T, TS, PPV, false, CB>), dim3(grid), dim3(256), 0,    \
                               ctx.stream, tiles, tile0, boxes, nslot, src, slot_op, Op, op_stride, \
                               X, nparts, out, tgt, sl);                                          \
        break;
    switch (Pp) {
        YK_TILE_CASE(16)
        YK_TILE_CASE(32)
        YK_TILE_CASE(48)
        YK_TILE_CASE(64)
        default:
            throw Error{YK_ERR_INTERNAL, "no matrix-core kernel for this padded order"};
    }
#undef YK_TILE_CASE
    check_launch(ctx, "k_tile_gemm");
    if (tgt) {
        if (slab->ntgt > 0)
            hipLaunchKernelGGL(k_slab_reduce_csr, dim3((unsigned)((slab->ntgt + 3) / 4)), dim3(256), 0, ctx.stream,
                               slab->ntgt, slab->tgt, slab->off, slab->rows, sl, Pp, out);
        check_launch(ctx, "k_slab_reduce_csr");
    } else if (nparts > 1) {
        hipLaunchKernelGGL(k_slab_reduce_parts, dim3((unsigned)ntiles, (unsigned)(NC * Pp / 256)), dim3(256), 0,
                           ctx.stream, tiles, tile0, boxes, nparts, NC, sl, Pp, out);
        check_launch(ctx, "k_slab_reduce_parts");
    }
}

__global__ void k_to_float(int64_t n, const double *__restrict__ a, float *__restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}

// ----------------------------------------------------------- leaf kernel ---
// Near field in scaled coordinates: separations are multiplied by 1/(2 alpha),
// so the squared scaled separation is t = r^2/(4 alpha^2) itself and
//     K0(r/alpha)            = h(t) A(t) + B(t),           h = -(1/2) ln t,
//     4 K1(r/alpha)/(r/alpha) = 1/t - 2 h(t) C(t) - D(t)
// for t <= 1 (series in bessel_tables.h); larger t use the Chebyshev forms.
template <int NT, typename T>
__device__ __forceinline__ T horner_n(const T (&c)[YK_NSER64], T t) {
    T s = c[NT - 1];
#pragma unroll
    for (int k = NT - 2; k >= 0; --k) s = __builtin_fma(s, t, c[k]);
    return s;
}

// h(t) = -(1/2) ln t for a positive normal t.  With t = m 2^e, m in [1/2, 1),
// piece i of [1/2, 1) is given by the top eight fraction bits of m; the table
// holds rc_i ~ 1/c_i (c_i the piece's centre) and (1/2) ln rc_i, and
// -(1/2) ln m = (1/2) ln rc_i - (1/2) log1p(m rc_i - 1) with |m rc_i - 1| < 2^-9,
// where five terms of the log1p series leave an error below r^6/12 < 2^-57.
// ln 2 is split so that e * ln2_hi is exact.
__device__ __forceinline__ double neg_half_log(double t, const double2 *__restrict__ tab) {
    const int e = __builtin_amdgcn_frexp_exp(t);
    const double m = __builtin_amdgcn_frexp_mant(t);
    const int i = (__double2hiint(m) >> 12) & (YK_LOG_TAB - 1);
    const double2 c = tab[i];
    const double r = __builtin_fma(m, c.x, -1.0);
    double s = __builtin_fma(r, -0.1, 0.125);
    s = __builtin_fma(s, r, -1.0 / 6.0);
    s = __builtin_fma(s, r, 0.25);
    s = __builtin_fma(s, r, -0.5);
    const double de = (double)e;
    constexpr double h2_hi = -0.5 * 6.93147180369123816490e-01;   // -(1/2) 0x3FE62E42FEE00000
    constexpr double h2_lo = -0.5 * 1.90821492927058770002e-10;
    return __builtin_fma(de, h2_hi, c.y + __builtin_fma(de, h2_lo, s * r));
}

// The forms for large arguments as calls (kCall): inlined, the series of every
// loop share the registers with their constants.  Called wherever many wavefronts
// hide what a call costs; see pick_leaf_kernel for the other case.
__device__ __forceinline__ double k1oz4_large(double t) {
    const double z = 2.0 * sqrt(t);
    return 4.0 * k1_large(z) / z;
}
__device__ __attribute__((noinline)) double k0_large_c(double t) { return k0_large(2.0 * sqrt(t)); }
__device__ __attribute__((noinline)) double k1oz4_large_c(double t) { return k1oz4_large(t); }
template <int NT, bool kSmallOnly, bool kCall = true>
__device__ __forceinline__ double near_k0(double t, const double2 *__restrict__ tab) {
    if (kSmallOnly || t <= 1.0)
        return __builtin_fma(neg_half_log(t, tab), horner_n<NT>(yk_ser_A, t), horner_n<NT>(yk_ser_B, t));
    if constexpr (kCall) return k0_large_c(t);
    else return k0_large(2.0 * sqrt(t));
}
// 4 K1(z)/z with t = z^2/4
template <int NT, bool kSmallOnly, bool kCall = true>
__device__ __forceinline__ double near_k1oz4(double t, const double2 *__restrict__ tab) {
    if (kSmallOnly || t <= 1.0) {
        const double h2 = 2.0 * neg_half_log(t, tab);
        return fast_rcp(t) - __builtin_fma(h2, horner_n<NT>(yk_ser_C, t), horner_n<NT>(yk_ser_D, t));
    }
    if constexpr (kCall) return k1oz4_large_c(t);
    else return k1oz4_large(t);
}

template <int NT>
__device__ __forceinline__ float horner_nf(const float (&c)[YK_NSER32], float t) {
    float s = c[NT - 1];
#pragma unroll
    for (int k = NT - 2; k >= 0; --k) s = s * t + c[k];
    return s;
}
template <bool kSmallOnly>
__device__ __forceinline__ float near_k0_f(float t) {
    if (kSmallOnly || t <= 1.0f) {
        const float lt = __logf(t);
        return -0.5f * lt * horner_nf<YK_NSER32>(yk_ser_A_f, t) + horner_nf<YK_NSER32>(yk_ser_B_f, t);
    }
    return k0_large_f(2.0f * sqrtf(t));
}
template <bool kSmallOnly>
__device__ __forceinline__ float near_k1oz4_f(float t) {
    if (kSmallOnly || t <= 1.0f) {
        const float lt = __logf(t);
        return 1.0f / t + lt * horner_nf<YK_NSER32>(yk_ser_C_f, t) - horner_nf<YK_NSER32>(yk_ser_D_f, t);
    }
    const float z = 2.0f * sqrtf(t);
    return 4.0f * k1_large_f(z) / z;
}

// Near-field accumulation policy: FP64 (series and sums in double) or FP32
// (separations and the dipole dot product in double, the Bessel series, the
// logarithm and the accumulation in float).
template <int NT, bool kSmallOnly, bool kF32, bool kCall>
struct Near {
    using acc_t = typename std::conditional<kF32, float, double>::type;
    static __device__ __forceinline__ acc_t charge(double q, double t, const double2 *tab) {
        if constexpr (kF32) return (float)q * near_k0_f<kSmallOnly>((float)t);
        else return q * near_k0<NT, kSmallOnly, kCall>(t, tab);
    }
    // dot = (x - y).(d n_y) in scaled coordinates; the caller multiplies the
    // sum by 1/(2 alpha), which turns dot * 4K1(z)/z into (1/alpha) K1(z) (x-y).(d n)/r
    static __device__ __forceinline__ acc_t dipole(double dot, double t, const double2 *tab) {
        if constexpr (kF32) return (float)dot * near_k1oz4_f<kSmallOnly>((float)t);
        else return dot * near_k1oz4<NT, kSmallOnly, kCall>(t, tab);
    }
};

// The pairs' arithmetic bounds it (one pair at a time per lane and more wavefronts
// beat two in flight: the two pairs' registers cost a wavefront per SIMD; a
// coincident pair is masked, not branched around).
// One wavefront per item: up to 64 targets of one leaf.  With c targets, the
// 64 lanes form g = floor(64/c) groups of c lanes; lane l serves target l mod c
// and walks every g-th source of the leaf's U list, so at most c - 1 lanes
// idle.  U-list sources are staged into LDS (scaled coordinates and strengths)
// in chunks of kLeafStage; the group partial sums are combined through LDS at
// the end.  The result is the near field alone (k_l2p adds the far field).
constexpr int kLeafStage = 192;

// the longest U list (9 in a uniform tree; the adaptive one's 2:1 balance
// bounds it by 13)
constexpr int kLeafU = 16;
struct LeafLds {
    double x[kLeafStage], y[kLeafStage], a[kLeafStage], b[kLeafStage];
    // per source set: flat end of each U-list leaf's sources, their first index less the flat begin
    int end[2][kLeafU], beg[2][kLeafU];
};
struct LeafArgs {
    const int2 *items;
    const int32_t *lrange, *uoff, *ulist;
    const double *px, *py, *qs, *dns;
    int64_t off1;
    int has_q, has_d, mask;
    double inv2a, dip_scale;
    double *outs;
};
// one item by the calling wavefront (sync: over the wavefront; the log table is ready after the first)
template <int NT, bool kSmallOnly, bool kF32, bool kCall = true, typename Sync>
__device__ __forceinline__ void leaf_item(const int2 item, const LeafArgs &A, LeafLds &S,
                                          const double2 *__restrict__ s_log, Sync sync) {
    const int li = item.x;
    const int lane = threadIdx.x & 63;
    int rs[3], re[3], ntot = 0;
    for (int s = 0; s < 3; ++s) {
        rs[s] = A.lrange[li * 6 + 2 * s];
        re[s] = (A.mask >> s) & 1 ? A.lrange[li * 6 + 2 * s + 1] : rs[s];
        ntot += re[s] - rs[s];
    }
    const int u0 = A.uoff[li], nu = A.uoff[li + 1] - u0;
    // U-list source ranges of the two source sets (lanes 0 to 15 charges, 16 to
    // 31 dipoles), in LDS for the lanes' searches below
    {
        const int u = lane & 15, set = (lane >> 4) & 1;
        int a = 0, n = 0;
        if (u < nu && (set == 0 ? A.has_q : A.has_d)) {
            const int ul = A.ulist[u0 + u];
            a = A.lrange[ul * 6 + 2 * set];
            n = A.lrange[ul * 6 + 2 * set + 1] - a;
        }
        int end = n;
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) {
            const int o = __shfl_up(end, m, 16);
            if (u >= m) end += o;
        }
        if (lane < 32) {
            S.end[set][u] = end;
            S.beg[set][u] = a - (end - n);
        }
    }
    sync();
    const int tb = item.y;
    const int c = min(64, ntot - tb);          // >= 1 by construction of the items
    const int g = 64 / c;
    const int ti = lane % c, sub = lane / c;
    const bool valid = sub < g;
    int k = tb + ti, t = -1;
    for (int s = 0; s < 3; ++s) {
        const int n = re[s] - rs[s];
        if (t < 0 && k < n) t = rs[s] + k;
        k -= n;
    }
    // separations are formed from the unscaled coordinates and then scaled:
    // the difference of two nearby coordinates is exact, whereas scaling
    // first would round each coordinate, which costs digits in (x - y).n for
    // the nearly tangential pairs of densely sampled, tightly curved curves
    const double xs = A.px[t], ys = A.py[t];
    using NearT = Near<NT, kSmallOnly, kF32, kCall>;
    typename NearT::acc_t near_q = 0, near_d = 0;
    for (int set = 0; set < 2; ++set) {
        const int ntot_s = S.end[set][kLeafU - 1];
        for (int c0 = 0; c0 < ntot_s; c0 += kLeafStage) {
            const int cn = min(kLeafStage, ntot_s - c0);
            sync();
            // cooperative gather of flat source indices [c0, c0 + cn) into LDS
            for (int f = lane; f < cn; f += 64) {
                int u = 0;   // its leaf: the first whose end is beyond it
#pragma unroll
                for (int m = kLeafU / 2; m >= 1; m >>= 1)
                    if (S.end[set][u + m - 1] <= c0 + f) u += m;
                const int j = S.beg[set][u] + c0 + f;
                S.x[f] = A.px[j];
                S.y[f] = A.py[j];
                if (set == 0) {
                    S.a[f] = A.qs[j];
                } else {
                    const int64_t jd = j - A.off1;
                    S.a[f] = A.dns[2 * jd];
                    S.b[f] = A.dns[2 * jd + 1];
                }
            }
            sync();
            if (valid) {
                // full passes (every lane's source index in range), then the tail
                const int nfull = cn - cn % g;
                if (set == 0) {
                    auto pair = [&](int j) {
                        const double dx = (xs - S.x[j]) * A.inv2a, dy = (ys - S.y[j]) * A.inv2a;
                        const double tt = __builtin_fma(dx, dx, dy * dy);
                        const bool on = tt > 0.0;
                        const auto v = NearT::charge(S.a[j], on ? tt : 1.0, s_log);
                        near_q += on ? v : 0;
                    };
#pragma unroll 1
                    for (int jj = 0; jj < nfull; jj += g) pair(jj + sub);
                    if (nfull + sub < cn) pair(nfull + sub);
                } else {
                    auto pair = [&](int j) {
                        const double dx = (xs - S.x[j]) * A.inv2a, dy = (ys - S.y[j]) * A.inv2a;
                        const double tt = __builtin_fma(dx, dx, dy * dy);
                        const bool on = tt > 0.0;
                        const auto v =
                            NearT::dipole(__builtin_fma(dx, S.a[j], dy * S.b[j]), on ? tt : 1.0, s_log);
                        near_d += on ? v : 0;
                    };
#pragma unroll 1
                    for (int jj = 0; jj < nfull; jj += g) pair(jj + sub);
                    if (nfull + sub < cn) pair(nfull + sub);
                }
            }
        }
    }
    sync();
    S.x[lane] = valid ? (double)near_q + A.dip_scale * (double)near_d : 0.0;
    sync();
    if (sub == 0) {
        double tot = 0.0;
        for (int gi = 0; gi < g; ++gi) tot += S.x[ti + gi * c];
        A.outs[t] = tot * kInv2Pi;
    }
}

template <int NT, bool kSmallOnly, bool kF32 = false, bool kCall = true>
__global__ __launch_bounds__(64) void k_leaf(LeafArgs A) {
    __shared__ LeafLds S;
    __shared__ double2 s_log[YK_LOG_TAB];
    if constexpr (!kF32)
        for (int i = threadIdx.x; i < YK_LOG_TAB; i += 64)
            s_log[i] = make_double2(yk_log_tab[2 * i], yk_log_tab[2 * i + 1]);
    leaf_item<NT, kSmallOnly, kF32, kCall>(A.items[xcd_remap(blockIdx.x, gridDim.x)], A, S, s_log, [] { __syncthreads(); });
}

// The adaptive tree's items in one launch: the items are ordered by the series
// their pair distances need (kLeafKinds, the slowest first), four to a
// workgroup, which share the table of logarithms.  One launch per class of
// leaves (level, coarser neighbour) left the GPU to the last wavefronts of each
// of some 16 classes, several of them of a few dozen leaves: on 1.5 M clustered
// points 1,288 us, this launch 619 (of that, 173 registers at two wavefronts
// per SIMD instead of five would cost 450).
struct LeafKinds {
    int block[kLeafKinds + 1];   // first workgroup of each kind (a multiple of 8: every XCD takes part in each)
    int item[kLeafKinds + 1];    // first item
};
struct WaveSync {
    __device__ __forceinline__ void operator()() const {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
};
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_leaf_kinds(LeafArgs A, LeafKinds K) {
    __shared__ LeafLds S[4];
    __shared__ double2 s_log[YK_LOG_TAB];
    for (int i = threadIdx.x; i < YK_LOG_TAB; i += 256)
        s_log[i] = make_double2(yk_log_tab[2 * i], yk_log_tab[2 * i + 1]);
    __syncthreads();   // (the wavefronts are independent from here on)
    int k = 0;
    while (k < kLeafKinds - 1 && (int)blockIdx.x >= K.block[k + 1]) ++k;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int it = K.item[k] + 4 * xcd_remap(blockIdx.x - K.block[k], K.block[k + 1] - K.block[k]) + w;
    if (it >= K.item[k + 1]) return;
    const int2 item = A.items[it];
    switch (k) {
    case 0: leaf_item<14, false, false>(item, A, S[w], s_log, WaveSync()); break;
    case 1: leaf_item<14, true, false>(item, A, S[w], s_log, WaveSync()); break;
    case 2: leaf_item<10, true, false>(item, A, S[w], s_log, WaveSync()); break;
    case 3: leaf_item<8, true, false>(item, A, S[w], s_log, WaveSync()); break;
    case 4: leaf_item<6, true, false>(item, A, S[w], s_log, WaveSync()); break;
    default: leaf_item<5, true, false>(item, A, S[w], s_log, WaveSync()); break;
    }
}

// ------------------------------------------------- cached near field ---
// The near-field values depend on the points and alpha only, so a tree can
// keep them: k_near_build writes them once per target set, k_near_apply then
// forms the sums from them (an HBM-bound pass instead of Bessel series).
// Both walk the items exactly as k_leaf does; entries are source-major and
// target-minor per item, so a wavefront's loads are contiguous.
struct ItemSetup {
    int c, g, ti, sub, t, nq, nd;
    bool valid;
};

// Leaf ranges and U-list source ranges of an item (into the LDS arrays qa, qn,
// da, dn_, one entry per neighbour), and this lane's target.  q_on / d_on
// select which source sets are counted; NTB threads share the item.
template <int NTB = 64>
__device__ __forceinline__ ItemSetup item_setup(int2 item, const int32_t *__restrict__ lrange,
                                                const int32_t *__restrict__ uoff,
                                                const int32_t *__restrict__ ulist, int q_on, int d_on,
                                                int mask, int *qa, int *qn, int *da, int *dn_) {
    const int li = item.x, lane = threadIdx.x;
    int rs[3], re[3], ntot = 0;
    for (int s = 0; s < 3; ++s) {
        rs[s] = lrange[li * 6 + 2 * s];
        re[s] = (mask >> s) & 1 ? lrange[li * 6 + 2 * s + 1] : rs[s];
        ntot += re[s] - rs[s];
    }
    const int u0 = uoff[li], nu = uoff[li + 1] - u0;
    if (lane < 9) {
        const int u = lane;
        int a = 0, an = 0, b2 = 0, bn = 0;
        if (u < nu) {
            const int ul = ulist[u0 + u];
            a = lrange[ul * 6];
            an = q_on ? lrange[ul * 6 + 1] - a : 0;
            b2 = lrange[ul * 6 + 2];
            bn = d_on ? lrange[ul * 6 + 3] - b2 : 0;
        }
        qa[u] = a; qn[u] = an; da[u] = b2; dn_[u] = bn;
    }
    __syncthreads();
    ItemSetup r;
    r.nq = 0;
    r.nd = 0;
    for (int u = 0; u < 9; ++u) {
        r.nq += qn[u];
        r.nd += dn_[u];
    }
    r.c = min(64, ntot - item.y);
    r.g = NTB / r.c;
    r.ti = lane % r.c;
    r.sub = lane / r.c;
    r.valid = r.sub < r.g;
    int k = item.y + r.ti;
    r.t = -1;
    for (int s = 0; s < 3; ++s) {
        const int n = re[s] - rs[s];
        if (r.t < 0 && k < n) r.t = rs[s] + k;
        k -= n;
    }
    return r;
}

// sorted index of flat U-list source f of a set (counts cnt, starts st)
__device__ __forceinline__ int flat_source(int f, const int *cnt, const int *st) {
    int u = 0;
    while (u < 8 && f >= cnt[u]) { f -= cnt[u]; ++u; }
    return st[u] + f;
}

template <int NT, bool kSmallOnly, bool kF32>
__global__ __launch_bounds__(64) void k_near_build(
    const int2 *__restrict__ items, const int32_t *__restrict__ lrange,
    const int32_t *__restrict__ uoff, const int32_t *__restrict__ ulist,
    const double *__restrict__ px, const double *__restrict__ py, int q_on, int d_on, int mask,
    double inv2a, const int64_t *__restrict__ qoff, const int64_t *__restrict__ doff,
    typename std::conditional<kF32, float, double>::type *__restrict__ Mq,
    typename std::conditional<kF32, float, double>::type *__restrict__ Md) {
    using VT = typename std::conditional<kF32, float, double>::type;
    __shared__ double s_x[kLeafStage], s_y[kLeafStage];
    __shared__ double2 s_log[YK_LOG_TAB];
    __shared__ int qa[9], qn[9], da[9], dn_[9];
    const int ib = xcd_remap(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x;
    if constexpr (!kF32)
        for (int i = lane; i < YK_LOG_TAB; i += 64) s_log[i] = make_double2(yk_log_tab[2 * i], yk_log_tab[2 * i + 1]);
    const ItemSetup it = item_setup(items[ib], lrange, uoff, ulist, q_on, d_on, mask, qa, qn, da, dn_);
    const double xs = px[it.t], ys = py[it.t];   // unscaled: see k_leaf
    for (int set = 0; set < 2; ++set) {
        const int ntot_s = set == 0 ? it.nq : it.nd;
        VT *Mb = set == 0 ? Mq + qoff[ib] : Md + 2 * doff[ib];
        for (int c0 = 0; c0 < ntot_s; c0 += kLeafStage) {
            const int cn = min(kLeafStage, ntot_s - c0);
            __syncthreads();
            for (int f = lane; f < cn; f += 64) {
                const int j = flat_source(c0 + f, set == 0 ? qn : dn_, set == 0 ? qa : da);
                s_x[f] = px[j];
                s_y[f] = py[j];
            }
            __syncthreads();
            if (!it.valid) continue;
            for (int j = it.sub; j < cn; j += it.g) {
                const double dx = (xs - s_x[j]) * inv2a, dy = (ys - s_y[j]) * inv2a;
                const double tt = __builtin_fma(dx, dx, dy * dy);
                const int64_t e = (int64_t)(c0 + j) * it.c + it.ti;
                if (set == 0) {
                    double v = 0.0;
                    if (tt > 0.0) {
                        if constexpr (kF32) v = (double)near_k0_f<kSmallOnly>((float)tt);
                        else v = near_k0<NT, kSmallOnly>(tt, s_log);
                    }
                    Mb[e] = (VT)v;
                } else {
                    double k = 0.0;
                    if (tt > 0.0) {
                        if constexpr (kF32) k = (double)near_k1oz4_f<kSmallOnly>((float)tt);
                        else k = near_k1oz4<NT, kSmallOnly>(tt, s_log);
                    }
                    Mb[2 * e] = (VT)(dx * k);
                    Mb[2 * e + 1] = (VT)(dy * k);
                }
            }
        }
    }
}

// NTB = 64, or 256 for trees with too few items to fill the GPU (the layout
// of the values does not depend on how many lanes share a target)
// sources per lane whose values are in flight together: an item of a densely
// sampled curve (58 targets, 130 dipoles) is one wavefront's chain of such
// batches (200,003 points: 176 us with 8 charges or 4 dipoles and two loads per
// dipole, 144 us with 16 and 8; the symmetric kernel, whose registers five
// wavefronts per SIMD share, takes 8 of either: 223 us with 16, 211 with 8)
constexpr int kNearBatch = 16;

// batch(N, full, j0) over cn sources, gs at a time: sources j0, j0 + gs, ...,
// j0 + (N-1) gs of each lane group, all in range or (the last batch) masked
template <int NB, typename Batch>
__device__ __forceinline__ void source_batches(int cn, int gs, Batch batch) {
    int j0 = 0;
    for (; j0 + NB * gs <= cn; j0 += NB * gs) batch(std::integral_constant<int, NB>(), std::true_type(), j0);
    const int r = cn - j0;
    if (r <= 0) return;
    if (NB > 8 && r > 8 * gs) batch(std::integral_constant<int, NB>(), std::false_type(), j0);
    else if (r > 4 * gs) batch(std::integral_constant<int, 8>(), std::false_type(), j0);
    else if (r > 2 * gs) batch(std::integral_constant<int, 4>(), std::false_type(), j0);
    else batch(std::integral_constant<int, 2>(), std::false_type(), j0);
}

// Values of an item's block, streamed past the caches or through them.  The line
// lies where an item has one wavefront (2,048 items): fewer items' values stay in
// cache between the passes of a solve (28,672 nodes, P2M and near field 26 us
// streaming, 21 not; 1,536 nodes 18 and 13), those of large trees are read from
// memory once per pass (200,003 points, 739 MB: the near field 132 us, 149
// otherwise; 400,000, 724 MB: 125 and 150; 120,000, 281 MB: 65 and 70).  What
// decides is the values' size against the 256 MB of the last cache, so that
// trees of 2,048 items and more with less than that lose by the rule: 70,000
// points, 69 MB 40 and 32 us (the pass 107 and 105), 106 MB 34 and 27 (109 and
// 107); 110,000 nodes, 120 MB 35 and 28 (222 and 215); 200,000 nodes, 197 MB 45
// and 41 (330 both).
template <bool kStream, typename T> __device__ __forceinline__ T near_value(const char *p) {
    if constexpr (kStream) return __builtin_nontemporal_load(reinterpret_cast<const T *>(p));
    else return *reinterpret_cast<const T *>(p);
}
// acc plus lane group sub's share (of g) of the sums of target t's values
// against cn staged charges a (dipoles a, b): blk the values' block from the
// first of them, c targets per source.  One 32-bit offset per load; the last
// batch is masked, not cut into smaller ones whose round trips would add up.
template <int NB, bool kStream, typename VT>
__device__ __forceinline__ double chg_rows(const VT *blk, int c, int g, int t, int sub, int cn, const double *a,
                                           double acc) {
    c = __builtin_amdgcn_readfirstlane(c);
    g = __builtin_amdgcn_readfirstlane(g);
    const char *base = reinterpret_cast<const char *>(blk);
    source_batches<NB>(cn, g, [&](auto N, auto full, int j0) {
        VT m[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int j = j0 + u * g + sub;
            m[u] = near_value<kStream, VT>(base + (full || j < cn ? (uint32_t)(t + j * c) : 0u) * (uint32_t)sizeof(VT));
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int j = j0 + u * g + sub;
            acc = __builtin_fma((double)m[u], full || j < cn ? a[j] : 0.0, acc);
        }
    });
    return acc;
}
template <int NB, bool kStream, typename VT>
__device__ __forceinline__ double dip_rows(const VT *blk, int c, int g, int t, int sub, int cn, const double *a,
                                           const double *b, double acc) {
    using Pair = typename Pair2<VT>::type;
    c = __builtin_amdgcn_readfirstlane(c);
    g = __builtin_amdgcn_readfirstlane(g);
    const char *base = reinterpret_cast<const char *>(blk);
    source_batches<NB>(cn, g, [&](auto N, auto full, int j0) {
        Pair m[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int j = j0 + u * g + sub;
            m[u] =
                near_value<kStream, Pair>(base + (full || j < cn ? (uint32_t)(t + j * c) : 0u) * (uint32_t)sizeof(Pair));
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int j = j0 + u * g + sub;
            const bool on = full || j < cn;
            acc = __builtin_fma((double)m[u].x, on ? a[j] : 0.0, __builtin_fma((double)m[u].y, on ? b[j] : 0.0, acc));
        }
    });
    return acc;
}

// the pass's side of a cached near field (both layouts)
template <typename VT>
struct NearPass {
    Strengths st;
    int64_t off1;
    int has_q, has_d;
    const int64_t *qoff, *doff;
    const VT *Mq, *Md;
    double dip_scale;
    double *outs;
};
// both orders of every charge pair stored
struct NearFull {
    const int2 *items;
    const int32_t *lrange, *uoff, *ulist;
    int q_on, d_on, mask;
};
template <typename VT, int NTB>
__device__ __forceinline__ void near_apply(int ib, const NearFull &nf, const NearPass<VT> &np, double *lds) {
    double *s_a = lds, *s_b = s_a + (NTB > kLeafStage ? NTB : kLeafStage);
    __shared__ int qa[9], qn[9], da[9], dn_[9];
    const int2 *__restrict__ items = nf.items;
    const int32_t *__restrict__ lrange = nf.lrange, *__restrict__ uoff = nf.uoff, *__restrict__ ulist = nf.ulist;
    const int q_on = nf.q_on, d_on = nf.d_on, mask = nf.mask, has_q = np.has_q, has_d = np.has_d;
    const int64_t off1 = np.off1;
    const int64_t *__restrict__ qoff = np.qoff, *__restrict__ doff = np.doff;
    const VT *__restrict__ Mq = np.Mq, *__restrict__ Md = np.Md;
    const double dip_scale = np.dip_scale;
    double *__restrict__ outs = np.outs;
    const int lane = threadIdx.x;
    const ItemSetup it = item_setup<NTB>(items[ib], lrange, uoff, ulist, q_on, d_on, mask, qa, qn, da, dn_);
    double near_q = 0.0, near_d = 0.0;
    for (int set = 0; set < 2; ++set) {
        if ((set == 0 && !has_q) || (set == 1 && !has_d)) continue;
        const int ntot_s = set == 0 ? it.nq : it.nd;
        for (int c0 = 0; c0 < ntot_s; c0 += kLeafStage) {
            const int cn = min(kLeafStage, ntot_s - c0);
            __syncthreads();
            for (int f = lane; f < cn; f += NTB) {
                const int j = flat_source(c0 + f, set == 0 ? qn : dn_, set == 0 ? qa : da);
                if (set == 0) {
                    s_a[f] = np.st.charge(j);
                } else {
                    const double2 d = np.st.dipole(j, off1);
                    s_a[f] = d.x;
                    s_b[f] = d.y;
                }
            }
            __syncthreads();
            if (!it.valid) continue;
            if (set == 0)
                near_q = chg_rows<kNearBatch, NTB == 64>(Mq + qoff[ib] + (int64_t)c0 * it.c, it.c, it.g, it.ti, it.sub,
                                                         cn, s_a, near_q);
            else
                near_d = dip_rows<kNearBatch / 2, NTB == 64>(Md + 2 * (doff[ib] + (int64_t)c0 * it.c), it.c, it.g,
                                                             it.ti, it.sub, cn, s_a, s_b, near_d);
        }
    }
    __syncthreads();
    s_a[lane] = it.valid ? near_q + dip_scale * near_d : 0.0;
    __syncthreads();
    if (it.sub == 0) {
        double tot = 0.0;
        for (int gi = 0; gi < it.g; ++gi) tot += s_a[it.ti + gi * it.c];
        outs[it.t] = tot * kInv2Pi;
    }
}

template <int NTB> constexpr int kNearFullLds = (NTB > kLeafStage ? NTB : kLeafStage) + kLeafStage;
template <typename VT, int NTB>
__global__ __launch_bounds__(NTB) void k_near_apply(NearFull nf, NearPass<VT> np) {
    __shared__ double lds[kNearFullLds<NTB>];
    near_apply<VT, NTB>(xcd_remap(blockIdx.x, gridDim.x), nf, np, lds);
}

// ---------------------------------------------------- symmetric near field --
// The charge-to-charge values K0(|x - y|/alpha) are symmetric in the two
// points.  When no leaf holds more than 64 charges (and the charges are among
// the targets), the block of each unordered pair of neighbouring leaves {A, B}
// is stored once, with the leaf of smaller index
// (its owner), and the owner's item applies it both ways: to its own charges
// (a sum over B's charges) and, transposed, to B's charges (a sum over its
// own), the latter written to B's incoming slot, which k_l2p adds.  A leaf's
// own block is stored whole.  A leaf's charges lead its targets, so they all
// fall in its first item.  Per item (starting at a
// multiple of four entries) the charge values are, source major and target
// minor: (1) the item's charges as targets against the charges of the owned
// neighbours (the leaf itself and those of larger index, in U-list order),
// each source's row padded with zeros to a multiple of four targets, (2) its
// other targets against the charges of all neighbours.  The dipole values keep
// the layout of k_near_build.
//
// owned charge count of each U-list entry (lanes < 9; published by the
// barrier in item_setup)
__device__ __forceinline__ void owned_counts(int li, const int32_t *__restrict__ lrange,
                                             const int32_t *__restrict__ uoff, const int32_t *__restrict__ ulist,
                                             int *qo) {
    const int lane = threadIdx.x;
    if (lane < 9) {
        const int u0 = uoff[li], nu = uoff[li + 1] - u0;
        int o = 0;
        if (lane < nu) {
            const int ul = ulist[u0 + lane];
            if (ul >= li) o = lrange[ul * 6 + 1] - lrange[ul * 6];
        }
        qo[lane] = o;
    }
}

// sorted index of the k-th target of a leaf (sets in order, those of the mask)
__device__ __forceinline__ int item_target(int li, int k, const int32_t *__restrict__ lrange, int mask) {
    for (int s = 0; s < 3; ++s) {
        const int rs = lrange[li * 6 + 2 * s], n = (mask >> s) & 1 ? lrange[li * 6 + 2 * s + 1] - rs : 0;
        if (k < n) return rs + k;
        k -= n;
    }
    return -1;
}

template <int NT, bool kSmallOnly, bool kF32>
__global__ __launch_bounds__(64) void k_near_build_sym(
    const int2 *__restrict__ items, const int32_t *__restrict__ lrange, const int32_t *__restrict__ uoff,
    const int32_t *__restrict__ ulist, const double *__restrict__ px, const double *__restrict__ py, int mask,
    double inv2a, const int64_t *__restrict__ qoff,
    typename std::conditional<kF32, float, double>::type *__restrict__ Mq) {
    using VT = typename std::conditional<kF32, float, double>::type;
    __shared__ double2 s_log[YK_LOG_TAB];
    __shared__ int qa[9], qn[9], da[9], dn_[9], qo[9];
    const int ib = xcd_remap(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x;
    if constexpr (!kF32)
        for (int i = lane; i < YK_LOG_TAB; i += 64) s_log[i] = make_double2(yk_log_tab[2 * i], yk_log_tab[2 * i + 1]);
    const int2 item = items[ib];
    const int li = item.x;
    owned_counts(li, lrange, uoff, ulist, qo);
    const ItemSetup it = item_setup(item, lrange, uoff, ulist, 1, 0, mask, qa, qn, da, dn_);
    int nown = 0;
    for (int u = 0; u < 9; ++u) nown += qo[u];
    // (the mask has the charges; they lead a leaf's targets, all in its first item)
    const int rs0 = lrange[li * 6], nA0 = item.y == 0 ? lrange[li * 6 + 1] - rs0 : 0;
    const int cB = it.c - nA0;
    auto value = [&](int t, int j) -> VT {
        const double dx = (px[t] - px[j]) * inv2a, dy = (py[t] - py[j]) * inv2a;
        const double tt = __builtin_fma(dx, dx, dy * dy);
        double v = 0.0;
        if (tt > 0.0) {
            if constexpr (kF32) v = (double)near_k0_f<kSmallOnly>((float)tt);
            else v = near_k0<NT, kSmallOnly>(tt, s_log);
        }
        return (VT)v;
    };
    VT *M1 = Mq + qoff[ib];
    const int cA4 = (nA0 + 3) & ~3;
    const int64_t n1 = (int64_t)cA4 * nown;
    for (int64_t e = lane; e < n1; e += 64) {
        const int f = (int)(e / cA4), t = (int)(e % cA4);
        M1[e] = t < nA0 ? value(rs0 + t, flat_source(f, qo, qa)) : (VT)0;
    }
    VT *M2 = M1 + n1;
    const int64_t n2 = (int64_t)cB * it.nq;
    for (int64_t e = lane; e < n2; e += 64) {
        const int f = (int)(e / cB), k = (int)(e % cB);
        M2[e] = value(item_target(li, item.y + nA0 + k, lrange, mask), flat_source(f, qn, qa));
    }
}

// Per-item descriptor of the symmetric near field (built with the plan): for
// the nine U-list entries the first charge, the charge count, the owned charge
// count, the first dipole and the dipole count (entries 0-44), the item's
// target ranges per set, empty for sets outside the mask (45-47 first, 48-50
// end), its first target (51); and per entry the incoming slot it writes.
constexpr int kItemDesc = 52;

template <int NTB>
__device__ __forceinline__ ItemSetup setup_from_desc(const int *d) {
    const int lane = threadIdx.x;
    ItemSetup r;
    r.nq = 0;
    r.nd = 0;
    for (int u = 0; u < 9; ++u) {
        r.nq += d[9 + u];
        r.nd += d[36 + u];
    }
    int ntot = 0;
    for (int s = 0; s < 3; ++s) ntot += d[48 + s] - d[45 + s];
    const int y = d[51];
    r.c = min(64, ntot - y);
    r.g = NTB / r.c;
    r.ti = lane % r.c;
    r.sub = lane / r.c;
    r.valid = r.sub < r.g;
    int k = y + r.ti;
    r.t = -1;
    for (int s = 0; s < 3; ++s) {
        const int n = d[48 + s] - d[45 + s];
        if (r.t < 0 && k < n) r.t = d[45 + s] + k;
        k -= n;
    }
    return r;
}

// Sources per lane and batch in the owned charge block (each lane has this
// many quarter rows of four values in flight).
constexpr int kSymRounds = 4;

// four consecutive values (16-byte aligned for float, 32 for double), read once
// (double: the two halves of a 32-byte piece are two loads, which the first
// level cache serves with one request when they are not marked streaming:
// 199 -> 183 us over 2^20 uniform points)
__device__ __forceinline__ void load4(const double *p, double (&o)[4]) {
    const yk_dpair a = *reinterpret_cast<const yk_dpair *>(p);
    const yk_dpair b = *(reinterpret_cast<const yk_dpair *>(p) + 1);
    o[0] = a.x;
    o[1] = a.y;
    o[2] = b.x;
    o[3] = b.y;
}
__device__ __forceinline__ void load4(const float *p, double (&o)[4]) {
    const yk_f4 a = __builtin_nontemporal_load(reinterpret_cast<const yk_f4 *>(p));
    o[0] = a.x;
    o[1] = a.y;
    o[2] = a.z;
    o[3] = a.w;
}

// each charge pair stored once
struct NearSym {
    const int32_t *desc;
    const int64_t *desc_dst;
    double *inc;
};
template <int NTB> constexpr int kNearSymLds = (NTB > kLeafStage ? NTB : kLeafStage) + kLeafStage + 64 + 4 * NTB;
template <typename VT, int NTB>
__device__ __forceinline__ void near_apply_sym(int ib, const NearSym &ns, const NearPass<VT> &np, double *lds) {
    double *s_a = lds, *s_b = s_a + (NTB > kLeafStage ? NTB : kLeafStage);
    double *s_res = s_b + kLeafStage, *s_p = s_res + 64;   // s_p: direct sums of part (1), four targets per lane
    __shared__ int s_d[kItemDesc], s_pre[9];
    __shared__ int64_t s_dst[9];
    const int32_t *__restrict__ desc = ns.desc;
    const int64_t *__restrict__ desc_dst = ns.desc_dst, *__restrict__ qoff = np.qoff, *__restrict__ doff = np.doff;
    const VT *__restrict__ Mq = np.Mq, *__restrict__ Md = np.Md;
    const int has_q = np.has_q, has_d = np.has_d;
    const int64_t off1 = np.off1;
    const double dip_scale = np.dip_scale;
    double *__restrict__ outs = np.outs, *__restrict__ inc = ns.inc;
    const int lane = threadIdx.x;
    // the item's descriptor: one round trip instead of the chain leaf -> U list -> ranges
    if (lane < kItemDesc) s_d[lane] = desc[(int64_t)ib * kItemDesc + lane];
    if (lane < 9) s_dst[lane] = desc_dst[(int64_t)ib * 9 + lane];
    if (lane < 64) s_res[lane] = 0.0;
    __syncthreads();
    const int *qa = s_d, *qn = s_d + 9, *qo = s_d + 18, *da = s_d + 27, *dn_ = s_d + 36;
    const ItemSetup it = setup_from_desc<NTB>(s_d);
    // first owned source of each U-list entry (published by part (1)'s barriers)
    if (lane < 9) {
        int a = 0;
        for (int u = 0; u < lane; ++u) a += qo[u];
        s_pre[lane] = a;
    }
    const int c = it.c;
    // the leaf's charges (at most 64) lead its targets, all in its first item
    const int rs0 = s_d[45], nA0 = s_d[51] == 0 ? s_d[48] - rs0 : 0;
    int nown = 0;
    for (int u = 0; u < 9; ++u) nown += qo[u];
    // (1) the item's charges against the owned charges, both ways.  A lane
    // takes four consecutive targets (one quarter row) of four sources per
    // batch, read as vectors; it sums the direct products over its sources in
    // registers for the whole block and the transposed ones over its targets,
    // then over the tb lanes that share the sources (shuffles within a
    // wavefront: the lanes of a source never straddle one).
    if (has_q && nA0 > 0) {
        const int cA = nA0, cA4 = (cA + 3) & ~3, tb = cA4 >> 2;
        const int nf = 64 / tb, nfb = (NTB / 64) * nf;
        const int wl = lane & 63, lt = wl % tb;
        const int fs = (lane >> 6) * nf + wl / tb;
        const bool vA = wl / tb < nf;
        double qa4[4], y4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = 4 * lt + i;
            qa4[i] = (vA && t < cA) ? np.st.charge(rs0 + t) : 0.0;
            y4[i] = 0.0;
        }
        const VT *Mb = Mq + qoff[ib] + 4 * lt;
        for (int c0 = 0; c0 < nown; c0 += kLeafStage) {
            const int cn = min(kLeafStage, nown - c0);
            double w[kSymRounds][4];
            // rounds of a batch that hold sources (the same for all lanes)
            int nr = 0;
            auto load_batch = [&](int r0) {
                nr = min(kSymRounds, (cn - r0 + nfb - 1) / nfb);
#pragma unroll
                for (int j = 0; j < kSymRounds; ++j) {
                    const int f = r0 + j * nfb + fs;
                    if (j < nr && vA && f < cn) {
                        load4(Mb + (int64_t)(c0 + f) * cA4, w[j]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) w[j][i] = 0.0;
                    }
                }
            };
            // the first batch is in flight while the sources' charges are staged
            load_batch(0);
            __syncthreads();
            for (int f = lane; f < cn; f += NTB) s_a[f] = np.st.charge(flat_source(c0 + f, qo, qa));
            __syncthreads();
            for (int r0 = 0; r0 < cn; r0 += kSymRounds * nfb) {
                if (r0 > 0) load_batch(r0);
                double z[kSymRounds];
#pragma unroll
                for (int j = 0; j < kSymRounds; ++j) {
                    z[j] = 0.0;
                    if (j >= nr) continue;
                    const int f = r0 + j * nfb + fs;
                    const double qb = (vA && f < cn) ? s_a[f] : 0.0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        y4[i] = __builtin_fma(w[j][i], qb, y4[i]);
                        z[j] = __builtin_fma(w[j][i], qa4[i], z[j]);
                    }
                }
                for (int k = 1; k < tb; k <<= 1) {
                    const bool in = lt + k < tb;
#pragma unroll
                    for (int j = 0; j < kSymRounds; ++j) {
                        if (j >= nr) continue;
                        const double o = __shfl_down(z[j], k, 64);
                        z[j] += in ? o : 0.0;
                    }
                }
                if (vA && lt == 0) {
#pragma unroll
                    for (int j = 0; j < kSymRounds; ++j) {
                        const int f = r0 + j * nfb + fs;
                        if (f >= cn) break;
                        // the U-list entry of owned source c0 + f: the last one
                        // starting at or before it (empty entries share the
                        // next one's start)
                        const int ff = c0 + f;
                        int u = 0;
#pragma unroll
                        for (int k = 1; k < 9; ++k) u += ff >= s_pre[k] ? 1 : 0;
                        const int64_t d = s_dst[u];
                        if (d >= 0) inc[d + ff - s_pre[u]] = z[j] * kInv2Pi;
                    }
                }
            }
        }
        // the direct sums over the source slots: lane (slot, lt) holds targets 4 lt .. 4 lt + 3
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) s_p[4 * lane + i] = vA ? y4[i] : 0.0;
        __syncthreads();
        if (lane < cA) {
            double tot = 0.0;
            for (int q = 0; q < nfb; ++q) {
                const int ln = (q / nf) * 64 + (q % nf) * tb + (lane >> 2);
                tot += s_p[4 * ln + (lane & 3)];
            }
            s_res[lane] += tot;
        }
    }
    // (2) the item's other targets against all neighbouring charges
    const int cB = c - nA0;
    if (has_q && cB > 0 && it.nq > 0) {
        const int gB = NTB / cB, tiB = lane % cB, subB = lane / cB;
        const bool vB = subB < gB;
        const VT *Mb = Mq + qoff[ib] + (int64_t)((nA0 + 3) & ~3) * nown;
        double acc = 0.0;
        for (int c0 = 0; c0 < it.nq; c0 += kLeafStage) {
            const int cn = min(kLeafStage, it.nq - c0);
            __syncthreads();
            for (int f = lane; f < cn; f += NTB) s_a[f] = np.st.charge(flat_source(c0 + f, qn, qa));
            __syncthreads();
            if (!vB) continue;
            acc = chg_rows<8, NTB == 64>(Mb + (int64_t)c0 * cB, cB, gB, tiB, subB, cn, s_a, acc);
        }
        __syncthreads();
        s_a[lane] = vB ? acc : 0.0;
        __syncthreads();
        if (lane < cB) {
            double tot = 0.0;
            for (int s = 0; s < gB; ++s) tot += s_a[s * cB + lane];
            s_res[nA0 + lane] += tot;
        }
    }
    // (3) every target against the dipoles (layout of k_near_build)
    if (has_d && it.nd > 0) {
        double acc = 0.0;
        for (int c0 = 0; c0 < it.nd; c0 += kLeafStage) {
            const int cn = min(kLeafStage, it.nd - c0);
            __syncthreads();
            for (int f = lane; f < cn; f += NTB) {
                const double2 d = np.st.dipole(flat_source(c0 + f, dn_, da), off1);
                s_a[f] = d.x;
                s_b[f] = d.y;
            }
            __syncthreads();
            if (!it.valid) continue;
            acc = dip_rows<8, NTB == 64>(Md + 2 * (doff[ib] + (int64_t)c0 * c), c, it.g, it.ti, it.sub, cn, s_a, s_b,
                                         acc);
        }
        __syncthreads();
        s_a[lane] = it.valid ? acc : 0.0;
        __syncthreads();
        if (lane < c) {
            double tot = 0.0;
            for (int s = 0; s < it.g; ++s) tot += s_a[s * c + lane];
            s_res[lane] += dip_scale * tot;
        }
    }
    __syncthreads();
    if (lane < c) outs[it.t] = s_res[lane] * kInv2Pi;
}

template <typename VT, int NTB>
__global__ __launch_bounds__(NTB) __attribute__((amdgpu_waves_per_eu(5))) void k_near_apply_sym(NearSym ns,
                                                                                                NearPass<VT> np) {
    __shared__ double lds[kNearSymLds<NTB>];
    near_apply_sym<VT, NTB>(xcd_remap(blockIdx.x, gridDim.x), ns, np, lds);
}

// P2M (cached rows) and the cached near field of a small tree in one launch,
// the strengths read through the permutation: both need only them, the near
// field's items are the longer chains and go first, and the far field's
// launches that follow are too short to hide a second stream's events behind.
template <typename VT, bool SYM>
__global__ __launch_bounds__(256) void k_p2m_near(P2MApply pa, NearFull nf, NearSym ns, NearPass<VT> np, int nitems) {
    constexpr int kLds = kNearSymLds<256> > kP2MApplyLds ? kNearSymLds<256> : kP2MApplyLds;
    __shared__ double lds[kLds];
    if ((int)blockIdx.x < nitems) {   // (whole workgroups)
        if constexpr (SYM) near_apply_sym<VT, 256>(blockIdx.x, ns, np, lds);
        else near_apply<VT, 256>(blockIdx.x, nf, np, lds);
    } else {
        p2m_apply(blockIdx.x - nitems, pa, np.st, np.off1, np.has_q, np.has_d, lds);
    }
}

using NearBuild64 = void (*)(const int2 *, const int32_t *, const int32_t *, const int32_t *,
                             const double *, const double *, int, int, int, double, const int64_t *,
                             const int64_t *, double *, double *);
using NearBuild32 = void (*)(const int2 *, const int32_t *, const int32_t *, const int32_t *,
                             const double *, const double *, int, int, int, double, const int64_t *,
                             const int64_t *, float *, float *);

NearBuild64 pick_near_build64(int nt, bool small_only) {
    if (small_only) {
        if (nt <= 5) return k_near_build<5, true, false>;
        if (nt <= 6) return k_near_build<6, true, false>;
        if (nt <= 8) return k_near_build<8, true, false>;
        if (nt <= 10) return k_near_build<10, true, false>;
        return k_near_build<14, true, false>;
    }
    return k_near_build<14, false, false>;
}
NearBuild32 pick_near_build32(bool small_only) {
    return small_only ? k_near_build<8, true, true> : k_near_build<8, false, true>;
}
using NearBuildSym64 = void (*)(const int2 *, const int32_t *, const int32_t *, const int32_t *,
                                const double *, const double *, int, double, const int64_t *, double *);
using NearBuildSym32 = void (*)(const int2 *, const int32_t *, const int32_t *, const int32_t *,
                                const double *, const double *, int, double, const int64_t *, float *);
NearBuildSym64 pick_near_build_sym64(int nt, bool small_only) {
    if (small_only) {
        if (nt <= 5) return k_near_build_sym<5, true, false>;
        if (nt <= 6) return k_near_build_sym<6, true, false>;
        if (nt <= 8) return k_near_build_sym<8, true, false>;
        if (nt <= 10) return k_near_build_sym<10, true, false>;
        return k_near_build_sym<14, true, false>;
    }
    return k_near_build_sym<14, false, false>;
}
NearBuildSym32 pick_near_build_sym32(bool small_only) {
    return small_only ? k_near_build_sym<8, true, true> : k_near_build_sym<8, false, true>;
}

using LeafKernel = void (*)(LeafArgs);

// L2P reads its leaf's expansion once per point.  The points of a workgroup are
// consecutive in leaf order, so the leaves they span (at most kL2PRows, points
// of one set) are staged in LDS: all rows' loads are in flight together, and the
// series' loop waits on no memory.  Coefficient k lies at k + 1, so that the pair
// 2m - 1, 2m is one aligned read.
constexpr int kL2PRows = 32, kL2PStride = 66;
constexpr int kL2PLds = kL2PRows * kL2PStride;
template <typename RowOf>
__device__ __forceinline__ bool l2p_stage(double *s_rows, int64_t n, int64_t toff1, int64_t toff2,
                                          const int32_t *__restrict__ pleaf, int Pp, int32_t &first, RowOf row_of) {
    const int64_t t0 = (int64_t)blockIdx.x * 256, te = min(t0 + 256, n);
    first = pleaf[t0];
    const int rows = pleaf[te - 1] - first + 1;
    // (the points of one set are in leaf order; two sets' are not)
    const bool one_set = !(t0 < toff1 && toff1 < te) && !(t0 < toff2 && toff2 < te);
    if (!one_set || rows < 1 || rows > kL2PRows || Pp > 64) return false;   // (the whole workgroup)
    const int lane = threadIdx.x & 63;
    if (lane < Pp)
#pragma unroll 8
        for (int r = threadIdx.x >> 6; r < rows; r += 4) s_rows[r * kL2PStride + 1 + lane] = row_of(first + r)[lane];
    return true;
}
// What a point needs beside the series, all read before the rows are waited for
// (one after the other, these loads were most of the time of a small tree's
// pass).  Points beyond the end read the last one's.
struct L2PPoint {
    int64_t t;
    int set;
    int32_t leaf, dst;
    double x, y, near, bx, diag;
    bool on;
    __device__ __forceinline__ L2PPoint(int64_t n, int64_t toff1, int64_t toff2, int mask, const int32_t *pleaf,
                                        const double *px, const double *py, const double *outs, const int32_t *perm,
                                        const double *bw, const double *bk, const double *bxv, double inv_alpha2) {
        const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
        t = min(t0, n - 1);
        set = (t >= toff1) + (t >= toff2);
        on = t0 < n && ((mask >> set) & 1);
        leaf = pleaf[t];
        dst = perm[t];
        x = px[t];
        y = py[t];
        near = outs[t];
        bx = diag = 0.0;
        if (set == 1 && bxv) {
            bx = bxv[dst];
            diag = dl_diag_weight(bw[dst], bk[dst], inv_alpha2);
        }
    }
    // double-layer operator: x - 2 (DL + corrected diagonal)
    __device__ __forceinline__ void store(double v, bool op, double *out0, double *out1, double *out2) const {
        double *o = set == 0 ? out0 : set == 1 ? out1 : out2;
        o[dst] = set == 1 && op ? bx - 2.0 * (v + diag * bx) : v;
    }
};
// the series at scaled offset (wx, wy): Horner in z with G_m = F_m(y)/F_m(Y),
// F_m downwards; at(k) is coefficient k, 2 pi times the value returned
template <typename At>
__device__ __forceinline__ double l2p_series(double wx, double wy, double invR, const double *sc, int nser,
                                             const double *ify, const double *cnn, int p, At at) {
    const double yv = 0.25 * (wx * wx + wy * wy);
    const double zx = wx * invR, zy = wy * invR;
    double F1, F2;
    f_start(yv, sc, nser, F1, F2);
    double sr = 0.0, si = 0.0;
#pragma unroll 4
    for (int m = p; m >= 1; --m) {
        const double F0 = F1 + yv * F2 * cnn[m];
        const double gm = F0 * ify[m];
        const double cr = at(2 * m - 1) * gm, ci = at(2 * m) * gm;
        const double nr = sr * zx - si * zy + cr;
        si = sr * zy + si * zx + ci;
        sr = nr;
        F2 = F1;
        F1 = F0;
    }
    const double F0 = F1 + yv * F2 * cnn[0];
    return at(0) * F0 * ify[0] + 2.0 * (sr * zx - si * zy);
}

// L2P: one thread per target point, adding the local expansion of the
// point's leaf to the near-field sum already in outs.  The level's tables are staged in LDS.
__global__ __launch_bounds__(256) void k_l2p(
    int64_t n, int64_t toff1, int64_t toff2, int mask, const int32_t *__restrict__ pleaf,
    int64_t leaf_base, const double *__restrict__ bcx, const double *__restrict__ bcy,
    const double *__restrict__ px, const double *__restrict__ py, const double *__restrict__ Lc,
    double inv_alpha, double invR, const double *__restrict__ invFY, const double *__restrict__ cnn,
    const double *__restrict__ sc, int nser, int p, int Pp, const double *__restrict__ outs,
    const int32_t *__restrict__ perm, double *__restrict__ out0, double *__restrict__ out1,
    double *__restrict__ out2, const double *__restrict__ bw, const double *__restrict__ bk,
    const double *__restrict__ bx, const double *__restrict__ inc, const int64_t *__restrict__ inc_base,
    const int32_t *__restrict__ inc_cnt, const int32_t *__restrict__ lrange) {
    extern __shared__ double dyn[];
    __shared__ double s_rows[kL2PLds];
    double *t_cnn = dyn;               // [p+1]
    double *t_ify = t_cnn + p + 1;     // [p+1]
    double *t_sc = t_ify + p + 1;      // [2 nser]
    for (int i = threadIdx.x; i < p + 1; i += blockDim.x) {
        t_cnn[i] = cnn[i];
        t_ify[i] = invFY[i];
    }
    for (int i = threadIdx.x; i < 2 * nser; i += blockDim.x) t_sc[i] = sc[i];
    const L2PPoint pt(n, toff1, toff2, mask, pleaf, px, py, outs, perm, bw, bk, bx, inv_alpha * inv_alpha);
    const int32_t lb = pt.leaf;
    const int64_t b = leaf_base + lb;
    const double wx = (pt.x - bcx[b]) * inv_alpha, wy = (pt.y - bcy[b]) * inv_alpha;
    int32_t first = 0;
    const bool staged = l2p_stage(s_rows, n, toff1, toff2, pleaf, Pp, first,
                                  [&](int32_t leaf) { return Lc + (leaf_base + leaf) * Pp; });
    // the incoming slots of the symmetric near field (charge targets), of which
    // a leaf has one per neighbour that owns their pair block: eight at once
    constexpr int kIn = 8;
    double in[kIn];
    int32_t n_in = 0, n0 = 0;
    int64_t in_base = 0;
    if (pt.set == 0 && inc) {
        const int32_t s0 = lrange[lb * 6];
        n0 = lrange[lb * 6 + 1] - s0;
        in_base = inc_base[lb] + (pt.t - s0);
        n_in = inc_cnt[lb];
#pragma unroll
        for (int k = 0; k < kIn; ++k) in[k] = n_in > k ? inc[in_base + (int64_t)k * n0] : 0.0;
    }
    __syncthreads();
    if (!pt.on) return;
    double far;
    if (staged) {
        const double *Lb = s_rows + (lb - first) * kL2PStride + 1;
        far = l2p_series(wx, wy, invR, t_sc, nser, t_ify, t_cnn, p, [&](int k) { return Lb[k]; });
    } else {
        const double *Lb = Lc + b * Pp;
        far = l2p_series(wx, wy, invR, t_sc, nser, t_ify, t_cnn, p, [&](int k) { return Lb[k]; });
    }
    // near field + far field, written straight to the caller's array of the set
    double v = pt.near + far * kInv2Pi;
    if (n_in > 0) {
#pragma unroll
        for (int k = 0; k < kIn; ++k) v += in[k];
        for (int k = kIn; k < n_in; ++k) v += inc[in_base + (int64_t)k * n0];
    }
    pt.store(v, bx != nullptr, out0, out1, out2);
}

// ------------------------------------------------------- adaptive tree ---
// beyond this scaled distance K_0 < 1e-250: the pair is dropped (also keeps
// K_0 and the ratio K_1/K_0 away from underflow)
constexpr double kFarRho = 600.0;
// The products T_n = I_n(R_l) K_n(rho) of the W and X translations, from the
// level's table rI[l] = {I_0(R_l), r_n = I_n(R_l)/I_{n-1}(R_l)} and the upward
// recurrence of K (stable for K): with A_n = I_n K_{n-1} and B_n = I_n K_{n+1} =
// A_n + (2n/rho) T_n, T_{n+1} = r_{n+1} B_n and A_{n+1} = r_{n+1} T_n.  Every
// factor stays in range however small the box, all terms are positive, and no
// order divides (a division per order was two thirds of the arithmetic).

// {K_0, K_1}(z), called and not inlined: inlined into a loop over sources, the
// some hundred constants of its two branches are kept in registers across the
// loop (256 VGPRs, one wavefront per SIMD, scalar spills).  On 1.5 M clustered
// points k_ad_p2l took 341 us inlined, 113 with the call at four wavefronts per
// SIMD, k_ad_m2p 113 and 83.
__device__ __attribute__((noinline)) double2 k01_called(double z) {
    double2 r;
    k01(z, r.x, r.y);
    return r;
}

// W list (M2P): the multipole of every box of the leaf's W list evaluated at
// the leaf's targets, phi(x) = sum_n M_n F^K_n((x - c)/alpha) =
// M_0 K_0 + 2 sum_{n>=1} Re(M_n e^{in theta}) K_n, added to the near-field
// sums in outs.  One wavefront per leaf, a lane per target; each target sums
// its boxes in list order (deterministic, no atomics).
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_ad_m2p(
    const int32_t *__restrict__ wleaves, const int32_t *__restrict__ woff, const int32_t *__restrict__ wl,
    const int32_t *__restrict__ lrange, int mask, const int32_t *__restrict__ blevel,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ M, const double *__restrict__ rI, int p, int Pp,
    double inv_alpha, double *__restrict__ outs) {
    const int li = wleaves[blockIdx.x];
    const int w0 = woff[li], w1 = woff[li + 1];
    int rs[3], rn[3], ntot = 0;
    for (int st = 0; st < 3; ++st) {
        rs[st] = lrange[li * 6 + 2 * st];
        rn[st] = (mask >> st) & 1 ? lrange[li * 6 + 2 * st + 1] - rs[st] : 0;
        ntot += rn[st];
    }
    // a leaf with few targets (at most 16 or 32) splits its W list among 4 or
    // 2 lane groups, whose partial sums meet in a fixed shuffle order
    const int G = ntot <= 16 ? 4 : ntot <= 32 ? 2 : 1, T = 64 / G;
    const int g = threadIdx.x / T, kl = threadIdx.x - g * T;
    for (int kb = 0; kb < ntot; kb += T) {
        const int k = kb + kl;
        int t = -1;
        double acc = 0.0;
        if (k < ntot) {
            int r = k;
            for (int st = 0; st < 3; ++st) {
                if (t < 0 && r < rn[st]) t = rs[st] + r;
                r -= rn[st];
            }
            const double x = px[t], y = py[t];
            for (int w = w0 + g; w < w1; w += G) {
                const int32_t d = wl[w];
                const double *Md = M + (int64_t)d * Pp;
                const double *ri = rI + (int64_t)blevel[d] * (p + 3);
                const double wx = (x - bcx[d]) * inv_alpha, wy = (y - bcy[d]) * inv_alpha;
                const double rho = sqrt(wx * wx + wy * wy), ir = 1.0 / rho;
                if (rho > kFarRho) continue;          // below 1e-250 of the box's sources
                const double c = wx * ir, sn = wy * ir;
                const double2 k01v = k01_called(rho);
                double T = ri[0] * k01v.x, A = ri[0] * k01v.y;   // T_0; A_0 = I_0 K_1
                const double T0 = T;
                double sum = 0.0, m2 = 0.0;
                double er = 1.0, ei = 0.0;            // e^{i n theta}
#pragma unroll 4
                for (int n = 1; n <= p; ++n) {
                    const double B = A + m2 * ir * T;             // I_{n-1} K_n
                    A = ri[n] * T;
                    T = ri[n] * B;                                // T_n
                    m2 += 2.0;
                    const double nr = er * c - ei * sn;
                    ei = er * sn + ei * c;
                    er = nr;
                    sum += T * (Md[2 * n - 1] * er - Md[2 * n] * ei);
                }
                sum = Md[0] * T0 + 2.0 * sum;
                acc += sum;
            }
        }
        if (G == 4) acc += __shfl_xor(acc, 16, 64);
        if (G >= 2) acc += __shfl_xor(acc, 32, 64);
        if (t >= 0 && g == 0) outs[t] += acc * kInv2Pi;
    }
}

// Sums over a wavefront's sources, eight orders at a time: every lane writes
// its source's terms to LDS (row 2i the real, 2i + 1 the imaginary part of the
// chunk's order i), then lane (row l / 4, part l % 4) adds up every fourth entry
// of its row.  The row stride puts the 32 entries that half a wavefront reads
// in different banks.  Nine KB per wavefront leave the occupancy to the
// registers.
constexpr int kSumStride = 68;
constexpr int kSumLds = 16 * kSumStride;
struct OrderSums {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};   // chunk c: orders 8c .. 8c + 7 (p <= 31)
    __device__ __forceinline__ void add(const double *sh, int c) {
        const double *r = sh + (threadIdx.x >> 2) * kSumStride + (threadIdx.x & 3);
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
            s0 += r[4 * k];
            s1 += r[4 * k + 4];
        }
        s0 += s1;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += k == c ? s0 : 0.0;
    }
    // put(output, sum) for the outputs 0 .. 2p, each from one lane
    template <typename Put> __device__ __forceinline__ void store(int p, Put put) {
        const int row = threadIdx.x >> 2, im = row & 1;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double v = acc[c];
            v += dpp_d<0xB1>(v);    // quad_perm [1,0,3,2]
            v += dpp_d<0x4E>(v);    // quad_perm [2,3,0,1]
            const int n = 8 * c + (row >> 1);
            if ((threadIdx.x & 3) == 0 && n <= p && (n > 0 || !im)) put(n == 0 ? 0 : 2 * n - 1 + im, v);
        }
    }
};

// X list (P2L): the sources of every leaf of the box's X list into the box's
// local expansion (scaled, Lh_m = L_m I_m(R_l)).  By Graf's addition theorem a
// charge q at w = (y - c)/alpha contributes L_m = q K_m(|w|) e^{-i m theta};
// a dipole D = d (n_x + i n_y), the normal derivative at y of that,
// L_m = -(1/(2 alpha)) [conj(D) K_{|m-1|} e^{-i(m-1) theta} + D K_{m+1}
// e^{-i(m+1) theta}]; with a + i b = D e^{-i theta}/(2 alpha) and A, B as above
// that is -(A + B) a cos(m theta) - (B - A) b sin(m theta) and
// (A + B) a sin(m theta) - (B - A) b cos(m theta).
// One wavefront per box, a lane per source.  FP64 issue bounds it (the orders
// and K0, K1), so lanes are kept busy: the sources of up to 64 leaves form one
// run, which the lanes take 64 at a time (leaf by leaf, leaves of some 15
// points left three lanes of four idle).
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_ad_p2l(
    const int32_t *__restrict__ xbox, const int32_t *__restrict__ xoff, const int32_t *__restrict__ xl,
    const int32_t *__restrict__ lrange, int has_q, int has_d, const int32_t *__restrict__ blevel,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ qs, const double *__restrict__ dns, int64_t off1,
    const double *__restrict__ rI, int p, int Pp, double inv_alpha, double *__restrict__ Lc) {
    __shared__ double sh[kSumLds];
    __shared__ int s_end[64], s_beg[64];   // flat end of each leaf's sources; their first index less the flat begin
    const int lane = threadIdx.x;
    const int32_t d = xbox[blockIdx.x];
    const double *ri = rI + (int64_t)blevel[d] * (p + 3);
    const double cx = bcx[d], cy = bcy[d], h = 0.5 * inv_alpha;
    const int xe = xoff[blockIdx.x + 1];
    OrderSums sums;
    for (int x0 = xoff[blockIdx.x]; x0 < xe; x0 += 64) {
        for (int set = 0; set < 2; ++set) {
            if ((set == 0 && !has_q) || (set == 1 && !has_d)) continue;
            int a = 0, n = 0;
            if (x0 + lane < xe) {
                const int32_t c = xl[x0 + lane];
                a = lrange[c * 6 + 2 * set];
                n = lrange[c * 6 + 2 * set + 1] - a;
            }
            int end = n;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const int o = __shfl_up(end, m, 64);
                if (lane >= m) end += o;
            }
            const int tot = __shfl(end, 63, 64);
            __syncthreads();
            s_end[lane] = end;
            s_beg[lane] = a - (end - n);
            __syncthreads();
            for (int base = 0; base < tot; base += 64) {
                const int f = base + lane;
                int k = 0;   // the leaf of source f: the first whose end is beyond it
#pragma unroll
                for (int m = 32; m >= 1; m >>= 1)
                    if (s_end[k + m - 1] <= f) k += m;
                bool on = f < tot;
                const int j = on ? s_beg[k] + f : 0;
                double wx = 1.0, wy = 0.0;
                if (on) {
                    wx = (px[j] - cx) * inv_alpha;
                    wy = (py[j] - cy) * inv_alpha;
                }
                double rho = sqrt(wx * wx + wy * wy);
                if (rho > kFarRho) {
                    on = false;
                    rho = wx = 1.0;
                    wy = 0.0;
                }
                const double ir = 1.0 / rho;
                const double co = wx * ir, sn = wy * ir;
                const double2 k01v = k01_called(rho);
                double T = ri[0] * k01v.x, A = ri[0] * k01v.y;   // T_0; at order 0, A = B = I_0 K_1
                double m2 = 0.0, er = 1.0, ei = 0.0;               // 2m, e^{i m theta}
                auto orders = [&](auto emit) {
                    for (int c = 0; 8 * c <= p; ++c) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int m = 8 * c + i;
                            if (m > p) break;
                            const double ct = m2 * ir * T, B = A + ct;
                            emit(sh + 2 * i * kSumStride + lane, T, A + B, ct);
                            A = ri[m + 1] * T;
                            T = ri[m + 1] * B;
                            m2 += 2.0;
                            const double nr = er * co - ei * sn;
                            ei = er * sn + ei * co;
                            er = nr;
                        }
                        __syncthreads();
                        sums.add(sh, c);
                        __syncthreads();
                    }
                };
                if (set == 0) {
                    const double q = on ? qs[j] : 0.0;
                    orders([&](double *row, double t, double, double) {
                        const double qt = q * t;
                        row[0] = qt * er;
                        row[kSumStride] = -qt * ei;
                    });
                } else {
                    const double Dx = on ? h * dns[2 * (j - off1)] : 0.0, Dy = on ? h * dns[2 * (j - off1) + 1] : 0.0;
                    const double ra = Dx * co + Dy * sn, rb = Dy * co - Dx * sn;
                    orders([&](double *row, double, double ab, double ct) {
                        const double sa = ab * ra, tb = ct * rb;
                        row[0] = -(sa * er + tb * ei);
                        row[kSumStride] = sa * ei - tb * er;
                    });
                }
            }
        }
    }
    sums.store(p, [&](int o, double v) { Lc[(int64_t)d * Pp + o] += v; });
}

// P2M, one wavefront per leaf (entry of leaf_list, or every leaf: leaf_base plus
// it is the box), a lane per point: for few leaves, where k_p2m_quad's chains of points
// per lane leave the GPU idle and its unrolled code is fetched for a few
// wavefronts only.  Per chunk of eight orders, the highest first: F_n further
// down, then the terms with the powers of conj(z) from the chunk's first order
// up, summed over the lanes as OrderSums says.  blevel: the box's level (its
// tables); null: all at level lev.
// Up to kP2MWaveLeaves leaves (of some 15 points): 4.4 k leaves 15 us against
// 19 by quads, 9 k 23 against 20, 18 k 38 against 24 (order 24).
constexpr int64_t kP2MWaveLeaves = 6144;
struct P2MTables {
    const int32_t *blevel;
    int lev;
    const double *sc;           // F_{p+1}, F_{p+2} series, sc_stride per level
    const int32_t *nser_lv;     // null: nser
    const double *invR_lv;      // null: invR
    const double *invFY, *da, *db, *cnn;
    int sc_stride, nser;
    double invR;
};
__global__ __launch_bounds__(64) void k_p2m_wave(
    int64_t leaf_base, const int32_t *__restrict__ leaf_list, const int32_t *__restrict__ lrange,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ qs, const double *__restrict__ dns, int64_t off1,
    int has_q, int has_d, double inv_alpha, P2MTables tb, int p, int Pp, double *__restrict__ M, int accumulate) {
    __shared__ double sh[kSumLds];
    const int lane = threadIdx.x;
    const int64_t li = leaf_list ? leaf_list[blockIdx.x] : (int64_t)blockIdx.x, b = leaf_base + li;
    const int l = tb.blevel ? tb.blevel[b] : tb.lev;
    const double *ify = tb.invFY + (int64_t)l * (p + 2), *cnn = tb.cnn;
    const double *da = tb.da + (int64_t)l * (p + 2), *db = tb.db + (int64_t)l * (p + 2);
    const double *sc = tb.sc + (int64_t)l * tb.sc_stride;
    const int nser = tb.nser_lv ? tb.nser_lv[l] : tb.nser;
    const double invR = tb.invR_lv ? tb.invR_lv[l] : tb.invR;
    const double cx = bcx[b], cy = bcy[b];
    const int ctop = p >> 3;
    OrderSums sums;
    for (int set = 0; set < 2; ++set) {
        if ((set == 0 && !has_q) || (set == 1 && !has_d)) continue;
        const int s0 = lrange[li * 6 + 2 * set], e0 = lrange[li * 6 + 2 * set + 1];
        for (int base = s0; base < e0; base += 64) {
            const int j = min(base + lane, e0 - 1);
            const bool on = base + lane < e0;
            const double wx = (px[j] - cx) * inv_alpha, wy = (py[j] - cy) * inv_alpha;
            const double y = 0.25 * (wx * wx + wy * wy);
            const double zx = wx * invR, zy = -wy * invR;   // conj(w)/R
            double F1, F2;
            f_start(y, sc, nser, F1, F2);
            auto fnext = [&](int n) {   // F_n / F_n(Y), downwards from n = p
                const double F0 = F1 + y * F2 * cnn[n];
                F2 = F1;
                F1 = F0;
                return F0 * ify[n];
            };
            // conj(z)^2 and ^8, and the chunks' first powers 8c - set
            const double z2r = zx * zx - zy * zy, z2i = 2.0 * zx * zy;
            const double z4r = z2r * z2r - z2i * z2i, z4i = 2.0 * z2r * z2i;
            const double z8r = z4r * z4r - z4i * z4i, z8i = 2.0 * z4r * z4i;
            double u1r = z8r, u1i = z8i;
            if (set == 1) {   // conj(z)^7
                const double z3r = z2r * zx - z2i * zy, z3i = z2r * zy + z2i * zx;
                u1r = z4r * z3r - z4i * z3i;
                u1i = z4r * z3i + z4i * z3r;
            }
            const double u2r = u1r * z8r - u1i * z8i, u2i = u1r * z8i + u1i * z8r;
            const double u3r = u2r * z8r - u2i * z8i, u3i = u2r * z8i + u2i * z8r;
            auto first_power = [&](int c, double &wr, double &wi) {
                wr = c == 3 ? u3r : c == 2 ? u2r : c == 1 ? u1r : 1.0;
                wi = c == 3 ? u3i : c == 2 ? u2i : c == 1 ? u1i : 0.0;
            };
            auto up = [&](double &wr, double &wi) {
                const double nr = wr * zx - wi * zy;
                wi = wr * zy + wi * zx;
                wr = nr;
            };
            if (set == 0) {
                const double q = on ? qs[j] : 0.0;
                for (int c = ctop; c >= 0; --c) {
                    double g[8], wr, wi;
#pragma unroll
                    for (int i = 7; i >= 0; --i) g[i] = 8 * c + i <= p ? fnext(8 * c + i) : 0.0;
                    first_power(c, wr, wi);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const double t = q * g[i];
                        double *row = sh + 2 * i * kSumStride + lane;
                        row[0] = t * wr;
                        row[kSumStride] = t * wi;
                        up(wr, wi);
                    }
                    __syncthreads();
                    sums.add(sh, c);
                    __syncthreads();
                }
            } else {
                // term_n = h [a_n D Psi_{n+1} + b_n conj(D) Psi_{n-1}], Psi_k = G_k
                // conj(z)^k, Psi_{-1} = conj(Psi_1); h folded into D, E = D conj(z)^2
                const double h = on ? 0.5 * inv_alpha : 0.0;
                const double Dx = h * dns[2 * (j - off1)], Dy = h * dns[2 * (j - off1) + 1];
                const double Ex = Dx * z2r - Dy * z2i, Ey = Dx * z2i + Dy * z2r;
                auto gn = [&](int n) { return n <= p ? fnext(n) : n == p + 1 ? F1 * ify[n] : 0.0; };
                double g[10];   // G_{8c-1} .. G_{8c+8}
                g[1] = gn(8 * ctop + 8);
                g[0] = gn(8 * ctop + 7);
                for (int c = ctop; c >= 0; --c) {
                    g[9] = g[1];
                    g[8] = g[0];
#pragma unroll
                    for (int k = 7; k >= 1; --k) g[k] = gn(8 * c - 1 + k);
                    g[0] = c > 0 ? gn(8 * c - 1) : 0.0;
                    double wr, wi;   // conj(z)^(n-1)
                    first_power(c, wr, wi);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int n = 8 * c + i;
                        double *row = sh + 2 * i * kSumStride + lane;
                        if (n == 0) {   // the real part alone: (a + b) Re(D Psi_1)
                            row[0] = (da[0] + db[0]) * (g[2] * (Dx * zx - Dy * zy));
                            row[kSumStride] = 0.0;
                        } else if (n <= p) {
                            const double X = da[n] * g[i + 2], Y = db[n] * g[i];
                            const double tr = X * Ex + Y * Dx, ti = X * Ey - Y * Dy;
                            row[0] = tr * wr - ti * wi;
                            row[kSumStride] = tr * wi + ti * wr;
                            up(wr, wi);
                        }
                    }
                    __syncthreads();
                    sums.add(sh, c);
                    __syncthreads();
                }
            }
        }
    }
    double *Mb = M + b * Pp;
    sums.store(p, [&](int o, double v) { Mb[o] = accumulate ? Mb[o] + v : v; });
    if (!accumulate)
        for (int o = 2 * p + 1 + lane; o < Pp; o += 64) Mb[o] = 0.0;
}

// L2P of the adaptive tree: as k_l2p, with the leaf's level (and its tables)
// per point, all levels' tables in LDS; leaves coarser than lmin have no local
// expansion.
__global__ __launch_bounds__(256) void k_ad_l2p(
    int64_t n, int64_t toff1, int64_t toff2, int mask, const int32_t *__restrict__ pleaf,
    const int32_t *__restrict__ leaf_box, const int32_t *__restrict__ leaf_lev, int lmin,
    const double *__restrict__ bcx, const double *__restrict__ bcy, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ Lc, double inv_alpha,
    const double *__restrict__ invR_lv, const double *__restrict__ invFY, const double *__restrict__ cnn,
    const double *__restrict__ serc_lv, const int32_t *__restrict__ nser_lv, int nser_stride, int p, int Pp,
    const double *__restrict__ outs, const int32_t *__restrict__ perm, double *__restrict__ out0,
    double *__restrict__ out1, double *__restrict__ out2, const double *__restrict__ bw,
    const double *__restrict__ bk, const double *__restrict__ bx, int nlev) {
    extern __shared__ double dyn[];
    __shared__ double s_rows[kL2PLds];
    double *t_ify = dyn, *t_sc = t_ify + nlev * (p + 2);   // levels lmin .. lmin + nlev - 1
    for (int k = threadIdx.x; k < nlev * (p + 2); k += 256) t_ify[k] = invFY[(int64_t)lmin * (p + 2) + k];
    for (int k = threadIdx.x; k < nlev * 2 * nser_stride; k += 256)
        t_sc[k] = serc_lv[(int64_t)lmin * 2 * nser_stride + k];
    const L2PPoint pt(n, toff1, toff2, mask, pleaf, px, py, outs, perm, bw, bk, bx, inv_alpha * inv_alpha);
    const int32_t li = pt.leaf;
    const int l = leaf_lev[li];
    const int64_t b = leaf_box[li];
    const double wx = (pt.x - bcx[b]) * inv_alpha, wy = (pt.y - bcy[b]) * inv_alpha;
    int32_t first = 0;
    const bool staged = nlev > 0 && l2p_stage(s_rows, n, toff1, toff2, pleaf, Pp, first,
                                              [&](int32_t leaf) { return Lc + (int64_t)leaf_box[leaf] * Pp; });
    __syncthreads();
    if (!pt.on) return;
    double v = pt.near;
    if (l >= lmin) {
        const double *ify = t_ify + (l - lmin) * (p + 2), *sc = t_sc + (l - lmin) * 2 * nser_stride;
        double far;
        if (staged) {
            const double *Lb = s_rows + (li - first) * kL2PStride + 1;
            far = l2p_series(wx, wy, invR_lv[l], sc, nser_lv[l], ify, cnn, p, [&](int k) { return Lb[k]; });
        } else {
            const double *Lb = Lc + b * Pp;
            far = l2p_series(wx, wy, invR_lv[l], sc, nser_lv[l], ify, cnn, p, [&](int k) { return Lb[k]; });
        }
        v += far * kInv2Pi;
    }
    pt.store(v, bx != nullptr, out0, out1, out2);
}

// Pairs beyond the series, FP64: up to some number of items the forms for large
// arguments are inlined, for a wavefront's own chain of pairs is what there is to
// shorten; more items take the calls, which leave registers for more wavefronts.
// Near field, called and inlined, boxes of 3 or 4 alpha: 1,024 leaves of some 20
// points 166 and 135 us, 4,096 of 61 1,193 and 1,088, 8,239 of 40 1,121 and
// 1,063, 12,289 of 40 1,547 and 1,543, 16,384 of 60 3,262 and 3,321, 65,536 of 15
// 960 and 1,055.  Boxes of up to alpha, few of whose pairs are beyond the series:
// 1,024 leaves equal, 4,096 of 15 82 and 67, 5,085 of 40 402 and 403, of 60 635
// and 662, 6,735 of 15 80 and 89.
LeafKernel pick_leaf_kernel(int nt, double tmax, bool f32, int64_t items) {
    const bool small_only = tmax <= 1.0;
    if (f32) return small_only ? k_leaf<8, true, true> : k_leaf<8, false, true>;
    if (small_only) {
        if (nt <= 5) return k_leaf<5, true>;
        if (nt <= 6) return k_leaf<6, true>;
        if (nt <= 8) return k_leaf<8, true>;
        if (nt <= 10) return k_leaf<10, true>;
        return k_leaf<14, true>;
    }
    return items <= (tmax <= 2.0 ? 4608 : 12288) ? k_leaf<14, false, false, false> : k_leaf<14, false>;
}

}  // namespace

// one resident round of the persistent M2L: three workgroups per compute unit
int m2l_persist_grid(Context &ctx) {
    static int cus = 0;
    if (cus == 0) {
        int n = 0;
        YK_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, ctx.device));
        cus = n > 0 ? n : 256;
    }
    return 3 * cus;
}

// M2M over levels L-1 .. lmin: each parent box from its children (the
// adaptive tree's split boxes only: a leaf keeps its own multipole)
void fmm_m2m(Context &ctx, FmmPlan &pl) {
    StageTimer tmm(ctx, YK_STAGE_M2M);
    for (const ShiftGroup &gr : pl.m2m_groups) launch_m2m_group(ctx, pl, gr);
}

// M2L of dense V lists with 64 padded coefficients goes by sibling groups (its
// 98,304 multiply-adds per parent, empty lists or not, are below the 442,368 of
// the dense tiles for every filling of the lists; below 64 padded coefficients
// there is no such kernel), in FP64 also where sums in FP32 are asked for: on
// 2^20 points 0.11 ms, where the FP32 tiles take 0.24 and the multipoles' copies
// in FP32 another 0.02.
static bool use_sym(const FmmPlan &pl, const ActiveSet &as) {
    return pl.Pp == 64 && !as.m2l_sparse && as.n_sym_tiles > 0;
}

int64_t m2l_clear_len(const FmmPlan &pl, const ActiveSet &as) {
    if (!use_sym(pl, as)) return (int64_t)pl.nbox * pl.Pp;
    return as.n_sym_coarse > 0 ? 0 : pl.lev[as.sym_level].begin * (int64_t)pl.Pp;
}

// The M2L operators in FP32, for the routes that sum in it: sparse lists, or
// fewer than 64 padded coefficients.  Made on first use: most trees never read
// them (0.66 MB a level at 64 coefficients; converted and sent by the host with
// every tree, 0.3 of the 23.8 ms that the tables of 4,096 points take).
static const float *m2l_f32(Context &ctx, FmmPlan &pl) {
    const int64_t n = (int64_t)(pl.L + 1) * kNumOff * pl.Pp * pl.Pp;
    float *f = pl.m2lf.ensure(n);
    if (!pl.m2lf_built) {
        hipLaunchKernelGGL(k_to_float, dim3(nblk(n, 256)), dim3(256), 0, ctx.stream, n, pl.m2l.p, f);
        check_launch(ctx, "k_to_float");
        pl.m2lf_built = true;
    }
    return f;
}

// M2L of every level at once into the zeroed local expansions
void fmm_m2l(Context &ctx, FmmPlan &pl, ActiveSet &as, bool f32) {
    const int P = pl.P, Pp = pl.Pp;
    {
        // M2L of every level at once (levels are independent given the multipoles)
        StageTimer tl(ctx, YK_STAGE_M2L);
        // (FP32: 128-box tiles, two column blocks per wavefront, so each
        // operator fragment feeds two matrix-core steps)
        SlabPlan slab;
        slab.buf = &as.m2l_slab;
        slab.ntgt = as.n_csr_tgt;
        slab.tgt = as.csr_tgt.p;
        slab.off = as.csr_off.p;
        slab.rows = as.csr_rows.p;
        if (as.m2l_sparse && f32)
            launch_tile_gemm<float, float>(ctx, P, Pp, as.n_ptiles, as.m2l_ptiles.p, 0, as.m2l_piota.p,
                                           1, as.m2l_psrc.p, pl.iota40.p, m2l_f32(ctx, pl),
                                           (int64_t)kNumOff * Pp * Pp, pl.Mf.p, pl.Lc.p,
                                           as.m2l_ptgt.p, &slab, as.n_ptrans);
        else if (as.m2l_sparse)
            launch_tile_gemm<double, double>(ctx, P, Pp, as.n_ptiles, as.m2l_ptiles.p, 0,
                                             as.m2l_piota.p, 1, as.m2l_psrc.p, pl.iota40.p, pl.m2l.p,
                                             (int64_t)kNumOff * Pp * Pp, pl.M.p, pl.Lc.p,
                                             as.m2l_ptgt.p, &slab, as.n_ptrans);
        else if (f32 && !use_sym(pl, as))
            launch_tile_gemm<float, float, 2>(ctx, P, Pp, as.n_tiles_w, as.m2l_tiles_w.p, 0,
                                              as.m2l_boxes.p, kNumV, pl.vlist.p, pl.slot_oid.p,
                                              m2l_f32(ctx, pl), (int64_t)kNumOff * Pp * Pp, pl.Mf.p, pl.Lc.p,
                                              nullptr, &slab);
        else {
            // sibling groups at the levels they serve, the dense products by
            // box at the others (the leading tiles, which are level-major)
            int nt = as.n_tiles;
            if (use_sym(pl, as)) {
                nt = 0;
                if (as.n_sym_coarse == 0)
                    for (int l = pl.lmin; l < as.sym_level && l <= pl.L; ++l) nt += as.tile_count[l];
                launch_m2l_sym(ctx, pl, as);
            }
            if (Pp == 64 && P == 63 && nt >= m2l_persist_grid(ctx)) {
                hipLaunchKernelGGL(k_m2l_persist, dim3(m2l_persist_grid(ctx)), dim3(256), 0, ctx.stream,
                                   as.m2l_tiles.p, nt, as.m2l_boxes.p, pl.vlist.p, pl.slot_oid.p,
                                   pl.m2l.p, (int64_t)kNumOff * Pp * Pp, pl.M.p, pl.Lc.p);
                check_launch(ctx, "k_m2l_persist");
            } else
                launch_tile_gemm<double, double, 1>(ctx, P, Pp, nt, as.m2l_tiles.p, 0, as.m2l_boxes.p, kNumV,
                                                    pl.vlist.p, pl.slot_oid.p, pl.m2l.p,
                                                    (int64_t)kNumOff * Pp * Pp, pl.M.p, pl.Lc.p, nullptr,
                                                    &slab);
        }
    }
}

// L2L top-down over levels lmin+1 .. L (each box pulls its parent's expansion)
void fmm_l2l(Context &ctx, FmmPlan &pl, ActiveSet &as) {
    StageTimer tl2(ctx, YK_STAGE_L2L);
    for (const ShiftGroup &gr : as.l2l_groups) launch_l2l_group(ctx, pl, as, gr);
}

static void launch_ad_l2p(Context &ctx, FmmPlan &pl, int mask, const double *outs, double *const out[3],
                          const BieFuse *bie) {
    const int nlev = std::max(0, pl.L - pl.lmin + 1);
    const size_t tabs = (size_t)nlev * (pl.p + 2 + 2 * pl.nser_stride) * sizeof(double);
    hipLaunchKernelGGL(k_ad_l2p, dim3(nblk(pl.N, 256)), dim3(256), tabs, ctx.stream, pl.N, pl.toff[1], pl.toff[2], mask,
                       pl.pleaf.p, pl.leaf_box.p, pl.leaf_lev.p, pl.lmin, pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p,
                       pl.Lc.p, 1.0 / pl.alpha, pl.invR_lv.p, pl.invFY.p, pl.cnn.p, pl.serc_lv.p, pl.nser_dev.p,
                       pl.nser_stride, pl.p, pl.Pp, outs, pl.perm.p, out[0], out[1], out[2], bie ? bie->w : nullptr,
                       bie ? bie->kappa : nullptr, (bie && bie->kappa) ? bie->sigma : nullptr, nlev);
    check_launch(ctx, "k_ad_l2p");
}

void fmm_adaptive_finish(Context &ctx, FmmPlan &pl, int mask, double *outs, double *const out[3]) {
    const int p = pl.p, Pp = pl.Pp;
    const double inv_alpha = 1.0 / pl.alpha;
    StageTimer tl(ctx, YK_STAGE_L2P);
    if (pl.n_wleaves > 0 && pl.lmin <= pl.L) {
        hipLaunchKernelGGL(k_ad_m2p, dim3((unsigned)pl.n_wleaves), dim3(64), 0, ctx.stream, pl.wleaves.p, pl.woff.p,
                           pl.wl.p, pl.lrange.p, mask, pl.blevel.p, pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p, pl.M.p,
                           pl.rI.p, p, Pp, inv_alpha, outs);
        check_launch(ctx, "k_ad_m2p");
    }
    launch_ad_l2p(ctx, pl, mask, outs, out, nullptr);
}

void fmm_run(Context &ctx, FmmPlan &pl, const double *q, const double *dn, double *const out[3],
             SumPrec prec, const BieFuse *bie, int keep_charge_m, int parts) {
    int mask = 0;
    for (int s = 0; s < 3; ++s)
        if (out[s] && pl.toff[s + 1] > pl.toff[s]) mask |= 1 << s;
    if (!mask) return;
    const int64_t n0 = pl.toff[1] - pl.toff[0], n1 = pl.toff[2] - pl.toff[1];
    if (bie && !bie->sigma) bie = nullptr;
    // The charges' leaf multipoles of a charges-only pass stay in M for a
    // later pass with the same charges (keep_charge_m 1, then 2); any other
    // pass may overwrite them, and the reusing pass adds the dipoles to them.
    if (keep_charge_m != 2) pl.mq_kept = false;
    const int has_q = (q && n0 > 0) ? 1 : 0, has_d = ((dn || bie) && n1 > 0) ? 1 : 0;
    const int L = pl.L, p = pl.p, P = pl.P, Pp = pl.Pp;
    const double inv_alpha = 1.0 / pl.alpha;
    double *outs = pl.outs.ensure(pl.N);
    pl.last_mask = mask;
    pl.last_has_q = has_q;
    pl.last_has_d = has_d;
    ActiveSet &as = get_active(ctx, pl, mask);
    // parts: bit 0 the near field, bit 1 the far field (the order check
    // evaluates them apart; the near field alone is then evaluated on the fly)
    const bool far = pl.lmin <= L && (has_q || has_d) && (parts & 2);
    const bool near_on = (parts & 1) != 0;
    const int64_t leaf_base = pl.lev[L].begin;
    const bool f32 = prec == SUM_FP32;

    // cached near field: (the near field alone, without the far field's L2P,
    // cannot use the symmetric cache's incoming slots: it is evaluated on the
    // fly, and so is the adaptive tree's)
    const bool want_cache = near_on && as.n_leaves > 0 && ctx.opt.near_cache_mb > 0 && (parts & 2) && !pl.adaptive;
    if (want_cache) ensure_near_layout(ctx, pl, as);
    const bool near_cached = want_cache && (as.near_q_len + 2 * as.near_d_len) * (f32 ? 4 : 8) <=
                                               ((int64_t)ctx.opt.near_cache_mb << 20);
    // cached P2M rows for small trees (there the compute kernel's chains are
    // latency-bound; for large ones it beats reading the rows) when they fit
    // the cache budget
    const bool p2m_cached = far && ctx.opt.near_cache_mb > 0 && pl.nleaf < 8192 && !pl.adaptive &&
                            (n0 + 2 * n1) * (int64_t)Pp * (int64_t)sizeof(double) <=
                                ((int64_t)ctx.opt.near_cache_mb << 20);
    // few items: four wavefronts each, which would otherwise leave the GPU
    // with under about eight wavefronts per CU
    const bool wide = as.n_items < 2048;
    // Small trees: P2M and the near field in one launch, which reads the
    // strengths through the permutation (k_p2m_near).  With more items the
    // near field outlasts P2M by so much that it goes to a second stream, under
    // the whole far field; large trees fill the GPU with either, and sharing it
    // was measured no faster than running the stages in turn.  (In one launch,
    // and the stages in turn: a density solve on 28,672 nodes, 15 operator
    // applications, 1.62 and 1.80 ms; right-hand side and step on 64^2 cells and
    // 512 nodes 0.95 and 1.04 ms; a pass over 4,096 + 1,536 points 61 and 71 us.
    // With the second stream the solve took 1.75 when one launch took 1.63.)
    const bool merged = far && near_cached && p2m_cached && wide && !(ctx.opt.debug_flags & 2);
    const bool overlap = !merged && !(ctx.opt.debug_flags & 2) && pl.nleaf < 8192 && near_on;

    double *qs = nullptr, *dns = nullptr;
    Strengths st;
    if (merged) {
        st.perm = pl.perm.p;
        st.q = q;
        if (bie) {
            st.w = bie->w;
            st.sigma = bie->sigma;
            st.normal = bie->normal;
        } else {
            st.dn = dn;
        }
    } else {
        qs = pl.qs.ensure(n0 > 0 ? n0 : 1);
        dns = pl.dns.ensure(n1 > 0 ? 2 * n1 : 1);
        st.qs = qs;
        st.dns = dns;
        StageTimer tg(ctx, YK_STAGE_GATHER);
        if (has_q) {
            hipLaunchKernelGGL(k_gather_q, dim3(nblk(n0, 256)), dim3(256), 0, ctx.stream, n0, pl.perm.p, q, qs);
            check_launch(ctx, "k_gather_q");
        }
        if (has_d && bie) {
            hipLaunchKernelGGL(k_gather_dn_form, dim3(nblk(n1, 256)), dim3(256), 0, ctx.stream, pl.toff[1], n1,
                               pl.perm.p, bie->w, bie->sigma, bie->normal, dns);
            check_launch(ctx, "k_gather_dn_form");
        } else if (has_d) {
            hipLaunchKernelGGL(k_gather_dn, dim3(nblk(n1, 256)), dim3(256), 0, ctx.stream, pl.toff[1], n1,
                               pl.perm.p, dn, dns);
            check_launch(ctx, "k_gather_dn");
        }
    }
    // an evaluation of the near field's values on their first use
    const bool small_only = pl.near_tmax <= 1.0;
    const int q_on = n0 > 0 ? 1 : 0, d_on = n1 > 0 ? 1 : 0;
    auto build_near = [&](hipStream_t stream) {
        bool &built = f32 ? as.near32 : as.near64;
        if (built) return;
        StageTimer tb(ctx, YK_STAGE_NEAR_BUILD, stream);
        // (symmetric: charge values by the first kernel, dipole values by the second)
        const int q_full = as.near_sym ? 0 : q_on;
        const bool second = !as.near_sym || d_on;
        if (f32) {
            float *mq = as.nq32.ensure(std::max<int64_t>(as.near_q_len, 1));
            float *md = as.nd32.ensure(std::max<int64_t>(2 * as.near_d_len, 1));
            if (as.near_sym)
                hipLaunchKernelGGL(pick_near_build_sym32(small_only), dim3(as.n_items), dim3(64), 0, stream,
                                   as.leaf_items.p, pl.lrange.p, pl.ulist_off.p, pl.ulist.p, pl.px.p, pl.py.p, mask,
                                   0.5 * inv_alpha, as.item_qoff.p, mq);
            if (second)
                hipLaunchKernelGGL(pick_near_build32(small_only), dim3(as.n_items), dim3(64), 0, stream,
                                   as.leaf_items.p, pl.lrange.p, pl.ulist_off.p, pl.ulist.p, pl.px.p, pl.py.p, q_full,
                                   d_on, mask, 0.5 * inv_alpha, as.item_qoff.p, as.item_doff.p, mq, md);
        } else {
            double *mq = as.nq64.ensure(std::max<int64_t>(as.near_q_len, 1));
            double *md = as.nd64.ensure(std::max<int64_t>(2 * as.near_d_len, 1));
            if (as.near_sym)
                hipLaunchKernelGGL(pick_near_build_sym64(pl.near_terms, small_only), dim3(as.n_items), dim3(64), 0,
                                   stream, as.leaf_items.p, pl.lrange.p, pl.ulist_off.p, pl.ulist.p, pl.px.p, pl.py.p,
                                   mask, 0.5 * inv_alpha, as.item_qoff.p, mq);
            if (second)
                hipLaunchKernelGGL(pick_near_build64(pl.near_terms, small_only), dim3(as.n_items), dim3(64), 0, stream,
                                   as.leaf_items.p, pl.lrange.p, pl.ulist_off.p, pl.ulist.p, pl.px.p, pl.py.p, q_full,
                                   d_on, mask, 0.5 * inv_alpha, as.item_qoff.p, as.item_doff.p, mq, md);
        }
        check_launch(ctx, "k_near_build");
        built = true;
    };
    const NearFull nfull{as.leaf_items.p, pl.lrange.p, pl.ulist_off.p, pl.ulist.p, q_on, d_on, mask};
    NearSym nsym{as.sym_desc.p, as.sym_desc_dst.p, nullptr};
    if (near_cached && as.near_sym && has_q) nsym.inc = as.inc.ensure(std::max<int64_t>(as.inc_len, 1));
    const double *sym_inc = near_cached && as.near_sym ? nsym.inc : nullptr;   // incoming slots (for k_l2p)
    auto near_pass = [&](auto vt) {
        using VT = decltype(vt);
        NearPass<VT> np;
        np.st = st;
        np.off1 = pl.toff[1];
        np.has_q = has_q;
        np.has_d = has_d;
        np.qoff = as.item_qoff.p;
        np.doff = as.item_doff.p;
        if constexpr (std::is_same<VT, float>::value) {
            np.Mq = as.nq32.p;
            np.Md = as.nd32.p;
        } else {
            np.Mq = as.nq64.p;
            np.Md = as.nd64.p;
        }
        np.dip_scale = 0.5 * inv_alpha;
        np.outs = outs;
        return np;
    };

    // near field: independent of the far field until L2P
    bool near_done = merged;
    auto launch_near = [&]() {
        near_done = true;
        if (!near_on) {   // far field alone: L2P adds it to zeros
            launch_fill(ctx, pl.N, 0.0, outs);
            return;
        }
        if (overlap) {
            ensure_side_stream(ctx);
            YK_HIP(hipEventRecord(ctx.ev_fork, ctx.stream));
            YK_HIP(hipStreamWaitEvent(ctx.side, ctx.ev_fork, 0));
        }
        hipStream_t near_stream = overlap ? ctx.side : ctx.stream;
        if (as.n_leaves > 0) {
            if (near_cached) {
                build_near(near_stream);
                StageTimer tl(ctx, YK_STAGE_LEAF, near_stream);
                const dim3 blk(wide ? 256 : 64);
                auto apply = [&](auto vt) {
                    using VT = decltype(vt);
                    if (as.near_sym) {
                        auto kern = wide ? k_near_apply_sym<VT, 256> : k_near_apply_sym<VT, 64>;
                        hipLaunchKernelGGL(kern, dim3(as.n_items), blk, 0, near_stream, nsym, near_pass(vt));
                    } else {
                        auto kern = wide ? k_near_apply<VT, 256> : k_near_apply<VT, 64>;
                        hipLaunchKernelGGL(kern, dim3(as.n_items), blk, 0, near_stream, nfull, near_pass(vt));
                    }
                };
                if (f32) apply(0.f);
                else apply(0.0);
                check_launch(ctx, "k_near_apply");
            } else {
                StageTimer tl(ctx, YK_STAGE_LEAF, near_stream);
                LeafArgs la{as.leaf_items.p, pl.lrange.p, pl.ulist_off.p, pl.ulist.p, pl.px.p, pl.py.p, qs, dns,
                            pl.toff[1], has_q, has_d, mask, 0.5 * inv_alpha, 0.5 * inv_alpha, outs};
                if (!pl.adaptive) {
                    hipLaunchKernelGGL(pick_leaf_kernel(pl.near_terms, pl.near_tmax, f32, as.n_items),
                                       dim3(as.n_items), dim3(64), 0, near_stream, la);
                } else if (f32) {
                    // the kind with large arguments, then the others (one series serves them)
                    const int n_large = as.item_kind[1];
                    if (n_large > 0)
                        hipLaunchKernelGGL((k_leaf<8, false, true>), dim3(n_large), dim3(64), 0, near_stream, la);
                    la.items += n_large;
                    if (as.n_items > n_large)
                        hipLaunchKernelGGL((k_leaf<8, true, true>), dim3(as.n_items - n_large), dim3(64), 0,
                                           near_stream, la);
                } else {
                    LeafKinds lk;
                    int blocks = 0;
                    for (int k = 0; k <= kLeafKinds; ++k) {
                        lk.block[k] = blocks;
                        lk.item[k] = as.item_kind[k];
                        if (k < kLeafKinds) blocks += ((as.item_kind[k + 1] - as.item_kind[k] + 3) / 4 + 7) / 8 * 8;
                    }
                    hipLaunchKernelGGL(k_leaf_kinds, dim3(blocks), dim3(256), 0, near_stream, la, lk);
                }
                check_launch(ctx, "k_leaf");
            }
        }
        if (overlap) YK_HIP(hipEventRecord(ctx.ev_join, ctx.side));
    };
    const size_t lvl = (size_t)(p + 2);
    bool lc_clear = false;   // Lc already cleared (by the cached P2M kernel)
    const int64_t lc_len = m2l_clear_len(pl, as);
    if (far && pl.adaptive) {
        // P2M at the leaves of every level from lmin on, with the level's tables
        // (leaves coarser than lmin need no multipole)
        StageTimer tm(ctx, YK_STAGE_P2M);
        pl.mq_kept = false;
        const int64_t nl = pl.n_p2m;
        auto quad4 = p == 8 ? k_p2m_quad<8> : p == 12 ? k_p2m_quad<12> : p == 16 ? k_p2m_quad<16>
                   : p == 20 ? k_p2m_quad<20> : p == 24 ? k_p2m_quad<24> : p == 28 ? k_p2m_quad<28>
                   : p == 31 ? k_p2m_quad<31> : nullptr;
        YK_REQUIRE(quad4 != nullptr, "no P2M kernel for this order");
        if (nl > 0 && nl < kP2MWaveLeaves) {
            const P2MTables tb{pl.blevel.p, 0, pl.serc_lv.p, pl.nser_dev.p, pl.invR_lv.p, pl.invFY.p, pl.dipa.p,
                               pl.dipb.p, pl.cnn.p, 2 * pl.nser_stride, 0, 0.0};
            hipLaunchKernelGGL(k_p2m_wave, dim3((unsigned)nl), dim3(64), 0, ctx.stream, 0, pl.p2m_list.p, pl.alr.p,
                               pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p, qs, dns, pl.toff[1], has_q, has_d, inv_alpha, tb,
                               p, Pp, pl.M.p, 0);
            check_launch(ctx, "k_p2m_wave");
        } else if (nl > 0) {
            const size_t tabs = (2 * (size_t)pl.nser_stride + 4 * (size_t)(p + 2)) * sizeof(double);
            hipLaunchKernelGGL(quad4, dim3((unsigned)pl.n_p2m_tiles), dim3(64), tabs, ctx.stream, pl.alr.p, pl.bcx.p,
                               pl.bcy.p, pl.px.p, pl.py.p, qs, dns, pl.toff[1], has_q, has_d, inv_alpha, pl.invFY.p,
                               pl.dipa.p, pl.dipb.p, pl.cnn.p, pl.serc_lv.p, Pp, pl.M.p, pl.p2m_list.p,
                               pl.p2m_tiles.p, pl.nser_dev.p, pl.invR_lv.p, 2 * pl.nser_stride);
            check_launch(ctx, "k_p2m_quad");
        }
    }
    if (far) {
        // upward pass
        if (!pl.adaptive) {
        if (p2m_cached && !pl.p2m_rows_built) {
            // cached rows (built on first use)
            StageTimer tb(ctx, YK_STAGE_NEAR_BUILD);
            double *rq = pl.p2m_rq.ensure(std::max<int64_t>(n0 * Pp, 1));
            double *rd = pl.p2m_rd.ensure(std::max<int64_t>(2 * n1 * Pp, 1));
            double *gs = pl.p2m_gs.ensure(std::max<int64_t>((n0 + n1) * (p + 2), 1));
            hipLaunchKernelGGL(k_p2m_rows, dim3(nblk(n0 + n1, 256)), dim3(256), 0, ctx.stream, n0, n1,
                               pl.toff[1], pl.pleaf.p, leaf_base, pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p,
                               inv_alpha, 1.0 / pl.lev[L].R, pl.invFY.p + L * lvl, pl.dipa.p + L * lvl,
                               pl.dipb.p + L * lvl, pl.cnn.p, pl.serc.p, pl.nser, p, Pp, rq, rd, gs);
            check_launch(ctx, "k_p2m_rows");
            YK_HIP(hipStreamSynchronize(ctx.stream));
            pl.p2m_gs.release();
            pl.p2m_rows_built = true;
        }
        const P2MApply pa{leaf_base,    pl.nleaf, pl.lrange.p, pl.p2m_rq.p, pl.p2m_rd.p, P, Pp, pl.M.p,
                          pl.Lc.p, lc_len};
        if (merged) {
            build_near(ctx.stream);
            StageTimer tm(ctx, YK_STAGE_LEAF);
            const dim3 grid((unsigned)(as.n_items + pl.nleaf));
            auto both = [&](auto vt) {
                using VT = decltype(vt);
                auto kern = as.near_sym ? k_p2m_near<VT, true> : k_p2m_near<VT, false>;
                hipLaunchKernelGGL(kern, grid, dim3(256), 0, ctx.stream, pa, nfull, nsym, near_pass(vt), (int)as.n_items);
            };
            if (f32) both(0.f);
            else both(0.0);
            check_launch(ctx, "k_p2m_near");
            lc_clear = true;
        } else {
        StageTimer tm(ctx, YK_STAGE_P2M);
        if (p2m_cached) {
            hipLaunchKernelGGL(k_p2m_apply, dim3((unsigned)pl.nleaf), dim3(256), 0, ctx.stream, pa, st, pl.toff[1],
                               has_q, has_d);
            check_launch(ctx, "k_p2m_apply");
            lc_clear = true;
        } else {
        auto half = p == 8 ? k_p2m_half<8> : p == 12 ? k_p2m_half<12> : p == 16 ? k_p2m_half<16>
                  : p == 20 ? k_p2m_half<20> : p == 24 ? k_p2m_half<24> : p == 28 ? k_p2m_half<28>
                  : p == 31 ? k_p2m_half<31> : nullptr;
        YK_REQUIRE(half != nullptr, "no P2M kernel for this order");
        // a wavefront per leaf: all leaves when they are few, else (list) those
        // that hold dipoles, whose points are dense along the curves; charges
        // too unless add_only
        const bool many = pl.nleaf >= 8192;
        auto by_wave = [&](const int32_t *list, int64_t nl, int with_q, int with_d, int add_only) {
            const P2MTables tb{nullptr, L, pl.serc.p, nullptr, nullptr, pl.invFY.p, pl.dipa.p, pl.dipb.p, pl.cnn.p,
                               0, pl.nser, 1.0 / pl.lev[L].R};
            hipLaunchKernelGGL(k_p2m_wave, dim3((unsigned)nl), dim3(64), 0, ctx.stream, leaf_base,
                               list, pl.lrange.p, pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p, qs, dns, pl.toff[1],
                               with_q, with_d, inv_alpha, tb, p, Pp, pl.M.p, add_only);
        };
        if (many && keep_charge_m == 2 && pl.mq_kept && has_q) {
            // the charges' leaf multipoles of the keeping pass are still in M:
            // the dipoles are added to them
            if (has_d && pl.n_dleaves > 0) by_wave(pl.dleaves.p, pl.n_dleaves, 0, 1, 1);
            pl.mq_kept = false;
        } else if (many) {
            // charges in two halves of the orders on the leaves without
            // dipoles (all leaves when there are none), then the leaves with
            // dipoles, charges and dipoles together
            const int split_d = has_d && pl.n_dleaves > 0;
            // (the two kernels write disjoint leaves, but running the dipole
            // leaves' one on a second stream was measured no faster: the
            // other fills the GPU)
            const size_t tabh = (2 * (size_t)pl.nser + 2 * (size_t)(p + 2)) * sizeof(double);
            hipLaunchKernelGGL(half, dim3((unsigned)((pl.nleaf + 15) / 16), 2), dim3(64), tabh, ctx.stream,
                               leaf_base, pl.nleaf, pl.lrange.p, pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p, qs,
                               has_q, inv_alpha, 1.0 / pl.lev[L].R, pl.invFY.p + L * lvl, pl.cnn.p, pl.serc.p,
                               pl.nser, Pp, pl.M.p, split_d, pl.Lc.p, lc_len);
            lc_clear = true;
            if (keep_charge_m == 1 && has_q && !has_d) pl.mq_kept = true;
            if (split_d) by_wave(pl.dleaves.p, pl.n_dleaves, has_q, 1, 0);
        } else {
            by_wave(nullptr, pl.nleaf, has_q, has_d, 0);
        }
        check_launch(ctx, "k_p2m");
        }
        }
        }
        if (!near_done) launch_near();
        fmm_m2m(ctx, pl);
        if (f32 && !use_sym(pl, as)) {
            const int64_t nm = pl.nbox * (int64_t)Pp;
            float *mf = pl.Mf.ensure(nm);
            hipLaunchKernelGGL(k_to_float, dim3(nblk(nm, 256)), dim3(256), 0, ctx.stream, nm, pl.M.p, mf);
            check_launch(ctx, "k_to_float");
        }
        // downward pass
        // a fill kernel rather than a memset node: this pass may be captured in a graph
        if (!lc_clear) launch_fill(ctx, lc_len, 0.0, pl.Lc.p);
        {
            fmm_m2l(ctx, pl, as, f32);
            if (pl.adaptive && pl.n_xbox > 0) {
                // X lists: coarser leaves' sources straight into the local
                // expansions (before L2L passes them down)
                StageTimer tx(ctx, YK_STAGE_M2L);
                hipLaunchKernelGGL(k_ad_p2l, dim3((unsigned)pl.n_xbox), dim3(64), 0, ctx.stream, pl.xbox.p, pl.xoff.p,
                                   pl.xl.p, pl.lrange.p, has_q, has_d, pl.blevel.p, pl.bcx.p, pl.bcy.p, pl.px.p,
                                   pl.py.p, qs, dns, pl.toff[1], pl.rI.p, p, Pp, inv_alpha, pl.Lc.p);
                check_launch(ctx, "k_ad_p2l");
            }
            fmm_l2l(ctx, pl, as);
        }
    }
    if (!near_done) launch_near();
    if (overlap) YK_HIP(hipStreamWaitEvent(ctx.stream, ctx.ev_join, 0));
    if (far && pl.adaptive && as.n_leaves > 0) {
        StageTimer tl(ctx, YK_STAGE_L2P);
        if (pl.n_wleaves > 0) {
            // W lists: finer boxes' multipoles at the leaves' targets
            hipLaunchKernelGGL(k_ad_m2p, dim3((unsigned)pl.n_wleaves), dim3(64), 0, ctx.stream, pl.wleaves.p,
                               pl.woff.p, pl.wl.p, pl.lrange.p, mask, pl.blevel.p, pl.bcx.p, pl.bcy.p, pl.px.p,
                               pl.py.p, pl.M.p, pl.rI.p, p, Pp, inv_alpha, outs);
            check_launch(ctx, "k_ad_m2p");
        }
        launch_ad_l2p(ctx, pl, mask, outs, out, bie);
        return;   // L2P wrote the outputs
    }
    if (far && as.n_leaves > 0) {
        StageTimer tl(ctx, YK_STAGE_L2P);
        const size_t lsh = (size_t)(2 * (p + 1) + 2 * pl.nser) * sizeof(double);
        hipLaunchKernelGGL(k_l2p, dim3(nblk(pl.N, 256)), dim3(256), lsh, ctx.stream, pl.N, pl.toff[1],
                           pl.toff[2], mask, pl.pleaf.p, leaf_base, pl.bcx.p, pl.bcy.p, pl.px.p, pl.py.p,
                           pl.Lc.p, inv_alpha, 1.0 / pl.lev[L].R, pl.invFY.p + L * lvl, pl.cnn.p,
                           pl.serc.p, pl.nser, p, Pp, outs, pl.perm.p, out[0], out[1], out[2],
                           bie ? bie->w : nullptr, bie ? bie->kappa : nullptr,
                           (bie && bie->kappa) ? bie->sigma : nullptr, sym_inc, as.inc_base.p, as.inc_cnt.p,
                           pl.lrange.p);
        check_launch(ctx, "k_l2p");
        return;   // L2P wrote the outputs
    }
    StageTimer tsc(ctx, YK_STAGE_SCATTER);
    for (int s = 0; s < 3; ++s) {
        if (!((mask >> s) & 1)) continue;
        const int64_t n = pl.toff[s + 1] - pl.toff[s];
        hipLaunchKernelGGL(k_scatter_out, dim3(nblk(n, 256)), dim3(256), 0, ctx.stream, pl.toff[s], n,
                           pl.perm.p, outs, out[s]);
        check_launch(ctx, "k_scatter_out");
        if (s == 1 && bie && bie->kappa)
            launch_bie_finish(ctx, n, bie->w, bie->kappa, pl.alpha, bie->sigma, out[1], out[1]);
    }
}

}  // namespace yk
