// shifts.hip -- M2M and L2L (the parent-child shifts) on the FP64 matrix
// cores, subtrees of up to three levels per workgroup.
//
// M2M: a parent's multipole is the sum over its four children of S[c] M_c;
// L2L: child c gets E[c] L_parent added.  A workgroup owns the subtree below
// one box: M2M computes its boxes at three levels, finest first, L2L its
// children at three levels, coarsest first, and what one level produces stays
// in LDS as the next one's operand.  The columns are the parents, four to a
// v_mfma_f64_4x4x4 (four row blocks of one 16-row tile, the same four columns
// each), so a level costs what its boxes need; the operators are kept in the
// order the lanes consume them and stream from L2 through a ring of registers.
// Bound by latency: descriptor, coefficient rows, then per level a chain of 32
// or more operator fragments from L2 and the matrix-core steps they feed.
// A padding row of a product is 0 x the source: zero, or NaN where the source's
// own row is not finite (setting it to zero in the stores took 1% of a pass over
// 7,147 nodes and 50,021 targets).  It lasts for the pass: M2M writes its boxes'
// rows whole, and M2L, or the clearing before it, those of L.
// Measured (one launch per level before): the 28,672-node boundary tree's five
// levels 27 us of M2M and 20 of L2L in ten launches, now 20 + 18 in four; 2^20
// points 61 + 66 us, now 49 + 62 (the finest level 20 -> 20 and 29 -> 28: its
// coefficients' 42 and 75 MB take 8 and 15).
#include "fmm.h"

namespace yk {

namespace {

typedef double sh_d2 __attribute__((ext_vector_type(2)));
typedef double sh_d4 __attribute__((ext_vector_type(4)));

constexpr int kShRing = 8;     // operator fragments in flight per wavefront
constexpr int kShFrag = 128;   // doubles of a fragment: 64 lanes x 2

__device__ __forceinline__ int sh_remap(int b, int n) {   // consecutive subtrees on one XCD
    const int x = b % 8;
    return x * (n / 8) + min(x, n % 8) + b / 8;
}

// contraction pair kappa (indices 2 kappa, 2 kappa + 1) of parent j in LDS, of
// K pairs: [four parents][pair][parent][2], the groups of four 64 bytes off a
// multiple of the bank period
template <int K>
__device__ __forceinline__ int sh_slot(int kappa, int j) {
    return ((j >> 2) * (4 * K + 4) + 4 * kappa + (j & 3)) * 2;
}
template <int K, int G> constexpr int sh_size = G * (4 * K + 4) * 2;   // doubles of G groups

// Operator fragments of parent level l from the dense operators (column-major,
// [level][4][PP * PP]).  up: [row tile][4 PP / 8 eights][lane][2], down:
// [child][PP / 8 eights][row tile][lane][2]; lane l holds row l % 16 of the
// tile and indices 2 (l / 16) + {0, 1} of the eight.
__global__ void k_shift_ops(int64_t n, int PP, const double *__restrict__ m2m, const double *__restrict__ l2l,
                            double *__restrict__ up, double *__restrict__ down) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int per = 4 * PP * PP, NR = PP / 16, NQ = PP / 8;
    const int64_t l = t / per;
    const int f = (int)(t % per);
    const int e = f & 1, lane = (f >> 1) & 63, frag = f >> 7;
    const int row = lane & 15, kk = 2 * (lane >> 4) + e;
    const double *S = m2m + l * per, *E = l2l + l * per;
    {
        const int rt = frag / (4 * NQ), q = frag % (4 * NQ), c = q / NQ, k = 8 * (q % NQ) + kk;
        up[t] = S[((int64_t)c * PP + k) * PP + 16 * rt + row];
    }
    {
        const int c = frag / (NQ * NR), r = frag % (NQ * NR), k = 8 * (r / NR) + kk;
        down[t] = E[((int64_t)c * PP + k) * PP + 16 * (r % NR) + row];
    }
}

// 16 parents' columns: NT row tiles, NQ eights of contraction indices
template <int NT, int NQ>
__device__ __forceinline__ void sh_columns(const double *B, const sh_d2 *Ap, sh_d2 *ring, int lane, sh_d4 *out) {
    constexpr int NF = NQ * NT, NA = NT == 1 ? 2 : 1;   // (two sums where there is one row tile)
    const int g = lane >> 4, col = lane & 15;
    sh_d4 acc[NT][NA];
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int i = 0; i < NA; ++i) acc[r][i] = sh_d4{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const sh_d2 b = *reinterpret_cast<const sh_d2 *>(B + sh_slot<4 * NQ>(4 * q + g, col));
        sh_d2 a[NT];
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            const int f = q * NT + r;
            a[r] = ring[f % kShRing];
            if (f + kShRing < NF) ring[f % kShRing] = Ap[(f + kShRing) * 64];
        }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int r = 0; r < NT; ++r)
                acc[r][x % NA] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r][x], b[x], acc[r][x % NA], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < NT; ++r) {
        out[r] = acc[r][0];
        if (NA == 2) out[r] += acc[r][NA - 1];
    }
}

// The product of a level: NT row tiles, NQ eights of contraction indices, cnt
// parents; put(row of the NT tiles, parent, value) takes the results.  The ring
// holds the first fragments on entry.  Up to eight parents go as one or two
// groups of four; for more the 16-column step costs no more than four groups
// and reads each operand from LDS once instead of four times.
template <int NG, int NT, int NQ, typename Put>
__device__ __forceinline__ void sh_groups(const double *B, const sh_d2 *Ap, sh_d2 *ring, int lane, Put put) {
    constexpr int NF = NQ * NT;
    const int g = lane >> 4, j = lane & 3;
    double acc[NT][NG][2];
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int i = 0; i < NG; ++i) acc[r][i][0] = acc[r][i][1] = 0.0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        sh_d2 b[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) b[i] = *reinterpret_cast<const sh_d2 *>(B + sh_slot<4 * NQ>(4 * q + g, 4 * i + j));
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            const int f = q * NT + r;
            const sh_d2 a = ring[f % kShRing];
            if (f + kShRing < NF) ring[f % kShRing] = Ap[(f + kShRing) * 64];
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                acc[r][i][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a.x, b[i].x, acc[r][i][0], 0, 0, 0);
                acc[r][i][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a.y, b[i].y, acc[r][i][1], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int i = 0; i < NG; ++i)
            put(16 * r + 4 * ((lane >> 2) & 3) + (lane >> 4), 4 * i + j, acc[r][i][0] + acc[r][i][1]);
}
template <int NT, int NQ, typename Put>
__device__ __forceinline__ void sh_multiply(int cnt, const double *B, const sh_d2 *Ap, sh_d2 *ring, int lane, Put put) {
    if (cnt <= 4) {
        sh_groups<1, NT, NQ>(B, Ap, ring, lane, put);
        return;
    }
    if (cnt <= 8) {
        sh_groups<2, NT, NQ>(B, Ap, ring, lane, put);
        return;
    }
    sh_d4 out[NT];
    sh_columns<NT, NQ>(B, Ap, ring, lane, out);
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) put(16 * r + (lane >> 4) + 4 * i, lane & 15, out[r][i]);
}

// M2M of a subtree; the descriptor's layout is at kUp* in fmm.h
template <int PP>
__global__ __launch_bounds__(256) void k_m2m(const int32_t *__restrict__ desc, int nlev, int l,
                                             const double *__restrict__ Op, double *__restrict__ M) {
    constexpr int NR = PP / 16, NQ = 4 * PP / 8, HP = PP / 2, K = 4 * HP, LD = PP + 1;
    __shared__ double B0[sh_size<K, 4>], B1[2][sh_size<K, 1>], S[16 * LD];
    __shared__ int32_t d[kUpDesc];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const bool mul = w < NR;
    const int64_t wf = (int64_t)(mul ? w : 0) * NQ * kShFrag;
    sh_d2 ring[kShRing];
    {
        const sh_d2 *Ap = reinterpret_cast<const sh_d2 *>(Op + (int64_t)l * 4 * PP * PP + wf) + lane;
#pragma unroll
        for (int i = 0; i < kShRing; ++i)
            if (i < NQ) ring[i] = Ap[i * 64];
    }
    if (tid < kUpDesc) d[tid] = desc[(int64_t)sh_remap(blockIdx.x, gridDim.x) * kUpDesc + tid];
    __syncthreads();
    // the finest level's children, and the coarser levels' that are leaves
    // (zeros where a child is absent or comes from the level before)
    constexpr int N0 = 64 * HP / 256, N1 = (20 * HP + 255) / 256;
    const int rows0 = 4 * d[0];
    sh_d2 v0[N0], v1[N1];
#pragma unroll
    for (int i = 0; i < N0; ++i) {
        const int e = tid + 256 * i, r = e / HP, p = e % HP;
        const int32_t b = r < rows0 ? d[kUpChild + r] : -1;
        v0[i] = sh_d2{0.0, 0.0};
        if (b >= 0) v0[i] = reinterpret_cast<const sh_d2 *>(M + (int64_t)b * PP)[p];
    }
    if (nlev > 1) {
#pragma unroll
        for (int i = 0; i < N1; ++i) {
            const int e = tid + 256 * i, r = e / HP, p = e % HP;
            const int32_t b = r < 20 ? d[kUpChild + 64 + r] : -1;
            v1[i] = sh_d2{0.0, 0.0};
            if (b >= 0) v1[i] = reinterpret_cast<const sh_d2 *>(M + (int64_t)b * PP)[p];
        }
    }
#pragma unroll
    for (int i = 0; i < N0; ++i) {
        const int e = tid + 256 * i, r = e / HP, p = e % HP;
        *reinterpret_cast<sh_d2 *>(B0 + sh_slot<K>((r & 3) * HP + p, r >> 2)) = v0[i];
    }
    if (nlev > 1) {
#pragma unroll
        for (int i = 0; i < N1; ++i) {
            const int e = tid + 256 * i, r = e / HP, p = e % HP;
            if (r < 20) {
                const int k = r < 16 ? 0 : 1, rr = r - 16 * k;
                *reinterpret_cast<sh_d2 *>(B1[k] + sh_slot<K>((rr & 3) * HP + p, rr >> 2)) = v1[i];
            }
        }
    }
    __syncthreads();
    for (int k = 0; k < nlev; ++k) {
        const int cnt = d[k];
        const sh_d2 *Ap = reinterpret_cast<const sh_d2 *>(Op + (int64_t)(l - k) * 4 * PP * PP + wf) + lane;
        if (mul)
            sh_multiply<1, NQ>(cnt, k == 0 ? B0 : B1[k - 1], Ap, ring, lane,
                               [&](int row, int j, double v) { S[j * LD + 16 * w + row] = v; });
        if (k + 1 < nlev) {
            const sh_d2 *An = reinterpret_cast<const sh_d2 *>(Op + (int64_t)(l - k - 1) * 4 * PP * PP + wf) + lane;
#pragma unroll
            for (int i = 0; i < kShRing; ++i)
                if (i < NQ) ring[i] = An[i * 64];
        }
        __syncthreads();
        const int32_t *box = d + kUpBox + (k == 0 ? 0 : k == 1 ? 16 : 20), *link = d + kUpLink + (k == 0 ? 0 : 16);
        for (int e = tid; e < cnt * PP; e += 256) {
            const int j = e / PP, i = e % PP;
            const double v = S[j * LD + i];
            M[(int64_t)box[j] * PP + i] = v;
            if (k + 1 < nlev) B1[k][sh_slot<K>((link[j] & 3) * HP + (i >> 1), link[j] >> 2) + (i & 1)] = v;
        }
        __syncthreads();
    }
}

// L2L of a subtree; the descriptor's layout is at kDown* in fmm.h
template <int PP>
__global__ __launch_bounds__(256) void k_l2l(const int32_t *__restrict__ desc, int nlev, int l,
                                             const double *__restrict__ Op, double *__restrict__ L) {
    constexpr int NR = PP / 16, NQ = PP / 8, HP = PP / 2, LD = PP + 1;
    __shared__ double B[3][sh_size<HP, 4>], S[64 * LD];
    __shared__ int32_t d[kDownDesc];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int64_t wf = (int64_t)w * NQ * NR * kShFrag;
    sh_d2 ring[kShRing];
    {
        const sh_d2 *Ap = reinterpret_cast<const sh_d2 *>(Op + (int64_t)(l - 1) * 4 * PP * PP + wf) + lane;
#pragma unroll
        for (int i = 0; i < kShRing; ++i)
            if (i < NQ * NR) ring[i] = Ap[i * 64];
    }
    if (tid < kDownDesc) d[tid] = desc[(int64_t)sh_remap(blockIdx.x, gridDim.x) * kDownDesc + tid];
    __syncthreads();
    sh_d2 root{0.0, 0.0};
    if (tid < HP) root = reinterpret_cast<const sh_d2 *>(L + (int64_t)d[3] * PP)[tid];
    // what the children hold (level 0: 4 rows, level 1: 16, level 2: 64)
    constexpr int N = PP / 16;   // elements per thread of 4 rows: 4 PP / 256
    constexpr int E1 = (4 * PP + 255) / 256, E2 = 16 * PP / 256, E3 = 64 * PP / 256;
    static_assert(N >= 1, "");
    double old1[E1], old2[E2], old3[E3];
    auto fetch = [&](int k, int i) -> double {
        const int e = tid + 256 * i, s = e / PP;
        const int32_t b = s < 4 * d[k] ? d[kDownChild + (k == 0 ? 0 : k == 1 ? 4 : 20) + s] : -1;
        return b >= 0 ? L[(int64_t)b * PP + e % PP] : 0.0;
    };
#pragma unroll
    for (int i = 0; i < E1; ++i) old1[i] = fetch(0, i);
    if (nlev > 1) {
#pragma unroll
        for (int i = 0; i < E2; ++i) old2[i] = fetch(1, i);
    }
    if (nlev > 2) {
#pragma unroll
        for (int i = 0; i < E3; ++i) old3[i] = fetch(2, i);
    }
    if (tid < HP) *reinterpret_cast<sh_d2 *>(B[0] + sh_slot<HP>(tid, 0)) = root;
    __syncthreads();
    auto level = [&](int k, const double *old, auto count) {
        constexpr int NE = decltype(count)::value;
        const int cnt = d[k];
        const sh_d2 *Ap = reinterpret_cast<const sh_d2 *>(Op + (int64_t)(l - 1 + k) * 4 * PP * PP + wf) + lane;
        sh_multiply<NR, NQ>(cnt, B[k], Ap, ring, lane, [&](int row, int j, double v) { S[(4 * j + w) * LD + row] = v; });
        if (k + 1 < nlev) {
            const sh_d2 *An = reinterpret_cast<const sh_d2 *>(Op + (int64_t)(l + k) * 4 * PP * PP + wf) + lane;
#pragma unroll
            for (int i = 0; i < kShRing; ++i)
                if (i < NQ * NR) ring[i] = An[i * 64];
        }
        __syncthreads();
        const int base = k == 0 ? 0 : k == 1 ? 4 : 20;
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = tid + 256 * i, s = e / PP, o = e % PP;
            const int32_t b = s < 4 * cnt ? d[kDownChild + base + s] : -1;
            if (b >= 0) {
                const double v = old[i] + S[s * LD + o];
                L[(int64_t)b * PP + o] = v;
                const int32_t j = k + 1 < nlev ? d[kDownLink + base + s] : -1;
                if (j >= 0) B[k + 1][sh_slot<HP>(o >> 1, j) + (o & 1)] = v;
            }
        }
        __syncthreads();
    };
    level(0, old1, std::integral_constant<int, E1>{});
    if (nlev > 1) level(1, old2, std::integral_constant<int, E2>{});
    if (nlev > 2) level(2, old3, std::integral_constant<int, E3>{});
}

// One level of up to 16 boxes of no common subtree (levels of many boxes:
// their workgroups fill the GPU by themselves, and four of them share a compute
// unit).
template <int PP>
__global__ __launch_bounds__(256, 4) void k_m2m_wide(const int32_t *__restrict__ desc, const double *__restrict__ Op,
                                                     double *__restrict__ M) {
    constexpr int NR = PP / 16, NQ = 4 * PP / 8, HP = PP / 2, K = 4 * HP, LD = PP + 1, N0 = 64 * HP / 256;
    __shared__ double B[sh_size<K, 4>];
    __shared__ int32_t d[kUpDesc];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const bool mul = w < NR;
    const sh_d2 *Ap = reinterpret_cast<const sh_d2 *>(Op + (int64_t)(mul ? w : 0) * NQ * kShFrag) + lane;
    sh_d2 ring[kShRing];
#pragma unroll
    for (int i = 0; i < kShRing; ++i)
        if (i < NQ) ring[i] = Ap[i * 64];
    if (tid < kUpDesc) d[tid] = desc[(int64_t)sh_remap(blockIdx.x, gridDim.x) * kUpDesc + tid];
    __syncthreads();
    const int cnt = d[0];
    sh_d2 v[N0];
#pragma unroll
    for (int i = 0; i < N0; ++i) {
        const int e = tid + 256 * i, r = e / HP, p = e % HP;
        const int32_t b = r < 4 * cnt ? d[kUpChild + r] : -1;
        v[i] = sh_d2{0.0, 0.0};
        if (b >= 0) v[i] = reinterpret_cast<const sh_d2 *>(M + (int64_t)b * PP)[p];
    }
#pragma unroll
    for (int i = 0; i < N0; ++i) {
        const int e = tid + 256 * i, r = e / HP, p = e % HP;
        *reinterpret_cast<sh_d2 *>(B + sh_slot<K>((r & 3) * HP + p, r >> 2)) = v[i];
    }
    __syncthreads();
    double *S = B;
    sh_d4 out = sh_d4{0, 0, 0, 0};
    if (mul) sh_columns<1, NQ>(B, Ap, ring, lane, &out);
    __syncthreads();
    if (mul)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[(lane & 15) * LD + 16 * w + (lane >> 4) + 4 * i] = out[i];
    __syncthreads();
    for (int e = tid; e < cnt * PP; e += 256) M[(int64_t)d[kUpBox + e / PP] * PP + e % PP] = S[(e / PP) * LD + e % PP];
}

// The same for L2L: desc holds the parents per workgroup (0), their rows (3 ..
// 18) and their children (20 ..).
template <int PP>
__global__ __launch_bounds__(256, 3) void k_l2l_wide(const int32_t *__restrict__ desc, const double *__restrict__ Op,
                                                     double *__restrict__ L) {
    constexpr int NR = PP / 16, NQ = PP / 8, HP = PP / 2, LD = PP + 1, NP = (16 * HP + 255) / 256, NE = 64 * PP / 256;
    __shared__ double B[sh_size<HP, 4>], S[64 * LD];
    __shared__ int32_t d[kDownDesc];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const sh_d2 *Ap = reinterpret_cast<const sh_d2 *>(Op + (int64_t)w * NQ * NR * kShFrag) + lane;
    sh_d2 ring[kShRing];
#pragma unroll
    for (int i = 0; i < kShRing; ++i)
        if (i < NQ * NR) ring[i] = Ap[i * 64];
    if (tid < kDownDesc) d[tid] = desc[(int64_t)sh_remap(blockIdx.x, gridDim.x) * kDownDesc + tid];
    __syncthreads();
    const int cnt = d[0];
    sh_d2 v[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int e = tid + 256 * i, r = e / HP, p = e % HP;
        v[i] = sh_d2{0.0, 0.0};
        if (r < cnt) v[i] = reinterpret_cast<const sh_d2 *>(L + (int64_t)d[kDownWide + r] * PP)[p];
    }
    double old[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = tid + 256 * i, s = e / PP;
        const int32_t b = s < 4 * cnt ? d[kDownWide + 16 + s] : -1;
        old[i] = b >= 0 ? L[(int64_t)b * PP + e % PP] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int e = tid + 256 * i, r = e / HP, p = e % HP;
        if (r < 16) *reinterpret_cast<sh_d2 *>(B + sh_slot<HP>(p, r)) = v[i];
    }
    __syncthreads();
    sh_d4 out[NR];
    sh_columns<NR, NQ>(B, Ap, ring, lane, out);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[(4 * (lane & 15) + w) * LD + 16 * r + (lane >> 4) + 4 * i] = out[r][i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = tid + 256 * i, s = e / PP, o = e % PP;
        const int32_t b = s < 4 * cnt ? d[kDownWide + 16 + s] : -1;
        if (b >= 0) L[(int64_t)b * PP + o] = old[i] + S[s * LD + o];
    }
}

}  // namespace

void build_shift_ops(Context &ctx, FmmPlan &pl) {
    const int64_t n = (int64_t)(pl.L + 1) * 4 * pl.Pp * pl.Pp;
    double *u = pl.up_op.ensure(n), *d = pl.down_op.ensure(n);
    hipLaunchKernelGGL(k_shift_ops, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx.stream, n, pl.Pp, pl.m2m.p,
                       pl.l2l.p, u, d);
    check_launch(ctx, "k_shift_ops");
}

#define YK_SHIFT_CASES(KERN, ...)                                                                              \
    switch (pl.Pp) {                                                                                           \
        case 32: hipLaunchKernelGGL(KERN<32>, dim3(grid), dim3(256), 0, ctx.stream, __VA_ARGS__); break;       \
        case 48: hipLaunchKernelGGL(KERN<48>, dim3(grid), dim3(256), 0, ctx.stream, __VA_ARGS__); break;       \
        case 64: hipLaunchKernelGGL(KERN<64>, dim3(grid), dim3(256), 0, ctx.stream, __VA_ARGS__); break;       \
        default: throw Error{YK_ERR_INTERNAL, "no shift kernel for this padded order"};                        \
    }

void launch_m2m_group(Context &ctx, FmmPlan &pl, const ShiftGroup &gr) {
    if (gr.n <= 0) return;
    const unsigned grid = (unsigned)gr.n;
    const int64_t per = (int64_t)4 * pl.Pp * pl.Pp;
    if (gr.wide) YK_SHIFT_CASES(k_m2m_wide, pl.up_desc.p + gr.first * kUpDesc, pl.up_op.p + gr.level * per, pl.M.p)
    else YK_SHIFT_CASES(k_m2m, pl.up_desc.p + gr.first * kUpDesc, gr.nlev, gr.level, pl.up_op.p, pl.M.p)
    check_launch(ctx, "k_m2m");
}

void launch_l2l_group(Context &ctx, FmmPlan &pl, ActiveSet &as, const ShiftGroup &gr) {
    if (gr.n <= 0) return;
    const unsigned grid = (unsigned)gr.n;
    const int64_t per = (int64_t)4 * pl.Pp * pl.Pp;
    if (gr.wide) YK_SHIFT_CASES(k_l2l_wide, as.down_desc.p + gr.first * kDownDesc, pl.down_op.p + (gr.level - 1) * per, pl.Lc.p)
    else YK_SHIFT_CASES(k_l2l, as.down_desc.p + gr.first * kDownDesc, gr.nlev, gr.level, pl.down_op.p, pl.Lc.p)
    check_launch(ctx, "k_l2l");
}
#undef YK_SHIFT_CASES

}  // namespace yk
