// FP64 linear algebra of the boundary-MPS fit: Householder QR of the tall
// (chi * phys) x chi site matrices (the gauge moves of the one-site fit), norms,
// renormalisation, Philox initial guesses.
//
// QR is a tall-skinny (TSQR) tree: the rows are split into balanced blocks, each
// block is factored by one workgroup (Householder), the stacked n x n R factors
// are factored the same way level by level, and the explicit thin Q is formed
// top-down by applying each block's reflectors to its chunk of the parent Q.
// Up to 64 columns a block is at most QR_REG_ROWS rows in registers (k_qr_reg),
// else, and where the order of the sums must stay (QrArgs::keep_sums), at most
// QR_LDS / n rows in LDS (k_qr_leaf, k_qr_form).  Matrices with more than 64
// columns that do not fit one block fall back to a one-workgroup factorisation
// in global memory.
#include "kernels.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

namespace tnk {
namespace {

constexpr int QR_NT = 256;
constexpr int CQR_ROWS = 32;  // rows of a CholeskyQR pass staged in LDS at a time
constexpr int SUM_E = 8;      // entries per workgroup of the partial-sum reduction
constexpr int QR_LDS = 8192;  // complex doubles held by one workgroup (128 KiB)
constexpr int QR_G = QR_NT / 64;

struct MatDesc {
    const void *p; int esz; int64_t bs, rs, cs; int conj;
};
struct MatOut {
    void *p; int esz; int64_t bs, rs, cs; int conj;
};

__device__ inline double2 ld_c(const void *base, int esz, int64_t off, int conj) {
    double2 v;
    if (esz == 16) {
        v = reinterpret_cast<const double2 *>(base)[off];
    } else {
        const float2 f = reinterpret_cast<const float2 *>(base)[off];
        v.x = f.x; v.y = f.y;
    }
    if (conj) v.y = -v.y;
    return v;
}
__device__ inline void st_c(void *base, int esz, int64_t off, double2 v, int conj) {
    if (conj) v.y = -v.y;
    if (esz == 16) {
        reinterpret_cast<double2 *>(base)[off] = v;
    } else {
        reinterpret_cast<float2 *>(base)[off] = make_float2((float)v.x, (float)v.y);
    }
}
__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ inline double2 cmulc(double2 a, double2 b) {  // conj(a) * b
    return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

__device__ inline double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// Block sum over QR_NT threads; every thread receives the result.
__device__ inline double block_sum(double v, double *red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < QR_NT / 64; ++i) s += red[i];
    return s;
}

// Block maximum over QR_NT threads; every thread receives the result.
__device__ inline double block_max(double v, double *red) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double m = 0.0;
#pragma unroll
    for (int i = 0; i < QR_NT / 64; ++i) m = fmax(m, red[i]);
    return m;
}

// Below this sum of squares a column's norm is recomputed from values scaled
// by its largest modulus: squares of entries under ~1e-154 fall into the
// subnormal range (or to zero) and would give an inaccurate norm.
constexpr double HH_SMALL2 = 1e-280;

// In-place Householder factorisation of X (rows x n, leading dimension ld).
// After return: X[i][j], i >= j, holds reflector j normalised to v_j[0] = 1
// (the 1 stored on the diagonal); X[i][j], i < j, holds R; beta[j] = R[j][j];
// tau[j] = 2 / ||v_j||^2 = (|alpha| + sigma) / sigma, between 1 and 2 (0 for a
// zero column).  H_j = I - tau_j v_j v_j^H is Hermitian and unitary; A = H_0 ...
// H_{k-1} R.  With the normalised reflector nothing in the step scales like
// 1 / sigma^2, so columns whose remaining norm is far below the others' (the
// rank-deficient matrices of gauged site tensors) stay finite and exact.
__device__ void hh_factor(double2 *X, int rows, int n, int ld, double2 *beta, double *tau,
                          double *red, double2 *wpart) {
    const int t = threadIdx.x;
    const int kmax = rows < n ? rows : n;
    for (int j = 0; j < kmax; ++j) {
        double s = 0.0;
        for (int i = j + t; i < rows; i += QR_NT) {
            const double2 x = X[(int64_t)i * ld + j];
            s += x.x * x.x + x.y * x.y;
        }
        s = block_sum(s, red);
        double sigma = sqrt(s);
        if (s < HH_SMALL2) {  // uniform over the block
            double cm = 0.0;
            for (int i = j + t; i < rows; i += QR_NT) {
                const double2 x = X[(int64_t)i * ld + j];
                cm = fmax(cm, fmax(fabs(x.x), fabs(x.y)));
            }
            cm = block_max(cm, red);
            double s2 = 0.0;
            if (cm > 0.0) {
                for (int i = j + t; i < rows; i += QR_NT) {
                    const double2 x = X[(int64_t)i * ld + j];
                    const double xr = x.x / cm, xi = x.y / cm;
                    s2 += xr * xr + xi * xi;
                }
            }
            s2 = block_sum(s2, red);
            sigma = cm > 0.0 ? cm * sqrt(s2) : 0.0;
        }
        const double2 alpha = X[(int64_t)j * ld + j];
        const double aabs = hypot(alpha.x, alpha.y);
        __syncthreads();
        double tj = 0.0;
        double2 bj = make_double2(0.0, 0.0);
        if (sigma > 0.0) {
            const double2 ph = aabs > 0.0 ? make_double2(alpha.x / aabs, alpha.y / aabs) : make_double2(1.0, 0.0);
            const double d = aabs + sigma;  // |v_j[0]| before normalisation
            bj = make_double2(-ph.x * sigma, -ph.y * sigma);
            tj = d / sigma;
            // v_j[i] = x_i / (ph d) below the diagonal (divisions, not a
            // reciprocal: d may be subnormal)
            for (int i = j + 1 + t; i < rows; i += QR_NT) {
                const double2 x = X[(int64_t)i * ld + j];
                const double2 xc = cmulc(ph, x);  // conj(ph) x
                X[(int64_t)i * ld + j] = make_double2(xc.x / d, xc.y / d);
            }
            if (t == 0) X[(int64_t)j * ld + j] = make_double2(1.0, 0.0);
        }
        if (t == 0) { beta[j] = bj; tau[j] = tj; }
        __syncthreads();
        if (tj == 0.0) continue;
        const int g = t >> 6;
        for (int cb = j + 1; cb < n; cb += 64) {
            const int c = cb + (t & 63);
            double2 w = make_double2(0.0, 0.0);
            if (c < n) {
                for (int i = j + g; i < rows; i += QR_G) {
                    const double2 v = X[(int64_t)i * ld + j];
                    const double2 x = X[(int64_t)i * ld + c];
                    const double2 p = cmulc(v, x);
                    w.x += p.x; w.y += p.y;
                }
            }
            wpart[g * 64 + (t & 63)] = w;
            __syncthreads();
            if (c < n) {
                double2 ws = make_double2(0.0, 0.0);
#pragma unroll
                for (int q = 0; q < QR_G; ++q) { ws.x += wpart[q * 64 + (t & 63)].x; ws.y += wpart[q * 64 + (t & 63)].y; }
                ws.x *= tj; ws.y *= tj;
                for (int i = j + g; i < rows; i += QR_G) {
                    const double2 v = X[(int64_t)i * ld + j];
                    const double2 p = cmul(v, ws);
                    double2 &x = X[(int64_t)i * ld + c];
                    x.x -= p.x; x.y -= p.y;
                }
            }
            __syncthreads();
        }
    }
}

// Y <- H_0 ... H_{k-1} Y for Y (rows x nq, leading dim ldy); reflectors in V
// (rows x k part of a rows x ldv array), tau[k].
__device__ void hh_apply(double2 *Y, int rows, int nq, int ldy, const double2 *V, int ldv, int k,
                         const double *tau, double2 *wpart) {
    const int t = threadIdx.x;
    const int g = t >> 6;
    for (int j = k - 1; j >= 0; --j) {
        const double tj = tau[j];
        if (tj == 0.0) continue;
        for (int cb = 0; cb < nq; cb += 64) {
            const int c = cb + (t & 63);
            double2 w = make_double2(0.0, 0.0);
            if (c < nq) {
                for (int i = j + g; i < rows; i += QR_G) {
                    const double2 v = V[(int64_t)i * ldv + j];
                    const double2 y = Y[(int64_t)i * ldy + c];
                    const double2 p = cmulc(v, y);
                    w.x += p.x; w.y += p.y;
                }
            }
            wpart[g * 64 + (t & 63)] = w;
            __syncthreads();
            if (c < nq) {
                double2 ws = make_double2(0.0, 0.0);
#pragma unroll
                for (int q = 0; q < QR_G; ++q) { ws.x += wpart[q * 64 + (t & 63)].x; ws.y += wpart[q * 64 + (t & 63)].y; }
                ws.x *= tj; ws.y *= tj;
                for (int i = j + g; i < rows; i += QR_G) {
                    const double2 v = V[(int64_t)i * ldv + j];
                    const double2 p = cmul(v, ws);
                    double2 &y = Y[(int64_t)i * ldy + c];
                    y.x -= p.x; y.y -= p.y;
                }
            }
            __syncthreads();
        }
    }
}

struct LeafArgs {
    MatDesc in;              // level input (row i, col j), rows x n
    int rows, n, nb, top;
    char *ws; int64_t ws_bs;  // workspace base and per-batch stride (bytes)
    size_t v_off, t_off, b_off, rs_off;
    MatOut R; int want_r;    // top only: k x n
    const int *only_if;      // see QrArgs (register kernels)
};

__global__ void __launch_bounds__(QR_NT) k_qr_leaf(LeafArgs a) {
    extern __shared__ double2 lds[];
    __shared__ double red[QR_NT / 64];
    __shared__ double2 wpart[QR_NT];
    __shared__ double2 sbeta[128];  // k <= 90 whenever one block holds the matrix
    __shared__ double stau[128];
    const int blk = blockIdx.x;
    const int bt = blockIdx.y;
    const int r0 = (int)(((int64_t)blk * a.rows) / a.nb);
    const int r1 = (int)(((int64_t)(blk + 1) * a.rows) / a.nb);
    const int len = r1 - r0;
    const int n = a.n;
    double2 *X = lds;
    char *wb = a.ws + (int64_t)bt * a.ws_bs;
    const char *inb = reinterpret_cast<const char *>(a.in.p) + (int64_t)bt * a.in.bs * a.in.esz;
    for (int e = threadIdx.x; e < len * n; e += QR_NT) {
        const int i = e / n, j = e % n;
        X[e] = ld_c(inb, a.in.esz, (int64_t)(r0 + i) * a.in.rs + (int64_t)j * a.in.cs, a.in.conj);
    }
    __syncthreads();
    hh_factor(X, len, n, n, sbeta, stau, red, wpart);
    __syncthreads();
    const int k = len < n ? len : n;
    double2 *Vb = reinterpret_cast<double2 *>(wb + a.v_off) + (int64_t)r0 * n;
    for (int e = threadIdx.x; e < len * n; e += QR_NT) Vb[e] = X[e];
    double *tb = reinterpret_cast<double *>(wb + a.t_off) + (int64_t)blk * n;
    double2 *bb = reinterpret_cast<double2 *>(wb + a.b_off) + (int64_t)blk * n;
    for (int j = threadIdx.x; j < n; j += QR_NT) {
        tb[j] = j < k ? stau[j] : 0.0;
        bb[j] = j < k ? sbeta[j] : make_double2(0.0, 0.0);
    }
    if (!a.top) {
        double2 *Rb = reinterpret_cast<double2 *>(wb + a.rs_off) + (int64_t)blk * n * n;
        for (int e = threadIdx.x; e < n * n; e += QR_NT) {
            const int i = e / n, j = e % n;
            double2 v = make_double2(0.0, 0.0);
            if (i < k) {
                if (j == i) v = sbeta[i];
                else if (j > i) v = X[i * n + j];
            }
            Rb[e] = v;
        }
    } else if (a.want_r) {
        char *rb = reinterpret_cast<char *>(a.R.p) + (int64_t)bt * a.R.bs * a.R.esz;
        for (int e = threadIdx.x; e < k * n; e += QR_NT) {
            const int i = e / n, j = e % n;
            double2 v = make_double2(0.0, 0.0);
            if (j == i) v = sbeta[i];
            else if (j > i) v = X[i * n + j];
            st_c(rb, a.R.esz, (int64_t)i * a.R.rs + (int64_t)j * a.R.cs, v, a.R.conj);
        }
    }
}

struct FormArgs {
    int rows, n, nb, k, top, level0;
    char *ws; int64_t ws_bs;
    size_t v_off, t_off, b_off, x_off, q_off;  // x_off: parent Q ((nb n) x k), q_off: this level's Q
    MatOut out;                          // level 0 destination
    const int *only_if;                  // see QrArgs (register kernels)
};

__global__ void __launch_bounds__(QR_NT) k_qr_form(FormArgs a) {
    extern __shared__ double2 lds[];
    __shared__ double2 wpart[QR_NT];
    const int blk = blockIdx.x;
    const int bt = blockIdx.y;
    const int r0 = (int)(((int64_t)blk * a.rows) / a.nb);
    const int r1 = (int)(((int64_t)(blk + 1) * a.rows) / a.nb);
    const int len = r1 - r0;
    const int n = a.n, k = a.k;
    const int kb = len < n ? len : n;
    char *wb = a.ws + (int64_t)bt * a.ws_bs;
    double2 *Y = lds;  // len x k
    const double2 *X = a.top ? nullptr : reinterpret_cast<const double2 *>(wb + a.x_off);
    for (int e = threadIdx.x; e < len * k; e += QR_NT) {
        const int i = e / k, c = e % k;
        double2 v = make_double2(0.0, 0.0);
        if (i < kb) {
            if (a.top) v = make_double2(i == c ? 1.0 : 0.0, 0.0);
            else v = X[((int64_t)blk * n + i) * k + c];
        }
        Y[e] = v;
    }
    __syncthreads();
    const double2 *Vb = reinterpret_cast<const double2 *>(wb + a.v_off) + (int64_t)r0 * n;
    const double *tb = reinterpret_cast<const double *>(wb + a.t_off) + (int64_t)blk * n;
    hh_apply(Y, len, k, k, Vb, n, kb, tb, wpart);
    if (a.level0) {
        char *ob = reinterpret_cast<char *>(a.out.p) + (int64_t)bt * a.out.bs * a.out.esz;
        for (int e = threadIdx.x; e < len * k; e += QR_NT) {
            const int i = e / k, c = e % k;
            st_c(ob, a.out.esz, (int64_t)(r0 + i) * a.out.rs + (int64_t)c * a.out.cs, Y[e], a.out.conj);
        }
    } else {
        double2 *qb = reinterpret_cast<double2 *>(wb + a.q_off) + (int64_t)r0 * k;
        for (int e = threadIdx.x; e < len * k; e += QR_NT) qb[e] = Y[e];
    }
}

// The same level of the tree with the block in registers: a workgroup of NT
// threads is G = NT / NC row groups of NC lanes (NC = 16, 32 or 64 >= n), a lane
// holds one column of its group's rows, row i in register i / G of group i % G.
// A step is bound by its serial chain (a reciprocal square root, a division, one
// barrier), so everything else is kept off it: a group reads the pivot column's
// entries of its own rows from the owning lane (no LDS), and one reduction over
// the groups carries both the column's norm and its products with all other
// columns.  The reflector stays unnormalised in its column, p = (ph d, x_j+1, ..),
// d = |x_j| + sigma, with its factor f = ph / d in the column's lanes:
// v = conj(f) p, v_j = 1.  At the top of the tree the reflectors, still in
// registers, are applied to the identity in the same launch.  Measured against
// the LDS kernels (five barriers a step), Q and R: 128 x 64 237 for 600 us, 4096 x
// 64 1.46 for 3.69 ms, 128 x 32 122 for 346, 32 of 128 x 16 29 for 234, 64 x 16 24
// for 109; with the pivot column through shuffles or twice a step, and divisions and
// square roots of the library, 339, 2.08, 141, 48 and 46.  512 threads serve 64 columns as well as 256 (338 and 367 us; 1024: 474);
// up to 32 columns 256 are no slower than 512 and leave room for more blocks.
constexpr int QR_REG_ROWS = 128;
// A column whose sum of squares s is outside [REG_SMALL2, REG_LARGE2] is scaled to s
// near 1 for its step: the pivot's square (kept down to 2^-106 s), the column's
// products with columns of any other size and their quotients by its norm stay
// normal numbers.  (A pivot of subnormal square gave a phase off by 1e-12, and Q with
// it; columns of 1e-290 after ones of 1e-150 lost their R.)
constexpr double REG_SMALL2 = 1e-40, REG_LARGE2 = 1e20;
__device__ __forceinline__ bool out_of_range(double s) {  // s >= 0 or NaN: one comparison of the upper words
    constexpr unsigned lo = (unsigned)(__builtin_bit_cast(unsigned long long, REG_SMALL2) >> 32);
    constexpr unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, REG_LARGE2) >> 32);
    return (unsigned)(__builtin_bit_cast(unsigned long long, s) >> 32) - lo > hi - lo;
}

__device__ inline double lane_get(double v, int lane) {
    const int2 a = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(a.x, lane),
                                                __builtin_amdgcn_readlane(a.y, lane)));
}

// Column j's value in every lane of its group (j the same in all lanes).
template <int NC> __device__ __forceinline__ double2 column(double2 v, int j) {
    if constexpr (NC == 64) return make_double2(lane_get(v.x, j), lane_get(v.y, j));
    const int src = (threadIdx.x & 63 & ~(NC - 1)) | j;
    return make_double2(__shfl(v.x, src, 64), __shfl(v.y, src, 64));
}

// Lane K of each row of 16 lanes, to the whole row.
template <int K> __device__ __forceinline__ double row_lane(double v) {
    const int2 a = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(a.x, 0x150 + K, 0xf, 0xf, false),
                                                __builtin_amdgcn_mov_dpp(a.y, 0x150 + K, 0xf, 0xf, false)));
}
// 1 / sqrt(d) for d > 0 in the normal range: the hardware estimate r and one step of
// third order, r (1 + y / 2 + 3 y^2 / 8) with y = 1 - d r^2.
__device__ __forceinline__ double rsqrt3(double d) {
    const double r = __builtin_amdgcn_rsq(d);
    const double y = fma(-d * r, r, 1.0);
    return fma(r * y, fma(y, 0.375, 0.5), r);
}
// 1 / d for d > 0 in the normal range: the hardware estimate and two Newton steps.
__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
}
template <int J, int RT> __device__ __forceinline__ void row_lanes(const double2 (&V)[RT], double2 (&p)[RT]) {
#pragma unroll
    for (int r = 0; r < RT; ++r) p[r] = make_double2(row_lane<J>(V[r].x), row_lane<J>(V[r].y));
}
template <int RT> __device__ __forceinline__ void row_lanes(const double2 (&V)[RT], int j, double2 (&p)[RT]) {
    switch (j) {
        case 0: row_lanes<0>(V, p); break;
        case 1: row_lanes<1>(V, p); break;
        case 2: row_lanes<2>(V, p); break;
        case 3: row_lanes<3>(V, p); break;
        case 4: row_lanes<4>(V, p); break;
        case 5: row_lanes<5>(V, p); break;
        case 6: row_lanes<6>(V, p); break;
        case 7: row_lanes<7>(V, p); break;
        case 8: row_lanes<8>(V, p); break;
        case 9: row_lanes<9>(V, p); break;
        case 10: row_lanes<10>(V, p); break;
        case 11: row_lanes<11>(V, p); break;
        case 12: row_lanes<12>(V, p); break;
        case 13: row_lanes<13>(V, p); break;
        case 14: row_lanes<14>(V, p); break;
        default: row_lanes<15>(V, p); break;
    }
}
// Rows 0, 0, 2, 2 of 16 lanes of v, or rows 1, 1, 3, 3.
__device__ __forceinline__ double row_pair(double v, bool odd) {
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    const uint2 d = __builtin_bit_cast(uint2, v);
    const v2u x = __builtin_amdgcn_permlane16_swap(d.x, d.x, false, false);
    const v2u y = __builtin_amdgcn_permlane16_swap(d.y, d.y, false, false);
    return __builtin_bit_cast(double, odd ? make_uint2(x.y, y.y) : make_uint2(x.x, y.x));
}
// p = column j of V, every lane its own group's rows (j the same in all lanes): once
// a step, on the vector unit.  Through shuffles, once for the products and again for
// the update, this was most of a step.
template <int NC, int RT> __device__ __forceinline__ void pivot_column(const double2 (&V)[RT], int j, double2 (&p)[RT]) {
    if constexpr (NC == 64) {
#pragma unroll
        for (int r = 0; r < RT; ++r) p[r] = make_double2(lane_get(V[r].x, j), lane_get(V[r].y, j));
    } else if constexpr (NC == 32) {
        double2 half[RT];
        const bool odd = j >= 16;
#pragma unroll
        for (int r = 0; r < RT; ++r) half[r] = make_double2(row_pair(V[r].x, odd), row_pair(V[r].y, odd));
        row_lanes(half, j & 15, p);
    } else {
        row_lanes(V, j, p);
    }
}

template <int NC, int NT> struct QrRegShared {
    double2 part[2][NT / 64][NC];  // [parity of the reduction][wave][column]
    double2 row[2][NC];      // the pivot row
};

// Adds the row groups of a wave (its lanes of equal column): halves, then rows of 16.
__device__ __forceinline__ double half_add(double v) {
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    const uint2 d = __builtin_bit_cast(uint2, v);
    const v2u x = __builtin_amdgcn_permlane32_swap(d.x, d.x, false, false);
    const v2u y = __builtin_amdgcn_permlane32_swap(d.y, d.y, false, false);
    return __builtin_bit_cast(double, make_uint2(x.x, y.x)) + __builtin_bit_cast(double, make_uint2(x.y, y.y));
}
template <int NC> __device__ __forceinline__ double2 group_add(double2 v) {
    if constexpr (NC < 64) v = make_double2(half_add(v.x), half_add(v.y));
    if constexpr (NC < 32)
        v = make_double2(row_pair(v.x, false) + row_pair(v.x, true), row_pair(v.y, false) + row_pair(v.y, true));
    return v;
}

// p = 0 in the rows i = g + G r < lo (lo <= NC, so only the first registers have any).
template <int NC, int NT, int RT>
__device__ __forceinline__ void reg_mask(double2 (&p)[RT], int lo) {
    constexpr int G = NT / NC;
    const int g = threadIdx.x / NC;
#pragma unroll
    for (int r = 0; r < RT; ++r)
        if (r * G < NC) {
            const bool live = g + G * r >= lo;
            p[r] = make_double2(live ? p[r].x : 0.0, live ? p[r].y : 0.0);
        }
}

// sum_i conj(p_i) y_i over the wave's rows.
template <int NC, int RT>
__device__ __forceinline__ double2 reg_dot(const double2 (&p)[RT], const double2 (&Y)[RT]) {
    double2 s[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        double2 &a = s[r & 1];
        a.x = fma(p[r].x, Y[r].x, a.x);
        a.y = fma(p[r].x, Y[r].y, a.y);
        a.x = fma(p[r].y, Y[r].y, a.x);
        a.y = fma(-p[r].y, Y[r].x, a.y);
    }
    return group_add<NC>(make_double2(s[0].x + s[1].x, s[0].y + s[1].y));
}

// y_i -= p_i u.
template <int RT>
__device__ __forceinline__ void reg_take(const double2 (&p)[RT], double2 (&Y)[RT], double2 u) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        Y[r].x = fma(-p[r].x, u.x, Y[r].x);
        Y[r].y = fma(-p[r].x, u.y, Y[r].y);
        Y[r].x = fma(p[r].y, u.y, Y[r].x);
        Y[r].y = fma(-p[r].y, u.x, Y[r].y);
    }
}

// Householder steps on X; the lanes of column j end with R[j][j] in beta, tau_j
// and f_j.  A column out of range is scaled by a power of two (its reflector does not
// change with scale) and its step taken again; one that is still too small for its
// squares after three times 2^400 is zero, with tau = 0.
template <int NC, int NT, int RT>
__device__ __forceinline__ void reg_factor(double2 (&X)[RT], int rows, int n, double2 &beta, double &tau, double2 &fac,
                                           QrRegShared<NC, NT> &sh) {
    constexpr int G = NT / NC;
    const int col = threadIdx.x % NC, g = threadIdx.x / NC, w = threadIdx.x >> 6;
    beta = make_double2(0.0, 0.0);
    fac = make_double2(0.0, 0.0);
    tau = 0.0;
    const int kmax = rows < n ? rows : n;
    int pb = 0, ups = 0, ex = 0;  // scalings of this column, and their exponent
    for (int j = 0; j < kmax;) {
        pb ^= 1;
        double2 p[RT];
        pivot_column<NC>(X, j, p);
        reg_mask<NC, NT>(p, j + 1);
        const double2 part = reg_dot<NC>(p, X);
        if ((threadIdx.x & 63) < NC) sh.part[pb][w][col] = part;
        const int rj = j / G;  // the pivot row's register
        double2 mine = make_double2(0.0, 0.0);
#pragma unroll
        for (int r = 0; r < RT; ++r)
            if (r * G < NC) mine = make_double2(r == rj ? X[r].x : mine.x, r == rj ? X[r].y : mine.y);
        if (g == j % G) sh.row[pb][col] = mine;
        __syncthreads();
        double2 dot = make_double2(0.0, 0.0);
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NT / 64; ++q) {
            const double2 d = sh.part[pb][q][col];
            dot.x += d.x;
            dot.y += d.y;
            s += sh.part[pb][q][j].x;
        }
        const double2 xj = sh.row[pb][col], alpha = sh.row[pb][j];
        const double a2 = alpha.x * alpha.x + alpha.y * alpha.y;
        s += a2;
        // s is the same in every thread, and so is every branch on it
        if (out_of_range(s) && ups < 4 && s < INFINITY) {
            if (s < HH_SMALL2 && ups == 3) {
                ups = ex = 0;
                ++j;
                continue;
            }
            const int e = s < HH_SMALL2 ? 400 : -(ilogb(s) / 2);
            ++ups;
            ex += e;
            const double up = ldexp(1.0, e);
#pragma unroll
            for (int r = 0; r < RT; ++r)
                if (col == j && g + G * r >= j) { X[r].x *= up; X[r].y *= up; }
            continue;
        }
        // an alpha below the rounding of sigma counts as zero (its square may underflow)
        const bool some = a2 > s * 0x1p-106;
        const double is = rsqrt3(s), sigma = s * is;
        const double ia = some ? rsqrt3(a2) : 0.0, d = a2 * ia + sigma, id = recip(d);
        // u = tau conj(f) v^H x_c with v^H x_c = x_jc + f sum_{i > j} conj(x_ij) x_ic:
        // tau |f|^2 = 1 / (sigma d), tau conj(f) = conj(ph) / sigma
        const double2 ph = make_double2(some ? alpha.x * ia : 1.0, alpha.y * ia);
        const double isd = is * id;
        const double2 px = cmulc(ph, xj);
        const double2 u = make_double2(col > j ? fma(px.x, is, dot.x * isd) : 0.0,
                                       col > j ? fma(px.y, is, dot.y * isd) : 0.0);
        if (col == j) {
            beta = make_double2(ldexp(-ph.x * sigma, -ex), ldexp(-ph.y * sigma, -ex));
            tau = d * is;
            fac = make_double2(ph.x * id, ph.y * id);
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
            if (r * G < NC) {  // the reflector's first entry
                const bool first = g == j % G && r == rj, at = first && col == j;
                p[r] = make_double2(first ? ph.x * d : p[r].x, first ? ph.y * d : p[r].y);
                X[r] = make_double2(at ? ph.x * d : X[r].x, at ? ph.y * d : X[r].y);
            }
        reg_take(p, X, u);
        ups = ex = 0;
        ++j;
    }
}

// Y <- H_0 ... H_{k-1} Y, the reflectors in V (lanes of column j, with tau and f).
template <int NC, int NT, int RT>
__device__ __forceinline__ void reg_apply(double2 (&Y)[RT], const double2 (&V)[RT], int k, double tau, double2 fac,
                                          QrRegShared<NC, NT> &sh) {
    const int col = threadIdx.x % NC, w = threadIdx.x >> 6;
    const double t2 = tau * (fac.x * fac.x + fac.y * fac.y);  // tau conj(f) f
    int pb = 0;
    for (int j = k - 1; j >= 0; --j) {
        const double tj = column<NC>(make_double2(t2, 0.0), j).x;
        if (__builtin_amdgcn_readfirstlane(tj == 0.0)) continue;  // the same in every thread
        pb ^= 1;
        double2 p[RT];
        pivot_column<NC>(V, j, p);
        reg_mask<NC, NT>(p, j);
        const double2 part = reg_dot<NC>(p, Y);
        if ((threadIdx.x & 63) < NC) sh.part[pb][w][col] = part;
        __syncthreads();
        double2 ws = make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < NT / 64; ++q) {
            const double2 d = sh.part[pb][q][col];
            ws.x += d.x;
            ws.y += d.y;
        }
        reg_take(p, Y, make_double2(tj * ws.x, tj * ws.y));
    }
}

template <int NC, int NT, int RT>
__device__ __forceinline__ void reg_store_q(const FormArgs &f, const double2 (&Y)[RT], int r0, int len, char *wb) {
    constexpr int G = NT / NC;
    const int col = threadIdx.x % NC, g = threadIdx.x / NC;
    char *ob = f.level0 ? reinterpret_cast<char *>(f.out.p) + (int64_t)blockIdx.y * f.out.bs * f.out.esz : nullptr;
    double2 *qb = reinterpret_cast<double2 *>(wb + f.q_off);
    if (col >= f.k) return;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int i = g + G * r;
        if (i >= len) continue;
        if (ob) st_c(ob, f.out.esz, (int64_t)(r0 + i) * f.out.rs + (int64_t)col * f.out.cs, Y[r], f.out.conj);
        else qb[(int64_t)(r0 + i) * f.k + col] = Y[r];
    }
}

// Factors one block of a level; at the top also forms its Q (f).
template <int NC, int NT, int RT, bool TOP>
__global__ void __launch_bounds__(NT, NT / 256) k_qr_reg(LeafArgs a, FormArgs f) {
    __shared__ QrRegShared<NC, NT> sh;
    constexpr int G = NT / NC;
    const int blk = blockIdx.x, bt = blockIdx.y, n = a.n;
    if (a.only_if && !(a.only_if[bt] & 4)) return;  // uniform over the block
    const int col = threadIdx.x % NC, g = threadIdx.x / NC;
    const int r0 = (int)(((int64_t)blk * a.rows) / a.nb);
    const int r1 = (int)(((int64_t)(blk + 1) * a.rows) / a.nb);
    const int len = r1 - r0, k = len < n ? len : n;
    char *wb = a.ws + (int64_t)bt * a.ws_bs;
    const char *inb = reinterpret_cast<const char *>(a.in.p) + (int64_t)bt * a.in.bs * a.in.esz;
    double2 X[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int i = g + G * r;
        X[r] = i < len && col < n ? ld_c(inb, a.in.esz, (int64_t)(r0 + i) * a.in.rs + (int64_t)col * a.in.cs, a.in.conj)
                                  : make_double2(0.0, 0.0);
    }
    double2 beta, fac;
    double tau;
    reg_factor<NC, NT, RT>(X, len, n, beta, tau, fac, sh);
    // R: beta on the diagonal, the registers above it
    if (col < n && (!TOP || a.want_r)) {
        double2 *Rb = TOP ? nullptr : reinterpret_cast<double2 *>(wb + a.rs_off) + (int64_t)blk * n * n;
        char *rb = TOP ? reinterpret_cast<char *>(a.R.p) + (int64_t)bt * a.R.bs * a.R.esz : nullptr;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int i = g + G * r;
            if (i >= (TOP ? k : n)) continue;
            const bool diag = i < k && col == i, up = i < k && col > i;
            const double2 v = make_double2(diag ? beta.x : up ? X[r].x : 0.0, diag ? beta.y : up ? X[r].y : 0.0);
            if (TOP) st_c(rb, a.R.esz, (int64_t)i * a.R.rs + (int64_t)col * a.R.cs, v, a.R.conj);
            else Rb[i * n + col] = v;
        }
    }
    if constexpr (TOP) {
        double2 Y[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) Y[r] = make_double2(g + G * r == col && col < k ? 1.0 : 0.0, 0.0);
        __syncthreads();  // the last step's reads of the partial sums
        reg_apply<NC, NT, RT>(Y, X, k, tau, fac, sh);
        reg_store_q<NC, NT, RT>(f, Y, r0, len, wb);
    } else {
        if (col >= n) return;
        double2 *Vb = reinterpret_cast<double2 *>(wb + a.v_off) + (int64_t)r0 * n;
#pragma unroll
        for (int r = 0; r < RT; ++r)
            if (g + G * r < len) Vb[(int64_t)(g + G * r) * n + col] = X[r];
        if (g == 0) {
            reinterpret_cast<double *>(wb + a.t_off)[(int64_t)blk * n + col] = tau;
            reinterpret_cast<double2 *>(wb + a.b_off)[(int64_t)blk * n + col] = fac;
        }
    }
}

// Applies the reflectors of one block below the top to its chunk of the parent Q.
template <int NC, int NT, int RT>
__global__ void __launch_bounds__(NT, NT / 256) k_qr_reg_form(FormArgs f) {
    __shared__ QrRegShared<NC, NT> sh;
    constexpr int G = NT / NC;
    const int blk = blockIdx.x, n = f.n, k = f.k;
    if (f.only_if && !(f.only_if[blockIdx.y] & 4)) return;  // uniform over the block
    const int col = threadIdx.x % NC, g = threadIdx.x / NC;
    const int r0 = (int)(((int64_t)blk * f.rows) / f.nb);
    const int r1 = (int)(((int64_t)(blk + 1) * f.rows) / f.nb);
    const int len = r1 - r0, kb = len < n ? len : n;
    char *wb = f.ws + (int64_t)blockIdx.y * f.ws_bs;
    const double2 *Vb = reinterpret_cast<const double2 *>(wb + f.v_off) + (int64_t)r0 * n;
    const double2 *P = reinterpret_cast<const double2 *>(wb + f.x_off);
    double2 V[RT], Y[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int i = g + G * r;
        V[r] = i < len && col < n ? Vb[(int64_t)i * n + col] : make_double2(0.0, 0.0);
        Y[r] = i < kb && col < k ? P[((int64_t)blk * n + i) * k + col] : make_double2(0.0, 0.0);
    }
    const double tau = col < n ? reinterpret_cast<const double *>(wb + f.t_off)[(int64_t)blk * n + col] : 0.0;
    const double2 fac = col < n ? reinterpret_cast<const double2 *>(wb + f.b_off)[(int64_t)blk * n + col]
                                : make_double2(0.0, 0.0);
    reg_apply<NC, NT, RT>(Y, V, kb, tau, fac, sh);
    reg_store_q<NC, NT, RT>(f, Y, r0, len, wb);
}

// One level of the tree: columns rounded up to 16, 32 or 64 lanes, registers for
// blocks of at most 32, 64 or 128 rows.
template <int NC, int NT, int ROWS> void launch_reg_rows(const LeafArgs *a, const FormArgs &f, dim3 g, hipStream_t s) {
    constexpr int R = ROWS * NC / NT;
    const dim3 b(NT);
    if (!a) hipLaunchKernelGGL((k_qr_reg_form<NC, NT, R>), g, b, 0, s, f);
    else if (a->top) hipLaunchKernelGGL((k_qr_reg<NC, NT, R, true>), g, b, 0, s, *a, f);
    else hipLaunchKernelGGL((k_qr_reg<NC, NT, R, false>), g, b, 0, s, *a, f);
}
template <int NC, int NT> void launch_reg_level(const LeafArgs *a, const FormArgs &f, int rows_per_block, dim3 g,
                                                hipStream_t s) {
    if (rows_per_block <= 32) launch_reg_rows<NC, NT, 32>(a, f, g, s);
    else if (rows_per_block <= 64) launch_reg_rows<NC, NT, 64>(a, f, g, s);
    else launch_reg_rows<NC, NT, QR_REG_ROWS>(a, f, g, s);
}

void launch_reg(const LeafArgs *a, const FormArgs &f, int n, int rows_per_block, dim3 g, hipStream_t s) {
    if (n <= 16) launch_reg_level<16, 256>(a, f, rows_per_block, g, s);
    else if (n <= 32) launch_reg_level<32, 256>(a, f, rows_per_block, g, s);
    else launch_reg_level<64, 512>(a, f, rows_per_block, g, s);
}

// Fallback: one workgroup per matrix, matrix in global workspace.
struct GlobalQrArgs {
    MatDesc in; int m, n;
    char *ws; int64_t ws_bs;
    size_t w_off, y_off, t_off, b_off;
    MatOut Q; MatOut R; int want_r;
    int batch;
    const int *only_if;  // optional [batch]: factor only the items whose flag has bit 4 set
};

// One workgroup per matrix; the workgroups loop over the batch (workspace slot
// = blockIdx.x), skipping the items not flagged in only_if when it is given.
__global__ void __launch_bounds__(QR_NT) k_qr_global(GlobalQrArgs a) {
    __shared__ double red[QR_NT / 64];
    __shared__ double2 wpart[QR_NT];
    const int m = a.m, n = a.n, k = m < n ? m : n;
    char *wb = a.ws + (int64_t)blockIdx.x * a.ws_bs;
    double2 *X = reinterpret_cast<double2 *>(wb + a.w_off);
    double2 *Y = reinterpret_cast<double2 *>(wb + a.y_off);
    double *tau = reinterpret_cast<double *>(wb + a.t_off);
    double2 *beta = reinterpret_cast<double2 *>(wb + a.b_off);
    for (int bt = blockIdx.x; bt < a.batch; bt += gridDim.x) {
        if (a.only_if && !(a.only_if[bt] & 4)) continue;  // uniform over the block
        const char *inb = reinterpret_cast<const char *>(a.in.p) + (int64_t)bt * a.in.bs * a.in.esz;
        __syncthreads();  // the previous item's last reads of the workspace
        for (int64_t e = threadIdx.x; e < (int64_t)m * n; e += QR_NT) {
            const int i = (int)(e / n), j = (int)(e % n);
            X[e] = ld_c(inb, a.in.esz, (int64_t)i * a.in.rs + (int64_t)j * a.in.cs, a.in.conj);
        }
        __syncthreads();
        hh_factor(X, m, n, n, beta, tau, red, wpart);
        __syncthreads();
        for (int64_t e = threadIdx.x; e < (int64_t)m * k; e += QR_NT) {
            const int i = (int)(e / k), c = (int)(e % k);
            Y[e] = make_double2(i == c ? 1.0 : 0.0, 0.0);
        }
        __syncthreads();
        hh_apply(Y, m, k, k, X, n, k, tau, wpart);
        char *qb = reinterpret_cast<char *>(a.Q.p) + (int64_t)bt * a.Q.bs * a.Q.esz;
        for (int64_t e = threadIdx.x; e < (int64_t)m * k; e += QR_NT) {
            const int i = (int)(e / k), c = (int)(e % k);
            st_c(qb, a.Q.esz, (int64_t)i * a.Q.rs + (int64_t)c * a.Q.cs, Y[e], a.Q.conj);
        }
        if (a.want_r) {
            char *rb = reinterpret_cast<char *>(a.R.p) + (int64_t)bt * a.R.bs * a.R.esz;
            for (int64_t e = threadIdx.x; e < (int64_t)k * n; e += QR_NT) {
                const int i = (int)(e / n), j = (int)(e % n);
                double2 v = make_double2(0.0, 0.0);
                if (j == i) v = beta[i];
                else if (j > i) v = X[(int64_t)i * n + j];
                st_c(rb, a.R.esz, (int64_t)i * a.R.rs + (int64_t)j * a.R.cs, v, a.R.conj);
            }
        }
    }
}

struct TsqrLevel {
    int rows, nb;
    size_t v_off, t_off, b_off, rs_off, q_off;  // byte offsets inside one batch item's workspace
};

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Blocks of the tree in registers: the block's columns are one per lane.
bool use_reg(int n, int keep_sums) { return n <= 64 && !keep_sums; }

// Plans the TSQR tree; returns per-batch workspace bytes.
size_t plan_tsqr(int m, int n, int keep_sums, std::vector<TsqrLevel> &lv) {
    lv.clear();
    const int rb = use_reg(n, keep_sums) ? QR_REG_ROWS : QR_LDS / n;
    int rows = m;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    while (true) {
        TsqrLevel L;
        L.rows = rows;
        L.nb = (rows + rb - 1) / rb;
        if (L.nb < 1) L.nb = 1;
        L.v_off = take((size_t)rows * n * 16);
        L.t_off = take((size_t)L.nb * n * 8);
        L.b_off = take((size_t)L.nb * n * 16);
        L.rs_off = (L.nb > 1) ? take((size_t)L.nb * n * n * 16) : 0;
        L.q_off = lv.empty() ? 0 : take((size_t)rows * n * 16);
        lv.push_back(L);
        if (L.nb == 1) break;
        rows = L.nb * n;
    }
    return off;
}

bool use_tsqr(int m, int n) { return n <= 64 || (int64_t)m * n <= QR_LDS; }

size_t global_qr_bytes(int m, int n, size_t *w, size_t *y, size_t *t, size_t *b) {
    const int k = m < n ? m : n;
    size_t off = 0;
    *w = off; off += align256((size_t)m * n * 16);
    *y = off; off += align256((size_t)m * k * 16);
    *t = off; off += align256((size_t)k * 8);
    *b = off; off += align256((size_t)k * 16);
    return off;
}

// ---------------------------------------------------------------- CholeskyQR
// Matrices of up to 64 columns, padded to P = 1..4 blocks of 16: the Gram
// matrices, the triangular products and the block steps of the Cholesky
// factorisation run on v_mfma_f64_16x16x4 (four real products per complex one),
// with the operands in LDS as planar (re, im) arrays.  A lane l of a fragment
// holds (row or column l % 16, k = l / 16); a result register r holds (row 4 r +
// l / 16, column l % 16).
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int CB = 16;         // block edge
template <int LD> struct CMat { double (*re)[LD]; double (*im)[LD]; };
template <int P> constexpr int CLD = CB * P + 2;  // padded LDS row of P blocks
struct CAcc { v4d re, im; };

__device__ __forceinline__ void acc_zero(CAcc &c) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c.re[r] = c.im[r] = 0.0;
}
__device__ __forceinline__ void acc_mma(CAcc &c, double ar, double ai, double br, double bi) {
    c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, c.re, 0, 0, 0);
    c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, c.im, 0, 0, 0);
    c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, bi, c.re, 0, 0, 0);
    c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, c.im, 0, 0, 0);
}
// c += op(A) B over 16 k indices: op(A)(m, k) = A[ar + m][ac + k], or with HERM
// conj(A[ar + k][ac + m]); B(k, n) = B[br + k][bc + n].
template <bool HERM, int LA, int LB>
__device__ __forceinline__ void acc_block(CAcc &c, CMat<LA> A, int ar, int ac, CMat<LB> B, int br, int bc, int lane) {
    const int x = lane & 15, q = lane >> 4;
#pragma unroll
    for (int k = 0; k < CB; k += 4) {
        const int i = HERM ? ar + k + q : ar + x, j = HERM ? ac + x : ac + k + q;
        const double pr = A.re[i][j], pi = A.im[i][j];
        acc_mma(c, pr, HERM ? -pi : pi, B.re[br + k + q][bc + x], B.im[br + k + q][bc + x]);
    }
}
// M[r0.., c0..] (a 16 x 16 block) = s * c, or += with ADD.
template <bool ADD, int LD>
__device__ __forceinline__ void acc_store(const CAcc &c, CMat<LD> M, int r0, int c0, double s, int lane) {
    const int x = lane & 15, q = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double &re = M.re[r0 + 4 * r + q][c0 + x], &im = M.im[r0 + 4 * r + q][c0 + x];
        re = (ADD ? re : 0.0) + s * c.re[r];
        im = (ADD ? im : 0.0) + s * c.im[r];
    }
}

// out[a] = lane 16 a + x of v, in every lane (x = lane % 16): swaps of half waves,
// then of rows of 16 lanes.
__device__ __forceinline__ void rows4(double v, double (&out)[4]) {
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    const uint2 d = __builtin_bit_cast(uint2, v);
    unsigned int o[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const unsigned int x = h ? d.y : d.x;
        const v2u p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        const v2u a = __builtin_amdgcn_permlane16_swap(p.x, p.x, false, false);
        const v2u b = __builtin_amdgcn_permlane16_swap(p.y, p.y, false, false);
        o[h][0] = a.x; o[h][1] = a.y; o[h][2] = b.x; o[h][3] = b.y;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = __builtin_bit_cast(double, make_uint2(o[0][i], o[1][i]));
}

// One wave: a 16 x 16 Hermitian block w (in full) becomes R (upper) and e becomes
// R^{-H} e: elimination on the pair [w | e] in panels of four rows.  Each lane
// carries the panel's four rows of its column of both halves through the panel's own
// elimination (the four pivots, one after another, in every lane alike); the rows
// below take the rank-4 update as one matrix instruction per real product, whose
// operands are the panel's rows as the accumulator layout holds them.  A pivot
// below cl is raised to it (returns true).  Bound by the issue of one wave: some
// 220 instructions and 8 matrix products a panel.
template <int PN, int A>
__device__ __forceinline__ void diag_pivot(double (&w)[2][4], double (&e)[2][4], double cl, bool &bad, int x) {
    double d = row_lane<4 * PN + A>(w[0][A]);
    if (!(d >= cl)) {  // the same in every lane
        bad = true;
        d = cl > 0.0 ? cl : 1e-300;
    }
    const double rs = rsqrt3(d);
    w[0][A] = x == 4 * PN + A ? d * rs : w[0][A] * rs;
    w[1][A] *= rs;
    e[0][A] *= rs;
    e[1][A] *= rs;
    auto below = [&](auto bc) {
        constexpr int B = decltype(bc)::value;
        if constexpr (B < 4) {
            const double cr = row_lane<4 * PN + (B & 3)>(w[0][A]), ci = row_lane<4 * PN + (B & 3)>(w[1][A]);
            w[0][B] = fma(-cr, w[0][A], fma(-ci, w[1][A], w[0][B]));
            w[1][B] = fma(-cr, w[1][A], fma(ci, w[0][A], w[1][B]));
            e[0][B] = fma(-cr, e[0][A], fma(-ci, e[1][A], e[0][B]));
            e[1][B] = fma(-cr, e[1][A], fma(ci, e[0][A], e[1][B]));
        }
    };
    below(std::integral_constant<int, A + 1>());
    below(std::integral_constant<int, A + 2>());
    below(std::integral_constant<int, A + 3>());
}
template <int PN>
__device__ __forceinline__ void diag_panel(CAcc &w, CAcc &e, CAcc &R, CAcc &F, double cl, bool &bad, int lane) {
    const int x = lane & 15, q = lane >> 4;
    double wp[2][4], ep[2][4];
    rows4(w.re[PN], wp[0]);
    rows4(w.im[PN], wp[1]);
    rows4(e.re[PN], ep[0]);
    rows4(e.im[PN], ep[1]);
    diag_pivot<PN, 0>(wp, ep, cl, bad, x);
    diag_pivot<PN, 1>(wp, ep, cl, bad, x);
    diag_pivot<PN, 2>(wp, ep, cl, bad, x);
    diag_pivot<PN, 3>(wp, ep, cl, bad, x);
    auto own = [&](double a, double b, double c, double d) {
        const double lo = q == 0 ? a : b, hi = q == 2 ? c : d;
        return q < 2 ? lo : hi;
    };
    const double wr = own(wp[0][0], wp[0][1], wp[0][2], wp[0][3]), wi = own(wp[1][0], wp[1][1], wp[1][2], wp[1][3]);
    const double er = own(ep[0][0], ep[0][1], ep[0][2], ep[0][3]), ei = own(ep[1][0], ep[1][1], ep[1][2], ep[1][3]);
    R.re[PN] = wr; R.im[PN] = wi;
    F.re[PN] = er; F.im[PN] = ei;
    if constexpr (PN < 3) {  // (the rows of finished panels are overwritten with what is not read again)
        acc_mma(w, -wr, wi, wr, wi);
        __builtin_amdgcn_sched_barrier(0);  // the next panel waits for these four
        acc_mma(e, -wr, wi, er, ei);
        diag_panel<PN + 1>(w, e, R, F, cl, bad, lane);
    }
}
template <int LD> __device__ __forceinline__ void acc_load(CAcc &c, CMat<LD> M, int r0, int c0, int lane) {
    const int x = lane & 15, q = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        c.re[r] = M.re[r0 + 4 * r + q][c0 + x];
        c.im[r] = M.im[r0 + 4 * r + q][c0 + x];
    }
}

// W (P x P blocks, the diagonal blocks Hermitian in full, the blocks above them
// filled) = R^H R: R replaces W's upper part and E receives R^{-1} (upper blocks).
// NW >= P waves; returns whether a pivot was raised (wave 0).  Right-looking over
// panels of 16: P waves factor the diagonal block, all alike, each with one of the
// P blocks that R_pp^{-H} is due on as its right half: the identity (its result is
// E_pp^H), the rest of the panel's row of W, the column of E above it (transposed).
// So the panel needs no products of its own; the trailing updates are spread over
// all waves.  With SAME, E is W (P <= 2): R is not kept.
template <int P, int NW, bool SAME, int LD>
__device__ __forceinline__ bool chol_blocks(CMat<LD> W, CMat<LD> E, double cl, int wave, int lane) {
    static_assert(NW >= P && NW > 1 && (!SAME || P <= 2), "chol_blocks");
    const int x = lane & 15, q = lane >> 4;
    bool bad = false;
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
        const int o = CB * p;
        const int j = wave <= P - 1 - p ? p + wave : P - 1 - wave;  // right half: block pj of W, or of E for j < p
        CAcc w, e;
        if (wave < P) {
            acc_load(w, W, o, o, lane);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * r + q;
                if (j > p) {
                    e.re[r] = W.re[o + i][CB * j + x];
                    e.im[r] = W.im[o + i][CB * j + x];
                } else if (j < p) {
                    e.re[r] = E.re[CB * j + x][o + i];
                    e.im[r] = -E.im[CB * j + x][o + i];
                } else {
                    e.re[r] = i == x ? 1.0 : 0.0;
                    e.im[r] = 0.0;
                }
            }
        }
        __syncthreads();
        if (wave < P) {
            CAcc R, F;
            diag_panel<0>(w, e, R, F, cl, bad, lane);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * r + q;
                if (j > p) {
                    W.re[o + i][CB * j + x] = F.re[r];
                    W.im[o + i][CB * j + x] = F.im[r];
                } else if (j < p) {
                    E.re[CB * j + x][o + i] = F.re[r];
                    E.im[CB * j + x][o + i] = -F.im[r];
                } else {
                    if constexpr (!SAME) {
                        W.re[o + i][o + x] = x >= i ? R.re[r] : 0.0;
                        W.im[o + i][o + x] = x > i ? R.im[r] : 0.0;
                    }
                    E.re[o + x][o + i] = x <= i ? F.re[r] : 0.0;
                    E.im[o + x][o + i] = x <= i ? -F.im[r] : 0.0;
                }
            }
        }
        __syncthreads();
        if (p == P - 1) break;
        if constexpr (SAME && P == 2) {  // E_01 takes the place of R_01 once both products have read it
            CAcc c;
            acc_zero(c);
            if (wave == 0) acc_block<true>(c, W, 0, CB, W, 0, CB, lane);
            if (wave == 1) acc_block<false>(c, E, 0, 0, W, 0, CB, lane);
            __syncthreads();
            if (wave == 0) acc_store<true>(c, W, CB, CB, -1.0, lane);
            if (wave == 1) acc_store<false>(c, E, 0, CB, -1.0, lane);
        } else {
            int t = 0;
            for (int i = p + 1; i < P; ++i) {
                for (int jj = i; jj < P; ++jj) {  // W_ij -= R_pi^H R_pj
                    if (t++ % NW != wave) continue;
                    CAcc c;
                    acc_zero(c);
                    acc_block<true>(c, W, o, CB * i, W, o, CB * jj, lane);
                    acc_store<true>(c, W, CB * i, CB * jj, -1.0, lane);
                }
                for (int k = 0; k <= p; ++k) {    // E_ki -= E_kp R_pi (nothing there yet at k = p)
                    if (t++ % NW != wave) continue;
                    CAcc c;
                    acc_zero(c);
                    acc_block<false>(c, E, CB * k, o, W, o, CB * i, lane);
                    if (k < p) acc_store<true>(c, E, CB * k, CB * i, -1.0, lane);
                    else acc_store<false>(c, E, CB * k, CB * i, -1.0, lane);
                }
            }
        }
        __syncthreads();
    }
    return bad;
}

// Mean diagonal of the n x n matrix in W (every thread gets it), then the shift
// and a diagonal of that mean on the padding.  Ends with a barrier.
template <int LD>
__device__ __forceinline__ double chol_scale(CMat<LD> W, int n, int np, double shift, double *red) {
    const int t = threadIdx.x;
    if (t < 64) {
        double v = t < n ? W.re[t][t] : 0.0;
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        const double scale = v / n;
        if (t < n) W.re[t][t] += shift * scale;
        else if (t < np) W.re[t][t] = scale > 0.0 ? scale : 1.0;
        if (t == 0) *red = scale;
    }
    __syncthreads();
    return *red;
}

// Cholesky factor and inverse, one workgroup per matrix (see launch_chol_inv).
// A 64 x 64 call takes 24 us, 32 x 32 11.3; with one pivot at a time, its row through
// shuffles, and the products of the panel apart, 33 and 12.8.  A diagonal block is
// 7700 cycles, the trailing updates of a 64 x 64 matrix 12700 in all, the load and
// the store 7300.  Adding up 16 partial Gram matrices here instead of in a launch
// before it costs more (16.8 for 14 us): one CU reads them.
template <int P, int NW>
__global__ void __launch_bounds__(64 * NW, 2) k_chol_inv(const double2 *G, int n, double shift,
                                                        double clamp, double2 *Rinv, double2 *Rf, int *flags,
                                                        int first) {
    __shared__ double sm[4][CB * P][CLD<P>];
    __shared__ double red;
    const CMat<CLD<P>> W{sm[0], sm[1]}, E{sm[2], sm[3]};
    const int b = blockIdx.x, t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int64_t nn = (int64_t)n * n;
    constexpr int NP = CB * P, NT = 64 * NW, PER = (NP * NP + NT - 1) / NT;
    double2 g[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        // only the upper triangle is given; elsewhere the first element stands in
        const int e = t + NT * u, i = e / NP, j = e % NP;
        g[u] = G[b * nn + (j >= i && j < n ? i * n + j : 0)];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = t + NT * u, i = e / NP, j = e % NP;
        if (j < i || i >= NP) continue;
        const double2 v = j < n ? g[u] : make_double2(0.0, 0.0);
        W.re[i][j] = v.x;
        W.im[i][j] = i == j ? 0.0 : v.y;
        if (j > i && j / CB == i / CB) {
            W.re[j][i] = v.x;
            W.im[j][i] = -v.y;
        }
    }
    __syncthreads();
    const double scale = chol_scale(W, n, NP, shift, &red);
    const bool bad = chol_blocks<P, NW, false>(W, E, clamp * scale, wave, lane);
    if (t == 0 && flags) flags[b] = (first ? 0 : flags[b]) | (bad ? 4 : 0);
    double2 *Ob = Rinv + b * nn;
    double2 *Fb = Rf ? Rf + b * nn : nullptr;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = t + NT * u, i = e / NP, j = e % NP;
        if (i >= n || j >= n) continue;
        const bool up = j >= i;
        Ob[i * n + j] = up ? make_double2(E.re[i][j], E.im[i][j]) : make_double2(0.0, 0.0);
        if (Fb) Fb[i * n + j] = up ? make_double2(W.re[i][j], W.im[i][j]) : make_double2(0.0, 0.0);
    }
}

// One pass of CholeskyQR over a block of p.rb rows of a (batch x m x n, n <= 16 P)
// complex matrix, CQR_ROWS rows staged in LDS at a time: the rows are read through
// p.src's strides (complex64 or complex128, conjugated if asked), multiplied by
// the inverse factor p.Ri of the previous pass when given (Y = X Ri, Ri upper
// triangular: the zero blocks are skipped), written to the contiguous complex128
// rows p.X and/or through p.dst's strides, and their Gram matrix Y^H Y (upper
// triangle) is written to p.part[b][block] when p.part is given.  Two row tiles
// by P column tiles of the product and P (P + 1) / 2 tiles of the Gram matrix
// are dealt to the four waves so that each has the same number of k steps (at P =
// 4) and keeps its Gram tiles in registers over the staged chunks.  With the
// products on the vector unit a pass was bound by its LDS reads: 28 us on 4096 x
// 64, now 14 (the whole orthonormalisation 146 for 285 us; 512 x 32 66 for 146).
template <int P>
__global__ void __launch_bounds__(256) k_cqr_rows(CqrPass p) {
    constexpr int NP = CB * P;
    constexpr int TG = P * (P + 1) / 2;          // Gram tiles
    constexpr int GW = (TG + 3) / 4;             // of one wave
    __shared__ double sX[2][CQR_ROWS][CLD<P>];
    __shared__ double sY[2][CQR_ROWS][CLD<P>];
    __shared__ double sR[2][NP][CLD<P>];
    const CMat<CLD<P>> X{sX[0], sX[1]}, Yr{sY[0], sY[1]}, Ri{sR[0], sR[1]};
    const int t = threadIdx.x, b = blockIdx.y, n = p.n, wave = t >> 6, lane = t & 63;
    const int r_beg = blockIdx.x * p.rb, r_end = min(p.m, r_beg + p.rb);
    const bool apply = p.Ri != nullptr;
    const bool by_col = p.s_cs != 1;             // source contiguous along rows
    constexpr int LX = CQR_ROWS * NP / 256;
    double2 xv[LX];
    auto load = [&](int r0) {                    // one chunk, all loads issued together
        const int nr = min(CQR_ROWS, r_end - r0);
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int e = t + 256 * i;
            const int r = by_col ? e % CQR_ROWS : e / NP, c = by_col ? e / CQR_ROWS : e % NP;
            xv[i] = (r < nr && c < n) ? ld_c(p.src, p.s_esz, (int64_t)b * p.s_bs + (int64_t)(r0 + r) * p.s_rs +
                                                                 (int64_t)c * p.s_cs, p.s_conj)
                                      : make_double2(0.0, 0.0);
        }
    };
    load(r_beg);
    if (apply) {
        const double2 *Rb = reinterpret_cast<const double2 *>(p.Ri) + (int64_t)b * n * n;
        double2 rv[NP * NP / 256];
#pragma unroll
        for (int i = 0; i < NP * NP / 256; ++i) {
            const int e = t + 256 * i, r = e / NP, c = e % NP;
            rv[i] = r < n && c < n ? Rb[r * n + c] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int i = 0; i < NP * NP / 256; ++i) {
            const int e = t + 256 * i, r = e / NP, c = e % NP;
            Ri.re[r][c] = rv[i].x;
            Ri.im[r][c] = rv[i].y;
        }
    }
    CAcc g[GW];
#pragma unroll
    for (int i = 0; i < GW; ++i) acc_zero(g[i]);
    for (int r0 = r_beg; r0 < r_end; r0 += CQR_ROWS) {
        const int nr = min(CQR_ROWS, r_end - r0);
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int e = t + 256 * i;
            const int r = by_col ? e % CQR_ROWS : e / NP, c = by_col ? e / CQR_ROWS : e % NP;
            X.re[r][c] = xv[i].x;
            X.im[r][c] = xv[i].y;
        }
        __syncthreads();
        if (r0 + CQR_ROWS < r_end) load(r0 + CQR_ROWS);
        CMat<CLD<P>> Y = X;
        if (apply) {
            // row tile wave % 2; waves 0, 1 take the outer columns, 2, 3 the inner ones
#pragma unroll
            for (int c = 0; c < P; ++c) {
                const bool outer = c == 0 || c == P - 1;
                if ((P <= 2 ? c % 2 == 0 : outer) != (wave < 2)) continue;
                CAcc a;
                acc_zero(a);
                for (int k = 0; k <= c; ++k) acc_block<false>(a, X, CB * (wave & 1), CB * k, Ri, CB * k, CB * c, lane);
                acc_store<false>(a, Yr, CB * (wave & 1), CB * c, 1.0, lane);
            }
            __syncthreads();
            Y = Yr;
        }
        if (p.X)
            for (int e = t; e < nr * n; e += 256) {
                const int r = e / n, c = e % n;
                reinterpret_cast<double2 *>(p.X)[((int64_t)b * p.m + r0 + r) * n + c] = make_double2(Y.re[r][c], Y.im[r][c]);
            }
        if (p.dst)
            for (int e = t; e < nr * n; e += 256) {
                int r, c;
                if (p.d_cs != 1) { c = e / nr; r = e % nr; }
                else { r = e / n; c = e % n; }
                st_c(p.dst, p.d_esz, (int64_t)b * p.d_bs + (int64_t)(r0 + r) * p.d_rs + (int64_t)c * p.d_cs,
                     make_double2(Y.re[r][c], Y.im[r][c]), p.d_conj);
            }
        if (p.part) {
            int q = 0;
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
                for (int j = i; j < P; ++j, ++q)
                    if (q % 4 == wave) {
#pragma unroll
                        for (int k = 0; k < CQR_ROWS; k += CB)
                            acc_block<true>(g[q / 4], Y, k, CB * i, Y, k, CB * j, lane);
                    }
        }
        __syncthreads();
    }
    if (p.part) {
        double2 *G = reinterpret_cast<double2 *>(p.part) + ((int64_t)b * gridDim.x + blockIdx.x) * n * n;
        int q = 0;
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = i; j < P; ++j, ++q)
                if (q % 4 == wave) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = CB * i + 4 * r + (lane >> 4), col = CB * j + (lane & 15);
                        if (row < n && col < n) G[row * n + col] = make_double2(g[q / 4].re[r], g[q / 4].im[r]);
                    }
                }
    }
}

// The whole orthonormalisation of one matrix in one workgroup, n <= 32 columns and
// at most CQR1_ROWS rows (135 KiB of LDS), which stay there through the three
// passes: Gram matrix (each wave a share of the rows, the partial sums added in
// wave order), its factor's inverse in place, rows times inverse.  flags[b] as from
// launch_chol_inv.  Replaces eleven launches where a matrix alone cannot fill the
// chip: 256 x 32 takes 76 us, 32 of 128 x 16 24 (103 before), 64 x 16 19 (96).
constexpr int CQR1_ROWS = 256;
constexpr int XLD = 33;  // padded LDS row of 32 complex doubles
template <int P, int NW>
__global__ void __launch_bounds__(64 * NW, 2) k_cqr_one(QrArgs a, double shift, int *flags) {
    extern __shared__ double2 lds[];                 // X [rows of 16][XLD]
    __shared__ double sW[2][CB * P][CLD<P>];
    __shared__ double red;
    constexpr int NP = CB * P;
    const CMat<CLD<P>> W{sW[0], sW[1]};
    const int t = threadIdx.x, b = blockIdx.x, m = a.m, n = a.n, wave = t >> 6, lane = t & 63;
    const int x = lane & 15, q = lane >> 4;
    const int mt = (m + CB - 1) / CB;                // row tiles
    const bool by_col = a.a_cs != 1;
    for (int e = t; e < mt * CB * NP; e += 64 * NW) {
        const int r = by_col ? e % (mt * CB) : e / NP, c = by_col ? e / (mt * CB) : e % NP;
        lds[r * XLD + c] = r < m && c < n ? ld_c(a.A, a.a_esz, (int64_t)b * a.a_bs + (int64_t)r * a.a_rs +
                                                                   (int64_t)c * a.a_cs, a.a_conj)
                                          : make_double2(0.0, 0.0);
    }
    bool bad = false;
    for (int pass = 0; pass < 3; ++pass) {
        __syncthreads();
        CAcc g[P][P];
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = i; j < P; ++j) acc_zero(g[i][j]);
        for (int r = wave; r < mt; r += NW)
#pragma unroll
            for (int k = 0; k < CB; k += 4) {
                double2 v[P];
#pragma unroll
                for (int i = 0; i < P; ++i) v[i] = lds[(CB * r + k + q) * XLD + CB * i + x];
#pragma unroll
                for (int i = 0; i < P; ++i)
#pragma unroll
                    for (int j = i; j < P; ++j) acc_mma(g[i][j], v[i].x, -v[i].y, v[j].x, v[j].y);
            }
        for (int w = 0; w < NW; ++w) {
            if (wave == w)
#pragma unroll
                for (int i = 0; i < P; ++i)
#pragma unroll
                    for (int j = i; j < P; ++j) {
                        if (w == 0) acc_store<false>(g[i][j], W, CB * i, CB * j, 1.0, lane);
                        else acc_store<true>(g[i][j], W, CB * i, CB * j, 1.0, lane);
                    }
            __syncthreads();
        }
        const double scale = chol_scale(W, n, NP, pass == 0 ? shift : 0.0, &red);
        bad |= chol_blocks<P, NW, true>(W, W, (pass == 0 ? 1e-300 : 1e-14) * scale, wave, lane);
        for (int r = wave; r < mt; r += NW) {
            CAcc y[P];
#pragma unroll
            for (int c = 0; c < P; ++c) acc_zero(y[c]);
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
                for (int k = 0; k < CB; k += 4) {
                    const double2 v = lds[(CB * r + x) * XLD + CB * i + k + q];
#pragma unroll
                    for (int c = i; c < P; ++c)
                        acc_mma(y[c], v.x, v.y, W.re[CB * i + k + q][CB * c + x], W.im[CB * i + k + q][CB * c + x]);
                }
#pragma unroll
            for (int c = 0; c < P; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    lds[(CB * r + 4 * k + q) * XLD + CB * c + x] = make_double2(y[c].re[k], y[c].im[k]);
        }
    }
    __syncthreads();
    const bool q_col = a.q_cs != 1;
    for (int e = t; e < m * n; e += 64 * NW) {
        const int r = q_col ? e % m : e / n, c = q_col ? e / m : e % n;
        st_c(a.Q, a.q_esz, (int64_t)b * a.q_bs + (int64_t)r * a.q_rs + (int64_t)c * a.q_cs, lds[r * XLD + c], a.q_conj);
    }
    if (t == 0) flags[b] = bad ? 4 : 0;
}

// G[b][e] = sum over p of parts[b][p][e] (e < nn), in a fixed order: 256
// threads per SUM_E entries, each of the 256 / SUM_E slices sums the parts
// p = slice, slice + slices, ... in order, then the slices are added in order.
__global__ void __launch_bounds__(256) k_sum_parts(const double2 *parts, int nparts, int nn, double2 *G) {
    constexpr int SL = 256 / SUM_E;
    __shared__ double2 red[SL][SUM_E];
    const int t = threadIdx.x, b = blockIdx.y;
    const int el = t % SUM_E, sl = t / SUM_E;
    const int e = blockIdx.x * SUM_E + el;
    double2 acc = make_double2(0.0, 0.0);
    if (e < nn) {
        const double2 *P = parts + (int64_t)b * nparts * nn + e;
        for (int q = sl; q < nparts; q += SL) {
            const double2 v = P[(int64_t)q * nn];
            acc.x += v.x;
            acc.y += v.y;
        }
    }
    red[sl][el] = acc;
    __syncthreads();
    if (sl == 0 && e < nn) {
        double2 r = red[0][el];
        for (int q = 1; q < SL; ++q) {
            r.x += red[q][el].x;
            r.y += red[q][el].y;
        }
        G[(int64_t)b * nn + e] = r;
    }
}

// x[i] *= (re + i im), complex128.
__global__ void __launch_bounds__(256) k_scale(double2 *x, int64_t n, double re, double im) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double2 v = x[i];
        x[i] = make_double2(v.x * re - v.y * im, v.x * im + v.y * re);
    }
}

__global__ void __launch_bounds__(256) k_strided_copy(const char *in, int ie, int64_t ibs, int64_t irs, int64_t ics,
                                                     char *out, int oe, int64_t obs, int64_t ors, int64_t ocs, int m,
                                                     int n, int batch, int conj) {
    const int64_t per = (int64_t)m * n, total = per * batch;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int b = (int)(e / per);
        const int64_t r = e - (int64_t)b * per;
        const int i = (int)(r / n), j = (int)(r - (int64_t)i * n);
        double2 v = ld_c(in, ie, (int64_t)b * ibs + (int64_t)i * irs + (int64_t)j * ics, conj);
        st_c(out, oe, (int64_t)b * obs + (int64_t)i * ors + (int64_t)j * ocs, v, 0);
    }
}

}  // namespace

hipError_t launch_chol_inv(const double *G, int n, int batch, double shift, double clamp, double *Rinv, double *Rf,
                           int *flags, int first, hipStream_t s) {
    if (n > 64 || n < 1) return hipErrorInvalidValue;
    const double2 *g = reinterpret_cast<const double2 *>(G);
    double2 *ri = reinterpret_cast<double2 *>(Rinv), *rf = reinterpret_cast<double2 *>(Rf);
    auto go = [&](auto kernel, int nt) {
        hipLaunchKernelGGL(kernel, dim3(batch), dim3(nt), 0, s, g, n, shift, clamp, ri, rf, flags, first);
    };
    if (n <= 16) go(k_chol_inv<1, 4>, 256);
    else if (n <= 32) go(k_chol_inv<2, 4>, 256);
    else if (n <= 48) go(k_chol_inv<3, 8>, 512);
    else go(k_chol_inv<4, 8>, 512);
    return hipGetLastError();
}

bool cqr_one_fits(int m, int n) { return n <= 32 && m <= CQR1_ROWS; }

hipError_t launch_cqr_one(const QrArgs &a, double shift, int *flags, hipStream_t s) {
    if (a.m <= 0 || a.n <= 0 || a.batch <= 0) return hipSuccess;
    if (!cqr_one_fits(a.m, a.n) || a.R || !flags) return hipErrorInvalidValue;
    const size_t lds = (size_t)((a.m + CB - 1) / CB * CB) * XLD * sizeof(double2);
    auto go = [&](auto kernel, int nt) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)(CQR1_ROWS * XLD * sizeof(double2)));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(a.batch), dim3(nt), lds, s, a, shift, flags);
        return hipGetLastError();
    };
    // two waves a SIMD once each has two row tiles or more: 256 x 32 80 -> 76 us, 64 x 32
    // 43 -> 45
    if (a.m <= 128) return a.n <= 16 ? go(k_cqr_one<1, 4>, 256) : go(k_cqr_one<2, 4>, 256);
    return a.n <= 16 ? go(k_cqr_one<1, 8>, 512) : go(k_cqr_one<2, 8>, 512);
}

int cqr_rows_per_block(int m) {
    // one staged chunk per workgroup (the passes are latency-bound: more
    // workgroups, each with a short chain), at most 1024 blocks per matrix
    const int per = (m + 1023) / 1024;
    return std::max(CQR_ROWS, (per + CQR_ROWS - 1) / CQR_ROWS * CQR_ROWS);
}

hipError_t launch_sum_parts(const double *parts, int nparts, int n, int batch, double *G, hipStream_t s) {
    if (n < 1 || nparts < 1 || batch < 1) return hipSuccess;
    if (batch > 65535) return hipErrorInvalidValue;
    const int nn = n * n;
    hipLaunchKernelGGL(k_sum_parts, dim3((nn + SUM_E - 1) / SUM_E, batch), dim3(256), 0, s,
                       reinterpret_cast<const double2 *>(parts), nparts, nn, reinterpret_cast<double2 *>(G));
    return hipGetLastError();
}

hipError_t launch_cqr_pass(const CqrPass &p, hipStream_t s) {
    if (p.m <= 0 || p.batch <= 0) return hipSuccess;
    if (p.n < 1 || p.n > 64 || p.rb < CQR_ROWS || p.rb % CQR_ROWS) return hipErrorInvalidValue;
    if (p.batch > 65535) return hipErrorInvalidValue;
    const int nblk = (p.m + p.rb - 1) / p.rb;
    const dim3 g(nblk, p.batch), t(256);
    if (p.n <= 16) hipLaunchKernelGGL(k_cqr_rows<1>, g, t, 0, s, p);
    else if (p.n <= 32) hipLaunchKernelGGL(k_cqr_rows<2>, g, t, 0, s, p);
    else if (p.n <= 48) hipLaunchKernelGGL(k_cqr_rows<3>, g, t, 0, s, p);
    else hipLaunchKernelGGL(k_cqr_rows<4>, g, t, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_scale(void *x, int64_t n, double re, double im, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_scale, dim3((unsigned)g), dim3(256), 0, s, reinterpret_cast<double2 *>(x), n, re, im);
    return hipGetLastError();
}

hipError_t launch_strided_copy(const void *in, int ie, int64_t ibs, int64_t irs, int64_t ics, void *out, int oe,
                               int64_t obs, int64_t ors, int64_t ocs, int m, int n, int batch, int conj,
                               hipStream_t s) {
    const int64_t total = (int64_t)m * n * batch;
    if (total <= 0) return hipSuccess;
    int64_t g = (total + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_strided_copy, dim3((unsigned)g), dim3(256), 0, s, reinterpret_cast<const char *>(in), ie, ibs,
                       irs, ics, reinterpret_cast<char *>(out), oe, obs, ors, ocs, m, n, batch, conj);
    return hipGetLastError();
}

// workgroups (and workspace slots) of the fallback: at most 512, and at most
// 16 MiB of workspace (at least one slot)
static int qr_fallback_slots(int m, int n, int batch) {
    size_t w, y, t, b;
    const size_t per = global_qr_bytes(m, n, &w, &y, &t, &b);
    const size_t cap = (size_t)16 << 20;
    const int by_cap = (int)std::max<size_t>(1, cap / std::max<size_t>(per, 1));
    return std::max(1, std::min(std::min(batch, 512), by_cap));
}

size_t qr_fallback_workspace_bytes(int m, int n, int batch) {
    if (m <= 0 || n <= 0 || batch <= 0) return 0;
    size_t w, y, t, b;
    return global_qr_bytes(m, n, &w, &y, &t, &b) * (size_t)qr_fallback_slots(m, n, batch);
}

hipError_t launch_qr_fallback(const QrArgs &q, const int *flags, void *workspace, hipStream_t s) {
    const int m = q.m, n = q.n;
    if (m <= 0 || n <= 0 || q.batch <= 0) return hipSuccess;
    if (!flags || !workspace) return hipErrorInvalidValue;
    GlobalQrArgs g;
    const size_t per = global_qr_bytes(m, n, &g.w_off, &g.y_off, &g.t_off, &g.b_off);
    g.in = MatDesc{q.A, q.a_esz, q.a_bs, q.a_rs, q.a_cs, q.a_conj};
    g.m = m; g.n = n; g.ws = reinterpret_cast<char *>(workspace); g.ws_bs = (int64_t)per;
    g.Q = MatOut{q.Q, q.q_esz, q.q_bs, q.q_rs, q.q_cs, q.q_conj};
    g.R = MatOut{q.R, q.r_esz, q.r_bs, q.r_rs, q.r_cs, q.r_conj};
    g.want_r = q.R != nullptr;
    g.batch = q.batch;
    g.only_if = flags;
    hipLaunchKernelGGL(k_qr_global, dim3(qr_fallback_slots(m, n, q.batch)), dim3(QR_NT), 0, s, g);
    return hipGetLastError();
}

size_t qr_workspace_bytes(int m, int n, int batch, int keep_sums) {
    if (m <= 0 || n <= 0) return 0;
    std::vector<TsqrLevel> lv;
    size_t w, y, t, b;
    const size_t per = use_tsqr(m, n) ? plan_tsqr(m, n, keep_sums, lv) : global_qr_bytes(m, n, &w, &y, &t, &b);
    return per * (size_t)batch;
}

hipError_t launch_qr(const QrArgs &q, void *workspace, hipStream_t s) {
    const int m = q.m, n = q.n;
    if (m <= 0 || n <= 0 || q.batch <= 0) return hipSuccess;
    if (q.only_if && !use_reg(n, q.keep_sums)) return hipErrorInvalidValue;
    const int k = m < n ? m : n;
    char *ws = reinterpret_cast<char *>(workspace);
    MatDesc in{q.A, q.a_esz, q.a_bs, q.a_rs, q.a_cs, q.a_conj};
    MatOut qo{q.Q, q.q_esz, q.q_bs, q.q_rs, q.q_cs, q.q_conj};
    MatOut ro{q.R, q.r_esz, q.r_bs, q.r_rs, q.r_cs, q.r_conj};
    if (!use_tsqr(m, n)) {
        GlobalQrArgs g;
        const size_t per = global_qr_bytes(m, n, &g.w_off, &g.y_off, &g.t_off, &g.b_off);
        g.in = in; g.m = m; g.n = n; g.ws = ws; g.ws_bs = (int64_t)per;
        g.Q = qo; g.R = ro; g.want_r = q.R != nullptr;
        g.batch = q.batch;
        g.only_if = nullptr;
        hipLaunchKernelGGL(k_qr_global, dim3(q.batch), dim3(QR_NT), 0, s, g);
        return hipGetLastError();
    }
    std::vector<TsqrLevel> lv;
    const size_t per = plan_tsqr(m, n, q.keep_sums, lv);
    const size_t lds_bytes = (size_t)QR_LDS * 16;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_qr_leaf),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_qr_form),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        attr_set = true;
    }
    auto form_of = [&](int L) {
        FormArgs f;
        f.rows = lv[L].rows; f.n = n; f.nb = lv[L].nb; f.k = k;
        f.top = (L + 1 == (int)lv.size()); f.level0 = (L == 0);
        f.ws = ws; f.ws_bs = (int64_t)per;
        f.v_off = lv[L].v_off; f.t_off = lv[L].t_off; f.b_off = lv[L].b_off;
        f.x_off = f.top ? 0 : lv[L + 1].q_off;
        f.q_off = lv[L].q_off;
        f.out = qo;
        f.only_if = q.only_if;
        return f;
    };
    for (size_t L = 0; L < lv.size(); ++L) {
        LeafArgs a;
        if (L == 0) a.in = in;
        else a.in = MatDesc{ws + lv[L - 1].rs_off, 16, (int64_t)(per / 16), n, 1, 0};
        a.rows = lv[L].rows; a.n = n; a.nb = lv[L].nb; a.top = (L + 1 == lv.size());
        a.ws = ws; a.ws_bs = (int64_t)per;
        a.v_off = lv[L].v_off; a.t_off = lv[L].t_off; a.b_off = lv[L].b_off; a.rs_off = lv[L].rs_off;
        a.R = ro; a.want_r = (q.R != nullptr);
        a.only_if = q.only_if;
        if (use_reg(n, q.keep_sums)) {
            launch_reg(&a, form_of((int)L), n, (lv[L].rows + lv[L].nb - 1) / lv[L].nb, dim3(lv[L].nb, q.batch), s);
        } else {
            hipLaunchKernelGGL(k_qr_leaf, dim3(lv[L].nb, q.batch), dim3(QR_NT), lds_bytes, s, a);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    for (int L = (int)lv.size() - 1; L >= 0; --L) {
        const FormArgs f = form_of(L);
        if (!use_reg(n, q.keep_sums)) {
            hipLaunchKernelGGL(k_qr_form, dim3(lv[L].nb, q.batch), dim3(QR_NT), lds_bytes, s, f);
        } else if (!f.top) {
            launch_reg(nullptr, f, n, (lv[L].rows + lv[L].nb - 1) / lv[L].nb, dim3(lv[L].nb, q.batch), s);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tnk
