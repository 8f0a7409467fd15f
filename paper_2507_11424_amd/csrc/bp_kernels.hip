// Kernels of belief propagation on the norm network and of the loop BP error
// (Methods, BP contraction and Eqs. avBPError / loopBPerror; Appendix, the
// message update rule and "Computing the BP Error").  All arithmetic FP64
// complex (double2).  The contractions of the message updates run on the
// GETT engine; these kernels embed the site tensors in a uniform padded
// layout, normalise and exchange the messages, form the BP free energy, gather
// the loop matrices and find their eigenvalues.
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace tnk {
namespace {

constexpr int NT = 256;

__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ inline double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ inline double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ inline double cabsv(double2 a) { return hypot(a.x, a.y); }
__device__ inline double2 csqrt(double2 z) {
    const double r = cabsv(z);
    if (r == 0.0) return make_double2(0.0, 0.0);
    double x = sqrt(0.5 * (r + fabs(z.x)));
    double y = 0.5 * z.y / x;
    if (z.x >= 0.0) return make_double2(x, y);
    if (z.y < 0.0) { x = -x; y = -y; }
    return make_double2(fabs(y), x);  // sqrt for Re z < 0: (|Im|/(2x), sign(Im) x)
}

__device__ double block_sum(double v, double *red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int h = NT / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

__device__ double block_max(double v, double *red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int h = NT / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h]);
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// One message per block b = z * 4 + leg (legs 0..3 = up, left, down, right):
// the message site z sends through `leg`, out[leg][z] (Dm x Dm), becomes its
// Hermitian part divided by its Frobenius norm and is stored as the message
// into the neighbour w = nbr[z][leg] through the opposite leg; dmax[b] is the
// largest element change (0 for legs without a bond).
__global__ void __launch_bounds__(NT) k_bp_update(const double2 *out, double2 *msg, const int *nbr, int N, int Dm,
                                                 double *dmax) {
    __shared__ double red[NT];
    const int b = blockIdx.x;
    const int z = b >> 2, leg = b & 3;
    const int w = nbr[b];
    if (w < 0) {
        if (threadIdx.x == 0) dmax[b] = 0.0;
        return;
    }
    const int n2 = Dm * Dm;
    const double2 *m = out + ((int64_t)leg * N + z) * n2;
    double2 *dst = msg + ((int64_t)w * 4 + ((leg + 2) & 3)) * n2;
    double s = 0.0;
    for (int e = threadIdx.x; e < n2; e += NT) {
        const int i = e / Dm, j = e % Dm;
        const double2 h = cscale(cadd(m[i * Dm + j], cconj(m[j * Dm + i])), 0.5);
        s += cabs2(h);
    }
    s = block_sum(s, red);
    const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    double dm = 0.0;
    for (int e = threadIdx.x; e < n2; e += NT) {
        const int i = e / Dm, j = e % Dm;
        const double2 h = cscale(cadd(m[i * Dm + j], cconj(m[j * Dm + i])), 0.5 * inv);
        const double2 o = dst[e];
        dm = fmax(dm, fmax(fabs(h.x - o.x), fabs(h.y - o.y)));
        dst[e] = h;
    }
    dm = block_max(dm, red);
    if (threadIdx.x == 0) dmax[b] = (s > 0.0 && isfinite(s)) ? dm : INFINITY;
}

__global__ void __launch_bounds__(NT) k_max(const double *x, int n, double *out) {
    __shared__ double red[NT];
    double m = 0.0;
    for (int i = threadIdx.x; i < n; i += NT) m = fmax(m, x[i]);
    m = block_max(m, red);
    if (threadIdx.x == 0) *out = m;
}

// Per site z: zv[z] = sum_ij outr[z][i][j] msg[z][right][i][j] (the pair closed
// with all four messages); ze[z][0 / 1] = sum_ij msg[z][right / down] *
// msg[w][left / up] for the bond to the right / below (1 if absent).
__global__ void __launch_bounds__(NT) k_bp_values(const double2 *outr, const double2 *msg, const int *nbr, int N,
                                                 int Dm, double2 *zv, double2 *ze) {
    __shared__ double red[NT];
    const int z = blockIdx.x;
    const int n2 = Dm * Dm;
    const double2 *o = outr + (int64_t)z * n2;
    const double2 *mr = msg + ((int64_t)z * 4 + 3) * n2;
    double2 acc = make_double2(0.0, 0.0);
    for (int e = threadIdx.x; e < n2; e += NT) acc = cadd(acc, cmul(o[e], mr[e]));
    const double vr = block_sum(acc.x, red), vi = block_sum(acc.y, red);
    if (threadIdx.x == 0) zv[z] = make_double2(vr, vi);
    for (int k = 0; k < 2; ++k) {
        const int leg = k == 0 ? 3 : 2;  // right, down
        const int w = nbr[z * 4 + leg];
        double2 a = make_double2(0.0, 0.0);
        if (w >= 0) {
            const double2 *m1 = msg + ((int64_t)z * 4 + leg) * n2;
            const double2 *m2 = msg + ((int64_t)w * 4 + ((leg + 2) & 3)) * n2;
            for (int e = threadIdx.x; e < n2; e += NT) a = cadd(a, cmul(m1[e], m2[e]));
        }
        const double er = block_sum(a.x, red), ei = block_sum(a.y, red);
        if (threadIdx.x == 0) ze[z * 2 + k] = w >= 0 ? make_double2(er, ei) : make_double2(1.0, 0.0);
    }
}

// out[0] = sum log|zv| - sum log|ze|, out[1] = the same sum of phases, in a
// fixed order (one wave: a lane per site, then a tree over the lanes; one lane
// alone took 235 us for 144 sites).
__global__ void __launch_bounds__(64) k_bp_logsum(const double2 *zv, const double2 *ze, int N, double *out) {
    double lz = 0.0, ph = 0.0;
    for (int z = threadIdx.x; z < N; z += 64) {
        lz += log(cabsv(zv[z]));
        ph += atan2(zv[z].y, zv[z].x);
        for (int k = 0; k < 2; ++k) {
            const double2 e = ze[z * 2 + k];
            lz -= log(cabsv(e));
            ph -= atan2(e.y, e.x);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        lz += __shfl_xor(lz, o);
        ph += __shfl_xor(ph, o);
    }
    if (threadIdx.x == 0) {
        out[0] = lz;
        out[1] = remainder(ph, 2.0 * M_PI);
    }
}

// mats[q] (n x n, n = Dm^2) <- the pair tensor tab[q] = (buffer offset, flag):
// flag 0 copies [i][j], flag 1 transposes.
__global__ void __launch_bounds__(NT) k_gather_mats(const double2 *pairs, const int64_t *off, const int *trans,
                                                   int n, double2 *mats) {
    const int q = blockIdx.x;
    const double2 *src = pairs + off[q];
    double2 *dst = mats + (int64_t)q * n * n;
    const int t = trans[q];
    for (int e = threadIdx.x; e < n * n; e += NT) {
        const int i = e / n, j = e % n;
        dst[e] = t ? src[(int64_t)j * n + i] : src[e];
    }
}

// Eigenvalues of one general complex n x n matrix per workgroup (the matrix is
// overwritten): Householder reduction to upper Hessenberg form, then the
// shifted QR algorithm with Givens rotations on the active window, Wilkinson
// shifts (an exceptional shift every 11th iteration without deflation) and
// deflation when |h[k][k-1]| <= eps (|h[k][k]| + |h[k-1][k-1]|) (Golub and Van
// Loan, Matrix Computations, 7.4-7.5).  eps[q] = 1 - max|lambda| / sum|lambda|;
// info[q] = 0, or 1 if the iteration limit (30 n per eigenvalue) was hit.
//
// Bound by the chain of rotations, one square root and one division each: NT
// lanes share every other part.  A lane owns one column in the products from
// the left (it carries the column's entry of the current row in registers, so
// a rotation reads one new row) and one row in those from the right; the
// rotation is formed by every lane from its owner's two entries.  Up to 64
// columns one wave does it, without barriers, the entries handed round by
// lane reads; above, four waves through LDS.  The matrix sits in LDS up to
// EIG_LDS_N columns (row length n + 1: a lane per row reads without bank
// conflicts), else in place.  tn_bp on a 12 x 12 brick at D = 8 (its 55 loop
// matrices have n = 64) went from 195 ms, one lane per matrix, to 36 ms.
// The matrix is first scaled by a power of two to entries of at most 1, so the
// squares of entries underflow only below 1e-154 of the largest.
constexpr int EIG_LDS_N = 96;
__device__ inline double2 lane_read(double2 v, int lane) {
    const int2 a = __builtin_bit_cast(int2, v.x), b = __builtin_bit_cast(int2, v.y);
    const int2 c = make_int2(__builtin_amdgcn_readlane(a.x, lane), __builtin_amdgcn_readlane(a.y, lane));
    const int2 d = make_int2(__builtin_amdgcn_readlane(b.x, lane), __builtin_amdgcn_readlane(b.y, lane));
    return make_double2(__builtin_bit_cast(double, c), __builtin_bit_cast(double, d));
}

template <int NTH, bool IN_LDS>
__global__ void __launch_bounds__(NTH) k_eig(double2 *mats, int n, double2 *lam, double *eps, int *info) {
    extern __shared__ double2 hl[];
    constexpr int NW = NTH / 64;
    __shared__ double2 va[NTH], vb[NTH];   // reflector; rotations x / r, y / r
    __shared__ double2 ls[NTH];            // eigenvalues of the scaled matrix
    __shared__ double2 hand[2][2];         // the current rotation's entries (NW > 1)
    __shared__ double red[NW];
    __shared__ int redi[NW];
    const int q = blockIdx.x, t = threadIdx.x;
    double2 *G = mats + (int64_t)q * n * n;
    double2 *H = IN_LDS ? hl : G;
    const int ld = IN_LDS ? n + 1 : n;
#define AT(i, j) H[(int64_t)(i) * ld + (j)]
    auto reduce = [&](double v, bool mx) {  // sum or maximum over the block, to every thread
        for (int o = 32; o > 0; o >>= 1) {
            const double u = __shfl_xor(v, o);
            v = mx ? fmax(v, u) : v + u;
        }
        if constexpr (NW > 1) {
            __syncthreads();
            if ((t & 63) == 0) red[t >> 6] = v;
            __syncthreads();
            v = red[0];
            for (int i = 1; i < NW; ++i) v = mx ? fmax(v, red[i]) : v + red[i];
        }
        return v;
    };
    double big = 0.0;
    for (int e = t; e < n * n; e += NTH) big = fmax(big, fmax(fabs(G[e].x), fabs(G[e].y)));
    big = reduce(big, true);
    int ex = 0;
    if (big > 0.0 && isfinite(big)) ex = ilogb(big);
    for (int e = t; e < n * n; e += NTH) {
        const double2 g = G[e];
        AT(e / n, e % n) = make_double2(ldexp(g.x, -ex), ldexp(g.y, -ex));
    }
    __syncthreads();
    // Householder to Hessenberg: zero H[k+2.., k]
    for (int k = 0; k + 2 < n; ++k) {
        const double2 x = t > k && t < n ? AT(t, k) : make_double2(0.0, 0.0);
        const double tail2 = reduce(t > k + 1 ? cabs2(x) : 0.0, false);
        if (tail2 <= 1e-300) continue;  // uniform
        const double2 x0 = AT(k + 1, k);
        const double a2 = cabs2(x0), a0 = sqrt(a2), xn = sqrt(a2 + tail2);
        const double2 ph = a0 > 0.0 ? cscale(x0, 1.0 / a0) : make_double2(1.0, 0.0);
        // v = x + ph |x| e1, H <- (I - 2 v v^H / v^H v) H (I - ...)
        const double2 v0 = cadd(x0, cscale(ph, xn));
        const double beta = 2.0 / (cabs2(v0) + tail2);
        va[t] = t == k + 1 ? v0 : x;
        __syncthreads();
        if (t > k && t < n) {  // left: column t, rows k+1..n-1
            double2 s = make_double2(0.0, 0.0);
            for (int i = k + 1; i < n; ++i) s = cadd(s, cmul(cconj(va[i]), AT(i, t)));
            s = cscale(s, beta);
            for (int i = k + 1; i < n; ++i) AT(i, t) = csub(AT(i, t), cmul(va[i], s));
        }
        __syncthreads();
        if (t < n) {           // right: row t, columns k+1..n-1
            double2 s = make_double2(0.0, 0.0);
            for (int j = k + 1; j < n; ++j) s = cadd(s, cmul(AT(t, j), va[j]));
            s = cscale(s, beta);
            for (int j = k + 1; j < n; ++j) AT(t, j) = csub(AT(t, j), cmul(s, cconj(va[j])));
            if (t > k) AT(t, k) = t == k + 1 ? cscale(ph, -xn) : make_double2(0.0, 0.0);
        }
        __syncthreads();
    }
    int hi = n - 1, iter = 0, bad = 0;
    const double ulp = 2.220446049250313e-16;
    while (hi >= 0) {  // hi, iter and l are the same in every thread
        if (hi == 0) {
            if (t == 0) ls[0] = AT(0, 0);
            break;
        }
        // the window l..hi: the lowest row reached from hi without a negligible subdiagonal
        bool small = false;
        if (t >= 1 && t <= hi) {
            const double s = cabsv(AT(t, t)) + cabsv(AT(t - 1, t - 1));
            small = cabsv(AT(t, t - 1)) <= ulp * (s > 0.0 ? s : 1.0);
            if (small) AT(t, t - 1) = make_double2(0.0, 0.0);  // read by this thread alone
        }
        const unsigned long long bal = __ballot(small);
        int l = bal ? (t & ~63) + 63 - __clzll((long long)bal) : 0;
        if constexpr (NW > 1) {
            if ((t & 63) == 0) redi[t >> 6] = l;
            __syncthreads();
            l = redi[0];
            for (int i = 1; i < NW; ++i) l = max(l, redi[i]);
        }
        if (l == hi) {
            if (t == 0) ls[hi] = AT(hi, hi);
            --hi;
            iter = 0;
            __syncthreads();  // the next scan rewrites redi
            continue;
        }
        if (++iter > 30 * n) {
            bad = 1;
            if (t <= hi) ls[t] = AT(t, t);
            break;
        }
        // Wilkinson shift: eigenvalue of the trailing 2x2 closer to h[hi][hi]
        double2 mu;
        if (iter % 11 == 0) {
            mu = cadd(AT(hi, hi), make_double2(0.75 * cabsv(AT(hi, hi - 1)), 0.0));
        } else {
            const double2 a = AT(hi - 1, hi - 1), b = AT(hi - 1, hi), c = AT(hi, hi - 1), d = AT(hi, hi);
            const double2 tr2 = cscale(cadd(a, d), 0.5);
            const double2 dd = cscale(csub(a, d), 0.5);
            const double2 disc = csqrt(cadd(cmul(dd, dd), cmul(b, c)));
            const double2 m1 = cadd(tr2, disc), m2 = csub(tr2, disc);
            mu = cabs2(csub(m1, d)) < cabs2(csub(m2, d)) ? m1 : m2;
        }
        __syncthreads();
        // one QR step on the window: H - mu I = Q R, H <- R Q + mu I.  Rotation k
        // takes (x, y) = (h[k][k], h[k+1][k]) to (r, 0): rows k, k+1 become
        // (conj(x) row_k + conj(y) row_k+1) / r and (x row_k+1 - y row_k) / r.
        const bool col = t >= l && t <= hi;
        double2 cur = col ? AT(l, t) : make_double2(0.0, 0.0);
        if (t == l) cur = csub(cur, mu);
        double2 nxt = col ? AT(l + 1, t) : make_double2(0.0, 0.0);
        for (int k = l; k < hi; ++k) {
            double2 row = nxt;
            if (t == k + 1) row = csub(row, mu);
            if (k + 2 <= hi && col) nxt = AT(k + 2, t);  // one row ahead
            double2 x, y;
            if constexpr (NW == 1) {
                x = lane_read(cur, k);
                y = lane_read(row, k);
            } else {
                if (t == k) { hand[k & 1][0] = cur; hand[k & 1][1] = row; }
                __syncthreads();
                x = hand[k & 1][0];
                y = hand[k & 1][1];
            }
            const double r2 = cabs2(x) + cabs2(y);
            if (r2 > 0.0) {
                const double inv = 1.0 / sqrt(r2);
                x = cscale(x, inv);
                y = cscale(y, inv);
            } else {
                x = make_double2(1.0, 0.0);
                y = make_double2(0.0, 0.0);
            }
            if (t == 0) { va[k] = x; vb[k] = y; }
            if (t >= k && t <= hi) AT(k, t) = cadd(cmul(cconj(x), cur), cmul(cconj(y), row));
            cur = csub(cmul(x, row), cmul(y, cur));
        }
        if (t == hi) AT(hi, hi) = cur;
        __syncthreads();
        // columns k, k+1 of rows l..k+1, by rows: row t starts at column t - 1 (its
        // subdiagonal entry was annihilated) or at the window's first column
        if (col) {
            const int k0 = t > l ? t - 1 : l;
            double2 a = t > l ? make_double2(0.0, 0.0) : AT(l, l);
            for (int k = k0; k < hi; ++k) {
                const double2 b = AT(t, k + 1), x = va[k], y = vb[k];
                double2 o = cadd(cmul(a, x), cmul(b, y));
                if (t == k) o = cadd(o, mu);
                AT(t, k) = o;
                a = csub(cmul(b, cconj(x)), cmul(a, cconj(y)));
            }
            if (t == hi) a = cadd(a, mu);
            AT(t, hi) = a;
        }
        __syncthreads();
    }
    __syncthreads();
#undef AT
    const double a = t < n ? cabsv(ls[t]) : 0.0;
    const double mx = reduce(a, true), sm = reduce(a, false);
    if (t < n) lam[(int64_t)q * n + t] = make_double2(ldexp(ls[t].x, ex), ldexp(ls[t].y, ex));
    if (t == 0) {
        eps[q] = sm > 0.0 ? 1.0 - mx / sm : 0.0;
        info[q] = bad;
    }
}

}  // namespace

hipError_t launch_bp_update(const void *out, void *msg, const int *nbr, int N, int Dm, double *dmax, double *delta,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_bp_update, dim3(N * 4), dim3(NT), 0, s, static_cast<const double2 *>(out),
                       static_cast<double2 *>(msg), nbr, N, Dm, dmax);
    if (delta) hipLaunchKernelGGL(k_max, dim3(1), dim3(NT), 0, s, dmax, N * 4, delta);
    return hipGetLastError();
}

hipError_t launch_bp_free_energy(const void *outr, const void *msg, const int *nbr, int N, int Dm, void *zv,
                                 void *ze, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_bp_values, dim3(N), dim3(NT), 0, s, static_cast<const double2 *>(outr),
                       static_cast<const double2 *>(msg), nbr, N, Dm, static_cast<double2 *>(zv),
                       static_cast<double2 *>(ze));
    hipLaunchKernelGGL(k_bp_logsum, dim3(1), dim3(64), 0, s, static_cast<const double2 *>(zv),
                       static_cast<const double2 *>(ze), N, out);
    return hipGetLastError();
}

hipError_t launch_gather_mats(const void *pairs, const int64_t *off, const int *trans, int count, int n, void *mats,
                              hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_mats, dim3(count), dim3(NT), 0, s, static_cast<const double2 *>(pairs), off, trans, n,
                       static_cast<double2 *>(mats));
    return hipGetLastError();
}

hipError_t launch_eig(void *mats, int n, int batch, void *lam, double *eps, int *info, hipStream_t s) {
    if (batch <= 0) return hipSuccess;
    if (n < 1 || n > BP_EIG_NMAX) return hipErrorInvalidValue;
    double2 *m = static_cast<double2 *>(mats), *l = static_cast<double2 *>(lam);
    const size_t lds = (size_t)n * (n + 1) * sizeof(double2);
    constexpr int most = EIG_LDS_N * (EIG_LDS_N + 1) * (int)sizeof(double2);
    if (n <= 64) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_eig<64, true>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_eig<64, true>), dim3(batch), dim3(64), lds, s, m, n, l, eps, info);
    } else if (n <= EIG_LDS_N) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_eig<256, true>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_eig<256, true>), dim3(batch), dim3(256), lds, s, m, n, l, eps, info);
    } else {
        hipLaunchKernelGGL((k_eig<256, false>), dim3(batch), dim3(256), 0, s, m, n, l, eps, info);
    }
    return hipGetLastError();
}

}  // namespace tnk
