// Symmetric eigensolvers in FP64: cyclic two-sided Jacobi with the round-robin
// ("circle method") ordering, so that every round rotates n/2 disjoint index pairs
// in parallel.  Order n <= 96 (the Rayleigh-Ritz subspace matrix): one workgroup, A and V in
// LDS.  Larger orders (the natural-orbital, recanonicalisation, exact-1p-block and
// natural-auxiliary-function matrices, one or a batch): the same ordering over blocks of 16
// rows, each round diagonalising the block pairs' sub-matrices in LDS and applying their
// orthogonal factors to A and V on the matrix cores, two launches per round of block pairs.
#include "internal.h"
#include <algorithm>
#include <cmath>
#include <vector>

namespace adc3 {

typedef double d4e __attribute__((ext_vector_type(4)));

namespace {

// player in slot i in round r (np players, np even; player 0 fixed, the others rotate by r); slots k and
// np - 1 - k are paired
__device__ inline int rr_pos(int i, int r, int np) { return i == 0 ? 0 : 1 + (i - 1 + r) % (np - 1); }
// the same slot's player one round later, and the slot one round later of the player in slot x
__device__ inline int rr_next(int x, int np) { return x == 0 ? 0 : (x == np - 1 ? 1 : x + 1); }
__device__ inline int rr_prev(int x, int np) { return x == 0 ? 0 : (x == 1 ? np - 1 : x - 1); }

__device__ inline void pair_of(int r, int k, int np, int& p, int& q) {
    const int a = rr_pos(k, r, np), b = rr_pos(np - 1 - k, r, np);
    p = min(a, b);
    q = max(a, b);
}

// 1 / sqrt(x) and 1 / x from the hardware's start values (relative error about 2^-23) and N Newton steps (two
// reach FP64 rounding); normal, positive x only
template <int N>
__device__ inline double rsqrt_n(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int k = 0; k < N; ++k) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}
template <int N>
__device__ inline double rcp_n(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int k = 0; k < N; ++k) y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// The rotation (c, s) that annihilates apq: t = tan = sgn(d) b / (|d| + sqrt(d^2 + b^2)) with d = aqq - app,
// b = 2 apq, c = 1/sqrt(1 + t^2), s = t c.  A round's rotations are one dependent chain of FP64 arithmetic
// between two barriers, so there is no division, library square root or branch in it.  NT, NC: Newton steps of
// the angle and of the normalisation (the rotation is orthogonal to the accuracy of NC; an angle off by 2^-23,
// NT = 0, leaves that share of apq).  The matrix is scaled to norm about 1, so that the squares do not overflow;
// where they underflow, both entries are below 1e-145 of the norm and nothing is rotated.
template <int NT, int NC>
__device__ inline void rot_of(double app, double aqq, double apq, double& c, double& s) {
    const double d = aqq - app, b = 2.0 * apq;
    const double h2 = fma(d, d, b * b);
    const double h = h2 * rsqrt_n<NT>(h2);
    const double t0 = (d >= 0.0 ? b : -b) * rcp_n<NT>(fabs(d) + h);
    const bool none = h2 < 1e-290;
    const double t = none ? 0.0 : t0;
    c = rsqrt_n<NC>(fma(t, t, 1.0));
    s = t * c;
}

// power of two that brings a matrix of squared norm tot to norm about 1 (tot normal and finite)
__device__ inline double norm_scale(double tot) { return ldexp(1.0, -(__builtin_amdgcn_frexp_exp(tot) >> 1)); }

// ---------------- small: one workgroup, matrix and vectors in LDS ----------------
constexpr int SMALL_MAX = 96;

// Cyclic Jacobi on a symmetric np x np matrix (np even, at most SMALL_MAX) held in LDS (row stride ld), one
// workgroup of NTH threads: sweeps of np - 1 rounds of np/2 disjoint rotations, until the off-diagonal squared
// norm is at most 1e-30 of the total, or is within 100 times that and no longer halves, or max_sweeps.  V [nv][np] (same
// stride) accumulates the rotations on its columns.
// A round is a dependent chain (pivots, rotation, update), so it is latency bound: 0.30 us at order 40 with
// library divisions and square roots and the index arithmetic inside; here the indices advance in registers,
// the rotations of a round are computed by the first wave while the others still apply the previous round's to
// V, and the elements of A to be updated are loaded before the rotations are known.
template <int NTH>
__device__ void jacobi_lds(double* A, double* V, int np, int nv, int ld, int max_sweeps) {
    constexpr int MI = NTH >= 1024 ? 3 : 1;  // 2x2 blocks of A per thread: (np/2)^2 <= MI * NTH
    __shared__ double cs[2][SMALL_MAX / 2], sn[2][SMALL_MAX / 2];
    __shared__ double red[2][NTH / 64];
    const int tid = threadIdx.x;
    const int npair = np / 2, items = npair * npair;
    double prev = INFINITY;
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int t = tid; t < np * np; t += NTH) {
            const int i = t / np, j = t - (t / np) * np;
            const double a = A[i * ld + j];
            tot += a * a;
            if (i != j) off += a * a;
        }
        for (int o = 32; o > 0; o >>= 1) {
            off += __shfl_down(off, o, 64);
            tot += __shfl_down(tot, o, 64);
        }
        if ((tid & 63) == 0) { red[0][tid >> 6] = off; red[1][tid >> 6] = tot; }
        __syncthreads();
        double offs = 0.0, tots = 0.0;
        for (int k = 0; k < NTH / 64; ++k) { offs += red[0][k]; tots += red[1][k]; }
        __syncthreads();
        if (offs <= 1e-30 * tots || offs == 0.0) break;
        if (offs <= 1e-28 * tots && offs > 0.5 * prev) break;  // at the rounding floor (see offnorm_sum_kernel)
        prev = offs;
        const double scale = norm_scale(tots);
        // A is kept in slot order: rows and columns k, np - 1 - k are paired in every round, and each rotated
        // element is written where its players sit one round later, so that no address depends on the round
        // (after np - 1 rounds every player is back).  This thread's blocks: row pair k1, column pair k2.
        int in[MI], out[MI][4], k1[MI], k2[MI];
        const int dq = np - 1;
#pragma unroll
        for (int m = 0; m < MI; ++m) {
            const int t = min(tid + m * NTH, items - 1);
            k1[m] = t / npair;
            k2[m] = t - k1[m] * npair;
            in[m] = k1[m] * ld + k2[m];
            const int r0 = rr_prev(k1[m], np) * ld, r1 = rr_prev(dq - k1[m], np) * ld;
            const int c0 = rr_prev(k2[m], np), c1 = rr_prev(dq - k2[m], np);
            out[m][0] = r0 + c0; out[m][1] = r0 + c1; out[m][2] = r1 + c0; out[m][3] = r1 + c1;
        }
        // V stays in player order, on the threads past the first wave: pair vk in rows vi, vi + vst, ...
        const int vst = (NTH - 64) / npair, vi = (tid - 64) / npair, vk = (tid - 64) - vi * npair;
        int va = vk, vb = dq - vk;
        auto v_update = [&](int buf) {
            const double c = cs[buf][vk], s = sn[buf][vk];
            if (vi < vst)
                for (int i = vi; i < nv; i += vst) {
                    const double vip = V[i * ld + va], viq = V[i * ld + vb];
                    V[i * ld + va] = c * vip - s * viq;
                    V[i * ld + vb] = s * vip + c * viq;
                }
            va = rr_next(va, np);
            vb = rr_next(vb, np);
        };
        for (int r = 0; r < np - 1; ++r) {
            const int buf = r & 1;
            double x00[MI], x01[MI], x10[MI], x11[MI];
            if (tid < npair) {
                const int p = tid, q = dq - tid;
                double c, s;
                rot_of<2, 2>(scale * A[p * ld + p], scale * A[q * ld + q], scale * A[p * ld + q], c, s);
                cs[buf][tid] = c; sn[buf][tid] = s;
            } else if (tid >= 64 && r > 0) {
                v_update(buf ^ 1);
            }
#pragma unroll
            for (int m = 0; m < MI; ++m) {
                const int iq = in[m] + (dq - 2 * k1[m]) * ld, dc = dq - 2 * k2[m];
                x00[m] = A[in[m]]; x01[m] = A[in[m] + dc];
                x10[m] = A[iq]; x11[m] = A[iq + dc];
            }
            __syncthreads();
            // rows rotated first, then columns; the annihilated elements are set to zero
#pragma unroll
            for (int m = 0; m < MI; ++m) {
                if (tid + m * NTH >= items) break;
                const double c1 = cs[buf][k1[m]], s1 = sn[buf][k1[m]], c2 = cs[buf][k2[m]], s2 = sn[buf][k2[m]];
                const double y00 = c1 * x00[m] - s1 * x10[m], y10 = s1 * x00[m] + c1 * x10[m];
                const double y01 = c1 * x01[m] - s1 * x11[m], y11 = s1 * x01[m] + c1 * x11[m];
                const bool pivot = k1[m] == k2[m];
                A[out[m][0]] = c2 * y00 - s2 * y01;
                A[out[m][1]] = pivot ? 0.0 : s2 * y00 + c2 * y01;
                A[out[m][2]] = pivot ? 0.0 : c2 * y10 - s2 * y11;
                A[out[m][3]] = s2 * y10 + c2 * y11;
            }
            __syncthreads();
        }
        if (tid >= 64) v_update((np - 2) & 1);
        __syncthreads();
    }
}

// threads of the one-workgroup solver at order n: a thread per 2x2 block of A up to n = 64
inline int small_threads(int n) {
    const int h = (n + 1) / 2;
    return h * h <= 256 ? 256 : h * h <= 512 ? 512 : 1024;
}

// One workgroup per matrix A[blockIdx.x][n][n].  desc < 0: eigenpairs as the solver leaves them; 0 / 1: sorted
// ascending / descending (ties by position), each vector's largest |.| entry positive (the first of equals).  A's rows
// lda apart, (A + A^T)/2 if sym; sorted: also w to host and V w^-1/2 to coef where given.
template <int NTH>
__global__ __launch_bounds__(NTH) void jacobi_small_kernel(const double* Ag, int lda, int sym, int n, double* w, double* Vg,
                                                           int desc, double* coef, double* host) {
    extern __shared__ double sm[];
    __shared__ int rank[SMALL_MAX];
    __shared__ double sgn[SMALL_MAX], ww[SMALL_MAX];
    const int np = n + (n & 1), ld = np + 1;
    double* A = sm;
    double* V = sm + (size_t)np * ld;
    const int tid = threadIdx.x;
    const long long nn = (long long)n * n;
    Ag += (long long)blockIdx.x * n * lda;
    Vg += blockIdx.x * nn;
    w += (long long)blockIdx.x * n;
    for (int t = tid; t < np * np; t += NTH) {
        const int i = t / np, j = t - (t / np) * np;
        double a = (i < n && j < n) ? Ag[i * lda + j] : 0.0;
        if (sym && i < n && j < n) a = 0.5 * (a + Ag[j * lda + i]);
        A[i * ld + j] = a;  // odd n: a zero row and column, never rotated
        if (i < n) V[i * ld + j] = (i == j) ? 1.0 : 0.0;
    }
    __syncthreads();
    jacobi_lds<NTH>(A, V, np, n, ld, 60);
    if (desc < 0) {
        for (int t = tid; t < n * n; t += NTH) {
            const int i = t / n, j = t - (t / n) * n;
            Vg[t] = V[i * ld + j];
        }
        for (int i = tid; i < n; i += NTH) w[i] = A[i * ld + i];
        return;
    }
    if (tid < n) ww[tid] = A[tid * ld + tid];
    __syncthreads();
    if (tid < n) {
        const double wi = ww[tid];
        int rk = 0;
        double best = -1.0, sg = 1.0;
        for (int j = 0; j < n; ++j) {
            const double wj = ww[j];
            rk += desc ? (wj > wi || (wj == wi && j < tid)) : (wj < wi || (wj == wi && j < tid));
            const double x = V[j * ld + tid];
            if (fabs(x) > best) { best = fabs(x); sg = x < 0 ? -1.0 : 1.0; }
        }
        rank[tid] = rk;
        sgn[tid] = sg;
        w[rk] = wi;
        if (host) host[rk] = wi;
    }
    __syncthreads();
    for (int t = tid; t < n * n; t += NTH) {
        const int i = t / n, j = t - (t / n) * n;
        const double x = sgn[j] * V[i * ld + j];
        Vg[i * n + rank[j]] = x;
        if (coef) coef[i * n + rank[j]] = ww[j] > 0.0 ? x / sqrt(ww[j]) : 0.0;
    }
}

// Off-diagonal and total squared norms of the active matrices, in ONORM partial sums each (grid (ONORM, batch)),
// then summed in a fixed order by one wave per matrix, which marks a matrix done whose off-diagonal norm has
// reached the threshold or is not finite.  (One workgroup per matrix took 120 us per check at n = 600.)
constexpr int ONORM = 64;
__global__ void offnorm_part_kernel(const double* A, int n, double* part, const int* active) {
    const int bm = blockIdx.y;
    if (!active[bm]) return;
    const double* Ab = A + (long long)bm * n * n;
    double off = 0.0, tot = 0.0;
    for (int i = blockIdx.x; i < n; i += ONORM)
        for (int j = threadIdx.x; j < n; j += blockDim.x) {
            const double a = Ab[(long long)i * n + j];
            tot += a * a;
            if (i != j) off += a * a;
        }
    __shared__ double r1[4], r2[4];
    for (int o = 32; o > 0; o >>= 1) {
        off += __shfl_down(off, o, 64);
        tot += __shfl_down(tot, o, 64);
    }
    if ((threadIdx.x & 63) == 0) { r1[threadIdx.x >> 6] = off; r2[threadIdx.x >> 6] = tot; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double* p = part + 2 * ((long long)bm * ONORM + blockIdx.x);
        p[0] = ((r1[0] + r1[1]) + r1[2]) + r1[3];
        p[1] = ((r2[0] + r2[1]) + r2[2]) + r2[3];
    }
}

// nrm[2b] is kept from check to check: a matrix within 100 times the threshold whose off-diagonal norm did not halve
// since the last check is at its rounding floor and done as well.  Slow convergence further up is no floor: with a large
// cluster of eigenvalues the off-diagonal norm falls linearly from about 1e-24 of the total on (a 150-fold eigenvalue at
// n = 200; ended there, the residual is 6e-13 of the norm, here 8e-16).  The metric matrices of the NAF step, whose
// eigenvalues fall off fast, do the same (from 1e-22 on at n = 201) and take two more sweeps of eleven for it.
__global__ __launch_bounds__(64) void offnorm_sum_kernel(const double* part, int n, double* nrm, int* active) {
    const int bm = blockIdx.x;
    if (!active[bm]) return;
    double off = part[2 * ((long long)bm * ONORM + threadIdx.x)], tot = part[2 * ((long long)bm * ONORM + threadIdx.x) + 1];
    for (int o = 32; o > 0; o >>= 1) {
        off += __shfl_down(off, o, 64);
        tot += __shfl_down(tot, o, 64);
    }
    if (threadIdx.x == 0) {
        const double prev = nrm[2 * bm];
        nrm[2 * bm] = off;
        nrm[2 * bm + 1] = tot;
        // the rounding of the blocks' products leaves off-diagonal elements of about eps times the diagonal:
        // off^2 / tot of 2.5e-33 n measured (n = 200 .. 600), so the threshold grows with n
        const double thr = fmax(1e-30, 1e-32 * n) * tot;
        if (!(off == off && tot == tot) || !(tot < INFINITY) || off <= thr || off == 0.0 ||
            (off <= 100.0 * thr && off > 0.5 * prev))
            active[bm] = 0;
    }
}

// ascending (desc=0) or descending (desc=1) order; ties by index; sign: largest |.| of each column positive
// (first index on ties).  A workgroup ranks 16 columns, 16 threads a column, and writes them in place of their
// rank; the second kernel copies the sorted pairs back.  (One workgroup for everything took 570 us at n = 600.)
__global__ __launch_bounds__(256) void sort_rank_kernel(const double* w, const double* V, int n, int desc, double* wtmp,
                                                        double* Vtmp) {
    __shared__ int rk[16][17], at[16][17];
    __shared__ double bs[16][17];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int i = blockIdx.x * 16 + tx;
    int rank = 0, arg = n;
    double best = -1.0;
    if (i < n) {
        const double wi = w[i];
        for (int j = ty; j < n; j += 16) {
            const double wj = w[j];
            rank += desc ? (wj > wi || (wj == wi && j < i)) : (wj < wi || (wj == wi && j < i));
            const double x = fabs(V[(long long)j * n + i]);
            if (x > best) { best = x; arg = j; }
        }
    }
    rk[tx][ty] = rank; bs[tx][ty] = best; at[tx][ty] = arg;
    __syncthreads();
    if (i >= n) return;
    rank = 0;
    best = -1.0;
    arg = n;
    for (int k = 0; k < 16; ++k) {
        rank += rk[tx][k];
        const double x = bs[tx][k];
        if (x > best || (x == best && at[tx][k] < arg)) { best = x; arg = at[tx][k]; }
    }
    const double sgn = (arg < n && V[(long long)arg * n + i] < 0) ? -1.0 : 1.0;
    if (ty == 0) wtmp[rank] = w[i];
    for (int r = ty; r < n; r += 16) Vtmp[(long long)r * n + rank] = sgn * V[(long long)r * n + i];
}
__global__ void sort_copy_kernel(double* w, double* V, int n, const double* wtmp, const double* Vtmp) {
    const long long nn = (long long)n * n, st = (long long)gridDim.x * blockDim.x;
    const long long t0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    for (long long t = t0; t < nn; t += st) V[t] = Vtmp[t];
    for (long long t = t0; t < n; t += st) w[t] = wtmp[t];
}

// ---------------- large: block Jacobi, two launches per round of block pairs ----------------
// The matrix is cut into blocks of BJ rows (the last one shorter).  Every round pairs the blocks in the
// same round-robin order as the scalar rounds (with a bye when their count is odd); bj_solve_kernel runs one
// Jacobi sweep in LDS on each pair's symmetric sub-matrix (at most BSUB rows) and writes its orthogonal factor
// Q_k; bj_apply_kernel then applies every pair's factor at once, A <- P^T A P and V^T <- P^T V^T with P
// block-diagonal over the pairs' index sets, a 32 x 32 tile per workgroup on the matrix cores.  Every element of
// A lies in exactly one tile, so A is updated in place; the vectors are kept transposed (rows), which makes
// their update the first half of A's.
// Blocks of 16 (sub-matrices of 32, a 2x2 block per thread): a round costs a solve of 31 dependent scalar rounds
// and two launches, and one inner sweep is enough (the outer sweeps number the same, 9 at n = 200 and 11 at
// n = 600 on a uniform spectrum, with one or two inner sweeps and with blocks of 16 or 32).  Measured against
// blocks of 32 with two inner sweeps of the scalar code above and the tiles' products on the vector ALUs:
// n = 600 146 -> 10.5 ms, n = 200 16.0 -> 2.7 ms, five of n = 200 17.7 -> 3.1 ms (uniform spectra); a round's solve
// 226 -> 15.7 us and its application 50 -> 6-8 us.  At n = 600 two thirds of the old time went into sweeps past
// convergence: the threshold lay below the rounding floor of the off-diagonal norm (see offnorm_sum_kernel).
constexpr int BJ = 16, BSUB = 2 * BJ, BL = BSUB + 1;

// global row of local index t of the pair (blocks I, J) or -1 past the matrix (short last block, bye)
__device__ inline int bj_row(int t, int I, int J, int nblk, int n) {
    const int blk = t < BJ ? I : J;
    const int row = blk * BJ + (t & (BJ - 1));
    return (blk < nblk && row < n) ? row : -1;
}

// grid (npb / 2, batch), 512 threads; Q [batch][npb / 2][BSUB][BSUB] (identity on rows past the matrix)
__global__ __launch_bounds__(512) void bj_solve_kernel(const double* A, double* Q, int n, int nblk, int npb, int r,
                                                       const double* nrm, const int* active) {
    const int bm = blockIdx.y;
    if (!active[bm]) return;
    const double* Ab = A + (long long)bm * n * n;
    double* Qb = Q + ((long long)bm * (npb / 2) + blockIdx.x) * BSUB * BSUB;
    int I, J;
    pair_of(r, blockIdx.x, npb, I, J);
    __shared__ double S[2][BSUB * BL], V2[2][BSUB * BL];
    const int tid = threadIdx.x;
    const double scale = 0.5 * norm_scale(nrm[2 * bm + 1]);
    for (int t = tid; t < BSUB * BSUB; t += 512) {
        const int i = t / BSUB, j = t % BSUB;
        const int gi = bj_row(i, I, J, nblk, n), gj = bj_row(j, I, J, nblk, n);
        S[0][i * BL + j] =
            (gi >= 0 && gj >= 0) ? scale * Ab[(long long)gi * n + gj] + scale * Ab[(long long)gj * n + gi] : 0.0;
        V2[0][i * BL + j] = i == j ? 1.0 : 0.0;
    }
    __syncthreads();
    // One sweep.  S and V's columns are kept in slot order: pairs are slots k, 31 - k in every round, and rotated
    // elements are written where their players sit one round later, in the other of two buffers: no address
    // depends on the round, and a round has one barrier.  Waves 0-3: thread (k1, k2) owns the 2x2 block of pairs
    // k1, k2 of S and forms both rotations from the pivots itself; waves 4-7: V's columns of pair k2 in rows k1
    // and k1 + 16.  (With the players' indices advanced per round and V on the same four waves, a round took
    // 0.6 us, most of it instruction issue.)
    const int k1 = (tid >> 4) & 15, k2 = tid & 15;
    const int n0 = rr_prev(k2, BSUB), n1 = rr_prev(BSUB - 1 - k2, BSUB);
    if (tid < 256) {
        const int r0 = rr_prev(k1, BSUB) * BL, r1 = rr_prev(BSUB - 1 - k1, BSUB) * BL;
        const int i0 = k1 * BL + k2, i1 = (BSUB - 1 - k1) * BL + k2, dc = BSUB - 1 - 2 * k2;
        const int d1 = k1 * (BL + 1), e1 = (BSUB - 1 - k1) * (BL + 1), o1 = k1 * BL + BSUB - 1 - k1;
        const int d2 = k2 * (BL + 1), e2 = (BSUB - 1 - k2) * (BL + 1), o2 = k2 * BL + BSUB - 1 - k2;
        const bool pivot = k1 == k2;
        auto round = [&](const double* X, double* Y) {
            double u1, w1, u2, w2;
            const double x00 = X[i0], x01 = X[i0 + dc], x10 = X[i1], x11 = X[i1 + dc];
            rot_of<0, 1>(X[d1], X[e1], X[o1], u1, w1);
            rot_of<0, 1>(X[d2], X[e2], X[o2], u2, w2);
            const double y00 = u1 * x00 - w1 * x10, y10 = w1 * x00 + u1 * x10;
            const double y01 = u1 * x01 - w1 * x11, y11 = w1 * x01 + u1 * x11;
            Y[r0 + n0] = u2 * y00 - w2 * y01;
            Y[r0 + n1] = pivot ? 0.0 : w2 * y00 + u2 * y01;
            Y[r1 + n0] = pivot ? 0.0 : u2 * y10 - w2 * y11;
            Y[r1 + n1] = w2 * y10 + u2 * y11;
            __syncthreads();
        };
        for (int h = 0; h < BSUB / 2 - 1; ++h) {
            round(S[0], S[1]);
            round(S[1], S[0]);
        }
        round(S[0], S[1]);
    } else {
        const int i0 = k1 * BL + k2, dc = BSUB - 1 - 2 * k2;
        const int d2 = k2 * (BL + 1), e2 = (BSUB - 1 - k2) * (BL + 1), o2 = k2 * BL + BSUB - 1 - k2;
        const int ro = k1 * BL;
        auto round = [&](const double* X, const double* Vi, double* Vo) {
            double u, w;
            const double a0 = Vi[i0], a1 = Vi[i0 + dc], b0 = Vi[i0 + 16 * BL], b1 = Vi[i0 + 16 * BL + dc];
            rot_of<0, 1>(X[d2], X[e2], X[o2], u, w);
            Vo[ro + n0] = u * a0 - w * a1;
            Vo[ro + n1] = w * a0 + u * a1;
            Vo[ro + 16 * BL + n0] = u * b0 - w * b1;
            Vo[ro + 16 * BL + n1] = w * b0 + u * b1;
            __syncthreads();
        };
        for (int h = 0; h < BSUB / 2 - 1; ++h) {
            round(S[0], V2[0], V2[1]);
            round(S[1], V2[1], V2[0]);
        }
        round(S[0], V2[0], V2[1]);
    }
    const double* V = V2[1];
    double* G = V2[0];
    if (tid >= 256) {
        __syncthreads();
        return;
    }
    // one Newton-Schulz step, Q = V (3 I - V^T V) / 2, takes the factor's departure from orthogonality (the
    // rounding of its many rotations) from e to about e^2, so that it does not add up over the rounds
    // applied to the eigenvectors; a wave per 16 x 16 quadrant of each product
    const int lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = lane >> 4;
    const int r0 = (wave >> 1) * 16, c0 = (wave & 1) * 16;
    d4e g = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < BSUB; k += 4)
        g = __builtin_amdgcn_mfma_f64_16x16x4f64(V[(k + lk) * BL + r0 + lr], V[(k + lk) * BL + c0 + lr], g, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) G[(r0 + lk + 4 * e) * BL + c0 + lr] = g[e];
    __syncthreads();
    d4e h = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < BSUB; k += 4)
        h = __builtin_amdgcn_mfma_f64_16x16x4f64(V[(r0 + lr) * BL + k + lk], G[(k + lk) * BL + c0 + lr], h, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = r0 + lk + 4 * e, j = c0 + lr;
        Qb[i * BSUB + j] = 1.5 * V[i * BL + j] - 0.5 * h[e];
    }
}

// grid (npb / 2 + ceil(n / 32), npb / 2, batch), 256 threads: pair y's rows; x < npb / 2 the columns of pair x of
// A, else 32 columns of the transposed vectors Vt.  A wave per 16 x 16 quadrant; fragments straight from memory
// (L2), the half-transformed tile through LDS.
__global__ __launch_bounds__(256) void bj_apply_kernel(double* A, double* Vt, const double* Q, int n, int nblk, int npb,
                                                       int r, const int* active) {
    const int bm = blockIdx.z;
    if (!active[bm]) return;
    const int npair = npb / 2;
    const long long nn = (long long)n * n;
    const double* Qb = Q + (long long)bm * npair * BSUB * BSUB;
    const double* Qr = Qb + (long long)blockIdx.y * BSUB * BSUB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const int i0 = (wave >> 1) * 16, j0 = (wave & 1) * 16;
    int I, J;
    pair_of(r, blockIdx.y, npb, I, J);
    const bool isA = (int)blockIdx.x < npair;
    double* X = (isA ? A : Vt) + bm * nn;
    int CI = 0, CJ = 0, col;
    if (isA) {
        pair_of(r, blockIdx.x, npb, CI, CJ);
        col = bj_row(j0 + lr, CI, CJ, nblk, n);
    } else {
        col = ((int)blockIdx.x - npair) * 32 + j0 + lr;
        if (col >= n) col = -1;
    }
    // Q_r^T X: step s contracts local rows 4 s + lk
    d4e t = {0.0, 0.0, 0.0, 0.0};
    double xb[8], qa[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int row = bj_row(4 * s + lk, I, J, nblk, n);
        xb[s] = (row >= 0 && col >= 0) ? X[(long long)row * n + col] : 0.0;
        qa[s] = Qr[(4 * s + lk) * BSUB + i0 + lr];
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) t = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[s], xb[s], t, 0, 0, 0);
    __shared__ double T[BSUB * BL];
    if (isA) {
        const double* Qc = Qb + (long long)blockIdx.x * BSUB * BSUB;
        double qc[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) qc[s] = Qc[(4 * s + lk) * BSUB + j0 + lr];
#pragma unroll
        for (int e = 0; e < 4; ++e) T[(i0 + lk + 4 * e) * BL + j0 + lr] = t[e];
        __syncthreads();
        t = d4e{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 8; ++s)
            t = __builtin_amdgcn_mfma_f64_16x16x4f64(T[(i0 + lr) * BL + 4 * s + lk], qc[s], t, 0, 0, 0);
    } else {
        __syncthreads();  // the other row half of these columns has been read
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = bj_row(i0 + lk + 4 * e, I, J, nblk, n);
        if (row >= 0 && col >= 0) X[(long long)row * n + col] = t[e];
    }
}

// Vt = I, and a copy of A for the Rayleigh quotients
__global__ void bj_start_kernel(const double* A, double* A0, double* Vt, int n) {
    const long long nn = (long long)n * n, o = blockIdx.y * nn;
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < nn; t += (long long)gridDim.x * blockDim.x) {
        A0[o + t] = A[o + t];
        Vt[o + t] = (t / n == t % n) ? 1.0 : 0.0;
    }
}

// w[b][i] = v_i^T A0 v_i / v_i^T v_i for 16 vectors (rows of Vt) per workgroup: the rotated diagonal carries the
// rounding of every round (2e-15 relative), the Rayleigh quotient only that of its own products (6e-16); 16
// waves deal out the 16-column tiles of Vt A0, which goes to W.
__global__ __launch_bounds__(1024) void bj_rayleigh_kernel(const double* A0, const double* Vt, int n, double* w, double* W) {
    const long long o = (long long)blockIdx.y * n * n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const int i0 = blockIdx.x * 16, nt = (n + 15) / 16;
    const bool irow = i0 + lr < n;
    const double* vr = Vt + o + (long long)(irow ? i0 + lr : 0) * n;
    double num[4] = {0, 0, 0, 0}, den[4] = {0, 0, 0, 0};
    for (int c = wave; c < nt; c += 16) {
        const int col = c * 16 + lr;
        d4e acc = {0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < n; k += 4) {
            const int kk = k + lk;
            const double a = (irow && kk < n) ? vr[kk] : 0.0;
            const double b = (kk < n && col < n) ? A0[o + (long long)kk * n + col] : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + lk + 4 * e;
            const bool in = i < n && col < n;
            const double v = in ? Vt[o + (long long)i * n + col] : 0.0;
            if (in) W[o + (long long)i * n + col] = acc[e];
            num[e] += acc[e] * v;
            den[e] += v * v;
        }
    }
    __shared__ double sn[16][16], sd[16][16];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        for (int q = 8; q > 0; q >>= 1) {
            num[e] += __shfl_down(num[e], q, 16);
            den[e] += __shfl_down(den[e], q, 16);
        }
        if (lr == 0) { sn[wave][lk + 4 * e] = num[e]; sd[wave][lk + 4 * e] = den[e]; }
    }
    __syncthreads();
    if (threadIdx.x < 16 && i0 + (int)threadIdx.x < n) {
        double a = 0.0, b = 0.0;
        for (int k = 0; k < 16; ++k) { a += sn[k][threadIdx.x]; b += sd[k][threadIdx.x]; }
        w[(long long)blockIdx.y * n + i0 + threadIdx.x] = a / b;
    }
}

// The rotated vectors carry the rounding of every round too: V^T A0 V is diagonal only to 28 eps of the norm at
// n = 600 (14 at n = 200), which an eigenvector pair shows divided by its gap.  One first-order correction from the
// input matrix takes that out:  x_j += sum_i E_ij x_i  with, for r = I - V^T V and the residuals q_j = A0 x_j - w_j x_j,
//   E_ij = x_i . q_j / (w_j - w_i),   E_ji = r_ij - E_ij,   E_ii = r_ii / 2,
// and E_ij = E_ji = r_ij / 2 (orthogonality alone) for a pair whose rotation would exceed 2^-18: close clusters, whose
// vectors are any basis of their space.  Both elements of a pair come from one workgroup and one decision, so the
// correction is antisymmetric up to r; applied as E + E^2 / 2 + E^3 / 6 it is orthogonal to the rounding, which loose clusters
// need (400 eigenvalues within 1e-8: V^T V - I 3e-13 with E alone, where the rotations leave 1e-13).
// grid (nt (nt + 1) / 2, batch), 256 threads: the 16 x 16 tile pair (i tile <= j tile), K dealt to the waves; E[i][j].
__global__ __launch_bounds__(256) void bj_correct_kernel(const double* Vt, const double* W, const double* w, int n, double* E) {
    const long long o = (long long)blockIdx.y * n * n;
    const double* wb = w + (long long)blockIdx.y * n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const int nt = (n + 15) / 16;
    int ti = 0, p = blockIdx.x;
    while (p >= nt - ti) { p -= nt - ti; ++ti; }
    const int tj = ti + p, i = ti * 16 + lr, j = tj * 16 + lr;
    const bool ii = i < n, ij = j < n;
    const double* vi = Vt + o + (long long)(ii ? i : 0) * n;
    const double* vj = Vt + o + (long long)(ij ? j : 0) * n;
    const double* Wj = W + o + (long long)(ij ? j : 0) * n;
    const double wj = ij ? wb[j] : 0.0;
    d4e g = {0.0, 0.0, 0.0, 0.0}, q = g;
    for (int k0 = 16 * wave; k0 < n; k0 += 64)  // step s: k = k0 + 4 lk + s on both sides
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = k0 + 4 * lk + s;
            const double a = (ii && k < n) ? vi[k] : 0.0, b = (ij && k < n) ? vj[k] : 0.0;
            const double c = (ij && k < n) ? fma(-wj, b, Wj[k]) : 0.0;
            g = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, g, 0, 0, 0);
            q = __builtin_amdgcn_mfma_f64_16x16x4f64(a, c, q, 0, 0, 0);
        }
    __shared__ double sg[4][256], sq[4][256];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sg[wave][(lk + 4 * e) * 16 + lr] = g[e];
        sq[wave][(lk + 4 * e) * 16 + lr] = q[e];
    }
    __syncthreads();
    const int t = threadIdx.x, x = ti * 16 + (t >> 4), y = tj * 16 + (t & 15);
    if (x > y || y >= n) return;
    const double gs = ((sg[0][t] + sg[1][t]) + sg[2][t]) + sg[3][t], qs = ((sq[0][t] + sq[1][t]) + sq[2][t]) + sq[3][t];
    const double gap = wb[y] - wb[x], r = (x == y ? 1.0 : 0.0) - gs;
    const bool rot = x != y && fabs(qs) <= 0x1p-18 * fabs(gap);
    const double exy = rot && gap != 0.0 ? qs / gap : 0.5 * r;
    E[o + (long long)x * n + y] = exy;
    if (x != y) E[o + (long long)y * n + x] = r - exy;
}

// Out[j][k] = Vt[j][k] + f sum_i E[i][j] T[i][k], or as Out[k][j] (COLS: vectors as columns): grid (nt, nt, batch), 256
// threads, a 16 x 16 tile (j, k), i dealt to the waves; through LDS, so that lanes run along Out's rows.
template <bool COLS>
__global__ __launch_bounds__(256) void bj_update_kernel(const double* Vt, const double* E, const double* T, double f, int n,
                                                        double* Out) {
    const long long o = (long long)blockIdx.z * n * n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const int j0 = blockIdx.x * 16, k0 = blockIdx.y * 16, j = j0 + lr, k = k0 + lr;
    d4e d = {0.0, 0.0, 0.0, 0.0};
    for (int i0 = 16 * wave; i0 < n; i0 += 64)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int i = i0 + 4 * s + lk;
            const double a = (i < n && j < n) ? E[o + (long long)i * n + j] : 0.0;
            const double b = (i < n && k < n) ? T[o + (long long)i * n + k] : 0.0;
            d = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0);
        }
    __shared__ double sd[4][16][17];
#pragma unroll
    for (int e = 0; e < 4; ++e) sd[wave][lk + 4 * e][lr] = d[e];
    __shared__ double vt[16][17];
    const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
    vt[r][c] = (j0 + r < n && k0 + c < n) ? Vt[o + (long long)(j0 + r) * n + k0 + c] : 0.0;
    __syncthreads();
    const int x = COLS ? c : r, y = COLS ? r : c;  // element (j0 + x, k0 + y)
    if (j0 + x >= n || k0 + y >= n) return;
    Out[o + (COLS ? (long long)(k0 + y) * n + j0 + x : (long long)(j0 + x) * n + k0 + y)] =
        vt[x][y] + f * (((sd[0][x][y] + sd[1][x][y]) + sd[2][x][y]) + sd[3][x][y]);
}
}  // namespace

// once per process (thread-safe initialisation; retried if it throws)
static void small_attr() {
    static const bool set = [] {
        const int lds = (int)(2 * SMALL_MAX * (SMALL_MAX + 1) * sizeof(double));
        HIPCHK(hipFuncSetAttribute((const void*)jacobi_small_kernel<256>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        HIPCHK(hipFuncSetAttribute((const void*)jacobi_small_kernel<512>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        HIPCHK(hipFuncSetAttribute((const void*)jacobi_small_kernel<1024>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        return true;
    }();
    (void)set;
}

static void eig_small_batch(const double* A, int lda, int sym, int n, int nb, double* w, double* V, int desc, double* coef,
                            double* host, hipStream_t s) {
    if (g_dry) return;
    if (n <= 0 || nb <= 0) return;
    if (n > SMALL_MAX) fail(-1, "eig_small: n too large");
    small_attr();
    const int np = n + (n & 1);
    const size_t lds = 2 * (size_t)np * (np + 1) * sizeof(double);
    auto go = [&](auto kern, int nth) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(nth), lds, s, A, lda, sym, n, w, V, desc, coef, host);
    };
    switch (small_threads(n)) {
        case 256: go(jacobi_small_kernel<256>, 256); break;
        case 512: go(jacobi_small_kernel<512>, 512); break;
        default: go(jacobi_small_kernel<1024>, 1024);
    }
    LAUNCHCHK();
}

void eig_small_sorted(const double* A, int n, double* w, double* V, int desc, hipStream_t s) {
    eig_small_batch(A, n, 0, n, 1, w, V, desc ? 1 : 0, nullptr, nullptr, s);
}

void eig_small_gram(const double* A, int lda, int n, double* w, double* V, int desc, double* coef, double* host,
                    hipStream_t s) {
    eig_small_batch(A, lda, 1, n, 1, w, V, desc ? 1 : 0, coef, host, s);
}

namespace {
// doubles of scratch the block solver takes for nb matrices of order n: the pairs' factors, the matrices'
// copies, the transposed vectors, norms, flags
size_t block_scratch(int n, int nb) {
    const long long nblk = (n + BJ - 1) / BJ, npair = (nblk + (nblk & 1)) / 2;
    return (size_t)nb * npair * BSUB * BSUB + 2 * (size_t)nb * n * n + (size_t)nb * (2 * ONORM + 3) + 8;
}

// nb symmetric matrices of order n > SMALL_MAX, [nb][n][n]: eigenvalues w [nb][n] (unsorted) and
// eigenvectors V [nb][n][n] (columns), A overwritten; each matrix stops at its own convergence.
void eig_block(double* A, int n, int nb, double* w, double* V, double* scratch, hipStream_t s) {
    const long long nn = (long long)n * n;
    const int nblk = (n + BJ - 1) / BJ, npb = nblk + (nblk & 1), npair = npb / 2;
    double* Q = scratch;
    double* A0 = Q + (long long)nb * npair * BSUB * BSUB;    // [nb][n][n]
    double* Vt = A0 + nb * nn;                               // [nb][n][n]
    double* part = Vt + nb * nn;                             // [nb][ONORM][2]
    double* nrm = part + (long long)nb * 2 * ONORM;          // [nb][2]
    int* active = (int*)(nrm + 2 * (long long)nb);           // [nb]
    std::vector<int> hact(nb, 1);
    std::vector<double> hn(2 * (size_t)nb, INFINITY);
    HIPCHK(hipMemcpyAsync(active, hact.data(), nb * sizeof(int), hipMemcpyHostToDevice, s));
    HIPCHK(hipMemcpyAsync(nrm, hn.data(), 2 * nb * sizeof(double), hipMemcpyHostToDevice, s));
    for (int b0 = 0; b0 < nb; b0 += 65535) {
        const int c = std::min(65535, nb - b0);
        hipLaunchKernelGGL(bj_start_kernel, dim3(256, c), dim3(256), 0, s, A + b0 * nn, A0 + b0 * nn, Vt + b0 * nn, n);
    }
    LAUNCHCHK();
    const dim3 gs(npair, nb), ga(npair + (n + 31) / 32, npair, nb);
    for (int sweep = 0; sweep < 60; ++sweep) {
        // a matrix that is not (block) diagonal to begin with takes at least four sweeps: no check before
        if (sweep == 0 || sweep >= 4) {
            hipLaunchKernelGGL(offnorm_part_kernel, dim3(ONORM, nb), dim3(256), 0, s, A, n, part, active);
            hipLaunchKernelGGL(offnorm_sum_kernel, dim3(nb), dim3(64), 0, s, part, n, nrm, active);
            LAUNCHCHK();
            std::vector<int> now(nb);
            HIPCHK(hipMemcpyAsync(now.data(), active, nb * sizeof(int), hipMemcpyDeviceToHost, s));
            HIPCHK(hipMemcpyAsync(hn.data(), nrm, 2 * nb * sizeof(double), hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            int left = 0;
            for (int b = 0; b < nb; ++b) {
                if (hact[b] && !now[b] && (!std::isfinite(hn[2 * b]) || !std::isfinite(hn[2 * b + 1])))
                    fail(-4, "eigensolver: non-finite matrix");
                hact[b] = now[b];
                left += now[b];
            }
            if (left == 0) break;
        }
        for (int r = 0; r < npb - 1; ++r) {
            hipLaunchKernelGGL(bj_solve_kernel, gs, dim3(512), 0, s, A, Q, n, nblk, npb, r, nrm, active);
            hipLaunchKernelGGL(bj_apply_kernel, ga, dim3(256), 0, s, A, Vt, Q, n, nblk, npb, r, active);
        }
        LAUNCHCHK();
    }
    // A is free from here on (it takes Vt A0), and A0 after the quotients (it takes the correction E):
    // V = Vt + E^T (Vt + E^T (Vt + E^T Vt / 3) / 2), by way of V and A
    const int nt = (n + 15) / 16;
    hipLaunchKernelGGL(bj_rayleigh_kernel, dim3(nt, nb), dim3(1024), 0, s, A0, Vt, n, w, A);
    hipLaunchKernelGGL(bj_correct_kernel, dim3(nt * (nt + 1) / 2, nb), dim3(256), 0, s, Vt, A, w, n, A0);
    const dim3 gu(nt, nt, nb);
    hipLaunchKernelGGL(bj_update_kernel<false>, gu, dim3(256), 0, s, Vt, A0, Vt, 1.0 / 3.0, n, V);
    hipLaunchKernelGGL(bj_update_kernel<false>, gu, dim3(256), 0, s, Vt, A0, V, 0.5, n, A);
    hipLaunchKernelGGL(bj_update_kernel<true>, gu, dim3(256), 0, s, Vt, A0, A, 1.0, n, V);
    LAUNCHCHK();
}
}  // namespace

// the block solver's factors, copies, norms and flags
size_t eig_large_scratch(int n) { return block_scratch(n, 1); }

void eig_large(double* A, int n, double* w, double* V, double* scratch, hipStream_t s) {
    eig_batched(A, n, 1, w, V, scratch, s);
}

// the block solver's factors, copies, norms and flags of the nb matrices
size_t eig_batched_scratch(int n, int nb) { return block_scratch(n, nb); }

void eig_batched(double* A, int n, int nb, double* w, double* V, double* scratch, hipStream_t s) {
    if (g_dry) return;
    ProfScope prof(PROF_EIG, s, 0.0, 0.0);
    if (n <= 0 || nb <= 0) return;
    if (n <= SMALL_MAX) {
        eig_small_batch(A, n, 0, n, nb, w, V, -1, nullptr, nullptr, s);
        return;
    }
    eig_block(A, n, nb, w, V, scratch, s);
}

void k_sort_eig(double* w, double* V, int n, int desc, double* wtmp, double* Vtmp, hipStream_t s) {
    if (g_dry) return;
    if (n <= 0) return;
    hipLaunchKernelGGL(sort_rank_kernel, dim3((n + 15) / 16), dim3(256), 0, s, w, V, n, desc, wtmp, Vtmp);
    hipLaunchKernelGGL(sort_copy_kernel, dim3((unsigned)std::min(256, (n * n + 255) / 256)), dim3(256), 0, s, w, V, n,
                       wtmp, Vtmp);
    LAUNCHCHK();
}

}  // namespace adc3
