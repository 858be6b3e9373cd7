// Deterministic FP64 reductions used by the Davidson solver.
//
// Inner products G = X Y^T of a few long vectors are a GEMM with a huge K: the K
// axis is cut into fixed chunks, each chunk is one batch of the matrix-core GEMM
// (every vector element is read once; ~n/1024 workgroups keep the chip busy), and
// the per-chunk partial Gram blocks are summed by one workgroup per output element
// in a fixed order -- the result does not depend on scheduling.
#include "internal.h"
#include <algorithm>

namespace adc3 {

namespace {
inline long long chunk_of(long long n) { return std::max<long long>(256, (n + 8191) / 8192); }

// G[p*ldg + q] = sum_c partial[c][r][s] with (r,s) = (p,q) or (q,p) when swapped.  m0 >= 0: G is the block of columns
// m0 .. of a symmetric matrix (G = matrix + m0): the element goes to its mirrored place too, and of the block's own square
// (rows m0 ..) the upper half counts.
__global__ void sum_partials_kernel(const double* partial, long long nchunk, int M, int N, int swapped, double* G,
                                    int ldg, int m0) {
    const int t = blockIdx.x;  // output element of the partial [M][N] block
    const long long MN = (long long)M * N;
    double acc = 0.0;
    for (long long c = threadIdx.x; c < nchunk; c += blockDim.x) acc += partial[c * MN + t];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    __shared__ double red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = red[0] + red[1] + red[2] + red[3];
        int r = t / N, q = t % N;
        const int i = swapped ? q : r, j = swapped ? r : q;
        if (m0 >= 0 && i - m0 > j) return;
        G[(long long)i * ldg + j] = s;
        if (m0 >= 0) G[(long long)(m0 + j) * ldg + i - m0] = s;
    }
}
// Small Gram blocks (at most 64 products, e.g. residual norms and the Gram of a new block): one pass on the vector ALUs,
// bound by the stream over the rows.  A workgroup takes one chunk of the long axis, all np (<= PG) rows of X against all
// nq (<= NQ) rows of Y, two elements of each row per thread and step with every row's load in flight together; the products
// accumulate in registers, a butterfly that halves the values held per step reduces them over the wave (63 exchanges for
// 64 products, not 64 x 6), and the workgroup writes partial[c][p][q], all in a fixed order.  16 rows against one at
// n = 185000: 63 us with each row's load waited for and 64 rows unrolled, 7.6 now; 5 against 5 at n = 230000: 24 and 9.
typedef double d2v __attribute__((ext_vector_type(2), aligned(8)));

template <int H, int NV>
__device__ inline void wave_halve(double (&v)[NV], int lane) {
    // lanes with bit H set keep the upper half of the values
    if constexpr (NV > 1) {
        constexpr int h = NV / 2;
        const bool up = lane & H;
        double w[h];
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const double send = up ? v[i] : v[i + h], keep = up ? v[i + h] : v[i];
            w[i] = keep + __shfl_xor(send, H, 64);
        }
        wave_halve<H / 2, h>(w, lane);
        v[0] = w[0];
    } else if constexpr (H > 0) {
        v[0] += __shfl_xor(v[0], H, 64);
        wave_halve<H / 2, 1>(v, lane);
    }
}

template <int NQ, int PG>
__global__ __launch_bounds__(256) void dots_small_kernel(const double* X, long long ldx, int np, const double* Y,
                                                         long long ldy, int nq, long long n, long long chunk,
                                                         double* partial) {
    constexpr int NV = PG * NQ;  // a power of two, at most 64
    const long long c0 = (long long)blockIdx.x * chunk, c1 = min(n, c0 + chunk);
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    for (long long t = c0 + 2 * threadIdx.x; t < c1; t += 512) {
        const bool two = t + 1 < c1;
        d2v x[PG], y[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double* r = Y + min(q, nq - 1) * ldy + t;
            if (two) y[q] = *(const d2v*)r;
            else y[q] = d2v{*r, 0.0};
        }
#pragma unroll
        for (int p = 0; p < PG; ++p) {
            x[p] = d2v{0.0, 0.0};
            if (p < np) {
                const double* r = X + p * ldx + t;
                if (two) x[p] = *(const d2v*)r;
                else x[p] = d2v{*r, 0.0};
            }
        }
#pragma unroll
        for (int p = 0; p < PG; ++p)
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[p * NQ + q] += x[p].x * y[q].x + x[p].y * y[q].y;
    }
    __shared__ double red[4][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_halve<32, NV>(acc, lane);
    // value k sits in the lanes whose top bits spell k
    constexpr int L = 64 / NV;
    if (lane % L == 0) red[wave][lane / L] = acc[0];
    __syncthreads();
    const int k = threadIdx.x;
    if (k < NV) {
        const int p = k / NQ, q = k % NQ;
        if (p < np && q < nq)
            partial[((long long)blockIdx.x * np + p) * nq + q] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

// Y[q][t] = alpha * sum_p C[p][q] X[p][t] + beta * Y[q][t] for nq <= NQ rows: each thread E elements
// (stride 256), the coefficients uniform across the wave, X streamed once.
template <int NQ, int E>
__global__ __launch_bounds__(256) void lincomb_kernel(double* Y, long long ldy, int nq, const double* X, long long ldx,
                                                      int np, const double* C, int ldc, long long n, double alpha,
                                                      double beta) {
    const long long base = (long long)blockIdx.x * (256 * E) + threadIdx.x;
    double acc[E][NQ];
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[e][q] = 0.0;
    for (int p = 0; p < np; ++p) {
        double x[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const long long t = base + 256LL * e;
            x[e] = t < n ? X[p * ldx + t] : 0.0;
        }
        const double* cp = C + (long long)p * ldc;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double c = q < nq ? cp[q] : 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e][q] += c * x[e];
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q >= nq) break;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const long long t = base + 256LL * e;
            if (t < n) {
                double* y = Y + q * ldy + t;
                *y = alpha * acc[e][q] + (beta == 0.0 ? 0.0 : beta * *y);
            }
        }
    }
}

// Rayleigh-Ritz vectors and residuals of nq <= NQ roots in one pass over V and S (rows 0..m-1 of n):
//   X[q] = sum_p Y[p][q] V[p],   R[q] = sum_p Y[p][q] S[p] - th[q] X[q],   part[block][q] = partial |R[q]|^2
// bound by the stream of V and S (o=16 v=120, 5 roots, m = 30: 27 us for 0.13 GB, 55 as
// two products, a residual pass and a Gram).
template <int NQ>
__global__ __launch_bounds__(256) void ritz_kernel(const double* V, const double* S, long long n, int m, const double* Y,
                                                   int ldy, int nq, const double* th, double* X, double* R, double* part,
                                                   int ldp) {
    double nrm[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) nrm[q] = 0.0;
    for (long long t = 2 * ((long long)blockIdx.x * 256 + threadIdx.x); t < n; t += 512LL * gridDim.x) {
        const bool two = t + 1 < n;
        auto ld = [&](const double* p) {
            if (two) return *(const d2v*)p;
            return d2v{*p, 0.0};
        };
        d2v x[NQ], ax[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) x[q] = ax[q] = d2v{0.0, 0.0};
#pragma unroll 4
        for (int p = 0; p < m; ++p) {
            const d2v a = ld(V + p * n + t), b = ld(S + p * n + t);
            const double* c = Y + (long long)p * ldy;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const double y = q < nq ? c[q] : 0.0;
                x[q] += y * a;
                ax[q] += y * b;
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (q >= nq) break;
            const d2v r = ax[q] - th[q] * x[q];
            nrm[q] += r.x * r.x + r.y * r.y;
            double *xo = X + q * n + t, *ro = R + q * n + t;
            if (two) {
                *(d2v*)xo = x[q];
                *(d2v*)ro = r;
            } else {
                *xo = x[q].x;
                *ro = r.x;
            }
        }
    }
    __shared__ double red[4][NQ];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_halve<32, NQ>(nrm, lane);
    constexpr int L = 64 / NQ;
    if (lane % L == 0) red[wave][lane / L] = nrm[0];
    __syncthreads();
    const int q = threadIdx.x;
    if (q < nq) part[(long long)blockIdx.x * ldp + q] = ((red[0][q] + red[1][q]) + red[2][q]) + red[3][q];
}

// host[q] = sum_b part[b][q], host[nr + q] = ev[q] (host memory the device can write), th[q] = ev[q]
__global__ __launch_bounds__(256) void ritz_norms_kernel(const double* part, int nb, int nr, const double* ev, double* th,
                                                         double* host) {
    const int q = blockIdx.x;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) acc += part[(long long)b * nr + q];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    __shared__ double red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        host[q] = red[0] + red[1] + red[2] + red[3];
        host[nr + q] = ev[q];
        th[q] = ev[q];
    }
}

// T[q] = f_q (T[q] - sum_p C[p][q] V[p]) for nq <= NQ rows, f_q = 1 / sqrt(C[m + q][q]) (0 where that is not positive) if
// scale, else 1: new directions brought to unit length and projected against V in one pass, C holding the inner
// products with V's rows and, below them, with the directions themselves.
template <int NQ>
__global__ __launch_bounds__(256) void project_kernel(double* T, const double* V, long long n, int m, const double* C,
                                                      int ldc, int nq, int scale) {
    double f[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const double g = scale && q < nq ? C[(long long)(m + q) * ldc + q] : 1.0;
        f[q] = g > 0.0 ? 1.0 / sqrt(g) : 0.0;
    }
    for (long long t = 2 * ((long long)blockIdx.x * 256 + threadIdx.x); t < n; t += 512LL * gridDim.x) {
        const bool two = t + 1 < n;
        auto ld = [&](const double* p) {
            if (two) return *(const d2v*)p;
            return d2v{*p, 0.0};
        };
        d2v x[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) x[q] = q < nq ? ld(T + q * n + t) : d2v{0.0, 0.0};
#pragma unroll 4
        for (int p = 0; p < m; ++p) {
            const d2v a = ld(V + p * n + t);
            const double* c = C + (long long)p * ldc;
#pragma unroll
            for (int q = 0; q < NQ; ++q) x[q] -= (q < nq ? c[q] : 0.0) * a;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (q >= nq) break;
            const d2v y = f[q] > 0.0 ? f[q] * x[q] : d2v{0.0, 0.0};
            double* o = T + q * n + t;
            if (two) *(d2v*)o = y;
            else *o = y.x;
        }
    }
}

template <int NQ>
void launch_lincomb(double* Y, long long ldy, int nq, const double* X, long long ldx, int np, const double* C, int ldc,
                    long long n, double alpha, double beta, hipStream_t s) {
    constexpr int E = NQ <= 8 ? 4 : 2;
    const long long nb = (n + 256 * E - 1) / (256 * E);
    hipLaunchKernelGGL((lincomb_kernel<NQ, E>), dim3((unsigned)nb), dim3(256), 0, s, Y, ldy, nq, X, ldx, np, C, ldc, n,
                       alpha, beta);
}

template <int NQ, int PG>
void launch_dots_small(const double* X, long long ldx, int np, const double* Y, long long ldy, int nq, long long n,
                       long long chunk, long long nchunk, double* partial, hipStream_t s) {
    if constexpr (PG > NQ) {
        if (np <= PG / 2) {
            launch_dots_small<NQ, PG / 2>(X, ldx, np, Y, ldy, nq, n, chunk, nchunk, partial, s);
            return;
        }
    }
    hipLaunchKernelGGL((dots_small_kernel<NQ, PG>), dim3((unsigned)nchunk), dim3(256), 0, s, X, ldx, np, Y, ldy, nq, n, chunk,
                       partial);
}
}  // namespace

size_t dots_partial_elems(int np, int nq, long long n) {
    return (size_t)(n / chunk_of(n) + 2) * np * nq;
}

void k_dots(const double* X, long long ldx, int np, const double* Y, long long ldy, int nq, long long n, double* G,
            int ldg, double* partial, hipStream_t s, int mirror) {
    if (g_dry) return;
    if (np <= 0 || nq <= 0) return;
    // rows of the GEMM = the smaller set (skinny tiles when it is <= 16)
    const bool swapped = nq < np;
    const double* A = swapped ? Y : X;
    const double* B = swapped ? X : Y;
    const long long lda = swapped ? ldy : ldx, ldb = swapped ? ldx : ldy;
    const int M = swapped ? nq : np, N = swapped ? np : nq;
    const long long MN = (long long)M * N;
    // at most 64 products with one row group: the vector-ALU pass (A's rows against B's columns, the
    // partials laid out [chunk][M][N] as the GEMM's)
    if (n > 0 && M <= 8 && N <= 16 && (long long)N * ((M + 3) / 4 * 4) <= 64) {
        // three workgroups a CU for long vectors, one step per workgroup for short ones
        const long long ch = std::max<long long>(1, (n + 768 * 512 - 1) / (768 * 512)) * 512;
        const long long nch = (n + ch - 1) / ch;
        if (nch <= 65535 && nch * MN <= (long long)dots_partial_elems(np, nq, n)) {
            // rows of the output: the N operand rows against M (<= 8) operand rows
            if (M <= 1) launch_dots_small<1, 16>(B, ldb, N, A, lda, M, n, ch, nch, partial, s);
            else if (M <= 2) launch_dots_small<2, 16>(B, ldb, N, A, lda, M, n, ch, nch, partial, s);
            else if (M <= 4) launch_dots_small<4, 16>(B, ldb, N, A, lda, M, n, ch, nch, partial, s);
            else launch_dots_small<8, 8>(B, ldb, N, A, lda, M, n, ch, nch, partial, s);
            LAUNCHCHK();
            // partial[c][r][m] with r over the N operand: the transposed block of the GEMM's layout
            hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)MN), dim3(256), 0, s, partial, nch, N, M,
                               swapped ? 0 : 1, G, ldg, mirror);
            LAUNCHCHK();
            return;
        }
    }
    // up to 16 x 256 products: the fragment-streaming skinny kernel (partials [chunk][M][N] as the GEMM's)
    if (n > 0 && M <= 16 && N <= 256) {
        const long long nch = abt_skinny(M, N, n, A, lda, B, ldb, partial, (long long)dots_partial_elems(np, nq, n), s);
        if (nch > 0) {
            hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)MN), dim3(256), 0, s, partial, nch, M, N,
                               swapped ? 1 : 0, G, ldg, mirror);
            LAUNCHCHK();
            return;
        }
    }
    const long long CH = chunk_of(n);
    long long nchunk = (n + CH - 1) / CH;
    if (nchunk == 0) {
        k_fill(partial, MN, 0.0, s);
        nchunk = 1;
    } else {
        if (nchunk > 65535) fail(-1, "k_dots: vectors too long");
        Gemm g;
        g.M = M; g.N = N; g.K = (int)CH;
        g.Klast = (int)(n - (nchunk - 1) * CH);
        g.A = A; g.sAm = lda; g.sAk = 1; g.bA0 = CH;
        g.B = B; g.sBk = 1; g.sBn = ldb; g.bB0 = CH;
        g.C = partial; g.sCm = N; g.sCn = 1; g.bC0 = MN;
        g.nb0 = (int)nchunk;
        gemm(g, s);
    }
    hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)MN), dim3(256), 0, s, partial, nchunk, M, N,
                       swapped ? 1 : 0, G, ldg, mirror);
    LAUNCHCHK();
}

void k_ritz(const double* V, const double* S, long long n, int m, const double* Y, int ldy, int nr, const double* ev,
           double* X, double* R, double* part, double* th, double* host, hipStream_t s) {
    if (g_dry || nr <= 0 || n <= 0) return;
    const int nb = (int)std::min<long long>(2048, (n + 511) / 512);
    for (int q0 = 0; q0 < nr; q0 += 8) {
        const int nq = std::min(8, nr - q0);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, V, S, n, m, Y + q0, ldy, nq, ev + q0, X + q0 * n, R + q0 * n,
                               part + q0, nr);
        };
        if (nq <= 1) go(ritz_kernel<1>);
        else if (nq <= 2) go(ritz_kernel<2>);
        else if (nq <= 4) go(ritz_kernel<4>);
        else go(ritz_kernel<8>);
    }
    hipLaunchKernelGGL(ritz_norms_kernel, dim3(nr), dim3(256), 0, s, part, nb, nr, ev, th, host);
    LAUNCHCHK();
}

void k_project(double* T, int nq, const double* V, int m, long long n, const double* C, int ldc, int scale, hipStream_t s) {
    if (g_dry || nq <= 0 || n <= 0) return;
    if (nq > 16) fail(-1, "k_project: more than 16 rows");
    const int nb = (int)std::min<long long>(4096, (n + 511) / 512);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, T, V, n, m, C, ldc, nq, scale); };
    if (nq <= 1) go(project_kernel<1>);
    else if (nq <= 2) go(project_kernel<2>);
    else if (nq <= 4) go(project_kernel<4>);
    else if (nq <= 8) go(project_kernel<8>);
    else go(project_kernel<16>);
    LAUNCHCHK();
}

void k_lincomb(double* Y, long long ldy, int nq, const double* X, long long ldx, int np, const double* C, int ldc,
               long long n, double alpha, double beta, hipStream_t s) {
    if (g_dry) return;
    if (nq <= 0 || n <= 0) return;
    // few output rows: the streaming kernel (one pass over X, coefficients in scalar registers)
    if (nq <= 16 && np <= 128 && (n + 1023) / 1024 <= 0x7fffffffLL) {
        if (nq <= 1) launch_lincomb<1>(Y, ldy, nq, X, ldx, np, C, ldc, n, alpha, beta, s);
        else if (nq <= 2) launch_lincomb<2>(Y, ldy, nq, X, ldx, np, C, ldc, n, alpha, beta, s);
        else if (nq <= 4) launch_lincomb<4>(Y, ldy, nq, X, ldx, np, C, ldc, n, alpha, beta, s);
        else if (nq <= 8) launch_lincomb<8>(Y, ldy, nq, X, ldx, np, C, ldc, n, alpha, beta, s);
        else launch_lincomb<16>(Y, ldy, nq, X, ldx, np, C, ldc, n, alpha, beta, s);
        LAUNCHCHK();
        return;
    }
    for (long long c0 = 0; c0 < n; c0 += 2000000000LL) {
        long long nn = std::min<long long>(n - c0, 2000000000LL);
        Gemm g;
        g.M = nq; g.N = (int)nn; g.K = np;
        g.A = C; g.sAm = 1; g.sAk = ldc;
        g.B = X + c0; g.sBk = ldx; g.sBn = 1;
        g.C = Y + c0; g.sCm = ldy; g.sCn = 1;
        g.alpha = alpha; g.beta = beta;
        gemm(g, s);
    }
}

}  // namespace adc3
