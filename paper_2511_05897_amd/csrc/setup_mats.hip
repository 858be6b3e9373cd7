// Matrices of a context's setup over occupied-virtual pairs, and the passes that assemble its tensors from them.
//
// The o^3 v^3 contractions of the setup all run over one (occupied, virtual) pair, so their operands are kept as
// (ov) x (ov) matrices with rows of ldm = ov rounded up to even (16-byte rows for the k-major GEMM tiles; the pad
// column is never read into a result):
//   g [(ia)][(jb)] = (ia|jb)      h [(ia)][(jb)] = (ij|ab)       (both symmetric)
//   Tm[(ia)][(jb)] = T_ij^ab      Tx[(ia)][(jb)] = T_ij^ba       S = 2 Tm - Tx
// The second-order doubles and the ring part of M11 need the same two products (see build_ctx in adc.hip),
//   RB = Tm h - S g,   RC = -Tx h,
// three GEMMs where the terms written out one by one are eleven, each with its operands permuted.  A whole context
// with its first sigma vector: o=20 v=200 X=128 97.0 -> 71.5 ms (of which 40 ms are the two coupling products over
// (k,d), 63 TFLOP/s), o=9 v=83 X=249 4.46 -> 2.09 ms (230 -> 153 launches of which most are launch bound).
// The kernels here are streams (32 x 32 tiles transposed through LDS where an index pair is exchanged), bound by
// HBM: at o=20 v=200 uz_form_kernel moves 6.4 GB in 1.32 ms (4.9 TB/s; the permutes and passes it replaces took
// 4.6 ms), ovvv_perm_kernel 2.6 GB in 0.50 ms, pair_comb_kernel 0.26-0.38 GB in 0.07 ms.
#include "internal.h"
#include <algorithm>

namespace adc3 {

namespace {
constexpr int TS = 32;

// Tm[(ia)][(jb)] = g[(ia)][(jb)] / (e_i + e_j - e_a - e_b), and the same as blocks T[i][j][a][b]
__global__ void amp_mat_kernel(const double* g, const double* eo, const double* ev, int o, int v, long long ld, double* Tm,
                               double* T) {
    const int ov = o * v;
    for (int ia = blockIdx.y; ia < ov; ia += gridDim.y) {
        const int i = ia / v, a = ia - i * v;
        for (int jb = blockIdx.x * blockDim.x + threadIdx.x; jb < ov; jb += gridDim.x * blockDim.x) {
            const int j = jb / v, b = jb - j * v;
            const double t = g[ia * ld + jb] / (eo[i] + eo[j] - ev[a] - ev[b]);
            if (Tm) Tm[ia * ld + jb] = t;
            T[(((long long)i * o + j) * v + a) * v + b] = t;
        }
    }
}

struct PairView {  // element (i, j, a, b) at i si + j sj + a sr + b
    long long si, sj, sr;
};

// out(i,j,a,b) = ca in(i,j,a,b) + cb in(i,j,b,a)
__global__ __launch_bounds__(256) void pair_comb_kernel(double* out, PairView vo, const double* in, PairView vi, int o,
                                                        int v, int nt, double ca, double cb) {
    __shared__ double t2[TS][TS + 1];
    const int ta = blockIdx.x / nt, tb = blockIdx.x - ta * nt;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int ij = blockIdx.y; ij < o * o; ij += gridDim.y) {
        const int i = ij / o, j = ij - i * o;
        const double* X = in + i * vi.si + j * vi.sj;
        double* Y = out + i * vo.si + j * vo.sj;
        __syncthreads();
        for (int r = ty; r < TS; r += 8) {  // the mirrored tile: rows b, columns a
            const int b = tb * TS + r, a = ta * TS + tx;
            t2[r][tx] = (a < v && b < v) ? X[b * vi.sr + a] : 0.0;
        }
        __syncthreads();
        for (int r = ty; r < TS; r += 8) {
            const int a = ta * TS + r, b = tb * TS + tx;
            if (a < v && b < v) Y[a * vo.sr + b] = ca * X[a * vi.sr + b] + cb * t2[tx][r];
        }
    }
}

// U[(ia)][(jb)] = (LH[i][j][a][b] - RB[(ia)][(jb)] - RB[(jb)][(ia)] + RC[(ja)][(ib)] + RC[(ib)][(ja)]) / (e_i + e_j - e_a - e_b)
__global__ __launch_bounds__(256) void doubles_kernel(double* U, const double* LH, const double* RB, const double* RC,
                                                      const double* eo, const double* ev, int o, int v, long long ld,
                                                      int nt) {
    __shared__ double t1[TS][TS + 1], t2[TS][TS + 1];
    const int ta = blockIdx.x / nt, tb = blockIdx.x - ta * nt;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int ij = blockIdx.y; ij < o * o; ij += gridDim.y) {
        const int i = ij / o, j = ij - i * o;
        const long long bij = (long long)i * v * ld + (long long)j * v, bji = (long long)j * v * ld + (long long)i * v;
        __syncthreads();
        for (int r = ty; r < TS; r += 8) {
            const int b = tb * TS + r, a = ta * TS + tx;
            const bool in = a < v && b < v;
            t1[r][tx] = in ? RB[bji + b * ld + a] : 0.0;
            t2[r][tx] = in ? RC[bij + b * ld + a] : 0.0;
        }
        __syncthreads();
        for (int r = ty; r < TS; r += 8) {
            const int a = ta * TS + r, b = tb * TS + tx;
            if (a >= v || b >= v) continue;
            const double y = LH[((long long)ij * v + a) * v + b] - (RB[bij + a * ld + b] + t1[tx][r]) +
                             (RC[bji + a * ld + b] + t2[tx][r]);
            U[bij + a * ld + b] = y / (eo[i] + eo[j] - ev[a] - ev[b]);
        }
    }
}

// G2[(k,d)][(a,c)] = V1[(k,a)][(c,d)] for a < nc (rows of G2 of length ldg)
__global__ __launch_bounds__(256) void ovvv_perm_kernel(double* G2, long long ldg, const double* V1, int nc, int v, int nt) {
    __shared__ double t[TS][TS + 1];
    const int tc = blockIdx.x / nt, td = blockIdx.x - tc * nt;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int a = blockIdx.y;
    const long long k = blockIdx.z;
    const double* X = V1 + (k * nc + a) * (long long)v * v;
    for (int r = ty; r < TS; r += 8) {
        const int c = tc * TS + r, d = td * TS + tx;
        if (c < v && d < v) t[r][tx] = X[(long long)c * v + d];
    }
    __syncthreads();
    for (int r = ty; r < TS; r += 8) {
        const int d = td * TS + r, c = tc * TS + tx;
        if (c < v && d < v) G2[(k * v + d) * ldg + (long long)a * v + c] = t[tx][r];
    }
}

// U_z[a][i][b][c] = S + sqrt3 A over (b,c) of
//   D[b][c] = F[(a,b)][(i,c)] + U_z[a][i][b][c] - x2 (C1[(i,b)][(a,c)] + C2[(i,c)][(a,b)])
// (level 2: C1 = C2 = null and U_z is not read).  A workgroup takes a tile pair (tb <= tc) of one (a, i).
__global__ __launch_bounds__(256) void uz_form_kernel(double* Uz, const double* F, const double* C1, const double* C2,
                                                      long long ldc, double x2, int nc, int o, int v) {
    const double s3 = 1.73205080756887729353;
    __shared__ double d1[TS][TS + 1], d2[TS][TS + 1], u1[TS][TS + 1], u2[TS][TS + 1];
    const int nt = (v + TS - 1) / TS;
    int tb = 0, p = blockIdx.x;
    while (p >= nt - tb) { p -= nt - tb; ++tb; }
    const int tc = tb + p;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const long long ov = (long long)o * v;
    for (long long ai = blockIdx.y; ai < (long long)nc * o; ai += gridDim.y) {
        const int a = (int)(ai / o), i = (int)(ai - (long long)a * o);
        const double* Fa = F + (long long)a * v * ov + (long long)i * v;  // [b][.. c], rows of ov
        double* Ua = Uz + ai * v * v;
        const double* C1a = C1 ? C1 + (long long)i * v * ldc + (long long)a * v : nullptr;  // [b][c], rows of ldc
        const double* C2a = C2 ? C2 + (long long)i * v * ldc + (long long)a * v : nullptr;  // [c][b], rows of ldc
        __syncthreads();
        for (int r = ty; r < TS; r += 8) {
            const int b = tb * TS + r, c = tc * TS + tx;  // D[b][c]
            double x = 0.0, y = 0.0;
            if (b < v && c < v) {
                x = Fa[b * ov + c];
                if (C1) { x += Ua[(long long)b * v + c] - x2 * C1a[b * ldc + c]; y = C2a[b * ldc + c]; }
            }
            d1[r][tx] = x;
            u2[r][tx] = y;  // C2 at (c' = b, b' = c)
            const int b2 = tc * TS + r, c2 = tb * TS + tx;  // D[b2][c2], the mirrored tile
            x = 0.0;
            y = 0.0;
            if (b2 < v && c2 < v) {
                x = Fa[b2 * ov + c2];
                if (C1) { x += Ua[(long long)b2 * v + c2] - x2 * C1a[b2 * ldc + c2]; y = C2a[b2 * ldc + c2]; }
            }
            d2[r][tx] = x;
            u1[r][tx] = y;  // C2 at (c' = b2, b' = c2)
        }
        __syncthreads();
        double w1[4], w2[4];
        for (int q = 0; q < 4; ++q) {
            const int r = ty + 8 * q;
            // D[b][c] = d1[b][c] - x2 C2[c][b], with C2[c][b] = u1[c][b]; D[c][b] = d2[c][b] - x2 u2[b][c]
            w1[q] = d1[r][tx] - x2 * u1[tx][r];  // (b = r, c = tx)
            w2[q] = d2[r][tx] - x2 * u2[tx][r];  // (b2 = r, c2 = tx)
        }
        __syncthreads();
        for (int q = 0; q < 4; ++q) { d1[ty + 8 * q][tx] = w1[q]; d2[ty + 8 * q][tx] = w2[q]; }
        __syncthreads();
        for (int r = ty; r < TS; r += 8) {
            const int b = tb * TS + r, c = tc * TS + tx;
            if (b < v && c < v) {
                const double x = d1[r][tx], y = d2[tx][r];
                Ua[(long long)b * v + c] = 0.5 * (x + y) + s3 * 0.5 * (x - y);
            }
            const int b2 = tc * TS + r, c2 = tb * TS + tx;
            if (tb != tc && b2 < v && c2 < v) {
                const double x = d2[r][tx], y = d1[tx][r];
                Ua[(long long)b2 * v + c2] = 0.5 * (x + y) + s3 * 0.5 * (x - y);
            }
        }
    }
}
}  // namespace

void k_amp_mat(const double* g, const double* eo, const double* ev, int o, int v, long long ld, double* Tm, double* T,
               hipStream_t s) {
    if (g_dry || o <= 0 || v <= 0) return;
    hipLaunchKernelGGL(amp_mat_kernel, dim3((unsigned)std::min((o * v + 255) / 256, 64), (unsigned)std::min(o * v, 65535)), dim3(256), 0, s,
                       g, eo, ev, o, v, ld, Tm, T);
    LAUNCHCHK();
}

static PairView view(long long ld, int o, int v) {
    // ld > 0: matrix [(ia)][(jb)] with rows of ld; 0: blocks [i][j][a][b]
    if (ld > 0) return PairView{v * ld, v, ld};
    return PairView{(long long)o * v * v, (long long)v * v, v};
}

void k_pair_comb(double* out, long long ldo, const double* in, long long ldi, int o, int v, double ca, double cb,
                 hipStream_t s) {
    if (g_dry || o <= 0 || v <= 0) return;
    const int nt = (v + TS - 1) / TS;
    hipLaunchKernelGGL(pair_comb_kernel, dim3((unsigned)(nt * nt), (unsigned)std::min(o * o, 65535)), dim3(256), 0, s, out,
                       view(ldo, o, v), in, view(ldi, o, v), o, v, nt, ca, cb);
    LAUNCHCHK();
}

void k_doubles(double* U, const double* LH, const double* RB, const double* RC, const double* eo, const double* ev, int o,
               int v, long long ld, hipStream_t s) {
    if (g_dry || o <= 0 || v <= 0) return;
    const int nt = (v + TS - 1) / TS;
    hipLaunchKernelGGL(doubles_kernel, dim3((unsigned)(nt * nt), (unsigned)std::min(o * o, 65535)), dim3(256), 0, s, U, LH, RB,
                       RC, eo, ev, o, v, ld, nt);
    LAUNCHCHK();
}

void k_ovvv_perm(double* G2, long long ldg, const double* V1, int o, int nc, int v, hipStream_t s) {
    if (g_dry || o <= 0 || v <= 0 || nc <= 0) return;
    const int nt = (v + TS - 1) / TS;
    hipLaunchKernelGGL(ovvv_perm_kernel, dim3((unsigned)(nt * nt), (unsigned)nc, (unsigned)o), dim3(256), 0, s, G2, ldg, V1, nc,
                       v, nt);
    LAUNCHCHK();
}

void k_uz_form(double* Uz, const double* F, const double* C1, const double* C2, long long ldc, double x2, int nc, int o,
               int v, hipStream_t s) {
    if (g_dry || o <= 0 || v <= 0 || nc <= 0) return;
    const int nt = (v + TS - 1) / TS;
    const long long rows = (long long)nc * o;
    hipLaunchKernelGGL(uz_form_kernel, dim3((unsigned)(nt * (nt + 1) / 2), (unsigned)std::min<long long>(rows, 65535)), dim3(256),
                       0, s, Uz, F, C1, C2, ldc, x2, nc, o, v);
    LAUNCHCHK();
}

}  // namespace adc3
