// The data passes around the products of a level-3 sigma pass.
//
//   k_sigma_prep: the 2p1h part z of nv vectors -> the ladder's packed rows w+- (ladder_sa.hip) and the operands of the
//     particle-hole products, k-major for the tiles that copy both operands into LDS:
//       Y2t[(j,d)][(n,a)] = x[n][j][a][d],  Y3t = x[n][j][d][a],  Y1t = 2 x[n][j][a][d] - x[n][j][d][a]
//     (x = z_S + z_A/sqrt3 per block; Y2t and Y3t side by side in rows of 2 nv v)
//   k_sigma_fin: sigma_z += x1 (ladder + S(d) + sqrt3 A(d)), d[n][i][a][b] = -E2[(n,a)][(i,b)] - E3[(n,b)][(i,a)],
//     with the K-chunk partial sums of the ladder's and the particle-hole product summed on the way in, in order.
//
// Both are streams.  They replace thirteen launches of a pass (copies, pack, transposes, operand build, split-K
// reductions, unpack, final sums); a small sigma is bound by its launches (a kernel in a dependent chain takes at least
// 4.7 us), a large one saves the round trips of the intermediate forms.  Whole sigma without and with
// them: o=4 v=20 3 vectors 93 -> 46 us, o=13 v=91 5 vectors 396 -> 267, o=20 v=200 5 vectors 4.57 -> 4.39 ms (43 us, 251 us
// and 4.1 ms since the ladder's tiles take 4-row strips).
#include "internal.h"
#include <algorithm>

namespace adc3 {

namespace {
__device__ inline long long pidx(int a, int b, int v) {  // a <= b
    return (long long)a * v - (long long)a * (a - 1) / 2 + (b - a);
}
__device__ inline long long qidx(int a, int b, int v) {  // a < b
    return (long long)a * (v - 1) - (long long)a * (a - 1) / 2 + (b - a - 1);
}

// A workgroup takes the tile pair (tc <= td) of 16 x 16 elements for 16 rows m = (n, j): 128-byte runs on every side
// (along d and c of z, along c and d of the operands' columns, along m of the k-major packed rows).  16 waves a workgroup:
// a small sigma has few tile pairs and waits for each (one vector of o=16 v=120, 37 workgroups: 26 us with four waves,
// 9.3 with 16; five of o=20 v=200: 42 and 35).
constexpr int PT = 16, PR = 17, PM = PT * PR + 1;  // tile, LDS row stride, stride between rows m

struct SigmaPrep {
    const double* z; long long ldz;  // vector n's z at z + n ldz
    int nv, o, v;
    double *Ws, *Wa;                 // packed rows: k-major [pair][ldt] (ldt > 0) or row-major [m][lp], [m][lm]; or null
    long long ldt, lp, lm;
    double *Y1, *Y23;                // [(j,d)][ldy1], [(j,d)][ldy]
    long long ldy1, ldy;
    double* Y0; int nrow0;           // nrow0 rows of ldy before Y23: the second half (columns nv v ..) is zeroed
};

__global__ __launch_bounds__(1024) void sigma_prep_kernel(SigmaPrep g) {
    __shared__ double A[PT * PM], B[PT * PM];
    const int v = g.v, o = g.o, M = g.nv * o, vv = v * v;
    const int nt = (v + PT - 1) / PT, npr = nt * (nt + 1) / 2;
    const int tx = threadIdx.x & 15, ty = (threadIdx.x >> 4) & 15, tz = threadIdx.x >> 8;  // tz: four rows m at a time
    const int m0 = blockIdx.y * PT, mn = min(PT, M - m0), half = g.nv * v;
    // the zero half of the rows before Y23, dealt to the whole grid
    for (int r = blockIdx.y * gridDim.x + blockIdx.x; r < g.nrow0; r += gridDim.x * gridDim.y)
        for (int c = threadIdx.x; c < half; c += 1024) g.Y0[r * g.ldy + half + c] = 0.0;
    if ((int)blockIdx.x == npr) {
        // padding of the packed rows (pairs np .. lp, nm .. lm)
        const long long np = (long long)v * (v + 1) / 2, nm = (long long)v * (v - 1) / 2;
        if (g.Ws) {
            for (int t = threadIdx.x; t < 8 * mn; t += 1024) {
                const int k = t & 7, m = m0 + (t >> 3);
                if (np + k < g.lp) g.Ws[g.ldt ? (np + k) * g.ldt + m : m * g.lp + np + k] = 0.0;
                if (nm + k < g.lm) g.Wa[g.ldt ? (nm + k) * g.ldt + m : m * g.lm + nm + k] = 0.0;
            }
        }
        return;
    }
    int tc = 0, p = blockIdx.x;
    while (p >= nt - tc) { p -= nt - tc; ++tc; }
    const int td = tc + p, c0 = tc * PT, d0 = td * PT;
    {
        const int c = c0 + ty, d = d0 + tx, c2 = c0 + tx, d2 = d0 + ty;
        const bool in = c < v && d < v, im = c2 < v && d2 < v;
        double ra[4], rb[4];  // every load issued before the first is waited for
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int mm = min(m0 + 4 * tz + m, M - 1), n = mm / o, j = mm - n * o;
            const double* zb = g.z + n * g.ldz + (long long)j * vv;
            ra[m] = in ? zb[c * v + d] : 0.0;    // z[c][d]
            rb[m] = im ? zb[d2 * v + c2] : 0.0;  // z[d][c]
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            A[(4 * tz + m) * PM + ty * PR + tx] = ra[m];
            B[(4 * tz + m) * PM + ty * PR + tx] = rb[m];
        }
    }
    __syncthreads();
    if (g.Ws) {
        if (g.ldt) {
            for (int e = threadIdx.x >> 4; e < PT * PT; e += 64) {  // lanes along m
                const int ci = e >> 4, di = e & 15, c = c0 + ci, d = d0 + di;
                if (c > d || d >= v || tx >= mn) continue;
                const double x = A[tx * PM + ci * PR + di], y = B[tx * PM + di * PR + ci];
                const long long m = m0 + tx;
                if (c == d) {
                    g.Ws[pidx(c, c, v) * g.ldt + m] = x;
                } else {
                    g.Ws[pidx(c, d, v) * g.ldt + m] = x + y;
                    g.Wa[qidx(c, d, v) * g.ldt + m] = x - y;
                }
            }
        } else {
            const int c = c0 + ty, d = d0 + tx;  // lanes along d
            if (c <= d && d < v)
                for (int m = tz; m < mn; m += 4) {
                    const double x = A[m * PM + ty * PR + tx], y = B[m * PM + tx * PR + ty];
                    if (c == d) {
                        g.Ws[(m0 + m) * g.lp + pidx(c, c, v)] = x;
                    } else {
                        g.Ws[(m0 + m) * g.lp + pidx(c, d, v)] = x + y;
                        g.Wa[(m0 + m) * g.lm + qidx(c, d, v)] = x - y;
                    }
                }
        }
    }
    const double is3 = 0.57735026918962576451;  // 1/sqrt(3)
    for (int m = tz; m < mn; m += 4) {
        const int n = (m0 + m) / o, j = (m0 + m) - n * o;
        {  // rows (j, d = d0 + ty), columns (n, c = c0 + tx)
            const int c = c0 + tx, d = d0 + ty;
            if (c < v && d < v) {
                const double x = A[m * PM + tx * PR + ty], y = B[m * PM + ty * PR + tx];  // z[c][d], z[d][c]
                const double sy = 0.5 * (x + y), an = 0.5 * (x - y) * is3;
                const long long row = (long long)j * v + d, col = (long long)n * v + c;
                g.Y23[row * g.ldy + col] = sy + an;
                g.Y23[row * g.ldy + half + col] = sy - an;
                g.Y1[row * g.ldy1 + col] = 2.0 * (sy + an) - (sy - an);
            }
        }
        if (tc != td) {  // rows (j, c = c0 + ty), columns (n, d = d0 + tx)
            const int c = c0 + ty, d = d0 + tx;
            if (c < v && d < v) {
                const double x = A[m * PM + ty * PR + tx], y = B[m * PM + tx * PR + ty];
                const double sy = 0.5 * (x + y), an = 0.5 * (x - y) * is3;
                const long long row = (long long)j * v + c, col = (long long)n * v + d;
                g.Y23[row * g.ldy + col] = sy - an;
                g.Y23[row * g.ldy + half + col] = sy + an;
                g.Y1[row * g.ldy1 + col] = 2.0 * (sy - an) - (sy + an);
            }
        }
    }
}

struct SigmaFin {
    double* out; long long ldo;               // vector n's sigma_z at out + n ldo
    const double *Cs, *Ca;                    // ladder in pair blocks: partial sums [nl][M][lp], [nl][M][lm]
    int nl; long long lp, lm;
    const double* L;                          // or (Cs null) as [M][v][v]
    const double* E; int ne; long long echunk;  // particle-hole products [ne chunks][2 nv v][o v]
    int nv, o, v;
    double x1;
};

// A workgroup takes the tile pair (ta <= tb) of 32 x 32 elements of one row m: a thread one element and its mirror.  The
// chunks of an element are summed in turn; the loads in flight come from the 16 waves of a workgroup, two per CU (with
// four waves and four elements a thread: 46 against 25 us at o=13 v=91, 105 against 72 us at o=20 v=200, 5 vectors; the
// second moves 0.2 GB).
__global__ __launch_bounds__(1024) void sigma_fin_kernel(SigmaFin g) {
    constexpr int T = 32;
    __shared__ double e2[T][T + 1], f2[T][T + 1], l2[T][T + 1];
    const double s3 = 1.73205080756887729353;
    const int v = g.v, o = g.o, nt = (v + T - 1) / T;
    const long long M = (long long)g.nv * o, ov = (long long)o * v, Mph = (long long)g.nv * v;
    int ta = 0, p = blockIdx.x;
    while (p >= nt - ta) { p -= nt - ta; ++ta; }
    const int tb = ta + p, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int a = ta * T + ty, b = tb * T + tx, aa = ta * T + tx, bb = tb * T + ty;  // (a,b) and, transposed, (bb,aa)
    const bool in = a < v && b < v, im = bb < v && aa < v;
    for (long long m = blockIdx.y; m < M; m += gridDim.y) {
        const long long n = m / o, i = m - n * o;
        const double* E2 = g.E + (n * v) * ov + i * v;          // [a][b], rows of ov
        const double* E3 = g.E + (Mph + n * v) * ov + i * v;
        double* out = g.out + n * g.ldo + i * v * v;
        const double o1 = in ? out[a * v + b] : 0.0, o2 = im && ta != tb ? out[bb * v + aa] : 0.0;
        double e1 = 0.0, f1 = 0.0, e2r = 0.0, f2r = 0.0, l1 = 0.0, l2r = 0.0;
        for (int c = 0; c < g.ne; ++c) {
            const long long oc = c * g.echunk;
            if (in) { e1 += E2[oc + a * ov + b]; f1 += E3[oc + a * ov + b]; }
            if (im) { e2r += E2[oc + bb * ov + aa]; f2r += E3[oc + bb * ov + aa]; }
        }
        if (g.Cs) {
            double sp = 0.0, sm = 0.0;
            if (a <= b && b < v) {
                const double *cs = g.Cs + m * g.lp + pidx(a, b, v), *ca = g.Ca + m * g.lm + qidx(a, b, v);
                for (int c = 0; c < g.nl; ++c, cs += M * g.lp, ca += M * g.lm) {
                    sp += *cs;
                    if (a < b) sm += *ca;
                }
            }
            l1 = sp + sm;
            l2r = sp - sm;  // the ladder's (b, a)
        } else {
            const double* L = g.L + m * v * v;
            if (in) l1 = L[a * v + b];
            if (im) l2r = L[bb * v + aa];
        }
        __syncthreads();
        e2[ty][tx] = e2r;
        f2[ty][tx] = f2r;
        if (!g.Cs) l2[ty][tx] = l2r;
        __syncthreads();
        const double dab = -e1 - f2[tx][ty], dba = -e2[tx][ty] - f1;
        const double sy = 0.5 * (dab + dba), an = s3 * 0.5 * (dab - dba);
        const double oab = l1 + sy + an, oba = (g.Cs ? l2r : l2[tx][ty]) + sy - an;
        __syncthreads();
        if (ta != tb || ty <= tx) e2[tx][ty] = oba;  // the mirrored value, at [b][a]; a diagonal tile holds both triangles
        __syncthreads();
        if (ta == tb) {
            if (in) out[a * v + b] = o1 + g.x1 * (ty <= tx ? oab : e2[ty][tx]);
        } else {
            if (in) out[a * v + b] = o1 + g.x1 * oab;
            if (im) out[bb * v + aa] = o2 + g.x1 * e2[ty][tx];
        }
    }
}
}  // namespace

void k_sigma_prep(const double* z, long long ldz, int nv, int o, int v, double* Ws, double* Wa, long long ldt, double* Y1,
                  long long ldy1, double* Y0, int nrow0, double* Y23, long long ldy, hipStream_t s) {
    if (g_dry || nv <= 0 || o <= 0 || v <= 0) return;
    SigmaPrep g;
    g.z = z; g.ldz = ldz; g.nv = nv; g.o = o; g.v = v;
    g.Ws = Ws; g.Wa = Wa; g.ldt = ldt; g.lp = sa_lp(v); g.lm = sa_lm(v);
    g.Y1 = Y1; g.ldy1 = ldy1; g.Y23 = Y23; g.ldy = ldy; g.Y0 = Y0; g.nrow0 = nrow0;
    const int nt = (v + PT - 1) / PT;
    hipLaunchKernelGGL(sigma_prep_kernel, dim3((unsigned)(nt * (nt + 1) / 2 + 1), (unsigned)((nv * o + PT - 1) / PT)), dim3(1024),
                       0, s, g);
    LAUNCHCHK();
}

void k_sigma_fin(double* out, long long ldo, const double* Cs, const double* Ca, int nl, const double* L, const double* E,
                 int ne, long long echunk, int nv, int o, int v, double x1, hipStream_t s) {
    if (g_dry || nv <= 0 || o <= 0 || v <= 0) return;
    SigmaFin g;
    g.out = out; g.ldo = ldo; g.Cs = Cs; g.Ca = Ca; g.nl = nl; g.lp = sa_lp(v); g.lm = sa_lm(v); g.L = L;
    g.E = E; g.ne = ne; g.echunk = echunk; g.nv = nv; g.o = o; g.v = v; g.x1 = x1;
    const int nt = (v + 31) / 32;
    hipLaunchKernelGGL(sigma_fin_kernel, dim3((unsigned)(nt * (nt + 1) / 2), (unsigned)std::min(nv * o, 65535)), dim3(1024), 0,
                       s, g);
    LAUNCHCHK();
}

}  // namespace adc3
