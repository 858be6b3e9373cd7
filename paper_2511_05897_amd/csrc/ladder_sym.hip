// C = Z G for the two symmetric pair blocks of the stored ladder and few rows (M <= 20), reading half of each G.
//
// With few rows the product is bound by the stream of G (8 n^2 bytes; 2 M n^2 flops), so each element above the diagonal
// is read once and serves both its row and its column: column block J (256 columns) streams the rows above it and its
// diagonal block in slabs of 16 rows, k-major Z and the slab giving
//   C[m][n] += sum_k Z[m][k] G[k][n]        n in J, accumulated in registers over the slabs     (product 1)
//   C[m][k] += sum_n Z[m][n] G[k][n]        k the slab's rows, complete for this J at once      (product 2, not for the
//                                           diagonal block)
// both on the matrix cores (16 rows and a 4-row strip, as ladder_f64t_kernel).  The slabs of all J form one list,
// dealt to 256 workgroups per pair block in equal runs (two workgroups a CU over both blocks), so the triangle is balanced
// whatever its shape; slabs go straight into LDS one ahead.  Product 1 leaves a partial sum per workgroup and J, product 2
// one per J and k; a second launch adds them in a fixed order.  o=20 v=200, 20 rows, both blocks:
// 761 us (4.2 TB/s over half of both G) and 62 for the sums, where the row-major kernel streamed all of G in 1180 and 14.
// What bounds it is the slab in flight behind the current one, two workgroups a CU.
#include "internal.h"
#include <algorithm>

namespace adc3 {

namespace {
typedef double d2y __attribute__((ext_vector_type(2)));
typedef double d4y __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* sy_lds_t;

constexpr int SB = 256, SS = 16, SLD = SB + 2;  // column block, slab rows, LDS row stride (doubles)
constexpr int SWG = 256;                        // workgroups per pair block
constexpr unsigned SY_OOR = 0xFFFFFFF0u;

struct SymArgs {
    const double* Z;  // [n][ldz]
    const double* G;  // [n][ldg]
    double *P1, *P2;  // [slot][M][n]; J's rows k < 256 J at M 256 J (J - 1) / 2, as [M][256 J]
    double* C;        // [M][n]
    long long ldz, ldg;
    int n, per;       // order, slabs per workgroup
};
struct SymPair {
    SymArgs b[2];
    int M;
};

__host__ __device__ inline int sym_start(int J) { return 8 * J * (J + 1); }  // J's first slab in the list
__host__ __device__ inline int sym_slabs(int n, int J) {                     // J's slabs
    const int rows = n < (J + 1) * SB ? n : (J + 1) * SB;
    return (rows + SS - 1) / SS;
}

template <int EX>
__global__ __launch_bounds__(256, 2) void ladder_sym_kernel(SymPair p) {
    constexpr int R = 16 + 4 * EX;
    const SymArgs& g = p.b[blockIdx.y];
    const int M = p.M, n = g.n;
    __shared__ __attribute__((aligned(16))) double G0[SS * SLD], G1[SS * SLD];
    __shared__ __attribute__((aligned(16))) double Z0[SS * R], Z1[SS * R];
    __shared__ double Ps[4][R * 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int nblk = (n + SB - 1) / SB, total = sym_start(nblk - 1) + sym_slabs(n, nblk - 1);
    const int s0 = blockIdx.x * g.per, s1 = min(total, s0 + g.per);
    int J = 0;
    while (J + 1 < nblk && sym_start(J + 1) <= s0) ++J;
    for (int s = s0; s < s1; ++J) {
        const int first = sym_start(J), ka = (s - first) * SS, kb = min(first + sym_slabs(n, J), s1);
        const int kend = (kb - first) * SS;  // this workgroup's rows of J: ka .. kend (the last slab may pass n)
        s = kb;
        const int n0 = J * SB, cw = 64 * wave;
        // product 2's rows of Z over the wave's 64 columns: step 2 t + j contracts columns 8 t + 2 lk + j
        double f[16], fx[EX > 0 ? EX : 1][16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int c = n0 + cw + 8 * (t >> 1) + 2 * lk + (t & 1);
            f[t] = (c < n && lr < M) ? g.Z[c * g.ldz + lr] : 0.0;
#pragma unroll
            for (int e = 0; e < EX; ++e) {
                const int m = 16 + 4 * e + (lr & 3);
                fx[e][t] = (c < n && m < M) ? g.Z[c * g.ldz + m] : 0.0;
            }
        }
        d4y acc[2][2];
        double ax[EX > 0 ? EX : 1][2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[h][j] = d4y{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < EX; ++e) ax[e][h][j] = 0.0;
            }
        auto issue = [&](double(&Gb)[SS * SLD], double(&Zb)[SS * R], int k0) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(g.G + (long long)k0 * g.ldg + n0), (short)0, 0x7fffffff, 0x00020000);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int row = 4 * wave + r, col = 128 * h + 2 * lane;
                    const unsigned off =
                        (k0 + row < n && n0 + col < n) ? (unsigned)(row * (int)g.ldg + col) * 8u : SY_OOR;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (sy_lds_t)&Gb[row * SLD + 128 * h], 16, off, 0, 0, 0);
                }
            // the slab's rows of Z are contiguous: 16 ldz doubles, two a lane
            const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(g.Z + k0 * g.ldz), (short)0, (int)(min(SS, n - k0) * g.ldz * 8), 0x00020000);
            if (64 * wave < 8 * (int)g.ldz) {
                const unsigned l = tid;
                if (l < 8 * (unsigned)g.ldz)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rz, (sy_lds_t)&Zb[128 * wave], 16, 16 * l, 0, 0, 0);
            }
        };
        // product 2's results of a slab, stored after the next slab's loads are issued
        double o0 = 0.0, o1 = 0.0;
        int ok = n0;
        double* P2 = g.P2 + (long long)M * SB * J * (J - 1) / 2;
        auto flush = [&] {
            if (ok + lr >= n0) return;
            const int m = tid >> 4;
            if (m < M) P2[(long long)m * n0 + ok + lr] = o0;
            if (EX > 0 && tid < 64 * EX && 16 + m < M) P2[(long long)(16 + m) * n0 + ok + lr] = o1;
        };
        auto step = [&](const double(&Gb)[SS * SLD], const double(&Zb)[SS * R], int k0) {
            const bool two = k0 < n0;  // uniform; blocks above the diagonal one
            if (two) {
                d4y d0 = d4y{0.0, 0.0, 0.0, 0.0}, d1 = d0;
                double x0[EX > 0 ? EX : 1], x1[EX > 0 ? EX : 1];
#pragma unroll
                for (int e = 0; e < EX; ++e) x0[e] = x1[e] = 0.0;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const d2y b = *(const d2y*)&Gb[lr * SLD + cw + 8 * t + 2 * lk];
                    d0 = __builtin_amdgcn_mfma_f64_16x16x4f64(f[2 * t], b.x, d0, 0, 0, 0);
                    d1 = __builtin_amdgcn_mfma_f64_16x16x4f64(f[2 * t + 1], b.y, d1, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < EX; ++e) {
                        x0[e] = __builtin_amdgcn_mfma_f64_4x4x4f64(fx[e][2 * t], b.x, x0[e], 0, 0, 0);
                        x1[e] = __builtin_amdgcn_mfma_f64_4x4x4f64(fx[e][2 * t + 1], b.y, x1[e], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) Ps[wave][(lk + 4 * r) * 16 + lr] = d0[r] + d1[r];
#pragma unroll
                for (int e = 0; e < EX; ++e) Ps[wave][(16 + 4 * e + lk) * 16 + lr] = x0[e] + x1[e];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 4 * j + lk;  // lane (m = lr, k); rows past M are never written
                const double z = Zb[k * (int)g.ldz + lr];
                double zs[EX > 0 ? EX : 1];
#pragma unroll
                for (int e = 0; e < EX; ++e) zs[e] = Zb[k * (int)g.ldz + 16 + 4 * e + (lr & 3)];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const d2y b = *(const d2y*)&Gb[k * SLD + cw + 32 * h + 2 * lr];
                    acc[h][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(z, b.x, acc[h][0], 0, 0, 0);
                    acc[h][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(z, b.y, acc[h][1], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < EX; ++e) {
                        ax[e][h][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(zs[e], b.x, ax[e][h][0], 0, 0, 0);
                        ax[e][h][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(zs[e], b.y, ax[e][h][1], 0, 0, 0);
                    }
                }
            }
            ok = n0;
            if (two) {
                // the barrier without the wait on the copies in flight that __syncthreads() would add
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                ok = k0;
                o0 = ((Ps[0][tid] + Ps[1][tid]) + Ps[2][tid]) + Ps[3][tid];
                if (EX > 0 && tid < 64 * EX) {
                    const int i = 256 + tid;
                    o1 = ((Ps[0][i] + Ps[1][i]) + Ps[2][i]) + Ps[3][i];
                }
            }
        };
        auto sync = [] {
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        };
        issue(G0, Z0, ka);
        sync();
        int k0 = ka;
        for (; k0 + SS < kend; k0 += 2 * SS) {
            issue(G1, Z1, k0 + SS);
            flush();
            step(G0, Z0, k0);
            sync();
            if (k0 + 2 * SS < kend) issue(G0, Z0, k0 + 2 * SS);
            flush();
            step(G1, Z1, k0 + SS);
            sync();
        }
        flush();
        if (k0 < kend) {
            step(G0, Z0, k0);
            flush();
            sync();
        }
        double* P1 = g.P1 + (long long)(blockIdx.x - first / g.per) * M * n;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int c = n0 + cw + 32 * h + 2 * lr + j;
                if (c >= n) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (lk + 4 * r < M) P1[(long long)(lk + 4 * r) * n + c] = acc[h][j][r];
#pragma unroll
                for (int e = 0; e < EX; ++e)
                    if (16 + 4 * e + lk < M) P1[(long long)(16 + 4 * e + lk) * n + c] = ax[e][h][j];
            }
    }
}

// C[m][n] = the partial sums of n's block from product 1, then of the blocks to its right from product 2
__global__ __launch_bounds__(256) void ladder_sym_sum_kernel(SymPair p) {
    const SymArgs& g = p.b[blockIdx.z];
    const int M = p.M, n = g.n, c = blockIdx.x * 256 + threadIdx.x, m = blockIdx.y, b = blockIdx.x;
    if (c >= n) return;
    const int nblk = (n + SB - 1) / SB, first = sym_start(b), w0 = first / g.per;
    const int slots = (first + sym_slabs(n, b) - 1) / g.per - w0 + 1;
    double acc = 0.0;
#pragma unroll 4
    for (int k = 0; k < slots; ++k) acc += g.P1[((long long)k * M + m) * n + c];
#pragma unroll 8
    for (int J = b + 1; J < nblk; ++J)
        acc += g.P2[(long long)M * SB * J * (J - 1) / 2 + (long long)m * SB * J + c];
    g.C[(long long)m * n + c] = acc;
}

int sym_per(int n) {
    const int nblk = (n + SB - 1) / SB, total = sym_start(nblk - 1) + sym_slabs(n, nblk - 1);
    return (total + SWG - 1) / SWG;
}
long long sym_elems(int M, int n, long long& p1) {
    const long long nblk = (n + SB - 1) / SB;
    // most runs that meet in one column block: the last one's slabs, and one at each end
    p1 = ((sym_slabs(n, (int)nblk - 1) + sym_per(n) - 1) / sym_per(n) + 1) * (long long)M * n;
    return p1 + M * SB * nblk * (nblk - 1) / 2;
}
}  // namespace

bool ladder_sym_fits(int M, long long np, long long nm, long long partial) {
    if (M < 1 || M > 20 || np < SB || nm < SB || np > (1 << 20)) return false;
    long long a, b;
    return sym_elems(M, (int)np, a) + sym_elems(M, (int)nm, b) <= partial;
}

void ladder_sym(int M, const double* Zp, const double* Zm, long long ldz, const double* Gp, int np, const double* Gm, int nm,
                double* Cp, double* Cm, double* partial, hipStream_t s) {
    if (g_dry) return;
    SymPair a;
    a.M = M;
    for (int i = 0; i < 2; ++i) {
        SymArgs& g = a.b[i];
        g.n = i ? nm : np;
        g.Z = i ? Zm : Zp;
        g.G = i ? Gm : Gp;
        g.C = i ? Cm : Cp;
        g.ldz = ldz;
        g.ldg = g.n;
        g.per = sym_per(g.n);
        long long p1;
        const long long all = sym_elems(M, g.n, p1);
        g.P1 = partial;
        g.P2 = partial + p1;
        partial += all;
    }
    const dim3 grid(SWG, 2), wg(256);
    if (M <= 16) hipLaunchKernelGGL(ladder_sym_kernel<0>, grid, wg, 0, s, a);
    else hipLaunchKernelGGL(ladder_sym_kernel<1>, grid, wg, 0, s, a);
    hipLaunchKernelGGL(ladder_sym_sum_kernel, dim3((unsigned)((np + 255) / 256), M, 2), wg, 0, s, a);
    LAUNCHCHK();
}

}  // namespace adc3
