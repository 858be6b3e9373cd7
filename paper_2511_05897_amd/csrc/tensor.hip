// Two-operand tensor contraction expressed as one GEMM on the matrix cores.
//
//   out[...] = alpha * sum_K A[...] B[...] + beta * out[...]
//
// Labels are single letters; an operand has at most 4 axes.  Labels shared by A
// and B and absent from the output are contracted (K); labels of A in the output
// form the GEMM rows (M), labels of B in the output the columns (N).  An operand
// whose axes are already ordered [M..,K..] / [K..,M..] (resp. [K..,N..] /
// [N..,K..]) is used in place through strides; otherwise it is permuted once into
// a workspace buffer.  The output is written through strides when its axes read
// [M..,N..] or [N..,M..], else through a permuted temporary.
#include "internal.h"
#include "tensor.h"
#include <algorithm>
#include <cmath>
#include <cstring>

namespace adc3 {

thread_local bool g_dry = false;

namespace {
struct Parsed {
    std::string a, b, o;
};
Parsed parse(const char* spec) {
    Parsed p;
    const char* comma = std::strchr(spec, ',');
    const char* arrow = std::strstr(spec, "->");
    if (!comma || !arrow) fail(-1, std::string("ein2: bad spec ") + spec);
    p.a.assign(spec, comma);
    p.b.assign(comma + 1, arrow);
    p.o.assign(arrow + 2);
    return p;
}
long long prod_dims(const std::string& labels, const std::string& from, const int* dims) {
    long long n = 1;
    for (char c : labels) n *= dims[from.find(c)];
    return n;
}
// permutation that reorders `from` into `to` (to[k] = from[perm[k]])
void perm_of(const std::string& from, const std::string& to, int* perm) {
    for (size_t k = 0; k < to.size(); ++k) perm[k] = (int)from.find(to[k]);
}
// pad to 4D with leading unit axes
void permute_any(double* out, const double* in, const std::string& from, const int* dims, const std::string& to,
                 double alpha, double beta, hipStream_t s) {
    int d4[4] = {1, 1, 1, 1}, p4[4] = {0, 1, 2, 3};
    int nd = (int)from.size();
    int off = 4 - nd;
    for (int k = 0; k < nd; ++k) d4[off + k] = dims[k];
    int perm[4];
    perm_of(from, to, perm);
    for (int k = 0; k < nd; ++k) p4[off + k] = off + perm[k];
    for (int k = 0; k < off; ++k) p4[k] = k;
    k_permute4(out, in, d4, p4, alpha, beta, s);
}
}  // namespace

// The tile and K split of a k-major product: the least modelled time over row tiles of 16 tm rows and K chunks.
// A workgroup's slab of 16 k keeps each of a CU's four matrix cores busy for 512 cycles per 16 rows; a CU with one workgroup
// also waits for the slab's loads (about 700 cycles), with two that mostly overlaps (400); B streams from HBM once per
// row tile; a split adds a pass over the partial sums and a launch.  (The sigma ladder at o=13 v=91, 65 rows, on this
// choice: 101 us for both pair blocks; measured choices for one block at a time, used for both: 162.)
void km_shape(long long M, long long N, long long K, long long partial, int kcmax, int& tm, int& mt, int& kc) {
    const long long ntn = (N + 127) / 128, nb = (M + 15) / 16;
    double best = 1e300;
    for (int t = (int)std::min<long long>(8, nb); t >= 1; --t) {
        const long long m = (nb + t - 1) / t;
        if (m > 65535) continue;
        const double blocks = ladder_t_rows(M, m) / 16.0;
        for (int c = 1; c <= 32; ++c) {
            const long long k = ((K + c - 1) / c + 15) / 16 * 16, n = (K + k - 1) / k;
            if (k > kcmax || (n > 1 && n * M * N > partial) || (c > 1 && k < 64)) continue;
            const double w = (double)m * ntn * n, slabs = (double)k / 16;
            double cost = std::ceil(w / 256.0) * slabs * (512.0 * blocks + (w <= 256 ? 700.0 : 400.0)) + 3000.0;
            cost = std::max(cost, 8.0 * (double)m * N * K / 5.2e12 * 2.2e9);  // B streamed once per row tile
            if (n > 1) cost += 7000.0 + 2.2e9 * (8.0 * (n + 1) * M * N) / 3.5e12;
            if (cost < best) { best = cost; tm = t; mt = (int)m; kc = (int)k; }
        }
    }
}

void gemm_km(Arena& ws, long long M, long long N, long long K, double alpha, const double* A, long long lda,
             const double* B, long long ldb, double beta, double* C, long long ldc, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    const size_t mark = ws.mark();
    // 16-byte rows (offsets relative to the workspace, so that the counting dry runs decide alike)
    const uintptr_t base = ws.base ? (uintptr_t)ws.base : ARENA_COUNT_BASE;
    auto even = [&](const double* X, long long& ld, long long cols) {
        if (ld % 2 == 0 && (((uintptr_t)X - base) & 15) == 0) return X;
        const long long n = cols + (cols & 1);
        double* t = ws.take<double>((size_t)std::max<long long>(K * n, 1));
        k_copy2d(t, n, X, ld, K, cols, 1.0, 0.0, s);
        ld = n;
        return (const double*)t;
    };
    const bool tile = 2.0 * (double)M * (double)N * (double)K >= 4e6 && M >= 16 && N >= 32 && K >= 16;
    if (tile) {
        A = even(A, lda, M);
        B = even(B, ldb, N);
        if (!g_dry && ladder_t_supported((int)M, (int)N, (int)K, A, lda, B, ldb) && ladder_t_min_chunks((int)K, lda, ldb) == 1) {
            int tm = 0, mt = 0, kc = 0;
            km_shape(M, N, K, g_gemm_scratch ? g_gemm_scratch_n : 0, (int)((K + 15) / 16 * 16), tm, mt, kc);
            if (tm > 0) {
                ladder_gemm_t_shape((int)M, (int)N, (int)K, alpha, A, lda, B, ldb, beta, C, ldc, tm, mt, kc, g_gemm_scratch, s);
                ws.release(mark);
                return;
            }
        }
    }
    Gemm g;
    g.M = (int)M; g.N = (int)N; g.K = (int)K;
    g.A = A; g.sAm = 1; g.sAk = lda;
    g.B = B; g.sBk = ldb; g.sBn = 1;
    g.C = C; g.sCm = ldc; g.sCn = 1;
    g.alpha = alpha; g.beta = beta;
    gemm(g, s);
    ws.release(mark);
}

void ein2(Arena& ws, const char* spec, double alpha, const double* A, const int* adims, const double* B,
          const int* bdims, double beta, double* C, hipStream_t s) {
    Parsed p = parse(spec);
    std::string Ml, Nl, Kl;
    for (char c : p.o) {
        bool ina = p.a.find(c) != std::string::npos, inb = p.b.find(c) != std::string::npos;
        if (ina && inb) fail(-1, std::string("ein2: batch label unsupported in ") + spec);
        if (ina) Ml += c;
        else if (inb) Nl += c;
        else fail(-1, std::string("ein2: output label not in inputs: ") + spec);
    }
    for (char c : p.a)
        if (p.b.find(c) != std::string::npos && p.o.find(c) == std::string::npos) Kl += c;
    for (char c : p.b)
        if (p.o.find(c) == std::string::npos && p.a.find(c) == std::string::npos)
            fail(-1, std::string("ein2: dangling label in ") + spec);
    for (char c : p.a)
        if (p.o.find(c) == std::string::npos && p.b.find(c) == std::string::npos)
            fail(-1, std::string("ein2: dangling label in ") + spec);
    // output dims
    int odims[4];
    for (size_t k = 0; k < p.o.size(); ++k) {
        char c = p.o[k];
        size_t ia = p.a.find(c);
        odims[k] = (ia != std::string::npos) ? adims[ia] : bdims[p.b.find(c)];
    }
    const long long M = prod_dims(Ml, p.a, adims), N = prod_dims(Nl, p.b, bdims), K = prod_dims(Kl, p.a, adims);
    size_t mark = ws.mark();
    Gemm g;
    g.M = (int)M; g.N = (int)N; g.K = (int)K;
    g.alpha = alpha;
    if (M > 2147483647LL || N > 2147483647LL || K > 2147483647LL) fail(-1, "ein2: dimension too large");
    // A contraction of some size runs on the k-major tiles (gemm_km): both operands as [K..][M..], [K..][N..], in
    // place or permuted once (cheap next to the GEMM), row-major output; where the output reads [N..][M..] the
    // operands change places.  Measured at o=9 v=83: the 64 x 64 tile with operands through registers takes 51 us
    // for 747^3 (144 workgroups, a load's latency per 16-deep slab), this path 17-25 us.
    const bool kmajor = 2.0 * (double)M * (double)N * (double)K >= 5e7 && M >= 32 && N >= 32 && K >= 16;
    if (kmajor) {
        const bool swap = p.o == Nl + Ml;
        const double *X = swap ? B : A, *Y = swap ? A : B;
        const std::string &xl = swap ? p.b : p.a, &yl = swap ? p.a : p.b, &rl = swap ? Nl : Ml, &cl = swap ? Ml : Nl;
        const int *xd = swap ? bdims : adims, *yd = swap ? adims : bdims;
        const long long R = swap ? N : M, Cc = swap ? M : N;
        if (xl != Kl + rl) {
            double* t = ws.take<double>(K * R);
            permute_any(t, X, xl, xd, Kl + rl, 1.0, 0.0, s);
            X = t;
        }
        if (yl != Kl + cl) {
            double* t = ws.take<double>(K * Cc);
            permute_any(t, Y, yl, yd, Kl + cl, 1.0, 0.0, s);
            Y = t;
        }
        if (p.o == rl + cl) {
            gemm_km(ws, R, Cc, K, alpha, X, R, Y, Cc, beta, C, Cc, s);
        } else {
            double* t = ws.take<double>(M * N);
            gemm_km(ws, R, Cc, K, alpha, X, R, Y, Cc, 0.0, t, Cc, s);
            int tdims[4];
            const std::string tl = rl + cl;
            for (size_t k = 0; k < tl.size(); ++k) tdims[k] = odims[p.o.find(tl[k])];
            permute_any(C, t, tl, tdims, p.o, 1.0, beta, s);
        }
        ws.release(mark);
        return;
    }
    // A
    if (p.a == Ml + Kl) { g.A = A; g.sAm = K; g.sAk = 1; }
    else if (p.a == Kl + Ml) { g.A = A; g.sAm = 1; g.sAk = M; }
    else {
        double* t = ws.take<double>(M * K);
        permute_any(t, A, p.a, adims, Ml + Kl, 1.0, 0.0, s);
        g.A = t; g.sAm = K; g.sAk = 1;
    }
    // B
    if (p.b == Kl + Nl) { g.B = B; g.sBk = N; g.sBn = 1; }
    else if (p.b == Nl + Kl) { g.B = B; g.sBk = 1; g.sBn = K; }
    else {
        double* t = ws.take<double>(K * N);
        permute_any(t, B, p.b, bdims, Kl + Nl, 1.0, 0.0, s);
        g.B = t; g.sBk = N; g.sBn = 1;
    }
    // C
    if (p.o == Ml + Nl) { g.C = C; g.sCm = N; g.sCn = 1; g.beta = beta; gemm(g, s); }
    else if (p.o == Nl + Ml) { g.C = C; g.sCm = 1; g.sCn = M; g.beta = beta; gemm(g, s); }
    else {
        double* t = ws.take<double>(M * N);
        g.C = t; g.sCm = N; g.sCn = 1; g.beta = 0.0;
        gemm(g, s);
        int tdims[4];
        std::string tl = Ml + Nl;
        for (size_t k = 0; k < tl.size(); ++k) tdims[k] = odims[p.o.find(tl[k])];
        permute_any(C, t, tl, tdims, p.o, 1.0, beta, s);
    }
    ws.release(mark);
}

}  // namespace adc3
