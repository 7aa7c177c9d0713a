// sign(T) e_1 for the small projected matrix of the direct two-sided Lanczos
// method (section "Short recurrences": f(H_k) of the k x k projected matrix,
// the last term of the cost proposition of the direct method, which dominates at
// small volumes if it is O(k^3)).
//
// First route: the eigenvalues alone and a rational function, O(k^2)
// (sign_by_poles below).  Second route, for small k and where the first cannot
// vouch for its result: complex Schur form T = Z S Z^H by the implicit single-shift QR
// algorithm on the (tridiagonal, hence Hessenberg) input; eigenvectors of the
// triangular S by back substitution; then
//   sign(T) e_1 = Z X sign(Lambda) X^{-1} Z^H e_1,
// where X (unit upper triangular) holds the eigenvectors of S.  Z is never
// formed: the QR sweeps record their rotations, and Z^H e_1 and Z u are two
// replays of them (O(1) per rotation instead of a length-k column update).
// The sweeps work on separate real and imaginary planes, apply the column part
// of each rotation along rows after the sweep wherever the sweep no longer reads
// it, and are built for AVX2/FMA as well as for the baseline x86-64 set.
#include "small_sign.h"
#include "sgn_internal.h"

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdlib>
#include <limits>
#include <memory>
#include <string>
#include <vector>

namespace sgn {

using zc = std::complex<double>;

namespace {

struct Mat {
    int n;
    std::vector<zc> a;  // row-major
    explicit Mat(int n_) : n(n_), a((size_t)n_ * n_, zc(0, 0)) {}
    zc &operator()(int i, int j) { return a[(size_t)i * n + j]; }
    zc operator()(int i, int j) const { return a[(size_t)i * n + j]; }
};

inline double cabs1(zc z) { return std::abs(z.real()) + std::abs(z.imag()); }

// Complex product written out: std::complex's operator* goes through a library
// routine that handles infinities and NaNs, several times slower in these loops
// (all values here are finite).
inline zc cmul(zc a, zc b)
{
    return zc(a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real());
}

// Givens (c real, s complex) with G [x; y] = [r; 0], G = [[c, s], [-conj(s), c]].
inline void givens(zc x, zc y, double &c, zc &s)
{
    const double ax = std::abs(x), ay = std::abs(y);
    if (ay == 0.0) {
        c = 1.0;
        s = 0.0;
        return;
    }
    if (ax == 0.0) {
        c = 0.0;
        s = std::conj(y) / ay;
        return;
    }
    const double nrm = std::hypot(ax, ay);
    c = ax / nrm;
    s = (x / ax) * std::conj(y) / nrm;
}

// One plane rotation of the QR sweeps: columns m, m+1 of Z are replaced by
// (c Z_m + conj(s) Z_{m+1}, -s Z_m + c Z_{m+1}), i.e. Z <- Z G with
// G = [c, -s; conj(s), c] on (m, m+1).
struct Rot {
    int m;
    double c;
    zc s;
};

// The sweep kernels are inlined into two builds of the Schur routine (below).
#define SGN_INLINE inline __attribute__((always_inline))

// A square matrix as two row-major planes (real and imaginary parts): the rotation
// loops of the QR sweeps then run on plain double arrays, which the compiler vectorises.
struct Planes {
    int n;
    std::vector<double> re, im;
    explicit Planes(const Mat &A) : n(A.n), re((size_t)A.n * A.n), im((size_t)A.n * A.n)
    {
        for (size_t q = 0; q < A.a.size(); ++q) {
            re[q] = A.a[q].real();
            im[q] = A.a[q].imag();
        }
    }
    zc get(int i, int j) const { return zc(re[(size_t)i * n + j], im[(size_t)i * n + j]); }
    void set(int i, int j, zc v)
    {
        re[(size_t)i * n + j] = v.real();
        im[(size_t)i * n + j] = v.imag();
    }
    double *rr(int i) { return re.data() + (size_t)i * n; }
    double *ri(int i) { return im.data() + (size_t)i * n; }
    void store(Mat &A) const
    {
        for (size_t q = 0; q < A.a.size(); ++q) A.a[q] = zc(re[q], im[q]);
    }
};

// Rows a, b <- G [a; b] over len entries, G = [[c, s], [-conj(s), c]].
SGN_INLINE void rotate_row_pair(double *__restrict ar, double *__restrict ai, double *__restrict br,
                            double *__restrict bi, int len, double c, double sr, double si)
{
    for (int j = 0; j < len; ++j) {
        const double xr = ar[j], xi = ai[j], yr = br[j], yi = bi[j];
        ar[j] = c * xr + sr * yr - si * yi;
        ai[j] = c * xi + sr * yi + si * yr;
        br[j] = c * yr - sr * xr - si * xi;
        bi[j] = c * yi - sr * xi + si * xr;
    }
}

// Rotations of one sweep from the right, applied along R rows at once: for q = 0..cnt-1 in order,
// (row[m], row[m+1]) <- (row[m] c + row[m+1] conj(s), row[m+1] c - row[m] s) with m = m0 + q and
// (c, s) = (gc[q], gsr[q] + i gsi[q]).  The entry moving right is carried in registers (each entry
// is read and written once); the R rows are independent chains, interleaved for the pipelines.
template <int R>
SGN_INLINE void rotate_rows_right(double *const *re, double *const *im, const double *gc, const double *gsr,
                              const double *gsi, int m0, int cnt)
{
    if (cnt <= 0) return;
    double tr[R], ti[R];
    for (int r = 0; r < R; ++r) {
        tr[r] = re[r][m0];
        ti[r] = im[r][m0];
    }
    for (int q = 0; q < cnt; ++q) {
        const double c = gc[q], sr = gsr[q], si = gsi[q];
        const int m = m0 + q;
        for (int r = 0; r < R; ++r) {
            const double yr = re[r][m + 1], yi = im[r][m + 1];
            re[r][m] = c * tr[r] + sr * yr + si * yi;
            im[r][m] = c * ti[r] + sr * yi - si * yr;
            const double nr = c * yr - sr * tr[r] + si * ti[r];
            const double ni = c * yi - sr * ti[r] - si * tr[r];
            tr[r] = nr;
            ti[r] = ni;
        }
    }
    for (int r = 0; r < R; ++r) {
        re[r][m0 + cnt] = tr[r];
        im[r][m0 + cnt] = ti[r];
    }
}

// The sweep's rotations m = max(l, i) .. ihi-1 on rows i = i0 .. i1-1 of P (row i is touched by
// rotation m only if i <= m + 2; rows i <= m are the ones left for after the sweep).
SGN_INLINE void rotate_rows_after_sweep(Planes &P, int i0, int i1, int l, int ihi, const std::vector<double> &gc,
                             const std::vector<double> &gsr, const std::vector<double> &gsi)
{
    constexpr int R = 4;
    int i = i0;
    for (; i + R <= i1; i += R) {
        // rows i..i+R-1 start at max(l, row); bring the earlier ones up to the last row's start
        const int mc = std::max(l, i + R - 1);
        for (int r = 0; r < R - 1; ++r) {
            const int m0 = std::max(l, i + r);
            double *pr[1] = {P.rr(i + r)}, *pi[1] = {P.ri(i + r)};
            rotate_rows_right<1>(pr, pi, gc.data() + (m0 - l), gsr.data() + (m0 - l), gsi.data() + (m0 - l), m0,
                                 std::min(mc, ihi) - m0);
        }
        if (mc >= ihi) continue;
        double *pr[R], *pi[R];
        for (int r = 0; r < R; ++r) {
            pr[r] = P.rr(i + r);
            pi[r] = P.ri(i + r);
        }
        rotate_rows_right<R>(pr, pi, gc.data() + (mc - l), gsr.data() + (mc - l), gsi.data() + (mc - l), mc,
                             ihi - mc);
    }
    for (; i < i1; ++i) {
        const int m0 = std::max(l, i);
        double *pr[1] = {P.rr(i)}, *pi[1] = {P.ri(i)};
        rotate_rows_right<1>(pr, pi, gc.data() + (m0 - l), gsr.data() + (m0 - l), gsi.data() + (m0 - l), m0,
                             ihi - m0);
    }
}

// Complex Schur decomposition of upper Hessenberg H (overwritten by S).  The unitary
// factor is accumulated into *Z, or, with Z null, its rotations are appended to *rots
// (Z = G_1 G_2 ... in that order).  Returns false if the iteration did not converge.
//
// Within a sweep, rotation m acts on rows m, m+1 (from the left) and on columns m, m+1
// (from the right).  Its column part is needed at once only on rows m+1 and m+2, which
// the next rotation reads; rows 0..m are touched by no later row rotation of the sweep,
// so their column rotations are applied after the sweep, along the rows (contiguous in
// the row-major storage) instead of down the columns.
SGN_INLINE bool hessenberg_schur_body(Mat &Hm, Mat *Zm, std::vector<Rot> *rots)
{
    const int n = Hm.n;
    Planes H(Hm);
    std::unique_ptr<Planes> Z(Zm ? new Planes(*Zm) : nullptr);
    const double ulp = std::numeric_limits<double>::epsilon();
    const double smallnum = std::numeric_limits<double>::min() * (n / ulp);
    int ihi = n - 1;
    int its = 0, total = 0;
    const int max_total = 60 * std::max(n, 10);
    std::vector<double> gc, gsr, gsi;
    gc.reserve(n);
    gsr.reserve(n);
    gsi.reserve(n);
    while (ihi >= 0) {
        // look for a negligible subdiagonal entry
        int l = ihi;
        for (; l > 0; --l) {
            const double tst = cabs1(H.get(l - 1, l - 1)) + cabs1(H.get(l, l));
            if (cabs1(H.get(l, l - 1)) <= std::max(ulp * tst, smallnum)) {
                H.set(l, l - 1, 0.0);
                break;
            }
        }
        if (l == ihi) {  // 1x1 block converged
            --ihi;
            its = 0;
            continue;
        }
        if (++total > max_total) return false;
        ++its;
        // shift
        zc sigma;
        if (its % 11 == 10) {  // exceptional shift
            sigma = H.get(ihi, ihi) + 0.75 * std::abs(H.get(ihi, ihi - 1).real());
        } else {
            const zc a = H.get(ihi - 1, ihi - 1), b = H.get(ihi - 1, ihi), c = H.get(ihi, ihi - 1),
                     d = H.get(ihi, ihi);
            const zc tr2 = 0.5 * (a + d);
            const zc disc = std::sqrt(0.25 * (a - d) * (a - d) + b * c);
            const zc e1 = tr2 + disc, e2 = tr2 - disc;
            sigma = (std::abs(e1 - d) <= std::abs(e2 - d)) ? e1 : e2;
        }
        // implicit single-shift QR sweep on rows/columns l..ihi
        gc.clear();
        gsr.clear();
        gsi.clear();
        for (int m = l; m < ihi; ++m) {
            zc x, y;
            if (m == l) {
                x = H.get(l, l) - sigma;
                y = H.get(l + 1, l);
            } else {
                x = H.get(m, m - 1);
                y = H.get(m + 1, m - 1);
            }
            double c;
            zc s;
            givens(x, y, c, s);
            // rows m, m+1  (all columns from the bulge column to the end: full Schur form)
            const int j0 = (m == l ? l : m - 1);
            rotate_row_pair(H.rr(m) + j0, H.ri(m) + j0, H.rr(m + 1) + j0, H.ri(m + 1) + j0, n - j0, c, s.real(),
                            s.imag());
            if (m > l) H.set(m + 1, m - 1, 0.0);
            // columns m, m+1 on rows m+1, m+2 now; rows 0..m after the sweep
            const int imax = std::min(m + 2, ihi);
            for (int i = m + 1; i <= imax; ++i) {
                const zc t1 = H.get(i, m), t2 = H.get(i, m + 1);
                H.set(i, m, t1 * c + cmul(t2, std::conj(s)));
                H.set(i, m + 1, t2 * c - cmul(t1, s));
            }
            gc.push_back(c);
            gsr.push_back(s.real());
            gsi.push_back(s.imag());
            if (rots) rots->push_back({m, c, s});
        }
        rotate_rows_after_sweep(H, 0, ihi, l, ihi, gc, gsr, gsi);
        if (Z) {
            // every row of Z takes every rotation of the sweep
            constexpr int R = 4;
            int i = 0;
            for (; i + R <= n; i += R) {
                double *pr[R], *pi[R];
                for (int r = 0; r < R; ++r) {
                    pr[r] = Z->rr(i + r);
                    pi[r] = Z->ri(i + r);
                }
                rotate_rows_right<R>(pr, pi, gc.data(), gsr.data(), gsi.data(), l, ihi - l);
            }
            for (; i < n; ++i) {
                double *pr[1] = {Z->rr(i)}, *pi[1] = {Z->ri(i)};
                rotate_rows_right<1>(pr, pi, gc.data(), gsr.data(), gsi.data(), l, ihi - l);
            }
        }
    }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < i; ++j) H.set(i, j, 0.0);
    H.store(Hm);
    if (Z) Z->store(*Zm);
    return true;
}

// The same routine built for x86-64 with AVX2 and FMA and for the baseline instruction set,
// chosen once from the host's CPU features (SGN_HOST_ISA=baseline in the environment forces
// the baseline build).
__attribute__((target("avx2,fma"))) bool hessenberg_schur_avx2(Mat &H, Mat *Z, std::vector<Rot> *rots)
{
    return hessenberg_schur_body(H, Z, rots);
}

bool hessenberg_schur_base(Mat &H, Mat *Z, std::vector<Rot> *rots) { return hessenberg_schur_body(H, Z, rots); }

bool host_avx2()
{
    static const bool avx2 = [] {
        const char *isa = std::getenv("SGN_HOST_ISA");
        if (isa && std::string(isa) == "baseline") return false;
        return __builtin_cpu_supports("avx2") && __builtin_cpu_supports("fma");
    }();
    return avx2;
}

bool hessenberg_schur(Mat &H, Mat *Z, std::vector<Rot> *rots)
{
    return host_avx2() ? hessenberg_schur_avx2(H, Z, rots) : hessenberg_schur_base(H, Z, rots);
}

}  // namespace

namespace {

// ---------------------------------------------------------------------------- rational route
// sign(T) e_1 in O(k^2): eigenvalues by the QL iteration on the complex symmetric tridiagonal similar to T, then
// the rational function g_s(cT) e_1 of Eq. (pfe_s) with the scale and the number of poles that make it the sign
// at every one of those eigenvalues far below rounding, each pole a pair of tridiagonal solves.  It is taken
// only when it can vouch for its result (see sign_by_poles); otherwise the Schur route below runs.
// k = 400 of the direct method, one core of a server: 149 ms by the Schur form, 9 ms here, and the result is
// closer to the exact one (k = 250: 2e-13 by the Schur form, 3e-16 here).

constexpr int kPolesMinSize = 24;     // below, the Schur form costs microseconds
// More poles than this (an eigenvalue near the imaginary axis): the Schur route.  A pole and its conjugate, twice,
// take 13 k ns, the Schur form k^3 ns, so the limit grows with k^2 and stays below where they meet (k = 400: 5000).
inline int poles_max(int k) { return std::max(512, (int)std::min<int64_t>((int64_t)k * k / 32, 1 << 20)); }
constexpr double kPolesTruncation = 1e-20;  // |g_s(c lambda) - sign lambda| at every eigenvalue, below this
constexpr double kPolesAgree = 1e-11;       // two evaluations with other poles agree to this, relative

// Eigenvalues of the complex symmetric tridiagonal matrix with diagonal d and off-diagonal e (e[k-1] unused):
// implicit QL with Wilkinson shifts and complex orthogonal rotations.  False if a rotation does not exist or is
// large (complex orthogonal matrices are not bounded), or an eigenvalue takes too many sweeps.
SGN_INLINE bool symmetric_ql_body(std::vector<zc> &d, std::vector<zc> &e)
{
    const int n = (int)d.size();
    const double eps = std::numeric_limits<double>::epsilon();
    auto inv = [](zc a) {
        const double q = 1.0 / std::norm(a);
        return zc(a.real() * q, -a.imag() * q);
    };
    for (int l = 0; l < n; ++l) {
        for (int iter = 0;; ++iter) {
            int m = l;
            for (; m + 1 < n; ++m)
                if (cabs1(e[m]) <= eps * (cabs1(d[m]) + cabs1(d[m + 1]))) break;
            if (m == l) break;
            if (iter >= 60) return false;
            // shift: the eigenvalue of the leading 2 x 2 block closer to d[l]
            const zc g0 = cmul(d[l + 1] - d[l], 0.5 * inv(e[l]));
            const zc r0 = std::sqrt(cmul(g0, g0) + 1.0);
            const zc t0 = std::abs(g0 + r0) >= std::abs(g0 - r0) ? g0 + r0 : g0 - r0;
            if (!(std::norm(t0) > 0.0)) return false;
            zc g = d[m] - d[l] + cmul(e[l], inv(t0));
            zc s = 1.0, c = 1.0, p = 0.0;
            for (int i = m - 1; i >= l; --i) {
                const zc f = cmul(s, e[i]), b = cmul(c, e[i]);
                // r = sqrt(f^2 + g^2), either root (written out: the library's complex square root guards against
                // over- and underflow, which would end this route anyway)
                const zc q2 = cmul(f, f) + cmul(g, g);
                const double rn = std::sqrt(std::norm(q2));  // |r|^2
                const double h = std::sqrt(0.5 * (rn + std::abs(q2.real()))), v = 0.5 * q2.imag() / h;
                const zc r = q2.real() >= 0.0 ? zc(h, v) : zc(v, h);
                if (!(rn > 1e-12 * (std::norm(f) + std::norm(g)))) return false;  // |c|, |s| up to 1e6
                const zc ri(r.real() / rn, -r.imag() / rn);
                e[i + 1] = r;
                s = cmul(f, ri);
                c = cmul(g, ri);
                const zc q = d[i + 1] - p;
                const zc w = cmul(d[i] - q, s) + 2.0 * cmul(c, b);
                p = cmul(s, w);
                d[i + 1] = q + p;
                g = cmul(c, w) - b;
            }
            d[l] -= p;
            e[l] = g;
            e[m] = 0.0;
        }
    }
    return true;
}

// y += sum_j w_j (c T - z_j)^{-1} e_1 for W shifts z_j at once (lane j of every inner loop), without pivoting:
// q_i = c d_i - z - c^2 sub_i sup_i / q_{i+1} from the last row up, x_1 = 1 / q_1, x_{i+1} = -c sub_i x_i / q_{i+1}.
// A pivot that happens to be small is followed by one as large, and the products of the two are accurate.
constexpr int kPoleLanes = 8;
SGN_INLINE void tridiagonal_poles_body(int k, const zc *diag, const zc *sub, const zc *sup, double c, const double *zi,
                                       const double *w, std::vector<double> &work, zc *y)
{
    constexpr int W = kPoleLanes;
    work.resize((size_t)2 * W * k);
    double *qr = work.data(), *qi = qr + (size_t)W * k;  // 1 / q_i
    double br[W], bi[W];
    for (int i = k - 1; i >= 0; --i) {
        double tr = 0.0, ti = 0.0;
        if (i + 1 < k) {
            const zc t = (c * c) * cmul(sub[i], sup[i]);
            tr = t.real();
            ti = t.imag();
        }
        const double dr = c * diag[i].real(), di = c * diag[i].imag();
        double *orow = qr + (size_t)W * i, *oi = qi + (size_t)W * i;
        const double *nr = i + 1 < k ? orow + W : orow, *ni = i + 1 < k ? oi + W : oi;
        for (int j = 0; j < W; ++j) {
            const double ur = i + 1 < k ? nr[j] : 0.0, ui = i + 1 < k ? ni[j] : 0.0;
            br[j] = dr - (tr * ur - ti * ui);
            bi[j] = di - zi[j] - (tr * ui + ti * ur);
        }
        for (int j = 0; j < W; ++j) {
            const double q = 1.0 / (br[j] * br[j] + bi[j] * bi[j]);
            orow[j] = br[j] * q;
            oi[j] = -bi[j] * q;
        }
    }
    double xr[W], xi[W];
    for (int j = 0; j < W; ++j) {
        xr[j] = qr[j];
        xi[j] = qi[j];
    }
    for (int i = 0; i < k; ++i) {
        double ar = 0.0, ai = 0.0;
        for (int j = 0; j < W; ++j) {
            ar += w[j] * xr[j];
            ai += w[j] * xi[j];
        }
        y[i] += zc(ar, ai);
        if (i + 1 == k) break;
        const double sr = -c * sub[i].real(), si = -c * sub[i].imag();
        const double *nr = qr + (size_t)W * (i + 1), *ni = qi + (size_t)W * (i + 1);
        for (int j = 0; j < W; ++j) {
            const double pr = sr * xr[j] - si * xi[j], pi = sr * xi[j] + si * xr[j];
            xr[j] = pr * nr[j] - pi * ni[j];
            xi[j] = pr * ni[j] + pi * nr[j];
        }
    }
}

__attribute__((target("avx2,fma"))) bool symmetric_ql_avx2(std::vector<zc> &d, std::vector<zc> &e)
{
    return symmetric_ql_body(d, e);
}
bool symmetric_ql_base(std::vector<zc> &d, std::vector<zc> &e) { return symmetric_ql_body(d, e); }
__attribute__((target("avx2,fma"))) void tridiagonal_poles_avx2(int k, const zc *diag, const zc *sub, const zc *sup,
                                                                double c, const double *zi, const double *w,
                                                                std::vector<double> &work, zc *y)
{
    tridiagonal_poles_body(k, diag, sub, sup, c, zi, w, work, y);
}
void tridiagonal_poles_base(int k, const zc *diag, const zc *sub, const zc *sup, double c, const double *zi,
                            const double *w, std::vector<double> &work, zc *y)
{
    tridiagonal_poles_body(k, diag, sub, sup, c, zi, w, work, y);
}

// y = g_s(cT) e_1: g_s(t) = sum_i omega_i / 2 [1 / (t + i tau_i) + 1 / (t - i tau_i)], tau_i = tan theta_i,
// omega_i = 1 / (s cos^2 theta_i), theta_i = pi (i - 1/2) / (2s)
void sign_poles(int k, const zc *diag, const zc *sub, const zc *sup, int s, double c, bool avx2,
                std::vector<double> &work, zc *y)
{
    std::fill(y, y + k, zc(0.0, 0.0));
    double zi[kPoleLanes], w[kPoleLanes];
    int n = 0;
    auto flush = [&]() {
        for (; n < kPoleLanes; ++n) {  // unused lanes: weight 0 at a harmless shift
            zi[n] = 1.0;
            w[n] = 0.0;
        }
        if (avx2) tridiagonal_poles_avx2(k, diag, sub, sup, c, zi, w, work, y);
        else tridiagonal_poles_base(k, diag, sub, sup, c, zi, w, work, y);
        n = 0;
    };
    for (int i = 1; i <= s; ++i) {
        const double th = M_PI * (i - 0.5) / (2.0 * s), cs = std::cos(th), tau = std::tan(th);
        for (double sg : {1.0, -1.0}) {
            zi[n] = sg * tau;
            w[n] = 0.5 / (s * cs * cs);
            if (++n == kPoleLanes) flush();
        }
    }
    if (n) flush();
}

// Returns true with sign(T) e_1 in y and the smallest |Re lambda| in *minre if
//  - the QL iteration converges and its eigenvalues reproduce trace(T) and trace(T^2),
//  - no eigenvalue is so near the imaginary axis (relative to its modulus and the spectrum's extent) that the
//    truncation kPolesTruncation takes more than poles_max poles, and
//  - a second evaluation with another scale and more poles agrees to kPolesAgree.
bool sign_by_poles(int k, const zc *diag, const zc *sub, const zc *sup, double tnorm, bool avx2, zc *y, double *minre)
{
    if (k < kPolesMinSize) return false;
    std::vector<zc> d(diag, diag + k), e(k, zc(0.0, 0.0));
    zc tr = 0.0, tr2 = 0.0;
    for (int i = 0; i < k; ++i) {
        tr += d[i];
        tr2 += cmul(d[i], d[i]);
        if (i + 1 < k) {
            const zc b = cmul(sub[i], sup[i]);
            tr2 += 2.0 * b;
            e[i] = std::sqrt(b);
        }
    }
    if (!(avx2 ? symmetric_ql_avx2(d, e) : symmetric_ql_base(d, e))) return false;
    zc s1 = 0.0, s2 = 0.0;
    double lo = std::numeric_limits<double>::infinity(), hi = 0.0, re = lo;
    for (const zc &l : d) {
        s1 += l;
        s2 += cmul(l, l);
        const double a = std::abs(l);
        lo = std::min(lo, a);
        hi = std::max(hi, a);
        re = std::min(re, std::abs(l.real()));
    }
    if (!(std::abs(s1 - tr) <= 1e-10 * k * tnorm) || !(std::abs(s2 - tr2) <= 1e-10 * k * tnorm * tnorm)) return false;
    if (!(lo > 1e-8 * tnorm) || !std::isfinite(hi)) return false;
    const int limit = poles_max(k);
    // |(1 - z)/(1 + z)| over z = c lambda in the right half plane (by the symmetry of g_s), c the mean of the circles
    auto poles = [&](double c) {
        double rho = 0.0;
        for (const zc &l : d) {
            const zc z = (l.real() > 0 ? c : -c) * l;
            rho = std::max(rho, std::norm(zc(1.0, 0.0) - z) / std::norm(zc(1.0, 0.0) + z));
        }
        if (!(rho < 1.0)) return limit + 1;
        const double need = std::log(0.5 * kPolesTruncation) / std::log(std::max(rho, 1e-6));  // rho = |.|^2: |.|^(2s)
        return need < (double)limit ? std::max(8, (int)std::ceil(need)) : limit + 1;
    };
    const double c1 = 1.0 / std::sqrt(lo * hi), c2 = 1.07 * c1;
    const int n1 = poles(c1), n2 = poles(c2) + 4;
    if (n1 > limit || n2 > limit) return false;
    std::vector<double> work;
    std::vector<zc> y1(k);
    sign_poles(k, diag, sub, sup, n1, c1, avx2, work, y1.data());
    sign_poles(k, diag, sub, sup, n2, c2, avx2, work, y);
    double num = 0.0, den = 0.0;
    for (int i = 0; i < k; ++i) {
        num += std::norm(y[i] - y1[i]);
        den += std::norm(y[i]);
    }
    if (!(den > 0.0) || !(num <= kPolesAgree * kPolesAgree * den)) return false;
    *minre = re;
    return true;
}

}  // namespace

int small_sign_e1(int k, const std::complex<double> *diag, const std::complex<double> *sub,
                  const std::complex<double> *sup, std::complex<double> *y, SmallSignInfo *info)
{
    if (k <= 0) return 1;
    Mat S(k);
    double tnorm = 0.0;
    for (int i = 0; i < k; ++i) {
        S(i, i) = diag[i];
        if (i + 1 < k) {
            S(i + 1, i) = sub[i];
            S(i, i + 1) = sup[i];
        }
    }
    for (int i = 0; i < k; ++i) {
        double row = std::abs(diag[i]);
        if (i + 1 < k) row += std::abs(sup[i]);
        if (i > 0) row += std::abs(sub[i - 1]);
        tnorm = std::max(tnorm, row);
    }
    double re_poles = 0.0;
    if (sign_by_poles(k, diag, sub, sup, tnorm, host_avx2(), y, &re_poles)) {
        if (info) {
            info->min_abs_re = re_poles;
            info->norm = tnorm;
        }
        return 0;
    }
    std::vector<Rot> rots;
    if (!hessenberg_schur(S, nullptr, &rots)) return 2;
    // eigenvalues and the imaginary-axis check
    double minre = std::numeric_limits<double>::infinity();
    std::vector<double> sgn(k);
    for (int i = 0; i < k; ++i) {
        const double re = S(i, i).real();
        minre = std::min(minre, std::abs(re));
        sgn[i] = re > 0 ? 1.0 : -1.0;
    }
    if (info) {
        info->min_abs_re = minre;
        info->norm = tnorm;
    }
    if (!(minre > 1e-12 * tnorm)) return 3;
    // eigenvectors of S: column i of X with X(i, i) = 1, X(j > i, i) = 0, built in a
    // contiguous vector (the sums run along rows of S) and kept as row i of Xt = X^T
    const double ulp = std::numeric_limits<double>::epsilon();
    const double smin = std::max(ulp * tnorm, std::numeric_limits<double>::min());
    Mat Xt(k);
    std::vector<zc> xv(k);
    double cond_est = 1.0;
    for (int i = 0; i < k; ++i) {
        xv[i] = 1.0;
        const zc lam = S(i, i);
        for (int j = i - 1; j >= 0; --j) {
            const zc *srow = &S(j, 0);
            double ar = 0.0, ai = 0.0;
            for (int l = j + 1; l <= i; ++l) {
                ar += srow[l].real() * xv[l].real() - srow[l].imag() * xv[l].imag();
                ai += srow[l].real() * xv[l].imag() + srow[l].imag() * xv[l].real();
            }
            zc den = S(j, j) - lam;
            if (std::abs(den) < smin) den = smin;
            xv[j] = -zc(ar, ai) / den;
        }
        double cn = 0.0;
        for (int j = 0; j <= i; ++j) {
            cn += std::norm(xv[j]);
            Xt(i, j) = xv[j];
        }
        cond_est = std::max(cond_est, std::sqrt(cn));
    }
    if (info) info->eigvec_growth = cond_est;
    // q = Z^H e_1 (the first row of Z: e_1^T G_1 G_2 ..., conjugated);
    // c = X^{-1} q (unit upper triangular, solved column by column: rows of Xt)
    std::vector<zc> c(k, zc(0.0, 0.0));
    c[0] = 1.0;
    for (const Rot &g : rots) {
        const zc t1 = c[g.m], t2 = c[g.m + 1];
        c[g.m] = t1 * g.c + t2 * std::conj(g.s);
        c[g.m + 1] = -t1 * g.s + t2 * g.c;
    }
    for (int i = 0; i < k; ++i) c[i] = std::conj(c[i]);
    for (int j = k - 1; j > 0; --j) {
        const zc cj = c[j];
        const zc *xrow = &Xt(j, 0);
        for (int i = 0; i < j; ++i) c[i] -= cmul(xrow[i], cj);
    }
    // u = X sign(Lambda) c ; y = Z u
    std::vector<zc> u(k, zc(0, 0));
    for (int j = 0; j < k; ++j) {
        const zc cj = sgn[j] * c[j];
        const zc *xrow = &Xt(j, 0);
        for (int i = 0; i <= j; ++i) u[i] += cmul(xrow[i], cj);
    }
    // y = Z u = G_1 (G_2 (... u)): the rotations in reverse order
    for (auto it = rots.rbegin(); it != rots.rend(); ++it) {
        const zc t1 = u[it->m], t2 = u[it->m + 1];
        u[it->m] = it->c * t1 - it->s * t2;
        u[it->m + 1] = std::conj(it->s) * t1 + it->c * t2;
    }
    for (int i = 0; i < k; ++i) y[i] = u[i];
    return 0;
}

int small_eig(int n, const std::complex<double> *a, std::complex<double> *lam, std::complex<double> *vec)
{
    if (n <= 0) return 1;
    Mat H(n), Z(n);
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) H(i, j) = a[(size_t)i * n + j];
    for (int i = 0; i < n; ++i) Z(i, i) = 1.0;
    // Householder reduction to upper Hessenberg form, H = Z^H A Z
    for (int k = 0; k + 2 < n; ++k) {
        double xn = 0.0;
        for (int i = k + 1; i < n; ++i) xn += std::norm(H(i, k));
        xn = std::sqrt(xn);
        if (xn == 0.0) continue;
        const zc x0 = H(k + 1, k);
        const zc ph = std::abs(x0) > 0.0 ? x0 / std::abs(x0) : zc(1.0, 0.0);
        std::vector<zc> v(n, zc(0, 0));
        for (int i = k + 1; i < n; ++i) v[i] = H(i, k);
        v[k + 1] += ph * xn;  // v = x + e^{i arg x0} ||x|| e_1: no cancellation
        double vn = 0.0;
        for (int i = k + 1; i < n; ++i) vn += std::norm(v[i]);
        vn = std::sqrt(vn);
        for (int i = k + 1; i < n; ++i) v[i] /= vn;
        for (int j = 0; j < n; ++j) {  // H = (I - 2 v v^H) H
            zc d = 0.0;
            for (int i = k + 1; i < n; ++i) d += std::conj(v[i]) * H(i, j);
            for (int i = k + 1; i < n; ++i) H(i, j) -= 2.0 * v[i] * d;
        }
        for (int i = 0; i < n; ++i) {  // H = H (I - 2 v v^H), Z = Z (I - 2 v v^H)
            zc d = 0.0, e = 0.0;
            for (int j = k + 1; j < n; ++j) {
                d += H(i, j) * v[j];
                e += Z(i, j) * v[j];
            }
            for (int j = k + 1; j < n; ++j) {
                H(i, j) -= 2.0 * d * std::conj(v[j]);
                Z(i, j) -= 2.0 * e * std::conj(v[j]);
            }
        }
        for (int i = k + 2; i < n; ++i) H(i, k) = 0.0;
    }
    if (!hessenberg_schur(H, &Z, nullptr)) return 2;
    double tnorm = 0.0;
    for (int i = 0; i < n; ++i)
        for (int j = i; j < n; ++j) tnorm = std::max(tnorm, std::abs(H(i, j)));
    const double smin = std::max(std::numeric_limits<double>::epsilon() * tnorm, std::numeric_limits<double>::min());
    for (int i = 0; i < n; ++i) {
        lam[i] = H(i, i);
        // eigenvector of the triangular factor, X(i) = 1, back substitution above it
        std::vector<zc> x(n, zc(0, 0));
        x[i] = 1.0;
        for (int j = i - 1; j >= 0; --j) {
            zc acc = 0.0;
            for (int l = j + 1; l <= i; ++l) acc += H(j, l) * x[l];
            zc den = H(j, j) - lam[i];
            if (std::abs(den) < smin) den = smin;
            x[j] = -acc / den;
        }
        double nrm = 0.0;
        std::vector<zc> u(n, zc(0, 0));
        for (int r = 0; r < n; ++r) {
            for (int l = 0; l <= i; ++l) u[r] += Z(r, l) * x[l];
            nrm += std::norm(u[r]);
        }
        nrm = std::sqrt(nrm);
        for (int r = 0; r < n; ++r) vec[(size_t)r * n + i] = u[r] / nrm;
    }
    return 0;
}

}  // namespace sgn

extern "C" sgn_status sgn_small_sign(int k, const double *diag, const double *sub, const double *sup, double *y,
                                     double *min_abs_re)
{
    using zc = std::complex<double>;
    return sgn::guard([&] {
        SGN_REQUIRE(k >= 1 && diag && y && (k == 1 || (sub && sup)), "sgn_small_sign: bad arguments");
        for (int i = 0; i < 2 * k; ++i) SGN_REQUIRE(std::isfinite(diag[i]), "sgn_small_sign: diag not finite");
        for (int i = 0; i < 2 * (k - 1); ++i)
            SGN_REQUIRE(std::isfinite(sub[i]) && std::isfinite(sup[i]), "sgn_small_sign: sub/sup not finite");
        sgn::SmallSignInfo info;
        const int rc = sgn::small_sign_e1(k, reinterpret_cast<const zc *>(diag), reinterpret_cast<const zc *>(sub),
                                          reinterpret_cast<const zc *>(sup), reinterpret_cast<zc *>(y), &info);
        if (rc == 3) throw sgn::Failure{SGN_ERR_IMAG_AXIS, "sgn_small_sign: eigenvalue on the imaginary axis"};
        if (rc != 0) throw sgn::Failure{SGN_ERR_BREAKDOWN, "sgn_small_sign: QR iteration did not converge"};
        if (min_abs_re) *min_abs_re = info.min_abs_re;
    });
}
