// Host model of the index arithmetic of the two-factor x and y passes
// (k_fft_two): the same expressions as the kernel's, thread by thread, over
// every length the planner gives them, with full and pruned inputs and windows,
// ragged last workgroups and grids whose lines do not fill a block of columns.
// Checks that every access lies in its buffer, that every LDS slot and every
// output is written exactly once, and (small sizes, in float64) that the two passes
// are the zero-padded DFT of the grid.
#include "hvox_internal.hpp"

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <random>

using namespace hvox;
typedef std::complex<double> C;

#define CHECK(x)                                                                                     \
    do {                                                                                             \
        ++g_chk;                                                                                     \
        if (!(x)) { printf("line %d: %s (nx %d ny %d)\n", __LINE__, #x, g_nx, g_ny); exit(1); }       \
    } while (0)

static long long g_chk = 0;
static int g_nx, g_ny;
static const double kTau = 6.283185307179586476925287;
static C turn(double t) { return std::polar(1.0, kTau * (t - std::rint(t))); }

struct Axis { int n, n1, w, wst; };

static void run(int dtype, Axis X, Axis Y, int n1z, bool transform)
{
    uint8_t f[2][2];
    g_nx = X.n; g_ny = Y.n;
    CHECK(factor_two(X.n, dtype, f[0]) && factor_two(Y.n, dtype, f[1]));
    const int kC = kFft2Block, nb = (int)fft2_blocks(X.w);
    const size_t item = dtype == HVOX_F64 ? 16 : 8;
    std::vector<C> G((size_t)X.n1 * Y.n1 * n1z), A_((size_t)kC * nb * Y.n1 * n1z), B_((size_t)X.w * Y.w * n1z);
    std::vector<int> wa(A_.size(), 0), wb(B_.size(), 0);
    std::mt19937 gen(3);
    std::normal_distribution<double> normal;
    for (C &v : G) v = C(normal(gen), normal(gen));
    for (int pass = 0; pass < 2; ++pass) {
        const Axis &Q = pass ? Y : X;
        const int A = f[pass][0], B = f[pass][1], n = Q.n, half = Q.n1 / 2;
        const int L = fft2_lines(A, B, dtype), row = fft2_row(B), ls = fft2_line(A, B);
        const int threads = (L * A + 63) / 64 * 64;
        CHECK(A * B == n && A >= B && threads >= 64 && threads <= kFft2Threads && L * ls * item <= 65536);
        CHECK(row % 2 == 1 && ls % 32 == 8 && ls >= A * row);
        const int lines = pass == 0 ? n1z * Y.n1 : n1z * nb * kC;
        std::vector<C> &S = pass ? A_ : G, &D = pass ? B_ : A_;
        std::vector<int> &wd = pass ? wb : wa;
        for (int tile = 0; tile * L < lines; ++tile) {
            const int line0 = tile * L;
            std::vector<C> ex((size_t)L * ls);
            std::vector<int> we(ex.size(), 0);
            for (int t = 0; t < threads; ++t) {
                int j, b;
                if (pass == 0) { j = t / B; b = t - j * B; }
                else { const int g = t / (kC * B), r = t - g * (kC * B); b = r / kC; j = g * kC + (r - b * kC); }
                const int li = line0 + j;
                bool on = j < L && li < lines;
                int64_t base;
                uint32_t off, step;
                if (pass == 0) {
                    base = (int64_t)line0 * X.n1;
                    off = (uint32_t)(j * X.n1);
                    step = 1;
                } else {
                    const int zb0 = line0 / kC, zb = li / kC, c = li - zb * kC, z = zb / nb;
                    on = on && (zb - z * nb) * kC + c < X.w;
                    base = (int64_t)zb0 * Y.n1 * kC;
                    off = (uint32_t)((zb - zb0) * Y.n1 * kC + c);
                    step = kC;
                }
                if (!on) continue;
                CHECK(b >= 0 && b < B);
                const uint32_t front = off + (uint32_t)(b + half) * step, back = front - (uint32_t)n * step;
                std::vector<C> v(A);
                for (int a = 0; a < A; ++a) {
                    const bool lo = b < half - a * B, hi = b >= n - half - a * B;
                    const int cell = (lo ? half : half - n) + a * B + b;
                    if (!lo && !hi) continue;
                    CHECK(cell >= 0 && cell < Q.n1);
                    const int64_t at = base + (uint32_t)((lo ? front : back) + (uint32_t)(a * B) * step);
                    CHECK(at >= 0 && at < (int64_t)S.size());
                    if (pass == 0) CHECK(at == (int64_t)li * X.n1 + cell);
                    else CHECK(wa[at] == 1);   // written by the x pass
                    v[a] = S[at];
                }
                for (int k = 0; k < A; ++k) {
                    C x = 0.0;
                    if (transform) for (int a = 0; a < A; ++a) x += v[a] * turn(-(double)(a * k) / A);
                    const int at = j * ls + b + k * row;
                    CHECK(at >= 0 && at < L * ls && ++we[at] == 1);
                    ex[at] = x * turn(-(double)(k * b) / n);
                }
            }
            for (int t = 0; t < threads; ++t) {
                int j, k;
                if (pass == 0) { const int g = t / (kC * A), r = t - g * (kC * A); k = r / kC; j = g * kC + (r - k * kC); }
                else { j = t / A; k = t - j * A; }
                const int li = line0 + j;
                bool on = j < L && li < lines;
                const int q0 = k - Q.wst, wcnt = Q.w;
                int64_t base;
                uint32_t off;
                if (pass == 0) {
                    const int lz0 = line0 / Y.n1, lz = li / Y.n1, ly = li - lz * Y.n1;
                    base = (int64_t)lz0 * nb * Y.n1 * kC;
                    off = (uint32_t)((lz - lz0) * nb * Y.n1 + ly) * kC;
                } else {
                    const int zb0 = line0 / kC, z0 = zb0 / nb, x0 = (zb0 - z0 * nb) * kC, first = z0 * X.w + x0;
                    const int zb = li / kC, z = zb / nb, x = (zb - z * nb) * kC + (li - zb * kC);
                    on = on && x < X.w;
                    base = (int64_t)first * wcnt;
                    off = (uint32_t)((z * X.w + x - first) * wcnt);
                }
                if (!on) continue;
                CHECK(k >= 0 && k < A);
                for (int i = 0; i < B; ++i) {
                    C x = 0.0;
                    for (int b = 0; b < B; ++b) {
                        CHECK(we[j * ls + k * row + b] == 1);
                        if (transform) x += ex[j * ls + k * row + b] * turn(-(double)(b * i) / B);
                    }
                    int q = q0 + A * i;
                    if (q >= wcnt) q -= n;
                    if (q < 0) continue;
                    CHECK(q < wcnt);
                    const uint32_t plane = Y.n1 * kC;
                    CHECK(plane < (1u << 24));
                    const int64_t at = base + off + (pass == 0 ? (uint32_t)(q >> 2) * plane + (q & (kC - 1)) : (uint32_t)q);
                    CHECK(at >= 0 && at < (int64_t)D.size() && ++wd[at] == 1);
                    D[at] = x;
                }
            }
        }
        long long written = 0;
        for (int w : wd) written += w;
        CHECK(written == (pass ? (long long)X.w * Y.w * n1z : (long long)X.w * Y.n1 * n1z));
    }
    if (!transform) return;
    for (int m = 0; m < 30; ++m) {
        const int z = gen() % n1z, x = gen() % X.w, y = gen() % Y.w;
        C r = 0.0;
        for (int a = 0; a < Y.n1; ++a)
            for (int b = 0; b < X.n1; ++b)
                r += G[((size_t)z * Y.n1 + a) * X.n1 + b] *
                     turn(-(double)(x + X.wst) * (b - X.n1 / 2) / X.n - (double)(y + Y.wst) * (a - Y.n1 / 2) / Y.n);
        CHECK(std::abs(B_[((size_t)z * X.w + x) * Y.w + y] - r) < 1e-12 * X.n1 * Y.n1);
    }
}

int main(int argc, char **argv)
{
    const int dtype = argc > 1 ? atoi(argv[1]) : 0;
    std::vector<int> ns;
    for (int n = 2; n <= kFftMaxLen; n += 2) {
        uint8_t f[2];
        if (factor_two(n, dtype, f)) ns.push_back(n);
    }
    std::mt19937 gen(1);
    auto axis = [&](int n, int kind) {   // pruned input and window, full input, full window
        Axis a;
        a.n = n;
        a.n1 = kind == 1 ? n : std::max(2, n * 2 / 3 / 2 * 2);
        const int R = n / 3 + 2;
        if (kind == 2 || 2 * R + 1 >= n) { a.w = n; a.wst = 0; }
        else { a.w = 2 * R + 1; a.wst = -R; }
        return a;
    };
    for (int n : ns)
        for (int kind = 0; kind < 3; ++kind) {
            const int m = ns[gen() % ns.size()];
            run(dtype, axis(n, kind), axis(m, gen() % 3), 1 + gen() % 2, n * m < 20000);
        }
    printf("lengths %zu longest %d checks %lld\n", ns.size(), ns.back(), g_chk);
    return 0;
}
