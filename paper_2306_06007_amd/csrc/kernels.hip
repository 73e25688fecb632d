// HIP kernels of the HVOX library for gfx950 (MI355X): the hot path of the
// chunked 3D type-3 NUFFT (HVOX Sect. 3 and 3.1) and of its block-level
// direct evaluation.
//
// Data layout in HBM
//  * coordinates: float64 structure-of-arrays [3][n] in chunk order;
//  * user data:   complex (float2 / double2) in user order, gathered through
//                 the chunk-order permutation (Sect. 4, chunk-order views), or
//                 already in chunk order (pre-ordered plans);
//  * occupancy:   one bit per grid-1 tile (32 x 8 x 8 cells), set when the
//                 tile holds sources; spreading writes only those tiles and
//                 the x pass reads the others as zeros;
//  * grids:       per batch of sub-problems and per data row of a pass one
//                 workspace copy with three regions:
//                 G holds every pair's grid 1 as [n1z][n1y][n1x]; where both
//                 lengths have two factors the x pass writes its kept window to
//                 A in blocks of four columns ([n1z][wx/4][n1y][4]), which the y
//                 pass reads; other lengths go line-major to B ([n1z][n1y][wx])
//                 and through a tiled transpose to A ([n1z][wx][n1y]).  The y
//                 pass writes B ([n1z][wx][wy]), and the z pass reads its lines
//                 strided and writes A as [wx][wy][wz] (z fastest), which the
//                 interpolation reads;
//  * accumulator: float64 complex per target (chunk order); directions without
//                 NUFFT sub-problems and deterministic plans may keep partial sums
//                 of the direct sum beside it ([layer][target]), added up in order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "hvox_internal.hpp"

namespace hvox {

template <typename T> struct C2;
template <> struct C2<float> { using type = float2; };
template <> struct C2<double> { using type = double2; };
template <typename T> using cplx = typename C2<T>::type;

template <typename T> __device__ __forceinline__ cplx<T> mk(T a, T b) { cplx<T> r; r.x = a; r.y = b; return r; }
template <typename T> __device__ __forceinline__ cplx<T> cadd(cplx<T> a, cplx<T> b) { return mk<T>(a.x + b.x, a.y + b.y); }
template <typename T> __device__ __forceinline__ cplx<T> csub(cplx<T> a, cplx<T> b) { return mk<T>(a.x - b.x, a.y - b.y); }
template <typename T> __device__ __forceinline__ cplx<T> cmul(cplx<T> a, cplx<T> b)
{
    return mk<T>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <typename T> __device__ __forceinline__ cplx<T> cscale(cplx<T> a, T s) { return mk<T>(a.x * s, a.y * s); }
// multiply by s*i (s = +1 or -1)
template <typename T> __device__ __forceinline__ cplx<T> cmuli(cplx<T> a, T s) { return mk<T>(-s * a.y, s * a.x); }

// exponential of semicircle ES(z) = exp(beta (sqrt(1 - z^2) - 1)), |z| < 1
__device__ __forceinline__ float es_kernel(float z, float beta)
{
    // hardware square root and base-2 exponential (about 1 ulp each): far
    // below the kernel's own truncation error at any float32 tolerance
    float q = 1.0f - z * z;
    return q > 0.0f ? __builtin_amdgcn_exp2f(beta * 1.44269504088896341f * (__builtin_amdgcn_sqrtf(q) - 1.0f)) : 0.0f;
}
__device__ __forceinline__ double es_kernel(double z, double beta)
{
    double q = 1.0 - z * z;
    return q > 0.0 ? exp(beta * (sqrt(q) - 1.0)) : 0.0;
}

// exp(2 pi i s f) for a phase f in cycles, evaluated in float64 after
// reduction to [-1/2, 1/2]
__device__ __forceinline__ double2 cis_cycles(double f, double s)
{
    double r = f - rint(f);
    double sn, cs;
    sincospi(2.0 * r, &sn, &cs);
    return make_double2(cs, s * sn);
}

__device__ __forceinline__ int64_t find_segment(const int64_t *__restrict__ prefix, int n, int64_t g)
{
    int lo = 0, hi = n - 1;          // largest p with prefix[p] <= g
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// floor(a / d) for 0 <= a < 2^21, given rd = 1/d as a float.  (a + 1/2) / d
// is at least 1/(2d) away from every integer while the float product is off
// by at most (a + 1/2) / d * 2^-22 < 1/(2d), so truncation gives the exact
// quotient: a few full-rate instructions instead of a 32-bit integer division.
__device__ __forceinline__ int small_div(int a, float rd)
{
    return static_cast<int>((static_cast<float>(a) + 0.5f) * rd);
}
static_assert(kFftElems < (1 << 21), "FFT workgroup indices must stay below 2^21 for small_div");

// 1/d for small_div from the hardware reciprocal (within 1 ulp: the product
// in small_div then stays inside the 2^-22 budget above)
__device__ __forceinline__ float small_rcp(int d) { return __builtin_amdgcn_rcpf(static_cast<float>(d)); }
static_assert(int64_t(kFftMaxLen / kTileX) * (kFftMaxLen / kTileY) * (kFftMaxLen / kTileZ) < (int64_t(1) << 31),
              "grid-1 tiles of a sub-problem must fit 31 bits");

// ---------------------------------------------------------------------------
// accumulator clear
// ---------------------------------------------------------------------------
// (and of the direct sum's item queue, if given)
__global__ void k_zero(double *__restrict__ p, int64_t n, unsigned long long *__restrict__ queue)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (queue && i == 0) *queue = 0;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0.0;
}

// ---------------------------------------------------------------------------
// deconvolution factors 1 / prod_d Psi_hat(nu_d) of every target, where
// nu_d = (s_d - s_c,d) h_d and Psi_hat(nu) = (w/2) int_{-1}^{1} ES(z) cos(pi nu w z) dz
// (Gauss-Legendre; aq = weight * ES(node)).
// ---------------------------------------------------------------------------
__global__ void k_deconv(const double *__restrict__ xyz, int64_t n, const int32_t *__restrict__ chunk_of,
                         const double *__restrict__ ctr, const double *__restrict__ hscale,
                         const double *__restrict__ zq, const double *__restrict__ aq, int nq, int w,
                         double *__restrict__ out)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int32_t c = chunk_of[k];
    double prod = 1.0;
    for (int d = 0; d < 3; ++d) {
        double nu = (xyz[d * n + k] - ctr[3 * c + d]) * hscale[3 * c + d];
        double s = 0.0;
        for (int q = 0; q < nq; ++q) s += aq[q] * cospi(nu * w * zq[q]);
        prod *= 0.5 * w * s;
    }
    out[k] = 1.0 / prod;
}

// ---------------------------------------------------------------------------
// spreading (type-3 step 1, Sect. 3):
//   b_l = sum_n c'_n prod_d ES((l_d - t_nd) 2/w),  c'_n = c_n exp(2 pi i iota s_c.x'_n),
// with t_n = (x_n - x_c) * kscale (grid-1 units) and l in [-n1/2, n1/2)^3.
// ---------------------------------------------------------------------------

// grid-1 footprint of a source: first cell (local index l + n1/2) and the
// float64 grid coordinate; shared by the binning and the spreading kernels so
// that both see exactly the same cells.
__device__ __forceinline__ void source_footprint(const PairDev &P, const double *__restrict__ xyz, int64_t nsrc,
                                                 int64_t n, int w, double xp[3], double t[3], int c0[3])
{
    for (int d = 0; d < 3; ++d) {
        xp[d] = xyz[d * nsrc + n] - P.xc[d];
        t[d] = xp[d] * P.kscale[d];
        c0[d] = (int)ceil(t[d] - 0.5 * w) + P.n1[d] / 2;
    }
}

// Plan-time binning: every (sub-problem, source) pair is listed under each
// grid-1 tile its w^3 footprint touches.  Pass 1 (cursor == nullptr)
// counts, pass 2 scatters the pair's index in the batch's staging order to
// the offsets the host computed.
__global__ void k_bin_points(const PairDev *__restrict__ pairs, const int64_t *__restrict__ prefix, int npairs,
                             int64_t total, const double *__restrict__ xyz, int64_t nsrc, int w,
                             int32_t *__restrict__ counts, unsigned long long *__restrict__ cursor,
                             int32_t *__restrict__ records)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const int p = (int)find_segment(prefix, npairs, g);
    const PairDev &P = pairs[p];
    const int64_t n = P.src_off + (g - prefix[p]);
    double xp[3], t[3];
    int c0[3];
    source_footprint(P, xyz, nsrc, n, w, xp, t, c0);
    const int tdim[3] = {kTileX, kTileY, kTileZ};
    int lo[3], hi[3];
    for (int d = 0; d < 3; ++d) {
        lo[d] = max(0, c0[d]) / tdim[d];
        hi[d] = min(P.n1[d] - 1, c0[d] + w - 1);
        hi[d] = hi[d] < 0 ? -1 : hi[d] / tdim[d];
        hi[d] = min(hi[d], P.ntile[d] - 1);
    }
    for (int tz = lo[2]; tz <= hi[2]; ++tz)
        for (int ty = lo[1]; ty <= hi[1]; ++ty)
            for (int tx = lo[0]; tx <= hi[0]; ++tx) {
                const int64_t tile = P.tile0 + ((int64_t)tz * P.ntile[1] + ty) * P.ntile[0] + tx;
                if (cursor == nullptr) {
                    atomicAdd(counts + tile, 1);
                } else {
                    const unsigned long long pos = atomicAdd(cursor + tile, 1ull);
                    records[pos] = (int32_t)g;   // batches hold fewer than 2^31 sources
                }
            }
}

// Gather + pre-phase of a batch's sources (type-3 centring, the source side):
// c'_n = c_perm(n) exp(2 pi i iota s_c.(x_n - x_c)) for every source of every
// sub-problem of the batch, in the batch's order (sub-problem, then chunk
// order), staged with its kernel footprint on grid 1 for the spreading pass
// (computed once per source instead of once per tile it touches).  The phase
// and the footprint are float64.  With several data rows in the pass (the
// ntrans rows of Sect. 4), the footprint and phase factor are computed once
// and the further rows' values go to xval, row-major with stride xstride.
template <typename T>
__global__ void k_prephase(const PairDev *__restrict__ pairs, const int64_t *__restrict__ pprefix, int npairs,
                           int64_t total, const double *__restrict__ xyz, int64_t nsrc,
                           const int32_t *__restrict__ perm, const cplx<T> *__restrict__ in, int64_t in_stride,
                           int nr, StagedSrc<T> *__restrict__ stage, cplx<T> *__restrict__ xval, int64_t xstride,
                           double iota, int w)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const int p = (int)find_segment(pprefix, npairs, g);
    const PairDev &P = pairs[p];
    const int64_t n = P.src_off + (g - pprefix[p]);
    double xp[3], t[3];
    int c0[3];
    source_footprint(P, xyz, nsrc, n, w, xp, t, c0);
    double ph = 0.0;
    for (int d = 0; d < 3; ++d) ph += P.sc[d] * xp[d];
    const double2 e = cis_cycles(ph, iota);
    const int64_t u = perm ? perm[n] : n;   // no permutation: data already in chunk order
    const cplx<T> c = in[u];
    StagedSrc<T> s;
    s.v[0] = T(c.x * e.x - c.y * e.y);
    s.v[1] = T(c.x * e.y + c.y * e.x);
    for (int d = 0; d < 3; ++d) {
        s.frac[d] = T((double)(c0[d] - P.n1[d] / 2) - t[d]);
        s.c0[d] = c0[d];
    }
    stage[g] = s;
    // further data rows of the pass: the same phase factor, values only
    for (int r = 1; r < nr; ++r) {
        const cplx<T> cr = in[r * in_stride + u];
        xval[(r - 1) * xstride + g] = mk<T>(T(cr.x * e.x - cr.y * e.y), T(cr.x * e.y + cr.y * e.x));
    }
}

// eight consecutive LDS values (16-byte aligned) as wide reads
__device__ __forceinline__ void load8(const float *p, float v[8])
{
    const float4 a = reinterpret_cast<const float4 *>(p)[0], b = reinterpret_cast<const float4 *>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const double *p, double v[8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double2 a = reinterpret_cast<const double2 *>(p)[i];
        v[2 * i] = a.x;
        v[2 * i + 1] = a.y;
    }
}

// Spreading by grid-1 tile: one workgroup per tile.  Thread (x, y) of the
// 32 x 8 face owns the kTileZ cells of its column (a wavefront per 8 x 8 patch
// of the face); the tile's sources are staged kSpreadBatch at a time in LDS
// (pre-phased value, footprint origin relative to the tile, the 2w x and y
// kernel values in the source's frame and the kTileZ z values in the tile's
// frame, zero outside the footprint), every thread adds the contributions that
// fall in its column with two wide LDS reads and 2 kTileZ FMAs per source, and
// the whole tile is written once (no atomics; for a given plan the result is
// deterministic).  A crowded tile (more than kSpreadSplit sources) is split
// into parts, one workgroup each: the first stores like any tile, the others
// (a second launch) add their sums atomically on top (float atomics: the
// rounding order of those cells varies from run to run).  The tile's sub-problem, corner and source list come from
// one plan-time descriptor (the binning), each source's value and footprint
// from the pre-phase pass.  NR data rows share one evaluation of the kernel
// weights (row r's grid is the r-th copy of the batch workspace, ws_stride
// complex elements apart).
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_spread(const PairDev *__restrict__ pairs,
                                                const SpreadTile *__restrict__ tiles,
                                                const int32_t *__restrict__ records,
                                                const StagedSrc<T> *__restrict__ staged,
                                                const cplx<T> *__restrict__ xval, int64_t xstride,
                                                cplx<T> *__restrict__ ws, int64_t ws_stride,
                                                const T *__restrict__ precor, int w, T beta, T two_over_w, float rwk)
{
    static_assert(kTileZ == 8, "the z weights of a source are read as 8 values");
    // per staged source: kTileZ z values in the tile's frame, then w x and w y
    // values in the source's frame (rows a multiple of 16 bytes)
    constexpr int kKv = kTileZ + 2 * kWMax;
    static_assert(kKv % 4 == 0, "16-byte rows");
    __shared__ __align__(16) T kv[kSpreadBatch][kKv];
    __shared__ T frac[kSpreadBatch][3];
    __shared__ cplx<T> val[NR][kSpreadBatch];
    __shared__ int org[kSpreadBatch][3];
    const int tid = threadIdx.x;
    const SpreadTile tile = tiles[blockIdx.x];
    const int ox = tile.org[0], oy = tile.org[1], oz = tile.org[2];
    // each wavefront owns an 8 x 8 patch of columns (x fastest): a w-wide
    // footprint meets one or two of the four wavefronts instead of all of them
    static_assert(kTileX == 32 && kTileY == 8, "8 x 8 column patches per wavefront");
    const int x = (tid & 7) + 8 * (tid >> 6), y = (tid >> 3) & 7;
    const int wk = 2 * w + kTileZ;   // kernel values per staged source
    T accr[NR][kTileZ], acci[NR][kTileZ];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int z = 0; z < kTileZ; ++z) accr[r][z] = acci[r][z] = T(0);

    for (int base = 0; base < tile.cnt; base += kSpreadBatch) {
        const int cnt = min(kSpreadBatch, tile.cnt - base);
        __syncthreads();
        if (tid < cnt) {
            const int32_t rec = records[tile.r0 + base + tid];
            const StagedSrc<T> sc = staged[rec];
            for (int d = 0; d < 3; ++d) frac[tid][d] = sc.frac[d];
            org[tid][0] = sc.c0[0] - ox;
            org[tid][1] = sc.c0[1] - oy;
            org[tid][2] = sc.c0[2] - oz;
            val[0][tid] = mk<T>(sc.v[0], sc.v[1]);
#pragma unroll
            for (int r = 1; r < NR; ++r) val[r][tid] = xval[(r - 1) * xstride + rec];
        }
        __syncthreads();
        // one branch-free evaluation per entry: z entries take their offset
        // from the tile, x and y entries from the footprint origin
        for (int i = tid; i < cnt * wk; i += 256) {
            const int j = small_div(i, rwk), r = i - __mul24(j, wk);
            const int rr = r - kTileZ;
            const int d = r < kTileZ ? 2 : (rr >= w ? 1 : 0);
            const int q = r < kTileZ ? r - (&org[0][0])[__mul24(j, 3) + 2] : rr - (d ? w : 0);
            const T k = es_kernel(((&frac[0][0])[__mul24(j, 3) + d] + T(q)) * two_over_w, beta);
            (&kv[0][0])[__mul24(j, kKv) + r] = (unsigned)q < (unsigned)w ? k : T(0);
        }
        __syncthreads();
        for (int j = 0; j < cnt; ++j) {
            const int qx = x - org[j][0], qy = y - org[j][1];
            if ((unsigned)qx >= (unsigned)w || (unsigned)qy >= (unsigned)w) continue;
            const T kxy = kv[j][kTileZ + qx] * kv[j][kTileZ + w + qy];
            T kz[kTileZ];
            load8(kv[j], kz);
            // the kernel weights of this source serve every data row
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const T vr = val[r][j].x * kxy, vi = val[r][j].y * kxy;
#pragma unroll
                for (int z = 0; z < kTileZ; ++z) {
                    accr[r][z] += vr * kz[z];
                    acci[r][z] += vi * kz[z];
                }
            }
        }
    }
    const PairDev &P = pairs[tile.pair];
    const int gx = ox + x, gy = oy + y;
    if (gx < P.n1[0] && gy < P.n1[1]) {
        // the pre-correction 1/Phi_hat(l/n2) of the inner FFT, separable, on the way out
        const T fxy = precor[P.precor[0] + gx] * precor[P.precor[1] + gy];
#pragma unroll
        for (int z = 0; z < kTileZ; ++z) {
            const T f = fxy * precor[P.precor[2] + min(oz + z, P.n1[2] - 1)];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                accr[r][z] *= f;
                acci[r][z] *= f;
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            cplx<T> *grid = ws + r * ws_stride + P.bufG;   // row r's copy of the batch workspace
            if (tile.flags & kSpreadAdd) {
#pragma unroll
                for (int z = 0; z < kTileZ; ++z) {
                    const int gz = oz + z;
                    if (gz < P.n1[2]) {
                        T *c = reinterpret_cast<T *>(grid + ((int64_t)gz * P.n1[1] + gy) * P.n1[0] + gx);
                        atomicAdd(c, accr[r][z]);
                        atomicAdd(c + 1, acci[r][z]);
                    }
                }
            } else {
#pragma unroll
                for (int z = 0; z < kTileZ; ++z) {
                    const int gz = oz + z;
                    if (gz < P.n1[2])
                        grid[((int64_t)gz * P.n1[1] + gy) * P.n1[0] + gx] = mk<T>(accr[r][z], acci[r][z]);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// FFT passes (type-3 step 2: zero-padded FFT of the pre-corrected modes on grid 2).
// ---------------------------------------------------------------------------
// exp(2 pi i k / R) as (cos, sin), evaluated by the compiler: the angle is
// folded into [0, pi/4] with the quarter-turn and complement symmetries
// (integer arithmetic, exact) and the Taylor series summed there (eleven terms
// at |x| <= pi/4 leave a truncation below 1e-22).
constexpr double kPiRoots = 3.14159265358979323846;
constexpr double taylor_sin(double x)
{
    double t = x, s = x;
    for (int i = 1; i < 12; ++i) { t *= -x * x / ((2.0 * i) * (2.0 * i + 1.0)); s += t; }
    return s;
}
constexpr double taylor_cos(double x)
{
    double t = 1.0, s = 1.0;
    for (int i = 1; i < 12; ++i) { t *= -x * x / ((2.0 * i - 1.0) * (2.0 * i)); s += t; }
    return s;
}
template <int R> struct Roots {
    double c[R], s[R];
    constexpr Roots() : c(), s()
    {
        for (int k = 0; k < R; ++k) {
            const int q = (4 * k) / R, r = 4 * k - q * R;   // angle (pi/2)(q + r/R), 0 <= r < R
            double cr = 0.0, sr = 0.0;
            if (2 * r <= R) { const double x = kPiRoots / 2 * r / R; cr = taylor_cos(x); sr = taylor_sin(x); }
            else { const double x = kPiRoots / 2 * (R - r) / R; cr = taylor_sin(x); sr = taylor_cos(x); }
            for (int i = 0; i < q; ++i) { const double t = cr; cr = -sr; sr = t; }   // q quarter turns
            c[k] = cr;
            s[k] = sr;
        }
    }
};

template <typename T, int R> __device__ __forceinline__ void dft_small(cplx<T> *u, T s);

// R1 R2-point DFT in registers (Cooley-Tukey, one level): input q = R2 q1 + q2,
// output m = m1 + R1 m2.  An R1-point DFT over q1 for every q2, the twiddle
// w^(q2 m1) with w = exp(s 2 pi i / (R1 R2)), then an R2-point DFT over q2 for
// every m1.
template <typename T, int R1, int R2>
__device__ __forceinline__ void dft_two_factor(cplx<T> *u, T s)
{
    constexpr int R = R1 * R2;
    constexpr Roots<R> W{};
    cplx<T> t[R2][R1];
#pragma unroll
    for (int q2 = 0; q2 < R2; ++q2) {
#pragma unroll
        for (int q1 = 0; q1 < R1; ++q1) t[q2][q1] = u[R2 * q1 + q2];
        dft_small<T, R1>(t[q2], s);
#pragma unroll
        for (int m1 = 1; m1 < R1; ++m1) {
            const int k = (q2 * m1) % R;
            if (k == 0) continue;
            if ((4 * k) % R == 0) {   // a quarter turn: exact
                const int qt = 4 * k / R;
                t[q2][m1] = qt == 1 ? cmuli<T>(t[q2][m1], s)
                          : qt == 2 ? mk<T>(-t[q2][m1].x, -t[q2][m1].y) : cmuli<T>(t[q2][m1], -s);
            } else {
                const T c = T(W.c[k]), sn = s * T(W.s[k]);
                const cplx<T> a = t[q2][m1];
                t[q2][m1] = mk<T>(a.x * c - a.y * sn, a.y * c + a.x * sn);
            }
        }
    }
#pragma unroll
    for (int m1 = 0; m1 < R1; ++m1) {
        cplx<T> b[R2];
#pragma unroll
        for (int q2 = 0; q2 < R2; ++q2) b[q2] = t[q2][m1];
        dft_small<T, R2>(b, s);
#pragma unroll
        for (int m2 = 0; m2 < R2; ++m2) u[m1 + R1 * m2] = b[m2];
    }
}

// In-place R-point DFT u_m <- sum_q u_q exp(s 2 pi i q m / R), s = +-1.
template <typename T, int R>
__device__ __forceinline__ void dft_small(cplx<T> *u, T s)
{
    if constexpr (R == 2) {
        cplx<T> a = u[0], b = u[1];
        u[0] = cadd<T>(a, b);
        u[1] = csub<T>(a, b);
    } else if constexpr (R == 3) {
        const T h = T(0.86602540378443864676);
        cplx<T> t1 = cadd<T>(u[1], u[2]), t2 = csub<T>(u[1], u[2]);
        cplx<T> m = mk<T>(u[0].x - T(0.5) * t1.x, u[0].y - T(0.5) * t1.y);
        cplx<T> r = cmuli<T>(cscale<T>(t2, h), s);
        u[0] = cadd<T>(u[0], t1);
        u[1] = cadd<T>(m, r);
        u[2] = csub<T>(m, r);
    } else if constexpr (R == 4) {
        cplx<T> a = cadd<T>(u[0], u[2]), b = csub<T>(u[0], u[2]);
        cplx<T> c = cadd<T>(u[1], u[3]), d = csub<T>(u[1], u[3]);
        cplx<T> id = cmuli<T>(d, s);
        u[0] = cadd<T>(a, c);
        u[2] = csub<T>(a, c);
        u[1] = cadd<T>(b, id);
        u[3] = csub<T>(b, id);
    } else if constexpr (R == 8) {
        // two 4-point DFTs (even and odd inputs) joined with w^m, w = exp(s 2 pi i / 8)
        const T h = T(0.70710678118654752440);
        cplx<T> e[4] = {u[0], u[2], u[4], u[6]}, o[4] = {u[1], u[3], u[5], u[7]};
        dft_small<T, 4>(e, s);
        dft_small<T, 4>(o, s);
        const cplx<T> o1 = mk<T>(h * (o[1].x - s * o[1].y), h * (o[1].y + s * o[1].x));    // w^1 = (1 + i s)/sqrt2
        const cplx<T> o2 = cmuli<T>(o[2], s);                                              // w^2 = i s
        const cplx<T> o3 = mk<T>(-h * (o[3].x + s * o[3].y), h * (s * o[3].x - o[3].y));   // w^3 = (-1 + i s)/sqrt2
        u[0] = cadd<T>(e[0], o[0]);
        u[4] = csub<T>(e[0], o[0]);
        u[1] = cadd<T>(e[1], o1);
        u[5] = csub<T>(e[1], o1);
        u[2] = cadd<T>(e[2], o2);
        u[6] = csub<T>(e[2], o2);
        u[3] = cadd<T>(e[3], o3);
        u[7] = csub<T>(e[3], o3);
    } else if constexpr (R == 6) { dft_two_factor<T, 3, 2>(u, s);
    } else if constexpr (R == 9) { dft_two_factor<T, 3, 3>(u, s);
    } else if constexpr (R == 10) { dft_two_factor<T, 5, 2>(u, s);
    } else if constexpr (R == 12) { dft_two_factor<T, 4, 3>(u, s);
    } else if constexpr (R == 15) { dft_two_factor<T, 5, 3>(u, s);
    } else if constexpr (R == 16) { dft_two_factor<T, 4, 4>(u, s);
    } else if constexpr (R == 18) { dft_two_factor<T, 9, 2>(u, s);
    } else if constexpr (R == 20) { dft_two_factor<T, 5, 4>(u, s);
    } else if constexpr (R == 24) { dft_two_factor<T, 8, 3>(u, s);
    } else if constexpr (R == 25) { dft_two_factor<T, 5, 5>(u, s);
    } else if constexpr (R == 27) { dft_two_factor<T, 9, 3>(u, s);
    } else if constexpr (R == 30) { dft_two_factor<T, 6, 5>(u, s);
    } else if constexpr (R == 32) { dft_two_factor<T, 8, 4>(u, s);
    } else if constexpr (R == 36) { dft_two_factor<T, 9, 4>(u, s);
    } else if constexpr (R == 40) { dft_two_factor<T, 8, 5>(u, s);
    } else {
        static_assert(R == 5, "radix");
        const T c1 = T(0.30901699437494742410), c2 = T(-0.80901699437494742410);
        const T s1 = T(0.95105651629515357212), s2 = T(0.58778525229247312917);
        cplx<T> t1 = cadd<T>(u[1], u[4]), t2 = cadd<T>(u[2], u[3]);
        cplx<T> t3 = csub<T>(u[1], u[4]), t4 = csub<T>(u[2], u[3]);
        cplx<T> a1 = mk<T>(u[0].x + c1 * t1.x + c2 * t2.x, u[0].y + c1 * t1.y + c2 * t2.y);
        cplx<T> a2 = mk<T>(u[0].x + c2 * t1.x + c1 * t2.x, u[0].y + c2 * t1.y + c1 * t2.y);
        cplx<T> b1 = cmuli<T>(mk<T>(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y), s);
        cplx<T> b2 = cmuli<T>(mk<T>(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y), s);
        u[0] = cadd<T>(u[0], cadd<T>(t1, t2));
        u[1] = cadd<T>(a1, b1);
        u[4] = csub<T>(a1, b1);
        u[2] = cadd<T>(a2, b2);
        u[3] = csub<T>(a2, b2);
    }
}

// One Stockham stage of radix R on nl lines of length n held in LDS, in
// place: every thread first reads and transforms its butterflies into
// registers, then (after a barrier) writes them back in autosorted order.
// Butterfly i of a line: k = i mod p, inputs x[i + q n/R] twiddled by
// w^(k q n / (p R)), outputs at (i - k) R + k + m p.  The first stage
// (FIRST, p = 1) has k = 0: no twiddles.
template <typename T, int R, int NT, bool FIRST>
__device__ __forceinline__ void fft_stage(cplx<T> *lds, int nl, int n, int ls, int p, const cplx<T> *tw, T s)
{
    constexpr int MAXB = (fft_elems(NT) / R + NT - 1) / NT;
    const int nbf = n / R;
    const int total = nl * nbf;
    const int twstep = FIRST ? 0 : small_div(n, small_rcp(p * R));   // exact: p R divides n
    const int pR = p * R;
    const float rnbf = small_rcp(nbf), rp = FIRST ? 1.0f : small_rcp(p);
    cplx<T> v[MAXB][R];
    int obase[MAXB];
    // the thread index, opaque to the optimiser: otherwise the butterfly
    // indices of every radix case are hoisted out of the loop over stages and
    // held in registers across it (64 VGPRs, which halved the occupancy)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int c = 0; c < MAXB; ++c) {
        const int b = tid + c * NT;
        obase[c] = -1;
        if (b < total) {
            const int j = small_div(b, rnbf), i = b - __mul24(j, nbf);
            const int g = FIRST ? i : small_div(i, rp), k = FIRST ? 0 : i - __mul24(g, p);
            const int lb = __mul24(j, ls);   // line j starts at j * ls in LDS
            obase[c] = lb + __mul24(g, pR) + k;
            const int tk = __mul24(k, twstep);
#pragma unroll
            for (int q = 0; q < R; ++q) {
                cplx<T> u = lds[lb + i + __mul24(q, nbf)];
                // exponent q k twstep < n; the LDS table holds exp(s 2 pi i j/n), j < n
                if (!FIRST && q > 0) u = cmul<T>(u, tw[__mul24(q, tk)]);
                v[c][q] = u;
            }
            dft_small<T, R>(v[c], s);
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < MAXB; ++c) {
        if (obase[c] >= 0) {
#pragma unroll
            for (int m = 0; m < R; ++m) lds[obase[c] + __mul24(m, p)] = v[c][m];
        }
    }
    __syncthreads();
}

// A stage of any of the planner's radices (2, 3, 4, 5, 8, 9).
template <typename T, int NT, bool FIRST>
__device__ __forceinline__ void fft_stage_radix(int R, cplx<T> *lds, int nl, int n, int ls, int p, const cplx<T> *tw, T s)
{
    switch (R) {
    case 9: fft_stage<T, 9, NT, FIRST>(lds, nl, n, ls, p, tw, s); break;
    case 8: fft_stage<T, 8, NT, FIRST>(lds, nl, n, ls, p, tw, s); break;
    case 5: fft_stage<T, 5, NT, FIRST>(lds, nl, n, ls, p, tw, s); break;
    case 4: fft_stage<T, 4, NT, FIRST>(lds, nl, n, ls, p, tw, s); break;
    case 3: fft_stage<T, 3, NT, FIRST>(lds, nl, n, ls, p, tw, s); break;
    default: fft_stage<T, 2, NT, FIRST>(lds, nl, n, ls, p, tw, s); break;
    }
}

// One axis pass for every sub-problem of a batch.  Element e of an input
// line is mode l = e - nin/2, placed at FFT slot l mod n (zero elsewhere: the
// zero padding of grid 1 into grid 2 is never stored).  The x and y passes
// read contiguous lines; the z pass reads its lines strided (line j of the
// plane is element j of every z-slab, so consecutive lines sit in adjacent
// lanes).  The x pass reads grid-1 tiles that hold no source as zeros.  The second grid
// dimension runs over the data rows of the pass.  Output
// q of the kept window is FFT index (wstart + q) mod n, written line-major:
// out[line][q].
template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_fft_pass(const PairDev *__restrict__ pairs, const int64_t *__restrict__ prefix,
                                                 int npairs, int pass, cplx<T> *__restrict__ ws,
                                                 const cplx<T> *__restrict__ twtab,
                                                 const uint32_t *__restrict__ occ, int tw_off, T s,
                                                 int64_t ws_stride)
{
    static_assert(kTileX == 32, "a grid-1 tile spans 32 cells of an x line");
    ws += (int64_t)blockIdx.y * ws_stride;   // data row blockIdx.y: its copy of the batch workspace
    extern __shared__ unsigned char smem_raw[];
    cplx<T> *lds = reinterpret_cast<cplx<T> *>(smem_raw);
    cplx<T> *ltw = lds + tw_off;              // exp(s 2 pi i j/n), j < n, after the lines
    __shared__ uint32_t lmask[kFftMaxLines][kOccWords];   // x pass: occupancy bits of each line's tile row
    __shared__ int lbit0[kFftMaxLines];
    const int p = (int)find_segment(prefix, npairs, blockIdx.x);
    const PairDev &P = pairs[p];
    const int64_t tile = (int64_t)blockIdx.x - prefix[p];
    const int n = P.n2[pass], nin = P.n1[pass];
    const int wst = P.wstart[pass], wcnt = P.wcount[pass];
    int64_t lines;
    const cplx<T> *src;
    cplx<T> *dst;
    if (pass == 0) { lines = (int64_t)P.n1[2] * P.n1[1]; src = ws + P.bufG; dst = ws + P.bufB; }
    else if (pass == 1) { lines = (int64_t)P.n1[2] * P.wcount[0]; src = ws + P.bufA; dst = ws + P.bufB; }
    else { lines = (int64_t)P.wcount[0] * P.wcount[1]; src = ws + P.bufB; dst = ws + P.bufA; }
    const int L = P.lines_per_tile[pass];
    const int64_t line0 = tile * L;
    const int nl = (int)min((int64_t)L, lines - line0);
    const int half_in = nin / 2, half_n = n / 2;
    const int ls = fft_lds_stride(n);   // LDS line stride

    {
        // twiddles of this line length, staged with the data (sign s applied here)
        const cplx<T> *tw = twtab + P.tw[pass];
        for (int j = threadIdx.x; j < n; j += NT) {
            cplx<T> t = tw[j];
            t.y *= -s;   // table holds exp(-2 pi i j/n); s = -1 keeps it, +1 conjugates
            ltw[j] = t;
        }
    }
    if (pass == 0) {
        if ((int)threadIdx.x < nl) {
            const int64_t li = line0 + threadIdx.x;
            const int64_t lz = li / P.n1[1], ly = li - lz * P.n1[1];
            // tiles of this line's row: bit rowbit + tx is tile (tx, ly / 8, lz / 8) of the pair;
            // a tile without sources was never written and reads as zeros (no bitmap: all read)
            const int64_t rowbit = P.tile0 + ((lz / kTileZ) * P.ntile[1] + ly / kTileY) * P.ntile[0];
            lbit0[threadIdx.x] = (int)(rowbit & 31);
            for (int q = 0; q < kOccWords; ++q) lmask[threadIdx.x][q] = occ ? occ[(rowbit >> 5) + q] : ~0u;
        }
        __syncthreads();
    }
    // every thread loads its (at most) fft_elems(NT) / NT elements into
    // registers first, so the global loads are all in flight together, then
    // writes them to LDS
    constexpr int EPT = fft_elems(NT) / NT;
    static_assert(fft_elems(NT) % NT == 0, "FFT workgroup elements");
    const int ne = nl * n;
    cplx<T> v[EPT];
    if (pass < 2) {
        const cplx<T> *sb = src + line0 * nin;
        const float rn = small_rcp(n);
        int slot[EPT];
#pragma unroll
        for (int c = 0; c < EPT; ++c) {
            const int e = threadIdx.x + c * NT;
            v[c] = mk<T>(T(0), T(0));
            slot[c] = 0;
            if (e < ne) {
                const int j = small_div(e, rn), f = e - __mul24(j, n);
                const int l = f < half_n ? f : f - n;
                slot[c] = __mul24(j, ls) + f;
                bool take = l >= -half_in && l < half_in;
                if (pass == 0 && take) {
                    const int b = lbit0[j] + ((l + half_in) >> 5);
                    take = (lmask[j][b >> 5] >> (b & 31)) & 1u;
                }
                if (take) v[c] = sb[__mul24(j, nin) + l + half_in];
            }
        }
#pragma unroll
        for (int c = 0; c < EPT; ++c) {
            const int e = threadIdx.x + c * NT;
            if (e < ne) lds[slot[c]] = v[c];
        }
    } else {
        const cplx<T> *sb = src + line0;
        const float rl = small_rcp(nl);
        int slot[EPT];
#pragma unroll
        for (int c = 0; c < EPT; ++c) {
            const int e = threadIdx.x + c * NT;
            v[c] = mk<T>(T(0), T(0));
            slot[c] = -1;
            if (e < ne) {
                const int f = small_div(e, rl), j = e - __mul24(f, nl);
                const int l = f < half_n ? f : f - n;
                slot[c] = __mul24(j, ls) + f;
                if (l >= -half_in && l < half_in) v[c] = sb[(int64_t)(l + half_in) * lines + j];
            }
        }
#pragma unroll
        for (int c = 0; c < EPT; ++c)
            if (slot[c] >= 0) lds[slot[c]] = v[c];
    }
    __syncthreads();
    int pc = 1;
    for (int st = 0; st < P.nrad[pass]; ++st) {
        const int R = P.radix[pass][st];
        if (st == 0) fft_stage_radix<T, NT, true>(R, lds, nl, n, ls, pc, ltw, s);
        else fft_stage_radix<T, NT, false>(R, lds, nl, n, ls, pc, ltw, s);
        pc *= R;
    }
    // kept window: wstart is 0 (whole line) or -R with 2R < n, so wstart + q lies in (-n, n)
    cplx<T> *out = dst + line0 * wcnt;
    const float rw = small_rcp(wcnt);
    for (int e = threadIdx.x; e < nl * wcnt; e += NT) {
        const int j = small_div(e, rw), q = e - __mul24(j, wcnt);
        int m = wst + q;
        if (m < 0) m += n;
        out[e] = lds[__mul24(j, ls) + m];
    }
}

// ---------------------------------------------------------------------------
// x and y passes in two factors, n = A B.  Slot f = a B + b of a line, output
// m = k + A q:  X[k + A q] = sum_b w_B^(b q) [ w_n^(b k) sum_a w_A^(a k) x[a B + b] ].
// A thread takes column b: it loads its A elements straight into registers
// (zero padding and empty tiles are not read), transforms them, multiplies by the twiddles (table in the
// order [k][b]) and leaves them in LDS; a thread then takes row k, transforms its B
// values and writes its kept outputs straight from registers.
// Pass x reads contiguous lines and writes its window in blocks of kFft2Block
// columns, [z][x / 4][y][4]: four lines at a time fill 128-byte segments (float32), and
// pass y reads four neighbouring lines as one contiguous run.  No transpose.
//
// What bounds it: load, transform, exchange and store of a line follow each other,
// and registers let only three (float32, 168) or two wavefronts per SIMD (float64, 228)
// overlap them: leaving out loads, stores, transforms or twiddles each saved about a fifth.
// VALU is busy 45% of the time, traffic is 2.1 (x) and 3.3 TB/s (y, float32), 2.7 and 4.2
// TB/s (float64) of 4.7 for a copy.  Of the general passes it replaces (four or five radix
// stages of a 1200-point line, each with its index arithmetic, an LDS round
// trip and two barriers; a transpose between x and y), x + transpose + y took 26.1 ms on
// the 3 km dense mesh with every sub-problem a NUFFT (float32; now 15.5) and 11.0 ms on
// the 1 km one (float64; now 5.8).  Tried: several groups of lines per workgroup
// (8% slower), twiddles staged in LDS (4% slower: another barrier), smaller
// groups (10% slower), 128 registers (more spills; lengths up to 27 x 27 only).  One
// instance serves every factor: the 36- and 40-point transforms spill 40 (x) and 48 bytes (y)
// a lane in float32, and short lines run at the longest factor's registers.  Longer
// factors than 27 in float64 would take more than 256 registers.
// ---------------------------------------------------------------------------

// calls f with the compile-time constant equal to r (a factor of the planner's list)
template <int MAX, typename F> __device__ __forceinline__ void fft2_switch(int r, F &&f)
{
#define HVOX_CASE(R) case R: if constexpr (R <= MAX) f(std::integral_constant<int, R>{}); break;
    switch (r) {
        HVOX_CASE(3) HVOX_CASE(4) HVOX_CASE(5) HVOX_CASE(6) HVOX_CASE(8) HVOX_CASE(9) HVOX_CASE(10) HVOX_CASE(12) HVOX_CASE(15)
        HVOX_CASE(16) HVOX_CASE(18) HVOX_CASE(20) HVOX_CASE(24) HVOX_CASE(25) HVOX_CASE(27) HVOX_CASE(30)
        HVOX_CASE(32) HVOX_CASE(36) HVOX_CASE(40)
    default: break;
    }
#undef HVOX_CASE
}

// element at a 32-bit byte offset from a base that is uniform over the workgroup
template <typename V> __device__ __forceinline__ V &at_bytes(V *base, uint32_t off)
{
    using Byte = std::conditional_t<std::is_const_v<V>, const unsigned char, unsigned char>;
    return *reinterpret_cast<V *>(reinterpret_cast<Byte *>(base) + off);
}

template <typename T, int PASS, int SIGN>
__global__ __launch_bounds__(kFft2Threads, sizeof(T) == 8 ? 2 : 3) void k_fft_two(
    const PairDev *__restrict__ pairs, const int64_t *__restrict__ prefix, int npairs, cplx<T> *__restrict__ ws,
    const cplx<T> *__restrict__ twtab, const uint32_t *__restrict__ occ, int64_t ws_stride)
{
    static_assert(kTileX == 32 && kFft2MaxX <= 32 * kTileX, "a line's tiles fit a word");
    // over the direct sum's wavefronts, which never wait for memory (3 km dense mesh, automatic
    // choice: 8.7 -> 8.2 ms; the other NUFFT kernels gain nothing from it beside a long direct sum)
    __builtin_amdgcn_s_setprio(2);
    constexpr T s = T(SIGN);   // (a constant: the quarter turns of the DFTs cost nothing)
    constexpr int kType = sizeof(T) == 8 ? HVOX_F64 : HVOX_F32, kMax = fft2_max_factor(kType), kC = kFft2Block;
    constexpr uint32_t kB = sizeof(cplx<T>);
    extern __shared__ unsigned char smem_raw[];
    cplx<T> *ex = reinterpret_cast<cplx<T> *>(smem_raw);
    ws += (int64_t)blockIdx.y * ws_stride;   // data row blockIdx.y: its copy of the batch workspace
    const int p = (int)find_segment(prefix, npairs, blockIdx.x);
    const PairDev &P = pairs[p];
    const int A = P.two[PASS][0], B = P.two[PASS][1], n = P.n2[PASS], half_in = P.n1[PASS] / 2;
    const int L = fft2_lines(A, B, kType), row = fft2_row(B), ls = fft2_line(A, B);
    const int wx = P.wcount[0], n1x = P.n1[0], n1y = P.n1[1], n1z = P.n1[2];
    const int nb = (int)fft2_blocks(wx);          // blocks of columns in a grid plane
    const int lines = PASS == 0 ? n1z * n1y : n1z * nb * kC;   // (a region holds fewer than 2^31 elements)
    const int line0 = (int)(blockIdx.x - prefix[p]) * L;
    const int t = threadIdx.x;
    {
        // column b of line j: pass x along the line in adjacent lanes, pass y across the four lines of a block first
        int j, b;
        if (PASS == 0) { j = t / B; b = t - j * B; }
        else { const int g = t / (kC * B), r = t - g * (kC * B); b = r / kC; j = g * kC + (r - b * kC); }
        const int li = line0 + j;
        const cplx<T> *src;
        uint32_t off;                 // byte offset of the line's first cell
        uint32_t tiles = ~0u;         // occupied tiles of the line's row
        bool on = j < L && li < lines;
        if (PASS == 0) {
            src = ws + P.bufG + (int64_t)line0 * n1x;
            off = (uint32_t)(j * n1x) * kB;
            if (on && occ) {   // (padded: the word past a row's last tile may be read)
                const int lz = li / n1y, ly = li - lz * n1y;
                const int64_t bit = P.tile0 + ((int64_t)(lz / kTileZ) * P.ntile[1] + ly / kTileY) * P.ntile[0];
                const uint32_t *o = occ + (bit >> 5);
                tiles = __builtin_amdgcn_alignbit(o[1], o[0], (uint32_t)(bit & 31));
            }
        } else {
            // line c of block zb / z of plane z (the last block may hold columns past the window)
            const int zb0 = line0 / kC, zb = li / kC, c = li - zb * kC, z = zb / nb;
            on = on && (zb - z * nb) * kC + c < wx;
            src = ws + P.bufA + (int64_t)zb0 * n1y * kC;
            off = (uint32_t)((zb - zb0) * n1y * kC + c) * kB;
        }
        const cplx<T> *tw = twtab + P.tw[PASS];   // order [k][b]
        // slot f = a B + b holds mode f (f < half_in, cell f + half_in) or mode f - n (f >= n -
        // half_in, cell f - n + half_in), else zero
        constexpr uint32_t kStep = PASS == 0 ? kB : kB * kC;
        const uint32_t front = off + (uint32_t)(b + half_in) * kStep, back = front - (uint32_t)n * kStep;
        cplx<T> *to = ex + j * ls + b;
        fft2_switch<kMax>(A, [&](auto RA) {
            constexpr int R = decltype(RA)::value;
            cplx<T> v[R];
#pragma unroll
            for (int a = 0; a < R; ++a) {
                const bool lo = b < half_in - a * B, hi = b >= n - half_in - a * B;
                bool take = on && (lo || hi);
                if (PASS == 0) {
                    const int cell = (lo ? half_in : half_in - n) + a * B + b;
                    take = take && __builtin_amdgcn_ubfe(tiles, cell >> 5, 1);
                }
                v[a] = mk<T>(T(0), T(0));
                if (take) v[a] = at_bytes(src, (lo ? front : back) + (uint32_t)(a * B) * kStep);
            }
            dft_small<T, R>(v, s);
            if (on) {
                to[0] = v[0];
#pragma unroll
                for (int k = 1; k < R; ++k) {
                    const cplx<T> w = at_bytes(tw, (uint32_t)(k * B + b) * kB);   // exp(-2 pi i k b / n), conjugated for s = +1
                    to[k * row] = cmul<T>(v[k], mk<T>(w.x, SIGN < 0 ? w.y : -w.y));
                }
            }
        });
    }
    __syncthreads();
    {
        // row k of line j: pass x across four lines in adjacent lanes (its blocks of columns), pass y along the line
        int j, k;
        if (PASS == 0) { const int g = t / (kC * A), r = t - g * (kC * A); k = r / kC; j = g * kC + (r - k * kC); }
        else { j = t / A; k = t - j * A; }
        const int li = line0 + j;
        bool on = j < L && li < lines;
        // kept window: wstart is 0 (whole line) or -R with 2 R < n
        const int q0 = k - P.wstart[PASS], wcnt = P.wcount[PASS];
        cplx<T> *dst;
        uint32_t off;                 // byte offset of the line's first kept output
        if (PASS == 0) {
            const int lz0 = line0 / n1y, lz = li / n1y, ly = li - lz * n1y;
            dst = ws + P.bufA + (int64_t)lz0 * nb * n1y * kC;
            off = (uint32_t)((lz - lz0) * nb * n1y + ly) * (kC * kB);
        } else {
            const int zb0 = line0 / kC, z0 = zb0 / nb, x0 = (zb0 - z0 * nb) * kC, first = z0 * wx + x0;
            const int zb = li / kC, z = zb / nb, x = (zb - z * nb) * kC + (li - zb * kC);
            on = on && x < wx;
            dst = ws + P.bufB + (int64_t)first * wcnt;
            off = (uint32_t)((z * wx + x - first) * wcnt) * kB;
        }
        const cplx<T> *from = ex + j * ls + k * row;
        const uint32_t plane = n1y * kC;   // pass x: elements from a block of columns to the next
        if (on)
            fft2_switch<kMax>(B, [&](auto RB) {
                constexpr int R = decltype(RB)::value;
                cplx<T> u[R];
#pragma unroll
                for (int i = 0; i < R; ++i) u[i] = from[i];
                dft_small<T, R>(u, s);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    int q = q0 + A * i;
                    if (q >= wcnt) q -= n;
                    const uint32_t e = PASS == 0 ? __umul24(q >> 2, plane) + (q & (kC - 1)) : q;
                    if (q >= 0) at_bytes(dst, off + e * kB) = u[i];
                }
            });
    }
}

// Transpose of the x-pass output for the y pass: per z-slab, B[y][x'] ->
// A[x'][y], through a padded LDS tile so reads and writes are both coalesced.
template <typename T>
__global__ __launch_bounds__(256) void k_transpose(const PairDev *__restrict__ pairs, const int64_t *__restrict__ prefix,
                                                   int npairs, cplx<T> *__restrict__ ws, int64_t ws_stride)
{
    __shared__ cplx<T> tile[kTransposeTile][kTransposeTile + 1];
    ws += (int64_t)blockIdx.y * ws_stride;   // data row blockIdx.y
    const int p = (int)find_segment(prefix, npairs, blockIdx.x);
    const PairDev &P = pairs[p];
    const int64_t local = (int64_t)blockIdx.x - prefix[p];
    const int R = P.n1[1], C = P.wcount[0];
    const int tr = (R + kTransposeTile - 1) / kTransposeTile, tc = (C + kTransposeTile - 1) / kTransposeTile;
    const int64_t z = local / ((int64_t)tr * tc);
    const int rem = (int)(local - z * tr * tc);
    const int ti = rem / tc, tj = rem - ti * tc;
    const cplx<T> *in = ws + P.bufB + z * (int64_t)R * C;
    cplx<T> *out = ws + P.bufA + z * (int64_t)R * C;
    const int tx = threadIdx.x % kTransposeTile, ty = threadIdx.x / kTransposeTile;
    constexpr int rows_per_pass = 256 / kTransposeTile;
#pragma unroll
    for (int k = 0; k < kTransposeTile; k += rows_per_pass) {
        const int r = ti * kTransposeTile + ty + k, c = tj * kTransposeTile + tx;
        if (r < R && c < C) tile[ty + k][tx] = in[(int64_t)r * C + c];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTransposeTile; k += rows_per_pass) {
        const int c = tj * kTransposeTile + ty + k, r = ti * kTransposeTile + tx;
        if (r < R && c < C) out[(int64_t)c * R + r] = tile[tx][ty + k];
    }
}

// ---------------------------------------------------------------------------
// exp(2 pi i t) with t in revolutions, t reduced in float64 (phases of the
// interpolation epilogue and of the direct sum).
// ---------------------------------------------------------------------------
// exp(2 pi i t) for the float32 plan: fractional part in float64, then the
// hardware sine / cosine, whose argument is in revolutions.
__device__ __forceinline__ void cis_rev(double t, float &c, float &s)
{
    const float r = static_cast<float>(__builtin_amdgcn_fract(t));
    s = __builtin_amdgcn_sinf(r);
    c = __builtin_amdgcn_cosf(r);
}

// exp(2 pi i t) for the float64 plan: reduce t to the nearest quarter turn,
// t = q/4 + f with |f| <= 1/8, evaluate sin and cos of theta = 2 pi f by their
// Maclaurin series through theta^13 / theta^14 (truncation below 3e-14 on
// |theta| <= pi/4), then rotate by q quarter turns.
__device__ __forceinline__ void cis_rev(double t, double &c, double &s)
{
    const double q = rint(4.0 * t);
    const double f = fma(q, -0.25, t);
    const double th = 6.283185307179586476925287 * f;
    const double z = th * th;
    double ps = 1.0 / 6227020800.0;                 // 1/13!
    ps = fma(ps, -z, 1.0 / 39916800.0);             // 1/11!
    ps = fma(ps, -z, 1.0 / 362880.0);               // 1/9!
    ps = fma(ps, -z, 1.0 / 5040.0);                 // 1/7!
    ps = fma(ps, -z, 1.0 / 120.0);                  // 1/5!
    ps = fma(ps, -z, 1.0 / 6.0);                    // 1/3!
    const double sn = fma(-ps * z, th, th);
    double pc = 1.0 / 87178291200.0;                // 1/14!
    pc = fma(pc, -z, 1.0 / 479001600.0);            // 1/12!
    pc = fma(pc, -z, 1.0 / 3628800.0);              // 1/10!
    pc = fma(pc, -z, 1.0 / 40320.0);                // 1/8!
    pc = fma(pc, -z, 1.0 / 720.0);                  // 1/6!
    pc = fma(pc, -z, 1.0 / 24.0);                   // 1/4!
    pc = fma(pc, -z, 0.5);                          // 1/2!
    const double cs = fma(-pc, z, 1.0);
    const int k = static_cast<int>(q) & 3;
    const double s1 = (k & 1) ? cs : sn;
    const double c1 = (k & 1) ? sn : cs;
    s = (k & 2) ? -s1 : s1;
    c = (k == 1 || k == 2) ? -c1 : c1;
}

// exp(2 pi i t) in float64, t given in table steps (u = kCisTab t), from a
// table of exp(2 pi i k / kCisTab) (float64, filled on the host) and the Taylor
// terms of the remainder: with k = rint(u) and f = u - k in [-1/2, 1/2],
// exp(2 pi i t) = tab[k mod kCisTab] exp(i theta), theta = 2 pi f / kCisTab,
// |theta| <= pi / kCisTab; sin theta ~ theta - theta^3 / 6 and cos theta ~ 1 -
// theta^2 / 2 + theta^4 / 24 leave a truncation below theta^5 / 120 = 2.3e-15
// (kCisTab = 1024), the scale 2 pi / kCisTab folded into the coefficients.  k
// comes from one add of 1.5 2^52, which rounds u to an integer in
// round-to-nearest and leaves k + 2^51 in the low bits of the sum's mantissa
// (|u| < 2^51); the split u = k + f is exact.  Copies of a smaller table
// interleaved so that no two lanes meet on an LDS bank (256 entries, 16 copies,
// 64 KB, one more polynomial term) measured no faster with one data row and up
// to 18% slower with four (fewer wavefronts): bank conflicts do not bound the loop.
__device__ __forceinline__ void cis_tab(double u, const double2 *tab, double &c, double &s)
{
    static_assert((kCisTab & (kCisTab - 1)) == 0, "power-of-two table");
    constexpr double kRound = 6755399441055744.0;                 // 1.5 * 2^52
    constexpr double a1 = 6.283185307179586476925287 / kCisTab;   // theta = a1 f
    constexpr double a3 = -a1 * a1 * a1 / 6.0, b2 = -a1 * a1 / 2.0, b4 = a1 * a1 * a1 * a1 / 24.0;
    const double m = u + kRound;
    const double f = u - (m - kRound);                             // [-1/2, 1/2]
    const double2 e = tab[__double2loint(m) & (kCisTab - 1)];       // k + 2^51 = k mod kCisTab
    const double f2 = f * f;
    const double sn = f * fma(f2, a3, a1);
    const double cs = fma(f2, fma(f2, b4, b2), 1.0);
    c = fma(e.x, cs, -e.y * sn);
    s = fma(e.y, cs, e.x * sn);
}

// exp(2 pi i <a, b>) in float64: the products split exactly into a rounded
// part, reduced to a fraction of a turn, and its rounding error (no contraction:
// a fused p - rint(p) would count the error twice)
__device__ __forceinline__ void cis_dot(const double a[3], const double b[3], double &c, double &s)
{
#pragma clang fp contract(off)
    double f = 0.0, e = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double p = a[d] * b[d];
        e += fma(a[d], b[d], -p);
        f += p - rint(p);
    }
    cis_rev(f + e, c, s);
}

// ---------------------------------------------------------------------------
// interpolation + deconvolution + post-phase (type-3 steps 3-4):
//   f_k += exp(2 pi i iota s_k.x_c) / prod Psi_hat(.) * sum_m G_m prod_d ES((m_d - tau_kd) 2/w)
// A group of kInterpLanes lanes per target (four targets per wavefront,
// kInterpTargets targets of one sub-problem per workgroup);
// the lanes cover the (y, z) pairs of its w^3 window (z fastest, as the
// grid), loop over x, and reduce across the group.  Accumulation is float64
// (cross-sub-problem sums stay in double precision).  NR data rows share the
// kernel weights, addresses and post-phase of each target (row r reads the
// r-th copy of the batch workspace and adds into accumulator row r).
// ---------------------------------------------------------------------------
// two complex64 cells, aligned as one
typedef float F4 __attribute__((ext_vector_type(4), aligned(8)));

template <typename T, int NR>
__global__ __launch_bounds__(256) void k_interp(const PairDev *__restrict__ pairs, const int64_t *__restrict__ bprefix,
                                                int npairs, int64_t block0, const double *__restrict__ xyz,
                                                int64_t ntgt, const double *__restrict__ deconv,
                                                const cplx<T> *__restrict__ ws, int64_t ws_stride,
                                                double *__restrict__ acc, int64_t acc_stride, int w, T beta,
                                                double iota, int det)
{
    __shared__ T ker[kInterpTargets][3 * kWMax];
    const int sub = threadIdx.x & (kInterpLanes - 1), slot = threadIdx.x / kInterpLanes;
    const T two_over_w = T(2) / T(w);
    // every workgroup serves kInterpTargets consecutive targets of one sub-problem
    const int64_t blk = block0 + blockIdx.x;
    const int p = (int)find_segment(bprefix, npairs, blk);
    const PairDev &P = pairs[p];
    const int64_t local = (blk - bprefix[p]) * kInterpTargets + slot;
    const bool active = local < P.tgt_cnt;
    const int64_t k = P.tgt_off + (active ? local : 0);
    double s_k[3];
    int m0[3];
    for (int d = 0; d < 3; ++d) {
        s_k[d] = xyz[d * ntgt + k];
        const double tau = (s_k[d] - P.sc[d]) * P.tscale[d];
        m0[d] = (int)ceil(tau - 0.5 * w);
        for (int q = sub; q < w; q += kInterpLanes)
            ker[slot][d * w + q] = es_kernel(T((double)(m0[d] + q) - tau) * two_over_w, beta);
    }
    __syncthreads();
    T ar[NR], ai[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) ar[r] = ai[r] = T(0);
    if (active) {
        const int wx = P.wcount[0], wy = P.wcount[1], wz = P.wcount[2];
        const bool fx = wx == P.n2[0], fy = wy == P.n2[1], fz = wz == P.n2[2];   // whole (periodic) axis kept
        const int n2x = P.n2[0], n2y = P.n2[1], n2z = P.n2[2];
        const int sx = P.wstart[0], sy = P.wstart[1], sz = P.wstart[2];
        const cplx<T> *grid = ws + P.bufA;          // [wx][wy][wz], z fastest; row r at r * ws_stride
        const int xstride = wy * wz;
        // x cells eight at a time (the offsets and weights of a chunk shared by every
        // (y, z) row of the target and every data row); cells beyond the kernel support
        // or outside the kept window get weight 0 and the address of a cell the target
        // reads anyway (its last column, clamped into the window), so the loads carry
        // no branches and fetch no line the window does not need.  Each lane takes two
        // (y, z) rows per step, sixteen loads in flight per data row.
        auto column = [&](int e, T &kyz) -> const cplx<T> * {
            const int dy = e / w, dz = e - dy * w;
            int qy = m0[1] + dy - sy, qz = m0[2] + dz - sz;
            if (fy) { qy %= n2y; if (qy < 0) qy += n2y; }
            if (fz) { qz %= n2z; if (qz < 0) qz += n2z; }
            const bool ok = qy >= 0 && qy < wy && qz >= 0 && qz < wz;
            kyz = ok ? ker[slot][w + dy] * ker[slot][2 * w + dz] : T(0);
            return grid + (ok ? qy * wz + qz : 0);
        };
        // What bounds this gather is the number of loads and of the addresses worked out for
        // them, before the bytes: each lane waits for cells that its neighbours' lines mostly
        // hold already.  Float32 grids whose z axis is a window therefore read two neighbouring
        // z cells per 16-byte load (a 7 x 7 plane of columns takes 28 loads per x cell instead
        // of 49), with the same bytes in flight: four x cells of two pairs.  483 sub-problems
        // of a 3 km array, width 7: 7.8 ms -> 6.5 ms.  The last pair of an odd width starts one
        // cell early, with weight 0 on that cell; the window holds every target's whole
        // support, so no pair straddles its end.  A z axis kept whole may wrap between the two
        // cells, and a float64 cell is 16 bytes by itself: both read cell by cell below.
        bool pairs_done = false;
        if constexpr (sizeof(T) == 4) {
            if (!fz) {
                pairs_done = true;
                const int hw = (w + 1) / 2, ncol = w * hw;
                auto column2 = [&](int e, T &ka, T &kb) -> const cplx<T> * {
                    const int dy = e / hw, dz0 = 2 * (e - dy * hw), dz = min(dz0, w - 2);
                    int qy = m0[1] + dy - sy;
                    const int qz = m0[2] + dz - sz;
                    if (fy) { qy %= n2y; if (qy < 0) qy += n2y; }
                    const bool ok = qy >= 0 && qy < wy && qz >= 0 && qz + 1 < wz;
                    const T ky = ok ? ker[slot][w + dy] : T(0);
                    ka = dz == dz0 ? ky * ker[slot][2 * w + dz] : T(0);
                    kb = ky * ker[slot][2 * w + dz + 1];
                    return grid + (ok ? qy * wz + qz : 0);
                };
                for (int dx0 = 0; dx0 < w; dx0 += 4) {
                    int64_t xo[4];
                    T kx[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int dx = min(dx0 + u, w - 1);
                        int qx = m0[0] + dx - sx;
                        if (fx) { qx %= n2x; if (qx < 0) qx += n2x; }
                        const bool okx = dx0 + u < w && qx >= 0 && qx < wx;
                        kx[u] = okx ? ker[slot][dx] : T(0);
                        xo[u] = (int64_t)min(max(qx, 0), wx - 1) * xstride;
                    }
                    for (int e0 = sub; e0 < ncol; e0 += 2 * kInterpLanes) {
                        const int e1 = e0 + kInterpLanes;
                        const bool has1 = e1 < ncol;
                        T k0a, k0b, k1a, k1b;
                        const cplx<T> *col0 = column2(e0, k0a, k0b);
                        const cplx<T> *col1 = column2(has1 ? e1 : e0, k1a, k1b);   // no second: a repeat, weight 0
                        if (!has1) k1a = k1b = T(0);
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            const cplx<T> *c0 = col0 + r * ws_stride, *c1 = col1 + r * ws_stride;
                            F4 g0[4], g1[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                g0[u] = *reinterpret_cast<const F4 *>(c0 + xo[u]);
                                g1[u] = *reinterpret_cast<const F4 *>(c1 + xo[u]);
                            }
                            F4 s0 = {0, 0, 0, 0}, s1 = {0, 0, 0, 0};
#pragma unroll
                            for (int u = 0; u < 4; ++u)
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    s0[i] += g0[u][i] * kx[u];
                                    s1[i] += g1[u][i] * kx[u];
                                }
                            ar[r] += s0[0] * k0a + s0[2] * k0b + s1[0] * k1a + s1[2] * k1b;
                            ai[r] += s0[1] * k0a + s0[3] * k0b + s1[1] * k1a + s1[3] * k1b;
                        }
                    }
                }
            }
        }
        for (int dx0 = pairs_done ? w : 0; dx0 < w; dx0 += 8) {
            int64_t xo[8];
            T kx[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int dx = min(dx0 + u, w - 1);
                int qx = m0[0] + dx - sx;
                if (fx) { qx %= n2x; if (qx < 0) qx += n2x; }
                const bool okx = dx0 + u < w && qx >= 0 && qx < wx;
                kx[u] = okx ? ker[slot][dx] : T(0);
                xo[u] = (int64_t)min(max(qx, 0), wx - 1) * xstride;
            }
            for (int e0 = sub; e0 < w * w; e0 += 2 * kInterpLanes) {
                const int e1 = e0 + kInterpLanes;
                const bool has1 = e1 < w * w;
                T kyz0, kyz1;
                const cplx<T> *col0 = column(e0, kyz0);
                const cplx<T> *col1 = column(has1 ? e1 : e0, kyz1);   // no second row: a repeat, weight 0
                if (!has1) kyz1 = T(0);
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const cplx<T> *c0 = col0 + r * ws_stride, *c1 = col1 + r * ws_stride;
                    cplx<T> g0[8], g1[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        g0[u] = c0[xo[u]];
                        g1[u] = c1[xo[u]];
                    }
                    T s0r = T(0), s0i = T(0), s1r = T(0), s1i = T(0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        s0r += g0[u].x * kx[u];
                        s0i += g0[u].y * kx[u];
                        s1r += g1[u].x * kx[u];
                        s1i += g1[u].y * kx[u];
                    }
                    ar[r] += s0r * kyz0 + s1r * kyz1;
                    ai[r] += s0i * kyz0 + s1i * kyz1;
                }
            }
        }
    }
    // reduce over the target's lane group (xor offsets below the group size stay inside it)
#pragma unroll
    for (int r = 0; r < NR; ++r)
        for (int off = kInterpLanes / 2; off > 0; off >>= 1) {
            ar[r] += __shfl_xor(ar[r], off, 64);
            ai[r] += __shfl_xor(ai[r], off, 64);
        }
    if (active && sub == 0) {
        // post-phase exp(2 pi i iota s_k.x_c) in float64 in both precisions
        double ph = 0.0;
        for (int d = 0; d < 3; ++d) ph += s_k[d] * P.xc[d];
        double er, ei;
        cis_rev(iota * ph, er, ei);
        const double dk = deconv[k];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            double *a = acc + r * acc_stride;
            const double vr = (double)ar[r] * dk, vi = (double)ai[r] * dk;
            if (det) {
                // deterministic plans: no other workgroup of this launch adds into target k
                a[2 * k] += vr * er - vi * ei;
                a[2 * k + 1] += vr * ei + vi * er;
            } else {
                atomicAdd(a + 2 * k, vr * er - vi * ei);
                atomicAdd(a + 2 * k + 1, vr * ei + vi * er);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// direct evaluation of a sub-problem block (Sect. 3.1, last bullet; the
// eps = 0 mode of Sect. 4):  f_k += sum_n c_n exp(2 pi i iota s_k.x_n).
// A workgroup of 256 threads owns <= 512 targets (two per thread) and
// <= kDirectSeg sources, staged 256 at a time in LDS, for NT data rows at
// once (the phase factors are computed once and applied to every row).  Phases
// are float64 dot products (full rate on CDNA).  Float32 plans take them of the
// coordinates themselves, to 2^-32 turns or |t| 2^-53 for |t| turns (items of one or two
// sources: in float64 throughout).  Float64
// plans take them relative to the first source x_S of the staged tile and rotate
// the tile's sums by exp(2 pi i s_k.x_S), evaluated with exact products.  The
// sign iota multiplies the target coordinates, so the inner loop always
// accumulates c exp(+2 pi i t).
//
// What bounds it: VALU issue.  Per (target, source) the float32 loop issues three
// float64 FMAs (phase), a conversion and a scaling (fraction of a turn), sine and
// cosine, and per row four multiply-adds, two when every value of the staged tile is
// real (a real sky) or only the real part of the result is wanted: 11.1 instructions
// with one complex row, 9.1 with a real one.  Sine and cosine take two lane-cycles each
// and do not overlap with the rest; float32 multiply-adds on vector registers take 0.7 to
// 0.85.  A loop of the same instructions on registers alone takes 12.4 / 10.5 lane-cycles
// of the 2.4 GHz peak clock (five wavefronts per SIMD; four rows, at three, 23.1 / 15.9),
// and this one 12.4 / 10.6 (22.5 / 16.1): staging and LDS reads are hidden.  Matrix instructions for the
// multiply-adds (v_mfma_f32_4x4x1) do not overlap with the vector work and
// measured 15.1 lane-cycles a term against 12.0.  The float64 loop issues 21.25
// instructions (19.25 with real values), which take 22.5 (20.3) lane-cycles on registers
// alone, and takes 25.2 (22.9).  247,500 x 250,000, 10^12 term-rows/s, real / complex values, before
// (references per target and source tile, float64 fraction, one path for
// both kinds of values) and now:
//   float32, 1 row 3.00 -> 3.70 / 3.18, 4 rows 7.16 -> 9.8 / 7.0;
//   float64, 1 row 1.50 -> 1.71 / 1.56, 4 rows 3.64 -> 4.9 / 3.8.
// ---------------------------------------------------------------------------

// multiply-adds of a term: complex, real values only, real part of the result only
enum DirectMode { kDirectComplex, kDirectRealIn, kDirectRealOut };

// Float32 phase t + kPhaseMagic, accumulated as such by the FMAs: the sum of
// 1.5 2^20 keeps every |t| < 2^19 turns (the planner's kMaxMagicTurns bounds them
// with room) in one binade whose last bit is 2^-32 turns, so the
// low word of the double is the fraction of a turn in 32 bits.  Read as a signed
// integer, converted and scaled it is a float in [-1/2, 1/2] (an error of at most
// 2^-26 turns, less near zero), which the hardware sine and cosine take in
// revolutions.  A float64 fraction and its conversion hold a phase no better
// (2^-25 turns, [0, 1)) and take longer: 3.08e12 against 3.17e12 complex terms/s.
// One funnel shift of the upper 23 bits into the mantissa of a float in [1, 2) is
// faster (3.35e12), but its 2^-24 turns at every phase, zero included, are the larger part of a
// term's error: 3 points seen by 3,000, 2.2e-7 against 7.3e-8 (relative l2).
constexpr double kPhaseMagic = 1572864.0;

// The hardware cosine of a phase in [-1/2, 1/2] averages -5.0e-10 over a turn, not zero (in
// [0, 1): 3.7e-10, and the sine 4.1e-10): nothing to a term, but a sky of positive intensities
// adds it up in phase (1M points: an error of 4.2e-7 of the result, 1.5e-7 without).
// So every second source is taken half a turn further and its value negated: the averages of
// neighbours cancel.  Both halves cost nothing in the loop (the constant that
// the phase is summed onto, and the sign at the staging).
__device__ __forceinline__ double direct_half_turn(int j) { return j & 1 ? 0.5 : 0.0; }
template <typename T> __device__ __forceinline__ cplx<T> direct_value(cplx<T> c, int j)
{
    return sizeof(T) == 4 && (j & 1) ? mk<T>(-c.x, -c.y) : c;
}

// exp(2 pi i (t + half)) of the phase t = q.x for one (target, source): float32 plans
template <bool WIDE>
__device__ __forceinline__ void direct_cis(const double q[3], double x, double y, double z, double half, const double2 *,
                                           float &c, float &s)
{
    float r;
    if constexpr (WIDE) {   // phases beyond the magic range: float64 fraction
        r = static_cast<float>(__builtin_amdgcn_fract(fma(q[0], x, fma(q[1], y, fma(q[2], z, half)))));
    } else {
        const double m = fma(q[0], x, fma(q[1], y, fma(q[2], z, kPhaseMagic + half)));
        r = static_cast<float>(__double2loint(m)) * 0x1p-32f;   // [-1/2, 1/2] turns
    }
    s = __builtin_amdgcn_sinf(r);
    c = __builtin_amdgcn_cosf(r);
}
// float64 plans: the LDS phase table (q holds the target in table steps)
template <bool WIDE>
__device__ __forceinline__ void direct_cis(const double q[3], double x, double y, double z, double, const double2 *tab,
                                           double &c, double &s)
{
    cis_tab(fma(q[0], x, fma(q[1], y, q[2] * z)), tab, c, s);
}

// sources [jb, je) of the staged tile (a multiple of four) into the float64
// sums of the thread's two targets; partial sums of kRun terms in the plan's
// precision (64 in float32: the rounding of the running sum grows with its
// length, and a run of 64 instead of 256 costs 0.06 instructions a term)
template <typename T, int NT, bool WIDE, int MODE>
__device__ __forceinline__ void direct_tile(int jb, int je, const double q0[3], const double q1[3], const double *lx,
                                            const double *ly, const double *lz,
                                            const cplx<T> (*lc)[kDirectSrcTile], const double2 *ltab,
                                            double a0r[NT], double a0i[NT], double a1r[NT], double a1i[NT])
{
    constexpr int kRun = sizeof(T) == 4 ? 64 : kDirectSrcTile;
    for (int j0 = jb; j0 < je; j0 += kRun) {
        const int j1 = min(j0 + kRun, je);
        T b0r[NT], b0i[NT], b1r[NT], b1i[NT];
#pragma unroll
        for (int r = 0; r < NT; ++r) {   // float64: straight into the caller's sums
            b0r[r] = sizeof(T) == 4 ? T(0) : T(a0r[r]);
            b0i[r] = sizeof(T) == 4 ? T(0) : T(a0i[r]);
            b1r[r] = sizeof(T) == 4 ? T(0) : T(a1r[r]);
            b1i[r] = sizeof(T) == 4 ? T(0) : T(a1i[r]);
        }
        for (int j = j0; j < j1; j += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double x = lx[j + u], y = ly[j + u], z = lz[j + u];
                T c0, s0, c1, s1;
                direct_cis<WIDE>(q0, x, y, z, direct_half_turn(u), ltab, c0, s0);
                direct_cis<WIDE>(q1, x, y, z, direct_half_turn(u), ltab, c1, s1);
                // one phase factor per (target, source), applied to every row
#pragma unroll
                for (int r = 0; r < NT; ++r) {
                    const cplx<T> c = lc[r][j + u];
                    if constexpr (MODE == kDirectRealIn) {
                        b0r[r] = fma(c.x, c0, b0r[r]);
                        b0i[r] = fma(c.x, s0, b0i[r]);
                        b1r[r] = fma(c.x, c1, b1r[r]);
                        b1i[r] = fma(c.x, s1, b1i[r]);
                    } else {
                        b0r[r] = fma(c.x, c0, fma(-c.y, s0, b0r[r]));
                        b1r[r] = fma(c.x, c1, fma(-c.y, s1, b1r[r]));
                        if constexpr (MODE == kDirectComplex) {
                            b0i[r] = fma(c.x, s0, fma(c.y, c0, b0i[r]));
                            b1i[r] = fma(c.x, s1, fma(c.y, c1, b1i[r]));
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            a0r[r] = sizeof(T) == 4 ? a0r[r] + (double)b0r[r] : (double)b0r[r];
            a1r[r] = sizeof(T) == 4 ? a1r[r] + (double)b1r[r] : (double)b1r[r];
            if constexpr (MODE != kDirectRealOut) {
                a0i[r] = sizeof(T) == 4 ? a0i[r] + (double)b0i[r] : (double)b0i[r];
                a1i[r] = sizeof(T) == 4 ? a1i[r] + (double)b1i[r] : (double)b1i[r];
            }
        }
    }
}

template <typename T, int NT, int TILE, bool WIDE>
__device__ __forceinline__ void direct_item(const DirectItem it, const double *__restrict__ sxyz, int64_t nsrc,
                                            const double *__restrict__ txyz, int64_t ntgt,
                                            const int32_t *__restrict__ perm, const cplx<T> *__restrict__ in,
                                            int64_t in_stride, double *__restrict__ acc, int64_t acc_stride,
                                            double iota, int store, int layer0, int layers, int real_out,
                                            double (*lxyz)[kDirectSrcTile], cplx<T> (*lc)[kDirectSrcTile],
                                            const double2 *ltab)
{
    // TILE / 2 threads hold the targets; SL such slices divide the staged sources
    constexpr int kHalf = TILE / 2, SL = kDirectThreads / kHalf;
    static_assert(kHalf % 64 == 0 && SL * kHalf == kDirectThreads, "a wavefront lies in one slice");
    const int tid = threadIdx.x, tl = SL == 1 ? tid : tid & (kHalf - 1);
    const int slice = SL == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / kHalf);
    double *lx = lxyz[0], *ly = lxyz[1], *lz = lxyz[2];
    // two targets per thread: each staged source is read from LDS once for both
    const bool has0 = tl < it.tgt_cnt, has1 = tl + kHalf < it.tgt_cnt;
    const int64_t k0 = it.tgt_off + (has0 ? tl : 0);
    const int64_t k1 = it.tgt_off + (has1 ? tl + kHalf : 0);
    constexpr bool kRef = sizeof(T) == 8;   // phases relative to the staged tile's first source
    const double unit = kRef ? iota * kCisTab : iota;   // the sign enters through the phase
    double q0[3], q1[3];
    for (int d = 0; d < 3; ++d) {
        q0[d] = unit * txyz[d * ntgt + k0];
        q1[d] = unit * txyz[d * ntgt + k1];
    }
    double a0r[NT], a0i[NT], a1r[NT], a1i[NT];
#pragma unroll
    for (int r = 0; r < NT; ++r) a0r[r] = a0i[r] = a1r[r] = a1i[r] = 0.0;
    for (int s0 = 0; s0 < it.src_cnt; s0 += kDirectSrcTile) {
        const int cnt = min(kDirectSrcTile, it.src_cnt - s0);
        const int64_t nS = it.src_off + s0;
        double ref[3] = {0.0, 0.0, 0.0};
        if constexpr (kRef)
            for (int d = 0; d < 3; ++d) ref[d] = sxyz[d * nsrc + nS];
        __syncthreads();
        bool im = false;   // a staged value has an imaginary part (NaN included)
        {
            // entries beyond the last source hold zeros: the loop runs in fours
            const bool live = tid < cnt;
            const int64_t n = nS + (live ? tid : 0);
            lx[tid] = live ? sxyz[n] - ref[0] : 0.0;
            ly[tid] = live ? sxyz[nsrc + n] - ref[1] : 0.0;
            lz[tid] = live ? sxyz[2 * nsrc + n] - ref[2] : 0.0;
            const int64_t u = perm ? perm[n] : n;
#pragma unroll
            for (int r = 0; r < NT; ++r) {
                const cplx<T> c = live ? in[r * in_stride + u] : mk<T>(T(0), T(0));
                lc[r][tid] = direct_value<T>(c, tid);
                im |= !(c.y == T(0));
            }
        }
        const bool cplx_in = __syncthreads_or(im);
        const int c4 = (cnt + 3) & ~3, per = (c4 / 4 + SL - 1) / SL * 4;   // this slice's share
        const int jb = SL == 1 ? 0 : min(slice * per, c4), je = SL == 1 ? c4 : min(jb + per, c4);
        if constexpr (!kRef) {
            // one or two sources: their phases are the whole result, and hold float64
            if (it.src_cnt <= kDirectExactSrc) {
                for (int j = jb; j < min(je, cnt); ++j) {
                    const double x[3] = {lx[j], ly[j], lz[j]};
                    double c0, s0, c1, s1;
                    cis_dot(q0, x, c0, s0);
                    cis_dot(q1, x, c1, s1);
#pragma unroll
                    for (int r = 0; r < NT; ++r) {
                        const cplx<T> v = direct_value<T>(lc[r][j], j);   // (the value as it was)
                        const double cr = v.x, ci = v.y;
                        a0r[r] = fma(cr, c0, fma(-ci, s0, a0r[r]));
                        a0i[r] = fma(cr, s0, fma(ci, c0, a0i[r]));
                        a1r[r] = fma(cr, c1, fma(-ci, s1, a1r[r]));
                        a1i[r] = fma(cr, s1, fma(ci, c1, a1i[r]));
                    }
                }
            } else if (real_out)
                direct_tile<T, NT, WIDE, kDirectRealOut>(jb, je, q0, q1, lx, ly, lz, lc, ltab, a0r, a0i, a1r, a1i);
            else if (cplx_in)
                direct_tile<T, NT, WIDE, kDirectComplex>(jb, je, q0, q1, lx, ly, lz, lc, ltab, a0r, a0i, a1r, a1i);
            else direct_tile<T, NT, WIDE, kDirectRealIn>(jb, je, q0, q1, lx, ly, lz, lc, ltab, a0r, a0i, a1r, a1i);
        } else {
            double b0r[NT], b0i[NT], b1r[NT], b1i[NT];
#pragma unroll
            for (int r = 0; r < NT; ++r) b0r[r] = b0i[r] = b1r[r] = b1i[r] = 0.0;
            if (cplx_in)
                direct_tile<T, NT, WIDE, kDirectComplex>(jb, je, q0, q1, lx, ly, lz, lc, ltab, b0r, b0i, b1r, b1i);
            else direct_tile<T, NT, WIDE, kDirectRealIn>(jb, je, q0, q1, lx, ly, lz, lc, ltab, b0r, b0i, b1r, b1i);
            // tile reference phases (q / kCisTab is exact)
            double p0[3], p1[3], e0c, e0s, e1c, e1s;
            for (int d = 0; d < 3; ++d) {
                p0[d] = q0[d] * (1.0 / kCisTab);
                p1[d] = q1[d] * (1.0 / kCisTab);
            }
            cis_dot(p0, ref, e0c, e0s);
            cis_dot(p1, ref, e1c, e1s);
            // (fused by hand: left to the compiler, which product takes the fused form differs
            // between the instances for one row and for several, and with it a row's last bits)
#pragma unroll
            for (int r = 0; r < NT; ++r) {
#pragma clang fp contract(off)
                a0r[r] += fma(b0r[r], e0c, -b0i[r] * e0s);
                a0i[r] += fma(b0r[r], e0s, b0i[r] * e0c);
                a1r[r] += fma(b1r[r], e1c, -b1i[r] * e1s);
                a1i[r] += fma(b1r[r], e1s, b1i[r] * e1c);
            }
        }
    }
    // add the slices, halving their number: the upper half hands its sums over
    if constexpr (SL > 1) {
        double2 *red = reinterpret_cast<double2 *>(lxyz);
        static_assert(sizeof(double2) * (SL / 2) * TILE <= 3 * sizeof(double) * kDirectSrcTile, "the sums fit the stage");
#pragma unroll
        for (int r = 0; r < NT; ++r) {
#pragma unroll
            for (int h = SL / 2; h > 0; h /= 2) {
                __syncthreads();
                if (slice >= h && slice < 2 * h) {
                    red[(slice - h) * TILE + tl] = make_double2(a0r[r], a0i[r]);
                    red[(slice - h) * TILE + kHalf + tl] = make_double2(a1r[r], a1i[r]);
                }
                __syncthreads();
                if (slice < h) {
                    const double2 v0 = red[slice * TILE + tl], v1 = red[slice * TILE + kHalf + tl];
                    a0r[r] += v0.x;
                    a0i[r] += v0.y;
                    a1r[r] += v1.x;
                    a1i[r] += v1.y;
                }
            }
        }
        if (slice > 0) return;
    }
#pragma unroll
    for (int r = 0; r < NT; ++r) {
        double *ar = acc + r * acc_stride;
        if (store == kDirectSlab) {
            // the sums of this layer, added up afterwards (acc: the slabs)
            double2 *sl = reinterpret_cast<double2 *>(acc) + ((int64_t)r * layers + (it.layer - layer0)) * ntgt;
            if (has0) sl[k0] = make_double2(a0r[r], a0i[r]);
            if (has1) sl[k1] = make_double2(a1r[r], a1i[r]);
        } else if (store == kDirectAdd) {
            // items of one layer: no other workgroup of this launch adds to these targets
            if (has0) { ar[2 * k0] += a0r[r]; ar[2 * k0 + 1] += a0i[r]; }
            if (has1) { ar[2 * k1] += a1r[r]; ar[2 * k1 + 1] += a1i[r]; }
        } else {
            if (has0) {
                atomicAdd(ar + 2 * k0, a0r[r]);
                atomicAdd(ar + 2 * k0 + 1, a0i[r]);
            }
            if (has1) {
                atomicAdd(ar + 2 * k1, a1r[r]);
                atomicAdd(ar + 2 * k1 + 1, a1i[r]);
            }
        }
    }
}

// One workgroup per work item, or (persistent launches) workgroups that take
// items from a queue until it is empty: a capped grid leaves room on every CU
// for the kernels of the NUFFT sub-problems running beside the direct sum on
// another stream, and workgroups of CUs that those kernels slow down take fewer items (a
// fixed share per workgroup cost 5% with 8 workgroups per CU and 9% with 5, even with the GPU
// to itself).  Items stay source-segment-major across consecutive workgroups either way.
template <typename T, int NT, int TILE, bool WIDE>
__global__ __launch_bounds__(kDirectThreads) void k_direct(const DirectItem *__restrict__ items, int64_t nitems,
                                                           const double *__restrict__ sxyz, int64_t nsrc,
                                                           const double *__restrict__ txyz, int64_t ntgt,
                                                           const int32_t *__restrict__ perm,
                                                           const cplx<T> *__restrict__ in, int64_t in_stride,
                                                           double *__restrict__ acc, int64_t acc_stride, double iota,
                                                           int store, int layer0, int layers, int real_out,
                                                           const double2 *__restrict__ ctab,
                                                           unsigned long long *__restrict__ queue)
{
    static_assert(kDirectSrcTile == kDirectThreads && kDirectTile == 2 * kDirectThreads, "direct tiling");
    static_assert(kDirectSrcTile % 4 == 0, "the staged tile is walked in fours");
    __shared__ __align__(16) double lxyz[3][kDirectSrcTile];
    __shared__ __align__(16) cplx<T> lc[NT][kDirectSrcTile];
    __shared__ double2 ltab[sizeof(T) == 8 ? kCisTab : 1];   // float64 plans: the phase table
    if constexpr (sizeof(T) == 8) {
        for (int i = threadIdx.x; i < kCisTab; i += kDirectThreads) ltab[i] = ctab[i];
        // the first item's staging barrier orders these writes before any read
    }
    auto item = [&](int64_t w) {   // (starts with a barrier)
        direct_item<T, NT, TILE, WIDE>(items[w], sxyz, nsrc, txyz, ntgt, perm, in, in_stride, acc, acc_stride, iota,
                                       store, layer0, layers, real_out, lxyz, lc, ltab);
    };
    if (!queue) {
        if (blockIdx.x < nitems) item(blockIdx.x);
        return;
    }
    __shared__ int64_t next;
    for (;;) {
        if (threadIdx.x == 0) next = static_cast<int64_t>(atomicAdd(queue, 1ull));
        __syncthreads();
        const int64_t w = next;
        if (w >= nitems) return;   // every workgroup draws past the last item once
        item(w);
        __syncthreads();           // `next` is read, the staged sources are free
    }
}

// ---------------------------------------------------------------------------
// v plus a target's m stored layers (slab[l * n]), one after another: the sum of
// deterministic plans, the same for any split of the layers over launches and
// lanes, and as in-place items add it.  The G = 1 << lg lanes of a target load G
// layers at a time, the next G on the way while each adds them all in order, so
// that few targets with many layers do not wait for memory at every eighth addition
// (1 target, 1,954 layers: 101 us by one lane, 24 so; exchanged by shuffles 113).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 add_in_order(double2 v, const double2 *__restrict__ slab, int64_t n, int m, int lg,
                                                double2 *stage)
{
    if (lg == 0) {
#pragma unroll 8
        for (int l = 0; l < m; ++l) {
            const double2 s = slab[l * n];
            v.x += s.x;
            v.y += s.y;
        }
        return v;
    }
    // (a target's lanes lie in one wavefront, whose LDS accesses keep their order; m is one value for them)
    const int G = 1 << lg, g = threadIdx.x & (G - 1);
    double2 *mine = stage + threadIdx.x, *all = mine - g;
    double2 next = g < m ? slab[g * n] : make_double2(0.0, 0.0);
    for (int l0 = 0; l0 < m; l0 += G) {
        *mine = next;
        if (l0 + G + g < m) next = slab[(l0 + G + g) * n];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int cnt = min(G, m - l0);
#pragma unroll 16
        for (int i = 0; i < cnt; ++i) {
            v.x += all[i].x;
            v.y += all[i].y;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    return v;
}

// ---------------------------------------------------------------------------
// sums that direct items stored by layer: the accumulator takes layers
// [layer0, layer0 + layers) of every target in order (tgt_layers: layers of a
// target in all), after what it holds or (fresh) from zero.  Grid y: data rows.
// ---------------------------------------------------------------------------
__global__ void k_add_layers(double2 *__restrict__ acc, int64_t n, const double2 *__restrict__ slab, int layer0,
                             int layers, const int32_t *__restrict__ tgt_layers, int fresh, int lg)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, k = t >> lg;
    if (k >= n) return;   // (whole groups of lanes)
    acc += blockIdx.y * n;
    slab += (int64_t)blockIdx.y * layers * n;
    __shared__ double2 stage[256];
    const double2 v = add_in_order(fresh ? make_double2(0.0, 0.0) : acc[k], slab + k, n,
                                   min(layers, tgt_layers[k] - layer0), lg, stage);
    if ((t & ((1 << lg) - 1)) == 0) acc[k] = v;
}

// ---------------------------------------------------------------------------
// epilogue: cast the float64 sums to the plan's precision and scatter to user
// order (the inverse of the chunk-order gather, Sect. 4 Fig. 5).  The sums are
// the accumulator (if any) and the last stored layers (if any); G = 1 << lg lanes share
// a target's layers, each every G-th of them, so that few targets with many
// layers still fill the GPU; deterministic plans add them in order.  Grid y: data rows.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_finalize(const double2 *__restrict__ acc, int64_t n, const int32_t *__restrict__ perm,
                           cplx<T> *__restrict__ out, int real_only, const double2 *__restrict__ slab, int layer0,
                           int layers, const int32_t *__restrict__ tgt_layers, int det, int lg)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, k = t >> lg;
    const int g = (int)(t & ((1 << lg) - 1));
    if (k >= n) return;   // (whole groups)
    __shared__ double2 stage[256];
    double2 v = acc && (det || g == 0) ? acc[blockIdx.y * n + k] : make_double2(0.0, 0.0);
    if (slab && det) {
        v = add_in_order(v, slab + (int64_t)blockIdx.y * layers * n + k, n, min(layers, tgt_layers[k] - layer0), lg,
                         stage);
    } else if (slab) {
        slab += (int64_t)blockIdx.y * layers * n + k;
        const int m = min(layers, tgt_layers[k] - layer0);
        for (int l = g; l < m; l += 1 << lg) {
            const double2 s = slab[l * n];
            v.x += s.x;
            v.y += s.y;
        }
        for (int off = 1 << lg >> 1; off > 0; off >>= 1) {
            v.x += __shfl_xor(v.x, off, 64);
            v.y += __shfl_xor(v.y, off, 64);
        }
    }
    if (g == 0) out[blockIdx.y * n + (perm ? perm[k] : k)] = mk<T>(T(v.x), real_only ? T(0) : T(v.y));
}

// ---------------------------------------------------------------------------
// direction-dependent gains in separable form A_k(r_n) = sum_t a[t][k] b[t][n]:
// the rows a transform takes (scale) and the sum of the transformed rows
// (combine).  out[t][i] = w'[t][i] x[i] and out[i] = sum_t w'[t][i] y[t][i],
// w' = w or conj(w); the combination accumulates in float64.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_dde_scale(const cplx<T> *__restrict__ w, const cplx<T> *__restrict__ x, cplx<T> *__restrict__ out,
                            int64_t n, int terms, int conj_w)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const cplx<T> v = x[i];
    for (int t = 0; t < terms; ++t) {
        cplx<T> g = w[(int64_t)t * n + i];
        if (conj_w) g.y = -g.y;
        out[(int64_t)t * n + i] = cmul<T>(g, v);
    }
}

template <typename T>
__global__ void k_dde_combine(const cplx<T> *__restrict__ w, const cplx<T> *__restrict__ y, cplx<T> *__restrict__ out,
                              int64_t n, int terms, int conj_w, int real_only)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double re = 0.0, im = 0.0;
    for (int t = 0; t < terms; ++t) {
        const cplx<T> g = w[(int64_t)t * n + i], v = y[(int64_t)t * n + i];
        const double gi = conj_w ? -(double)g.y : (double)g.y;
        re += (double)g.x * v.x - gi * v.y;
        im += (double)g.x * v.y + gi * v.x;
    }
    out[i] = mk<T>(T(re), real_only ? T(0) : T(im));
}

// ---------------------------------------------------------------------------
// launch wrappers (host)
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(int64_t n, int per, int64_t cap)
{
    int64_t b = (n + per - 1) / per;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return static_cast<unsigned>(b);
}

hipError_t launch_zero(double *p, int64_t n, void *queue, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(n, 256 * 8, 65536)), dim3(256), 0, st, p, n,
                       static_cast<unsigned long long *>(queue));
    return hipGetLastError();
}

hipError_t launch_deconv(const double *xyz, int64_t n, const int32_t *chunk_of, const double *ctr,
                         const double *hscale, const double *zq, const double *aq, int nq, int w, double *out,
                         hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_deconv, dim3(blocks_for(n, 256, INT32_MAX)), dim3(256), 0, st, xyz, n, chunk_of, ctr,
                       hscale, zq, aq, nq, w, out);
    return hipGetLastError();
}

hipError_t launch_bin(const PairDev *pairs, const int64_t *prefix, int npairs, int64_t total, const double *xyz,
                      int64_t nsrc, int w, int32_t *counts, unsigned long long *cursor, int32_t *records,
                      hipStream_t st)
{
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_bin_points, dim3(blocks_for(total, 256, INT32_MAX)), dim3(256), 0, st, pairs, prefix, npairs,
                       total, xyz, nsrc, w, counts, cursor, records);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_prephase(const PairDev *pairs, const int64_t *pprefix, int npairs, int64_t total, const double *xyz,
                           int64_t nsrc, const int32_t *perm, const void *in, int64_t in_stride, int rows, void *stage,
                           void *xval, int64_t xstride, double iota, int w, hipStream_t st)
{
    if (total <= 0) return hipSuccess;
    if (rows < 1 || rows > kRowBatch) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_prephase<T>, dim3(blocks_for(total, 256, INT32_MAX)), dim3(256), 0, st, pairs, pprefix,
                       npairs, total, xyz, nsrc, perm, static_cast<const cplx<T> *>(in), in_stride, rows,
                       static_cast<StagedSrc<T> *>(stage), static_cast<cplx<T> *>(xval), xstride, iota, w);
    return hipGetLastError();
}

template <typename T, int NR>
static void spread_rows(const PairDev *pairs, const SpreadTile *tiles, int64_t ntiles, const int32_t *records,
                        const void *stage, const void *xval, int64_t xstride, void *ws, int64_t ws_stride,
                        const void *precor, int w, double beta, hipStream_t st)
{
    hipLaunchKernelGGL((k_spread<T, NR>), dim3(static_cast<unsigned>(ntiles)), dim3(256), 0, st, pairs, tiles, records,
                       static_cast<const StagedSrc<T> *>(stage), static_cast<const cplx<T> *>(xval), xstride,
                       static_cast<cplx<T> *>(ws), ws_stride, static_cast<const T *>(precor), w, T(beta), T(2.0 / w),
                       1.0f / static_cast<float>(2 * w + kTileZ));
}

template <typename T>
hipError_t launch_spread(const PairDev *pairs, const SpreadTile *tiles, int64_t ntiles, const int32_t *records,
                         const void *stage, const void *xval, int64_t xstride, int rows, void *ws, int64_t ws_stride,
                         const void *precor, int w, double beta, hipStream_t st)
{
    if (ntiles <= 0) return hipSuccess;
    switch (rows) {
    case 1: spread_rows<T, 1>(pairs, tiles, ntiles, records, stage, xval, xstride, ws, ws_stride, precor, w, beta, st); break;
    case 2: spread_rows<T, 2>(pairs, tiles, ntiles, records, stage, xval, xstride, ws, ws_stride, precor, w, beta, st); break;
    case 3: spread_rows<T, 3>(pairs, tiles, ntiles, records, stage, xval, xstride, ws, ws_stride, precor, w, beta, st); break;
    case 4: spread_rows<T, 4>(pairs, tiles, ntiles, records, stage, xval, xstride, ws, ws_stride, precor, w, beta, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_fft(const PairDev *pairs, const int64_t *prefix, int npairs, int64_t tiles, int pass, void *ws,
                      const void *tw, const uint32_t *occ, int lds_elems, int max_len, double sign, int rows,
                      int64_t ws_stride, hipStream_t st)
{
    if (tiles <= 0) return hipSuccess;
    if (rows < 1 || rows > kRowBatch) return hipErrorInvalidValue;
    // dynamic LDS: the lines of one workgroup, then the twiddle table of the longest line
    size_t lds = static_cast<size_t>(lds_elems + max_len) * sizeof(cplx<T>);
    const dim3 grid(static_cast<unsigned>(tiles), static_cast<unsigned>(rows));
    // workgroup size from the longest line of the batch (lines up to kFftSmallLen: 256 threads)
    const int threads = fft_threads(max_len);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, st, pairs, prefix, npairs, pass, static_cast<cplx<T> *>(ws),
                           static_cast<const cplx<T> *>(tw), occ, lds_elems, T(sign), ws_stride);
        return hipGetLastError();
    };
    return threads == kFftThreadsSmall ? go(k_fft_pass<T, kFftThreadsSmall>) : go(k_fft_pass<T, kFftThreads>);
}

template <typename T>
hipError_t launch_fft_two(const PairDev *pairs, const int64_t *prefix, int npairs, int64_t tiles, int pass, void *ws,
                          const void *tw, const uint32_t *occ, int lds_elems, int threads, double sign, int rows,
                          int64_t ws_stride, hipStream_t st)
{
    if (tiles <= 0) return hipSuccess;
    if (rows < 1 || rows > kRowBatch || pass < 0 || pass > 1 || threads < 64 || threads > kFft2Threads)
        return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(tiles), static_cast<unsigned>(rows));
    const size_t lds = sizeof(cplx<T>) * static_cast<size_t>(lds_elems);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, st, pairs, prefix, npairs, static_cast<cplx<T> *>(ws),
                           static_cast<const cplx<T> *>(tw), occ, ws_stride);
        return hipGetLastError();
    };
    if (pass == 0) return sign < 0.0 ? go(k_fft_two<T, 0, -1>) : go(k_fft_two<T, 0, 1>);
    return sign < 0.0 ? go(k_fft_two<T, 1, -1>) : go(k_fft_two<T, 1, 1>);
}

template <typename T>
hipError_t launch_transpose(const PairDev *pairs, const int64_t *prefix, int npairs, int64_t tiles, void *ws,
                            int rows, int64_t ws_stride, hipStream_t st)
{
    if (tiles <= 0) return hipSuccess;
    if (rows < 1 || rows > kRowBatch) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_transpose<T>, dim3(static_cast<unsigned>(tiles), static_cast<unsigned>(rows)), dim3(256), 0,
                       st, pairs, prefix, npairs, static_cast<cplx<T> *>(ws), ws_stride);
    return hipGetLastError();
}

template <typename T, int NR>
static hipError_t interp_rows(const PairDev *pairs, const int64_t *bprefix, int npairs, int64_t blocks,
                              const double *xyz, int64_t ntgt, const double *deconv, const void *ws,
                              int64_t ws_stride, double *acc, int64_t acc_stride, int w, double beta, double iota,
                              int det, hipStream_t st)
{
    for (int64_t b0 = 0; b0 < blocks; b0 += kMaxLaunchBlocks) {
        const int64_t nb = std::min<int64_t>(kMaxLaunchBlocks, blocks - b0);
        hipLaunchKernelGGL((k_interp<T, NR>), dim3(static_cast<unsigned>(nb)), dim3(256), 0, st, pairs, bprefix,
                           npairs, b0, xyz, ntgt, deconv, static_cast<const cplx<T> *>(ws), ws_stride, acc,
                           acc_stride, w, T(beta), iota, det);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T>
hipError_t launch_interp(const PairDev *pairs, const int64_t *bprefix, int npairs, int64_t blocks, const double *xyz,
                         int64_t ntgt, const double *deconv, const void *ws, int64_t ws_stride, double *acc,
                         int64_t acc_stride, int rows, int w, double beta, double iota, int det, hipStream_t st)
{
    if (blocks <= 0) return hipSuccess;
    switch (rows) {
    case 1: return interp_rows<T, 1>(pairs, bprefix, npairs, blocks, xyz, ntgt, deconv, ws, ws_stride, acc,
                                     acc_stride, w, beta, iota, det, st);
    case 2: return interp_rows<T, 2>(pairs, bprefix, npairs, blocks, xyz, ntgt, deconv, ws, ws_stride, acc,
                                     acc_stride, w, beta, iota, det, st);
    case 3: return interp_rows<T, 3>(pairs, bprefix, npairs, blocks, xyz, ntgt, deconv, ws, ws_stride, acc,
                                     acc_stride, w, beta, iota, det, st);
    case 4: return interp_rows<T, 4>(pairs, bprefix, npairs, blocks, xyz, ntgt, deconv, ws, ws_stride, acc,
                                     acc_stride, w, beta, iota, det, st);
    default: return hipErrorInvalidValue;
    }
}

// arguments of a direct-sum launch
template <typename T, int NT, int TILE, bool WIDE>
static hipError_t direct_grid(const DirectLaunch &d, hipStream_t st)
{
    if (d.nitems > kMaxLaunchBlocks * (int64_t(1) << 20)) return hipErrorInvalidValue;
    auto go = [&](const DirectItem *items, int64_t n, int64_t grid) {
        hipLaunchKernelGGL((k_direct<T, NT, TILE, WIDE>), dim3(static_cast<unsigned>(grid)), dim3(kDirectThreads), 0, st,
                           items, n, d.sxyz, d.nsrc, d.txyz, d.ntgt, d.perm, static_cast<const cplx<T> *>(d.in), d.nsrc,
                           d.acc, 2 * d.ntgt, d.iota, d.store, d.layer0, d.layers, d.real_out,
                           static_cast<const double2 *>(d.ctab),
                           static_cast<unsigned long long *>(d.grid_cap > 0 ? d.queue : nullptr));
        return hipGetLastError();
    };
    // persistent: at most grid_cap workgroups taking items from the queue
    if (d.grid_cap > 0 && d.queue == nullptr) return hipErrorInvalidValue;
    if (d.grid_cap > 0)
        return go(d.items, d.nitems, std::min<int64_t>(std::min<int64_t>(d.grid_cap, d.nitems), kMaxLaunchBlocks));
    // one workgroup per item, in launches of at most kMaxLaunchBlocks workgroups
    // (a dispatch counts its work-items in 32 bits)
    for (int64_t i0 = 0; i0 < d.nitems; i0 += kMaxLaunchBlocks) {
        const int64_t nb = std::min<int64_t>(kMaxLaunchBlocks, d.nitems - i0);
        const hipError_t e = go(d.items + i0, nb, nb);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, int NT>
static hipError_t direct_shape(const DirectLaunch &d, hipStream_t st)
{
    const bool narrow = d.tile == kDirectNarrow;
    if constexpr (sizeof(T) == 4)
        if (d.wide_phase)
            return narrow ? direct_grid<T, NT, kDirectNarrow, true>(d, st) : direct_grid<T, NT, kDirectTile, true>(d, st);
    return narrow ? direct_grid<T, NT, kDirectNarrow, false>(d, st) : direct_grid<T, NT, kDirectTile, false>(d, st);
}

template <typename T>
hipError_t launch_direct(const DirectLaunch &d, hipStream_t st)
{
    if (d.nitems <= 0) return hipSuccess;
    if (sizeof(T) == 8 && d.ctab == nullptr) return hipErrorInvalidValue;   // float64: the phase table
    if (d.tile != kDirectTile && d.tile != kDirectNarrow) return hipErrorInvalidValue;
    switch (d.rows) {
    case 1: return direct_shape<T, 1>(d, st);
    case 2: return direct_shape<T, 2>(d, st);
    case 3: return direct_shape<T, 3>(d, st);
    case 4: return direct_shape<T, 4>(d, st);
    default: return hipErrorInvalidValue;
    }
}

// lanes per target (a power of two): up to a wavefront, while the targets alone do not
// fill the GPU (2^18 threads) and every lane keeps two layers
static int layer_lanes_log2(int64_t n, int layers)
{
    int lg = 0;
    while (lg < 6 && (n << lg) < (int64_t(1) << 18) && (4 << lg) <= layers) ++lg;
    return lg;
}

hipError_t launch_add_layers(double *acc, int64_t n, const double *slab, int layer0, int layers,
                             const int32_t *tgt_layers, int fresh, int rows, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int lg = layer_lanes_log2(n, layers);
    hipLaunchKernelGGL(k_add_layers, dim3(blocks_for(n << lg, 256, INT32_MAX), static_cast<unsigned>(rows)), dim3(256),
                       0, st, reinterpret_cast<double2 *>(acc), n, reinterpret_cast<const double2 *>(slab), layer0,
                       layers, tgt_layers, fresh, lg);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_finalize(const double *acc, int64_t n, const int32_t *perm, void *out, int real_only,
                           const double *slab, int layer0, int layers, const int32_t *tgt_layers, int det, int rows,
                           hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int lg = slab ? layer_lanes_log2(n, layers) : 0;
    hipLaunchKernelGGL(k_finalize<T>, dim3(blocks_for(n << lg, 256, INT32_MAX), static_cast<unsigned>(rows)), dim3(256),
                       0, st, reinterpret_cast<const double2 *>(acc), n, perm, static_cast<cplx<T> *>(out), real_only,
                       reinterpret_cast<const double2 *>(slab), layer0, layers, tgt_layers, det, lg);
    return hipGetLastError();
}

template hipError_t launch_prephase<float>(const PairDev *, const int64_t *, int, int64_t, const double *, int64_t,
                                           const int32_t *, const void *, int64_t, int, void *, void *, int64_t, double,
                                           int, hipStream_t);
template hipError_t launch_prephase<double>(const PairDev *, const int64_t *, int, int64_t, const double *, int64_t,
                                            const int32_t *, const void *, int64_t, int, void *, void *, int64_t,
                                            double, int, hipStream_t);
template hipError_t launch_spread<float>(const PairDev *, const SpreadTile *, int64_t, const int32_t *, const void *,
                                         const void *, int64_t, int, void *, int64_t, const void *, int, double,
                                         hipStream_t);
template hipError_t launch_spread<double>(const PairDev *, const SpreadTile *, int64_t, const int32_t *, const void *,
                                         const void *, int64_t, int, void *, int64_t, const void *, int, double,
                                         hipStream_t);
template hipError_t launch_fft<float>(const PairDev *, const int64_t *, int, int64_t, int, void *, const void *,
                                      const uint32_t *, int, int, double, int, int64_t, hipStream_t);
template hipError_t launch_fft<double>(const PairDev *, const int64_t *, int, int64_t, int, void *, const void *,
                                      const uint32_t *, int, int, double, int, int64_t, hipStream_t);
template hipError_t launch_fft_two<float>(const PairDev *, const int64_t *, int, int64_t, int, void *, const void *,
                                          const uint32_t *, int, int, double, int, int64_t, hipStream_t);
template hipError_t launch_fft_two<double>(const PairDev *, const int64_t *, int, int64_t, int, void *, const void *,
                                          const uint32_t *, int, int, double, int, int64_t, hipStream_t);
template hipError_t launch_transpose<float>(const PairDev *, const int64_t *, int, int64_t, void *, int, int64_t,
                                            hipStream_t);
template hipError_t launch_transpose<double>(const PairDev *, const int64_t *, int, int64_t, void *, int, int64_t,
                                             hipStream_t);
template hipError_t launch_interp<float>(const PairDev *, const int64_t *, int, int64_t, const double *, int64_t,
                                         const double *, const void *, int64_t, double *, int64_t, int, int, double,
                                         double, int, hipStream_t);
template hipError_t launch_interp<double>(const PairDev *, const int64_t *, int, int64_t, const double *, int64_t,
                                          const double *, const void *, int64_t, double *, int64_t, int, int, double,
                                          double, int, hipStream_t);
template hipError_t launch_direct<float>(const DirectLaunch &, hipStream_t);
template hipError_t launch_direct<double>(const DirectLaunch &, hipStream_t);
template <typename T>
hipError_t launch_dde_scale(const void *w, const void *x, void *out, int64_t n, int terms, int conj_w, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dde_scale<T>, dim3(blocks_for(n, 256, INT32_MAX)), dim3(256), 0, st,
                       static_cast<const cplx<T> *>(w), static_cast<const cplx<T> *>(x), static_cast<cplx<T> *>(out), n,
                       terms, conj_w);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_dde_combine(const void *w, const void *y, void *out, int64_t n, int terms, int conj_w, int real_only,
                              hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dde_combine<T>, dim3(blocks_for(n, 256, INT32_MAX)), dim3(256), 0, st,
                       static_cast<const cplx<T> *>(w), static_cast<const cplx<T> *>(y), static_cast<cplx<T> *>(out), n,
                       terms, conj_w, real_only);
    return hipGetLastError();
}

template hipError_t launch_dde_scale<float>(const void *, const void *, void *, int64_t, int, int, hipStream_t);
template hipError_t launch_dde_scale<double>(const void *, const void *, void *, int64_t, int, int, hipStream_t);
template hipError_t launch_dde_combine<float>(const void *, const void *, void *, int64_t, int, int, int, hipStream_t);
template hipError_t launch_dde_combine<double>(const void *, const void *, void *, int64_t, int, int, int,
                                               hipStream_t);
template hipError_t launch_finalize<float>(const double *, int64_t, const int32_t *, void *, int, const double *, int, int,
                                             const int32_t *, int, int, hipStream_t);
template hipError_t launch_finalize<double>(const double *, int64_t, const int32_t *, void *, int, const double *, int, int,
                                             const int32_t *, int, int, hipStream_t);

}  // namespace hvox
