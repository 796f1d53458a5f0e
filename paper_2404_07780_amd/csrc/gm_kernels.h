// gm_kernels.h -- gfx950 kernels of libgmfit.
//
// Work decomposition.  A galaxy's cutout is processed in 32 x 32 output tiles
// by one 256-thread workgroup.  For a tile, the light (FP64) and its FP32
// derivatives with respect to every LM variable are evaluated on the tile's
// (32 + K - 1)^2 input region straight into LDS, one plane per quantity; the
// oversampled central window is evaluated once per model evaluation into a
// small LDS table.  Each thread then owns a 1 x 4 strip of outputs of every
// plane convolved with the PSF (true convolution, zero padding): the FP64
// light by vector FMAs, the FP32 planes on the matrix cores, row segments and
// taps from LDS (the FP64 light's taps at compiled sides above 15: scalar loads
// from memory); the results stay in registers.  When the planes of a model do
// not fit LDS together (or fit only one workgroup per CU) they are processed in
// NG groups, re-evaluating the profile per group (only the first group needs
// the FP64 light).  The fitting kernel turns the convolved planes into
// residuals and FP64 normal-equation sums without writing any image to memory.
//
// gm_fit_batch runs one persistent kernel: each workgroup pulls galaxies, in
// descending-cost order, from an atomic queue and runs the whole
// Levenberg-Marquardt iteration for a galaxy; its first two waves do the FP64
// Cholesky solves and accept or reject between evaluations.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "gmfit.h"
#include "gm_device.h"

namespace gm {

constexpr int TILE = 32;
constexpr int NT = 256;
constexpr int NWAVE = NT / 64;
constexpr int MAXP = 16;
constexpr int MAXWIN = 25;      // oversampled window of at most 5 x 5 pixels
constexpr int MAXOSF = 16;      // sub-samples per pixel side

struct Meta {
    int32_t h, w, k, pad;
    int64_t img_off, psf_off;
};

// Model description passed by value: internal LM index -> column of the
// caller's parameter vector (-1: fixed at fixedv, natural units).
struct ModelArgs {
    int p;
    int col[MAXP];
    double fixedv[MAXP];
    double cst[4];          // shape constants: component 0 at [0..1], component 1 at [2..3]
    double m0;
    int osf, osw;
    int nflux;              // components whose magnitude/amplitude is fitted (start-vector flux split)
};

struct BatchArgs {
    const Meta *meta;
    const float *data, *sigma, *psf;
    const uint8_t *omega;
};

__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Input-region geometry of a tile for PSF side K (row pitch IWP in elements).
__host__ __device__ constexpr int region_h(int K) { return TILE + K - 1; }
// Row pitch: the 32 outputs' 16-byte-aligned input segments need
// 28 + 4 ceil((K + 3) / 4) floats.
__host__ __device__ constexpr int region_wp(int K) { return 28 + 4 * ((K + 3 + 3) / 4); }

// FP64 light plane rows: with a pitch of 48 doubles (PSF side 15) the 16-byte
// reads of two rows two apart (one 16-lane group, strip_of) fall on the same
// LDS banks; rows with bit 1 set stored 2 doubles (16 bytes) further on read
// conflict-free.  The pitch has the 2 spare doubles this needs.
template <int KT>
__host__ __device__ constexpr bool shift64()
{
    return KT > 0 && region_wp(KT) == 48 && region_h(KT) + 2 <= 48;
}

// Output strip of thread tid in a tile: row r, columns 4 cg .. 4 cg + 3.  Wave
// w covers rows 8w .. 8w + 7, 8 lanes per row: lanes 0-31 the even rows, lanes
// 32-63 the odd ones, so that lanes l and l + 32 own the two rows of a row
// pair rp and the convolution can give each half of the wave a plane of its
// own over both rows (conv_pair).  A 16-lane group (which reads LDS together)
// holds row pairs rp and rp + 1, two rows apart: free of bank conflicts at a
// pitch of 16 (mod 32) floats (side 15).  At a pitch of 8 (mod 16) floats
// (sides 7, 9, 23, 25, 39, 41) it holds rp and rp + 2, four rows apart
// (4 x pitch = 32 mod 64), which is conflict-free there.
__host__ __device__ inline int strip_gap(int IWP) { return (IWP % 16 == 8) ? 4 : 2; }
__device__ inline void strip_of(int tid, int K, int &r, int &cg)
{
    const int lane = tid & 63, w = tid >> 6;
    cg = lane & 7;
    const int gi = (lane >> 4) & 1, j = (lane >> 3) & 1;
    const int rp = strip_gap(region_wp(K)) == 4 ? gi + 2 * j : 2 * gi + j;
    r = 8 * w + 2 * rp + (lane >> 5);
}

// Sum of an FP64 value over a wave's strips, every lane gets the total: within
// each row the eight strips by a shift-and-add ladder (row_shr 1, 2, 4), then
// row 2i + 1 + row 2i (strip_gap 2) or row i + 4 + row i (strip_gap 4) for
// i = 0..3, and those four sums in order.
__device__ inline double strip_sum(double v, int K)
{
    v += dpp_move<0x111>(v);
    v += dpp_move<0x112>(v);
    v += dpp_move<0x114>(v);
    if (strip_gap(region_wp(K)) == 4) {
        v += dpp_move<0x118>(v);
        return ((lane_value(v, 15) + lane_value(v, 47)) + lane_value(v, 31)) + lane_value(v, 63);
    }
    v += other_half(v);
    return ((lane_value(v, 7) + lane_value(v, 15)) + lane_value(v, 23)) + lane_value(v, 31);
}

// One row's eight strips (consecutive lanes' values in LDS), in the ladder's order.
__device__ inline double strip_row(const float *p)
{
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    return (((double)b.w + (double)b.z) + ((double)b.y + (double)b.x)) +
           (((double)a.w + (double)a.z) + ((double)a.y + (double)a.x));
}

// Plane groups: plane 0 (FP64) counts two units, the others one; groups are
// contiguous and balanced in units.
__host__ __device__ constexpr int group_bound(int npl, int ng, int g)
{
    if (g <= 0) return 0;
    if (g >= ng) return npl;
    int target = ((npl + 1) * g + ng - 1) / ng, acc = 0;
    for (int q = 0; q < npl; ++q) {
        acc += (q == 0 ? 2 : 1);
        if (acc >= target) return q + 1;
    }
    return npl;
}
__host__ __device__ constexpr int group_units(int npl, int ng, int g)
{
    int lo = group_bound(npl, ng, g), hi = group_bound(npl, ng, g + 1);
    return hi - lo + (lo == 0 ? 1 : 0);
}
__host__ __device__ constexpr int max_group_units(int npl, int ng)
{
    int m = 0;
    for (int g = 0; g < ng; ++g) m = group_units(npl, ng, g) > m ? group_units(npl, ng, g) : m;
    return m;
}

template <class F, int NG>
__host__ __device__ inline size_t planes_bytes(int K)
{
    return (size_t)max_group_units(F::NPL, NG) * region_h(K) * region_wp(K) * sizeof(float);
}

// ---------------------------------------------------------------- per-evaluation state in LDS
// Tiles a thread sums its FP32 partial products of g and J^T W J over before
// they are added, per wave, to FP64 running sums (EvalShared::nacc): a thread
// then never sums more than 4 x 16 = 64 pixels in FP32, whatever the cutout's
// size.  Cutouts of up to 16 tiles (128 x 128) never flush.
constexpr int FLUSH_TILES = 16;

template <class F>
struct EvalShared {
    typename F::Prep prep;
    double win0[F::NCOMP][MAXWIN];
    float win[F::NCOMP][MAXWIN][F::ND];
    double c2[NWAVE];                                     // per-wave chi^2
    int exact, pad;                                       // 1: strips with a NaN anew (conv_group)
    double nacc[NWAVE][F::P + F::P * (F::P + 1) / 2];     // per-wave FP64 sums of the flushed partials
};

// scratch needed by the window tables (in the plane buffer)
template <class F>
__host__ __device__ constexpr size_t window_scratch_bytes()
{
    return (size_t)MAXWIN * MAXOSF * (sizeof(double) + F::ND * sizeof(float));
}

// Dynamic LDS of the evaluating kernels: the plane buffer (which also hosts
// the window partial sums, the wave partial sums of the normal equations and
// the thread-0 solver temporaries), then a copy of the galaxy's PSF with rows
// padded to psf_pitch floats (16-byte aligned rows).
__host__ __device__ inline int psf_pitch(int K) { return (K + 3) & ~3; }
template <class F, int NG>
__host__ __device__ inline size_t lds_main_bytes(int K)
{
    size_t m = planes_bytes<F, NG>(K);
    const size_t sums = (size_t)NWAVE * (1 + F::P + F::P * (F::P + 1) / 2) * 8, solve = (size_t)3 * F::P * F::P * 8;
    m = m > sums ? m : sums;
    m = m > solve ? m : solve;
    m = m > window_scratch_bytes<F>() ? m : window_scratch_bytes<F>();
    return (m + 15) & ~(size_t)15;
}
template <class F, int NG>
__host__ __device__ inline size_t lds_total_bytes(int K)
{
    return lds_main_bytes<F, NG>(K) + (size_t)K * psf_pitch(K) * sizeof(float);
}

// Copy the PSF (K x K, global) into its LDS rows; the caller's next barrier
// publishes it.
template <class F, int NG>
__device__ inline const float *stage_psf(float *planes, const float *psf, int K)
{
    float *d = planes + lds_main_bytes<F, NG>(K) / sizeof(float);
    const int kp = psf_pitch(K);
    for (int i = threadIdx.x; i < K * K; i += NT) {
        const int u = i / K;
        d[u * kp + (i - u * K)] = psf[i];
    }
    return d;
}

// Scalar prologue + oversampled window tables.
// u: LDS (FP64, internal).  scratch: the idle plane buffer.
// Inlined by force, as the other parts of an evaluation: out of line, the
// compiler's choice in the larger kernels, arguments go through scratch memory
// and LDS is read by flat accesses (1,024 bulge + disk fits of 64 x 64 at a
// side of 9, eight trials: 9.1 ms, inline 7.7; their errors 1.14 and 0.98).
template <class F>
__device__ __forceinline__ void eval_prologue(const double *u, const ModelArgs &ma, int H, int W, EvalShared<F> &sh,
                                              float *scratch)
{
    const int tid = threadIdx.x;
    F::prep_all(u, ma.cst, ma.m0, H, W, ma.osf, ma.osw, tid, scratch, sh.prep);
    __syncthreads();
    const int f = ma.osf;
    const double invf = 1.0 / (double)f;
    double *sd = reinterpret_cast<double *>(scratch);
    float *sf = scratch + 2 * MAXWIN * MAXOSF;
#pragma unroll 1
    for (int c = 0; c < F::NCOMP; ++c) {
        const Geo &g = F::geo(sh.prep, c);
        const int ww = g.wj1 - g.wj0 + 1, wh = g.wi1 - g.wi0 + 1;
        if (ww <= 0 || wh <= 0) continue;
        const int nwin = ww * wh, items = nwin * f;
        // each item: one sub-row (t) of one window pixel, summed over s
        for (int it = tid; it < items; it += NT) {
            int pix = it / f, t = it - pix * f;
            int i = g.wi0 + pix / ww, j = g.wj0 + pix % ww;
            double aI = 0.0;
            float ad[F::ND];
#pragma unroll
            for (int q = 0; q < F::ND; ++q) ad[q] = 0.0f;
            const double dy = ((double)(H - i) - ((double)t + 0.5) * invf) - g.y0;
            // ILP samples side by side, added in order (no branch between a
            // sample's products and its sums, which the compiler contracts)
            int s = 0;
#pragma unroll 1
            for (; s + F::ILP <= f; s += F::ILP) {
                double I[F::ILP];
                float d[F::ILP][F::ND] = {};
#pragma unroll
                for (int n = 0; n < F::ILP; ++n) {
                    const double dx = ((double)j + ((double)(s + n) + 0.5) * invf) - g.x0;
                    F::template comp_pt<true, FORM_ROW>(sh.prep, c, dx, dy, I[n], d[n]);
                }
#pragma unroll
                for (int n = 0; n < F::ILP; ++n) {
                    aI += I[n];
#pragma unroll
                    for (int q = 0; q < F::ND; ++q) ad[q] += d[n][q];
                }
            }
            if (F::ILP > 1 && s < f) {
                const double dx = ((double)j + ((double)s + 0.5) * invf) - g.x0;
                double I;
                float d[F::ND] = {};
                F::template comp_pt<true, FORM_ROW>(sh.prep, c, dx, dy, I, d);
                aI += I;
#pragma unroll
                for (int q = 0; q < F::ND; ++q) ad[q] += d[q];
            }
            sd[it] = aI;
#pragma unroll
            for (int q = 0; q < F::ND; ++q) sf[it * F::ND + q] = ad[q];
        }
        __syncthreads();
        const double norm = 1.0 / (double)(f * f);
        // each thread sums one quantity of one pixel over its sub-rows
        for (int it = tid; it < nwin * (F::ND + 1); it += NT) {
            const int pix = it / (F::ND + 1), q = it - pix * (F::ND + 1);
            if (q == F::ND) {
                double s0 = 0.0;
#pragma unroll 4
                for (int t = 0; t < f; ++t) s0 += sd[pix * f + t];
                sh.win0[c][pix] = s0 * norm;
            } else {
                float s = 0.0f;
#pragma unroll 4
                for (int t = 0; t < f; ++t) s += sf[(pix * f + t) * F::ND + q];
                sh.win[c][pix][q] = s * (float)norm;
            }
        }
        __syncthreads();
    }
}

// Light (FP64 if F64) and derivative planes (dp[q - 1] for plane q) of the
// convolved components at the N pixels (i[n], j[n]).  The profile is evaluated
// at every pixel first, N independent chains of FP64 arithmetic side by side,
// and the pixels of the oversampled window then take the table's values.
template <class F, bool F64, int FORM, int N>
__device__ inline void planes_at(const EvalShared<F> &sh, const int (&i)[N], const int (&j)[N], int H,
                                 double (&v0)[N], float (&dp)[N][F::NPL - 1])
{
#pragma unroll
    for (int n = 0; n < N; ++n) {
        v0[n] = 0.0;
#pragma unroll
        for (int q = 0; q < F::NPL - 1; ++q) dp[n][q] = 0.0f;
    }
#pragma unroll
    for (int c = 0; c < F::NCOMP; ++c) {
        const Geo &g = F::geo(sh.prep, c);
        double I[N];
        float d[N][F::ND] = {};
        auto point = [&](int n) {
            const double dx = ((double)j[n] + 0.5) - g.x0;
            const double dy = ((double)(H - i[n]) - 0.5) - g.y0;
            F::template comp_pt<F64, FORM>(sh.prep, c, dx, dy, I[n], d[n]);
        };
        if (N > 1)
#pragma unroll
            for (int n = 0; n < N; ++n) point(n);
#pragma unroll
        for (int n = 0; n < N; ++n) {
            if (i[n] >= g.wi0 && i[n] <= g.wi1 && j[n] >= g.wj0 && j[n] <= g.wj1) {
                const int pix = (i[n] - g.wi0) * (g.wj1 - g.wj0 + 1) + (j[n] - g.wj0);
                I[n] = sh.win0[c][pix];
#pragma unroll
                for (int q = 0; q < F::ND; ++q) d[n][q] = sh.win[c][pix][q];
            } else if (N == 1) {
                point(n);
            }
            v0[n] += I[n];
            F::scatter(c, d[n], dp[n]);
        }
    }
}

// Fill the LDS planes LO..HI-1 of the input region of the tile at (ti0, tj0).
// Layout: if LO == 0 the FP64 light plane comes first (two float units),
// then the FP32 planes in order.  Region points outside the image are the
// convolution's zero padding; the points inside form a rectangle whose
// profile values are spread linearly over all threads of the workgroup.
template <class F, int LO, int HI, bool SH = false>
__device__ __forceinline__ void fill_region(const EvalShared<F> &sh, float *buf, int H, int W, int K, int ti0, int tj0)
{
    const int IH = region_h(K), IWP = region_wp(K), IW = TILE + K - 1, c = (K - 1) / 2;
    const int plane_sz = IH * IWP;
    double *b0 = reinterpret_cast<double *>(buf);
    float *bf = (LO == 0) ? buf + 2 * plane_sz : buf;
    constexpr int QLO = LO == 0 ? 1 : LO;
    // region rows r0..r1-1 and columns c0..c1-1 lie inside the image
    const int r0 = max(0, c - ti0), r1 = min(IH, H + c - ti0);
    const int c0 = max(0, c - tj0), c1 = min(IW, W + c - tj0);
    // region point (ri, ci); SH: rows with bit 1 set of the FP64 plane 2 further on
    auto store = [&](int ri, int ci, double v0, const float *dp) {
        const int idx = ri * IWP + ci;
        if constexpr (LO == 0) b0[SH ? idx + (ri & 2) : idx] = v0;
#pragma unroll
        for (int q = QLO; q < HI; ++q) bf[(q - QLO) * plane_sz + idx] = dp[q - 1];
    };
    const bool edge = r0 > 0 || r1 < IH || c0 > 0 || c1 < IW;
    if (edge) {
        float z[F::NPL - 1];
#pragma unroll
        for (int q = 0; q < F::NPL - 1; ++q) z[q] = 0.0f;
        for (int t = threadIdx.x; t < IH * IW; t += NT) {
            const int ri = t / IW, ci = t - ri * IW;
            if (ri < r0 || ri >= r1 || ci < c0 || ci >= c1) store(ri, ci, 0.0, z);
        }
    }
    const int nc = c1 - c0, npts = (r1 - r0) * nc;
    // row of a linear index by a float product: (t + 0.5) / nc is below the
    // row count (< 2^8) and at least 1/(2 nc) > 2^-9 away from an integer,
    // while the float rounding moves it by less than 2^-14
    const float rnc = 1.0f / (float)nc;
    // N points per thread and step (the last step's second may be none)
    constexpr int N = F::ILP, FORM = LO == 0 && HI == 1 ? FORM_LIGHT : FORM_POINT;
#pragma unroll 1
    for (int t = threadIdx.x; t < npts; t += N * NT) {
        int ri[N], ci[N], i[N], j[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int tn = n ? min(t + n * NT, npts - 1) : t;
            const int rr = (int)(((float)tn + 0.5f) * rnc);
            ri[n] = r0 + rr;
            ci[n] = c0 + (tn - rr * nc);
            i[n] = ti0 - c + ri[n];
            j[n] = tj0 - c + ci[n];
        }
        double v0[N];
        float dp[N][F::NPL - 1];
        planes_at<F, LO == 0, FORM, N>(sh, i, j, H, v0, dp);
#pragma unroll
        for (int n = 0; n < N; ++n)
            if (n == 0 || t + n * NT < npts) store(ri[n], ci[n], v0[n], dp[n]);
    }
}

// The PSF is read through the constant address space with a wave-uniform
// offset: such loads are scalar (s_load through the scalar cache) and the taps
// reach the FMAs as SGPR operands.
typedef __attribute__((address_space(4))) const float cfloat;

__device__ inline int64_t uniform64(int64_t x)
{
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)x);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// One PSF row (KT taps) against a row segment: acc[t] += sum_v p[v] seg[t + KT-1-v].
template <int KT, typename T, typename PR>
__device__ inline void row_fma(const T *seg, PR pr, T &a0, T &a1, T &a2, T &a3)
{
#pragma unroll
    for (int v = 0; v < KT; ++v) {
        const T pv = (T)pr[v];
        a0 = fma(pv, seg[KT - 1 - v], a0);
        a1 = fma(pv, seg[KT - v], a1);
        a2 = fma(pv, seg[KT + 1 - v], a2);
        a3 = fma(pv, seg[KT + 2 - v], a3);
    }
}

// Load the (KT + 3)-element row segment at p (16-byte aligned) into seg.
template <int KT, typename T>
__device__ inline void load_seg(const T *p, T *seg)
{
    constexpr int PER = 16 / sizeof(T);
    constexpr int NV = (KT + 3 + PER - 1) / PER;
    using V = typename std::conditional<sizeof(T) == 4, float4, double2>::type;
    const V *rp = reinterpret_cast<const V *>(p);
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        V t = rp[q];
        if constexpr (sizeof(T) == 4) {
            seg[4 * q] = t.x; seg[4 * q + 1] = t.y; seg[4 * q + 2] = t.z; seg[4 * q + 3] = t.w;
        } else {
            seg[2 * q] = t.x; seg[2 * q + 1] = t.y;
        }
    }
}

// Any PSF side, FP64: element by element of the row segment, from the far end
// (each accumulator then sees its taps in increasing order), the four taps an
// element meets sliding through registers; PSF rows from LDS (psl).
__device__ inline void conv64_any(const double *base, int r, int K, int IWP, const float *psl, double (&out)[4])
{
    double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    const int kp = psf_pitch(K);
    if (K == 1) {
        const double p = (double)psl[0];
        const double *rp = base + r * IWP;
        out[0] = fma(p, rp[0], 0.0);
        out[1] = fma(p, rp[1], 0.0);
        out[2] = fma(p, rp[2], 0.0);
        out[3] = fma(p, rp[3], 0.0);
        return;
    }
#pragma unroll 1
    for (int u = 0; u < K; ++u) {
        const double *rp = base + (r + K - 1 - u) * IWP;
        const float *pr = psl + u * kp;
        // element e = K + 2 - m meets tap m - 3 + t for output t
        double w1 = (double)pr[0], w2 = (double)pr[1], w3 = (double)pr[2];
        a3 = fma(w1, rp[K + 2], a3);
        a2 = fma(w1, rp[K + 1], a2);
        a3 = fma(w2, rp[K + 1], a3);
        a1 = fma(w1, rp[K], a1);
        a2 = fma(w2, rp[K], a2);
        a3 = fma(w3, rp[K], a3);
        // K - 3 elements meet four taps each: K is odd, two at a time
        double x0 = rp[K - 1], x1 = rp[K - 2];
        float n0 = pr[min(3, K - 1)], n1 = pr[min(4, K - 1)];
#pragma unroll 1
        for (int m = 3; m < K; m += 2) {
            const double e0 = x0, e1 = x1, p0 = (double)n0, p1 = (double)n1;
            if (m + 2 < K) {
                x0 = rp[K - m];
                x1 = rp[K - 1 - m];
                n0 = pr[m + 2];
                n1 = pr[m + 3];
            }
            a0 = fma(w1, e0, a0);
            a1 = fma(w2, e0, a1);
            a2 = fma(w3, e0, a2);
            a3 = fma(p0, e0, a3);
            a0 = fma(w2, e1, a0);
            a1 = fma(w3, e1, a1);
            a2 = fma(p0, e1, a2);
            a3 = fma(p1, e1, a3);
            w1 = w3;
            w2 = p0;
            w3 = p1;
        }
        a0 = fma(w1, rp[2], a0);
        a1 = fma(w2, rp[2], a1);
        a2 = fma(w3, rp[2], a2);
        a0 = fma(w2, rp[1], a0);
        a1 = fma(w3, rp[1], a1);
        a0 = fma(w3, rp[0], a0);
    }
    out[0] = a0; out[1] = a1; out[2] = a2; out[3] = a3;
}

// The taps of PSF row u from its LDS copy (rows of KP = psf_pitch floats).
template <int KP>
__device__ inline void load_taps(const float *psl, int u, float (&tp)[KP])
{
    const float4 *tv = reinterpret_cast<const float4 *>(psl + u * KP);
#pragma unroll
    for (int q = 0; q < KP / 4; ++q) {
        const float4 t = tv[q];
        tp[4 * q] = t.x; tp[4 * q + 1] = t.y; tp[4 * q + 2] = t.z; tp[4 * q + 3] = t.w;
    }
}

// ---------------------------------------------------------------- FP32 planes on the matrix cores
// A 1 x 4 strip against one PSF row is out[t] += sum_x seg[x] p[K - 1 + t - x]
// (x = 0 .. K + 2): for each x an outer product of four taps and one element
// per lane.  v_mfma_f32_4x4x1_16b_f32 does exactly that: its B operand and its
// four results belong to the lane, and its A operand, four values, is
// broadcast to all 16 blocks from the block the instruction names (cbsz = 4,
// abid), so one register holds the tap quadruples of 16 consecutive x (lane
// 4 b + t: x = b, output t; 0 outside the PSF).  It is a fused multiply-add
// with one rounding (also for denormals), and x runs downwards, so each
// accumulator sees the products of the scalar loop in its order: the results
// are the same bits (the extra products are 0 x finite; conv_group sees to
// strips with infinite elements).  A SIMD issues one instruction every 8.3
// cycles (a wave alone: 9.0 with two accumulators in turn, conv_pair, 8.5 with
// four, conv_quad), which replaces four FMAs at 2.5 cycles each (a wave alone:
// 4.9); matrix and vector instructions of two waves do not overlap (all
// measured), so what bounds the convolutions is the FMA
// units.  Before (FMAs with the taps in registers) and now, ms: 2,048 masked
// cutouts of 48-256 px, side 25: 326 -> 229; 256 of 64-128 px, side 31 (any-side
// loops, taps and elements one by one before): 907 -> 301; 16,384 of 64 x 64,
// side 15: 55.4 -> 52.8.
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int ABID>
__device__ inline f32x4 mfma_tap(float taps, float x, f32x4 acc)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(taps, x, acc, 4, ABID, 0);
}

// Registers of the tap quadruples of one PSF row.
__host__ __device__ constexpr int tap_regs(int K) { return (K + 3 + 15) / 16; }

// This lane's place in tap register j: column v of the PSF row, or none
// (FLIP: of the PSF flipped in both axes, whose row u is row K - 1 - u).
struct TapLane {
    int v;
    bool in;
};
template <bool FLIP = false>
__device__ inline TapLane tap_lane(int lane, int K, int j)
{
    const int v = K - 1 + (lane & 3) - (16 * j + (lane >> 2)), c = min(max(v, 0), K - 1);
    return TapLane{FLIP ? K - 1 - c : c, v >= 0 && v < K};
}

// seg[x] for x = X .. 0 against the taps of one PSF row, and (two rows) of the
// row before it.
template <int X>
__device__ inline void mfma_row(const float *t, const float *seg, f32x4 &a)
{
    if constexpr (X >= 0) {
        a = mfma_tap<X % 16>(t[X / 16], seg[X], a);
        mfma_row<X - 1>(t, seg, a);
    }
}
template <int X>
__device__ inline void mfma_row2(const float *t1, const float *t0, const float *s1, const float *s0, f32x4 &a1,
                                 f32x4 &a0)
{
    if constexpr (X >= 0) {
        a1 = mfma_tap<X % 16>(t1[X / 16], s1[X], a1);
        a0 = mfma_tap<X % 16>(t0[X / 16], s0[X], a0);
        mfma_row2<X - 1>(t1, t0, s1, s0, a1, a0);
    }
}

// Products before, LDS reads after: without it the compiler gathers the reads
// of both halves of an unrolled loop in front of the products, and the
// segments then need copies from register to register.
__device__ inline void keep_order(f32x4 &a) { asm volatile("" : "+v"(a)::"memory"); }
__device__ inline void keep_order(f32x4 &a, f32x4 &b) { asm volatile("" : "+v"(a), "+v"(b)::"memory"); }

// After a plane pair: lo, hi hold rows 2 rp, 2 rp + 1 of plane A in lanes 0-31
// and of plane B in lanes 32-63; exchanged, lo holds plane A and hi plane B at
// each lane's own row.
__device__ inline void split_pair(f32x4 &lo, f32x4 &hi)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float l = lo[t], h = hi[t];
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(h), false, false);
        lo[t] = __uint_as_float(s[0]);
        hi[t] = __uint_as_float(s[1]);
    }
}

// Two FP32 planes at once, one per half of the wave, over both rows of each
// lane's row pair: a row segment read from LDS serves PSF row u for the odd
// row and u - 1 for the even one, so K + 1 segments are read per pair of rows
// and plane instead of 2 K.  p: this lane's plane at the even row, PSF row 0
// (LDS row 2 rp + K - 1), column 4 cg.  The next segment and taps are read
// while the current ones are used.  KT odd, at least 3.
template <int KT>
__device__ inline void conv_pair(const float *p, const float *psl, f32x4 &lo, f32x4 &hi)
{
    constexpr int KP = (KT + 3) & ~3, IWP = 28 + 4 * ((KT + 3 + 3) / 4), SEG = ((KT + 3 + 3) / 4) * 4;
    constexpr int NR = tap_regs(KT);
    const int lane = threadIdx.x & 63;
    TapLane tl[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) tl[j] = tap_lane(lane, KT, j);
    auto taps = [&](int u, float (&t)[NR]) {
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const float x = psl[u * KP + tl[j].v];
            t[j] = tl[j].in ? x : 0.0f;
        }
    };
    f32x4 a0 = {0.0f, 0.0f, 0.0f, 0.0f}, a1 = a0;
    float sa[SEG], sb[SEG], ta[NR], tb[NR];
    taps(0, ta);
    load_seg<KT>(p + IWP, sa);
    taps(1, tb);
    load_seg<KT>(p, sb);
    mfma_row<KT + 2>(ta, sa, a1);
#pragma unroll 1
    for (int t = 1; t < KT; t += 2) {
        // sb, tb: row t; ta: the taps of row t - 1
        float tc[NR];
        taps(t + 1, tc);
        load_seg<KT>(p - t * IWP, sa);
        mfma_row2<KT + 2>(tb, ta, sb, sb, a1, a0);
        keep_order(a1, a0);
        taps(min(t + 2, KT - 1), ta);
        load_seg<KT>(p - (t + 1) * IWP, sb);
        mfma_row2<KT + 2>(tc, tb, sa, sa, a1, a0);
        keep_order(a1, a0);
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const float x = ta[j];
            ta[j] = tc[j];
            tb[j] = x;
        }
    }
    mfma_row<KT + 2>(ta, sb, a0);       // row KT, the even rows' last
    lo = a0;
    hi = a1;
}

// Two plane pairs at once (p and q as conv_pair's p): four accumulators in
// turn, so that no instruction waits for the one two before it (a pair alone
// needs a wait state on every third): 16,384 Sersic fits of 64 x 64 43.6 -> 41.9 ms.
template <int X>
__device__ inline void mfma_row4(const float *t1, const float *t0, const float *s, const float *z, f32x4 (&a)[4])
{
    if constexpr (X >= 0) {
        a[1] = mfma_tap<X % 16>(t1[X / 16], s[X], a[1]);
        a[0] = mfma_tap<X % 16>(t0[X / 16], s[X], a[0]);
        a[3] = mfma_tap<X % 16>(t1[X / 16], z[X], a[3]);
        a[2] = mfma_tap<X % 16>(t0[X / 16], z[X], a[2]);
        mfma_row4<X - 1>(t1, t0, s, z, a);
    }
}
__device__ inline void keep_order(f32x4 (&a)[4])
{
    asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3])::"memory");
}
template <int KT>
__device__ inline void conv_quad(const float *p, const float *q, const float *psl, f32x4 (&a)[4])
{
    constexpr int KP = (KT + 3) & ~3, IWP = 28 + 4 * ((KT + 3 + 3) / 4), SEG = ((KT + 3 + 3) / 4) * 4;
    constexpr int NR = tap_regs(KT);
    const int lane = threadIdx.x & 63;
    TapLane tl[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) tl[j] = tap_lane(lane, KT, j);
    auto taps = [&](int u, float (&t)[NR]) {
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const float x = psl[u * KP + tl[j].v];
            t[j] = tl[j].in ? x : 0.0f;
        }
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float sa[SEG], sb[SEG], za[SEG], zb[SEG], ta[NR], tb[NR];
    taps(0, ta);
    load_seg<KT>(p + IWP, sa);
    load_seg<KT>(q + IWP, za);
    taps(1, tb);
    load_seg<KT>(p, sb);
    load_seg<KT>(q, zb);
    mfma_row2<KT + 2>(ta, ta, sa, za, a[1], a[3]);
#pragma unroll 1
    for (int t = 1; t < KT; t += 2) {
        // sb, zb, tb: row t; ta: the taps of row t - 1
        float tc[NR];
        taps(t + 1, tc);
        load_seg<KT>(p - t * IWP, sa);
        load_seg<KT>(q - t * IWP, za);
        mfma_row4<KT + 2>(tb, ta, sb, zb, a);
        keep_order(a);
        taps(min(t + 2, KT - 1), ta);
        load_seg<KT>(p - (t + 1) * IWP, sb);
        load_seg<KT>(q - (t + 1) * IWP, zb);
        mfma_row4<KT + 2>(tc, tb, sa, za, a);
        keep_order(a);
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const float x = ta[j];
            ta[j] = tc[j];
            tb[j] = x;
        }
    }
    mfma_row2<KT + 2>(ta, ta, sb, zb, a[0], a[2]);      // row KT, the even rows' last
}

// One FP32 plane, each lane its own row (the odd plane out).  p: this lane's
// row at PSF row 0, column 4 cg.  FLIP: with the flipped PSF (a correlation).
template <int KT, bool FLIP = false>
__device__ inline void conv_one(const float *p, const float *psl, f32x4 &out)
{
    constexpr int KP = (KT + 3) & ~3, IWP = 28 + 4 * ((KT + 3 + 3) / 4), SEG = ((KT + 3 + 3) / 4) * 4;
    constexpr int NR = tap_regs(KT);
    const int lane = threadIdx.x & 63;
    TapLane tl[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) tl[j] = tap_lane<FLIP>(lane, KT, j);
    auto taps = [&](int u, float (&t)[NR]) {
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const float x = psl[(FLIP ? KT - 1 - u : u) * KP + tl[j].v];
            t[j] = tl[j].in ? x : 0.0f;
        }
    };
    f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
    float sa[SEG], sb[SEG], ta[NR], tb[NR];
    taps(0, ta);
    load_seg<KT>(p, sa);
#pragma unroll 1
    for (int u = 0; u + 1 < KT; u += 2) {
        taps(u + 1, tb);
        load_seg<KT>(p - (u + 1) * IWP, sb);
        mfma_row<KT + 2>(ta, sa, a);
        keep_order(a);
        taps(u + 2, ta);
        load_seg<KT>(p - (u + 2) * IWP, sa);
        mfma_row<KT + 2>(tb, sb, a);
        keep_order(a);
    }
    mfma_row<KT + 2>(ta, sa, a);
    out = a;
}

// Any PSF side K (odd): TWO planes per call as conv_pair (TWO), or one as
// conv_one.  Sixteen elements of the segment (one tap register) at a time, the
// next sixteen read while they are used; four-element groups past the segment
// are skipped, and elements past it in the last group are taken as 0.
struct Seg16 {
    f32x4 q[4];
};

template <int Q>
__device__ inline void mfma_quad(float t1, float t0, bool two, bool one, const f32x4 &x, f32x4 &a1, f32x4 &a0)
{
    if (two) {
        a1 = mfma_tap<4 * Q + 3>(t1, x[3], a1);
        a0 = mfma_tap<4 * Q + 3>(t0, x[3], a0);
        a1 = mfma_tap<4 * Q + 2>(t1, x[2], a1);
        a0 = mfma_tap<4 * Q + 2>(t0, x[2], a0);
        a1 = mfma_tap<4 * Q + 1>(t1, x[1], a1);
        a0 = mfma_tap<4 * Q + 1>(t0, x[1], a0);
        a1 = mfma_tap<4 * Q>(t1, x[0], a1);
        a0 = mfma_tap<4 * Q>(t0, x[0], a0);
    } else if (one) {
        a1 = mfma_tap<4 * Q + 3>(t1, x[3], a1);
        a1 = mfma_tap<4 * Q + 2>(t1, x[2], a1);
        a1 = mfma_tap<4 * Q + 1>(t1, x[1], a1);
        a1 = mfma_tap<4 * Q>(t1, x[0], a1);
    } else {
        a0 = mfma_tap<4 * Q + 3>(t0, x[3], a0);
        a0 = mfma_tap<4 * Q + 2>(t0, x[2], a0);
        a0 = mfma_tap<4 * Q + 1>(t0, x[1], a0);
        a0 = mfma_tap<4 * Q>(t0, x[0], a0);
    }
}

// a1: PSF row t of this lane's row (TWO: of the odd row), a0: PSF row t - 1 of
// the even row.  p: column 4 cg of this lane's plane and the LDS row of step 0.
template <bool TWO, bool FLIP = false>
__device__ inline void conv_any(const float *p, int K, int IWP, const float *psl, f32x4 &lo, f32x4 &hi)
{
    const int lane = threadIdx.x & 63, kp = psf_pitch(K), nx = K + 3, nj = tap_regs(K);
    const int steps = TWO ? K + 1 : K;
    f32x4 a0 = {0.0f, 0.0f, 0.0f, 0.0f}, a1 = a0;
    Seg16 x, y;
    float t1 = 0.0f, t0 = 0.0f, s1 = 0.0f, s0 = 0.0f;
    // the elements and taps of step t, register j
    auto load = [&](int t, int j, Seg16 &v, float &w1, float &w0) {
        const float *row = p - t * IWP + 16 * j;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            f32x4 e = {0.0f, 0.0f, 0.0f, 0.0f};
            if (16 * j + 4 * q < nx) {
                e = *reinterpret_cast<const f32x4 *>(row + 4 * q);
                if (16 * j + 4 * q + 2 >= nx) e[2] = e[3] = 0.0f;      // nx is even
            }
            v.q[q] = e;
        }
        const TapLane tl = tap_lane<FLIP>(lane, K, j);
        const int u = min(t, K - 1);
        const float c = psl[(FLIP ? K - 1 - u : u) * kp + tl.v];
        w1 = tl.in ? c : 0.0f;
        if (TWO) {
            const float b = psl[max(t - 1, 0) * kp + tl.v];
            w0 = tl.in ? b : 0.0f;
        }
    };
    int t = 0, j = nj - 1;
    load(t, j, x, t1, t0);
#pragma unroll 1
    while (true) {
        int tn = t, jn = j - 1;
        if (jn < 0) {
            jn = nj - 1;
            tn = t + 1;
        }
        const bool more = tn < steps;
        if (more) load(tn, jn, y, s1, s0);
        const bool two = TWO && t > 0 && t < K, one = t < K;
        const int left = nx - 16 * j;
        if (left > 12) mfma_quad<3>(t1, t0, two, one, x.q[3], a1, a0);
        if (left > 8) mfma_quad<2>(t1, t0, two, one, x.q[2], a1, a0);
        if (left > 4) mfma_quad<1>(t1, t0, two, one, x.q[1], a1, a0);
        mfma_quad<0>(t1, t0, two, one, x.q[0], a1, a0);
        if (!more) break;
        t = tn;
        j = jn;
        t1 = s1;
        t0 = s0;
        x = y;
    }
    lo = a0;
    hi = a1;
}

// Order products before the reads that follow, as keep_order.
__device__ inline void keep_order64(double (&a)[4])
{
    asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3])::"memory");
}

// Segment elements E0 .. E0 + N - 1 that taps V0 .. V1-1 of a row meet.
template <int KT, int V0, int V1, int E0>
struct Part64 {
    static constexpr int N = ((KT + 2 - V0) - E0 + 2) / 2 * 2;
    double seg[N];
    __device__ inline void load(const double *rp)
    {
        const double2 *vp = reinterpret_cast<const double2 *>(rp + E0);
#pragma unroll
        for (int q = 0; q < N / 2; ++q) {
            const double2 t = vp[q];
            seg[2 * q] = t.x;
            seg[2 * q + 1] = t.y;
        }
    }
    __device__ inline void add(const float *tp, double (&a)[4]) const
    {
#pragma unroll
        for (int v = V0; v < V1; ++v) {
            const double pv = (double)tp[v];
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t] = fma(pv, seg[KT - 1 - v + t - E0], a[t]);
        }
        keep_order64(a);
    }
};

// The FP64 light plane with PSF sides above 15, the taps as scalar loads, each
// row in two halves of taps (v < VS meet elements from ES on, v >= VS elements
// from 0).  Scalar loads and LDS reads share one counter and complete out of
// order with each other, so a wait between them is a wait for all: each half's
// reads (the second half's with the next row's taps) are issued in front of
// the other half's products and waited for behind them.  Bound by the FP64
// units (100 FMAs and 25 conversions a row at side 25): 21.5k cycles per tile
// with waits in front of each half, now 19.2k; with the taps from LDS 23k, with
// whole rows ahead the registers spill.
template <int KT>
__device__ inline void conv64_wide(const double *b64, const cfloat *psf, int r, double (&acc0)[4])
{
    constexpr int IWP = (28 + 4 * ((KT + 3 + 3) / 4));
    constexpr int ES = 4 * ((KT - 1) / 8), VS = KT - ES;
    Part64<KT, 0, VS, ES> a;
    Part64<KT, VS, KT, 0> b;
    double d[4] = {0.0, 0.0, 0.0, 0.0};
    float ta[KT], tb[KT];
    const double *rp = b64 + (r + KT - 1) * IWP;
    auto taps = [&](int u, float (&t)[KT]) {
#pragma unroll
        for (int v = 0; v < KT; ++v) t[v] = psf[u * KT + v];
    };
    taps(0, ta);
    a.load(rp);
#pragma unroll 1
    for (int u = 0; u + 1 < KT; u += 2) {
        b.load(rp - u * IWP);
        a.add(ta, d);
        a.load(rp - (u + 1) * IWP);
        taps(u + 1, tb);
        b.add(ta, d);
        b.load(rp - (u + 1) * IWP);
        a.add(tb, d);
        a.load(rp - (u + 2) * IWP);
        taps(u + 2, ta);
        b.add(tb, d);
    }
    b.load(rp - (KT - 1) * IWP);
    a.add(ta, d);
    b.add(ta, d);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc0[t] = d[t];
}

// The FP64 light plane with PSF sides up to 15.  Every load of the loop is an
// LDS read (the taps from the PSF's LDS copy, the segments from the plane),
// and LDS reads complete in order, so a wait covers exactly the reads a
// product needs: the segment and taps of the next PSF row are read while the
// current row is used.
template <int KT>
__device__ inline void conv64_rows(const double *b64, const float *psl, int r, double (&acc0)[4])
{
    constexpr int KP = (KT + 3) & ~3;
    constexpr int IWP = (28 + 4 * ((KT + 3 + 3) / 4));
    constexpr int SEG64 = ((KT + 3 + 1) / 2) * 2;
    constexpr bool SH = shift64<KT>();
    const int rr0 = r + KT - 1;
    auto row = [&](int u) {
        const int y = rr0 - u;
        return b64 + y * IWP + (SH ? (y & 2) : 0);
    };
    double d0 = 0.0, d1 = 0.0, d2 = 0.0, d3 = 0.0;
    double sa[SEG64], sb[SEG64];
    float ta[KP], tb[KP];
    load_taps<KP>(psl, 0, ta);
    load_seg<KT>(row(0), sa);
#pragma unroll 1
    for (int u = 0; u + 1 < KT; u += 2) {
        load_taps<KP>(psl, u + 1, tb);
        load_seg<KT>(row(u + 1), sb);
        row_fma<KT>(sa, ta, d0, d1, d2, d3);
        if (u + 2 < KT) {
            load_taps<KP>(psl, u + 2, ta);
            load_seg<KT>(row(u + 2), sa);
        }
        row_fma<KT>(sb, tb, d0, d1, d2, d3);
    }
    if (KT & 1) row_fma<KT>(sa, ta, d0, d1, d2, d3);
    acc0[0] = d0; acc0[1] = d1; acc0[2] = d2; acc0[3] = d3;
}

// The FP64 light plane for this thread's 1 x 4 strip.
template <int KT>
__device__ inline void conv64(const float *buf, int K, const cfloat *psf, const float *psl, int r, int cg,
                              double (&acc0)[4])
{
    const double *b64 = reinterpret_cast<const double *>(buf) + 4 * cg;
    if constexpr (KT > 15) conv64_wide<KT>(b64, psf, r, acc0);
    else if constexpr (KT > 0) conv64_rows<KT>(b64, psl, r, acc0);
    else conv64_any(b64, r, K, region_wp(K), psl, acc0);
}

// One FP32 plane by scalar products, each output's own taps alone: for strips
// in which the matrix cores met an infinite element (p as conv_one's).
__device__ inline void conv_strip(const float *p, int K, int IWP, const float *psl, float (&out)[4])
{
    const int kp = psf_pitch(K);
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int u = 0; u < K; ++u) {
        const float *rp = p - u * IWP, *pr = psl + u * kp;
        float s1 = rp[K], s2 = rp[K + 1], s3 = rp[K + 2];
#pragma unroll 4
        for (int v = 0; v < K; ++v) {
            const float s0 = rp[K - 1 - v], pv = pr[v];
            a[0] = fmaf(pv, s0, a[0]);
            a[1] = fmaf(pv, s1, a[1]);
            a[2] = fmaf(pv, s2, a[2]);
            a[3] = fmaf(pv, s3, a[3]);
            s3 = s2;
            s2 = s1;
            s1 = s0;
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) out[t] = a[t];
}

// Convolve planes LO..HI-1 for this thread's 1 x 4 output strip (tile row r,
// columns 4 cg .. 4 cg + 3): plane 0 in FP64 on the vector units, the FP32
// planes two at a time on the matrix cores.  KT > 0: compile-time PSF side;
// 0: any K.  A matrix instruction multiplies an element by zero for the
// outputs of the strip whose PSF does not reach it; an infinite element (a
// derivative beyond FP32's range) makes those NaN, so a strip that holds a NaN
// is convolved anew by scalar products where *exact is set (v_maximum3_f32,
// which keeps a NaN, looks at two values an instruction).
template <class F, int KT, int LO, int HI>
__device__ inline void conv_group(const float *__restrict__ buf, int K, const cfloat *psf, const float *psl, int r,
                                  int cg, double (&acc0)[4], float (&acc)[F::NPL][4], const int *exact)
{
    const int IH = region_h(K), IWP = region_wp(K);
    const int plane_sz = IH * IWP;
    constexpr int QLO = LO == 0 ? 1 : LO, NP = HI - QLO;
    const float *bf = ((LO == 0) ? buf + 2 * plane_sz : buf) + 4 * cg;
    if constexpr (LO == 0) conv64<KT>(buf, K, psf, psl, r, cg, acc0);
    const int half = (threadIdx.x >> 5) & 1;
    constexpr int NQ = KT > 0 && KT <= 25 ? NP / 4 * 4 : 0;
#pragma unroll
    for (int pl = 0; pl < NQ; pl += 4) {
        const float *p = bf + (pl + half) * plane_sz + ((r & ~1) + K - 1) * IWP;
        f32x4 a[4];
        conv_quad<KT>(p, p + 2 * plane_sz, psl, a);
#pragma unroll
        for (int k = 0; k < 4; k += 2) {
            split_pair(a[k], a[k + 1]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                acc[QLO + pl + k][t] = a[k][t];
                acc[QLO + pl + k + 1][t] = a[k + 1][t];
            }
        }
    }
#pragma unroll
    for (int pl = NQ; pl + 1 < NP; pl += 2) {
        const float *p = bf + (pl + half) * plane_sz + ((r & ~1) + K - 1) * IWP;
        f32x4 lo, hi;
        if constexpr (KT > 0) conv_pair<KT>(p, psl, lo, hi);
        else conv_any<true>(p + IWP, K, IWP, psl, lo, hi);
        split_pair(lo, hi);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc[QLO + pl][t] = lo[t];
            acc[QLO + pl + 1][t] = hi[t];
        }
    }
    if constexpr (NP & 1) {
        const float *p = bf + (NP - 1) * plane_sz + (r + K - 1) * IWP;
        f32x4 one, none;
        if constexpr (KT > 0) conv_one<KT>(p, psl, one);
        else conv_any<false>(p, K, IWP, psl, none, one);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[HI - 1][t] = one[t];
    }
    if constexpr (NP > 0) {
        if (uniform(*exact) == 0) return;
        float all = 0.0f;
#pragma unroll
        for (int q = QLO; q < HI; ++q)
#pragma unroll
            for (int t = 0; t < 4; t += 2)
                all = __builtin_elementwise_maximum(__builtin_elementwise_maximum(all, acc[q][t]), acc[q][t + 1]);
        if (__builtin_expect(all != all, 0)) {
            int tid = threadIdx.x, row, col;       // worked out anew: nothing is kept for this path
            asm volatile("" : "+v"(tid));
            strip_of(tid, K, row, col);
            const float *p = buf + (LO == 0 ? 2 * plane_sz : 0) + 4 * col + (row + K - 1) * IWP;
            unsigned which = 0;
#pragma unroll
            for (int q = QLO; q < HI; ++q) {
                const float x = (acc[q][0] + acc[q][1]) + (acc[q][2] + acc[q][3]);
                which |= (x != x ? 1u : 0u) << (q - QLO);
            }
#pragma unroll 1
            for (int pl = 0; pl < NP; ++pl) {
                if (!((which >> pl) & 1u)) continue;
                float o[4];
                conv_strip(p + pl * plane_sz, K, IWP, psl, o);
#pragma unroll
                for (int q = QLO; q < HI; ++q)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[q][t] = q - QLO == pl ? o[t] : acc[q][t];
            }
        }
    }
}

// All groups of one tile: fill, convolve, leave the buffer idle.
template <class F, int KT, int NG, int G = 0>
__device__ inline void tile_planes(const EvalShared<F> &sh, float *buf, int H, int W, int K, int ti0, int tj0,
                                   const cfloat *psf, const float *psl, int r, int cg, double (&acc0)[4],
                                   float (&acc)[F::NPL][4])
{
    if constexpr (G < NG) {
        constexpr int LO = group_bound(F::NPL, NG, G), HI = group_bound(F::NPL, NG, G + 1);
        fill_region<F, LO, HI, shift64<KT>()>(sh, buf, H, W, K, ti0, tj0);
        __syncthreads();
        conv_group<F, KT, LO, HI>(buf, K, psf, psl, r, cg, acc0, acc, &sh.exact);
        __syncthreads();
        tile_planes<F, KT, NG, G + 1>(sh, buf, H, W, K, ti0, tj0, psf, psl, r, cg, acc0, acc);
    }
}

// d M / d u_k at output column t of this thread's strip.
// (dx, dy): the pixel's offset from the cutout's centre (analytic sky columns).
template <class F>
__device__ inline float jac_at(int k, int t, const double (&acc0)[4], const float (&acc)[F::NPL][4], float dx,
                               float dy)
{
    if (F::analytic(k)) return F::analytic_value(k, dx, dy);
    if (k == F::DER) {
        float col[F::NPL];
#pragma unroll
        for (int q = 0; q < F::NPL; ++q) col[q] = acc[q][t];
        return F::derived(acc0[t], col);
    }
    return acc[F::plane(k)][t];
}

__device__ inline float pixel_weight(const BatchArgs &ba, int64_t idx, float &d)
{
    d = ba.data[idx];
    float s = ba.sigma[idx];
    bool ok = (ba.omega == nullptr || ba.omega[idx] != 0) && s > 0.0f && isfinite(s) && isfinite(d);
    return ok ? 1.0f / (s * s) : 0.0f;
}

// pixel_weight of the four pixels j0 .. j0 + 3 of the row starting at rowoff,
// read together (columns past W - 1 read pixel W - 1; the caller skips them):
// one wait for the strip instead of one per pixel.
__device__ inline void strip_weights(const BatchArgs &ba, int64_t rowoff, int j0, int W, float (&d)[4],
                                     float (&w)[4])
{
    float s[4];
    int m[4] = {1, 1, 1, 1};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int64_t idx = rowoff + min(j0 + t, W - 1);
        d[t] = ba.data[idx];
        s[t] = ba.sigma[idx];
    }
    if (ba.omega) {
#pragma unroll
        for (int t = 0; t < 4; ++t) m[t] = ba.omega[rowoff + min(j0 + t, W - 1)];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const bool ok = m[t] != 0 && s[t] > 0.0f && isfinite(s[t]) && isfinite(d[t]);
        w[t] = ok ? 1.0f / (s[t] * s[t]) : 0.0f;
    }
}

// A bootstrap replica (r >= 0) of galaxy g: every pixel weight is multiplied
// by a Poisson(1) deviate drawn from Philox4x32-10 keyed by (k0, k1), counter
// {pixel / 4, g, r, 1}, word pixel mod 4 (pixel: row-major index in the
// cutout).  r < 0: the plain weights.
struct BootArgs {
    uint32_t k0, k1;
    int g, r;
};

// Poisson(1) multipliers of the four consecutive pixels pix0 .. pix0 + 3.
__device__ inline void boot_weights(const BootArgs &bt, int64_t pix0, float (&m)[4])
{
    const uint32_t q0 = (uint32_t)(pix0 >> 2), off = (uint32_t)(pix0 & 3);
    const U4 a = philox4x32_10(U4{q0, (uint32_t)bt.g, (uint32_t)bt.r, 1u}, bt.k0, bt.k1);
    U4 b = a;
    if (off != 0) b = philox4x32_10(U4{q0 + 1u, (uint32_t)bt.g, (uint32_t)bt.r, 1u}, bt.k0, bt.k1);
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) m[t] = (float)poisson1(w[off + t]);
}

// ---------------------------------------------------------------- helpers
// A fit that needs many trials (up to 100, against ten for most) or has many
// tiles outlives the rest of its launch: 2,048 cutouts of 48-256 px on 256
// workgroups kept one workgroup busy for 220 ms, the others for 82 on
// average.  A workgroup that finds the queue empty therefore helps the fits
// still running, tile by tile: it takes the next tile of an evaluation, makes
// its convolved planes and leaves them in memory; the fit's own workgroup (the
// owner) takes tiles too and adds the products of all of them itself, in tile
// order, so a thread's FP32 sums see the same values in the same order and the
// results are the same bits with any number of helpers.
//
// An owner that sees idle workgroups claims one of kHelpSlots slots for the
// rest of its fit.  Per evaluation it writes the prologue's result (scalars
// and window tables) into the slot and opens a ticket {epoch, tiles, next};
// who adds one to `next` has that tile.  A tile's planes go to entry
// tile % kHelpRing of the slot, marked with help_seq(epoch, tile); the owner
// frees entries by advancing `added`.  The tile the owner waits for is held by
// a running workgroup, whose entry is free, so every wait ends; each is bounded
// by spin_limit all the same: past it the owner makes the tile itself and
// leaves the slot for good (a late helper can then only write to that slot).
// A helper leaves, and is no longer counted, when no fit ended and it found no
// tile for idle_limit, and when the running fits have fewer tiles than there
// are helpers: that gives its CU to the kernels of other streams (1,024 fits
// of 64 x 64, one image batch on another stream: done after 3.3 ms without
// helpers, 7.3 with all of them kept, 3.6 now; the fits 13.2, 7.2 and 7.4 ms).
// The board is zeroed before every launch; slots past n_slots are never used.
constexpr int kHelpSlots = 64;
constexpr int kHelpRing = 16;

struct HelpSlot {
    int owner;                    // 1: claimed
    int epoch;                    // of the last evaluation shared
    int src;                      // galaxy
    int added;                    // tiles of this evaluation the owner has added
    int seq[kHelpRing];
    int pad[12];
};
struct HelpBoard {                // the first six words: gm_help_counts
    int idle;                     // helpers
    int done;                     // queue entries finished
    int turned, left;             // workgroups that turned helpers; that left before the last fit's end
    int tiles, lost;              // tiles made by helpers; evaluations that went on without one
    int pad[10];
    unsigned long long ticket[kHelpSlots];      // epoch << 32 | tiles << 16 | next
    HelpSlot slot[kHelpSlots];
};

enum { HELP_NONE = 0, HELP_OWNER, HELP_HELPER };
enum { TILE_SUM = 0, TILE_STORE, TILE_LOAD };     // make + add, make + leave in memory, read + add

// A workgroup's part in a shared evaluation (wave-uniform).
struct HelpState {
    HelpBoard *board = nullptr;
    char *base = nullptr;         // the slots' memory
    int64_t stride = 0, limit = 0;
    int n_slots = 0, n_entries = 0;
    int role = HELP_NONE;
    int slot = -1;
    int epoch = 0;
    int tile = 0;                 // HELP_HELPER: the tile it took
    __device__ char *buf() const { return base + slot * stride; }
};

template <typename T>
__device__ inline T agent_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void agent_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// This wave's stores have reached the memory that all dies see (agent-scope
// stores write through).  What helpers and owners hand over is written and
// read by agent-scope accesses alone, stores_done and a barrier before the
// mark that publishes it: no release or acquire, whose L2 write-back and
// invalidation would hit every workgroup of the die (with them, 2,048 fits of
// 64 x 64 ran 12% slower helped than alone).
__device__ inline void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ inline int help_count(int *p, int n)
{
    return __hip_atomic_fetch_add(p, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int help_seq(int epoch, int tile) { return (epoch << 11) | (tile + 1); }
__device__ inline unsigned long long help_take(unsigned long long *ticket)
{
    return __hip_atomic_fetch_add(ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The part of EvalShared that the prologue fills (all but nacc).
template <class F>
__host__ __device__ constexpr size_t help_head_bytes()
{
    return sizeof(EvalShared<F>) - sizeof(double) * NWAVE * (F::P + F::P * (F::P + 1) / 2);
}
// Bytes of one ring entry (a tile's planes) and of one slot's memory.
template <class F>
__host__ __device__ constexpr size_t help_entry_bytes()
{
    return (size_t)NT * (4 * sizeof(double) + (F::NPL - 1) * 4 * sizeof(float));
}
template <class F>
__host__ __device__ constexpr size_t help_slot_bytes()
{
    return ((help_head_bytes<F>() + 255) & ~(size_t)255) + kHelpRing * help_entry_bytes<F>();
}

// One strip's values to or from a ring entry, as 8-byte words of coalesced
// agent-scope accesses (they reach the memory that all dies see).
template <class F, bool STORE>
__device__ inline void help_strip(char *buf, int tile, double (&acc0)[4], float (&acc)[F::NPL][4])
{
    unsigned long long *e = reinterpret_cast<unsigned long long *>(
        buf + ((help_head_bytes<F>() + 255) & ~(size_t)255) + (size_t)(tile % kHelpRing) * help_entry_bytes<F>());
    e += threadIdx.x;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (STORE) agent_store(e + t * NT, __builtin_bit_cast(unsigned long long, acc0[t]));
        else acc0[t] = __builtin_bit_cast(double, agent_load(e + t * NT));
    }
    e += 4 * NT;
#pragma unroll
    for (int q = 1; q < F::NPL; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            unsigned long long *w = e + (2 * (q - 1) + h) * NT;
            if (STORE) {
                agent_store(w, (unsigned long long)__float_as_uint(acc[q][2 * h]) |
                                   ((unsigned long long)__float_as_uint(acc[q][2 * h + 1]) << 32));
            } else {
                const unsigned long long v = agent_load(w);
                acc[q][2 * h] = __uint_as_float((unsigned)v);
                acc[q][2 * h + 1] = __uint_as_float((unsigned)(v >> 32));
            }
        }
}

// All threads: this workgroup's agent-scope stores so far, then *p = v.
template <typename T>
__device__ inline void help_publish(T *p, T v)
{
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) agent_store(p, v);
}

// Owner, all threads: a slot for this fit (kept until help_release).
template <class F>
__device__ inline bool help_claim(HelpState &hp, int *sh_help)
{
    if (hp.slot >= 0) return true;
    __syncthreads();
    if (threadIdx.x == 0) {
        int got = -1;
        for (int i = 0; i < 8 && got < 0; ++i) {
            const int k = (int)((blockIdx.x + 23 * i) % (unsigned)hp.n_slots);
            int free_ = 0;
            if (__hip_atomic_compare_exchange_strong(&hp.board->slot[k].owner, &free_, 1, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                got = k;
        }
        sh_help[0] = got;
        sh_help[1] = got >= 0 ? agent_load(&hp.board->slot[got].epoch) : 0;
    }
    __syncthreads();
    hp.slot = uniform(sh_help[0]);
    hp.epoch = uniform(sh_help[1]);
    return hp.slot >= 0;
}

// Owner, all threads, after the prologue: opens the evaluation's tickets.
template <class F>
__device__ inline void help_open(const EvalShared<F> &sh, HelpState &hp, int src, int ntiles)
{
    HelpSlot *hs = hp.board->slot + hp.slot;
    ++hp.epoch;
    unsigned long long *d = reinterpret_cast<unsigned long long *>(hp.buf());
    const unsigned long long *e = reinterpret_cast<const unsigned long long *>(&sh);
    for (int i = threadIdx.x; i < (int)(help_head_bytes<F>() / 8); i += NT) agent_store(d + i, e[i]);
    if (threadIdx.x == 0) {
        agent_store(&hs->src, src);
        agent_store(&hs->epoch, hp.epoch);
        agent_store(&hs->added, 0);
    }
    help_publish(hp.board->ticket + hp.slot,
                 ((unsigned long long)(unsigned)hp.epoch << 32) | ((unsigned long long)ntiles << 16));
}

// Owner, thread 0: what to do for tile `next`, the first not yet added: add it
// from the ring (TILE_LOAD), make and add it (TILE_SUM), or make a later tile
// for the ring (TILE_STORE).  held: a tile taken while the ring had no room
// for it (-1: none); drained: no tiles left to take.
__device__ inline int help_next(HelpState &hp, int next, int ntiles, int &held, int &drained, int &tile, int &lost)
{
    HelpSlot *hs = hp.board->slot + hp.slot;
    agent_store(&hs->added, next);
    const int *mark = hs->seq + next % kHelpRing;
    const int want = help_seq(hp.epoch, next);
    tile = next;
    if (lost) return TILE_SUM;
    if (agent_load(mark) == want) return TILE_LOAD;
    if (held < 0 && !drained) {
        const int t = (int)(help_take(hp.board->ticket + hp.slot) & 0xffff);
        if (t < ntiles) held = t;
        else drained = 1;
    }
    if (held >= 0 && held < next + kHelpRing) {
        tile = held;
        held = -1;
        return tile == next ? TILE_SUM : TILE_STORE;
    }
    const int64_t t0 = wall_clock64();
    while (agent_load(mark) != want) {
        if (wall_clock64() - t0 > hp.limit) {
            lost = 1;
            agent_store(hp.board->ticket + hp.slot, 0ull);
            help_count(&hp.board->lost, 1);
            return TILE_SUM;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    return TILE_LOAD;
}

// Helper, wave 0: takes a tile of some open evaluation into hp; false when
// every fit has ended, when the fits still running have work for fewer helpers
// (keep for each), or when no fit ended and no tile was found for idle_limit.
__device__ inline bool help_find(HelpState &hp, int n_entries, int keep, int64_t idle_limit)
{
    static_assert(kHelpSlots == 64, "one lane per slot");
    HelpBoard *bd = hp.board;
    const int lane = threadIdx.x & 63;
    const int turn = (int)(blockIdx.x & 63);
    int64_t t0 = wall_clock64();
    int seen = -1;
    for (;;) {
        const int done = uniform(agent_load(&bd->done));
        if (done >= n_entries) return false;
        const int64_t now = wall_clock64();
        if (done != seen) {
            seen = done;
            t0 = now;
        } else if (now - t0 > idle_limit) {
            if (lane == 0) {
                help_count(&bd->idle, -1);
                help_count(&bd->left, 1);
            }
            return false;
        }
        // lane l looks at slot (l + turn) mod 64, so that helpers spread
        const int k = (lane + turn) & 63;
        const unsigned long long tk = agent_load(bd->ticket + k);
        const unsigned long long open = __ballot((int)(tk & 0xffff) < (int)((tk >> 16) & 0xffff));
        if (open) {
            const int at = (__ffsll(open) - 1 + turn) & 63;
            unsigned long long got = 0;
            if (lane == 0) got = help_take(bd->ticket + at);
            const int lo = uniform((int)(unsigned)got), hi = uniform((int)(unsigned)(got >> 32));
            if ((lo & 0xffff) < ((lo >> 16) & 0xffff)) {
                hp.slot = at;
                hp.epoch = hi;
                hp.tile = lo & 0xffff;
                return true;
            }
        } else {
            const int idle = uniform(agent_load(&bd->idle));
            const int64_t use = (int64_t)keep * (n_entries - done);
            if (idle > use) {
                int go = 0;
                if (lane == 0) {
                    go = help_count(&bd->idle, -1) > use;
                    help_count(go ? &bd->left : &bd->idle, 1);
                }
                if (uniform(go)) return false;
            }
            // 0.4 us, or 3.5 to 14 with more helpers: hundreds of idle workgroups looking more often
            // slow the others' accesses, a few looking less often leave tiles waiting
            if (idle <= 32) __builtin_amdgcn_s_sleep(16);
            else
                for (int z = 0; z < min(4, 1 + idle / 64); ++z) __builtin_amdgcn_s_sleep(127);
        }
    }
}

// One model evaluation at u (LDS): chi^2, g = J^T W r and A = J^T W J
// (internal LM variables), written to out_chi2/out_g/out_A (LDS, A full
// P x P).  All threads of the workgroup call it.
//
// A team of tsize workgroups shares one evaluation: the workgroup of rank
// trank takes the tiles whose row-major index is trank modulo tsize, and its
// outputs are the partial sums over those tiles (tsize = 1: the whole image).
//
// With helpers (hp.role) the tiles of the image are shared as described above;
// a helper makes one tile's planes and returns.
template <class F, int KT, int NG>
__device__ __forceinline__ void evaluate(const double *u, const ModelArgs &ma, const BatchArgs &ba, const Meta &me,
                                         EvalShared<F> &sh, float *planes, double *out_chi2, double *out_g,
                                         double *out_A, const BootArgs &bt = BootArgs{0u, 0u, 0, -1}, int trank = 0,
                                         int tsize = 1, HelpState *hp = nullptr, int *sh_help = nullptr, int src = 0)
{
    constexpr int P = F::P;
    constexpr int NR = 1 + P + P * (P + 1) / 2;
    const int H = me.h, W = me.w, K = KT > 0 ? KT : me.k;
    const int tid = threadIdx.x;
    const int nty = (H + TILE - 1) / TILE, ntx = (W + TILE - 1) / TILE;
    const int ntiles = nty * ntx;
    const float *psl = stage_psf<F, NG>(planes, ba.psf + uniform64(me.psf_off), K);
    int role = hp ? hp->role : HELP_NONE;
    if (role == HELP_HELPER) {
        const unsigned long long *d = reinterpret_cast<const unsigned long long *>(hp->buf());
        unsigned long long *e = reinterpret_cast<unsigned long long *>(&sh);
        for (int i = tid; i < (int)(help_head_bytes<F>() / 8); i += NT) e[i] = agent_load(d + i);
        __syncthreads();
    } else {
        // a fit of several tiles asks for helpers when there is one for every
        // four running fits (512 bulge + disk fits of 128 x 128: 60 ms, with one for
        // every fit 63, for every sixteen 60; 256 of 64-128 px at a side of 31: 36, 38, 36)
        if (hp && hp->board && tid == NT - 1) {
            const int running = hp->n_entries - agent_load(&hp->board->done);
            sh_help[0] = ntiles > 1 && 4 * agent_load(&hp->board->idle) >= running;
        }
        eval_prologue<F>(u, ma, H, W, sh, planes);
        if (hp && hp->board && uniform(sh_help[0]) > 0) {
            role = help_claim<F>(*hp, sh_help) ? HELP_OWNER : HELP_NONE;
            if (role == HELP_OWNER) help_open<F>(sh, *hp, src, ntiles);
        }
    }
    const cfloat *psf = (const cfloat *)(ba.psf + uniform64(me.psf_off));
    // Per-thread partial sums: chi^2 in FP64 (it decides accept/reject), g and
    // A in FP32 over at most FLUSH_TILES tiles (64 pixels), then FP64.
    double c2 = 0.0;
    float red[NR - 1];
#pragma unroll
    for (int q = 0; q < NR - 1; ++q) red[q] = 0.0f;
    int r, cg;
    strip_of(tid, K, r, cg);
    const int lane = tid & 63, wave = tid >> 6;
    const int mine = (ntiles - trank + tsize - 1) / tsize;        // tiles of this workgroup
    const bool flushes = mine > FLUSH_TILES;                      // uniform over the workgroup
    if (flushes && lane == 0)
        for (int q = 0; q < NR - 1; ++q) sh.nacc[wave][q] = 0.0;
    int since_flush = 0;
    int next = trank;                                             // the first tile not yet added
    int held = -1, drained = 0, lost = 0;                         // thread 0: help_next
    while (next < ntiles) {
        int ti = next, mode = TILE_SUM;
        if (role == HELP_OWNER) {
            __syncthreads();
            if (tid == 0) {
                sh_help[1] = help_next(*hp, next, ntiles, held, drained, sh_help[0], lost);
                sh_help[2] = lost;
            }
            __syncthreads();
            ti = uniform(sh_help[0]);
            mode = uniform(sh_help[1]);
        } else if (role == HELP_HELPER) {
            ti = hp->tile;
            mode = TILE_STORE;
        }
        const int ty = ti / ntx, tx = ti - ty * ntx;
        const int ti0 = ty * TILE, tj0 = tx * TILE;
        double acc0[4];
        float acc[F::NPL][4];
        if (mode != TILE_LOAD) tile_planes<F, KT, NG>(sh, planes, H, W, K, ti0, tj0, psf, psl, r, cg, acc0, acc);
        if (mode == TILE_STORE) {
            HelpSlot *hs = hp->board->slot + hp->slot;
            if (role == HELP_HELPER) {
                // room in the ring: tile - kHelpRing has been added
                if (tid == 0) {
                    const int64_t t0 = wall_clock64();
                    int ok = 1;
                    while (agent_load(&hs->added) <= ti - kHelpRing && ok)
                        if (wall_clock64() - t0 > hp->limit) ok = 0;
                    sh_help[1] = ok;
                }
                __syncthreads();
                if (uniform(sh_help[1]) == 0) return;
            }
            help_strip<F, true>(hp->buf(), ti, acc0, acc);
            help_publish(hs->seq + ti % kHelpRing, help_seq(hp->epoch, ti));
            if (role == HELP_HELPER) {
                if (tid == 0) ++sh_help[3];
                return;
            }
            continue;
        }
        if (mode == TILE_LOAD) help_strip<F, false>(hp->buf(), ti, acc0, acc);
        next += tsize;
        if (since_flush == FLUSH_TILES) {
            // the FP32 partials of the last FLUSH_TILES tiles into the wave's FP64 sums
#pragma unroll
            for (int q = 0; q < NR - 1; ++q) {
                const double v = strip_sum((double)red[q], K);
                if (lane == 0) sh.nacc[wave][q] += v;
                red[q] = 0.0f;
            }
            since_flush = 0;
        }
        ++since_flush;
        const int i = ti0 + r;
        if (i < H) {
            float bw[4] = {1.0f, 1.0f, 1.0f, 1.0f};
            if (bt.r >= 0) boot_weights(bt, (int64_t)i * W + tj0 + 4 * cg, bw);
            float dv[4], wv[4];
            strip_weights(ba, me.img_off + (int64_t)i * W, tj0 + 4 * cg, W, dv, wv);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int j = tj0 + 4 * cg + t;
                if (j >= W) continue;
                const float d = dv[t];
                const float wgt = wv[t] * bw[t];
                if (wgt == 0.0f) continue;
                const double pdx = ((double)j + 0.5) - 0.5 * W, pdy = 0.5 * H - ((double)i + 0.5);
                const double res = (double)d - (acc0[t] + F::sky_at(sh.prep, pdx, pdy));
                c2 = fma((double)wgt * res, res, c2);
                const float wr = wgt * (float)res;
                const float fdx = (float)pdx, fdy = (float)pdy;
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    const float Jk = jac_at<F>(k, t, acc0, acc, fdx, fdy);
                    red[k] = fmaf(wr, Jk, red[k]);
                    const float wj = wgt * Jk;
#pragma unroll
                    for (int l = 0; l <= k; ++l) {
                        const float Jl = jac_at<F>(l, t, acc0, acc, fdx, fdy);
                        red[P + k * (k + 1) / 2 + l] = fmaf(wj, Jl, red[P + k * (k + 1) / 2 + l]);
                    }
                }
            }
        }
    }
    if (role == HELP_OWNER && uniform(sh_help[2]) != 0) {
        hp->board = nullptr;          // a tile never came: no more helpers for this fit, the slot stays claimed
        hp->slot = -1;
    }
    // Fixed-order reduction in FP64 through the idle plane buffer (after the last
    // tile's barrier), in the order of strip_sum and then the waves: the FP32
    // partials of as many sums as fit are written one row of NT floats per sum;
    // a thread then adds the two strip rows of one of the four terms of a
    // wave's sum, and another the four terms of each wave and the waves.
    double *terms = reinterpret_cast<double *>(planes);           // [sum of the chunk][wave][4]
    constexpr int QB = NWAVE * 4 * (int)sizeof(double) + NT * (int)sizeof(float);
    const int chunk = min(NR - 1, (int)(lds_main_bytes<F, NG>(K) / QB));
    const bool gap4 = strip_gap(region_wp(K)) == 4;
    {
        const double v = strip_sum(c2, K);
        if (lane == 0) sh.c2[wave] = v;
    }
#pragma unroll 1
    for (int q0 = 0; q0 < NR - 1; q0 += chunk) {
        const int n = min(chunk, NR - 1 - q0);
        float *rows = reinterpret_cast<float *>(terms + chunk * NWAVE * 4);
#pragma unroll
        for (int q = 0; q < NR - 1; ++q)
            if (q >= q0 && q < q0 + n) rows[(q - q0) * NT + tid] = red[q];
        __syncthreads();
        for (int t = tid; t < n * NWAVE * 4; t += NT) {
            const int i = t & 3, w = (t >> 2) & (NWAVE - 1), q = t / (NWAVE * 4);
            const float *p = rows + q * NT + 64 * w + (gap4 ? 16 * (i >> 1) + 32 * (i & 1) : 8 * i);
            terms[t] = strip_row(p + (gap4 ? 8 : 32)) + strip_row(p);
        }
        __syncthreads();
        for (int q = tid; q < n; q += NT) {
            double s = 0.0;
            for (int w = 0; w < NWAVE; ++w) {
                const double *t4 = terms + (q * NWAVE + w) * 4;
                double v = ((t4[0] + t4[1]) + t4[2]) + t4[3];
                if (flushes) v = sh.nacc[w][q0 + q] + v;
                s = w == 0 ? v : s + v;
            }
            const int e = q0 + q;
            if (e < P) {
                out_g[e] = s;
            } else {
                int k = 0;
                while ((k + 1) * (k + 2) / 2 <= e - P) ++k;
                const int l = e - P - k * (k + 1) / 2;
                out_A[k * P + l] = s;
                out_A[l * P + k] = s;
            }
        }
        __syncthreads();
    }
    if (tid == 0) *out_chi2 = ((sh.c2[0] + sh.c2[1]) + sh.c2[2]) + sh.c2[3];
    __syncthreads();
}

// ---------------------------------------------------------------- small FP64 algebra (one thread)
// Cholesky L L^T = M of a P x P matrix; returns false if not positive definite.
template <int P>
__device__ bool chol(const double *M, double *L)
{
    for (int i = 0; i < P * P; ++i) L[i] = 0.0;
    for (int j = 0; j < P; ++j) {
        double d = M[j * P + j];
        for (int k = 0; k < j; ++k) d -= L[j * P + k] * L[j * P + k];
        if (!(d > 0.0) || !isfinite(d)) return false;
        double lj = sqrt(d);
        L[j * P + j] = lj;
        for (int i = j + 1; i < P; ++i) {
            double s = M[i * P + j];
            for (int k = 0; k < j; ++k) s -= L[i * P + k] * L[j * P + k];
            L[i * P + j] = s / lj;
        }
    }
    return true;
}

template <int P>
__device__ void chol_solve(const double *L, const double *b, double *x)
{
    double y[P];
    for (int i = 0; i < P; ++i) {
        double s = b[i];
        for (int k = 0; k < i; ++k) s -= L[i * P + k] * y[k];
        y[i] = s / L[i * P + i];
    }
    for (int i = P - 1; i >= 0; --i) {
        double s = y[i];
        for (int k = i + 1; k < P; ++k) s -= L[k * P + i] * x[k];
        x[i] = s / L[i * P + i];
    }
}

template <int P>
__device__ void chol_inverse(const double *L, double *inv)
{
    for (int j = 0; j < P; ++j) {
        double e[P], col[P];
        for (int i = 0; i < P; ++i) e[i] = (i == j) ? 1.0 : 0.0;
        chol_solve<P>(L, e, col);
        for (int i = 0; i < P; ++i) inv[i * P + j] = col[i];
    }
}

// Fixed parameters: their rows and columns of A are replaced by the identity
// and their gradient by 0, so that they never move.
template <int P>
__device__ void project_fixed(const int *freev, double *A, double *g)
{
    for (int k = 0; k < P; ++k) {
        if (freev[k]) continue;
        for (int l = 0; l < P; ++l) {
            A[k * P + l] = 0.0;
            A[l * P + k] = 0.0;
        }
        A[k * P + k] = 1.0;
        g[k] = 0.0;
    }
}

// Bounds of the LM variables (natural units: centres inside the cutout,
// scales in [0.1, 2 max(H, W)] px, Sersic n in [0.2, 10], q in [0.05, 20]).

// Canonical form of every component: q > 1 -> (1/q, scale * q, theta + pi/2),
// then theta wrapped into [0, pi).  u in internal layout; natural output.
template <class F>
__device__ __forceinline__ void canonical_nat(const double *u, const int *freev, double *nat)
{
    for (int k = 0; k < F::P; ++k) nat[k] = u_to_nat(F::kind(k), u[k]);
    for (int c = 0; c < F::NCAN; ++c) {
        int iq, ith, is0, is1;
        F::canon(c, iq, ith, is0, is1);
        if (freev[iq] && freev[ith] && nat[iq] > 1.0) {
            double qo = nat[iq];
            nat[iq] = 1.0 / qo;
            if (is0 >= 0) nat[is0] *= qo;
            if (is1 >= 0) nat[is1] *= qo;
            nat[ith] += 90.0;
        }
        if (freev[ith]) {
            double pa = fmod(nat[ith], 180.0);
            if (pa < 0.0) pa += 180.0;
            if (pa >= 180.0) pa -= 180.0;
            nat[ith] = pa;
        }
    }
}

// Covariance errors of a fit, sqrt(diag (J^T W J)^-1) (Sec. 5.2), from the
// normal matrix of the last accepted evaluation (J^T W J at u), in natural
// units of the canonical form written by canonical_nat.  Where that form
// flips a component (q -> 1/q, each scale s -> s q, theta -> theta + pi/2),
// the model image is unchanged, so the Jacobian in the canonical variables is
// J Phi^-1 with Phi the Jacobian of the flip in the LM variables (ln s' =
// ln s + ln q, q' = 1/q) and the covariance becomes Phi (J^T W J)^-1 Phi^T:
// the errors gm_param_errors computes at the canonical parameters, without
// another evaluation.  Fixed slots have identity rows (as in the error
// kernel); a matrix that is not positive definite gives NaN.  One thread,
// every array in LDS and every loop rolled, so that it adds no registers to
// the fit's loops; scratch: 3 P^2 + 2 P doubles.  A is overwritten.
template <class F>
__device__ __forceinline__ void fit_errors(double *A, double *g, const double *u, const int *freev,
                                           const ModelArgs &ma, double *err, double *scratch)
{
    constexpr int P = F::P;
    double *L = scratch, *inv = L + P * P, *phi = inv + P * P, *nat = phi + P * P, *y = nat + P;
    project_fixed<P>(freev, A, g);
    // Cholesky A = L L^T
    bool ok = true;
#pragma unroll 1
    for (int j = 0; j < P && ok; ++j) {
        double d = A[j * P + j];
#pragma unroll 1
        for (int k = 0; k < j; ++k) d -= L[j * P + k] * L[j * P + k];
        if (!(d > 0.0) || !isfinite(d)) {
            ok = false;
            break;
        }
        const double lj = sqrt(d);
        L[j * P + j] = lj;
#pragma unroll 1
        for (int i = j + 1; i < P; ++i) {
            double t = A[i * P + j];
#pragma unroll 1
            for (int k = 0; k < j; ++k) t -= L[i * P + k] * L[j * P + k];
            L[i * P + j] = t / lj;
        }
    }
    if (!ok) {
#pragma unroll 1
        for (int k = 0; k < P; ++k)
            if (ma.col[k] >= 0) err[ma.col[k]] = NAN;
        return;
    }
    // inverse, column by column: L y = e_j, then L^T x = y
#pragma unroll 1
    for (int j = 0; j < P; ++j) {
#pragma unroll 1
        for (int i = 0; i < P; ++i) {
            double t = (i == j) ? 1.0 : 0.0;
#pragma unroll 1
            for (int k = 0; k < i; ++k) t -= L[i * P + k] * y[k];
            y[i] = t / L[i * P + i];
        }
#pragma unroll 1
        for (int i = P - 1; i >= 0; --i) {
            double t = y[i];
#pragma unroll 1
            for (int k = i + 1; k < P; ++k) t -= L[k * P + i] * inv[k * P + j];
            inv[i * P + j] = t / L[i * P + i];
        }
    }
    // Phi: identity, with the flip's rows for components canonical_nat flips
#pragma unroll 1
    for (int k = 0; k < P * P; ++k) phi[k] = (k % (P + 1) == 0) ? 1.0 : 0.0;
#pragma unroll 1
    for (int c = 0; c < F::NCAN; ++c) {
        int iq, ith, is0, is1;
        F::canon(c, iq, ith, is0, is1);
        const double q = u[iq];
        if (freev[iq] && freev[ith] && q > 1.0) {
            phi[iq * P + iq] = -1.0 / (q * q);
            if (is0 >= 0) phi[is0 * P + iq] = 1.0 / q;
            if (is1 >= 0) phi[is1 * P + iq] = 1.0 / q;
        }
    }
    canonical_nat<F>(u, freev, nat);
    // diag(Phi inv Phi^T)
#pragma unroll 1
    for (int a = 0; a < P; ++a) {
        if (ma.col[a] < 0) continue;
        double v = 0.0;
#pragma unroll 1
        for (int k = 0; k < P; ++k) {
            if (phi[a * P + k] == 0.0) continue;
            double t = 0.0;
#pragma unroll 1
            for (int l = 0; l < P; ++l) t += inv[k * P + l] * phi[a * P + l];
            v += phi[a * P + k] * t;
        }
        err[ma.col[a]] = sqrt(v) * fabs(dnat_du(F::kind(a), nat[a]));
    }
}

// ---------------------------------------------------------------- LM kernel
template <class F>
struct LMShared {
    double u[F::P], ut[F::P], g[F::P], gt[F::P], A[F::P * F::P], At[F::P * F::P];
    double Dg[F::P], sig[F::P], un[F::P];        // un: the damped step's point
    double chi2, chi2t, lambda;
    int freev[F::P];
    int t, status, fresh, apd, action, max_iter;
    int damped;               // the damped step: 1 factorised, 2 below the tolerance
    int gal;
    int tok;                  // team: the last wait ended in time
    int help[4];              // owner: a helper to be had, then tile / mode / lost of the next step;
                              // helper: slot / epoch / tile taken / tiles made
};

struct FitArgs {
    const int *order;
    const int *active;        // nullable: galaxies with active[g] == 0 are skipped
    int n_gal;
    int *queue;
    double *params, *chi2;
    int *niter, *status;
    double *err;              // nullable: covariance errors at the fit [n_gal][p]
    int max_iter;
    double lambda0, tol;
    // Refit (nullable refit_start): a galaxy whose fit from params ends other
    // than CONVERGED within first_max_iter trials, or whose valid[g] is 0 (its
    // params are not a usable start), is fitted again, at once and by the same
    // workgroup, from refit_start[g] with max_iter trials; niter counts the
    // trials of both fits and refit_code[g] (nullable) is 0 (first fit), 1
    // (unusable start) or 2 (refitted).
    const double *refit_start;
    const int *valid;
    int *refit_code;
    int first_max_iter;
    // Bootstrap (n_boot > 0): fit index i is replica i % n_boot of galaxy
    // i / n_boot (BootArgs, key (boot_k0, boot_k1)); n_gal counts fit indices.
    int n_boot;
    uint32_t boot_k0, boot_k1;
    // Teams (nullable items): queue entry i is items[i] instead of order[i];
    // n_gal then counts the entries.  A fit with team size G > 1 is served by
    // G workgroups through its TeamCtl (ctl[team]) and its G partial-sum
    // slots (part + team * part_stride + rank * NR); spin_limit bounds every
    // wait of a team member, in wall-clock ticks.
    const struct TeamItem *items;
    struct TeamCtl *ctl;
    double *part;
    int64_t part_stride;
    int64_t spin_limit;
    // Helpers (nullable; one workgroup per fit only): HelpBoard.
    struct HelpBoard *help;
    char *help_buf;
    int64_t help_stride;      // bytes of help_buf per slot
    int64_t idle_limit;       // helpers' wait for work
    int help_slots, help_keep;
    int grid_items;           // workgroups worth launching (at least the queue entries)
};

enum { ACT_EVAL = 0, ACT_RETRY = 1, ACT_DONE = 2 };

// ---------------------------------------------------------------- teams of workgroups
// A fit served by G workgroups: the leader (rank 0) runs the LM, and each
// evaluation is shared by the team -- the leader publishes the point (its
// LM variables and the command ACT_EVAL, epoch by epoch), every member
// evaluates its tiles and delivers its partial sums (chi^2, g, the lower
// triangle of A in FP64), the leader adds the G partials in rank order (a
// fixed order: results do not depend on timing) and takes the LM step.  The
// leader ends the team with ACT_DONE.  All G workgroups hold their queue
// entries at once (consecutive entries of the persistent grid, which is never
// smaller than a team), so every wait ends; each wait is nonetheless bounded
// by spin_limit, after which the fit ends with GM_ST_TEAM_TIMEOUT.
struct TeamItem {
    int32_t fit, rank, size, team;
};

struct TeamCtl {
    int cmd;                  // commands published so far (the epoch of the last one + 1)
    int action;               // the last command: ACT_EVAL or ACT_DONE
    int arrive;               // partial sums delivered so far, over all epochs
    int pad;
    double u[MAXP];           // the point of the last ACT_EVAL
};

__device__ inline int team_load(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}

// Thread 0: wait until *p >= target (acquire) or the limit passes; true if reached.
__device__ inline bool team_wait(const int *p, int target, int64_t limit)
{
    const int64_t t0 = wall_clock64();
    while (team_load(p) < target) {
        if (wall_clock64() - t0 > limit) return false;
        __builtin_amdgcn_s_sleep(2);
    }
    return true;
}

// Entry q of the NR = 1 + P + P (P + 1) / 2 sums of an evaluation: chi^2, g,
// then A's lower triangle row by row.
template <int P>
__device__ inline double sum_entry(int q, double chi2, const double *g, const double *A)
{
    if (q == 0) return chi2;
    if (q <= P) return g[q - 1];
    int e = q - 1 - P, k = 0;
    while ((k + 1) * (k + 2) / 2 <= e) ++k;
    return A[k * P + (e - k * (k + 1) / 2)];
}

template <int P>
__device__ inline void set_entry(int q, double v, double *chi2, double *g, double *A)
{
    if (q == 0) {
        *chi2 = v;
    } else if (q <= P) {
        g[q - 1] = v;
    } else {
        int e = q - 1 - P, k = 0;
        while ((k + 1) * (k + 2) / 2 <= e) ++k;
        const int l = e - k * (k + 1) / 2;
        A[k * P + l] = v;
        A[l * P + k] = v;
    }
}

// All threads: this workgroup's partial sums (LDS) into its slot, made visible
// at device scope before thread 0 counts the delivery.
template <int P>
__device__ inline void team_deliver(TeamCtl *ctl, double *slot, double chi2, const double *g, const double *A)
{
    constexpr int NR = 1 + P + P * (P + 1) / 2;
    for (int q = threadIdx.x; q < NR; q += NT) slot[q] = sum_entry<P>(q, chi2, g, A);
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(&ctl->arrive, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- wave-parallel LM step
// Two waves run the LM bookkeeping between evaluations.  Lane r < P holds row
// r of the P x P normal matrix; the Cholesky factorisation is row-parallel
// (the pivot column is broadcast with readlane at every step), the triangular
// solves are computed by every lane from broadcast values, the columns of the
// inverse factor by a lane each.  Sums run in the same order as the textbook
// one-thread algorithm.

// L (lane r: row r) of M (lane r: row r, overwritten); false if M is not
// positive definite.  Column by column, each column's products taken from the
// rest of M at once: an element still sees them in increasing column order.
template <int P>
__device__ inline bool chol_rows(double (&m)[P], double (&l)[P], int lane)
{
#pragma unroll
    for (int j = 0; j < P; ++j) {
        const double d = lane_value(m[j], j);
        if (!(d > 0.0) || !isfinite(d)) return false;
        const double ljj = sqrt(d);
        l[j] = lane > j ? m[j] / ljj : (lane == j ? ljj : 0.0);
#pragma unroll
        for (int c = j + 1; c < P; ++c) m[c] -= l[j] * lane_value(l[j], c);
    }
    return true;
}

// x = (L L^T)^-1 b, with b and the result as wave-uniform arrays.
template <int P>
__device__ inline void chol_solve_rows(const double (&l)[P], const double (&b)[P], double (&x)[P])
{
    double y[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        double t = b[i];
#pragma unroll
        for (int k = 0; k < i; ++k) t -= lane_value(l[k], i) * y[k];
        y[i] = t / lane_value(l[i], i);
    }
#pragma unroll
    for (int i = P - 1; i >= 0; --i) {
        double t = y[i];
#pragma unroll
        for (int k = i + 1; k < P; ++k) t -= lane_value(l[i], k) * x[k];
        x[i] = t / lane_value(l[i], i);
    }
}

// diag((L L^T)^-1)_c = sum_i (L^-1)_ic^2 at lane c (column c of L^-1 by lane c).
template <int P>
__device__ inline double chol_inv_diag_lane(const double (&l)[P], int lane)
{
    double z[P], acc = 0.0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        double t = (i == lane) ? 1.0 : 0.0;
#pragma unroll
        for (int k = 0; k < i; ++k) t -= lane_value(l[k], i) * z[k];      // z[k] = 0 for k < c
        z[i] = t / lane_value(l[i], i);
        acc += z[i] * z[i];
    }
    return acc;
}

// v limited to [lo, hi] by comparisons: a NaN stays NaN (fmin/fmax would
// replace it by a bound), so a non-finite start or step gives a non-finite
// chi^2 and is never taken for a point inside the bounds.
__device__ inline double clamp_to(double v, double lo, double hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

// Bounds of the LM variables (internal units: ln of scales, n and a, radians).
template <class F>
__device__ inline double clamp_var(int k, double v, int H, int W)
{
    const double big = 2.0 * (H > W ? H : W);
    switch (F::kind(k)) {
    case KX0: return clamp_to(v, 0.0, (double)W);
    case KY0: return clamp_to(v, 0.0, (double)H);
    case KSCALE: return clamp_to(v, log(0.1), log(big));
    case KN: return clamp_to(v, log(0.2), log(10.0));
    case KQ: return clamp_to(v, 0.05, 20.0);
    case KBOX: return clamp_to(v, -0.9, 2.0);
    case KFA: return clamp_to(v, log(0.1), log(10.0));
    case KFB: return clamp_to(v, -1.0, 1.95);
    case KKAL: return clamp_to(v, log(0.5), log(10.0));
    default: return v;
    }
}

template <class F>
__device__ void clamp_u(double *u, int H, int W)
{
    for (int k = 0; k < F::P; ++k) u[k] = clamp_var<F>(k, u[k], H, W);
}

// Waves 0 and 1 (the others pass its one barrier by themselves: the function
// is out of line and saves registers in scratch on entry, 71 -> 44 MB written
// by 8,192 fits of 64 x 64): absorb the evaluation just
// made (the start point, or a trial: accept if chi^2 decreased, else raise the
// damping), then choose the next trial point or finish.
//   Start: A, g from the evaluation, fixed rows/columns replaced by the
//     identity and their gradient by 0; lambda = lambda0.
//   Stop test at every newly accepted state: the undamped Gauss-Newton step
//     A^-1 g in units of sigma_k = sqrt([A^-1]_kk) below tol -> CONVERGED
//     (while A is not positive definite: the damped step against
//     1/sqrt(D_kk)).
//   Trial: (A + lambda D) delta = g with D = diag(max(A_kk, 1e-12 max A_kk))
//     of the current accepted A; a failed factorisation raises lambda by 10
//     and counts the trial; lambda > 1e9 -> STALLED; max_iter trials ->
//     MAXITER.
// Waves 0 and 1 both absorb; wave 0 then factorises A (stop test) while wave 1
// factorises A + lambda D (trial), and after a barrier wave 0 writes the
// outcome.  (One wave doing both in turn: 10k cycles per step, now 6k.)
template <class F>
__device__ void lm_step(LMShared<F> &s, const FitArgs &fa, int H, int W)
{
    constexpr int P = F::P;
    const int wave = uniform((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const bool row = lane < P;
    const int r = row ? lane : 0;
    bool fv[P];
#pragma unroll
    for (int k = 0; k < P; ++k) fv[k] = s.freev[k] != 0;
    bool fr = false;
#pragma unroll
    for (int k = 0; k < P; ++k)
        if (k == r) fr = fv[k];
    int t = s.t, action = s.action, status = s.status, fresh = s.fresh, apd = s.apd;
    double lambda = s.lambda, chi2 = s.chi2;
    double a[P];
    double gr, ur = s.u[r], dgr = s.Dg[r], sgr = s.sig[r];
    bool newA = false, accepted = false;
    if (t < 0 || action == ACT_EVAL) {
        const double chi2t = s.chi2t;
        const bool take = t < 0 || (isfinite(chi2t) && chi2t < chi2);
        if (take) {
#pragma unroll
            for (int k = 0; k < P; ++k) a[k] = (fr && fv[k]) ? s.At[r * P + k] : (r == k ? 1.0 : 0.0);
            gr = fr ? s.gt[r] : 0.0;
            newA = true;
            chi2 = chi2t;
            if (t < 0) {
                t = 0;
                if (!isfinite(chi2)) {
                    status = GM_ST_NONFINITE;
                    action = ACT_DONE;
                }
            } else {
                accepted = true;
                ur = s.ut[r];
                lambda = fmax(lambda / 10.0, 1e-9);
                fresh = 1;
            }
        } else {
            lambda *= 10.0;
            if (lambda > 1e9) {
                status = GM_ST_STALLED;
                action = ACT_DONE;
            }
        }
    }
    if (!newA) {
#pragma unroll
        for (int k = 0; k < P; ++k) a[k] = s.A[r * P + k];
        gr = s.g[r];
    }
    if (action != ACT_DONE && t >= s.max_iter) {
        status = GM_ST_MAXITER;
        action = ACT_DONE;
    }
    const bool step = action != ACT_DONE;
    double utr = ur, gv[P];
    bool stop = false;
    if (step) {
        t += 1;
#pragma unroll
        for (int k = 0; k < P; ++k) gv[k] = lane_value(gr, k);
        if (fresh) {
            double drr = 0.0;
#pragma unroll
            for (int k = 0; k < P; ++k)
                if (k == r) drr = a[k];
            double amax = 0.0;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double dk = lane_value(drr, k);
                if (fv[k] && dk > amax) amax = dk;
            }
            dgr = fr ? (drr > 1e-12 * amax ? drr : 1e-12 * amax) : 1.0;
        }
    }
    if (wave == 1) {
        // the damped step; conv: its test against 1/sqrt(D_kk), for an A that is not positive definite
        if (step) {
            double m[P], l[P];
#pragma unroll
            for (int k = 0; k < P; ++k) m[k] = a[k] + (k == r ? lambda * dgr : 0.0);
            const bool ok = chol_rows<P>(m, l, lane);
            bool conv = false;
            if (ok) {
                double dv[P];
                chol_solve_rows<P>(l, gv, dv);
                const double sg = fresh ? 1.0 / sqrt(dgr) : sgr;
                double smax = 0.0;
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    const double q = fabs(dv[k]) / lane_value(sg, k);
                    if (!(q <= smax)) smax = q;
                }
                conv = smax < fa.tol;
                double dr = 0.0;
#pragma unroll
                for (int k = 0; k < P; ++k)
                    if (k == r) dr = dv[k];
                utr = clamp_var<F>(r, ur + (fr ? dr : 0.0), H, W);
            }
            if (row) s.un[r] = utr;
            if (lane == 0) s.damped = (ok ? 1 : 0) | (conv ? 2 : 0);
        }
        __syncthreads();
        return;
    }
    if (step && fresh) {
        double m[P], l[P];
#pragma unroll
        for (int k = 0; k < P; ++k) m[k] = a[k];
        apd = chol_rows<P>(m, l, lane) ? 1 : 0;
        if (apd) {
            double dv[P];
            sgr = sqrt(chol_inv_diag_lane<P>(l, lane));
            chol_solve_rows<P>(l, gv, dv);
            double dr = 0.0, smax = 0.0;
#pragma unroll
            for (int k = 0; k < P; ++k)
                if (k == lane) dr = dv[k];
            const double ratio = fabs(dr) / sgr;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double q = lane_value(ratio, k);
                if (!(q <= smax)) smax = q;
            }
            if (smax < fa.tol) {
                t -= 1;
                status = GM_ST_CONVERGED;
                action = ACT_DONE;
                stop = true;
            }
        } else {
            sgr = 1.0 / sqrt(dgr);
        }
        fresh = 0;
    }
    __syncthreads();
    bool proposed = false;
    if (step && !stop) {
        const int damped = uniform(s.damped);
        if (!(damped & 1)) {
            lambda *= 10.0;
            if (lambda > 1e9) {
                status = GM_ST_STALLED;
                action = ACT_DONE;
            } else {
                action = ACT_RETRY;
            }
        } else if (!apd && (damped & 2)) {
            t -= 1;
            status = GM_ST_CONVERGED;
            action = ACT_DONE;
        } else {
            utr = s.un[r];
            proposed = true;
            action = ACT_EVAL;
        }
    }
    if (row) {
        if (newA) {
#pragma unroll
            for (int k = 0; k < P; ++k) s.A[r * P + k] = a[k];
            s.g[r] = gr;
        }
        if (accepted) s.u[r] = ur;
        if (proposed) s.ut[r] = utr;
        s.Dg[r] = dgr;
        s.sig[r] = sgr;
    }
    if (lane == 0) {
        s.t = t;
        s.action = action;
        s.status = status;
        s.fresh = fresh;
        s.apd = apd;
        s.lambda = lambda;
        s.chi2 = chi2;
    }
}

// The evaluation just made will be taken (as in lm_step), it was not exact,
// and a derivative was NaN at a pixel in use, which the diagonal of its A
// shows.  Most trials with infinite derivatives, which throw a magnitude far
// out, are rejected by their chi^2 (512 bulge + disk fits of 128 x 128 took
// 63 ms instead of 56 with the exact convolution at once).
template <class F>
__device__ inline bool lm_spoilt(const LMShared<F> &s, int exact)
{
    const int k = min((int)(threadIdx.x & 63), F::P - 1);
    const double d = s.At[k * F::P + k];
    const bool take = isfinite(s.chi2t) && (s.t < 0 || s.chi2t < s.chi2);
    return !exact && take && __ballot(d != d) != 0;
}

template <class F>
__device__ __forceinline__ void load_u(LMShared<F> &s, const ModelArgs &ma, const double *params)
{
    for (int k = 0; k < F::P; ++k) {
        int c = ma.col[k];
        double nat = c >= 0 ? params[c] : ma.fixedv[k];
        s.u[k] = nat_to_u(F::kind(k), nat);
        s.freev[k] = c >= 0;
    }
}

// Workgroups per CU that the kernels' register allocation targets.  At two (at
// most 256 VGPRs per lane) one workgroup's profile evaluation, prologue and LM
// step overlap the other's convolution where the plane buffers of two fit in
// LDS (measured 1.38x faster Sersic fits at 64 x 64, PSF side 15), and the
// matrix instructions' accumulators stay in VGPRs: with more registers allowed
// the compiler puts them into AGPRs, with copies in the convolution loops.
// Most one-component fits meet this budget with a few spilled registers outside
// their loops; those with nine and ten variables (boxy, tilted sky, free King
// and Ferrer) spill 20 to 60 at a side of 15, some of them inside, and are
// faster so than with one workgroup per CU all the same (1,024 boxy fits of
// 64 x 64, eight trials: 4.8 -> 4.5 ms; tilted sky: 3.6 -> 2.95).  The two-component
// models' normal-equation accumulators do not fit.
template <class F>
__host__ __device__ constexpr int min_wg()
{
    return F::NCOMP != 1 ? 1 : 2;
}

// Team steps around the one evaluation site of lm_fit_kernel.
// Leader: publish the point s.ut of the epoch-th shared evaluation.
template <class F>
__device__ inline void team_publish(const LMShared<F> &s, TeamCtl *ctl, int epoch)
{
    const int tid = threadIdx.x;
    if (tid < F::P) ctl->u[tid] = s.ut[tid];
    __threadfence();
    __syncthreads();
    if (tid == 0) {
        ctl->action = ACT_EVAL;
        __hip_atomic_store(&ctl->cmd, epoch + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Member: wait for the leader's command of the epoch-th evaluation; s.action
// and (for ACT_EVAL) s.ut take it.  A wait past the spin limit reads as ACT_DONE.
template <class F>
__device__ inline void team_command(LMShared<F> &s, const TeamCtl *ctl, int epoch, int64_t limit)
{
    if (threadIdx.x == 0) {
        // the command's fields are read atomically (never through a cache of
        // uniform loads), after the acquire of cmd
        const bool got = team_wait(&ctl->cmd, epoch + 1, limit);
        const int act = got ? __hip_atomic_load(&ctl->action, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ACT_DONE;
        s.action = act;
        if (act == ACT_EVAL)
            for (int k = 0; k < F::P; ++k)
                s.ut[k] = __hip_atomic_load(&ctl->u[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
}

// Leader, after its own delivery: wait for the team's tsize deliveries of the
// epoch-th evaluation and add the partial sums in rank order into s.chi2t,
// s.gt, s.At.  False if they did not arrive within the limit.
template <class F>
__device__ inline bool team_collect(LMShared<F> &s, TeamCtl *ctl, const double *slots, int tsize, int epoch,
                                    int64_t limit)
{
    constexpr int P = F::P, NR = 1 + P + P * (P + 1) / 2;
    const int tid = threadIdx.x;
    if (tid == 0) s.tok = team_wait(&ctl->arrive, tsize * (epoch + 1), limit) ? 1 : 0;
    __syncthreads();
    const bool ok = uniform(s.tok) != 0;
    if (ok) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        for (int q = tid; q < NR; q += NT) {
            double v = slots[q];
            for (int r = 1; r < tsize; ++r) v += slots[(int64_t)r * NR + q];
            set_entry<P>(q, v, &s.chi2t, s.gt, s.At);
        }
    }
    __syncthreads();
    return ok;
}

// Persistent LM fits: each workgroup takes queue entries (a fit, or one rank
// of a team sharing a fit) until the queue is empty.  One workgroup, or the
// leader of a team, runs the LM of its fit (a fit from params, then possibly
// the refit from refit_start); members follow the leader's commands.  The
// model is evaluated at a single site for all three roles.
template <class F, int KT, int NG>
__global__ __launch_bounds__(NT, min_wg<F>()) void lm_fit_kernel(ModelArgs ma, BatchArgs ba, FitArgs fa)
{
    extern __shared__ float4 dyn_lds[];
    float *planes = reinterpret_cast<float *>(dyn_lds);
    __shared__ EvalShared<F> esh;
    __shared__ LMShared<F> s;
    constexpr int NR = 1 + F::P + F::P * (F::P + 1) / 2;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) s.gal = atomicAdd(fa.queue, 1);
        __syncthreads();
        const int qi = uniform(s.gal);
        HelpState hp;
        hp.board = fa.help;
        hp.base = fa.help_buf;
        hp.stride = fa.help_stride;
        hp.n_slots = fa.help_slots;
        hp.n_entries = fa.n_gal;
        hp.limit = fa.spin_limit;
        const bool helper = qi >= fa.n_gal;
        if (helper && !fa.help) break;
        int g = 0, trank = 0, tsize = 1, team = 0;
        if (helper) {
            hp.role = HELP_HELPER;
            if (tid == 0) {
                help_count(&fa.help->idle, 1);
                help_count(&fa.help->turned, 1);
                s.help[3] = 0;
            }
        } else if (fa.items) {
            const TeamItem it = fa.items[qi];
            g = uniform(it.fit);
            trank = uniform(it.rank);
            tsize = uniform(it.size);
            team = uniform(it.team);
        } else {
            g = uniform(fa.order[qi]);
        }
        if (!helper && fa.active && uniform(fa.active[g]) == 0) {
            if (fa.help && tid == 0) help_count(&fa.help->done, 1);
            __syncthreads();      // s.gal is rewritten by thread 0 next
            continue;
        }
        if (tid == 0) esh.exact = tsize > 1;
        int src = fa.n_boot > 0 ? g / fa.n_boot : g;
        const BootArgs bt{fa.boot_k0, fa.boot_k1, src, fa.n_boot > 0 ? g - src * fa.n_boot : -1};
        Meta me = ba.meta[src];
        const bool member = trank > 0;
        TeamCtl *ctl = tsize > 1 ? fa.ctl + team : nullptr;
        double *slots = tsize > 1 ? fa.part + (int64_t)team * fa.part_stride : nullptr;
        // phase 0: the fit from params; phase 1: the refit from refit_start
        const bool refit = fa.refit_start != nullptr;
        const int first = (!member && !helper && refit && fa.valid && uniform(fa.valid[g]) == 0) ? 1 : 0;
        int t0 = 0, phase = first, epoch = 0;
        bool phase_start = !member && !helper;
        for (;;) {
            if (helper) {
                if (tid < 64) {
                    const bool any = help_find(hp, fa.n_gal, fa.help_keep, fa.idle_limit);
                    if (tid == 0) {
                        s.action = any ? ACT_EVAL : ACT_DONE;
                        s.help[0] = hp.slot;
                        s.help[1] = hp.epoch;
                        s.help[2] = hp.tile;
                    }
                }
                __syncthreads();
                if (uniform(s.action) == ACT_DONE) break;
                hp.slot = uniform(s.help[0]);
                hp.epoch = uniform(s.help[1]);
                hp.tile = uniform(s.help[2]);
                src = uniform(agent_load(&fa.help->slot[hp.slot].src));
                me = ba.meta[src];
            }
            if (phase_start) {
                if (tid == 0) {
                    load_u<F>(s, ma, (phase ? fa.refit_start : fa.params) + (int64_t)g * ma.p);
                    clamp_u<F>(s.u, me.h, me.w);
                    for (int k = 0; k < F::P; ++k) s.ut[k] = s.u[k];
                    s.t = -1;             // -1: the next evaluation is the start point
                    s.status = GM_ST_MAXITER;
                    s.max_iter = (refit && phase == 0) ? fa.first_max_iter : fa.max_iter;
                    s.lambda = fa.lambda0;
                    s.fresh = 1;
                    s.apd = 0;
                    s.chi2 = 0.0;
                    s.action = ACT_EVAL;
                    for (int k = 0; k < F::P; ++k) {
                        s.Dg[k] = 1.0;
                        s.sig[k] = 1.0;
                    }
                }
                __syncthreads();
                phase_start = false;
            }
            if (member) team_command<F>(s, ctl, epoch, fa.spin_limit);
            const int act = uniform(s.action);
            if (act == ACT_DONE) {
                if (member) break;
                if (uniform(s.status) == GM_ST_TEAM_TIMEOUT || phase == 1) break;
                if (!refit || uniform(s.status) == GM_ST_CONVERGED) {
                    t0 = -1;          // no refit
                    break;
                }
                t0 = uniform(s.t);
                __syncthreads();      // every thread has read s before thread 0 reloads it
                phase = 1;
                phase_start = true;
                continue;
            }
            if (act == ACT_EVAL) {
                if (tsize > 1 && !member) team_publish<F>(s, ctl, epoch);
                // the evaluation site: the whole image, this rank's tiles of it, or one tile for its owner
                evaluate<F, KT, NG>(s.ut, ma, ba, me, esh, planes, &s.chi2t, s.gt, s.At, bt, trank, tsize,
                                    &hp, s.help, src);
                if (helper) {
                    __syncthreads();
                    continue;
                }
                if (tsize > 1) {
                    team_deliver<F::P>(ctl, slots + (int64_t)trank * NR, s.chi2t, s.gt, s.At);
                    if (!member && !team_collect<F>(s, ctl, slots, tsize, epoch, fa.spin_limit)) {
                        if (tid == 0) {
                            s.status = GM_ST_TEAM_TIMEOUT;
                            s.action = ACT_DONE;
                        }
                        __syncthreads();
                        continue;
                    }
                    ++epoch;
                } else if (lm_spoilt<F>(s, esh.exact)) {
                    __syncthreads();
                    if (tid == 0) esh.exact = 1;      // once more
                    continue;
                }
            }
            if (!member) {
                if (uniform(tid >> 6) < 2) lm_step<F>(s, fa, me.h, me.w);
                else __syncthreads();         // lm_step's barrier
                if (tid == 0) esh.exact = tsize > 1;
            }
            __syncthreads();
        }
        if (helper) {
            if (tid == 0) help_count(&fa.help->tiles, s.help[3]);
            break;
        }
        if (member) {
            __syncthreads();          // s.gal is rewritten by thread 0 next
            continue;
        }
        if (tid == 0 && fa.help) {
            if (hp.slot >= 0)
                agent_store(&fa.help->slot[hp.slot].owner, 0);
            help_count(&fa.help->done, 1);
        }
        if (tsize > 1 && tid == 0) {
            // end the team (epoch + 2 exceeds every epoch a member can be waiting for)
            ctl->action = ACT_DONE;
            __hip_atomic_store(&ctl->cmd, epoch + 2, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (uniform(s.status) == GM_ST_TEAM_TIMEOUT) t0 = -1;
        if (tid == 0) {
            double nat[F::P];
            canonical_nat<F>(s.u, s.freev, nat);
            double *out = fa.params + (int64_t)g * ma.p;
            for (int k = 0; k < F::P; ++k)
                if (ma.col[k] >= 0) out[ma.col[k]] = nat[k];
            fa.chi2[g] = s.chi2;
            fa.niter[g] = s.t + (t0 > 0 ? t0 : 0);
            fa.status[g] = s.status;
            if (fa.refit_code) fa.refit_code[g] = t0 < 0 ? 0 : (first ? 1 : 2);
            if (fa.err)
                fit_errors<F>(s.A, s.g, s.u, s.freev, ma, fa.err + (int64_t)g * ma.p,
                              reinterpret_cast<double *>(planes));
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- covariance errors
struct ErrArgs {
    const double *params;
    double *err, *cov;
    int n_gal;
};

template <class F, int KT, int NG>
__global__ __launch_bounds__(NT) void errors_kernel(ModelArgs ma, BatchArgs ba, ErrArgs ea)
{
    extern __shared__ float4 dyn_lds[];
    float *planes = reinterpret_cast<float *>(dyn_lds);
    __shared__ EvalShared<F> esh;
    __shared__ LMShared<F> s;
    constexpr int P = F::P;
    const int tid = threadIdx.x;
    for (int g = blockIdx.x; g < ea.n_gal; g += gridDim.x) {
        const Meta me = ba.meta[g];
        if (tid == 0) {
            load_u<F>(s, ma, ea.params + (int64_t)g * ma.p);
            esh.exact = 1;
        }
        __syncthreads();
        evaluate<F, KT, NG>(s.u, ma, ba, me, esh, planes, &s.chi2, s.g, s.A);
        if (tid == 0) {
            // thread-0 temporaries in the idle plane buffer
            double *L = reinterpret_cast<double *>(planes);
            double *inv = L + P * P;
            project_fixed<P>(s.freev, s.A, s.g);
            const int p = ma.p;
            double *err = ea.err + (int64_t)g * p;
            double *cov = ea.cov ? ea.cov + (int64_t)g * p * p : nullptr;
            if (chol<P>(s.A, L)) {
                chol_inverse<P>(L, inv);
                for (int a = 0; a < P; ++a) {
                    if (ma.col[a] < 0) continue;
                    double na = u_to_nat(F::kind(a), s.u[a]);
                    double sa = dnat_du(F::kind(a), na);
                    err[ma.col[a]] = sqrt(inv[a * P + a]) * fabs(sa);
                    if (cov)
                        for (int b = 0; b < P; ++b) {
                            if (ma.col[b] < 0) continue;
                            double nb = u_to_nat(F::kind(b), s.u[b]);
                            cov[ma.col[a] * p + ma.col[b]] = sa * inv[a * P + b] * dnat_du(F::kind(b), nb);
                        }
                }
            } else {
                for (int a = 0; a < p; ++a) err[a] = NAN;
                if (cov)
                    for (int a = 0; a < p * p; ++a) cov[a] = NAN;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- model image / Jacobian
struct TileItem {
    int32_t gal, ty, tx, pad;
};

struct ImageArgs {
    const TileItem *tiles;
    int n_tiles;
    const double *params;
    float *out;          // model (mode 0) or Jacobian (mode 1)
    int mode;            // 2: adjoint, per-tile partials of J^T gin into part
    const float *gin;    // mode 2: weights of the pixels (image layout)
    double *part;        // mode 2: [n_tiles][P] partial sums (internal variable order)
};

// Mode 0 needs the light plane alone, in the LDS of a kernel with a group per
// plane, so that more workgroups share a CU: 768 images of 40-160 px at a side
// of 21 3.2 -> 0.6 ms, one of 64 x 64 32.4 -> 24.2 us (with every plane made and
// thrown away).  Bound by the prologue and the profile.
template <class F>
constexpr int kLightGroups = F::NPL;

template <class F, int KT, int NG>
__global__ __launch_bounds__(NT, 2) void image_kernel(ModelArgs ma, BatchArgs ba, ImageArgs ia)
{
    extern __shared__ float4 dyn_lds[];
    float *planes = reinterpret_cast<float *>(dyn_lds);
    __shared__ EvalShared<F> esh;
    __shared__ double su[F::P];
    __shared__ double sdu[F::P];        // d u / d p (natural units)
    __shared__ int sfree[F::P];
    __shared__ double sv[NWAVE][F::P];
    constexpr int P = F::P;
    const int tid = threadIdx.x;
    for (int it = blockIdx.x; it < ia.n_tiles; it += gridDim.x) {
        const TileItem ti = ia.tiles[it];
        const int g = uniform(ti.gal);
        const Meta me = ba.meta[g];
        const int H = me.h, W = me.w, K = KT > 0 ? KT : me.k;
        if (tid == 0) {
            esh.exact = 1;
            const double *pp = ia.params + (int64_t)g * ma.p;
            for (int k = 0; k < P; ++k) {
                int c = ma.col[k];
                su[k] = nat_to_u(F::kind(k), c >= 0 ? pp[c] : ma.fixedv[k]);
                sdu[k] = 1.0 / dnat_du(F::kind(k), u_to_nat(F::kind(k), su[k]));
                sfree[k] = c >= 0;
            }
        }
        const float *psl = ia.mode == 0 ? stage_psf<F, kLightGroups<F>>(planes, ba.psf + uniform64(me.psf_off), K)
                                        : stage_psf<F, NG>(planes, ba.psf + uniform64(me.psf_off), K);
        __syncthreads();
        eval_prologue<F>(su, ma, H, W, esh, planes);
        const int ti0 = ti.ty * TILE, tj0 = ti.tx * TILE;
        int r, cg;
        strip_of(tid, K, r, cg);
        double acc0[4];
        float acc[F::NPL][4];
        const cfloat *psf = (const cfloat *)(ba.psf + uniform64(me.psf_off));
        if (ia.mode == 0) {         // the light alone
            fill_region<F, 0, 1, shift64<KT>()>(esh, planes, H, W, K, ti0, tj0);
            __syncthreads();
            conv64<KT>(planes, K, psf, psl, r, cg, acc0);
        } else {
            tile_planes<F, KT, NG>(esh, planes, H, W, K, ti0, tj0, psf, psl, r, cg, acc0, acc);
        }
        const int i = ti0 + r;
        double v[P];
#pragma unroll
        for (int k = 0; k < P; ++k) v[k] = 0.0;
        if (i < H) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int j = tj0 + 4 * cg + t;
                if (j >= W) continue;
                const int64_t pix = (int64_t)i * W + j;
                const double pdx = ((double)j + 0.5) - 0.5 * W, pdy = 0.5 * H - ((double)i + 0.5);
                const float fdx = (float)pdx, fdy = (float)pdy;
                if (ia.mode == 0) {
                    ia.out[me.img_off + pix] = (float)(acc0[t] + F::sky_at(esh.prep, pdx, pdy));
                } else if (ia.mode == 1) {
                    float *jo = ia.out + (int64_t)ma.p * me.img_off;
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        if (!sfree[k]) continue;
                        float jv = jac_at<F>(k, t, acc0, acc, fdx, fdy);
                        jo[(int64_t)ma.col[k] * H * W + pix] = jv * (float)sdu[k];
                    }
                } else {
                    const double gw = (double)ia.gin[me.img_off + pix];
#pragma unroll
                    for (int k = 0; k < P; ++k) v[k] += (double)jac_at<F>(k, t, acc0, acc, fdx, fdy) * gw;
                }
            }
        }
        if (ia.mode == 2) {
            // fixed-order reduction: wave butterflies, then the waves in order
            const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double w = strip_sum(v[k], K);
                if (lane == 0) sv[wave][k] = w;
            }
            __syncthreads();
            if (tid < P) {
                double sacc = sv[0][tid];
                for (int w = 1; w < NWAVE; ++w) sacc += sv[w][tid];
                ia.part[(int64_t)it * P + tid] = sacc * sdu[tid];
            }
        }
        __syncthreads();
    }
}

// Sum of the tile partials of each galaxy (tiles tstart[g] .. tstart[g+1]-1, in
// order) into its gradient row; fixed columns of the row are left at 0.
static __global__ void vjp_reduce_kernel(int n_gal, int P, ModelArgs ma, const int *tstart, const double *part,
                                  double *grad)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_gal) return;
    double *row = grad + (int64_t)g * ma.p;
    for (int c = 0; c < ma.p; ++c) row[c] = 0.0;
    for (int k = 0; k < P; ++k) {
        if (ma.col[k] < 0) continue;
        double s = 0.0;
        for (int t = tstart[g]; t < tstart[g + 1]; ++t) s += part[(int64_t)t * P + k];
        row[ma.col[k]] = s;
    }
}

// ---------------------------------------------------------------- default guess
struct GuessArgs {
    double *params, *moments;
    int n_gal;
};

__device__ inline double block_sum(double v, double *sred)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) sred[wave] = v;
    __syncthreads();
    double s = sred[0];
    for (int w = 1; w < NWAVE; ++w) s += sred[w];
    return s;
}

// Image moments of one galaxy (all threads of the workgroup call this):
// sky0 = mean of the usable pixels in the 2-px frame; S = usable pixels with
// D - sky0 > 3 sigma; flux, flux-weighted centroid and central second moments
// over S; r0 = 1.1774 sqrt(lambda+), q0 = sqrt(lambda-/lambda+), theta0 =
// atan2(2 Mxy, Mxx - Myy) / 2, m_g = m0 - 2.5 log10 max(F0, 1e-3); fewer
// than 5 pixels in S: the cutout centre, r0 = 3, q0 = 1, theta0 = 0.
struct Moments {
    double sky0, f0, xc, yc, r0, q0, th0, mg, pk;
};

// Pixels per thread that a moments pass reads at once.
constexpr int kMomU = 4;

// This thread's pixels q0 + u NT (u < kMomU) of a cutout of npix pixels at
// off: data d, sigma s and ok = (pixel_weight != 0) (false past the cutout,
// whose reads take its last pixel), all reads issued before any value is
// used, the mask's in one uniform branch: one wait per batch.
__device__ inline void moment_pixels(const BatchArgs &ba, int64_t off, int q0, int npix, float (&d)[kMomU],
                                     float (&s)[kMomU], bool (&ok)[kMomU])
{
    int m[kMomU];
#pragma unroll
    for (int u = 0; u < kMomU; ++u) {
        const int64_t idx = off + min(q0 + u * NT, npix - 1);
        d[u] = ba.data[idx];
        s[u] = ba.sigma[idx];
        m[u] = 1;
    }
    if (ba.omega) {
#pragma unroll
        for (int u = 0; u < kMomU; ++u) m[u] = ba.omega[off + min(q0 + u * NT, npix - 1)];
    }
#pragma unroll
    for (int u = 0; u < kMomU; ++u) {
        const bool use = m[u] != 0 && s[u] > 0.0f && isfinite(s[u]) && isfinite(d[u]);
        ok[u] = q0 + u * NT < npix && (use ? 1.0f / (s[u] * s[u]) : 0.0f) != 0.0f;
    }
}

// A cutout of at most kMomPix pixels is read from memory once: each thread
// keeps its pixels (data, sigma, and a bit each for ok) in registers over the
// three passes (16,384 cutouts of 64 x 64: the guess 364 -> 270 us; more pixels
// than these leave too few workgroups per CU).  Batches past the cutout are
// left out (32 x 32: 190 -> 180 us; with the branches 64 x 64 takes 1% more).  Bound by instruction issue.
constexpr int kMomB = 4;                              // batches of kMomU pixels per thread
constexpr int kMomPix = kMomB * kMomU * NT;           // 4096: 64 x 64

struct MomPixels {
    float d[kMomB * kMomU], s[kMomB * kMomU];
    uint32_t ok;
};

__device__ inline void moment_read(const BatchArgs &ba, int64_t off, int npix, MomPixels &px)
{
    px.ok = 0;
#pragma unroll
    for (int b = 0; b < kMomB; ++b) {
        float d[kMomU], s[kMomU];
        bool ok[kMomU];
        moment_pixels(ba, off, threadIdx.x + b * kMomU * NT, npix, d, s, ok);
#pragma unroll
        for (int u = 0; u < kMomU; ++u) {
            px.d[b * kMomU + u] = d[u];
            px.s[b * kMomU + u] = s[u];
            px.ok |= (ok[u] ? 1u : 0u) << (b * kMomU + u);
        }
    }
}

// f(q, d, s, k) for each of this thread's usable pixels q = tid + k NT, k
// increasing (k: of a cutout whose pixels are kept).  `which`: the bits of the
// kept pixels it is called for.
template <bool KEPT, class Fn>
__device__ inline void moment_each(const BatchArgs &ba, int64_t off, int npix, const MomPixels &px, uint32_t which, Fn f)
{
    if constexpr (KEPT) {
        // each pixel is worked on anew in every pass: what the compiler would
        // carry over (row, column, FP64 value) costs the second workgroup per CU
        int t = threadIdx.x;
#pragma unroll
        for (int k = 0; k < kMomB * kMomU; ++k) {
            if (k % kMomU == 0 && k * NT >= npix) break;        // no more batches
            float d = px.d[k];
            asm volatile("" : "+v"(t), "+v"(d));
            if ((which >> k) & 1u) f(t + k * NT, d, px.s[k], k);
        }
    } else {
        for (int q0 = threadIdx.x; q0 < npix; q0 += kMomU * NT) {
            float d[kMomU], sg[kMomU];
            bool ok[kMomU];
            moment_pixels(ba, off, q0, npix, d, sg, ok);
#pragma unroll
            for (int u = 0; u < kMomU; ++u)
                if (ok[u]) f(q0 + u * NT, d[u], sg[u], 0);
        }
    }
}

// Block sums of N values at once, each in block_sum's order; sred: N NWAVE doubles.
template <int N>
__device__ inline void block_sums(double (&v)[N], double *sred)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int n = 0; n < N; ++n) v[n] = wave_sum(v[n]);
    __syncthreads();
    if (lane == 0)
#pragma unroll
        for (int n = 0; n < N; ++n) sred[n * NWAVE + wave] = v[n];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < N; ++n) {
        double s = sred[n * NWAVE];
        for (int w = 1; w < NWAVE; ++w) s += sred[n * NWAVE + w];
        v[n] = s;
    }
}
constexpr int kMomRed = 5 * NWAVE;        // doubles of LDS for image_moments

template <bool KEPT>
__device__ inline Moments image_moments(const BatchArgs &ba, const Meta &me, double m0, double *sred,
                                        const MomPixels &px, int tail)
{
    const int tid = threadIdx.x;
    const int H = me.h, W = me.w;
    // row of pixel q by a float product: cutouts are at most 1024 x 1024, so (q + 0.5) / W is
    // below 1024 and at least 1 / (2 W) >= 2^-11 away from an integer, while the float
    // rounding of the product moves it by less than 2^-13
    const int npix = H * W;
    const float rW = 1.0f / (float)W;
    auto row_of = [&](int q) { return (int)(((float)q + 0.5f) * rW); };
    const unsigned hin = max(H - 4, 0), win = max(W - 4, 0);
    double a2[2] = {0.0, 0.0};
    int n = 0;
    moment_each<KEPT>(ba, me.img_off, npix, px, px.ok, [&](int q, float d, float, int) {
        const int i = row_of(q), j = q - __mul24(i, W);
        if ((unsigned)(i - 2) >= hin || (unsigned)(j - 2) >= win) {       // the border, two pixels wide
            a2[0] += d;
            ++n;
        }
    });
    a2[1] = n;
    block_sums<2>(a2, sred);
    Moments mo;
    mo.sky0 = a2[1] > 0.0 ? a2[0] / a2[1] : 0.0;
    double a4[4] = {0.0, 0.0, 0.0, 0.0}, pk = 0.0;
    n = 0;
    uint32_t bright = 0;        // the kept pixels above 3 sigma
    moment_each<KEPT>(ba, me.img_off, npix, px, px.ok, [&](int q, float d, float s, int k) {
        const double dp = (double)d - mo.sky0;
        if (!(dp > 3.0 * (double)s)) return;
        bright |= 1u << k;
        const int i = row_of(q), j = q - __mul24(i, W);
        const double x = j + 0.5, y = (H - i) - 0.5;
        a4[0] += dp; a4[1] += dp * x; a4[2] += dp * y;
        ++n;
        pk = fmax(pk, dp);
    });
    a4[3] = n;
    {   // the peak's block maximum goes through the same barriers
        const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) pk = fmax(pk, __shfl_xor(pk, o, 64));
        __syncthreads();
        if (lane == 0) sred[4 * NWAVE + wave] = pk;
        block_sums<4>(a4, sred);
        pk = sred[4 * NWAVE];
        for (int w = 1; w < NWAVE; ++w) pk = fmax(pk, sred[4 * NWAVE + w]);
    }
    const double f0 = a4[0], fx = a4[1], fy = a4[2], cnt = a4[3];
    mo.f0 = f0;
    mo.pk = pk > 0.0 ? pk : 1.0;
    mo.xc = 0.5 * W; mo.yc = 0.5 * H; mo.r0 = 3.0; mo.q0 = 1.0; mo.th0 = 0.0;
    const bool have = cnt >= 5.0 && f0 > 0.0;
    double a3[3] = {0.0, 0.0, 0.0};
    if (have) {
        mo.xc = fx / f0;
        mo.yc = fy / f0;
        moment_each<KEPT>(ba, me.img_off, npix, px, bright, [&](int q, float d, float s, int) {
            const double dp = (double)d - mo.sky0;
            if (!KEPT && !(dp > 3.0 * (double)s)) return;
            const int i = row_of(q), j = q - __mul24(i, W);
            const double dx = j + 0.5 - mo.xc, dy = (H - i) - 0.5 - mo.yc;
            a3[0] += dp * dx * dx; a3[1] += dp * dy * dy; a3[2] += dp * dx * dy;
        });
    }
    block_sums<3>(a3, sred);
    if ((tid >> 6) != tail) return mo;
    double mxx = a3[0], myy = a3[1], mxy = a3[2];
    if (have) {
        mxx /= f0; myy /= f0; mxy /= f0;
        // which product is fused with the sum is written out, not left to the compiler
        const double df = mxx - myy;
        double tr = 0.5 * (mxx + myy), dd = sqrt(fma(df, 0.25 * df, mxy * mxy));
        double lp = tr + dd, lm = fmax(tr - dd, 0.0);
        mo.q0 = lp > 0.0 ? sqrt(lm / lp) : 1.0;
        mo.q0 = fmin(fmax(mo.q0, 0.1), 1.0);
        mo.th0 = 0.5 * atan2(2.0 * mxy, mxx - myy);
        mo.r0 = 1.1774 * sqrt(fmax(lp, 0.0));
        mo.r0 = fmin(fmax(mo.r0, 1.0), 0.25 * W);
    }
    mo.mg = m0 - 2.5 * log10(fmax(f0, 1e-3));
    return mo;
}

// Moments of a cutout of any size; px is filled where it is kept.  mg, r0, q0
// and th0 are the work of wave `tail` alone (1,400 instructions with the
// features'; it alternates from cutout to cutout, so that no SIMD has them all).
__device__ inline Moments cutout_moments(const BatchArgs &ba, const Meta &me, double m0, double *sred, MomPixels &px,
                                         int tail)
{
    if (me.h * me.w <= kMomPix) {
        moment_read(ba, me.img_off, me.h * me.w, px);
        return image_moments<true>(ba, me, m0, sred, px, tail);
    }
    return image_moments<false>(ba, me, m0, sred, px, tail);
}

// The default start of one galaxy from its image moments, written into its
// parameter row through the model's column map.
template <class F>
__device__ inline void moments_guess(const ModelArgs &ma, const Moments &mo, double *out)
{
    double pa0 = mo.th0 * 180.0 / kPi;
    if (pa0 < 0.0) pa0 += 180.0;
    double nat[F::P];
    const double ms = mo.mg + 2.5 * log10((double)(ma.nflux > 1 ? ma.nflux : 1));
    F::default_guess(mo.xc, mo.yc, ms, mo.r0, mo.q0, pa0, mo.sky0, mo.pk, nat);
    for (int k = 0; k < F::P; ++k)
        if (ma.col[k] >= 0) out[ma.col[k]] = nat[k];
}

template <class F>
__global__ __launch_bounds__(NT, 4) void guess_kernel(ModelArgs ma, BatchArgs ba, GuessArgs ga)
{
    __shared__ double sred[kMomRed];
    for (int g = blockIdx.x; g < ga.n_gal; g += gridDim.x) {
        const Meta me = ba.meta[g];
        const int tail = (g / 256) % NWAVE;
        MomPixels px;
        const Moments mo = cutout_moments(ba, me, ma.m0, sred, px, tail);
        if ((int)threadIdx.x == 64 * tail) {
            if (ga.moments) {
                double *m6 = ga.moments + (int64_t)g * 6;
                m6[0] = mo.xc - 0.5 * me.w; m6[1] = mo.yc - 0.5 * me.h; m6[2] = mo.mg;
                m6[3] = log(mo.r0); m6[4] = mo.q0; m6[5] = mo.th0;
            }
            moments_guess<F>(ma, mo, ga.params + (int64_t)g * ma.p);
        }
        __syncthreads();
    }
}

// The same start from moments a feature pass has already stored: mom8[g] =
// {sky0, F0, xc, yc, m_g, r0, q0, theta0} and the peak pk[g]; one thread per
// galaxy.
template <class F>
__global__ void guess_stored_kernel(ModelArgs ma, int n_gal, const double *mom8, const double *pk, double *params)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_gal) return;
    const double *o = mom8 + (int64_t)g * 8;
    Moments mo;
    mo.sky0 = o[0]; mo.f0 = o[1]; mo.xc = o[2]; mo.yc = o[3];
    mo.mg = o[4]; mo.r0 = o[5]; mo.q0 = o[6]; mo.th0 = o[7];
    mo.pk = pk[g];
    moments_guess<F>(ma, mo, params + (int64_t)g * ma.p);
}

static __global__ void fill_int_kernel(int *p, int v) { *p = v; }

// The work queue's counter and, if given, the helpers' board, zeroed before a launch.
static __global__ void fit_reset_kernel(int *queue, int *board, int n)
{
    if (threadIdx.x == 0) *queue = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) board[i] = 0;
}

static __global__ void fill_ints_kernel(int *p, int n, int v)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace gm
