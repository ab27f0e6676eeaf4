// smc_gmm_impl.hpp -- (templates over the number of components K) the tempered
// Bayesian Gaussian-mixture sampler of Section 5.2 on gfx950: prior draws, the
// mixture log-likelihood (and its gradient), the three Metropolis blocks
// (random walk or MALA), and the reweighting by the tempering increment.
//
// Per-particle parameters in unconstrained coordinates (rows of the state):
//   mu_j (rows 0..K-1), eta_j = log lambda_j (K..2K-1),
//   z_j = log(omega_j / omega_K) (2K..3K-2), then the cached log-likelihood
//   (row D = 3K-1), log prior (D+1) and, for MALA, the cached likelihood
//   gradient (D+2..2D+1).
//
// The likelihood is the hot loop: l = sum_k lse_j(c_j - lambda_j (y_k -
// mu_j)^2 / 2), c_j = log omega_j + eta_j / 2 - log(2 pi) / 2, i.e. n K
// "mixture terms" per particle, each a multiply-add, a square, an
// exponential and an addition, plus one logarithm per 128 points.  A
// workgroup holds 64 particles (one per lane) and W waves; wave w walks its
// own contiguous chunk of the data with wave-uniform
// (scalar) loads of y, every lane keeps its particle's 3K constants and its
// accumulators in registers, and the W partial sums are combined in wave
// order through LDS.  Nothing here is a dense contraction, so the vector ALU
// (FP64) is the roofline, not the matrix cores.  A population too small to
// fill the chip that way gives each particle 2^lsl neighbouring lanes, which
// share its data (gmm_split()).
#include <math.h>

#pragma once

#include "smc_internal.hpp"

namespace smc {

constexpr double kHalfLog2Pi = 0.91893853320467274178032973640562;
constexpr int GMM_RED_GROUP = 4;  // accumulators combined per LDS round
// doubles of the wave-combine buffer: wave 0 keeps its own sums in registers
constexpr int gmm_red_doubles(int W) { return GMM_RED_GROUP * (W - 1) * WAVE; }
// Where a Metropolis block reads and writes the particles' state: global
// memory both ways (each block its own launch or queue item) or, when one
// workgroup runs a step's blocks in sequence, global -> LDS for the first,
// LDS -> LDS between blocks and LDS -> global for the last.
constexpr int GMM_IO_GLOBAL = 0, GMM_IO_FIRST = 1, GMM_IO_LDS = 2, GMM_IO_LAST = 3;
// doubles of the LDS state copy of one 64-particle tile: D coordinates, the
// log-likelihood, the log prior and, for MALA, the D-gradient
constexpr int gmm_hand_doubles(int K, bool mala)
{
    return (mala ? 2 * (3 * K - 1) + 2 : 3 * K + 1) * WAVE;
}


// log omega_j (j = 0..K-1) from the K-1 logits, reference component K.
template <int K>
__device__ __forceinline__ void log_weights(const double (&phi)[3 * K - 1 > 0 ? 3 * K - 1 : 1],
                                            double (&logw)[K])
{
    double m = 0.0;
#pragma unroll
    for (int j = 0; j < K - 1; ++j)
        m = fmax(m, phi[2 * K + j]);
    double s = exp_d(-m);
#pragma unroll
    for (int j = 0; j < K - 1; ++j)
        s += exp_d(phi[2 * K + j] - m);
    const double lse = m + log_d(s);
#pragma unroll
    for (int j = 0; j < K - 1; ++j)
        logw[j] = phi[2 * K + j] - lse;
    logw[K - 1] = -lse;
}

template <int K>
__device__ __forceinline__ double log_prior(const double (&phi)[3 * K - 1 > 0 ? 3 * K - 1 : 1],
                                            const double (&logw)[K], const GmmPrior &pr)
{
    double a = 0.0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const double d = phi[j] - pr.mu_mean;
        a -= d * d * pr.inv_2var;
    }
#pragma unroll
    for (int j = 0; j < K; ++j)
        a += pr.shape * phi[K + j] - pr.rate * exp_d(phi[K + j]);
    if (K > 1) {
#pragma unroll
        for (int j = 0; j < K; ++j)
            a += pr.rho * logw[j];
    }
    return a;
}

// gradient of log_prior for the coordinates of one block
template <int K>
__device__ __forceinline__ double log_prior_grad(const double (&phi)[3 * K - 1 > 0 ? 3 * K - 1 : 1],
                                                 const double (&logw)[K], const GmmPrior &pr,
                                                 int q)
{
    if (q < K)
        return -(phi[q] - pr.mu_mean) * (2.0 * pr.inv_2var);
    if (q < 2 * K)
        return pr.shape - pr.rate * exp_d(phi[q]);
    return pr.rho * (1.0 - (double)K * exp_d(logw[q - 2 * K]));
}

// Per-lane mixture likelihood accumulator for one particle (Section 5.2.1):
// log p(y) = log sum_j exp(c_j - (lambda_j / 2) (y - mu_j)^2) with
// c_j = log omega_j + eta_j / 2 - log(2 pi) / 2, summed over the data.
//
// Fast form (K > 1): the density itself, up to a power of two of the
// parameter vector: s = sum_j 2^(SHIFT - a_j), a_j = u_j^2 + d_j with u_j =
// g_j (y - mu_j) = g_j y - g_j mu_j, g_j = sqrt(lambda_j log2(e) / 2), d_j =
// O - c_j log2(e) >= 0 and O the integer above the largest c_j log2(e).  Per
// term two multiply-adds, fraction and integer part, ten multiply-adds for
// the power, its scaling and the addition to s.  Nothing is factored out of
// s (SHIFT centres its range); the densities of two points are multiplied
// and split into exponent (summed as an integer) and mantissa (multiplied;
// one logarithm per FLUSH points).  A group of points with an s not above
// S_MIN in some lane -- a point some thirty-five standard deviations from
// every component, or a NaN -- is left out of that lane's sums, ends the
// segment, and repair() takes it again with the largest term factored out.
// After a second such group within FLUSH points, or when the first group of
// the chunk is one (a vector far from the data is out of range at most
// points), the wave takes the rest of its chunk in the safe form, which
// factors the largest term out of every point.  A wave with a parameter that
// is not finite takes the whole chunk in the safe form, and a sum that comes
// out NaN is taken again with zero for the terms that are not finite.
// One distant observation in every wave's part of the data, gradient at 2^16
// vectors of 1000 points: 342 -> 360 us at K = 6, 632 -> 642 at K = 12.
//
// Tournament form (K <= 8 without the gradient, K = 2 with it): the largest
// a_j = c_j log2(e) - u_j^2 is carried through K - 1 maxima, the loser of each
// match kept, so that only K - 1 powers 2^-(m - loser) are taken, s = 1 +
// their sum.  2 (K - 1) comparisons replace a power of 13 instructions, and
// no point is out of range; the gradient needs every term in its place, which
// two components get back by a selection.
//
// Bound: FP64 vector issue (every instruction of the loop is full rate).
// Per point 16 K + 3.5 instructions (fast form) or 17 K - 11 (tournament);
// factoring the maximum out of every point took 19 K + 3.  Value at K = 4,
// 2^14 vectors, 2000 points 95 -> 73 us; with the gradient at K = 6, 2^14
// vectors, 10^4 points 727 -> 673 us a call, 46 TFLOP/s.
//
// Gradient (GRAD): with responsibilities r_j = 2^(SHIFT - a_j) / s and
// lambda_j d_j = 2 ln2 g_j u_j, lambda_j d_j^2 / 2 = ln2 u_j^2:
//   d/d mu_j  = sum r_j lambda_j (y - mu_j)        = 2 ln2 g_j sum r_j u_j
//   d/d eta_j = sum r_j (1/2 - lambda_j d_j^2 / 2) = sum r_j / 2 - ln2 sum r_j u_j^2
// accumulated as sum r u (in gmu), sum r u^2 (in geta) and sum r (in gr)
// and converted once in finish().
// Largest K without the gradient that takes the tournament form: the two
// forms cross there (value of 2^14 vectors at 2000 points, us, tournament
// against product: K = 2 33 / 50, K = 4 73 / 86, K = 5 105 / 112, K = 6
// 117 / 122, K = 7 134 / 131, K = 8 150 / 150, K = 9 184 / 190, K = 10
// 197 / 192, K = 12 241 / 228, K = 16 327 / 296; of 2^16 at 1000: K = 7
// 275 / 273, K = 8 315 / 311, K = 9 359 / 346).  The tournament has no points
// out of range, so it keeps K = 7 and 8.
constexpr int TOURN_MAX_K = 8;

// SAFE_ONLY: the safe form throughout, for a gradient whose product form's
// registers would spill in its loop: K = 16 (2^14 vectors, 10^4 points: 3250 us
// a call against 2450) and, with the step's own registers, K = 15 (MALA step of
// 20000 particles, 400 points, 1870 us against 1020; the likelihood alone 1870
// in the product form, 1930 in the safe one).
template <int K, bool GRAD, bool SAFE_ONLY = GRAD && (K > 15)>
struct MixLik {
    // points per group: independent chains for the two waves a SIMD holds,
    // as far as the registers allow (the gradient keeps every term of the
    // group until its reciprocal is known)
    static constexpr int GROUP = K > 8 || (GRAD && K > 6) ? 1 : (GRAD || K > 4 ? 2 : 4);
    static constexpr bool TOURN = K > 1 && (GRAD ? K == 2 : K <= TOURN_MAX_K);
    // points per segment, one logarithm each (safe form: factors <= 16);
    // segments of 32 points cost 3 %
    static constexpr int FLUSH = 128;
    // s <= K 2^SHIFT <= 2^494; s > 2^-500 has a power above 2^-504, so every
    // s that counts, the product of two and its reciprocal are normal
    static constexpr int SHIFT = 490;
    static constexpr double S_MIN = 0x1p-500;
    // stand-in for a density out of range, and its log2
    static constexpr double OUT_S = 0x1p1000;
    static constexpr int OUT = 1000;
    double g[K], gm[K];
    double c[K];  // d_j, or c_j log2(e) in the safe form (fast == false) and for K = 1
    int off;      // O
    bool fast;    // uniform across the wave
    double ll;  // after chunk(): sum of log p(y_k) over the chunk
    double m2, lsum, prod;
    int ex;
    double gmu[GRAD ? K : 1], geta[GRAD ? K : 1], gr[GRAD ? K : 1];

    __device__ __forceinline__ void setup(const double (&phi)[3 * K - 1 > 0 ? 3 * K - 1 : 1],
                                          const double (&logw)[K])
    {
        bool ok = K > 1 && !SAFE_ONLY;
        double cmax = -INFINITY;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            g[j] = sqrt((0.5 * detail::kLog2e) * exp_d(phi[K + j]));
            gm[j] = g[j] * phi[j];
            c[j] = detail::kLog2e * (logw[j] + 0.5 * phi[K + j] - kHalfLog2Pi);
            ok = ok && fabs(c[j]) < 0x1p20 && g[j] < 0x1p500 && fabs(gm[j]) < 0x1p500;
            cmax = fmax(cmax, c[j]);
        }
        fast = __all(ok);
        off = 0;
        if (!TOURN && fast) {
            const double o = ceil(cmax);
            off = (int)o;
#pragma unroll
            for (int j = 0; j < K; ++j)
                c[j] = o - c[j];
        }
        reset();
    }

    __device__ __forceinline__ void reset()
    {
        ll = m2 = lsum = 0.0;
        prod = 1.0;
        ex = 0;
        if (GRAD) {
#pragma unroll
            for (int j = 0; j < K; ++j)
                gmu[j] = geta[j] = gr[j] = 0.0;
        }
    }

    // One point in the safe form: the maximum m of the a_j = cl_j - u_j^2
    // (cl_j = c_j log2(e)) factored out, s = sum_j 2^(a_j - m) in [1, K].
    // CLAMP: a_j = -inf or NaN is a zero term (without it the sums become
    // NaN).
    template <bool CLAMP>
    __device__ __forceinline__ void point(double y, const double (&cl)[K])
    {
        double e[K], u[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            u[j] = fma(g[j], y, -gm[j]);
            e[j] = fma(-u[j], u[j], cl[j]);
        }
        double m = e[0];
#pragma unroll
        for (int j = 1; j < K; ++j)
            m = fmax(m, e[j]);
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            e[j] = CLAMP ? exp2_nonpos(e[j] - m) : exp2_neg(m - e[j]);
            s = j == 0 ? e[0] : s + e[j];
        }
        m2 += m;
        prod *= s;
        if (GRAD) {
            const double inv = recip(s);
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const double r = e[j] * inv;
                const double ru = r * u[j];
                gmu[j] += ru;
                geta[j] = fma(ru, u[j], geta[j]);
                gr[j] += r;
            }
        }
    }

    // hardware estimate and two Newton steps (s and 1/s normal)
    static __device__ __forceinline__ double recip(double s)
    {
        double inv = __builtin_amdgcn_rcp(s);
        inv = fma(inv, fma(-s, inv, 1.0), inv);
        return fma(inv, fma(-s, inv, 1.0), inv);
    }

    // The terms and densities of N points (GROUP, or 1 for the remainder of a
    // chunk) in the fast form; whether every density is in range (false for
    // NaN).  No step of it can be contracted differently from one use to the
    // next, so in_range() gives the same answer.
    template <int N>
    __device__ __forceinline__ bool densities(const double (&y)[N], double (&u)[N][K],
                                              double (&e)[N][K], double (&s)[N])
    {
        bool good = true;
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                u[i][j] = fma(g[j], y[i], -gm[j]);
                e[i][j] = exp2_neg<SHIFT>(fma(u[i][j], u[i][j], c[j]));
                s[i] = j == 0 ? e[i][0] : s[i] + e[i][j];
            }
            good = good & (s[i] > S_MIN);
        }
        return good;
    }

    // Whether a point's density is in range: the sum of densities(), the terms
    // one at a time (few registers).
    __device__ __forceinline__ bool in_range(double y)
    {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const double u = fma(g[j], y, -gm[j]);
            const double e = exp2_neg<SHIFT>(fma(u, u, c[j]));
            s = j == 0 ? e : s + e;
            __builtin_amdgcn_sched_barrier(0);
        }
        return s > S_MIN;
    }

    // point<false>() with the constants of the fast form and the same bits, the
    // terms computed again for each of their uses and one at a time, so that
    // the loop around it keeps its registers.
    __device__ __forceinline__ void far_point(double y)
    {
        int o = off;
        asm volatile("" : "+v"(o));  // O - d_j stays here instead of K registers
        double m = 0.0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const double u = fma(g[j], y, -gm[j]);
            const double a = fma(-u, u, (double)o - c[j]);
            m = j == 0 ? a : fmax(m, a);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" : "+v"(y), "+v"(o));  // computed again
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const double u = fma(g[j], y, -gm[j]);
            const double e = exp2_neg(m - fma(-u, u, (double)o - c[j]));
            s = j == 0 ? e : s + e;
            __builtin_amdgcn_sched_barrier(0);
        }
        m2 += m;
        prod *= s;
        if (GRAD) {
            const double inv = recip(s);
            asm volatile("" : "+v"(y), "+v"(o));
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const double u = fma(g[j], y, -gm[j]);
                const double r = exp2_neg(m - fma(-u, u, (double)o - c[j])) * inv;
                const double ru = r * u;
                gmu[j] += ru;
                geta[j] = fma(ru, u, geta[j]);
                gr[j] += r;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // The group of N points at p that group() left out of some lanes' sums.
    template <int N>
    __device__ __forceinline__ void repair(const double *__restrict__ p)
    {
        bool good = true;
#pragma nounroll
        for (int i = 0; i < N; ++i)
            good = good & in_range(p[i]);
        if (!good) {
            m2 -= ((N + 1) / 2) * OUT + N * (off - SHIFT);
#pragma nounroll
            for (int i = 0; i < N; ++i)
                far_point(p[i]);
        }
    }

    // One point in the tournament form (finite parameters; a_j = -inf, from a
    // point that is not finite, makes the sums NaN or counts as zero).
    __device__ __forceinline__ void tournament(double y)
    {
        double e[K], u[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            u[j] = fma(g[j], y, -gm[j]);
            e[j] = fma(-u[j], u[j], c[j]);
        }
        if constexpr (GRAD) {  // K == 2
            const double d = e[0] - e[1];
            m2 += fmax(e[0], e[1]);
            const double w = exp2_neg(fabs(d));
            const double s = 1.0 + w;
            prod *= s;
            const double inv = recip(s), low = w * inv;
            const bool first = d >= 0.0;
            const double r[2] = {first ? inv : low, first ? low : inv};
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const double ru = r[j] * u[j];
                gmu[j] += ru;
                geta[j] = fma(ru, u[j], geta[j]);
                gr[j] += r[j];
            }
        } else {
            double m = e[0];
#pragma unroll
            for (int j = 1; j < K; ++j) {
                const double lo = fmin(m, e[j]);
                m = fmax(m, e[j]);
                e[j] = lo;
            }
            m2 += m;
            double s = 0.0;
#pragma unroll
            for (int j = 1; j < K; ++j)
                s += exp2_neg(m - e[j]);
            prod = fma(prod, s, prod);
        }
    }

    // Whether this lane has the group in its sums (false: for repair()).
    template <int N>
    __device__ __forceinline__ bool group(const double (&y)[N])
    {
        if constexpr (TOURN) {
#pragma unroll
            for (int i = 0; i < N; ++i)
                tournament(y[i]);
            return true;
        }
        double u[N][K], e[N][K], s[N];
        const bool good = densities<N>(y, u, e, s);
#pragma unroll
        for (int i = 0; i < N; i += 2) {
            const bool two = i + 1 < N;
            // no branch, so that the loads of the next group stay ahead: a
            // group out of range counts as a density OUT_S (taken back by
            // repair()), which leaves nothing of it in the gradient's sums
            const double p = two ? s[i] * s[two ? i + 1 : i] : s[i];
            const double q = good ? p : OUT_S;
            prod *= __builtin_amdgcn_frexp_mant(q);
            ex += __builtin_amdgcn_frexp_exp(q) + (two ? 2 : 1) * (off - SHIFT);
            if (GRAD) {
                static_assert(!GRAD || GROUP <= 2, "OUT_S covers a pair");
                const double iq = recip(q);
#pragma unroll
                for (int h = i; h < i + 2 && h < N; ++h) {
                    // 1 / s_h = (the other s) / q
                    const double inv = two ? iq * s[h == i ? i + (two ? 1 : 0) : i] : iq;
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        const double r = e[h][j] * inv;
                        const double ru = r * u[h][j];
                        gmu[j] += ru;
                        geta[j] = fma(ru, u[h][j], geta[j]);
                        gr[j] += r;
                    }
                }
            }
        }
        return good;
    }

    __device__ __forceinline__ void flush()
    {
        lsum += log_pos_d(prod);
        m2 += (double)ex;
        prod = 1.0;
        ex = 0;
    }

    // The constants of the safe form.
    __device__ __forceinline__ void safe_constants()
    {
#pragma unroll
        for (int j = 0; j < K; ++j)
            c[j] = (double)off - c[j];
        fast = false;
    }

    __device__ __forceinline__ void finish()
    {
        ll = fma(detail::kLn2, m2, lsum);
        if (GRAD) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                gmu[j] *= (2.0 * detail::kLn2) * g[j];
                geta[j] = fma(-detail::kLn2, geta[j], 0.5 * gr[j]);
            }
        }
    }

    // One point of a single component.
    __device__ __forceinline__ void single(double y)
    {
        const double u = fma(g[0], y, -gm[0]);
        m2 += fma(-u, u, c[0]);
        if (GRAD) {
            gmu[0] += u;
            geta[0] = fma(u, u, geta[0]);
            gr[0] += 1.0;
        }
    }

    // The points [k0, k1) (uniform across the wave) of this lane's particle.
    // Unsliced, every lane takes all of them: wave-uniform loads, the next
    // group fetched one group ahead.  SLICED, the 2^lsl lanes of a particle
    // share them, a group each in turn (neighbouring lanes read neighbouring
    // groups), the remainder point by point.
    template <bool SLICED>
    __device__ __forceinline__ void chunk(const double *__restrict__ y, int64_t k0, int64_t k1,
                                          int lsl)
    {
        const int slice = SLICED ? lane_id() & ((1 << lsl) - 1) : 0;
        const int one = SLICED ? 1 << lsl : 1;  // stride of single points
        int64_t k = k0;
        if constexpr (K == 1) {
            // three to five instructions a point: eight (sliced: four) to a wait
            // for loads, the next ones on their way
            constexpr int P = SLICED ? 4 : 8;
            k += slice;
            if (k + (int64_t)(P - 1) * one < k1) {
                double a[P];
#pragma unroll
                for (int i = 0; i < P; ++i)
                    a[i] = y[k + i * one];
                for (; k + (int64_t)(2 * P - 1) * one < k1; k += P * one) {
                    double b[P];
#pragma unroll
                    for (int i = 0; i < P; ++i)
                        b[i] = y[k + (P + i) * one];
#pragma unroll
                    for (int i = 0; i < P; ++i)
                        single(a[i]);
#pragma unroll
                    for (int i = 0; i < P; ++i)
                        a[i] = b[i];
                }
#pragma unroll
                for (int i = 0; i < P; ++i)
                    single(a[i]);
                k += P * one;
            }
            for (; k < k1; k += one)
                single(y[k]);
        } else {
            if constexpr (!SAFE_ONLY) {
                const int step = GROUP * one;
                const double *__restrict__ yg = y + slice * GROUP;  // this lane's groups
                // a group out of range that ends up to here changes the form
                int64_t quiet = k + step;
                while (fast && k + step <= k1) {
                    const int groups = (int)min((int64_t)(FLUSH / GROUP), (k1 - k) / step);
                    const double *__restrict__ p = yg + k;
                    double a[GROUP];
#pragma unroll
                    for (int i = 0; i < GROUP; ++i)
                        a[i] = p[i];
                    bool far = false;  // uniform across the wave
                    int r = 1;
                    for (; r < groups; ++r) {
                        double b[GROUP];
                        p += step;
#pragma unroll
                        for (int i = 0; i < GROUP; ++i)
                            b[i] = p[i];
                        const bool good = group<GROUP>(a);
                        far = !TOURN && __any(!good);
                        if (far)
                            break;
#pragma unroll
                        for (int i = 0; i < GROUP; ++i)
                            a[i] = b[i];
                    }
                    if (!far) {
                        const bool good = group<GROUP>(a);
                        far = !TOURN && __any(!good);
                    }
                    k += (int64_t)r * step;  // the segment, or up to the group out of range
                    flush();
                    if (far) {
                        repair<GROUP>(yg + k - step);
                        flush();
                        if (k <= quiet)
                            safe_constants();
                        quiet = k + (int64_t)FLUSH * one;
                    }
                }
                if ((SLICED || GROUP > 1) && fast && k < k1) {
                    bool good = true;
                    for (int64_t q = k + slice; q < k1; q += one) {
                        const double a[1] = {y[q]};
                        good = good & group<1>(a);
                    }
                    if (!TOURN && __any(!good)) {
                        flush();
#pragma nounroll
                        for (int64_t q = k + slice; q < k1; q += one)
                            repair<1>(y + q);
                    }
                    k = k1;
                }
            }
            flush();
            if constexpr (TOURN) {
                if (!fast)
                    m2 = __builtin_nan("");
                k = k1;
            }
            // the safe form, two points at a time while registers allow and
            // the next two fetched ahead of them
            k += slice;
            while (k < k1) {
                const int64_t kend = min(k + (int64_t)FLUSH * one, k1);
                if (K <= 8 && k + one < kend) {
                    double y0 = y[k], y1 = y[k + one];
                    for (; k + 3 * one < kend; k += 2 * one) {
                        const double n0 = y[k + 2 * one], n1 = y[k + 3 * one];
                        point<false>(y0, c);
                        point<false>(y1, c);
                        y0 = n0;
                        y1 = n1;
                    }
                    point<false>(y0, c);
                    point<false>(y1, c);
                    k += 2 * one;
                }
                for (; k < kend; k += one)
                    point<false>(y[k], c);
                flush();
            }
        }
        finish();
        // a term that is not finite: once more, clamped
        if (K > 1 && !TOURN && fast && __any(ll != ll))
            safe_constants();
        if (K > 1 && ll != ll) {
            reset();
#pragma nounroll
            for (k = k0 + slice; k < k1; k += one) {
                point<true>(y[k], c);
                flush();
            }
            finish();
        }
    }

    static constexpr int NACC = GRAD ? 1 + 3 * K : 1;
    __device__ __forceinline__ double &acc(int q)
    {
        if (q == 0)
            return ll;
        if (q <= K)
            return gmu[GRAD ? q - 1 : 0];
        if (q <= 2 * K)
            return geta[GRAD ? q - 1 - K : 0];
        return gr[GRAD ? q - 1 - 2 * K : 0];
    }
};

// Sums over the 2^lsl neighbouring lanes of a particle, complete in the last
// of them (the steps of the wave scan, as many as the slices need).
template <typename Lik>
__device__ __forceinline__ void combine_slices(Lik &L, int lsl)
{
#define SMC_SLICE_STEP(STEP, ...)                                                                 \
    if (lsl > STEP) {                                                                             \
        _Pragma("unroll") for (int q = 0; q < Lik::NACC; ++q)                                     \
            L.acc(q) += dpp::mov<__VA_ARGS__>(L.acc(q), 0.0);                                     \
    }
    SMC_SLICE_STEP(0, dpp::ROW_SHR1)
    SMC_SLICE_STEP(1, dpp::ROW_SHR2)
    SMC_SLICE_STEP(2, dpp::ROW_SHR4)
    SMC_SLICE_STEP(3, dpp::ROW_SHR8)
    SMC_SLICE_STEP(4, dpp::ROW_BCAST15, 0xA)
    SMC_SLICE_STEP(5, dpp::ROW_BCAST31, 0xC)
#undef SMC_SLICE_STEP
}

// Combines the accumulators of the W waves in wave order; wave 0 ends with
// the totals (SLICED: in the last lane of each particle).  `red` holds
// gmm_red_doubles(W).
template <bool SLICED, typename Lik>
__device__ __forceinline__ void combine_waves(Lik &L, int W, int lsl, double *red)
{
    constexpr int NACC = Lik::NACC;
    if (SLICED)
        combine_slices(L, lsl);
    const int w = wave_id(), lane = lane_id();
    for (int q0 = 0; q0 < NACC; q0 += GMM_RED_GROUP) {
        __syncthreads();
        if (w > 0) {
#pragma unroll
            for (int g = 0; g < GMM_RED_GROUP; ++g)
                if (q0 + g < NACC)
                    red[(g * (W - 1) + w - 1) * WAVE + lane] = L.acc(q0 + g);
        }
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int g = 0; g < GMM_RED_GROUP; ++g)
                if (q0 + g < NACC) {
                    double a = L.acc(q0 + g);
                    for (int v = 1; v < W; ++v)
                        a += red[(g * (W - 1) + v - 1) * WAVE + lane];
                    L.acc(q0 + g) = a;
                }
        }
    }
}

// Wave w's share [k0, k1) of the n data points (uniform across the wave).
__device__ __forceinline__ void data_chunk(int64_t nd, int W, int64_t *k0, int64_t *k1)
{
    const int w = __builtin_amdgcn_readfirstlane(wave_id());
    const int64_t per = (nd + W - 1) / W;
    *k0 = min((int64_t)w * per, nd);
    *k1 = min(*k0 + per, nd);
}

// The particle and column of a lane when 2^lsl neighbouring lanes share a
// particle (lsl = 0: one lane each): `tile` covers 64 >> lsl particles; the
// last lane of a particle leads (its sums are complete, its LDS column holds
// the particle's state).
struct LaneMap {
    int64_t i;  // particle
    int col;    // the particle's leading lane
    bool lead;
    __device__ __forceinline__ LaneMap(int64_t tile, int lsl)
    {
        const int lane = lane_id();
        i = tile * (WAVE >> lsl) + (lane >> lsl);
        col = lane | ((1 << lsl) - 1);
        lead = col == lane;
    }
};

// z-gradient from the accumulated responsibilities: sum_k (r_kj - omega_j)
template <int K>
__device__ __forceinline__ double z_grad(double gr_j, double logw_j, int64_t nd)
{
    return gr_j - (double)nd * exp_d(logw_j);
}

// ---------------------------------------------------------------------------
// Initialisation from the prior (Algorithm "gmm"): mu_j = xi + sd n_j
// (normals: call j/2), lambda_j = G_j / b with G_j ~ Gamma(a) (calls from
// 64 + 64 j), omega = H / sum H with H_j ~ Gamma(rho) (calls from
// 64 + 1024 + 64 j); then log prior and log-likelihood (and its gradient for
// MALA); log-weights 0.
// ---------------------------------------------------------------------------
template <int K, bool GRAD, bool SLICED>
__device__ __forceinline__ void gmm_init_tile(const Prob &P, int W, int64_t tile, int lsl)
{
    constexpr int D = 3 * K - 1;
    __shared__ double red[gmm_red_doubles(GMM_MAXW)];
    double *__restrict__ st = (double *)P.state[0];
    double *__restrict__ lw = P.lw;
    const int64_t n = P.n, nd = P.n_data;
    const double *__restrict__ y = P.data;
    const Key key = P.key;
    const uint32_t p = P.problem_id;
    const GmmPrior pr = P.prior;
    const double mu_sd = P.mu_sd;
    int32_t *__restrict__ counters = P.counters;
    const LaneMap lm(tile, SLICED ? lsl : 0);
    const int64_t i = lm.i;
    const bool valid = i < n;
    const uint32_t ii = (uint32_t)(valid ? i : 0);
    double phi[D > 0 ? D : 1];
#pragma unroll
    for (int j = 0; j < K; j += 2) {
        const double2 z = normal2(draw(key, ii, 0, TAG_INIT, (uint32_t)(j / 2), p));
        phi[j] = pr.mu_mean + mu_sd * z.x;
        if (j + 1 < K)
            phi[j + 1] = pr.mu_mean + mu_sd * z.y;
    }
    int fail = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const double G = gamma_draw(key, ii, 0, TAG_INIT, (uint32_t)(64 + 64 * j), p, pr.shape,
                                    &fail);
        phi[K + j] = log_d(G / pr.rate);
    }
    double H[K];
#pragma unroll
    for (int j = 0; j < K; ++j)
        H[j] = gamma_draw(key, ii, 0, TAG_INIT, (uint32_t)(64 + 64 * 16 + 64 * j), p, pr.rho,
                          &fail);
#pragma unroll
    for (int j = 0; j < K - 1; ++j)
        phi[2 * K + j] = log_d(H[j]) - log_d(H[K - 1]);
    double logw[K];
    log_weights<K>(phi, logw);
    MixLik<K, GRAD> L;
    L.setup(phi, logw);
    int64_t k0, k1;
    data_chunk(nd, W, &k0, &k1);
    L.template chunk<SLICED>(y, k0, k1, lsl);
    combine_waves<SLICED>(L, W, lsl, red);
    if (wave_id() == 0 && valid && lm.lead) {
#pragma unroll
        for (int q = 0; q < D; ++q)
            st[(int64_t)q * n + i] = phi[q];
        st[(int64_t)D * n + i] = L.ll;
        st[(int64_t)(D + 1) * n + i] = log_prior<K>(phi, logw, pr);
        if (GRAD) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                st[(int64_t)(D + 2 + j) * n + i] = L.gmu[j];
                st[(int64_t)(D + 2 + K + j) * n + i] = L.geta[j];
                if (j < K - 1)
                    st[(int64_t)(D + 2 + 2 * K + j) * n + i] = z_grad<K>(L.gr[j], logw[j], nd);
            }
        }
        lw[i] = 0.0;
        if (fail)
            atomicOr(&counters[CNT_ERR], SMC_DEVERR_GAMMA);
    }
}

template <int K, bool GRAD, bool SLICED>
__global__ __launch_bounds__(GMM_MAXW *WAVE) void gmm_init_kernel(Prob P, int W, int lsl)
{
    gmm_init_tile<K, GRAD, SLICED>(P, W, blockIdx.x, lsl);
}

// 2^lsl workgroups take the parts of each 64-particle tile of the map.
template <int K, bool GRAD, bool SLICED>
__global__ __launch_bounds__(GMM_MAXW *WAVE) void gmm_init_batch_kernel(
    const Prob *__restrict__ probs, const int2 *__restrict__ map, int W, int lsl)
{
    const int2 pm = map[SLICED ? blockIdx.x >> lsl : blockIdx.x];
    const int64_t tile = SLICED ? ((int64_t)pm.y << lsl) + (blockIdx.x & ((1u << lsl) - 1)) : pm.y;
    gmm_init_tile<K, GRAD, SLICED>(probs[pm.x], W, tile, lsl);
}

// ---------------------------------------------------------------------------
// One Metropolis block of every particle at tempering alpha (the three-block
// kernel of Section 5.2.1).  Random walk: phi'_b = phi_b + s n.  MALA:
// phi'_b = phi_b + s^2/2 g + s n, g the block gradient of prior + alpha x
// likelihood, with both proposal densities in the ratio.  Accept iff
// log u <= log r.  With `full` every row is written to the ping-pong
// partner (the first block after a resample call), the particle read through
// the pending ancestors when the resample happened; otherwise the accepted
// rows are updated in place.  Accepted proposals are counted into
// history[step][ACC0 + block] (integer-valued, so the order of the additions
// does not matter).
// ---------------------------------------------------------------------------
// The proposal of particle i for one block: loads phi, takes the normals, adds
// the drift (MALA).  Not kept across the data loop: what the decision needs of
// it is stashed in LDS.  All array indices are compile-time (the block's
// coordinates are selected by uniform branches), so the arrays are registers,
// not scratch.  fwd = sum over the block of (phi' - phi - drift)^2, the forward
// proposal term of MALA.
template <int K, bool MALA>
struct Proposal {
    static constexpr int D = 3 * K - 1;
    double phi[D > 0 ? D : 1];
    double prop[D > 0 ? D : 1];
    double logw0[K];
    double fwd;

    // `z`: the particle's normals, coordinate q at z[q * zn]
    __device__ __forceinline__ void build(const double *__restrict__ src, int64_t n, int64_t si,
                                          const double *z, int zn, int block, double alpha,
                                          double scale, const GmmPrior &pr)
    {
        const int off = block * K;
        const int dim = block == 2 ? K - 1 : K;
#pragma unroll
        for (int q = 0; q < D; ++q)
            phi[q] = src[(int64_t)q * n + si];
        log_weights<K>(phi, logw0);
        const double h2 = scale * scale;
        fwd = 0.0;
#pragma unroll
        for (int q = 0; q < D; ++q)
            prop[q] = phi[q];
#pragma unroll
        for (int q = 0; q < D; ++q) {
            const int mm = q - off;
            if (mm >= 0 && mm < dim) {
                double dr = 0.0;
                if (MALA) {
                    double g = log_prior_grad<K>(phi, logw0, pr, q);
                    if (alpha != 0.0)
                        g += alpha * src[(int64_t)(D + 2 + q) * n + si];
                    dr = 0.5 * h2 * g;
                }
                const double v = phi[q] + dr + scale * z[q * zn];
                prop[q] = v;
                const double a = v - phi[q] - dr;
                fwd += a * a;
            }
        }
    }
};

// Values of the epilogue that do not depend on the likelihood, computed
// before the data loop by the last wave and kept in LDS (one column per
// lane) until wave 0 takes the decision: the proposal's log prior, the
// proposed block coordinates and, for MALA, the forward proposal term, the
// prior gradient at the proposal (block coordinates) and the proposed mixture
// weights omega'_j (the z-gradient subtracts n omega'_j).
template <int K, bool MALA>
struct BlockStash {
    static constexpr int LPP = 0, FWD = 1, PROP = 2, GP = 2 + K, ZC = 2 + 2 * K;
    static constexpr int ROWS = MALA ? 2 + 3 * K - 1 : 2 + K;
};

template <int K, bool MALA>
constexpr int gmm_stash_doubles() { return BlockStash<K, MALA>::ROWS * WAVE; }

// One pair of normals (coordinates 2m, 2m + 1 of the block) or the logarithm of
// the accept uniform of block b, particle ii.  `z`: the block's first
// coordinate, `u`: its log U, in the particle's column of rows of `cols`.
template <int K>
__device__ __forceinline__ void draw_item(const Prob &P, uint32_t ii, uint32_t t, int sweep,
                                          bool pair, int b, int m, double *z, double *u, int cols)
{
    const uint4 w =
        draw(P.key, ii, t, pair ? TAG_MH_MU + (uint32_t)b : TAG_MH_ACCEPT,
             (uint32_t)(pair ? 64 * sweep + m : 4 * sweep + b), P.problem_id);
    const double l = log_pos_d(u53(w.x, w.y));
    if (pair) {
        const double2 v = normal2(w, l);
        z[2 * m * cols] = v.x;
        if (2 * m + 1 < (b == 2 ? K - 1 : K))
            z[(2 * m + 1) * cols] = v.y;
    } else {
        *u = l;
    }
}

// The random numbers of one sweep of a tile's particles: the D normals of the
// proposals and the logarithms of the blocks' accept uniforms.  None depends
// on the state, so they are drawn before the blocks, spread over the
// particle's lanes and the workgroup's waves -- pair or uniform r by lane r
// mod (W << lsl) -- where every lane of a particle used to draw every pair,
// one after the other, in each block's chain (about 250 dependent
// instructions each).  1000 particles of 1000 points, K = 4: 58 -> 51 us a
// step with its other launches; 16384: 124 -> 121 us.  Row q of `zs`:
// coordinate q; row D + b: log U of block b; one column a particle (WAVE >>
// lsl of them).
template <int K>
constexpr int gmm_draw_doubles() { return (3 * K - 1 + 3) * WAVE; }

template <int K, bool SLICED>
__device__ __forceinline__ void sweep_draws(const Prob &P, int W, int lsl, int64_t tile,
                                            uint32_t t, int sweep, double *zs)
{
    constexpr int D = 3 * K - 1, NB = K == 1 ? 2 : 3;
    constexpr int PK = (K + 1) / 2, PAIRS = 2 * PK + K / 2;  // K / 2 pairs for the K - 1 logits
    if (!SLICED)
        lsl = 0;
    const int lane = lane_id(), col = lane >> lsl, cols = WAVE >> lsl;
    const int64_t i = tile * cols + col;
    const uint32_t ii = (uint32_t)(i < P.n ? i : 0);
    for (int r = (wave_id() << lsl) + (lane & ((1 << lsl) - 1)); r < PAIRS + NB; r += W << lsl) {
        const bool pair = r < PAIRS;
        const int b = pair ? min(r / PK, 2) : r - PAIRS;
        draw_item<K>(P, ii, t, sweep, pair, b, r - b * PK, zs + b * K * cols + col,
                     zs + (D + b) * cols + col, cols);
    }
}

// The same of one block, one lane a particle: the normals to `z`, log U to `u`.
template <int K>
__device__ __forceinline__ void block_draws(const Prob &P, int W, int64_t tile, uint32_t t,
                                            int sweep, int b, double *z, double *u)
{
    const int lane = lane_id();
    const int64_t i = tile * WAVE + lane;
    const uint32_t ii = (uint32_t)(i < P.n ? i : 0);
    const int pairs = b == 2 ? K / 2 : (K + 1) / 2;
    for (int r = wave_id(); r < pairs + 1; r += W)
        draw_item<K>(P, ii, t, sweep, r < pairs, b, r, z + lane, u + lane, WAVE);
}

// `draws` (coordinate q in row q + z0) and `logu` (the block's numbers), `red`
// (gmm_red_doubles(W)), `stash` (gmm_stash_doubles<K, MALA>()) and, for the LDS
// hand-off modes `io`, `hand` (gmm_hand_doubles(K, MALA)) are the caller's LDS.
// With GMM_IO_GLOBAL the block reads `src` and writes `dst` (every row when
// `full`, else the accepted rows in place).
template <int K, bool MALA, bool SLICED>
__device__ __forceinline__ void gmm_block_tile(const Prob &P, const double *__restrict__ src,
                                               double *__restrict__ dst, int full, int W, int lsl,
                                               int64_t tile, int block, double alpha,
                                               double scale, int32_t step, const double *draws,
                                               int z0, const double *logu, double *red,
                                               double *stash, int io = GMM_IO_GLOBAL,
                                               double *hand = nullptr)
{
    constexpr int D = 3 * K - 1;
    using S = BlockStash<K, MALA>;
    const bool in_lds = io == GMM_IO_LDS || io == GMM_IO_LAST;
    const bool out_lds = io == GMM_IO_FIRST || io == GMM_IO_LDS;
    const bool out_all = full || io != GMM_IO_GLOBAL;
    const int32_t *__restrict__ anc = P.anc;
    const int64_t n = P.n, nd = P.n_data;
    const double *__restrict__ y = P.data;
    const GmmPrior pr = P.prior;
    double *__restrict__ hist = P.hist;
    const int64_t hist_len = P.hist_len;
    const bool gather = full && !in_lds && P.scalars[SMC_S_RESAMPLED] != 0.0;
    const int lane = lane_id();
    const LaneMap lm(tile, SLICED ? lsl : 0);
    const int64_t i = lm.i;
    const bool valid = i < n;
    // the state is read from column si of rows of length sn (global: the
    // particle or its ancestor; LDS: the particle's leading lane) and written
    // by that lane to column wi of rows of length wn
    const int64_t si = in_lds ? lm.col : (valid ? (gather ? (int64_t)anc[i] : i) : 0);
    const int64_t sn = in_lds ? WAVE : n;
    const double *__restrict__ rs = in_lds ? hand : src;
    double *__restrict__ ws = out_lds ? hand : dst;
    const int64_t wi = out_lds ? lane : i;
    const int64_t wn = out_lds ? WAVE : n;
    const int zn = SLICED ? WAVE >> lsl : WAVE;
    const int zcol = SLICED ? lane >> lsl : lane;
    const double *zs = draws + z0 * zn + zcol;
    const int off = block * K;
    const int dim = block == 2 ? K - 1 : K;
    const double h2 = scale * scale;
    MixLik<K, MALA, MALA && (K > 14)> L;
    {
        Proposal<K, MALA> Q;
        Q.build(rs, sn, si, zs, zn, block, alpha, scale, pr);
        double logw[K];
        log_weights<K>(Q.prop, logw);
        L.setup(Q.prop, logw);
        if (__builtin_amdgcn_readfirstlane(wave_id()) == W - 1) {
            stash[S::LPP * WAVE + lane] = log_prior<K>(Q.prop, logw, pr);
#pragma unroll
            for (int q = 0; q < D; ++q) {
                const int mm = q - off;
                if (mm >= 0 && mm < dim) {
                    stash[(S::PROP + mm) * WAVE + lane] = Q.prop[q];
                    if (MALA)
                        stash[(S::GP + mm) * WAVE + lane] = log_prior_grad<K>(Q.prop, logw, pr, q);
                }
            }
            if (MALA) {
                stash[S::FWD * WAVE + lane] = Q.fwd;
#pragma unroll
                for (int j = 0; j < K - 1; ++j)
                    stash[(S::ZC + j) * WAVE + lane] = exp_d(logw[j]);
            }
        }
    }
    int64_t k0, k1;
    data_chunk(nd, W, &k0, &k1);
    L.template chunk<SLICED>(y, k0, k1, lsl);
    double ll0 = 0.0, lp0 = 0.0;
    if (wave_id() == 0) {
        ll0 = rs[(int64_t)D * sn + si];
        lp0 = rs[(int64_t)(D + 1) * sn + si];
    }
    combine_waves<SLICED>(L, W, lsl, red);
    if (wave_id() != 0)
        return;
    double phi[D > 0 ? D : 1];
#pragma unroll
    for (int q = 0; q < D; ++q)
        phi[q] = rs[(int64_t)q * sn + si];
    const double lpp = stash[S::LPP * WAVE + lane];
    const double cur = alpha == 0.0 ? lp0 : lp0 + alpha * ll0;
    double logr = (alpha == 0.0 ? lpp : lpp + alpha * L.ll) - cur;
    double gnew[MALA ? D : 1];
    if (MALA) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            gnew[j] = L.gmu[j];
            gnew[K + j] = L.geta[j];
            if (j < K - 1)
                gnew[2 * K + j] = L.gr[j] - (double)nd * stash[(S::ZC + j) * WAVE + lane];
        }
        double bwd = 0.0;
#pragma unroll
        for (int q = 0; q < D; ++q) {
            const int mm = q - off;
            if (mm >= 0 && mm < dim) {
                double g2 = stash[(S::GP + mm) * WAVE + lane];
                if (alpha != 0.0)
                    g2 += alpha * gnew[q];
                const double b = phi[q] - stash[(S::PROP + mm) * WAVE + lane] - 0.5 * h2 * g2;
                bwd += b * b;
            }
        }
        logr += (stash[S::FWD * WAVE + lane] - bwd) / (2.0 * h2);
    }
    const bool acc = valid && lm.lead && logu[zcol] <= logr;
    if (lm.lead && (valid || out_lds)) {
        if (out_all) {
#pragma unroll
            for (int q = 0; q < D; ++q) {
                const int mm = q - off;
                const bool inb = mm >= 0 && mm < dim;
                ws[(int64_t)q * wn + wi] =
                    (acc && inb) ? stash[(S::PROP + (inb ? mm : 0)) * WAVE + lane] : phi[q];
            }
            ws[(int64_t)D * wn + wi] = acc ? L.ll : ll0;
            ws[(int64_t)(D + 1) * wn + wi] = acc ? lpp : lp0;
            if (MALA) {
#pragma unroll
                for (int q = 0; q < D; ++q)
                    ws[(int64_t)(D + 2 + q) * wn + wi] =
                        acc ? gnew[q] : rs[(int64_t)(D + 2 + q) * sn + si];
            }
        } else if (acc) {
#pragma unroll
            for (int q = 0; q < D; ++q) {
                const int mm = q - off;
                if (mm >= 0 && mm < dim)
                    ws[(int64_t)q * wn + wi] = stash[(S::PROP + mm) * WAVE + lane];
            }
            ws[(int64_t)D * wn + wi] = L.ll;
            ws[(int64_t)(D + 1) * wn + wi] = lpp;
            if (MALA) {
#pragma unroll
                for (int q = 0; q < D; ++q)
                    ws[(int64_t)(D + 2 + q) * wn + wi] = gnew[q];
            }
        }
    }
    // count accepted proposals of this wave
    const unsigned long long bal = __ballot(acc);
    if (lane == 0 && hist && step >= 0 && step < hist_len && bal)
        atomicAdd(&hist[(int64_t)step * SMC_HIST_COLS + SMC_H_ACC0 + block],
                  (double)__popcll(bal));
}

// The wave-combine buffer and the draws are the step kernel's dynamic LDS, as
// long as its waves need: with few data points a workgroup has one to four
// waves, and LDS decides how many of them a compute unit holds (MALA, K = 4,
// 2^16 particles of 50 points: 147 us at three workgroups a compute unit, the
// buffer as long as for eight waves, 77 at five).  For the same reason a single
// wave draws for one block at a time, into the rows that the proposal then
// takes (its lanes read only their own column), and two or four waves do it,
// into rows of their own, for as many components as the shorter buffer gains
// them a workgroup.  us a step, with the whole sweep's draws / by block (before
// the draws were spread): random walk, K = 11, 2^16 particles of 50 points 280 /
// 135 (137); MALA, K = 8, 288 / 145 (233); MALA, K = 14, 200000 of 200 points
// 3250 / 2230 (2950).  Where it gains nothing, its barriers cost 1 to 5 %.
constexpr bool gmm_draws_by_block(int K, int W, int lsl)
{
    return lsl == 0 && (W == 1 || (W < GMM_MAXW && K > 3 * W));
}

template <int K>
unsigned gmm_step_lds(int W, int lsl)
{
    const int draws = !gmm_draws_by_block(K, W, lsl) ? gmm_draw_doubles<K>() >> lsl
                      : W > 1                        ? K * WAVE
                                                     : 0;
    return sizeof(double) * (unsigned)(gmm_red_doubles(W) + draws);
}

// Waves a SIMD holds of gmm_step_kernel.  A random walk with K <= 4 fits two
// workgroups of eight waves on a compute unit (128 registers); MALA with K <= 3
// three waves (K = 2, 2^16 particles of 200 points: 95 us at the 171 registers
// it would take, 87 at 168; K = 3, 200000 of 200, 450 us at 192 registers, 373
// at 168), but for K = 3 where lanes share a particle (256 of 1000 points 7 %
// slower so).
constexpr int gmm_step_waves(int K, bool MALA, bool SLICED)
{
    return K <= 4 && !MALA ? 4 : (K <= 2 || (K == 3 && !SLICED) ? 3 : 2);
}

// All Metropolis blocks of a step (every sweep) in one launch: the tile's
// workgroup runs the blocks one after the other.  The first block reads
// `src` (through the ancestors when the step resampled and `full` is set)
// and leaves the tile's state in LDS; each later block reads the state the
// previous block's wave 0 left there (visible to the workgroup after the
// barrier), and the last one writes the whole state to `dst`.
template <int K, bool MALA, bool SLICED>
__global__ __launch_bounds__(GMM_MAXW *WAVE,
                             gmm_step_waves(K, MALA, SLICED)) void gmm_step_kernel(
    Prob P, const double *__restrict__ src, double *__restrict__ dst, int full, int W, int lsl,
    uint32_t t, int sweeps, double alpha, double s0, double s1, double s2, int32_t step)
{
    using S = BlockStash<K, MALA>;
    extern __shared__ double red[];
    __shared__ double stash[gmm_stash_doubles<K, MALA>() + WAVE];  // and a block's log U
    __shared__ double hand[gmm_hand_doubles(K, MALA)];
    constexpr int D = 3 * K - 1, nb = K == 1 ? 2 : 3;
    const bool by_block = !SLICED && gmm_draws_by_block(K, W, 0);
    const int cols = SLICED ? WAVE >> lsl : WAVE;
    double *zs = red + gmm_red_doubles(W);
    for (int sw = 0; sw < sweeps; ++sw) {
        if (!by_block) {
            if (sw > 0)
                __syncthreads();
            sweep_draws<K, SLICED>(P, W, lsl, blockIdx.x, t, sw, zs);
        }
        for (int b = 0; b < nb; ++b) {
            const bool first = sw == 0 && b == 0;
            const bool last = sw == sweeps - 1 && b == nb - 1;
            double *z = zs, *logu = zs + (D + b) * cols;
            __syncthreads();
            if (by_block) {
                if (W == 1)
                    z = stash + S::PROP * WAVE;
                logu = stash + S::ROWS * WAVE;
                block_draws<K>(P, W, blockIdx.x, t, sw, b, z, logu);
                __syncthreads();
            }
            gmm_block_tile<K, MALA, SLICED>(
                P, src, dst, first ? full : 0, W, lsl, blockIdx.x, b, alpha,
                b == 0 ? s0 : (b == 1 ? s1 : s2), step, z, by_block ? -b * K : 0, logu, red,
                stash, first ? GMM_IO_FIRST : (last ? GMM_IO_LAST : GMM_IO_LDS), hand);
        }
    }
}

// ---------------------------------------------------------------------------
// Log-likelihood (and gradient) for separate parameter arrays (the adjoint
// entry point).
// ---------------------------------------------------------------------------
// Four waves per SIMD (128 registers) up to four components: K = 4 with the
// gradient would take 141, and 2^16 vectors of 1000 points 249 us against 224
// (where lanes share a particle it spills six registers).
template <int K, bool GRAD, bool SLICED>
__global__ __launch_bounds__(GMM_MAXW *WAVE, K <= 4 ? 4 : 2) void gmm_loglik_kernel(
    const double *__restrict__ mu, const double *__restrict__ eta, const double *__restrict__ z,
    int64_t n, const double *__restrict__ y, int64_t nd, int W, int lsl, double *__restrict__ ll,
    double *__restrict__ grad)
{
    constexpr int D = 3 * K - 1;
    __shared__ double red[gmm_red_doubles(GMM_MAXW)];
    const LaneMap lm(blockIdx.x, SLICED ? lsl : 0);
    const int64_t i = lm.i;
    const bool valid = i < n;
    const int64_t si = valid ? i : 0;
    double phi[D > 0 ? D : 1];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        phi[j] = mu[(int64_t)j * n + si];
        phi[K + j] = eta[(int64_t)j * n + si];
        if (j < K - 1)
            phi[2 * K + j] = z[(int64_t)j * n + si];
    }
    double logw[K];
    log_weights<K>(phi, logw);
    MixLik<K, GRAD> L;
    L.setup(phi, logw);
    int64_t k0, k1;
    data_chunk(nd, W, &k0, &k1);
    L.template chunk<SLICED>(y, k0, k1, lsl);
    combine_waves<SLICED>(L, W, lsl, red);
    if (wave_id() == 0 && valid && lm.lead) {
        ll[i] = L.ll;
        if (GRAD) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                grad[(int64_t)j * n + i] = L.gmu[j];
                grad[(int64_t)(K + j) * n + i] = L.geta[j];
                if (j < K - 1)
                    grad[(int64_t)(2 * K + j) * n + i] = z_grad<K>(L.gr[j], logw[j], nd);
            }
        }
    }
}

// Host launchers of the K-templated kernels; explicitly instantiated in the
// smc_gmm_k*.hip translation units (compiled in parallel).
template <int K>
struct GmmK {
    static hipError_t init(Ctx &c, GmmSplit sp);
    static hipError_t step(Ctx &c, GmmSplit sp, int32_t step, int sweeps, double alpha,
                           const double (&scale)[3], bool gather_check);
    static hipError_t loglik(const double *mu, const double *eta, const double *z, int64_t n,
                             const double *y, int64_t nd, double *ll, double *grad, hipStream_t s);
    static hipError_t init_batch(const Prob *probs, const int2 *map, int64_t tiles, GmmSplit sp,
                                 bool mala, hipStream_t s);
};

template <int K>
hipError_t GmmK<K>::init(Ctx &c, GmmSplit sp)
{
    const dim3 grid((unsigned)ceil_div(c.n, WAVE >> sp.lsl)), block((unsigned)(sp.W * WAVE));
    const Prob P = make_prob(c);
#define SMC_INIT(GRAD, SLICED)                                                                    \
    hipLaunchKernelGGL((gmm_init_kernel<K, GRAD, SLICED>), grid, block, 0, c.stream, P, sp.W,     \
                       sp.lsl)
    if (c.cfg.move_kind == SMC_MOVE_MALA) {
        if (sp.lsl > 0)
            SMC_INIT(true, true);
        else
            SMC_INIT(true, false);
    } else {
        if (sp.lsl > 0)
            SMC_INIT(false, true);
        else
            SMC_INIT(false, false);
    }
#undef SMC_INIT
    return hipGetLastError();
}

template <int K>
hipError_t GmmK<K>::step(Ctx &c, GmmSplit sp, int32_t step, int sweeps, double alpha,
                         const double (&scale)[3], bool gather_check)
{
    const dim3 grid((unsigned)ceil_div(c.n, WAVE >> sp.lsl)), blk((unsigned)(sp.W * WAVE));
    const double *src = (const double *)c.state_ptr();
    double *dst = gather_check ? (double *)c.other_ptr() : (double *)c.state_ptr();
    const Prob P = make_prob(c);
    const unsigned lds = gmm_step_lds<K>(sp.W, sp.lsl);
    hipEvent_t e0, e1;
    const bool timed = c.prof_take(&e0, &e1);
#define SMC_STEP_ARGS                                                                             \
    P, src, dst, (int)gather_check, sp.W, sp.lsl, (uint32_t)step, sweeps, alpha, scale[0],        \
        scale[1], scale[2], step
#define SMC_STEP(MALA, SLICED)                                                                    \
    do {                                                                                          \
        if (timed)                                                                                \
            hipExtLaunchKernelGGL((gmm_step_kernel<K, MALA, SLICED>), grid, blk, lds, c.stream,   \
                                  e0, e1, 0, SMC_STEP_ARGS);                                      \
        else                                                                                      \
            hipLaunchKernelGGL((gmm_step_kernel<K, MALA, SLICED>), grid, blk, lds, c.stream,      \
                               SMC_STEP_ARGS);                                                    \
    } while (0)
    if (c.cfg.move_kind == SMC_MOVE_MALA) {
        if (sp.lsl > 0)
            SMC_STEP(true, true);
        else
            SMC_STEP(true, false);
    } else {
        if (sp.lsl > 0)
            SMC_STEP(false, true);
        else
            SMC_STEP(false, false);
    }
#undef SMC_STEP
#undef SMC_STEP_ARGS
    return hipGetLastError();
}

template <int K>
hipError_t GmmK<K>::loglik(const double *mu, const double *eta, const double *z, int64_t n,
                                  const double *y, int64_t nd, double *ll, double *grad,
                                  hipStream_t s)
{
    const GmmSplit sp = gmm_split(n, nd, K, GMM_SETUP_LOGLIK);
    const dim3 grid((unsigned)ceil_div(n, WAVE >> sp.lsl)), blk((unsigned)(sp.W * WAVE));
#define SMC_LOGLIK(GRAD, SLICED)                                                                  \
    hipLaunchKernelGGL((gmm_loglik_kernel<K, GRAD, SLICED>), grid, blk, 0, s, mu, eta, z, n, y,   \
                       nd, sp.W, sp.lsl, ll, grad)
    if (grad) {
        if (sp.lsl > 0)
            SMC_LOGLIK(true, true);
        else
            SMC_LOGLIK(true, false);
    } else {
        if (sp.lsl > 0)
            SMC_LOGLIK(false, true);
        else
            SMC_LOGLIK(false, false);
    }
#undef SMC_LOGLIK
    return hipGetLastError();
}

template <int K>
hipError_t GmmK<K>::init_batch(const Prob *probs, const int2 *map, int64_t tiles, GmmSplit sp,
                                      bool mala, hipStream_t s)
{
    const dim3 grid((unsigned)(tiles << sp.lsl)), blk((unsigned)(sp.W * WAVE));
#define SMC_INIT(GRAD, SLICED)                                                                    \
    hipLaunchKernelGGL((gmm_init_batch_kernel<K, GRAD, SLICED>), grid, blk, 0, s, probs, map,     \
                       sp.W, sp.lsl)
    if (mala) {
        if (sp.lsl > 0)
            SMC_INIT(true, true);
        else
            SMC_INIT(true, false);
    } else {
        if (sp.lsl > 0)
            SMC_INIT(false, true);
        else
            SMC_INIT(false, false);
    }
#undef SMC_INIT
    return hipGetLastError();
}


}  // namespace smc
