// Fold of the per-view sums into the normal equations and the regularised
// solve (eqs. 11-14, Algorithm 1 steps 5-6).
//
// L >= 1: four lanes per Gaussian.  Lane r owns the rows i = 4k + r of
//   A_g = sum_j V_gj phi_gj phi_gj^T  and  B_g = sum_j phi_gj S_gj^T
// and accumulates them over the views in FP64 registers (FP32 accumulation
// of A over tens of views loses ~1e-4 relative at the condition numbers the
// paper's Lambda produces).  The quad then factors A_g + w_g Lambda with a
// cooperative FP64 Cholesky and solves four right-hand-side columns at a
// time, all in registers; the factor stays there for further channel chunks.
// L = 0: A_g = w_g Y0^2 is a scalar and c_g = Y0 S_g / (w_g (Y0^2 + lambda_0)).
#include <algorithm>
#include <type_traits>

#include "gsc_internal.h"
#include "sh.h"

namespace gsc {

struct LamNB {
    double v[kMaxNb];
};

// The observed Gaussians of per-view sums (device): list[0 .. *n_list), and per
// Gaussian one bit per view that gave it weight.
struct ObsList {
    uint64_t* seen;
    uint32_t* list;
    uint32_t* counts;
    uint32_t* n_list;
    uint8_t* cls;
};

constexpr double kY0 = 0.28209479177387814;

__global__ void k_solve_dc(const SumRows sums, int64_t N, int C, double lam0,
                           float* __restrict__ coeffs, uint8_t* __restrict__ status,
                           float* __restrict__ wout) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= N) return;
    const float* s = sums.s + g * (int64_t)sums.s_stride;
    double w = sums.v[g * sums.v_stride];
    if (wout) wout[g] = (float)w;
    float* out = coeffs + g * C;
    if (w == 0.0) {
        for (int c = 0; c < C; ++c) out[c] = 0.0f;
        if (status) status[g] = GSC_G_UNOBSERVED;
        return;
    }
    double den = w * (kY0 * kY0 + lam0);
    for (int c = 0; c < C; ++c) out[c] = (float)(kY0 * (double)s[c] / den);
    if (status) status[g] = 0;
}

// Sum the per-view slots of every Gaussian over the views (L = 0 with
// per-view sums kept for the caller).
__global__ void k_sum_views(const float* __restrict__ VS, int n_views, int64_t N, int stride,
                            float* __restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N * stride) return;
    float a = 0.0f;
    for (int v = 0; v < n_views; ++v) a += VS[(int64_t)v * N * stride + i];
    out[i] = a;
}

// Broadcast lane `o` of each quad to the whole quad (DPP quad_perm [o,o,o,o]).
template <int O>
__device__ __forceinline__ double quad_bcast(double x) {
    constexpr int ctrl = O | (O << 2) | (O << 4) | (O << 6);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Lane u of each quad to the whole quad (u a constant once unrolled).
__device__ __forceinline__ float quad_bcast_f(float x, int u) {
    const int i = __float_as_int(x);
    switch (u) {
        case 0: return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x00, 0xF, 0xF, false));
        case 1: return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x55, 0xF, 0xF, false));
        case 2: return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xAA, 0xF, 0xF, false));
        default: return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xFF, 0xF, 0xF, false));
    }
}

// Sum over the quad (DPP quad_perm [1,0,3,2] then [2,3,0,1]); every lane of
// the quad gets the same value.
__device__ __forceinline__ double quad_sum(double x) {
    constexpr int x1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);
    constexpr int x2 = 2 | (3 << 2) | (0 << 4) | (1 << 6);
    x += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), x1, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), x1, 0xF, 0xF, false));
    x += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), x2, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), x2, 0xF, 0xF, false));
    return x;
}

__device__ __forceinline__ double quad_max(double x) {
    constexpr int x1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);
    constexpr int x2 = 2 | (3 << 2) | (0 << 4) | (1 << 6);
    x = fmax(x, __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), x1, 0xF, 0xF, false),
                                 __builtin_amdgcn_update_dpp(0, __double2loint(x), x1, 0xF, 0xF, false)));
    x = fmax(x, __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), x2, 0xF, 0xF, false),
                                 __builtin_amdgcn_update_dpp(0, __double2loint(x), x2, 0xF, 0xF, false)));
    return x;
}

// Unit direction from a camera centre (FP64) to a Gaussian mean, in FP64:
// the normal equations are assembled in FP64, and a direction rounded to
// binary32 would perturb A_g by an amount that weak regularisation does not
// damp.  1/|d| from the hardware reciprocal square root refined by three
// Newton steps y <- y (3/2 - n y^2 / 2), each of which squares the relative
// error (full FP64 from any start better than 2^-12), at a fraction of the
// cost of a square root and a division.
__device__ __forceinline__ void view_direction(float mx, float my, float mz, const double* centre,
                                               double* dir) {
    const double dx = (double)mx - centre[0];
    const double dy = (double)my - centre[1];
    const double dz = (double)mz - centre[2];
    const double n2 = dx * dx + dy * dy + dz * dz;
    if (!(n2 > 0.0)) {  // a mean at the camera centre: culled there, any unit vector will do
        dir[0] = 0.0;
        dir[1] = 0.0;
        dir[2] = 1.0;
        return;
    }
    double inv = __builtin_amdgcn_rsq(n2);
#pragma unroll
    for (int k = 0; k < 3; ++k) inv = inv * fma(-0.5 * n2 * inv, inv, 1.5);
    dir[0] = dx * inv;
    dir[1] = dy * inv;
    dir[2] = dz * inv;
}

// Broadcast from quad lane j & 3.
__device__ __forceinline__ double quad_from(double x, int j) {
    switch (j & 3) {
        case 0: return quad_bcast<0>(x);
        case 1: return quad_bcast<1>(x);
        case 2: return quad_bcast<2>(x);
        default: return quad_bcast<3>(x);
    }
}

// Fold + solve for L >= 1.  Four lanes (a quad) per Gaussian; lane r owns
// the rows i = 4k + r of A (lower triangle) and of the right-hand sides,
// four channels at a time, all in FP64 registers.  The quad walks the views
// that gave its Gaussian weight (seen, one bit per view), four at a time:
// lane r takes the r-th, loads its sums (the next four are in flight while
// four are folded), evaluates the SH basis of its direction and shares it
// through LDS; then all lanes fold the four views in order.  Quads of a wave
// have Gaussians seen by about as many views (the list is ordered by that
// number), as a wave walks as long as its longest.  The Cholesky factor is
// formed in place (column j broadcast within the quad; the owner of row j
// keeps 1/L_jj on the diagonal), forward substitution broadcasts each solved
// entry to the quad, and back substitution sums each column's products over
// the quad.
//
// Bound by FP64 issue and latency at one wave per SIMD.  100k Gaussians, 50
// views, 35% of them seen per observed Gaussian: 281 -> 95 us (before, every
// lane evaluated the basis of every view, seen or not, and every Gaussian took
// the condition iterations below).
//
// ADJ: adjoint solve for the backward pass.  VS then holds only the per-view
// visibilities (stride 1); the right-hand sides are read from `rhs`
// (dL/dc, [N][NB][C]) instead of being folded, the solution
// Bbar = (A + w Lambda)^{-1} dL/dc is written to `out`, and
// rho_g = sum_{m,c} lambda_m Bbar[m][c] cin[m][c] (cin = the forward
// coefficients) to rho[g].
template <int L, bool ADJ>
__global__ __launch_bounds__(64) void k_fold_solve(const ViewInfo* __restrict__ views, int n_views,
                                                   const float* __restrict__ means,
                                                   const float* __restrict__ VS, int vs_stride,
                                                   int64_t N, int C, LamNB lam, float kappa_max,
                                                   const float* __restrict__ rhs,
                                                   const float* __restrict__ cin,
                                                   float* __restrict__ coeffs,
                                                   float* __restrict__ rho,
                                                   uint8_t* __restrict__ status,
                                                   float* __restrict__ wout,
                                                   unsigned int* __restrict__ ill_count,
                                                   double* __restrict__ factor, ObsList obs) {
    constexpr int NB = (L + 1) * (L + 1);
    constexpr int RPL = (NB + 3) / 4;  // rows per lane
    constexpr int NP = (NB + 1) / 2;   // pairs of SH values
    __shared__ double2 sphi[NP][64];   // [pair][view of the four * 16 + quad]
    const int r = threadIdx.x & 3;
    // quad q takes the q-th observed Gaussian; a wave past the end of the list
    // has nothing to do (one wave per block: no block barrier below)
    const int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
    const bool valid = q < (int64_t)*obs.n_list;
    if (__builtin_amdgcn_ballot_w64(valid) == 0) return;
    const int64_t g = valid ? (int64_t)obs.list[q] : 0;
    const int stride = vs_stride;
    float mx = 0.f, my = 0.f, mz = 0.f;
    if (valid) {
        mx = means[3 * g];
        my = means[3 * g + 1];
        mz = means[3 * g + 2];
    }
    double sel[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) sel[e] = r == e ? 1.0 : 0.0;
    // accA[k][j]: row 4k+r, column j <= 4k+r; after the factorisation the
    // owner's diagonal entry holds 1/L_ii
    double accA[RPL][NB];
    bool failed = false;
    double wsum = 0.0, msum = 0.0;
    double rho_part = 0.0;
    const uint32_t tw = threadIdx.x >> 2;  // the quad
    const int words = (n_views + 63) / 64;
    const uint64_t* seen = obs.seen + g * (int64_t)words;
    for (int c0 = 0; c0 < C; c0 += 4) {
        const bool firstc = c0 == 0;
        double accB[RPL][4];
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (firstc) accA[k][j] = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) accB[k][c] = 0.0;
        }
        double wv = 0.0;
        const float* slot = VS + g * (int64_t)stride;
        const int64_t vstep = N * (int64_t)stride;
        struct Seen {
            int v;            // the lane's view, -1: none
            float V, S[4];
            double centre[3];
        };
        int wi = 0;
        uint64_t left = 0;
        const int nw = (!ADJ || firstc) ? words : 0;
        if (nw > 0 && valid) left = seen[0];
        auto next = [&](Seen& e) {
            // to the next word with views left (quads move on their own)
            while (left == 0 && ++wi < nw && valid) left = seen[wi];
            const uint64_t m1 = left & (left - 1), m2 = m1 & (m1 - 1), m3 = m2 & (m2 - 1);
            const uint64_t m = r == 0 ? left : (r == 1 ? m1 : (r == 2 ? m2 : m3));
            e.v = m != 0 ? 64 * wi + (int)__builtin_ctzll(m) : -1;
            left = m3 & (m3 - 1);
            const int v = e.v >= 0 ? e.v : 0;
            const float* p = slot + (int64_t)v * vstep;
            const float V = p[0];
            e.V = e.v >= 0 ? V : 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float s = 0.0f;
                if (!ADJ && c0 + c < C) s = p[1 + c0 + c];
                e.S[c] = e.v >= 0 ? s : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) e.centre[k] = views[v].centre[k];
        };
        // FIRST: also A and w (the first four channels)
        auto fold = [&](auto first) {
            constexpr bool FIRST = decltype(first)::value;
            Seen cur, nxt;
            next(cur);
            while (__builtin_amdgcn_ballot_w64(cur.v >= 0) != 0) {
            next(nxt);
            {
                double dir[3], phi[2 * NP];
                view_direction(mx, my, mz, cur.centre, dir);
                double ph[NB];
                sh_eval<double, L>(dir[0], dir[1], dir[2], ph);
#pragma unroll
                for (int j = 0; j < 2 * NP; ++j) phi[j] = j < NB ? ph[j < NB ? j : 0] : 0.0;
#pragma unroll
                for (int j = 0; j < NP; ++j) sphi[j][16 * r + tw] = make_double2(phi[2 * j], phi[2 * j + 1]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // (a view past a quad's last adds exact zeros)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double Vd = (double)quad_bcast_f(cur.V, u);
                double ph[2 * NP], own[RPL];
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const double2 p = sphi[j][16 * u + tw];
                    ph[2 * j] = p.x;
                    ph[2 * j + 1] = p.y;
                }
#pragma unroll
                for (int k = 0; k < RPL; ++k) {
                    own[k] = sel[0] * ph[4 * k];
#pragma unroll
                    for (int e = 1; e < 4; ++e)
                        if (4 * k + e < NB) own[k] = fma(sel[e], ph[4 * k + e < NB ? 4 * k + e : 0], own[k]);
                }
                if constexpr (FIRST) {
#pragma unroll
                    for (int k = 0; k < RPL; ++k) {
                        const double vo = Vd * own[k];
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            if (j < 4 * k + 4) accA[k][j] = fma(vo, ph[j], accA[k][j]);
                    }
                }
                if constexpr (!ADJ) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const double sc = (double)quad_bcast_f(cur.S[c], u);
#pragma unroll
                        for (int k = 0; k < RPL; ++k) accB[k][c] = fma(own[k], sc, accB[k][c]);
                    }
                }
                if constexpr (FIRST) wv += Vd;
            }
            __builtin_amdgcn_wave_barrier();  // the next four overwrite the values
            cur = nxt;
            }
        };
        if (firstc) {
            if (nw > 0) fold(std::true_type{});
        } else if constexpr (!ADJ) {
            if (nw > 0) fold(std::false_type{});
        }
        if (firstc) {
            wsum = wv;
            // regularise: the lane's own diagonal entries, selected arithmetically
#pragma unroll
            for (int k = 0; k < RPL; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * k + e < NB)
                        accA[k][4 * k + e < NB ? 4 * k + e : 0] =
                            fma(sel[e] * wsum, lam.v[4 * k + e < NB ? 4 * k + e : 0],
                                accA[k][4 * k + e < NB ? 4 * k + e : 0]);
            // trace of the matrix (for the condition estimate)
            if constexpr (!ADJ) {
                double t = 0.0;
#pragma unroll
                for (int k = 0; k < RPL; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (4 * k + e < NB) t = fma(sel[e], accA[k][4 * k + e < NB ? 4 * k + e : 0], t);
                msum = quad_sum(t);
            }
            // Right-looking Cholesky in registers.  Column j is scaled by its
            // owner rows, then each entry L[m][j] is broadcast from the lane
            // owning row m and every lane updates its own rows i >= m.
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                double djj;
                switch (j & 3) {
                    case 0: djj = quad_bcast<0>(accA[j >> 2][j]); break;
                    case 1: djj = quad_bcast<1>(accA[j >> 2][j]); break;
                    case 2: djj = quad_bcast<2>(accA[j >> 2][j]); break;
                    default: djj = quad_bcast<3>(accA[j >> 2][j]); break;
                }
                const bool bad = !(djj > 0.0);
                failed |= bad;
                const double d = bad ? 1.0 : sqrt(djj);
                const double id = 1.0 / d;
#pragma unroll
                for (int k = 0; k < RPL; ++k)
                    if (4 * k + 3 >= j) {
                        const int i = 4 * k + r;
                        accA[k][j] = i > j ? accA[k][j] * id : (i == j ? id : accA[k][j]);
                    }
#pragma unroll
                for (int m = j + 1; m < NB; ++m) {
                    double lmj;
                    switch (m & 3) {
                        case 0: lmj = quad_bcast<0>(accA[m >> 2][j]); break;
                        case 1: lmj = quad_bcast<1>(accA[m >> 2][j]); break;
                        case 2: lmj = quad_bcast<2>(accA[m >> 2][j]); break;
                        default: lmj = quad_bcast<3>(accA[m >> 2][j]); break;
                    }
#pragma unroll
                    for (int k = 0; k < RPL; ++k)
                        if (4 * k + 3 >= m) {  // rows 4k..4k+3 may reach column m
                            const bool act = 4 * k + r >= m;  // own row i = 4k + r needs i >= m
                            accA[k][m] = act ? fma(-accA[k][j], lmj, accA[k][m]) : accA[k][m];
                        }
                }
            }
            // keep the factor for refinement: row i at i (i + 1) / 2, 1/L_ii
            // on the diagonal, then w_g
            if constexpr (!ADJ) {
                if (factor != nullptr && valid) {
                    constexpr int NT = NB * (NB + 1) / 2;
                    double* F = factor + g * (int64_t)(NT + 1);
#pragma unroll
                    for (int k = 0; k < RPL; ++k) {
                        const int i = 4 * k + r;
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            if (j < 4 * k + 4 && j <= i && i < NB) F[i * (i + 1) / 2 + j] = accA[k][j];
                    }
                    if (r == 0) F[NT] = wsum;
                }
            }
        }
        if constexpr (ADJ) {
#pragma unroll
            for (int k = 0; k < RPL; ++k) {
                const int i = 4 * k + r;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    accB[k][c] = (valid && i < NB && c0 + c < C) ? (double)rhs[(g * NB + i) * C + c0 + c] : 0.0;
            }
        }
        // forward substitution L y = b: y_j = b_j / L_jj is broadcast from its
        // owner, and every lane updates its own rows m > j
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int kj = j >> 2;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double t = accB[kj][c] * accA[kj][j];
                double yj;
                switch (j & 3) {
                    case 0: yj = quad_bcast<0>(t); break;
                    case 1: yj = quad_bcast<1>(t); break;
                    case 2: yj = quad_bcast<2>(t); break;
                    default: yj = quad_bcast<3>(t); break;
                }
                accB[kj][c] = r == (j & 3) ? yj : accB[kj][c];
#pragma unroll
                for (int k = 0; k < RPL; ++k)
                    if (4 * k + 3 > j) {
                        const bool act = 4 * k + r > j && 4 * k + r < NB;
                        accB[k][c] = act ? fma(-accA[k][j], yj, accB[k][c]) : accB[k][c];
                    }
            }
        }
        // back substitution L^T x = y: x_i = (y_i - sum_{k>i} L_ki x_k) / L_ii,
        // the sum taken over each lane's solved rows, then over the quad
#pragma unroll
        for (int i = NB - 1; i >= 0; --i) {
            const int ki = i >> 2;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double p = 0.0;
#pragma unroll
                for (int k = 0; k < RPL; ++k)
                    if (4 * k + 3 > i) {
                        const bool act = 4 * k + r > i && 4 * k + r < NB;
                        p = act ? fma(accA[k][i], accB[k][c], p) : p;
                    }
                p = quad_sum(p);
                accB[ki][c] = r == (i & 3) ? (accB[ki][c] - p) * accA[ki][i] : accB[ki][c];
            }
        }
        const bool zero = wsum == 0.0 || failed;
        if (valid) {
            float* out = coeffs + g * NB * C;
#pragma unroll
            for (int k = 0; k < RPL; ++k) {
                const int i = 4 * k + r;
                if (i >= NB) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c0 + c >= C) continue;
                    out[i * C + c0 + c] = zero ? 0.0f : (float)accB[k][c];
                    if constexpr (ADJ) {
                        double lk = lam.v[4 * k];
#pragma unroll
                        for (int e = 1; e < 4; ++e)
                            if (4 * k + e < NB) lk = r == e ? lam.v[4 * k + e < NB ? 4 * k + e : 0] : lk;
                        if (!zero)
                            rho_part = fma(lk * accB[k][c], (double)cin[(g * NB + i) * C + c0 + c],
                                           rho_part);
                    }
                }
            }
        }
    }
    if constexpr (ADJ) {
        rho_part = quad_sum(rho_part);
        if (valid && r == 0) rho[g] = (float)rho_part;
        return;
    }
    // Condition.  lambda_min(M) >= w min(lambda) and lambda_max(M) <= tr M, and
    // the estimate below never exceeds kappa(M) = lambda_max / lambda_min: where
    // the bound does not reach kappa_max, nothing can be flagged and the
    // estimate is not needed (always so for the paper's Lambda, whose bound is
    // 1.3e5).  The 1e-6 covers the rounding of the sums.
    double lmin = lam.v[0];
#pragma unroll
    for (int j = 1; j < NB; ++j) lmin = fmin(lmin, lam.v[j]);
    const bool ask = valid && !failed && !(msum * (1.0 + 1e-6) <= (double)kappa_max * wsum * lmin);
    double kap = 0.0;
    if (__builtin_amdgcn_ballot_w64(ask) != 0) {
    // estimate from the extremes of 1/L_ii over the quad
    double imax = 0.0, imin = 1e300;
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        double dk = accA[k][4 * k];
#pragma unroll
        for (int e = 1; e < 4; ++e)
            if (4 * k + e < NB) dk = r == e ? accA[k][4 * k + e < NB ? 4 * k + e : 0] : dk;
        if (4 * k + r < NB) {
            imax = fmax(imax, dk);
            imin = fmin(imin, dk);
        }
    }
    imax = quad_max(imax);
    imin = -quad_max(-imin);
    // Extreme eigenvalues of M = L L^T: eight steps of power iteration give
    // lambda_max >= x^T M x / x^T x = |L^T x|^2 / |x|^2 (and lambda_max >=
    // max_i M_ii), eight of inverse iteration give 1/lambda_min >=
    // |L^{-1} x|^2 / |x|^2.  Their product is a lower bound of kappa(M) that
    // is close once the iterates align with the extreme eigenvectors (slowest
    // when the largest eigenvalues cluster); with the pivot ratio above it is
    // the estimate.  Vectors are distributed like the rows of L (row 4k + r
    // on lane r); the starts are golden-ratio sequences, free of the
    // symmetries of the SH basis that a regular start can share.
    double dia[RPL];  // the lane's own diagonal entries L_ii
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        double d = accA[k][4 * k];
#pragma unroll
        for (int e = 1; e < 4; ++e)
            if (4 * k + e < NB) d = r == e ? accA[k][4 * k + e < NB ? 4 * k + e : 0] : d;
        dia[k] = 1.0 / d;
    }
    auto lval = [&](int k, int j) {  // L[4k + r][j] for j <= 4k + r
        return 4 * k + r == j ? dia[k] : accA[k][j];
    };
    auto norm2 = [&](const double (&x)[RPL]) {
        double p = 0.0;
#pragma unroll
        for (int k = 0; k < RPL; ++k) p = 4 * k + r < NB ? fma(x[k], x[k], p) : p;
        return quad_sum(p);
    };
    auto lt_mul = [&](const double (&x)[RPL], double (&u)[RPL]) {  // u = L^T x
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            double p = 0.0;
#pragma unroll
            for (int k = 0; k < RPL; ++k)
                if (4 * k + 3 >= j) p = (4 * k + r >= j && 4 * k + r < NB) ? fma(lval(k, j), x[k], p) : p;
            p = quad_sum(p);
            if (r == (j & 3)) u[j >> 2] = p;
        }
    };
    auto l_mul = [&](const double (&u)[RPL], double (&z)[RPL]) {  // z = L u
#pragma unroll
        for (int k = 0; k < RPL; ++k) z[k] = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const double uj = quad_from(u[j >> 2], j);
#pragma unroll
            for (int k = 0; k < RPL; ++k)
                if (4 * k + 3 >= j) z[k] = (4 * k + r >= j && 4 * k + r < NB) ? fma(lval(k, j), uj, z[k]) : z[k];
        }
    };
    auto l_solve = [&](double (&x)[RPL]) {  // x <- L^{-1} x
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const double yj = quad_from(x[j >> 2] * accA[j >> 2][j], j);
            if (r == (j & 3)) x[j >> 2] = yj;
#pragma unroll
            for (int k = 0; k < RPL; ++k)
                if (4 * k + 3 > j) x[k] = (4 * k + r > j && 4 * k + r < NB) ? fma(-accA[k][j], yj, x[k]) : x[k];
        }
    };
    auto lt_solve = [&](double (&x)[RPL]) {  // x <- L^{-T} x
#pragma unroll
        for (int i = NB - 1; i >= 0; --i) {
            double p = 0.0;
#pragma unroll
            for (int k = 0; k < RPL; ++k)
                if (4 * k + 3 > i) p = (4 * k + r > i && 4 * k + r < NB) ? fma(accA[k][i], x[k], p) : p;
            p = quad_sum(p);
            if (r == (i & 3)) x[i >> 2] = (x[i >> 2] - p) * accA[i >> 2][i];
        }
    };
    double xp[RPL], xi[RPL], tmp[RPL];
    double mdiag = 0.0;  // max_i M_ii = max_i sum_j L_ij^2
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        const int i = 4 * k + r;
        const double fp = 0.6180339887498949 * i, fi = 0.7548776662466927 * i;
        xp[k] = i < NB ? 2.0 * (fp - floor(fp)) - 0.9 : 0.0;
        xi[k] = i < NB ? 2.0 * (fi - floor(fi)) - 0.9 : 0.0;
        double rn = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (j < 4 * k + 4) rn = (j <= i && i < NB) ? fma(lval(k, j), lval(k, j), rn) : rn;
        mdiag = fmax(mdiag, rn);
    }
    mdiag = quad_max(mdiag);
    double lmax_est = 0.0, sig = 0.0;
#pragma unroll 1
    for (int it = 0; it < 8; ++it) {
        const double np = norm2(xp), ni = norm2(xi);
        lt_mul(xp, tmp);
        lmax_est = norm2(tmp) / np;
        l_mul(tmp, xp);
        l_solve(xi);
        sig = norm2(xi) / ni;
        lt_solve(xi);
        const double sp = 1.0 / sqrt(norm2(xp)), si = 1.0 / sqrt(norm2(xi));
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            xp[k] *= sp;
            xi[k] *= si;
        }
    }
    kap = fmax((imax / imin) * (imax / imin), fmax(lmax_est, mdiag) * sig);
    }
    if (valid && r == 0) {
        if (wout) wout[g] = (float)wsum;
        uint8_t st = 0;
        if (wsum == 0.0) {
            st = GSC_G_UNOBSERVED;
        } else if (failed) {
            st = GSC_G_FAILED;
        } else {
            if (kap > (double)kappa_max) {
                st = GSC_G_ILL_COND;
                if (ill_count) atomicAdd(ill_count, 1u);
            }
        }
        if (status) status[g] = st;
    }
}

// Observed-list pre-pass (one Gaussian per thread, blocks of 1024): a
// Gaussian is observed when some view gave it weight.  Its views' weights are
// loaded eight at a time (independent loads in flight together); the views
// that gave it weight become its bits in `seen`.  Unobserved ones get their
// outputs here (zeros, a wave a row; GSC_G_UNOBSERVED, w = 0); the observed ones are
// put into one of kObsClasses classes by their number of views, most first, counted
// per block and class, and listed class by class.
constexpr int kObsClasses = 64;

// Past kObsSerial views the bits come from a launch of their own, a thread for 16
// views of a Gaussian: a block of 1024 alone waits for its views one group of loads
// after the other.  Fold and solve, 3 channels, us one launch / two: 4290 Gaussians
// 166 views 106 / 61, 100k 40 views 60 / 55, 500 40 views 35 / 29, 20k 24 views
// 31 / 31, 500 17 views 23 / 25.
constexpr int kObsSerial = 24;
__global__ __launch_bounds__(256) void k_obs_seen(const float* __restrict__ VS, int n_views, int64_t N, int stride,
                                                  uint16_t* __restrict__ seen) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= N) return;
    const int v0 = 16 * (int)blockIdx.y;
    float x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = v0 + u < n_views ? VS[((int64_t)(v0 + u) * N + g) * stride] : 0.0f;
    uint32_t bits = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) bits |= (uint32_t)(x[u] > 0.0f) << u;
    seen[g * (int64_t)gridDim.y + blockIdx.y] = (uint16_t)bits;  // (the lowest views first)
}

__global__ __launch_bounds__(1024) void k_obs_count(const float* __restrict__ VS, int n_views, int64_t N,
                                                    int stride, int64_t row, float* __restrict__ coeffs,
                                                    uint8_t* __restrict__ status, float* __restrict__ wout,
                                                    float* __restrict__ rho, ObsList obs) {
    __shared__ uint32_t cnt[kObsClasses];
    if (threadIdx.x < (unsigned)kObsClasses) cnt[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    uint32_t n = 0;
    if (g < N) {
        const int words = (n_views + 63) / 64;
        for (int w = 0; w < words; ++w) {
            uint64_t bits = 0;
            if (n_views > kObsSerial) {  // uniform
                bits = obs.seen[g * (int64_t)words + w];
            } else {
                for (int v0 = 0; v0 < n_views; v0 += 8) {
                    float x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = v0 + u < n_views ? VS[((int64_t)(v0 + u) * N + g) * stride] : 0.0f;
#pragma unroll
                    for (int u = 0; u < 8; ++u) bits |= (uint64_t)(x[u] > 0.0f) << (v0 + u);
                }
                obs.seen[g] = bits;
            }
            n += (uint32_t)__popcll(bits);
        }
        uint8_t cls = 255;
        if (n != 0u) {
            cls = (uint8_t)(kObsClasses - 1 - min((int)((uint64_t)n * kObsClasses / (uint64_t)(n_views + 1)), kObsClasses - 1));
            atomicAdd(&cnt[cls], 1u);
        } else {
            if (status) status[g] = GSC_G_UNOBSERVED;
            if (wout) wout[g] = 0.0f;
            if (rho) rho[g] = 0.0f;
        }
        obs.cls[g] = cls;
    }
    // Rows of zeros: short ones by their threads, others by the wave, one after the
    // other (a thread a row stores 4 bytes of 64 lines at a time: 250k rows of 1024
    // floats 2096 -> 747 us with the solve, of 27 76 -> 50; of 12 42 and 40, but 19
    // and 21 of 5k).
    const bool none = g < N && n == 0u;
    if (row < 16) {
        for (int64_t i = 0; none && i < row; ++i) coeffs[g * row + i] = 0.0f;
    } else {
        const int lane = (int)threadIdx.x & 63;
        for (uint64_t m = __builtin_amdgcn_ballot_w64(none); m != 0; m &= m - 1) {
            float* out = coeffs + (g - lane + __builtin_ctzll(m)) * row;
            for (int64_t i = lane; i < row; i += 64) out[i] = 0.0f;
        }
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)kObsClasses) obs.counts[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = cnt[threadIdx.x];
}

// (A class's Gaussians of one block come in any order: each is solved by itself.)
__global__ __launch_bounds__(1024) void k_obs_scatter(int64_t N, ObsList obs) {
    __shared__ uint32_t at[kObsClasses];
    if (threadIdx.x < (unsigned)kObsClasses) at[threadIdx.x] = obs.counts[(size_t)threadIdx.x * gridDim.x + blockIdx.x];
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const uint8_t cls = g < N ? obs.cls[g] : 255;
    if (cls != 255) obs.list[atomicAdd(&at[cls], 1u)] = (uint32_t)g;
}

namespace {
inline uint64_t obs_blocks(int64_t N) { return (uint64_t)((N + 1023) / 1024); }
}

// Layout: seen words (8-byte aligned first), list, class counts, scan scratch,
// total, class bytes.
int64_t fold_obs_words(int64_t N, int n_views) {
    const uint64_t nc = kObsClasses * obs_blocks(N);
    return 2 * N * (int64_t)((n_views + 63) / 64) + N + (int64_t)nc + (int64_t)scan_scratch_words(nc) + 2 + (N + 3) / 4;
}

// Lists the observed Gaussians of per-view sums VS; coeffs (rows of `row`
// floats), status, wout and rho (each optional but the first) get the
// unobserved ones' values.
static ObsList launch_obs_list(const float* VS, int n_views, int64_t N, int stride, int64_t row, float* coeffs,
                               uint8_t* status, float* wout, float* rho, uint32_t* scratch, hipStream_t s) {
    const int64_t words = (n_views + 63) / 64;
    const uint32_t nblk = (uint32_t)obs_blocks(N);
    ObsList o;
    o.seen = reinterpret_cast<uint64_t*>(scratch);
    o.list = scratch + 2 * N * words;
    o.counts = o.list + N;
    uint32_t* scr = o.counts + (size_t)kObsClasses * nblk;
    uint32_t* total = scr + scan_scratch_words((uint64_t)kObsClasses * nblk);
    o.n_list = total;
    o.cls = reinterpret_cast<uint8_t*>(total + 2);
    if (n_views > kObsSerial)
        hipLaunchKernelGGL(k_obs_seen, dim3((unsigned)((N + 255) / 256), (unsigned)(4 * words)), dim3(256), 0, s, VS,
                           n_views, N, stride, reinterpret_cast<uint16_t*>(o.seen));
    hipLaunchKernelGGL(k_obs_count, dim3(nblk), dim3(1024), 0, s, VS, n_views, N, stride, row, coeffs, status, wout,
                       rho, o);
    launch_scan(o.counts, o.counts, kObsClasses * nblk, total, scr, s);
    hipLaunchKernelGGL(k_obs_scatter, dim3(nblk), dim3(1024), 0, s, N, o);
    return o;
}

void launch_fold_solve(const ViewInfo* views, int n_views, const float* means, const float* VS,
                       bool per_view, int64_t N, int C, int sh_deg, const double* lam_nb,
                       float kappa_max, float* coeffs, uint8_t* status, float* wout,
                       float* dc_scratch, unsigned int* ill_count, hipStream_t s, double* factor,
                       uint32_t* obs_scratch, bool split) {
    if (N <= 0) return;
    if (sh_deg == 0) {
        const float* src = VS;
        if (per_view) {
            int64_t n = N * (int64_t)(C + 1);
            hipLaunchKernelGGL(k_sum_views, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, VS,
                               n_views, N, C + 1, dc_scratch);
            src = dc_scratch;
        }
        hipLaunchKernelGGL(k_solve_dc, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s,
                           sum_rows(const_cast<float*>(src), C, split ? N : 0), N, C,
                           lam_nb[0], coeffs, status, wout);
        return;
    }
    LamNB lam;
    for (int i = 0; i < kMaxNb; ++i) lam.v[i] = 0.0;
    int nb = (sh_deg + 1) * (sh_deg + 1);
    for (int i = 0; i < nb; ++i) lam.v[i] = lam_nb[i];
    // one wave (16 Gaussians) per block: at one wave per SIMD a block then
    // starts on any free SIMD, not only when four are free on one CU
    dim3 grid((unsigned)((N + 15) / 16)), block(64);
    const float* nf = nullptr;
    float* nw = nullptr;
    const ObsList obs = launch_obs_list(VS, n_views, N, C + 1, (int64_t)nb * C, coeffs, status, wout, nullptr,
                                        obs_scratch, s);
#define GSC_FOLD(LL)                                                                                        \
    hipLaunchKernelGGL((k_fold_solve<LL, false>), grid, block, 0, s, views, n_views, means, VS, C + 1, N, C, lam, \
                       kappa_max, nf, nf, coeffs, nw, status, wout, ill_count, factor, obs)
    switch (sh_deg) {
        case 1: GSC_FOLD(1); break;
        case 2: GSC_FOLD(2); break;
        default: GSC_FOLD(3); break;
    }
#undef GSC_FOLD
}

// ---- refinement (Algorithm 1, steps 8-10) --------------------------------
//
// One thread per Gaussian: fold the residual's per-view sums into
// B = sum_j phi_gj S_gj^T in FP64 (four channels at a time, the SH values of
// each view evaluated as in the fold above), form B - w_g Lambda c_g and solve
// with the factor stored by the first pass (forward substitution L y = rhs,
// back substitution L^T x = y, 1/L_ii kept on the diagonal), then c_g += x.
template <int L>
__global__ __launch_bounds__(256) void k_refine_update(const ViewInfo* __restrict__ views, int n_views,
                                                       const float* __restrict__ means,
                                                       const float* __restrict__ VS, int64_t N, int C,
                                                       LamNB lam, const double* __restrict__ factor,
                                                       const uint8_t* __restrict__ status,
                                                       float* __restrict__ coeffs) {
    constexpr int NB = (L + 1) * (L + 1);
    constexpr int NT = NB * (NB + 1) / 2;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= N) return;
    if (status[g] & (GSC_G_UNOBSERVED | GSC_G_FAILED)) return;
    const double* F = factor + g * (int64_t)(NT + 1);
    const double wg = F[NT];
    const float mx = means[3 * g], my = means[3 * g + 1], mz = means[3 * g + 2];
    const int stride = C + 1;
    const int64_t vstep = N * (int64_t)stride;
    float* out = coeffs + g * NB * C;
    for (int c0 = 0; c0 < C; c0 += 4) {
        double b[NB][4];
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
            for (int c = 0; c < 4; ++c) b[m][c] = 0.0;
        for (int v = 0; v < n_views; ++v) {
            const float* p = VS + (int64_t)v * vstep + g * stride;
            if (p[0] == 0.0f) continue;  // no contribution in this view
            double dir[3];
            view_direction(mx, my, mz, views[v].centre, dir);
            double ph[NB];
            sh_eval<double, L>(dir[0], dir[1], dir[2], ph);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double sc = c0 + c < C ? (double)p[1 + c0 + c] : 0.0;
#pragma unroll
                for (int m = 0; m < NB; ++m) b[m][c] = fma(ph[m], sc, b[m][c]);
            }
        }
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < C) b[m][c] = fma(-wg * lam.v[m], (double)out[m * C + c0 + c], b[m][c]);
        // L y = rhs
#pragma unroll
        for (int i = 0; i < NB; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double t = b[i][c];
#pragma unroll
                for (int j = 0; j < i; ++j) t = fma(-F[i * (i + 1) / 2 + j], b[j][c], t);
                b[i][c] = t * F[i * (i + 1) / 2 + i];
            }
        }
        // L^T x = y
#pragma unroll
        for (int i = NB - 1; i >= 0; --i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double t = b[i][c];
#pragma unroll
                for (int k = i + 1; k < NB; ++k) t = fma(-F[k * (k + 1) / 2 + i], b[k][c], t);
                b[i][c] = t * F[i * (i + 1) / 2 + i];
            }
        }
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < C) out[m * C + c0 + c] = (float)((double)out[m * C + c0 + c] + b[m][c]);
    }
}

// L = 0: the matrix is w_g (Y0^2 + lambda_0) and B = Y0 S_g (VS summed over views).
__global__ void k_refine_update_dc(const float* __restrict__ VS, int64_t N, int C, double lam0,
                                   const float* __restrict__ w, const uint8_t* __restrict__ status,
                                   float* __restrict__ coeffs) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= N) return;
    if (status[g] & (GSC_G_UNOBSERVED | GSC_G_FAILED)) return;
    const double wg = w[g];
    const float* sg = VS + g * (int64_t)(C + 1);
    const double den = wg * (kY0 * kY0 + lam0);
    for (int c = 0; c < C; ++c) {
        const double cg = coeffs[g * C + c];
        coeffs[g * C + c] = (float)(cg + (kY0 * (double)sg[1 + c] - wg * lam0 * cg) / den);
    }
}

void launch_refine_update(const ViewInfo* views, int n_views, const float* means, const float* VS,
                          int64_t N, int C, int sh_deg, const double* lam_nb, const double* factor,
                          const float* w, const uint8_t* status, float* coeffs, hipStream_t s) {
    if (N <= 0) return;
    const dim3 grid((unsigned)((N + 255) / 256)), block(256);
    if (sh_deg == 0) {
        hipLaunchKernelGGL(k_refine_update_dc, grid, block, 0, s, VS, N, C, lam_nb[0], w, status, coeffs);
        return;
    }
    LamNB lam;
    for (int i = 0; i < kMaxNb; ++i) lam.v[i] = 0.0;
    const int nb = (sh_deg + 1) * (sh_deg + 1);
    for (int i = 0; i < nb; ++i) lam.v[i] = lam_nb[i];
    switch (sh_deg) {
        case 1: hipLaunchKernelGGL((k_refine_update<1>), grid, block, 0, s, views, n_views, means, VS, N, C, lam, factor, status, coeffs); break;
        case 2: hipLaunchKernelGGL((k_refine_update<2>), grid, block, 0, s, views, n_views, means, VS, N, C, lam, factor, status, coeffs); break;
        default: hipLaunchKernelGGL((k_refine_update<3>), grid, block, 0, s, views, n_views, means, VS, N, C, lam, factor, status, coeffs); break;
    }
}

// L = 0 adjoint: A_g + w_g Lambda = w_g (Y0^2 + lambda_0).
__global__ void k_adjoint_dc(const float* __restrict__ W, int64_t N, int C, double lam0,
                             const float* __restrict__ gc, const float* __restrict__ cin,
                             float* __restrict__ bbar, float* __restrict__ rho) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= N) return;
    const double w = W[g];
    double r = 0.0;
    for (int c = 0; c < C; ++c) {
        const double b = w == 0.0 ? 0.0 : (double)gc[g * C + c] / (w * (kY0 * kY0 + lam0));
        bbar[g * C + c] = (float)b;
        r += lam0 * b * (double)cin[g * C + c];
    }
    rho[g] = (float)r;
}

void launch_adjoint_solve(const ViewInfo* views, int n_views, const float* means, const float* V,
                          bool per_view, int64_t N, int C, int sh_deg, const double* lam_nb,
                          const float* grad_coeffs, const float* coeffs, float* bbar, float* rho,
                          float* w_scratch, uint32_t* obs_scratch, hipStream_t s) {
    if (N <= 0) return;
    if (sh_deg == 0) {
        const float* src = V;
        if (per_view) {
            hipLaunchKernelGGL(k_sum_views, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, V,
                               n_views, N, 1, w_scratch);
            src = w_scratch;
        }
        hipLaunchKernelGGL(k_adjoint_dc, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, src, N,
                           C, lam_nb[0], grad_coeffs, coeffs, bbar, rho);
        return;
    }
    LamNB lam;
    for (int i = 0; i < kMaxNb; ++i) lam.v[i] = 0.0;
    int nb = (sh_deg + 1) * (sh_deg + 1);
    for (int i = 0; i < nb; ++i) lam.v[i] = lam_nb[i];
    dim3 grid((unsigned)((N + 15) / 16)), block(64);
    uint8_t* ns = nullptr;
    float* nw = nullptr;
    unsigned int* ni = nullptr;
    double* nd = nullptr;
    const ObsList obs = launch_obs_list(V, n_views, N, 1, (int64_t)nb * C, bbar, nullptr, nullptr, rho, obs_scratch, s);
#define GSC_ADJ(LL)                                                                                        \
    hipLaunchKernelGGL((k_fold_solve<LL, true>), grid, block, 0, s, views, n_views, means, V, 1, N, C, lam, 0.0f, \
                       grad_coeffs, coeffs, bbar, rho, ns, nw, ni, nd, obs)
    switch (sh_deg) {
        case 1: GSC_ADJ(1); break;
        case 2: GSC_ADJ(2); break;
        default: GSC_ADJ(3); break;
    }
#undef GSC_ADJ
}

}  // namespace gsc
