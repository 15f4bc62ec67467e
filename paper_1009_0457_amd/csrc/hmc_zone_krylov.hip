// hmc_zone_krylov.hip -- the zone solve (hmc_zone_kernels.h) by conjugate gradients, for the long
// relaxations of the 5^3 and 7^3 zones (h = 2 and 3).
//
// The n_r heavy-ball steps from rest apply a fixed polynomial of the zone's operator
// A = sum_v B_v^T C_v B_v to b = B_p^T t, and the trial needs one number of the result,
// Phi = -b.u + 1/2 u.A u.  Conjugate gradients from b reach the minimum of that form in far fewer
// applications of A (about 110 against n_r = 200 at h = 2, 170 against 400 at h = 3, for nickel), and
// their coefficients are the tridiagonal T of A in the Krylov basis, on which the n_r heavy-ball steps
// cost next to nothing.  So
//     Phi = Phi(x) + (Phi_T(n_r heavy-ball steps) - min Phi_T),
// the first term evaluated at the gradients' x as the other kernels do at their last displacement
// (its error is of second order in x's), the second, what n_r steps leave of the minimum (some 1e-7
// of the site's stored energy for the default n_r), from T: its heavy-ball steps in FP32 over a trial's lanes, the
// form of their result in double.
//
// A trial stops at the first even step where the residual |b - A x| has been below kKrylovTol |b| for
// two steps.  Measured in double precision for n_r = 20 .. 400 and h = 1, 2, 3 on random polycrystals,
// Phi is then within 20 kKrylovTol^2 |Phi| of the heavy-ball value, some 2e-8 of the site's stored
// energy (nickel; up to 1e-6 of max(|dPi|, W_p / 10) for shears five times as stiff one way as the other); the FP32
// tables leave 6e-8 of it either way.  The stop is each trial's own, so a trial's
// result does not depend on which trial shares its wavefront.  It also stops where its T is full.  The rule
// for taking this kernel (pays, below) leaves no trial far from its end there: for constants at the rule's edge
// trials in random, layered, checkered and uniform surroundings took at most 126 of the 128 steps at h = 2, and
// ones an eighth beyond the edge, cut off 6 steps early, were off by 6e-8 of max(|dPi|, W_p / 10) for n_r = 1000
// (double precision; an energy's error is of second order in the residual left).
//
// What bounds it is FP32 vector work, as in k_zone_lane, at 1.17 times the instructions a step.
// Measured per colour launch: 128^3 under load (h = 2, n_r = 200) 4.02 against 5.40 ms for
// heavy-ball steps, 50^3 (h = 3, n_r = 400) 1.21 against 2.65 ms.
//
// The layout is k_zone_lane's, with a trial's lanes at the start of a group of 32 (h = 2) or 64 (h = 3)
// so that the dot products are sums over whole DPP rows.  Lanes past a trial's own have zero
// stiffness and vectors that stay zero; they share the trial's LDS block, where they only ever write
// the zeros already there.  The stiffness of a voxel is held as the projectors P1, P2 on two of its
// crystal axes (12 registers in place of 21, for the vectors' sake).
#include <algorithm>
#include <cmath>

#include "hmc_device.h"
#include "hmc_zone_kernels.h"

namespace hmc {

namespace {

constexpr float kKrylovTol = 1e-4f;

template <int H>
struct KrylovShape {
    static constexpr int N = 2 * H + 1, NN = N + 1;
    static constexpr int LT = NN * N;                   // lanes per trial
    static constexpr int SL = LT <= 32 ? 32 : 64;       // lanes between trials
    static constexpr int TW = 64 / SL;                  // trials per wavefront
    static constexpr int ROW = NN * NN;                 // floats per (component, layer) row
    static constexpr int BODY = 3 * NN * ROW;
    // block stride: >= BODY + NN (zero gap), and = SL (mod 64) for conflict-free addressing
    static constexpr int TB = BODY + NN + ((SL - (BODY + NN) % 64) % 64 + 64) % 64;
    static constexpr int PAD = 8;                       // leading zeros of the force array
    static constexpr int P = H == 2 ? 4 : 3;            // entries of T per lane in the projected steps
    static constexpr int CAP = SL * P;                  // most Krylov steps
};

template <int CTRL>
__device__ __forceinline__ float dpp_all(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Sum over each group of SL = 32 or 64 lanes, in every lane (the same bits in all of them):
// butterflies within the DPP rows of 16, then exchanges of rows.
template <int SL>
__device__ __forceinline__ float group_sum(float v)
{
    v += dpp_all<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v += dpp_all<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += dpp_all<0x141>(v);   // row_half_mirror
    v += dpp_all<0x140>(v);   // row_mirror
    const auto a = __builtin_amdgcn_permlane16_swap((unsigned)__float_as_int(v), (unsigned)__float_as_int(v), false, false);
    v = __int_as_float((int)a[0]) + __int_as_float((int)a[1]);
    if (SL == 64) {
        const auto c =
            __builtin_amdgcn_permlane32_swap((unsigned)__float_as_int(v), (unsigned)__float_as_int(v), false, false);
        v = __int_as_float((int)c[0]) + __int_as_float((int)c[1]);
    }
    return v;
}

// Corner forces of one node layer, as node_forces: the own node's and the +y node's.
__device__ __forceinline__ void corner_forces(float L0, float L1, float L2, float& own, float& ny)
{
    const float Ab = (L2 - L0) + from_prev_lane(L2 + L0);
    const float Db = L1 + from_prev_lane(L1);
    own = Ab - Db;
    ny = Ab + Db;
}

struct KrylovArgs {
    ZoneArgs z;
    const float* Ptab;      // per-grain projectors (kProj)
    float lam, lam_lo, sgn;  // CubicTab's constants
    float inv_scale;        // C44 / 16: the kernel's operator is 16 / C44 times A
};

template <int H>
__global__ __launch_bounds__(64, 2) void k_zone_krylov(KrylovArgs ka)
{
    const ZoneArgs& a = ka.z;
    using S = KrylovShape<H>;
    constexpr int N = S::N, NN = S::NN, LT = S::LT, SL = S::SL, TW = S::TW, ROW = S::ROW, TB = S::TB, P = S::P;
    static_assert(3 * NN <= LT && TB % 64 == SL % 64 && TB >= S::BODY + NN && SL <= ROW, "layout");

    __shared__ float s_u[TW * TB];                                // the search direction
    __shared__ float s_n[S::PAD + TW * TB];                       // forces sent to the +y neighbour
    __shared__ float s_ctr[TW][18];                               // eps_p[6], t[6], t / |b| [6]
    __shared__ double s_nb2[TW];                                  // |b|^2
    __shared__ float2 s_T[TW][S::CAP];                            // (step length, residual^2) of each step

    const int li = threadIdx.x;
    const int zs = li / SL, l = li % SL;
    const bool member = l < LT;
    const int x = l % NN, y = l / NN;
    const bool vox = member && x < N;
    const bool centre_col = vox && x == H && y == H;
    const uint32_t count = *a.count;
    const float on_vox = vox ? 1.f : 0.f, lam = vox ? ka.lam : 0.f, lam_lo = vox ? ka.lam_lo : 0.f;

    float* const ub = s_u + zs * TB;                              // this lane's trial block
    float* const nbk = s_n + S::PAD + zs * TB;
    // top-row item: node column (l % NN, N), component l / NN, for the first 3 NN lanes
    const bool xon = l < 3 * NN;
    const int xcol = l % NN + NN * N, xj = xon ? l / NN : 0;
    const int m_cap = (a.nr < S::CAP ? a.nr : S::CAP) & ~1;

    // Gradients of the field v (own nodes) + the +y nodes in LDS at the lane's voxel column, layer by
    // layer (without the factor 1/4): calls f(k, strain of voxel k) in order.
    auto strains = [&](const float (&v)[NN][3], auto&& f) {
        float cn[3], cnn[3], Lp[3][3];
#pragma unroll
        for (int j = 0; j < 3; ++j) cn[j] = ub[(j * NN + 0) * ROW + l + NN];
#pragma unroll
        for (int z = 0; z < NN; ++z) {
            if (z + 1 < NN) {
#pragma unroll
                for (int j = 0; j < 3; ++j) cnn[j] = ub[(j * NN + z + 1) * ROW + l + NN];
            }
            float Lc[3][3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const float A = v[z][j] + cn[j], D = cn[j] - v[z][j];
                Lc[0][j] = from_next_lane(A) - A;
                Lc[1][j] = D + from_next_lane(D);
                Lc[2][j] = A + from_next_lane(A);
            }
            if (z >= 1) {
                float g[3][3];
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    g[j][0] = Lp[0][j] + Lc[0][j];
                    g[j][1] = Lp[1][j] + Lc[1][j];
                    g[j][2] = Lc[2][j] - Lp[2][j];
                }
                const float ev[6] = {g[0][0], g[1][1], g[2][2], g[1][2] + g[2][1], g[0][2] + g[2][0],
                                     g[0][1] + g[1][0]};
                f(z - 1, ev);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                cn[j] = cnn[j];
#pragma unroll
                for (int r = 0; r < 3; ++r) Lp[r][j] = Lc[r][j];
            }
        }
    };

    uint32_t n_solved = 0, n_accepted = 0;
    for (uint32_t base = (uint32_t)stride_block((int)blockIdx.x, (int)gridDim.x, a.order) * (uint32_t)TW; base < count;
         base += gridDim.x * (uint32_t)TW) {
        const uint32_t e = base + (uint32_t)zs;
        const bool active = member && e < count;

        float Cv[N][kProjUsed];
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
            for (int i = 0; i < kProjUsed; ++i) Cv[k][i] = 0.f;
        if (l == 0) {
            s_nb2[zs] = 0.0;
#pragma unroll
            for (int I = 0; I < 18; ++I) s_ctr[zs][I] = 0.f;
        }
        if (active) {
            const TrialEntry ent = a.list[e];
            const RepDev& R = a.reps[ent.qr >> 16];
            const TrialCtx tc = trial_ctx(a, ent.qr);
            const int K = tc.K;
            const int q_new = (int)(ent.qr & 0xffffu);
            const int px = (int)(ent.site % (uint32_t)K);
            const int py = (int)((ent.site / (uint32_t)K) % (uint32_t)K);
            const int pz = (int)(ent.site / ((uint32_t)K * (uint32_t)K));
            if (l == 0) {
                const int q_old = tc.spins[ent.site];
                float c[21], sp[6], s[6], eps[6], tt[6];
#pragma unroll
                for (int I = 0; I < 6; ++I) sp[I] = a.sigma[(int64_t)I * a.plane + tc.site_off + ent.site];
                load_sym(tc.Stab + (int64_t)q_old * kTab, c);
                symv(c, sp, eps);
                load_sym(tc.Ctab + (int64_t)q_new * kTab, c);
                symv(c, eps, tt);
                load_sym(tc.Ctab + (int64_t)q_old * kTab, c);
                symv(c, eps, s);
                // |B_p^T t|^2 = 1/2 sum_ij t_ij^2 (8 corners, each 1/4 of a signed row sum)
                double nb2 = 0.0;
#pragma unroll
                for (int I = 0; I < 6; ++I) {
                    tt[I] -= s[I];
                    nb2 += (I < 3 ? 0.5 : 1.0) * (double)tt[I] * (double)tt[I];
                }
                s_nb2[zs] = nb2;
                const double inv = nb2 > 0.0 ? 1.0 / sqrt(nb2) : 0.0;
#pragma unroll
                for (int I = 0; I < 6; ++I) {
                    s_ctr[zs][I] = eps[I];
                    s_ctr[zs][6 + I] = tt[I];
                    s_ctr[zs][12 + I] = (float)((double)tt[I] * inv);
                }
            }
            if (vox) {
                const float* Ptab = ka.Ptab + R.grain_off * kProj;
                const int gx = ((px + x - H) % K + K) % K, gy = ((py + y - H) % K + K) % K;
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const int gz = ((pz + k - H) % K + K) % K;
                    const int g = (centre_col && k == H) ? q_new : (int)tc.spins[gx + K * (gy + K * gz)];
                    cubic_row(Ptab, g, Cv[k]);
                }
            }
        }
        for (int i = li; i < TW * TB; i += 64) s_u[i] = 0.f;
        for (int i = li; i < S::PAD + TW * TB; i += 64) s_n[i] = 0.f;
        __syncthreads();

        // r = p = b / |b| on the trial site's eight corners (all own nodes of some lane)
        float u[NN][3], r[NN][3], p[NN][3], xu[NN], xr[NN];
        float rr;
        {
            const bool cx = member && (x == H || x == H + 1) && (y == H || y == H + 1);
            const float gx = cx ? (x == H ? -0.25f : 0.25f) : 0.f, gy = cx ? (y == H ? -0.25f : 0.25f) : 0.f;
            const float gz = cx ? 0.25f : 0.f;
            const float* t = &s_ctr[zs][12];
            const float fx = gx * t[0] + gy * t[5], fy = gx * t[5] + gy * t[1], fz = gx * t[4] + gy * t[3];
            float n = 0.f;
#pragma unroll
            for (int z = 0; z < NN; ++z) {
                const float sz = z == H ? -gz : z == H + 1 ? gz : 0.f;
                const bool on = z == H || z == H + 1;
                r[z][0] = on ? fx + sz * t[4] : 0.f;
                r[z][1] = on ? fy + sz * t[3] : 0.f;
                r[z][2] = on ? fz + sz * t[2] : 0.f;
                xu[z] = xr[z] = 0.f;
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    p[z][j] = r[z][j];
                    u[z][j] = 0.f;
                    n += r[z][j] * r[z][j];
                    if (on && member) ub[(j * NN + z) * ROW + l] = r[z][j];
                }
            }
            rr = group_sum<SL>(n);
        }
        const float tol = kKrylovTol * kKrylovTol * rr;
        __syncthreads();

        int m = 0;                                  // this trial's steps, set when it stops
        bool done = !(rr > 0.f) || m_cap == 0;      // b = 0 (or not finite): nothing to solve
        bool small = false;                         // the residual of the last two steps is
        auto step = [&](int k) {
            // ---- q = A p: voxels' strains, stresses, corner forces ----
            float q[NN][3];
            {
                float Pp[3], Qp[3], Rp[3];
                strains(p, [&](int kz, const float (&ev)[6]) {
                    float sv[6];
                    cubic_stress<float>(Cv[kz], lam, lam_lo, ka.sgn, on_vox, ev, sv);
                    const float Pn[3] = {sv[0], sv[5], sv[4]};
                    const float Qn[3] = {sv[5], sv[1], sv[3]};
                    const float Rn[3] = {sv[4], sv[3], sv[2]};
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const float PL = kz == 0 ? Pn[j] : Pp[j] + Pn[j];
                        const float QL = kz == 0 ? Qn[j] : Qp[j] + Qn[j];
                        const float RL = kz == 0 ? -Rn[j] : Rp[j] - Rn[j];
                        corner_forces(PL, QL, RL, q[kz][j], nbk[(j * NN + kz) * ROW + l]);
                        Pp[j] = Pn[j];
                        Qp[j] = Qn[j];
                        Rp[j] = Rn[j];
                    }
                });
                // top node layer: only voxel N-1 below it
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    corner_forces(Pp[j], Qp[j], Rp[j], q[NN - 1][j], nbk[(j * NN + NN - 1) * ROW + l]);
            }
            __syncthreads();
            // ---- step length, new residual, new direction ----
            float d[3] = {0.f, 0.f, 0.f}, n[3] = {0.f, 0.f, 0.f};
            float xq[NN], xp[NN];   // set and used in the item's lanes only
#pragma unroll
            for (int z = 0; z < NN; ++z)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    q[z][j] += nbk[(j * NN + z) * ROW + l - NN];
                    d[j] += q[z][j] * p[z][j];
                }
            if (xon) {
#pragma unroll
                for (int z = 0; z < NN; ++z) {
                    xq[z] = nbk[(xj * NN + z) * ROW + xcol - NN];
                    xp[z] = ub[(xj * NN + z) * ROW + xcol];
                    d[z % 3] += xq[z] * xp[z];
                }
            }
            const float pq = group_sum<SL>((d[0] + d[1]) + d[2]);
            const float gm = pq > 0.f && !done ? rr * __builtin_amdgcn_rcpf(pq) : 0.f;
            // (lanes past the trial's own have read the top row's forces: their r stays zero)
            const float gr = member ? gm : 0.f;
#pragma unroll
            for (int z = 0; z < NN; ++z)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    u[z][j] += gm * p[z][j];
                    r[z][j] -= gr * q[z][j];
                    n[j] += r[z][j] * r[z][j];
                }
            if (xon) {
#pragma unroll
                for (int z = 0; z < NN; ++z) {
                    xu[z] += gm * xp[z];
                    xr[z] -= gm * xq[z];
                    n[z % 3] += xr[z] * xr[z];
                }
            }
            const float rn = group_sum<SL>((n[0] + n[1]) + n[2]);
            const float bt = rr > 0.f ? rn * __builtin_amdgcn_rcpf(rr) : 0.f;
#pragma unroll
            for (int z = 0; z < NN; ++z)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    p[z][j] = r[z][j] + bt * p[z][j];
                    ub[(j * NN + z) * ROW + l] = p[z][j];
                }
            if (xon) {   // after the above: the lanes past the trial's own put zeros into the top row
#pragma unroll
                for (int z = 0; z < NN; ++z) ub[(xj * NN + z) * ROW + xcol] = xr[z] + bt * xp[z];
            }
            if (l == 0) s_T[zs][k] = make_float2(gm, rr);
            __syncthreads();
            small = !(rn > tol) && !(rr > tol);
            rr = rn;
        };
        for (int k = 0; k < m_cap; k += 2) {
            if (__builtin_amdgcn_ballot_w64(!done) == 0ull) break;
            if (H == 2) {
                step(k);
                step(k + 1);
            } else {   // one copy of the step: two of them spill at h = 3
#pragma unroll 1
                for (int i = k; i < k + 2; ++i) step(i);
            }
            if (!done && (small || k + 2 == m_cap)) {
                m = k + 2;   // small, or T full: its rest is below the FP32 tables' error, see above
                done = true;
            }
        }
        // ---- Phi(x) in units of |b|^2 and of the operator's: x published for the +y neighbours ----
#pragma unroll
        for (int z = 0; z < NN; ++z)
#pragma unroll
            for (int j = 0; j < 3; ++j) ub[(j * NN + z) * ROW + l] = u[z][j];
        if (xon) {
#pragma unroll
            for (int z = 0; z < NN; ++z) ub[(xj * NN + z) * ROW + xcol] = xu[z];
        }
        __syncthreads();
        double part;
        {
            double quad = 0.0, lin = 0.0;
            strains(u, [&](int kz, const float (&ev)[6]) {
                float sv[6];
                cubic_stress<float>(Cv[kz], lam, lam_lo, ka.sgn, on_vox, ev, sv);
#pragma unroll
                for (int I = 0; I < 6; ++I) quad += (double)ev[I] * (double)sv[I];
                if (kz == H && centre_col) {
#pragma unroll
                    for (int I = 0; I < 6; ++I) lin += (double)s_ctr[zs][12 + I] * (double)ev[I];
                }
            });
            part = vox ? 0.5 * quad - 0.25 * lin : 0.0;
        }

        // ---- what n_r heavy-ball steps leave of the minimum, on T: entries l P .. l P + P - 1 per
        // lane, in units where b = e_1: omega <- beta omega - rho T eta + e_1, eta <- eta + omega.  With
        // step lengths g_k, squared residuals r_k and s_k^2 = r_{k+1} / r_k,
        // T = sum_k (e_k + s_k e_{k+1}) (e_k + s_k e_{k+1})^T / g_k (no e_{m+1}).  The steps take T in
        // single precision: the form below is of second order in what that does to eta ----
        {
            const float rho = a.alpha * ka.inv_scale, beta = a.beta;
            const float2* T = s_T[zs];
            float D[P], O[P], eta[P], om[P];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const int i = l * P + q;
                const float2 t = T[i < m ? i : 0], lo = T[i > 0 && i < m ? i - 1 : 0], hi = T[i + 1 < m ? i + 1 : 0];
                const float ig = __builtin_amdgcn_rcpf(t.x), it = __builtin_amdgcn_rcpf(t.y);
                const float c = i > 0 ? t.y * __builtin_amdgcn_rcpf(lo.y * lo.x) : 0.f;
                D[q] = i < m ? -rho * (ig + c) : 0.f;
                O[q] = i + 1 < m ? -rho * (__builtin_amdgcn_sqrtf(hi.y * it) * ig) : 0.f;
                eta[q] = om[q] = 0.f;
            }
            const float Om = from_prev_lane(O[P - 1]);      // coupling to the previous lane's last entry
            const float e1 = l == 0 && m > 0 ? 1.f : 0.f;
            auto heavy_ball = [&]() {
                const float lo = from_prev_lane(eta[P - 1]), hi = from_next_lane(eta[0]);
                float t[P];
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    t[q] = q == 0 ? beta * om[q] + e1 : beta * om[q];
                    t[q] += (q == 0 ? Om : O[q - 1]) * (q == 0 ? lo : eta[q - 1]);
                    t[q] += O[q] * (q == P - 1 ? hi : eta[q + 1]);
                    om[q] = t[q] + D[q] * eta[q];
                }
#pragma unroll
                for (int q = 0; q < P; ++q) eta[q] += om[q];
            };
            for (int i = 0; i + 2 <= a.nr; i += 2) {
                heavy_ball();
                heavy_ball();
            }
            if (a.nr & 1) heavy_ball();
            // rho (-eta_1 + 1/2 rho eta.T eta) + 1/2 sum_k g_k r_k / r_1 (minus the minimum)
            const float hi = from_next_lane(eta[0]);
            double quad = 0.0, lin = l == 0 ? (double)eta[0] : 0.0, low = 0.0;
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const int i = l * P + q;
                if (i < m) {
                    const double en = (double)eta[q], ep = i + 1 < m ? (double)(q == P - 1 ? hi : eta[q + 1]) : 0.0;
                    const double f = i + 1 < m ? en + sqrt((double)T[i + 1].y / (double)T[i].y) * ep : en;
                    quad += f * f / (double)T[i].x;
                    low += (double)T[i].x * (double)T[i].y;
                }
            }
            const double rd = (double)rho;
            if (m > 0) part += rd * (0.5 * rd * quad - lin) + 0.5 * low / (double)T[0].y;
        }
#pragma unroll
        for (int o = SL / 2; o > 0; o >>= 1) part += __shfl_xor(part, o);
        if (active && l == 0) {
            const TrialEntry ent = a.list[e];
            const TrialCtx tc = trial_ctx(a, ent.qr);
            double dPi = part * s_nb2[zs] / (double)ka.inv_scale;
#pragma unroll
            for (int I = 0; I < 6; ++I) dPi += 0.5 * (double)s_ctr[zs][I] * (double)s_ctr[zs][6 + I];
            if (!isfinite(dPi)) atomicOr(a.nonfinite, (uint32_t)kNfZone);
            const double dE = tc.J * (double)ent.gb + tc.lambda * dPi;
            const bool accept = (dE <= 0.0) || ((double)ent.r1 < ldexp(exp(-dE / tc.kT), 32));
            a.acc[e] = accept ? 1 : 0;
            if (a.rec) {
                a.rec[tc.site_off + ent.site].dPi = (float)dPi;
                a.rec[tc.site_off + ent.site].flags = 1 | 4 | (accept ? 2 : 0);
            }
            n_solved += 1;
            n_accepted += accept ? 1 : 0;
        }
        __syncthreads();   // LDS is reused by the next group of trials
    }
    for (int off = 32; off > 0; off >>= 1) {
        n_solved += __shfl_xor(n_solved, off);
        n_accepted += __shfl_xor(n_accepted, off);
    }
    if (li == 0 && n_solved) {
        atomicAdd(&a.stats[stat_copy(blockIdx.x) + kStatSolves], (unsigned long long)n_solved);
        if (n_accepted) atomicAdd(&a.stats[stat_copy(blockIdx.x) + kStatAccepted], (unsigned long long)n_accepted);
    }
}

// Whether the relaxation of zone_steps heavy-ball steps is taken by conjugate gradients
// (k_zone_krylov).  With kappa = 4 lambda / mu, lambda the largest eigenvalue of the stiffness and
// mu = min(1/2 (C11 - C12), C44) / (2h+1)^2 the zone's slowest shear, a trial takes up to 3.7 sqrt(kappa)
// steps at h = 2 and 4.2 at h = 3 (random polycrystals of 25 sets of constants, C44 / mu from 0.1 to 10;
// 4 to 5.4 of them for crystals of little contrast, sqrt(kappa) < 25, which fill half of T).  They have
// to fit the kernel's T; and one costs 1.15 heavy-ball steps, a heavy-ball step on T 0.04 of one,
// so that gradients pay from zone_steps = 1.2 of them on, and are taken from 1.25 on.  Measured there, a pass by
// heavy-ball steps over one by gradients: h = 2, 149 steps 1.01 to 1.02 at 48^3 and 64^3, 0.93 at 16^3 to 32^3, whose
// launch lasts as long as its longest trial (1.0 from 160 steps on, 1.2 at 200); h = 3, 232 steps 1.24 at 48^3, 1.02 at
// 32^3, 0.96 below (1.0 from 245 on).
// And T has to resolve what the heavy-ball steps leave: m Krylov steps reproduce polynomials of degree 2m, and
// the steps' residual, of a higher one, only as far as it is smooth (slow modes not reached yet) or damped away,
// by beta^(n_r / 2) where the steps oscillate.  In double precision on random polycrystals the energies were off
// by 0.5 beta^n_r of themselves: by 5e-2 for beta = 0.99 and n_r = 200, by 1.5e-5 for 0.95; at beta^n_r = 1e-7
// (n_r = 149 .. 1000, alpha from a hundredth of the stability bound up to it) by 3e-7, the stop's share.
// Steps that are not stable for every mode are not taken on T either: alpha times the zone's largest eigenvalue at most
// 2 (1 + beta).  That eigenvalue is below 4 times the stiffest longitudinal modulus (0.87 to 0.90 of it in uniform and
// random zones of 11 sets of constants), a bound that leaves room for step lengths set for other constants nearby, as
// where a program changes C alone (4 lambda, half as large again for nickel, would send those back to the steps).
template <int H>
bool pays(const hmc_params& p)
{
    const double lam = std::max(p.C11 + 2 * p.C12, std::max(p.C11 - p.C12, 2 * p.C44));
    const double longitudinal = std::max(p.C11, std::max((p.C11 + p.C12 + 2 * p.C44) / 2,
                                                         (p.C11 + 2 * p.C12 + 4 * p.C44) / 3));   // <100>, <110>, <111>
    const bool stable = std::fabs(p.zone_beta) < 1.0 && p.zone_alpha >= 0.0 &&
                        p.zone_alpha * 4.0 * longitudinal <= 2.0 * (1.0 + p.zone_beta);
    if (!stable || std::pow(std::fabs(p.zone_beta), p.zone_steps) > 1e-7) return false;
    const double mu = std::min(0.5 * (p.C11 - p.C12), p.C44) / ((2 * H + 1) * (2 * H + 1));
    const double m = (H == 2 ? 3.6 : 4.0) * std::sqrt(4.0 * lam / mu);
    return m <= KrylovShape<H>::CAP && p.zone_steps >= 1.25 * m;
}

}  // namespace

bool krylov_pays(const hmc_params& p) { return p.zone_h == 2 ? pays<2>(p) : p.zone_h == 3 && pays<3>(p); }

void launch_zone_krylov(const hmc_params& p, int64_t max_list, const float* Ptab, hipStream_t stream, ZoneArgs za)
{
    KrylovArgs a;
    a.z = za;
    a.Ptab = Ptab;
    const double an = (p.C11 - p.C12 - 2.0 * p.C44) / p.C44, lam = p.C12 / p.C44 + an / 3.0;
    a.lam = (float)lam;
    a.lam_lo = (float)(lam - (double)a.lam);
    a.sgn = an < 0 ? -1.f : 1.f;
    a.inv_scale = (float)(p.C44 / 16.0);
    const int tw = p.zone_h == 2 ? KrylovShape<2>::TW : KrylovShape<3>::TW;
    // many more work-groups than resident slots: the hardware's dispatch balances the tail
    const unsigned g = (unsigned)std::min<int64_t>(std::max<int64_t>((max_list + tw - 1) / tw, 1), 65536);
    if (p.zone_h == 2) hipLaunchKernelGGL(k_zone_krylov<2>, dim3(g), dim3(64), 0, stream, a);
    else hipLaunchKernelGGL(k_zone_krylov<3>, dim3(g), dim3(64), 0, stream, a);
}

}  // namespace hmc
