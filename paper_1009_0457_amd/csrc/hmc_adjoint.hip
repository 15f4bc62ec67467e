// hmc_adjoint.hip -- reverse-mode derivative of the global explicit elastic solve (Sec. 5)
// with respect to the per-grain Euler angles and the applied stress.
//
// Forward (as hmc_stress_refresh with a cold start): E_0 = mean(S_q) Sigma, u_0 = w_0 = 0,
// then n explicit steps; U = 1/2 sum_v eps_v . C_v eps_v at the final state.  With the state
// of step t written (u_t, w_t, E_t, wE_t), the adjoint runs the recurrence backwards:
//
//   w~ = w^_{t+1} + u^_{t+1},  a = alpha w~          (nodal)
//   wE~ = wE^_{t+1} + E^_{t+1}, b = alphaE wE~       (6)
//   eta_v = B_v a + b / K^3,  tau_v = C_v eta_v      (per voxel: the adjoint stress)
//   u^_t = u^_{t+1} - sum_v B_v^T tau_v,   w^_t = beta w~
//   E^_t = E^_{t+1} - sum_v tau_v,         wE^_t = beta wE~
//   dU/dtheta_g += -sum_{v in g} eta_v . (dC_g/dtheta) eps_{t,v},   dU/dSigma += b
//
// from u^_n = sum_v B_v^T sigma_v, E^_n = sum_v sigma_v, w^_n = wE^_n = 0 and the direct
// term dU/dtheta_g += sum_{v in g} 1/2 eps_v . (dC_g/dtheta) eps_v; after step 0 the start
// E_0 = mean(S_q) Sigma adds E^_0 . (n_g/K^3) (dS_g/dtheta) Sigma and mean(S) E^_0.
//
// The stiffness-derivative terms are contracted as they arise and summed per voxel in FP64, as torques
// about the lab axes: turning a crystal by dw turns its projectors, dP_a = [W, P_a], so that with
// S(e) = (C11 - C12 - 2 C44) sum_a (P_a : e) P_a the change of eta.C eps is
//     tr(W (X - X^T)),   X = S(eps) eta + S(eta) eps,
// which needs no derivative table: G_v = 1/2 g(eps_n, eps_n) - sum_t g(eta_t, eps_t) with g the vector of
// those changes per unit turn about x, y and z.  An Euler angle turns the crystal about its own axis
// (z; the line of nodes; the crystal's z), along which G is taken at the end.  Per-grain sums use
// 64-bit fixed-point atomics (order-independent, so the result is deterministic).  Forward states are recovered from checkpoints every `ckpt_every` steps
// by recomputing one segment at a time.  The adjoint step is tiled like the forward step.
#include <cmath>
#include <cstring>
#include <vector>

#include "hmc_device.h"

namespace hmc {

constexpr double kFixScale = 1099511627776.0;   // 2^40
// Doubles per copy of the part of the adjoint state the adjoint steps advance (the slots
// kEb .. kWEt below), kept per step like the forward sequence's (E, wE); the tau sums between
// steps use the forward's fixed-point accumulators.
constexpr int kAdjSeq = 32;

struct AdjLayout {
    size_t ckpt, seg_u[2], seg_E[2], ub0, ub1, wb0, wb1, G, axes, low, dS, adj, asums, aseq, grad, total;
    int n_ck;          // checkpoints of segment starts
    size_t ck_bytes;   // bytes per checkpoint: u, w planes then 12 doubles
};

static size_t al256(size_t x) { return (x + 255) / 256 * 256; }

static AdjLayout adj_layout(const hmc_ctx_s* c, int n_steps, int k)
{
    AdjLayout L{};
    const size_t n3 = (size_t)c->reps[0].n3;
    const size_t Q = (size_t)c->reps[0].Q;
    L.n_ck = (n_steps + k - 1) / k + 1;          // + the final state
    L.ck_bytes = al256(6 * n3 * sizeof(float)) + 256;
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t at = o;
        o = al256(o + b);
        return at;
    };
    L.ckpt = take((size_t)L.n_ck * L.ck_bytes);
    // two segment buffers: one segment's adjoint steps read one while the next segment is
    // recomputed into the other
    for (int b = 0; b < 2; ++b) {
        L.seg_u[b] = take((size_t)(k + 1) * 3 * n3 * sizeof(float));
        L.seg_E[b] = take((size_t)(k + 1) * 8 * sizeof(double));
    }
    L.ub0 = take(3 * n3 * sizeof(float));
    L.ub1 = take(3 * n3 * sizeof(float));
    L.wb0 = take(3 * n3 * sizeof(float));
    L.wb1 = take(3 * n3 * sizeof(float));
    L.G = take(3 * n3 * sizeof(double));
    L.axes = take(Q * 9 * sizeof(double));
    L.low = take(Q * kProj * sizeof(float));
    L.dS = take(Q * 3 * kTab * sizeof(float));
    L.adj = take(64 * sizeof(double));
    L.asums = take(3 * kSumSlots * sizeof(unsigned long long));
    L.aseq = take(2 * kAdjSeq * sizeof(double));
    L.grad = take(Q * 3 * sizeof(unsigned long long));
    L.total = o;
    return L;
}

// Slots of the adjoint's small state block.
enum AdjSlot { kEb = 0, kWEb = 6, kB = 12, kSigb = 18, kWEt = 24, kE0 = 30, kAdjDoubles = 64 };

// Component I of the adjoint state after one more adjoint step whose tau sums are in `sums`
// (null: unchanged): E^ -= sum tau, wE^ = beta wE~, Sigma^ += b, wE~ = wE^ + E^, b = alphaE wE~.
__device__ __forceinline__ void adj_advance(const double* in, const unsigned long long* sums, int I, double betaE,
                                            double alphaE, double out[5])
{
    double Eb = in[kEb + I], wEb = in[kWEb + I], b = in[kB + I], Sb = in[kSigb + I], wt = in[kWEt + I];
    if (sums) {
        long long tot = 0;
#pragma unroll
        for (int c = 0; c < kSumCopies; ++c) tot += (long long)sums[c * 8 + I];
        Eb -= (double)tot / kSumScale;
        wEb = betaE * wt;
        Sb += b;
        wt = wEb + Eb;
        b = alphaE * wt;
    }
    out[0] = Eb;
    out[1] = wEb;
    out[2] = b;
    out[3] = Sb;
    out[4] = wt;
}

__device__ __forceinline__ void adj_store(double* dst, int I, const double v[5])
{
    dst[kEb + I] = v[0];
    dst[kWEb + I] = v[1];
    dst[kB + I] = v[2];
    dst[kSigb + I] = v[3];
    dst[kWEt + I] = v[4];
}

// The part of a cubic stress that turns with the crystal (a multiple of 1 commutes with every strain):
// q1 c1 + q2 c2 of cubic_stress, in units of C44 and FP64, with `l` what the rounding of the rows c left: turned,
// that rounding moves a torque by 5.4e-8 of its norm over random orientations (three tables of rounded
// derivatives: 2.5e-8).
template <class F>
__device__ __forceinline__ void turning_stress(const float c[kProjUsed], const float l[kProjUsed], float sgn,
                                               const F e[6], double s[6])
{
    double d[kProjUsed];
#pragma unroll
    for (int i = 0; i < kProjUsed; ++i) d[i] = (double)c[i] + (double)l[i];
    double p1 = d[0] * e[0], p2 = d[6] * e[0];
#pragma unroll
    for (int I = 1; I < 6; ++I) {
        p1 = fma(d[I], (double)e[I], p1);
        p2 = fma(d[6 + I], (double)e[I], p2);
    }
    const double q1 = sgn * fma(2.0, p1, p2), q2 = sgn * fma(2.0, p2, p1);
#pragma unroll
    for (int I = 0; I < 6; ++I) s[I] = fma(q2, d[6 + I], q1 * d[I]);
}

// m += (the vector of) S H - H S for a stress S and a strain H (engineering shears): the entries
// (y, z), (z, x) and (x, y).
template <class F>
__device__ __forceinline__ void add_commutator(const double S[6], const F e[6], double m[3])
{
    const double S0 = S[0], S1 = S[1], S2 = S[2], S3 = S[3], S4 = S[4], S5 = S[5];
    const double H0 = e[0], H1 = e[1], H2 = e[2], H3 = 0.5 * (double)e[3], H4 = 0.5 * (double)e[4],
                 H5 = 0.5 * (double)e[5];
    m[0] += S5 * H4 - S4 * H5 + (S1 - S2) * H3 + S3 * (H2 - H1);
    m[1] += S3 * H5 - S5 * H3 + (S2 - S0) * H4 + S4 * (H0 - H2);
    m[2] += S4 * H3 - S3 * H4 + (S0 - S1) * H5 + S5 * (H1 - H0);
}

// g = the changes of eta.C eps / C44 per unit turn of the crystal about x, y and z.
template <class F>
__device__ __forceinline__ void turning_work(const float c[kProjUsed], const float l[kProjUsed], float sgn,
                                             const F eta[6], const F eps[6], double g[3])
{
    double s[6];
    double m[3] = {0.0, 0.0, 0.0};
    turning_stress(c, l, sgn, eps, s);
    add_commutator(s, eta, m);
    turning_stress(c, l, sgn, eta, s);
    add_commutator(s, eps, m);
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = 2.0 * m[k];
}

struct AdjInitArgs {
    const int16_t* spins;
    CubicTab C;
    double lam;              // C.lam in full
    const float* low;        // Q x kProj: what the rounding of C's rows left
    const float* u;
    float* ub;
    float* wb;
    double* G;
    double* partials;
    const double* state;
    int K;
    int64_t n3;
};

// Final-state adjoint: u^_n = sum_v B_v^T sigma_v, G_v = 1/2 g(eps, eps) (in units of C44), partial sums of sigma.
// With the steps' rows (another rounding of the stiffness would leave forces that the final state does not have), and
// strain and stress in double, as the energy is formed: it is that energy's derivative at the state there is, whose
// error is then of second order in the state's.  The macroscopic strain, rounded, would be off alike in every voxel.
// Over 14 inputs, with E^ in double at the end too (k_adj_grad), the load derivative's error went from 5.2e-8 to 4.0e-8
// at 64^3 and from 5.3e-8 to 4.6e-8 at 40^3 (rms); the Euler derivatives' and the energy's stayed.
__global__ __launch_bounds__(256) void k_adj_init(AdjInitArgs a)
{
    const int K = a.K;
    const float zero[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < a.n3; n += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(n % K), y = (int)((n / K) % K), z = (int)(n / ((int64_t)K * K));
        double f[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int ca = c & 1, cb = (c >> 1) & 1, cc = c >> 2;
            const int vx = wrapk(x - ca, K), vy = wrapk(y - cb, K), vz = wrapk(z - cc, K);
            float row[kProjUsed], d[6];
            double e[6], s[6];
            voxel_strain(a.u, a.n3, K, vx, vy, vz, zero, d);
            const int g = a.spins[vx + (int64_t)K * (vy + (int64_t)K * vz)];
            cubic_row(a.C.P, g, row);
#pragma unroll
            for (int I = 0; I < 6; ++I) e[I] = a.state[kE + I] + (double)d[I];
            cubic_stress(row, a.lam, 0.0, (double)a.C.sgn, 1.0, e, s);
            const double sx = ca ? 0.25 : -0.25, sy = cb ? 0.25 : -0.25, sz = cc ? 0.25 : -0.25;
            f[0] += sx * s[0] + sy * s[5] + sz * s[4];
            f[1] += sx * s[5] + sy * s[1] + sz * s[3];
            f[2] += sx * s[4] + sy * s[3] + sz * s[2];
            if (c == 0) {
#pragma unroll
                for (int I = 0; I < 6; ++I) acc[I] += a.C.C44 * s[I];
                float low[kProjUsed];
                double gq[3];
                cubic_row(a.low, g, low);
                turning_work(row, low, a.C.sgn, e, e, gq);
#pragma unroll
                for (int q = 0; q < 3; ++q) a.G[(int64_t)q * a.n3 + n] = 0.5 * gq[q];
            }
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            a.ub[(int64_t)j * a.n3 + n] = (float)(a.C.C44 * f[j]);
            a.wb[(int64_t)j * a.n3 + n] = 0.f;
        }
    }
    block_sum_to<6>(a.partials, acc);
}

struct AdjStepArgs {
    const int16_t* spins;
    CubicTab C;
    const float* low;        // Q x kProj: what the rounding of C's rows left
    const float* ub_in;
    float* ub_out;
    const float* wb_in;      // read at neighbour nodes: ping-pong like ub
    float* wb_out;
    const float* u_t;        // forward displacement of step t
    const double* E_t;       // forward macroscopic strain of step t (6)
    const double* st_in;     // adjoint state the previous step started from (or the initial one)
    double* st_out;          // this step's (written by block 0)
    const unsigned long long* sums_in;   // the previous step's tau sums (null: first step)
    unsigned long long* sums_out;        // this step's
    unsigned long long* sums_clear;      // the next step's, cleared by block 0
    double* G;               // 3 planes
    int K, tile_z;
    float alpha, beta;
    double betaE, alphaE;
    int order;               // logical block order (hmc_set_block_order)
};

// G of the entries at `at` in its three planes, for subtract_from_G: only read where that stores.
template <bool ATOMIC>
__device__ __forceinline__ void read_G(const double* G, int64_t n3, int64_t at, double Gv[3])
{
    if (!ATOMIC)
#pragma unroll
        for (int k = 0; k < 3; ++k) Gv[k] = G[k * n3 + at];
}

// G -= g.  Only this voxel's thread adds to an entry, so the order of the sum is the steps' either way.  ATOMIC: an
// atomic nobody waits for (a backward step at 16^3 9.1 against 10.1 us, at 64^3 22.1 against 22.8), which the hardware
// may drop on fine-grained, managed or host memory: there G is read with the other fields and stored.
template <bool ATOMIC>
__device__ __forceinline__ void subtract_from_G(double* G, int64_t n3, int64_t at, const double Gv[3], const double g[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (ATOMIC)
            unsafeAtomicAdd(&G[k * n3 + at], -g[k]);
        else
            G[k * n3 + at] = Gv[k] - g[k];
    }
}

// tau = C eta / C44 and, where `owned`, the turning work, for a wavefront's voxels: of one grain with its rows
// from scalar loads, of several with each lane gathering its own.
__device__ __forceinline__ void adjoint_voxel(const CubicTab& T, const float* low, int q, bool owned,
                                              const float eta[6], const float eps[6], float tau[6], double g[3])
{
    const int q0 = __builtin_amdgcn_readfirstlane(q);
    float c[kProjUsed], l[kProjUsed];
    if (__builtin_amdgcn_ballot_w64(q != q0) == 0) {
        uniform_cubic_row(T.P, q0, c);
        cubic_stress(c, T, eta, tau);
        if (owned) {
            uniform_cubic_row(low, q0, l);
            turning_work(c, l, T.sgn, eta, eps, g);
        }
    } else {
        cubic_row(T.P, q, c);
        cubic_stress(c, T, eta, tau);
        if (owned) {
            cubic_row(low, q, l);
            turning_work(c, l, T.sgn, eta, eps, g);
        }
    }
}

// One adjoint step, tiled as the forward step (32 x 8 x tile_z nodes per block, layer-pair
// sums of the nodal fields and of the voxel stresses in LDS, previous layer in registers):
// the nodal field a = alpha (w^ + u^) and the forward displacement u_t give each voxel its
// adjoint strain eta and forward strain eps; tau = C eta is formed once per tile, and the
// voxels the block owns also add their torques to G (subtract_from_G) and tau to the block's sums.  Bound by VALU and
// LDS work (64^3: 38 % of the issue slots, 84 B of fields a node, from L2), so the torque counts:
// against three FP64 contractions with tables of 21 derivatives a grain it takes a backward step, forward
// recompute included, from 27.4 to 23.0 us at 64^3, 52.7 to 50.8 at 80^3 and 78.6 to 57.1 at 96^3.  Two wavefronts a SIMD (185
// registers) rather than three with spills: 22.8 against 23.9 us.
template <bool ATOMIC>
__global__ __launch_bounds__(256, 2) void k_adj_step(AdjStepArgs a)
{
    constexpr int NX = kTileX + 2, NY = kTileY + 2, VX = kTileX + 1, VY = kTileY + 1;
    constexpr int NP = (NX * NY + 255) / 256, VP = (kStepVox + 255) / 256;
    __shared__ float4 sAa[NY][NX], sUa[NY][NX];
    __shared__ float2 sAb[NY][NX], sUb[NY][NX];
    __shared__ float4 sPa[VY][VX], sPb[VY][VX];

    const int K = a.K;
    const int64_t n3 = (int64_t)K * K * K;
    const int ntx = (K + kTileX - 1) / kTileX, nty = (K + kTileY - 1) / kTileY, tz = a.tile_z;
    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);
    int b = lb;
    const int bx = b % ntx;
    b /= ntx;
    const int by = b % nty, bz = b / nty;
    const int x0 = bx * kTileX, y0 = by * kTileY, z0 = bz * tz;
    const int z1 = (z0 + tz < K) ? z0 + tz : K;
    // this step's adjoint state from the previous one and its tau sums (read after the
    // prologue's first barrier); block 0 records it and clears the sums of the step after
    __shared__ double sb[6];
    if (threadIdx.x < 6) {
        double v[5];
        adj_advance(a.st_in, a.sums_in, threadIdx.x, a.betaE, a.alphaE, v);
        sb[threadIdx.x] = v[2];
        if (lb == 0) adj_store(a.st_out, threadIdx.x, v);
    }
    if (lb == 0 && threadIdx.x < kSumSlots) a.sums_clear[threadIdx.x] = 0ull;
    float b3[6], E[6];
    const double inv_n3 = 1.0 / (double)n3;
#pragma unroll
    for (int I = 0; I < 6; ++I) E[I] = (float)a.E_t[I];
    const float alpha = a.alpha, beta = a.beta;
    const int t = threadIdx.x, lx = t % kTileX, ly = t / kTileX;
    const int nx = x0 + lx, ny = y0 + ly;
    const bool own = nx < K && ny < K;
    double acc[6] = {0, 0, 0, 0, 0, 0};

    int node_xy[NP], vox_xy[VP];
    bool vox_own[VP];   // only interior positions (k = 0) can be owned
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int i = t + 256 * k, ix = i % NX, iy = i / NX;
        node_xy[k] = wrap_tile(x0 - 1 + ix, K) + K * wrap_tile(y0 - 1 + iy, K);
    }
#pragma unroll
    for (int k = 0; k < VP; ++k) {
        int ix, iy;
        step_voxel_pos(t + 256 * k, ix, iy);
        vox_xy[k] = wrap_tile(x0 - 1 + ix, K) + K * wrap_tile(y0 - 1 + iy, K);
        vox_own[k] = t + 256 * k < kStepVox && ix >= 1 && iy >= 1 && x0 - 1 + ix < K && y0 - 1 + iy < K;
    }
    // the fetched node layer (w^, u^ for a, and u_t) at the thread's positions; the previous
    // layer's a and u_t stay in registers for the pair sums
    float fw[NP][3], fb[NP][3], fu[NP][3], prevA[NP][3], prevU[NP][3];
    int sp[VP];
    auto fetch_nodes = [&](int z) {
        const int64_t zoff = (int64_t)K * K * wrap_tile(z, K);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            if (t + 256 * k < NX * NY) {
                const int64_t n = node_xy[k] + zoff;
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    fw[k][j] = a.wb_in[j * n3 + n];
                    fb[k][j] = a.ub_in[j * n3 + n];
                    fu[k][j] = a.u_t[j * n3 + n];
                }
            }
        }
    };
    auto fetch_spins = [&](int z) {
        const int64_t zoff = (int64_t)K * K * wrap_tile(z, K);
#pragma unroll
        for (int k = 0; k < VP; ++k) {
            sp[k] = 0;
            if (t + 256 * k < kStepVox) sp[k] = a.spins[vox_xy[k] + zoff];
        }
    };
    // the fetched layer is z+1, prev* hold layer z: write the pair's entries
    auto store_pair = [&]() {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int i = t + 256 * k;
            if (i < NX * NY) {
                const int ix = i % NX, iy = i / NX;
                float an[3];
#pragma unroll
                for (int j = 0; j < 3; ++j) an[j] = alpha * (fw[k][j] + fb[k][j]);
                pair_node_entry(an, prevA[k], sAa[iy][ix], sAb[iy][ix]);
                pair_node_entry(fu[k], prevU[k], sUa[iy][ix], sUb[iy][ix]);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    prevA[k][j] = an[j];
                    prevU[k][j] = fu[k][j];
                }
            }
        }
    };
    auto take_prev = [&]() {
#pragma unroll
        for (int k = 0; k < NP; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                prevA[k][j] = alpha * (fw[k][j] + fb[k][j]);
                prevU[k][j] = fu[k][j];
            }
    };
    // adjoint stress of voxel position k (and, if owned, its angle contractions)
    auto voxel_adj = [&](int k, int q, bool owned, float tau[6], double gq[3]) {
        int ix, iy;
        step_voxel_pos(t + 256 * k, ix, iy);
        float eta[6], eps[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        pair_strain<NX>(sAa, sAb, ix, iy, b3, eta);
        if (owned) pair_strain<NX>(sUa, sUb, ix, iy, E, eps);
        adjoint_voxel(a.C, a.low, q, owned, eta, eps, tau, gq);
    };

    // prologue: node layers z0-1, z0 -> voxel layer z0-1 (kept in registers)
    fetch_nodes(z0 - 1);
    take_prev();
    fetch_nodes(z0);
    fetch_spins(z0 - 1);
    store_pair();
    __syncthreads();
#pragma unroll
    for (int I = 0; I < 6; ++I)   // the same in every lane: kept in scalar registers
        b3[I] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int((float)(sb[I] * inv_n3))));
    float tprev[VP][6];
#pragma unroll
    for (int k = 0; k < VP; ++k)
        if (t + 256 * k < kStepVox) {
            double unused[3];
            voxel_adj(k, sp[k], false, tprev[k], unused);
        }
    fetch_spins(z0);
    __syncthreads();

    for (int z = z0; z < z1; ++z) {
        fetch_nodes(z + 1);
        store_pair();                            // pair (z, z+1)
        int sp_cur[VP];
#pragma unroll
        for (int k = 0; k < VP; ++k) {
            sp_cur[k] = sp[k];
            asm volatile("" ::"v"(sp_cur[k]));   // take them before the loads below are issued
        }
        // requested in the order needed: G, the own nodes' w^ and u^, then the next layer's grains
        const int64_t zoff = (int64_t)K * K * z;
        double Gv[3];   // a thread without an owned voxel reads its place all the same
        read_G<ATOMIC>(a.G, n3, vox_xy[0] + zoff, Gv);
        float wn_in[3] = {0.f, 0.f, 0.f}, un_in[3] = {0.f, 0.f, 0.f};
        const int64_t n = nx + (int64_t)K * ny + zoff;
        if (own) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                wn_in[j] = a.wb_in[(int64_t)j * n3 + n];
                un_in[j] = a.ub_in[(int64_t)j * n3 + n];
            }
        }
        if (z + 1 < z1) fetch_spins(z + 1);
        __syncthreads();                         // the node pairs are complete
#pragma unroll
        for (int k = 0; k < VP; ++k) {
            const int i = t + 256 * k;
            if (i >= kStepVox) continue;
            int ix, iy;
            step_voxel_pos(i, ix, iy);
            const bool owned = k == 0 && vox_own[0];   // the halo (k >= 1) is never owned
            float tau[6];
            double gq[3] = {0.0, 0.0, 0.0};
            voxel_adj(k, sp_cur[k], owned, tau, gq);
            pair_voxel_entry(tau, tprev[k], sPa[iy][ix], sPb[iy][ix]);
#pragma unroll
            for (int I = 0; I < 6; ++I) tprev[k][I] = tau[I];
            if (owned) {
#pragma unroll
                for (int I = 0; I < 6; ++I) acc[I] += (double)tau[I];
                subtract_from_G<ATOMIC>(a.G, n3, vox_xy[0] + zoff, Gv, gq);
            }
        }
        __syncthreads();                         // the voxel pair is complete
        if (own) {
            const float quarter = (float)(0.25 * a.C.C44);
            float F[3];
            pair_force<VX>(sPa, sPb, lx, ly, F);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int64_t idx = (int64_t)j * n3 + n;
                a.ub_out[idx] = un_in[j] - quarter * F[j];
                a.wb_out[idx] = beta * (wn_in[j] + un_in[j]);
            }
        }
    }
    const double tot = block_total<6>(acc);
    if (threadIdx.x < 6)
        atomicAdd(a.sums_out + (lb & (kSumCopies - 1)) * 8 + threadIdx.x,
                  (unsigned long long)llrint(tot * (kSumScale * a.C.C44)));
}

// The adjoint step for tiles of depth 1, laid out as k_global_step_flat: every load at once, a thread a
// node column, a voxel column and an own-node column.  It serves the sizes whose blocks of one layer are
// all resident at once, where a step is one chain of loads and barriers: forward recompute and adjoint step
// together 10.8 -> 9.7 us at 16^3 and 11.3 -> 10.0 at 32^3 against k_adj_step.  From depth 2 on the
// halo's projector rows and three fields a layer cost more than the shorter chain saves (64^3: 18.0 us
// against 14.7), and k_adj_step is taken.
template <bool ATOMIC>
__global__ __launch_bounds__(kFlatThreads, 3) void k_adj_flat(AdjStepArgs a)
{
    constexpr int TZ = 1;
    constexpr int NX = kTileX + 2, NY = kTileY + 2, VX = kTileX + 1, VY = kTileY + 1;
    __shared__ float4 sAa[TZ + 1][NY][NX], sUa[TZ + 1][NY][NX];
    __shared__ float2 sAb[TZ + 1][NY][NX], sUb[TZ + 1][NY][NX];
    __shared__ float4 sPa[TZ][VY][VX], sPb[TZ][VY][VX];
    __shared__ double sb[6], red[6][4];

    const int K = a.K, KK = K * K;
    const int64_t n3 = (int64_t)KK * K;
    const int ntx = (K + kTileX - 1) / kTileX, nty = (K + kTileY - 1) / kTileY;
    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);
    int b = lb;
    const int bx = b % ntx;
    b /= ntx;
    const int by = b % nty, bz = b / nty;
    const int x0 = bx * kTileX, y0 = by * kTileY, z0 = bz * TZ;
    const int t = threadIdx.x;

    int vx, vy;
    step_voxel_pos(t, vx, vy);
    const bool vox = t < kStepVox;
    const bool owned = vox && vx >= 1 && vy >= 1 && x0 - 1 + vx < K && y0 - 1 + vy < K;
    const int vox_xy = wrap_tile(x0 - 1 + vx, K) + K * wrap_tile(y0 - 1 + vy, K);
    int sp[TZ + 1];
#pragma unroll
    for (int l = 0; l <= TZ; ++l) sp[l] = a.spins[vox_xy + (int64_t)KK * wrap_once(z0 - 1 + l, K)];
    const int ix = t % NX, iy = t / NX;
    const bool node = t < NX * NY;
    const int node_xy = wrap_tile(x0 - 1 + ix, K) + K * wrap_tile(y0 - 1 + iy, K);
    float wn[TZ + 2][3], bn[TZ + 2][3], un[TZ + 2][3];
#pragma unroll
    for (int l = 0; l < TZ + 2; ++l) {
        const int64_t n = node_xy + (int64_t)KK * wrap_once(z0 - 1 + l, K);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            wn[l][j] = a.wb_in[j * n3 + n];
            bn[l][j] = a.ub_in[j * n3 + n];
            un[l][j] = a.u_t[j * n3 + n];
        }
    }
    const int lx = t % kTileX, ly = t / kTileX;
    const bool own = t < kTileX * kTileY && x0 + lx < K && y0 + ly < K;
    const int64_t own_n = own ? x0 + lx + (int64_t)K * (y0 + ly) + (int64_t)KK * z0 : 0;
    double Et[6], Gv[3];
#pragma unroll
    for (int I = 0; I < 6; ++I) Et[I] = a.E_t[I];
    read_G<ATOMIC>(a.G, n3, vox_xy + (int64_t)KK * z0, Gv);
    float wo[TZ][3], uo[TZ][3];
#pragma unroll
    for (int l = 0; l < TZ; ++l)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            wo[l][j] = a.wb_in[j * n3 + own_n + (int64_t)KK * l];
            uo[l][j] = a.ub_in[j * n3 + own_n + (int64_t)KK * l];
        }
    if (t >= kFlatThreads - 64 && t < kFlatThreads - 64 + 6) {   // the last wavefront has no voxels
        const int I = t - (kFlatThreads - 64);
        double v[5];
        adj_advance(a.st_in, a.sums_in, I, a.betaE, a.alphaE, v);
        sb[I] = v[2];
        if (lb == 0) adj_store(a.st_out, I, v);
    }
    if (lb == 0 && t < kSumSlots) a.sums_clear[t] = 0ull;
    float c[TZ + 1][kProjUsed];
#pragma unroll
    for (int l = 0; l <= TZ; ++l) cubic_row(a.C.P, sp[l], c[l]);
    float low[kProjUsed];
    cubic_row(a.low, sp[1], low);
    if (node) {
#pragma unroll
        for (int l = 0; l < TZ + 2; ++l)
#pragma unroll
            for (int j = 0; j < 3; ++j) wn[l][j] = a.alpha * (wn[l][j] + bn[l][j]);
#pragma unroll
        for (int l = 0; l <= TZ; ++l) {
            pair_node_entry(wn[l + 1], wn[l], sAa[l][iy][ix], sAb[l][iy][ix]);
            pair_node_entry(un[l + 1], un[l], sUa[l][iy][ix], sUb[l][iy][ix]);
        }
    }
    __syncthreads();
    double acc[6] = {0, 0, 0, 0, 0, 0};
    if (vox) {
        const double inv_n3 = 1.0 / (double)n3;
        float b3[6], E[6], tau[2][6];
#pragma unroll
        for (int I = 0; I < 6; ++I) {
            b3[I] = (float)(sb[I] * inv_n3);
            E[I] = (float)Et[I];
        }
#pragma unroll
        for (int l = 0; l <= TZ; ++l) {
            float eta[6], eps[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            double g[3];
            const bool add = owned && l > 0;
            pair_strain<NX>(sAa[l], sAb[l], vx, vy, b3, eta);
            if (add) pair_strain<NX>(sUa[l], sUb[l], vx, vy, E, eps);
            cubic_stress(c[l], a.C, eta, tau[l & 1]);
            if (add) turning_work(c[l], low, a.C.sgn, eta, eps, g);
            if (l > 0) {
                pair_voxel_entry(tau[l & 1], tau[(l & 1) ^ 1], sPa[l - 1][vy][vx], sPb[l - 1][vy][vx]);
                if (add) {
#pragma unroll
                    for (int I = 0; I < 6; ++I) acc[I] += (double)tau[l & 1][I];
                    subtract_from_G<ATOMIC>(a.G, n3, vox_xy + (int64_t)KK * z0, Gv, g);
                }
            }
        }
    }
    if (t < kTileX * kTileY) {   // whole wavefronts; the halo's voxels (the others) are not owned
#pragma unroll
        for (int I = 0; I < 6; ++I) {
            const double v = wave_sum(acc[I]);
            if ((t & 63) == 0) red[I][t >> 6] = v;
        }
    }
    __syncthreads();
    if (t < 6) {
        const double tot = (red[t][0] + red[t][1]) + (red[t][2] + red[t][3]);
        atomicAdd(a.sums_out + (lb & (kSumCopies - 1)) * 8 + t,
                  (unsigned long long)llrint(tot * (kSumScale * a.C.C44)));
    }
    if (own) {
        const float quarter = (float)(0.25 * a.C.C44);
#pragma unroll
        for (int l = 0; l < TZ; ++l) {
            float F[3];
            pair_force<VX>(sPa[l], sPb[l], lx, ly, F);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int64_t idx = j * n3 + own_n + (int64_t)KK * l;
                a.ub_out[idx] = uo[l][j] - quarter * F[j];
                a.wb_out[idx] = a.beta * (wo[l][j] + uo[l][j]);
            }
        }
    }
}

// After the last adjoint step: the adjoint state block.
__global__ void k_adj_seq_fold(double* adj, const double* st_last, const unsigned long long* sums_last, double betaE,
                               double alphaE)
{
    const int I = threadIdx.x;
    if (I >= 6) return;
    double v[5];
    adj_advance(st_last, sums_last, I, betaE, alphaE, v);
    adj_store(adj, I, v);
}

// Starts the adjoint state from the per-block sums of the final stresses (fixed order):
// E^ = sum sigma, wE^ = 0, Sigma^ = 0, then wE~ = wE^ + E^ and b = alphaE wE~ for the first
// adjoint step (later steps advance the state themselves, adj_advance).
__global__ __launch_bounds__(256) void k_adj_E(double* adj, const double* partials, int nblocks, double alphaE)
{
    const int t = threadIdx.x;
    double s[6] = {0, 0, 0, 0, 0, 0};
    for (int bk = t; bk < nblocks; bk += 256)
#pragma unroll
        for (int I = 0; I < 6; ++I) s[I] += partials[(int64_t)bk * 8 + I];
    const double tot = block_total<6>(s);
    if (t < 6) {
        adj[kEb + t] = tot;
        adj[kWEb + t] = 0.0;
        adj[kSigb + t] = 0.0;
        adj[kWEt + t] = tot;
        adj[kB + t] = alphaE * tot;
    }
}

struct AdjGradArgs {
    const int16_t* spins;
    const float* Stab;
    const float* dS;    // Q x 3 x kTab
    const double* G;
    const double* axes; // Q x 3 x 3: the axis each Euler angle turns the grain about, times C44
    const double* adj;  // E^_0 at kEb
    double Sigma[6];
    unsigned long long* grad;   // Q x 3 fixed point
    double* partials;
    int64_t n3;
};

// Per voxel: the stiffness sums G_v along the three angles' axes plus the start-strain term
// (1/K^3) E^_0 . dS Sigma into its grain (fixed-point atomics); partial sums of S E^_0.
__global__ __launch_bounds__(256) void k_adj_grad(AdjGradArgs a)
{
    double Eb[6];
    const double inv_n3 = 1.0 / (double)a.n3;
#pragma unroll
    for (int I = 0; I < 6; ++I) Eb[I] = a.adj[kEb + I];
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < a.n3; v += (int64_t)gridDim.x * blockDim.x) {
        const int g = a.spins[v];
        double G[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) G[k] = a.G[(int64_t)k * a.n3 + v];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const float* ds = a.dS + ((int64_t)g * 3 + q) * kTab;
            const double* ax = a.axes + (int64_t)g * 9 + 3 * q;
            double val = ax[0] * G[0] + ax[1] * G[1] + ax[2] * G[2];
            int k = 0;
#pragma unroll
            for (int I = 0; I < 6; ++I)
#pragma unroll
                for (int J = I; J < 6; ++J) {
                    // start term: E^_0 . (dS Sigma) with the symmetric dS
                    const double sym = (I == J) ? Eb[I] * a.Sigma[I] : Eb[I] * a.Sigma[J] + Eb[J] * a.Sigma[I];
                    val += inv_n3 * (double)ds[k] * sym;
                    ++k;
                }
            const long long fx = llrint(val * kFixScale);
            atomicAdd(&a.grad[(int64_t)g * 3 + q], (unsigned long long)fx);
        }
        double se[6];
        symv21(a.Stab + (int64_t)g * kTab, Eb, se);
#pragma unroll
        for (int I = 0; I < 6; ++I) acc[I] += se[I];
    }
    block_sum_to<6>(a.partials, acc);
}

}  // namespace hmc

using namespace hmc;

namespace {

hmc_status afail(hmc_ctx c, hmc_status s, const char* m)
{
    c->err = m;
    return s;
}

hmc_status adev(hmc_ctx c, hipError_t e, const char* where)
{
    c->err = std::string(where) + ": " + hipGetErrorString(e);
    return HMC_EDEVICE;
}

#define ATRY(expr, where)                              \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return adev(c, e_, where); \
    } while (0)

int adj_blocks(int64_t n3)
{
    int64_t b = (n3 + 255) / 256;
    if (b > kMaxChunkBlocks) b = kMaxChunkBlocks;
    return (int)(b < 1 ? 1 : b);
}

// checkpoint j: u (3 planes), w (3 planes), then E, wE (12 doubles)
hmc_status save_ckpt(hmc_ctx c, char* base, const AdjLayout& L, int j)
{
    const size_t n3 = (size_t)c->reps[0].n3;
    char* ck = base + L.ckpt + (size_t)j * L.ck_bytes;
    ATRY(hipMemcpyAsync(ck, c->d.u[c->cur_u], 3 * n3 * sizeof(float), hipMemcpyDeviceToDevice, c->stream), "ckpt");
    ATRY(hipMemcpyAsync(ck + 3 * n3 * sizeof(float), c->d.w, 3 * n3 * sizeof(float), hipMemcpyDeviceToDevice,
                        c->stream),
         "ckpt");
    ATRY(hipMemcpyAsync(ck + al256(6 * n3 * sizeof(float)), c->d.state + kE, 12 * sizeof(double),
                        hipMemcpyDeviceToDevice, c->stream),
         "ckpt");
    return HMC_OK;
}

// restores checkpoint j with u into `u_dst`, on stream s
hmc_status load_ckpt(hmc_ctx c, char* base, const AdjLayout& L, int j, float* u_dst, hipStream_t s)
{
    const size_t n3 = (size_t)c->reps[0].n3;
    char* ck = base + L.ckpt + (size_t)j * L.ck_bytes;
    ATRY(hipMemcpyAsync(u_dst, ck, 3 * n3 * sizeof(float), hipMemcpyDeviceToDevice, s), "restore");
    ATRY(hipMemcpyAsync(c->d.w, ck + 3 * n3 * sizeof(float), 3 * n3 * sizeof(float), hipMemcpyDeviceToDevice, s),
         "restore");
    ATRY(hipMemcpyAsync(c->d.state + kE, ck + al256(6 * n3 * sizeof(float)), 12 * sizeof(double),
                        hipMemcpyDeviceToDevice, s),
         "restore");
    return HMC_OK;
}

hmc_status check_adj(hmc_ctx c, int n_steps, int k, void* ws, size_t bytes, AdjLayout* L)
{
    if (c->is_batch || c->n_rep != 1) return afail(c, HMC_ESTATE, "the adjoint acts on a single lattice");
    if (c->p.material_points == 8) return afail(c, HMC_ESTATE, "the adjoint covers one material point per voxel");
    if (!c->elastic_buffers) return afail(c, HMC_ESTATE, "elastic term disabled (lambda_el == 0)");
    if (n_steps < 1 || k < 1) return afail(c, HMC_EINVAL, "need n_steps >= 1 and ckpt_every >= 1");
    if (!ws || ((uintptr_t)ws % 256) != 0) return afail(c, HMC_EINVAL, "adjoint workspace must be 256-byte aligned");
    *L = adj_layout(c, n_steps, k);
    if (bytes < L->total) return afail(c, HMC_ESHAPE, "adjoint workspace too small");
    return HMC_OK;
}

}  // namespace

namespace hmc {
}

extern "C" {

size_t hmc_adjoint_workspace_bytes(hmc_ctx c, int32_t n_steps, int32_t ckpt_every)
{
    if (!c || c->n_rep != 1 || n_steps < 1 || ckpt_every < 1) return 0;
    return adj_layout(c, n_steps, ckpt_every).total;
}

hmc_status hmc_elastic_forward(hmc_ctx c, int32_t n_steps, int32_t ckpt_every, void* ws, size_t bytes, double* U)
{
    TraceRange range("hmc adjoint forward");
    if (!c) return HMC_EINVAL;
    c->err.clear();
    AdjLayout L;
    hmc_status st = check_adj(c, n_steps, ckpt_every, ws, bytes, &L);
    if (st != HMC_OK) return st;
    if (!U) return afail(c, HMC_EINVAL, "null output");
    if (!c->have_orient || !c->have_spins || !c->have_load)
        return afail(c, HMC_ESTATE, "forward needs orientations, spins and a load");
    char* base = (char*)ws;
    // cold start exactly as hmc_stress_refresh
    ATRY(launch_fill_f32(c->d.u[0], 0.f, 3 * c->total_sites, c->stream), "forward");
    ATRY(launch_fill_f32(c->d.w, 0.f, 3 * c->total_sites, c->stream), "forward");
    c->cur_u = 0;
    ATRY(launch_reuss(c), "forward");
    for (int t = 0; t < n_steps; t += ckpt_every) {
        st = save_ckpt(c, base, L, t / ckpt_every);
        if (st != HMC_OK) return st;
        ATRY(launch_global_steps(c, (t + ckpt_every < n_steps) ? ckpt_every : n_steps - t), "forward");
    }
    st = save_ckpt(c, base, L, L.n_ck - 1);   // final state
    if (st != HMC_OK) return st;
    ATRY(launch_global_final(c, true), "forward");
    double u = 0;
    ATRY(hipMemcpyAsync(&u, c->d.state + kU, sizeof u, hipMemcpyDeviceToHost, c->stream), "forward");
    ATRY(hipStreamSynchronize(c->stream), "forward");
    c->host_refresh_steps += n_steps;
    c->have_state = c->have_stress = true;
    c->adj_steps = n_steps;
    c->adj_every = ckpt_every;
    *U = u;
    return report_nonfinite(c);
}

hmc_status hmc_elastic_backward(hmc_ctx c, void* ws, size_t bytes, double dU, double* grad_euler,
                                double grad_sigma_MPa[6])
{
    if (!c) return HMC_EINVAL;
    TraceRange range("hmc adjoint backward");
    c->err.clear();
    if (c->adj_steps < 1) return afail(c, HMC_ESTATE, "no forward pass recorded");
    AdjLayout L;
    const int n = c->adj_steps, k = c->adj_every;
    hmc_status st = check_adj(c, n, k, ws, bytes, &L);
    if (st != HMC_OK) return st;
    if (!grad_euler || !grad_sigma_MPa) return afail(c, HMC_EINVAL, "null output");
    const RepDev& R = c->reps[0];
    const int64_t n3 = R.n3;
    const int Q = R.Q;
    char* base = (char*)ws;
    float* seg_u[2] = {(float*)(base + L.seg_u[0]), (float*)(base + L.seg_u[1])};
    double* seg_E[2] = {(double*)(base + L.seg_E[0]), (double*)(base + L.seg_E[1])};
    float* ub[2] = {(float*)(base + L.ub0), (float*)(base + L.ub1)};
    float* wb[2] = {(float*)(base + L.wb0), (float*)(base + L.wb1)};
    double* G = (double*)(base + L.G);
    double* axes = (double*)(base + L.axes);
    float* low = (float*)(base + L.low);
    float* dS = (float*)(base + L.dS);
    double* adj = (double*)(base + L.adj);
    unsigned long long* asums = (unsigned long long*)(base + L.asums);
    double* aseq = (double*)(base + L.aseq);
    unsigned long long* grad = (unsigned long long*)(base + L.grad);
    const int nb = adj_blocks(n3);

    // per-grain derivative tables
    {
        std::vector<float> hS((size_t)Q * 3 * kTab, 0.f), hl((size_t)Q * kProj, 0.f);
        std::vector<double> ax((size_t)Q * 9);
        for (int g = 0; g < Q; ++g) {
            const double* e = &c->euler[3 * (size_t)g];
            double dSd[3][36];
            grain_table_derivatives(e, c->p.C11, c->p.C12, c->p.C44, nullptr, dSd);
            for (int q = 0; q < 3; ++q)
                for (int i = 0; i < 6; ++i)
                    for (int j = i; j < 6; ++j)
                        hS[((size_t)g * 3 + q) * kTab + sym_index(i, j)] = (float)dSd[q][6 * i + j];
            // phi1 turns about z, Phi about the line of nodes Rz(phi1) x, phi2 about the crystal's z
            const double n[9] = {0.0, 0.0, 1.0, std::cos(e[0]), std::sin(e[0]), 0.0,
                                 std::sin(e[0]) * std::sin(e[1]), -std::cos(e[0]) * std::sin(e[1]), std::cos(e[1])};
            for (int k = 0; k < 9; ++k) ax[(size_t)g * 9 + k] = c->p.C44 * n[k];
            double A[3][3], proj[kProjUsed];
            bunge(e, A);
            axis_projectors(A, c->p.C11, c->p.C12, c->p.C44, proj);
            for (int k = 0; k < kProjUsed; ++k) hl[(size_t)g * kProj + k] = (float)(proj[k] - (double)(float)proj[k]);
        }
        ATRY(hipMemcpyAsync(low, hl.data(), hl.size() * sizeof(float), hipMemcpyHostToDevice, c->stream), "backward");
        ATRY(hipMemcpyAsync(axes, ax.data(), ax.size() * sizeof(double), hipMemcpyHostToDevice, c->stream), "backward");
        ATRY(hipMemcpyAsync(dS, hS.data(), hS.size() * sizeof(float), hipMemcpyHostToDevice, c->stream), "backward");
        ATRY(hipMemsetAsync(grad, 0, (size_t)Q * 3 * sizeof(unsigned long long), c->stream), "backward");
        ATRY(hipStreamSynchronize(c->stream), "backward");
    }

    // final state -> initial adjoint
    st = load_ckpt(c, base, L, L.n_ck - 1, c->d.u[0], c->stream);
    if (st != HMC_OK) return st;
    c->cur_u = 0;
    {
        AdjInitArgs a{c->d.spins, cubic_tab(c), cubic_lam(c), low, c->d.u[0], ub[0], wb[0], G, c->d.partials, c->d.state, R.K, n3};
        hipLaunchKernelGGL(k_adj_init, dim3(nb), dim3(256), 0, c->stream, a);
        hipLaunchKernelGGL(k_adj_E, dim3(1), dim3(256), 0, c->stream, adj, c->d.partials, nb, R.glob_alphaE);
        ATRY(hipGetLastError(), "backward: start");
    }
    int cur_b = 0, i_adj = 0;   // i_adj: adjoint steps taken
    // the first adjoint step adds into tau-sum buffer 0 (2 uint32 per 64-bit word)
    ATRY(launch_fill_u32((uint32_t*)asums, 0u, 2 * kSumSlots, c->stream), "backward: start");
    const int n_seg = (n + k - 1) / k;
    // tiles as deep as the forward step's (72^3, depth 4: 33.1 us a step with the recompute, 36.5 at 2)
    const int adj_depth = R.tile_z;
    // G's kind of memory, asked anew on each call: floating-point atomics on coarse-grained memory of this device alone
    hipPointerAttribute_t attr{};
    const bool plain_memory = hipPointerGetAttributes(&attr, G) == hipSuccess && attr.type == hipMemoryTypeDevice &&
                              !attr.isManaged && attr.allocationFlags == hipDeviceMallocDefault &&
                              attr.device == c->device;
    if (!plain_memory) (void)hipGetLastError();   // a refused query is no failure of the call
    // Segment j's forward states are recomputed from its checkpoint into buffer j & 1.  With
    // the auxiliary stream the recomputation of segment j-1 runs while the context's stream
    // takes segment j's adjoint steps (both are latency-bound at this size); events order
    // them: ev[0..1] "buffer b free", ev[2..3] "buffer b recomputed", ev[4] start.  With
    // profiling on, everything stays on the context's stream.
    const bool overlap = !c->profiling;
    hipStream_t rs = c->stream;
    if (overlap) {
        if (!c->aux_stream) {
            ATRY(hipStreamCreateWithFlags(&c->aux_stream, hipStreamNonBlocking), "backward: stream");
            for (auto& e : c->aux_ev) ATRY(hipEventCreateWithFlags(&e, hipEventDisableTiming), "backward: events");
        }
        rs = c->aux_stream;
        // the recomputation overwrites the context's w and (E, wE), which the start above read
        ATRY(hipEventRecord(c->aux_ev[4], c->stream), "backward: events");
        ATRY(hipStreamWaitEvent(rs, c->aux_ev[4], 0), "backward: events");
        ATRY(hipEventRecord(c->aux_ev[0], c->stream), "backward: events");
        ATRY(hipEventRecord(c->aux_ev[1], c->stream), "backward: events");
    }
    auto recompute = [&](int j) -> hmc_status {
        const int b = j & 1;
        const int t0 = j * k, t1 = (t0 + k < n) ? t0 + k : n;
        if (overlap) ATRY(hipStreamWaitEvent(rs, c->aux_ev[b], 0), "backward: events");
        hmc_status s2 = load_ckpt(c, base, L, j, seg_u[b], rs);
        if (s2 != HMC_OK) return s2;
        if (t1 - 1 > t0) {
            ATRY(seq_begin(c, rs), "backward: recompute");
            for (int t = t0; t + 1 < t1; ++t) {
                float* ut = seg_u[b] + (size_t)(t - t0) * 3 * n3;
                ATRY(seq_step(c, rs, t - t0, ut, ut + 3 * n3, seg_E[b] + (size_t)(t - t0) * 8),
                     "backward: recompute");   // records E_t
            }
            ATRY(seq_end(c, rs, t1 - 1 - t0), "backward: recompute");
        }
        ATRY(hipMemcpyAsync(seg_E[b] + (size_t)(t1 - 1 - t0) * 8, c->d.state + kE, 6 * sizeof(double),
                            hipMemcpyDeviceToDevice, rs),
             "backward: recompute");
        if (overlap) ATRY(hipEventRecord(c->aux_ev[2 + b], rs), "backward: events");
        return HMC_OK;
    };
    st = recompute(n_seg - 1);
    if (st != HMC_OK) return st;
    for (int j = n_seg - 1; j >= 0; --j) {
        const int b = j & 1;
        const int t0 = j * k, t1 = (t0 + k < n) ? t0 + k : n;
        if (j > 0) {
            st = recompute(j - 1);
            if (st != HMC_OK) return st;
        }
        if (overlap) ATRY(hipStreamWaitEvent(c->stream, c->aux_ev[2 + b], 0), "backward: events");
        // adjoint steps t1-1 .. t0
        for (int t = t1 - 1; t >= t0; --t) {
            AdjStepArgs a;
            a.spins = c->d.spins;
            a.C = cubic_tab(c);
            a.low = low;
            a.ub_in = ub[cur_b];
            a.ub_out = ub[1 - cur_b];
            a.wb_in = wb[cur_b];
            a.wb_out = wb[1 - cur_b];
            a.u_t = seg_u[b] + (size_t)(t - t0) * 3 * n3;
            a.E_t = seg_E[b] + (size_t)(t - t0) * 8;
            a.st_in = i_adj > 0 ? aseq + ((i_adj - 1) & 1) * kAdjSeq : adj;
            a.st_out = aseq + (i_adj & 1) * kAdjSeq;
            a.sums_in = i_adj > 0 ? asums + ((i_adj - 1) % 3) * kSumSlots : nullptr;
            a.sums_out = asums + (i_adj % 3) * kSumSlots;
            a.sums_clear = asums + ((i_adj + 1) % 3) * kSumSlots;
            a.G = G;
            a.K = R.K;
            a.tile_z = adj_depth;
            a.alpha = R.glob_alpha;
            a.beta = R.glob_beta;
            a.betaE = (double)R.glob_beta;
            a.alphaE = R.glob_alphaE;
            a.order = c->block_order;
            const int tok = prof_begin(c, kProfRefreshStep);
            // the adjoint step keeps 32 x 8 tiles whatever the forward step's rows
            const dim3 grid(tile_blocks_of(R.K, adj_depth, kTileY));
            if (adj_depth == 1 && plain_memory)
                hipLaunchKernelGGL(k_adj_flat<true>, grid, dim3(kFlatThreads), 0, c->stream, a);
            else if (adj_depth == 1)
                hipLaunchKernelGGL(k_adj_flat<false>, grid, dim3(kFlatThreads), 0, c->stream, a);
            else if (plain_memory)
                hipLaunchKernelGGL(k_adj_step<true>, grid, dim3(256), 0, c->stream, a);
            else
                hipLaunchKernelGGL(k_adj_step<false>, grid, dim3(256), 0, c->stream, a);
            prof_end(c, tok);
            ATRY(hipGetLastError(), "backward: step");
            cur_b = 1 - cur_b;
            ++i_adj;
        }
        if (overlap) ATRY(hipEventRecord(c->aux_ev[b], c->stream), "backward: events");
    }
    hipLaunchKernelGGL(k_adj_seq_fold, dim3(1), dim3(64), 0, c->stream, adj, aseq + ((i_adj - 1) & 1) * kAdjSeq,
                       asums + ((i_adj - 1) % 3) * kSumSlots, (double)R.glob_beta, R.glob_alphaE);
    ATRY(hipGetLastError(), "backward: step");
    // contractions and the start-strain terms
    {
        AdjGradArgs a;
        a.spins = c->d.spins;
        a.Stab = c->d.Stab;
        a.dS = dS;
        a.G = G;
        a.axes = axes;
        a.adj = adj;
        for (int I = 0; I < 6; ++I) a.Sigma[I] = R.Sigma[I];
        a.grad = grad;
        a.partials = c->d.partials;
        a.n3 = n3;
        hipLaunchKernelGGL(k_adj_grad, dim3(nb), dim3(256), 0, c->stream, a);
        ATRY(hipGetLastError(), "backward: gradient");
    }
    std::vector<unsigned long long> g((size_t)Q * 3);
    std::vector<double> parts((size_t)nb * 8);
    double ad[kAdjDoubles];
    ATRY(hipMemcpyAsync(g.data(), grad, g.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost, c->stream),
         "backward");
    ATRY(hipMemcpyAsync(parts.data(), c->d.partials, parts.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream),
         "backward");
    ATRY(hipMemcpyAsync(ad, adj, sizeof ad, hipMemcpyDeviceToHost, c->stream), "backward");
    ATRY(hipStreamSynchronize(c->stream), "backward");
    for (size_t i = 0; i < g.size(); ++i) grad_euler[i] = dU * (double)(long long)g[i] / kFixScale;
    for (int I = 0; I < 6; ++I) {
        double s = 0.0;   // mean(S) E^_0, folded in block order
        for (int b = 0; b < nb; ++b) s += parts[(size_t)b * 8 + I];
        // dU/dSigma in GPa^-1 * GPa*voxel; per MPa: x 1e-3
        grad_sigma_MPa[I] = dU * (ad[kSigb + I] + s / (double)n3) * 1e-3;
    }
    // leave the context at the final forward state
    st = load_ckpt(c, base, L, L.n_ck - 1, c->d.u[0], c->stream);
    if (st != HMC_OK) return st;
    c->cur_u = 0;
    ATRY(launch_global_final(c, true), "backward: restore");
    ATRY(hipStreamSynchronize(c->stream), "backward: restore");
    return HMC_OK;
}

}  // extern "C"
