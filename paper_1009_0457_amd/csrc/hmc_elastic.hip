// hmc_elastic.hip -- global quasi-static elastic state (Sec. 5) and lattice reductions.
//
// The periodic K^3 lattice carries one material point per site at the centre of a voxel
// whose 8 corners are background-grid nodes (K^3 nodes, periodic).  Unknowns: nodal
// displacement fluctuation u (3 planes of K^3) and macroscopic strain E (6); the strain of
// site v is E + B_v u, its stress C_{q_v} times that, and the load is the average stress
// Sigma.  One explicit step (damped dynamics written as a heavy ball, alpha = dt^2/m,
// beta = 1 - c dt):
//     r_n = -sum_{v at n} B_v(n)^T sigma_v,   w <- beta w + alpha r,   u <- u + w
//     r_E = Sigma - mean_v sigma_v,          wE <- beta wE + alphaE r_E,  E <- E + wE
// k_global_step_tiled does the node part for every node (reading u, writing the other u
// buffer, so no node sees a half-updated neighbour) and adds its blocks' stress sums into
// fixed-point accumulators; the next step's blocks first advance E from them, and
// k_seq_fold does so after a sequence's last step.  k_global_final writes the stress field
// the zone solves read.
#include <cmath>

#include "hmc_device.h"

namespace hmc {

struct GlobArgs {
    const int16_t* spins;
    CubicTab C;
    const float* uin;
    float* uout;
    float* w;
    const unsigned long long* sums_in;   // the previous step's stress sums (null: first step)
    unsigned long long* sums_out;        // this step's
    unsigned long long* sums_clear;      // the next step's, cleared here
    const double* st_in;     // (E, wE) the previous step started from, or the context's state
    int st_in_stride;        // doubles per replica in st_in
    double* st_out;          // (E, wE) of this step (kSeqState per replica)
    double* E_record;        // optional: receives the step's E (single lattice)
    const RepDev* reps;
    const int32_t* tile_rep;
    int64_t plane;
    int order;                           // logical block order (hmc_set_block_order)
    int single;                          // one replica, described here: no table to read first
    int K, tile_z;
    float alpha, beta;
};

// What a step's block needs of its replica at once.
struct StepRep {
    int r, K, tile_z, tile_first;
    float alpha, beta;
    int64_t site_off, grain_off;
};

__device__ __forceinline__ StepRep step_rep(const GlobArgs& a, int lb)
{
    if (a.single) return {0, a.K, a.tile_z, 0, a.alpha, a.beta, 0, 0};
    const int r = a.tile_rep[lb];
    const RepDev& R = a.reps[r];
    return {r, R.K, R.tile_z, R.tile_first, R.glob_alpha, R.glob_beta, R.site_off, R.grain_off};
}

// Tiled explicit step.  A block owns a 32 x 8 tile of nodes in x, y and marches through
// tile_z node layers in z, so each voxel stress is formed once per tile (1.3x with the halo
// voxels) instead of once per corner node (8x).  The trilinear element's sums are factored
// along z, where the march shares them between neighbouring layers:
//  * per node of the layer pair (z, z+1) and component: S = u(z+1) + u(z), D = u(z+1) - u(z);
//    a voxel's gradient is then 1/4 of (S10 - S00) + (S11 - S01) in x, (S01 - S00) + (S11 - S10)
//    in y and D00 + D10 + D01 + D11 in z over its four node columns;
//  * per voxel column of the layer pair (z-1, z): the stress sums P = s(z) + s(z-1) and
//    differences M = s(z) - s(z-1) that the three force components need (P of xx, yy, yz,
//    xz, xy; M of zz, yz, xz); a node's force is then 1/4 of a signed sum over its four
//    voxel columns.
// Each thread loads the same (x, y) positions of every layer, so the previous layer's
// displacements and stresses stay in its registers.  The own nodes' displacements pass
// through a three-layer LDS ring, which leaves two barriers per layer.  The interior voxels
// are formed in 8 x 8 patches, one per wavefront, so that a wavefront's voxels mostly share
// one grain and its stiffness comes through the scalar cache.
// (At most 128 VGPRs, so that four blocks share a CU: the LDS would allow five.)
// TY = 8 (256 threads, four blocks per CU), 16 (512 threads, two) or 32 (1024 threads, one):
// taller tiles load fewer halo nodes and voxels per owned node and re-read fewer y-halo rows
// of neighbouring tiles.  All give bit-identical results: wavefronts 4g .. 4g+3 of a tall tile
// hold exactly the voxels and sums of the g-th 8-row tile inside it, and each 8-row group's
// stress sums are totalled and rounded to fixed point on their own, as an 8-row block would.
// The own nodes' u and w are read and written once per step; with NT (lattices too large for
// the Infinity Cache) non-temporal accesses keep them from displacing the halo rows that
// neighbouring tiles read from L2 (512^3 on 16-row tiles: 1.73 -> 1.66 ms).
template <int TY, bool NT>
__global__ __launch_bounds__(32 * TY, TY == 8 ? 4 : TY == 16 ? 2 : 1) void k_global_step_tiled(GlobArgs a)
{
    constexpr int THREADS = kTileX * TY;
    constexpr int NX = kTileX + 2, NY = TY + 2, VX = kTileX + 1, VY = TY + 1;
    constexpr int NVOX = VX * VY;
    constexpr int NP = (NX * NY + THREADS - 1) / THREADS, VP = (NVOX + THREADS - 1) / THREADS;
    // LDS entries are vectors, so that each holds what one lane writes or reads at a time:
    // node pair (S0, D0, S1, D1) and (S2, D2); voxel pair (P_xx, P_yy, P_yz, P_xz) and
    // (P_xy, M_zz, M_yz, M_xz); own node (u0, u1, u2, -)
    __shared__ float4 sNa[NY][NX];
    __shared__ float2 sNb[NY][NX];
    __shared__ float4 sPa[VY][VX], sPb[VY][VX];
    __shared__ float4 sraw[3][TY][kTileX];

    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);   // neighbouring tiles share an L2
    const StepRep R = step_rep(a, lb);
    const int r = R.r, K = R.K;
    const int ntx = (K + kTileX - 1) / kTileX, nty = (K + TY - 1) / TY, tz = R.tile_z;
    int b = lb - R.tile_first;
    const int bx = b % ntx;
    b /= ntx;
    const int by = b % nty, bz = b / nty;
    const int x0 = bx * kTileX, y0 = by * TY, z0 = bz * tz;
    const int z1 = (z0 + tz < K) ? z0 + tz : K;
    const int16_t* spins = a.spins + R.site_off;
    CubicTab C = a.C;
    C.P += R.grain_off * kProj;
    const float* uin = a.uin + R.site_off;
    float* uout = a.uout + R.site_off;
    float* w = a.w + R.site_off;
    const int64_t P = a.plane;
    // this step's E (read after the prologue's first barrier); the replica's first block
    // records it and clears the accumulators of the step after
    __shared__ double sE[6];
    if (threadIdx.x < 6) {
        double E_I, wE_I;
        advance_E(a.reps[r], r, a.st_in, a.st_in_stride, a.sums_in, threadIdx.x, E_I, wE_I);
        sE[threadIdx.x] = E_I;
        if (lb == R.tile_first) {
            a.st_out[(int64_t)r * kSeqState + threadIdx.x] = E_I;
            a.st_out[(int64_t)r * kSeqState + 6 + threadIdx.x] = wE_I;
            if (a.E_record) a.E_record[threadIdx.x] = E_I;
        }
    }
    if (lb == R.tile_first && threadIdx.x < kSumSlots) a.sums_clear[(int64_t)r * kSumSlots + threadIdx.x] = 0ull;
    float E[6];
    const float alpha4 = (float)(0.25 * R.alpha * C.C44), beta = R.beta;
    const int t = threadIdx.x, lx = t % kTileX, ly = t / kTileX;
    const int nx = x0 + lx, ny = y0 + ly;
    const bool own = nx < K && ny < K;
    double acc[6] = {0, 0, 0, 0, 0, 0};

    // tile positions this thread loads (nodes) and forms (voxels), the same in every layer
    int node_xy[NP], vox_xy[VP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int i = t + THREADS * k, ix = i % NX, iy = i / NX;
        node_xy[k] = wrap_tile(x0 - 1 + ix, K) + K * wrap_tile(y0 - 1 + iy, K);
    }
#pragma unroll
    for (int k = 0; k < VP; ++k) {
        int ix, iy;
        step_voxel_pos<TY>(t + THREADS * k, ix, iy);
        vox_xy[k] = wrap_tile(x0 - 1 + ix, K) + K * wrap_tile(y0 - 1 + iy, K);
    }
    // Node layer z+2 and voxel layer z+1's grains are fetched into registers while layer z
    // is computed.
    float pf[NP][3], prev[NP][3];
    int sp[VP];
    auto fetch_nodes = [&](int z) {
        const int64_t zoff = (int64_t)K * K * wrap_tile(z, K);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int i = t + THREADS * k;
            if (i < NX * NY) {
                const int64_t n = node_xy[k] + zoff;
                pf[k][0] = uin[n];
                pf[k][1] = uin[P + n];
                pf[k][2] = uin[2 * P + n];
            }
        }
    };
    auto fetch_spins = [&](int z) {
        const int64_t zoff = (int64_t)K * K * wrap_tile(z, K);
#pragma unroll
        for (int k = 0; k < VP; ++k) {
            const int i = t + THREADS * k;
            sp[k] = 0;
            if (i < NVOX) sp[k] = spins[vox_xy[k] + zoff];
        }
    };
    // pf holds node layer z+1 and prev layer z: write the pair's S and D, and layer z+1's own
    // nodes into ring slot `raw`
    auto store_pair = [&](int raw) {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int i = t + THREADS * k;
            if (i < NX * NY) {
                const int ix = i % NX, iy = i / NX;
                pair_node_entry(pf[k], prev[k], sNa[iy][ix], sNb[iy][ix]);
#pragma unroll
                for (int j = 0; j < 3; ++j) prev[k][j] = pf[k][j];
                if (ix >= 1 && ix <= kTileX && iy >= 1 && iy <= TY)
                    sraw[raw][iy - 1][ix - 1] = make_float4(pf[k][0], pf[k][1], pf[k][2], 0.f);
            }
        }
    };
    // stress (in units of C44) of voxel position k of the layer whose node pair is in sNa / sNb
    // (grains in q)
    auto voxel_stress = [&](int k, int q, float s6[6]) {
        int ix, iy;
        step_voxel_pos<TY>(t + THREADS * k, ix, iy);
        float e[6];
        pair_strain<NX>(sNa, sNb, ix, iy, E, e);
        cubic_grains<NT>(C, q, e, s6);
    };

    // prologue: node layers z0-1, z0 -> voxel layer z0-1 (kept in registers)
    int ring = 0;                                // sraw slot of layer z
    fetch_nodes(z0 - 1);
#pragma unroll
    for (int k = 0; k < NP; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) prev[k][j] = pf[k][j];
    fetch_nodes(z0);
    fetch_spins(z0 - 1);
    store_pair(ring);
    __syncthreads();
#pragma unroll
    for (int I = 0; I < 6; ++I) E[I] = (float)sE[I];
    float sprev[VP][6];
#pragma unroll
    for (int k = 0; k < VP; ++k)
        if (t + THREADS * k < NVOX) voxel_stress(k, sp[k], sprev[k]);
    fetch_nodes(z0 + 1);
    fetch_spins(z0);
    __syncthreads();                             // the prologue's reads of sNa / sNb are done

    for (int z = z0; z < z1; ++z) {
        const int ring_next = ring == 2 ? 0 : ring + 1;
        store_pair(ring_next);                   // pair (z, z+1); own nodes of layer z+1
        // This layer's grains arrived during the last layer: take them now, so that no
        // later wait on them also waits for the loads issued below.  The own nodes' w is
        // needed first (at the end of this layer), so it is requested before the prefetch.
        int sp_cur[VP];
#pragma unroll
        for (int k = 0; k < VP; ++k) {
            sp_cur[k] = sp[k];
            asm volatile("" ::"v"(sp_cur[k]));
        }
        float wz[3] = {0.f, 0.f, 0.f};
        const int64_t n = nx + (int64_t)K * (ny + (int64_t)K * z);
        if (own) {
#pragma unroll
            for (int j = 0; j < 3; ++j) wz[j] = NT ? __builtin_nontemporal_load(&w[(int64_t)j * P + n]) : w[(int64_t)j * P + n];
        }
        if (z + 1 < z1) {
            fetch_nodes(z + 2);                  // in flight during this layer
            fetch_spins(z + 1);
        }
        __syncthreads();                         // the node pair is complete
#pragma unroll
        for (int k = 0; k < VP; ++k) {
            const int i = t + THREADS * k;
            if (i >= NVOX) continue;
            int ix, iy;
            step_voxel_pos<TY>(i, ix, iy);
            float s6[6];
            voxel_stress(k, sp_cur[k], s6);
            pair_voxel_entry(s6, sprev[k], sPa[iy][ix], sPb[iy][ix]);
#pragma unroll
            for (int I = 0; I < 6; ++I) sprev[k][I] = s6[I];
            const int gx = x0 - 1 + ix, gy = y0 - 1 + iy;
            if (ix >= 1 && iy >= 1 && gx < K && gy < K) {
#pragma unroll
                for (int I = 0; I < 6; ++I) acc[I] += (double)s6[I];
            }
        }
        __syncthreads();                         // the voxel pair is complete
        if (own) {
            float F[3];
            pair_force<VX>(sPa, sPb, lx, ly, F);
            const float4 u = sraw[ring][ly][lx];
            const float uz[3] = {u.x, u.y, u.z};
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int64_t idx = (int64_t)j * P + n;
                const float wn = __builtin_fmaf(-alpha4, F[j], beta * wz[j]);
                if (NT) {
                    __builtin_nontemporal_store(wn, &w[idx]);
                    __builtin_nontemporal_store(uz[j] + wn, &uout[idx]);
                } else {
                    w[idx] = wn;
                    uout[idx] = uz[j] + wn;
                }
            }
        }
        ring = ring_next;
    }
    const double tot = block_total_quads<6, TY / 8>(acc);
    const int k = threadIdx.x & 255;             // total k of the half threadIdx.x / 256
    if (k < 6) {
        const unsigned copy = (unsigned)(lb - R.tile_first + (threadIdx.x >> 8)) & (kSumCopies - 1);
        atomicAdd(a.sums_out + (int64_t)r * kSumSlots + copy * 8 + k,
                  (unsigned long long)llrint(tot * (kSumScale * C.C44)));
    }
}

// The step for shallow tiles (depth TZ = 1, 2 or 4: lattices whose blocks hardly fill the chip).  There the
// march above is a chain of memory latencies, a layer's loads after another's; here a block of six
// wavefronts issues every load of its 32 x 8 x TZ nodes at once (a thread a node column, a voxel column
// and an own-node column), so the chain is arguments, fields and spins, the spins' stiffness rows, stores.
// Voxels, sums and their order are those of the tiled step: the same bits.
// Measured per step (kernel trace): 16^3 at depth 1 8.4 us tiled, 5.6 so; 64^3 at depth 2 12.0 and 8.4.
template <int TZ>
__global__ __launch_bounds__(kFlatThreads, 3) void k_global_step_flat(GlobArgs a)
{
    constexpr int NX = kTileX + 2, NY = kTileY + 2, VX = kTileX + 1, VY = kTileY + 1;
    static_assert(NX * NY <= kFlatThreads && kStepVox <= kFlatThreads, "a thread a column");
    __shared__ float4 sNa[TZ + 1][NY][NX];
    __shared__ float2 sNb[TZ + 1][NY][NX];
    __shared__ float4 sPa[TZ][VY][VX], sPb[TZ][VY][VX];
    __shared__ double sE[6], red[6][4];

    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);
    const StepRep R = step_rep(a, lb);
    const int r = R.r, K = R.K;
    const int ntx = (K + kTileX - 1) / kTileX, nty = (K + kTileY - 1) / kTileY;
    int b = lb - R.tile_first;
    const int bx = b % ntx;
    b /= ntx;
    const int by = b % nty, bz = b / nty;
    const int x0 = bx * kTileX, y0 = by * kTileY, z0 = bz * TZ;
    const int16_t* spins = a.spins + R.site_off;
    const float* uin = a.uin + R.site_off;
    float* uout = a.uout + R.site_off;
    float* w = a.w + R.site_off;
    const int64_t P = a.plane;
    const int t = threadIdx.x;
    const int KK = K * K;

    // Every thread loads, from a valid place where it has none of its own, so that the loads follow each
    // other without a branch.  Spins first: the stiffness rows wait for them.
    int vx, vy;
    step_voxel_pos(t, vx, vy);
    const bool vox = t < kStepVox;
    const int vox_xy = wrap_tile(x0 - 1 + vx, K) + K * wrap_tile(y0 - 1 + vy, K);
    int sp[TZ + 1];
#pragma unroll
    for (int l = 0; l <= TZ; ++l) sp[l] = spins[vox_xy + (int64_t)KK * wrap_once(z0 - 1 + l, K)];
    const int ix = t % NX, iy = t / NX;
    const bool node = t < NX * NY;
    const int node_xy = wrap_tile(x0 - 1 + ix, K) + K * wrap_tile(y0 - 1 + iy, K);
    float un[TZ + 2][3];
#pragma unroll
    for (int l = 0; l < TZ + 2; ++l) {
        const int64_t n = node_xy + (int64_t)KK * wrap_once(z0 - 1 + l, K);
#pragma unroll
        for (int j = 0; j < 3; ++j) un[l][j] = uin[j * P + n];
    }
    const int lx = t % kTileX, ly = t / kTileX;
    const bool own = t < kTileX * kTileY && x0 + lx < K && y0 + ly < K;
    const int64_t own_n = own ? x0 + lx + (int64_t)K * (y0 + ly) + (int64_t)KK * z0 : 0;
    float wz[TZ][3], uz[TZ][3];
#pragma unroll
    for (int l = 0; l < TZ; ++l)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int64_t i = j * P + own_n + (TZ <= 2 || z0 + l < K ? (int64_t)KK * l : 0);
            wz[l][j] = w[i];
            uz[l][j] = uin[i];
        }
    if (t >= kFlatThreads - 64 && t < kFlatThreads - 64 + 6) {   // the last wavefront has no voxels
        const int I = t - (kFlatThreads - 64);
        double E_I, wE_I;
        advance_E(a.reps[r], r, a.st_in, a.st_in_stride, a.sums_in, I, E_I, wE_I);
        sE[I] = E_I;
        if (lb == R.tile_first) {
            a.st_out[(int64_t)r * kSeqState + I] = E_I;
            a.st_out[(int64_t)r * kSeqState + 6 + I] = wE_I;
            if (a.E_record) a.E_record[I] = E_I;
        }
    }
    if (lb == R.tile_first && t < kSumSlots) a.sums_clear[(int64_t)r * kSumSlots + t] = 0ull;
    const float* rows = a.C.P + R.grain_off * kProj;
    float c[TZ + 1][kProjUsed];
#pragma unroll
    for (int l = 0; l <= TZ; ++l) cubic_row(rows, sp[l], c[l]);
    if (node) {
#pragma unroll
        for (int l = 0; l <= TZ; ++l) pair_node_entry(un[l + 1], un[l], sNa[l][iy][ix], sNb[l][iy][ix]);
    }
    __syncthreads();
    double acc[6] = {0, 0, 0, 0, 0, 0};
    if (vox) {
        float E[6], s[2][6];
#pragma unroll
        for (int I = 0; I < 6; ++I) E[I] = (float)sE[I];
#pragma unroll
        for (int l = 0; l <= TZ; ++l) {
            float e[6];
            pair_strain<NX>(sNa[l], sNb[l], vx, vy, E, e);
            cubic_stress(c[l], a.C, e, s[l & 1]);
            if (l > 0) {
                pair_voxel_entry(s[l & 1], s[(l & 1) ^ 1], sPa[l - 1][vy][vx], sPb[l - 1][vy][vx]);
                if (vx >= 1 && vy >= 1 && x0 - 1 + vx < K && y0 - 1 + vy < K && (TZ <= 2 || z0 + l - 1 < K)) {
#pragma unroll
                    for (int I = 0; I < 6; ++I) acc[I] += (double)s[l & 1][I];
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
        const unsigned copy = (unsigned)(lb - R.tile_first) & (kSumCopies - 1);
        atomicAdd(a.sums_out + (int64_t)r * kSumSlots + copy * 8 + t,
                  (unsigned long long)llrint(tot * (kSumScale * a.C.C44)));
    }
    if (own) {
        const float alpha4 = (float)(0.25 * R.alpha * a.C.C44), beta = R.beta;
#pragma unroll
        for (int l = 0; l < TZ; ++l) {
            if (TZ > 2 && z0 + l >= K) break;   // the last tile of an edge that TZ does not divide
            float F[3];
            pair_force<VX>(sPa[l], sPb[l], lx, ly, F);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int64_t idx = j * P + own_n + (int64_t)KK * l;
                const float wn = __builtin_fmaf(-alpha4, F[j], beta * wz[l][j]);
                w[idx] = wn;
                uout[idx] = uz[l][j] + wn;
            }
        }
    }
}

// After a sequence's last step: the context's (E, wE), one block per replica.
__global__ void k_seq_fold(double* state, const double* st_last, const unsigned long long* sums_last,
                           const RepDev* reps)
{
    const int r = blockIdx.x, I = threadIdx.x;
    if (I >= 6) return;
    double E_I, wE_I;
    advance_E(reps[r], r, st_last, kSeqState, sums_last, I, E_I, wE_I);
    state[(int64_t)r * kStateDoubles + kE + I] = E_I;
    state[(int64_t)r * kStateDoubles + kWE + I] = wE_I;
}

struct FinalArgs {
    const int16_t* spins;
    const float* P;         // CubicTab's rows, and its constants in double
    double lam, sgn, C44;
    const float* u;
    float* sigma;       // may be null
    double* partials;
    const double* state;
    const RepDev* reps;
    const int32_t* node_rep;
    int64_t plane;
};

// The strain's sum and the stress are formed in double (once per refresh, and memory bound): what is
// left of the error is the displacements' and the table's.
__global__ __launch_bounds__(256) void k_global_final(FinalArgs a)
{
    const NodeRange nr = node_range(a.reps, a.node_rep);
    const RepDev& R = nr.R;
    const int K = R.K;
    const double* st = a.state + (int64_t)a.node_rep[blockIdx.x] * kStateDoubles;
    const int16_t* spins = a.spins + R.site_off;
    const float* Ptab = a.P + R.grain_off * kProj;
    const float* u = a.u + R.site_off;
    const float zero[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    double U[1] = {0.0};
    for (int64_t v = nr.first; v < R.n3; v += nr.stride) {
        const int x = (int)(v % K), y = (int)((v / K) % K), z = (int)(v / ((int64_t)K * K));
        float g[6], c[kProjUsed];
        voxel_strain(u, a.plane, K, x, y, z, zero, g);
        cubic_row(Ptab, spins[v], c);
        double e[6], s[6];
#pragma unroll
        for (int I = 0; I < 6; ++I) e[I] = st[kE + I] + (double)g[I];
        cubic_stress(c, a.lam, 0.0, a.sgn, 1.0, e, s);
        double d = 0.0;
#pragma unroll
        for (int I = 0; I < 6; ++I) {
            s[I] *= a.C44;
            d += s[I] * e[I];
        }
        U[0] += 0.5 * d;
        if (a.sigma)
#pragma unroll
            for (int I = 0; I < 6; ++I) a.sigma[(int64_t)I * a.plane + R.site_off + v] = (float)s[I];
    }
    block_sum_to<1>(a.partials, U);
}

// One block per replica: stored energy = fixed-order sum of the block partials.
// A non-finite stress or strain anywhere in the replica makes its energy non-finite, which
// raises kNfGlobal.
__global__ __launch_bounds__(256) void k_sum_U(double* state, const double* partials, const RepDev* reps,
                                               uint32_t* nonfinite)
{
    const RepDev R = reps[blockIdx.x];
    const int t = threadIdx.x;
    double s = 0.0;
    for (int b = t; b < R.node_blocks; b += 256) s += partials[(int64_t)(R.node_first + b) * 8];
    const double v[1] = {s};
    const double tot = block_total<1>(v);
    if (t == 0) {
        state[(int64_t)blockIdx.x * kStateDoubles + kU] = tot;
        if (!isfinite(tot)) atomicOr(nonfinite, (uint32_t)kNfGlobal);
    }
}

struct ReussArgs {
    const int16_t* spins;
    const float* Stab;
    double* partials;
    const RepDev* reps;
    const int32_t* node_rep;
};

// Per-block sums of S_{q_v} Sigma (the uniform-stress strain of each site).
__global__ __launch_bounds__(256) void k_reuss(ReussArgs a)
{
    const NodeRange nr = node_range(a.reps, a.node_rep);
    const RepDev& R = nr.R;
    const int16_t* spins = a.spins + R.site_off;
    const float* Stab = a.Stab + R.grain_off * kTab;
    float Sig[6];
#pragma unroll
    for (int I = 0; I < 6; ++I) Sig[I] = (float)R.Sigma[I];
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t v = nr.first; v < R.n3; v += nr.stride) {
        float e[6];
        symv21(Stab + (int64_t)spins[v] * kTab, Sig, e);
#pragma unroll
        for (int I = 0; I < 6; ++I) acc[I] += (double)e[I];
    }
    block_sum_to<6>(a.partials, acc);
}

// One block per replica: E = mean(S_q) Sigma, wE = 0.
__global__ __launch_bounds__(256) void k_reuss_E(double* state, const double* partials, const RepDev* reps)
{
    const RepDev R = reps[blockIdx.x];
    const int t = threadIdx.x;
    double s[6] = {0, 0, 0, 0, 0, 0};
    for (int b = t; b < R.node_blocks; b += 256)
#pragma unroll
        for (int I = 0; I < 6; ++I) s[I] += partials[(int64_t)(R.node_first + b) * 8 + I];
    const double tot = block_total<6>(s);
    if (t < 6) {
        double* st = state + (int64_t)blockIdx.x * kStateDoubles;
        st[kE + t] = tot / (double)R.n3;
        st[kWE + t] = 0.0;
    }
}

__global__ void k_zero_wE(double* state, int n_rep)
{
    for (int r = blockIdx.x; r < n_rep; r += gridDim.x)
        if (threadIdx.x < 6) state[(int64_t)r * kStateDoubles + kWE + threadIdx.x] = 0.0;
}

// ---- lattice reductions ----

// Unlike ordered pairs of neighbours.  A pair and its reverse are both unlike or neither, so each site looks in
// one of every two opposite directions (+x; +y with any x; +z with any x, y) and counts twice.  A thread takes two
// sites in a row, whose neighbours in a row are four sites read once; a block adds its sum to one of
// kCountCopies.  Bound by the reads, five rows a pair from cache (26 neighbours); before, with all 26
// neighbours of a site and an atomic a wavefront on one word, that word bound it: a call at 100^3 took 235 us,
// now 52 (copy and synchronisation included); one grain at 320^3 315 and 135.
template <int M>
__global__ __launch_bounds__(256) void k_unlike(const int16_t* spins, int K, int64_t n3, unsigned long long* out)
{
    unsigned int cnt = 0;
    const int Kh = K >> 1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n3 / 2;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = 2 * (int)(i % Kh), y = (int)((i / Kh) % K), z = (int)(i / ((int64_t)Kh * K));
        const int xm = x > 0 ? x - 1 : K - 1, xp = x + 2 < K ? x + 2 : 0;
        const int yp = y + 1 < K ? y + 1 : 0, ym = y > 0 ? y - 1 : K - 1, zp = z + 1 < K ? z + 1 : 0;
        auto row = [&](int yy, int zz) { return spins + (int64_t)K * (yy + (int64_t)K * zz); };
        const int16_t* r = row(y, z);
        const int a = r[x], b = r[x + 1];
        cnt += (a != b) + (b != r[xp]);
        if (M == 6) {
            const int16_t *ry = row(yp, z), *rz = row(y, zp);
            cnt += (a != ry[x]) + (b != ry[x + 1]) + (a != rz[x]) + (b != rz[x + 1]);
        } else {
            const int16_t* rows[4] = {row(yp, z), row(ym, zp), row(y, zp), row(yp, zp)};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int n0 = rows[k][xm], n1 = rows[k][x], n2 = rows[k][x + 1], n3_ = rows[k][xp];
                cnt += (a != n0) + (a != n1) + (a != n2) + (b != n1) + (b != n2) + (b != n3_);
            }
        }
    }
    block_count_to(out, cnt, 2);
}

// Sites by texture bin.  A lane adds to its own copy of the block's histogram, so that lanes of one bin (most
// of them) do not wait for each other.
__global__ __launch_bounds__(256) void k_texture(const int16_t* spins, const int32_t* bin, int64_t n3, int nbins,
                                                 unsigned long long* hist)
{
    __shared__ unsigned int h[64][32];
    for (int i = threadIdx.x; i < 64 * 32; i += 256) (&h[0][0])[i] = 0;
    __syncthreads();
    const int4* sp = reinterpret_cast<const int4*>(spins);   // n3 and a replica's offset are multiples of 8
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n3 / 8; i += (int64_t)gridDim.x * blockDim.x) {
        const int4 v = sp[i];
        const int w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            atomicAdd(&h[bin[w[k] & 0xffff]][threadIdx.x & 31], 1u);
            atomicAdd(&h[bin[(int)((unsigned)w[k] >> 16)]][threadIdx.x & 31], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < nbins) {
        unsigned int s = 0;
        for (int c = 0; c < 32; ++c) s += h[threadIdx.x][(c + threadIdx.x) & 31];
        if (s) atomicAdd(&hist[threadIdx.x], (unsigned long long)s);
    }
}

// ---- launchers ----

hipError_t launch_reuss(hmc_ctx_s* c)
{
    ReussArgs a;
    a.spins = c->d.spins;
    a.Stab = c->d.Stab;
    a.partials = c->d.partials;
    a.reps = c->d.reps;
    a.node_rep = c->d.node_rep;
    hipLaunchKernelGGL(k_reuss, dim3(c->node_blocks), dim3(256), 0, c->stream, a);
    hipLaunchKernelGGL(k_reuss_E, dim3(c->n_rep), dim3(256), 0, c->stream, c->d.state, c->d.partials, c->d.reps);
    return hipGetLastError();
}

hipError_t seq_begin(hmc_ctx_s* c, hipStream_t s)
{
    // the first step adds into buffer 0, which starts cleared; each step clears the next
    const int tok = s == c->stream ? prof_begin(c, kProfRefreshOther) : -1;
    // (buffers 0 and 1: 2 x kSumSlots 64-bit words per replica, 2 uint32 each)
    const hipError_t e = launch_fill_u32((uint32_t*)c->d.sums, 0u, 4 * (int64_t)c->n_rep * kSumSlots, s);
    prof_end(c, tok);
    return e;
}

hipError_t seq_step(hmc_ctx_s* c, hipStream_t s, int i, const float* uin, float* uout, double* E_record)
{
    const int64_t per = (int64_t)c->n_rep * kSumSlots;
    GlobArgs a;
    a.spins = c->d.spins;
    a.C = cubic_tab(c);
    a.uin = uin;
    a.uout = uout;
    a.w = c->d.w;
    a.sums_in = i > 0 ? c->d.sums + ((i - 1) % 3) * per : nullptr;
    a.sums_out = c->d.sums + (i % 3) * per;
    a.sums_clear = c->d.sums + ((i + 1) % 3) * per;
    a.st_in = i > 0 ? c->d.seq_state + (int64_t)((i - 1) & 1) * c->n_rep * kSeqState : c->d.state + kE;
    a.st_in_stride = i > 0 ? kSeqState : kStateDoubles;
    a.st_out = c->d.seq_state + (int64_t)(i & 1) * c->n_rep * kSeqState;
    a.E_record = E_record;
    a.reps = c->d.reps;
    a.tile_rep = c->d.tile_rep;
    a.order = c->block_order;
    a.plane = c->total_sites;
    a.single = c->n_rep == 1;
    a.K = c->reps[0].K;
    a.tile_z = c->reps[0].tile_z;
    a.alpha = c->reps[0].glob_alpha;
    a.beta = c->reps[0].glob_beta;
    const int tok = s == c->stream ? prof_begin(c, kProfRefreshStep) : -1;
    const dim3 g(c->tile_blocks);
    if (c->flat_depth == 1) {
        hipLaunchKernelGGL(k_global_step_flat<1>, g, dim3(kFlatThreads), 0, s, a);
    } else if (c->flat_depth == 2) {
        hipLaunchKernelGGL(k_global_step_flat<2>, g, dim3(kFlatThreads), 0, s, a);
    } else if (c->flat_depth == 4) {
        hipLaunchKernelGGL(k_global_step_flat<4>, g, dim3(kFlatThreads), 0, s, a);
    } else if (c->reps[0].tile_y == 32) {
        if (c->step_streams)
            hipLaunchKernelGGL((k_global_step_tiled<32, true>), g, dim3(kTileX * 32), 0, s, a);
        else
            hipLaunchKernelGGL((k_global_step_tiled<32, false>), g, dim3(kTileX * 32), 0, s, a);
    } else if (c->reps[0].tile_y == 16) {
        if (c->step_streams)
            hipLaunchKernelGGL((k_global_step_tiled<16, true>), g, dim3(kTileX * 16), 0, s, a);
        else
            hipLaunchKernelGGL((k_global_step_tiled<16, false>), g, dim3(kTileX * 16), 0, s, a);
    } else {
        if (c->step_streams)
            hipLaunchKernelGGL((k_global_step_tiled<8, true>), g, dim3(kTileX * 8), 0, s, a);
        else
            hipLaunchKernelGGL((k_global_step_tiled<8, false>), g, dim3(kTileX * 8), 0, s, a);
    }
    prof_end(c, tok);
    return hipGetLastError();
}

hipError_t seq_end(hmc_ctx_s* c, hipStream_t s, int n)
{
    if (n <= 0) return hipSuccess;
    const int64_t per = (int64_t)c->n_rep * kSumSlots;
    const int tok = s == c->stream ? prof_begin(c, kProfRefreshOther) : -1;
    hipLaunchKernelGGL(k_seq_fold, dim3(c->n_rep), dim3(64), 0, s, c->d.state,
                       c->d.seq_state + (int64_t)((n - 1) & 1) * c->n_rep * kSeqState,
                       c->d.sums + ((n - 1) % 3) * per, c->d.reps);
    prof_end(c, tok);
    return hipGetLastError();
}

hipError_t launch_global_steps(hmc_ctx_s* c, int n_steps)
{
    if (n_steps <= 0) return hipSuccess;
    hipError_t e = seq_begin(c, c->stream);
    for (int s = 0; s < n_steps && e == hipSuccess; ++s) {
        e = seq_step(c, c->stream, s, c->d.u[c->cur_u], c->d.u[1 - c->cur_u], nullptr);
        c->cur_u = 1 - c->cur_u;
    }
    if (e == hipSuccess) e = seq_end(c, c->stream, n_steps);
    return e;
}

hipError_t launch_global_final(hmc_ctx_s* c, bool write_sigma)
{
    FinalArgs a;
    a.spins = c->d.spins;
    a.P = c->d.Ptab;
    a.lam = cubic_lam(c);
    a.sgn = cubic_tab(c).sgn;
    a.C44 = c->p.C44;
    a.u = c->d.u[c->cur_u];
    a.sigma = write_sigma ? c->d.sigma : nullptr;
    a.partials = c->d.partials;
    a.state = c->d.state;
    a.reps = c->d.reps;
    a.node_rep = c->d.node_rep;
    a.plane = c->total_sites;
    const int tok = prof_begin(c, kProfRefreshOther);
    hipLaunchKernelGGL(k_global_final, dim3(c->node_blocks), dim3(256), 0, c->stream, a);
    hipLaunchKernelGGL(k_sum_U, dim3(c->n_rep), dim3(256), 0, c->stream, c->d.state, c->d.partials, c->d.reps,
                       c->d.counters + kNonFinite);
    prof_end(c, tok);
    return hipGetLastError();
}

hipError_t launch_zero_wE(hmc_ctx_s* c)
{
    hipLaunchKernelGGL(k_zero_wE, dim3(c->n_rep < 1024 ? c->n_rep : 1024), dim3(64), 0, c->stream, c->d.state,
                       c->n_rep);
    return hipGetLastError();
}

hipError_t launch_unlike_bonds(hmc_ctx_s* c, int rep)
{
    const RepDev& R = c->reps[rep];
    int64_t g = (R.n3 / 2 + 255) / 256;
    if (g > 2048) g = 2048;
    const int16_t* sp = c->d.spins + R.site_off;
    if (c->p.neighbors == 26)
        hipLaunchKernelGGL(k_unlike<26>, dim3((unsigned)g), dim3(256), 0, c->stream, sp, R.K, R.n3, c->d.bonds);
    else
        hipLaunchKernelGGL(k_unlike<6>, dim3((unsigned)g), dim3(256), 0, c->stream, sp, R.K, R.n3, c->d.bonds);
    return hipGetLastError();
}

hipError_t launch_texture(hmc_ctx_s* c, int rep, int nbins)
{
    const RepDev& R = c->reps[rep];
    int64_t g = (R.n3 / 8 + 255) / 256;
    if (g > 512) g = 512;
    hipLaunchKernelGGL(k_texture, dim3((unsigned)g), dim3(256), 0, c->stream, c->d.spins + R.site_off,
                       c->d.tex_bin + R.grain_off, R.n3, nbins, c->d.hist);
    return hipGetLastError();
}

}  // namespace hmc
