// hmc_mp8.hip -- the global quasi-static solve with 2 x 2 x 2 material points per background
// cell (the arrangement of the paper's MPM, Appendix: a fixed number of particles per cell, two
// per direction), a variant of the one-point-per-voxel default of hmc_elastic.hip.
//
// The mesh has (K/2)^3 periodic nodes at the corners of cells of 2 x 2 x 2 sites.  Every site is
// a material point with its own stiffness at local coordinates +-1/2 of its cell; its strain is
// the gradient of the trilinear interpolation of the cell's 8 corner displacements there (the
// cell edge is 2 sites, so d/dx = d/dxi), its nodal forces the transpose.  The relaxation is the
// default's: average-stress control of the macroscopic strain E, heavy-ball steps
//   w <- beta w + alpha r,  u <- u + w,   wE <- beta wE + alphaE (Sigma - <sigma>),  E <- E + wE,
// with the Reuss start and the warm start of the default.  Stable for alpha below the Polyak
// value of L = 8 x the largest Mandel eigenvalue of the stiffness (the identity material's
// Hessian peaks at 8 here, against 4 for one point per voxel).
//
// One step is one launch (k_mp8_step) for every replica of a batch.  A replica's node fields occupy the
// first (K/2)^3 entries of its slice of each displacement plane and alternate between the two displacement
// buffers; a sequence ends in the first.
#include <algorithm>

#include "hmc_device.h"

namespace hmc {

namespace {

// Weight of the edge at bit b (0 or 1) of a cell direction for the point at sub-position p
// there: the trilinear shape functions' factor 1 +- xi_p with xi_p = +-1/2.
__host__ __device__ constexpr float mp_w(int b, int p) { return b == p ? 1.5f : 0.5f; }

// Work-groups per replica of the final pass: one per 256 cells, at most 4096 (it strides
// beyond).  The same count alone and in a batch, so each replica's partial sums are the
// same numbers in the same order either way.
__host__ __device__ inline int mp8_blocks(int K)
{
    const int64_t Kc = K / 2, nc = Kc * Kc * Kc;
    const int64_t b = (nc + 255) / 256;
    return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

// The cells around a step's tile of nodes: one thread a cell column.
constexpr int kMp8Threads = 256;
// From this many blocks a launch (as many as run at once) the points' rows are a load on the vector cache
// rather than a wait: there a lane whose next point lies in the same grain keeps its row (320^3: 133 -> 117 us a
// step; 224^3 57 -> 46; 200^3 49.4 -> 48.7; but 64^3, whose waits it adds to, 8.7 -> 9.4, and 96^3 13.8 -> 15.1).
constexpr int kMp8KeepBlocks = 700;

struct Mp8StepArgs {
    const int16_t* spins;
    CubicTab C;
    const float* uin;        // 3 planes of `plane` floats; a replica's nodes first in its slice
    float* uout;
    float* w;
    const unsigned long long* sums_in;   // as in the one-point step (GlobArgs)
    unsigned long long* sums_out;
    unsigned long long* sums_clear;
    const double* st_in;
    int st_in_stride;
    double* st_out;
    const RepDev* reps;
    int64_t plane;
    int order;
};

// g(p, q) = s + 1/2 (+-d1) + 1/2 (+-d2) + 1/4 (+-+-d12): a bilinear function at the four +-1/2 from its sums and
// differences over the corners.
__device__ __forceinline__ void bilinear(float s, float d1, float d2, float d12, float g[2][2][3], int j)
{
    const float s0 = fmaf(-0.5f, d1, s), s1 = fmaf(0.5f, d1, s), t0 = fmaf(-0.5f, d12, d2), t1 = fmaf(0.5f, d12, d2);
    g[0][0][j] = fmaf(-0.5f, t0, s0);
    g[1][0][j] = fmaf(-0.5f, t1, s1);
    g[0][1][j] = fmaf(0.5f, t0, s0);
    g[1][1][j] = fmaf(0.5f, t1, s1);
}

// The sum of t over its four points and the differences along the first direction, the second and both.
__device__ __forceinline__ void plane_sums(const float t[2][2][3], int j, float& s, float& d1, float& d2, float& d12)
{
    const float s0 = t[0][0][j] + t[1][0][j], s1 = t[0][1][j] + t[1][1][j];
    const float e0 = t[1][0][j] - t[0][0][j], e1 = t[1][1][j] - t[0][1][j];
    s = s0 + s1;
    d2 = s1 - s0;
    d1 = e0 + e1;
    d12 = e1 - e0;
}

// One explicit step.  A block owns a tile of nodes and marches through its layers; a thread takes one
// column of the cells around them.  Per layer a thread reads its cell's four upper corners (the lower
// ones stay from the layer below) and its eight points' rows, forms gradients, stresses and the transpose, and puts
// what it gives the nodes between this layer and the one below into LDS, where each own node adds its four
// cells' parts and takes its heavy-ball step.  The stress sums become the next step's E as in the one-point step.
// Bound by VALU and, in polycrystals, the gather of the rows: about 950 operations a cell (8 x 35 of them the
// stresses, 96 the FP64 sums) keep the units busy 60 % of the time at 200^3, the vector cache as long.  A cell
// pass that wrote 24 corner forces a cell, a node pass that gathered them and a launch for the stress sums, as
// three launches, took 13.6 us at 16^3, 30.6 at 128^3, 89 at 200^3 and 362 at 320^3; this one 7.9, 19.4, 48.7
// and 115.
template <bool KEEP>
__global__ __launch_bounds__(kMp8Threads, 3) void k_mp8_step(Mp8StepArgs a)
{
    __shared__ float sF[2][12][kMp8Threads];   // the forces on a cell's four corner columns, two layers
    __shared__ double sE[6];
    const int r = blockIdx.y, t = threadIdx.x;
    const RepDev& R = a.reps[r];
    const int Kc = R.K >> 1, K = R.K, TX = R.mp_tile[0], TY = R.mp_tile[1], TZ = R.mp_tile[2];
    const int ntx = (Kc + TX - 1) / TX, nty = (Kc + TY - 1) / TY, ntz = (Kc + TZ - 1) / TZ;
    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);
    if (lb >= ntx * nty * ntz) return;   // the whole work-group leaves together
    if (t < 6) {
        double E_I, wE_I;
        advance_E(R, r, a.st_in, a.st_in_stride, a.sums_in, t, E_I, wE_I);
        sE[t] = E_I;
        if (lb == 0) {
            a.st_out[(int64_t)r * kSeqState + t] = E_I;
            a.st_out[(int64_t)r * kSeqState + 6 + t] = wE_I;
        }
    }
    if (lb == 0 && t < kSumSlots) a.sums_clear[(int64_t)r * kSumSlots + t] = 0ull;

    const int x0 = lb % ntx * TX, y0 = lb / ntx % nty * TY, z0 = lb / (ntx * nty) * TZ;
    const int z1 = min(z0 + TZ, Kc), vx = TX + 1;
    const int16_t* spins = a.spins + R.site_off;
    const float* uin = a.uin + R.site_off;
    const float* rows = a.C.P + R.grain_off * kProj;
    // the thread's cell column, (-1, -1) relative to the tile first; a thread without one takes the last
    const int ncell = vx * (TY + 1), tc = min(t, ncell - 1);
    const int cx = tc % vx, cy = tc / vx;
    const int X = wrap_once(x0 - 1 + cx, Kc), Y = wrap_once(y0 - 1 + cy, Kc);
    const int X1 = X + 1 < Kc ? X + 1 : 0, Y1 = Y + 1 < Kc ? Y + 1 : 0;
    const bool sums = t < ncell && cx >= 1 && cy >= 1 && x0 - 1 + cx < Kc && y0 - 1 + cy < Kc;
    const int corner[4] = {X + Kc * Y, X1 + Kc * Y, X + Kc * Y1, X1 + Kc * Y1};
    // its node
    const int lx = t % TX, ly = t / TX, nX = x0 + lx, nY = y0 + ly;
    const bool own = ly < TY && nX < Kc && nY < Kc;
    const int64_t node_xy = own ? nX + (int64_t)Kc * nY : 0;
    const int64_t layer = (int64_t)Kc * Kc;

    float lo[4][3], up[4][3], below[4][3];   // corner displacements; the layer below's forces on its upper corners
    int sp[4];                               // the points' grains, two of a row each
    auto fetch = [&](int z) {                // upper corners and points of cell layer z
        const int zc = wrap_once(z, Kc), zu = zc + 1 < Kc ? zc + 1 : 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) up[k][j] = uin[j * a.plane + zu * layer + corner[k]];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            sp[q] = *reinterpret_cast<const int*>(
                spins + 2 * X + (int64_t)K * (2 * Y + (q & 1) + (int64_t)K * (2 * zc + (q >> 1))));
    };
    fetch(z0 - 1);
    {
        const int zl = wrap_once(z0 - 1, Kc);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) lo[k][j] = uin[j * a.plane + zl * layer + corner[k]];
    }
    __syncthreads();
    float E[6];
#pragma unroll
    for (int I = 0; I < 6; ++I)   // the same in every lane: kept in scalar registers
        E[I] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int((float)sE[I])));
    double acc[6] = {0, 0, 0, 0, 0, 0};
    const float alpha = (float)(0.125 * R.glob_alpha * a.C.C44), beta = R.glob_beta;

    for (int z = z0 - 1; z < z1; ++z) {
        float wn[3], un[3];
        const int64_t n = node_xy + layer * max(z, z0);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            wn[j] = a.w[R.site_off + j * a.plane + n];
            un[j] = uin[j * a.plane + n];
        }
        // Differences along the edges first, then sums (+) and differences (-) over the other two directions:
        // in these a point's +-1/2 is a factor of +-1/2.  The name says which directions are differences.
        float gx[2][2][3], gy[2][2][3], gz[2][2][3];   // 8 d u / dx by (py, pz), d u / dy by (px, pz), dz by (px, py)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const float a0 = lo[1][j] - lo[0][j], a1 = lo[3][j] - lo[2][j];
            const float a2 = up[1][j] - up[0][j], a3 = up[3][j] - up[2][j];
            const float as0 = a0 + a1, ad0 = a1 - a0, as1 = a2 + a3, ad1 = a3 - a2;
            const float X = as0 + as1, XZ = as1 - as0, XY = ad0 + ad1, XYZ = ad1 - ad0;
            const float b0 = (lo[2][j] - lo[0][j]) + (lo[3][j] - lo[1][j]);
            const float b1 = (up[2][j] - up[0][j]) + (up[3][j] - up[1][j]);
            const float Yd = b0 + b1, YZ = b1 - b0;
            const float Zd = ((up[0][j] - lo[0][j]) + (up[1][j] - lo[1][j])) +
                             ((up[2][j] - lo[2][j]) + (up[3][j] - lo[3][j]));
            bilinear(X, XY, XZ, XYZ, gx, j);
            bilinear(Yd, XY, YZ, XYZ, gy, j);
            bilinear(Zd, XZ, YZ, XYZ, gz, j);
        }
        // tractions across x by (py, pz), y by (px, pz) and z by (px, py), summed over the cell's two points
        float tx[2][2][3], ty[2][2][3], tz[2][2][3];
        // from point to neighbouring point, so that most lanes have the next one's row already (KEEP)
        float c[kProjUsed];
        int have = -1;
        bool sx[2][2] = {}, sy[2][2] = {}, sz[2][2] = {};   // begun
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int p = i ^ (i >> 1), px = p & 1, py = (p >> 1) & 1, pz = p >> 2;
            const int pair = sp[p >> 1], q = px ? pair >> 16 : (int)(int16_t)pair;
            float e[6], s[6];
            if (!KEEP || q != have) cubic_row(rows, q, c);
            have = q;
            e[0] = fmaf(0.125f, gx[py][pz][0], E[0]);
            e[1] = fmaf(0.125f, gy[px][pz][1], E[1]);
            e[2] = fmaf(0.125f, gz[px][py][2], E[2]);
            e[3] = fmaf(0.125f, gz[px][py][1] + gy[px][pz][2], E[3]);
            e[4] = fmaf(0.125f, gz[px][py][0] + gx[py][pz][2], E[4]);
            e[5] = fmaf(0.125f, gy[px][pz][0] + gx[py][pz][1], E[5]);
            cubic_stress(c, a.C, e, s);
            if (sums && z >= z0)
#pragma unroll
                for (int I = 0; I < 6; ++I) acc[I] += (double)s[I];
            const float rx[3] = {s[0], s[5], s[4]}, ry[3] = {s[5], s[1], s[3]}, rz[3] = {s[4], s[3], s[2]};
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                tx[py][pz][j] = sx[py][pz] ? tx[py][pz][j] + rx[j] : rx[j];
                ty[px][pz][j] = sy[px][pz] ? ty[px][pz][j] + ry[j] : ry[j];
                tz[px][py][j] = sz[px][py] ? tz[px][py][j] + rz[j] : rz[j];
            }
            sx[py][pz] = sy[px][pz] = sz[px][py] = true;
        }
        float F[2][4][3];   // 8 times the forces on the lower and upper corners: the transpose
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            float X, Yd, Zd, XY, XZ, YZ, XYZ, d1, d2, d3;
            plane_sums(tx, j, X, XY, XZ, XYZ);
            plane_sums(ty, j, Yd, d1, YZ, d3);
            XY += d1;
            XYZ += d3;
            plane_sums(tz, j, Zd, d1, d2, d3);
            XZ += d1;
            YZ += d2;
            XYZ += d3;
#pragma unroll
            for (int bz = 0; bz < 2; ++bz) {
                const float h = bz ? 0.5f : -0.5f;
                const float px = fmaf(h, XZ, X), py = fmaf(h, YZ, Yd), pxy = fmaf(h, XYZ, XY);
                const float n0 = bz ? Zd - py : -Zd - py, n1 = bz ? Zd + py : py - Zd;   // by = 0, 1
                const float m0 = fmaf(-0.5f, pxy, px), m1 = fmaf(0.5f, pxy, px);
                F[bz][0][j] = n0 - m0;
                F[bz][1][j] = n0 + m0;
                F[bz][2][j] = n1 - m1;
                F[bz][3][j] = n1 + m1;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) lo[k][j] = up[k][j];
        if (z + 1 < z1) fetch(z + 1);
        if (z >= z0) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 3; ++j) sF[z & 1][3 * k + j][t] = F[0][k][j] + below[k][j];
            __syncthreads();   // two buffers: a layer's reads end before the barrier of the next
            if (own) {
                const int c = lx + vx * ly;   // the cell at (-1, -1) from the node
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const float f = (sF[z & 1][j][c + 1 + vx] + sF[z & 1][3 + j][c + vx]) +
                                    (sF[z & 1][6 + j][c + 1] + sF[z & 1][9 + j][c]);
                    const float wnew = fmaf(-alpha, f, beta * wn[j]);
                    a.w[R.site_off + j * a.plane + n] = wnew;
                    a.uout[R.site_off + j * a.plane + n] = un[j] + wnew;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) below[k][j] = F[1][k][j];
    }
    const double tot = block_total<6>(acc);
    if (t < 6)
        atomicAdd(a.sums_out + (int64_t)r * kSumSlots + (lb & (kSumCopies - 1)) * 8 + t,
                  (unsigned long long)llrint(tot * (kSumScale * a.C.C44)));
}

// The nodes back from the second displacement buffer after an odd number of steps.
__global__ __launch_bounds__(256) void k_mp8_back(const float* from, float* to, const RepDev* reps, int64_t plane)
{
    const RepDev& R = reps[blockIdx.y];
    const int64_t Kc = R.K >> 1, nc = Kc * Kc * Kc;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < nc; n += (int64_t)gridDim.x * blockDim.x)
#pragma unroll
        for (int j = 0; j < 3; ++j) to[j * plane + R.site_off + n] = from[j * plane + R.site_off + n];
}

struct Mp8FinalArgs {
    const int16_t* spins;
    CubicTab C;
    double lam;            // C.lam in full
    const float* u;
    float* sigma;          // 6 planes of point stresses (or null)
    double* partials;
    const double* state;
    const RepDev* reps;
    int64_t plane;
};

// Point stresses and stored energy (per-block partial sums).  Strain and stress are formed in double, as in the
// one-point solve's final pass.
__global__ __launch_bounds__(256) void k_mp8_final(Mp8FinalArgs a)
{
    const RepDev& R = a.reps[blockIdx.y];
    const int K = R.K, Kc = K >> 1, nb = mp8_blocks(K);
    if ((int)blockIdx.x >= nb) return;   // the whole work-group leaves together
    const int64_t nc = (int64_t)Kc * Kc * Kc;
    const int16_t* spins = a.spins + R.site_off;
    const float* rows = a.C.P + R.grain_off * kProj;
    const float* u = a.u + R.site_off;
    const double* st = a.state + (int64_t)blockIdx.y * kStateDoubles;
    double U[1] = {0.0};
    for (int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; cell < nc;
         cell += (int64_t)nb * blockDim.x) {
        const int X = (int)(cell % Kc), Y = (int)((cell / Kc) % Kc), Z = (int)(cell / ((int64_t)Kc * Kc));
        const int X1 = X + 1 < Kc ? X + 1 : 0, Y1 = Y + 1 < Kc ? Y + 1 : 0, Z1 = Z + 1 < Kc ? Z + 1 : 0;
        float uc[8][3];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int64_t node = (int64_t)((c & 1) ? X1 : X) +
                                 (int64_t)Kc * (((c >> 1) & 1 ? Y1 : Y) + (int64_t)Kc * ((c >> 2) & 1 ? Z1 : Z));
#pragma unroll
            for (int j = 0; j < 3; ++j) uc[c][j] = u[(int64_t)j * a.plane + node];
        }
        // differences along the cell's edges: D[d][e][j] for the 4 edges e parallel to d (e = the other two
        // bits, lower direction first); a point's gradient is d/dx = 1/8 sum_e w w D (cell edge 2 sites)
        float D[3][4][3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b1 = e & 1, b2 = e >> 1;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                D[0][e][j] = uc[1 + 2 * b1 + 4 * b2][j] - uc[0 + 2 * b1 + 4 * b2][j];
                D[1][e][j] = uc[b1 + 2 + 4 * b2][j] - uc[b1 + 0 + 4 * b2][j];
                D[2][e][j] = uc[b1 + 2 * b2 + 4][j] - uc[b1 + 2 * b2 + 0][j];
            }
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int px = p & 1, py = (p >> 1) & 1, pz = (p >> 2) & 1;
            const int64_t v = (int64_t)(2 * X + px) + (int64_t)K * ((2 * Y + py) + (int64_t)K * (2 * Z + pz));
            // point sub-positions along the two other directions of each d, lower first
            const int q1[3] = {py, px, px}, q2[3] = {pz, pz, py};
            float g[3][3], c[kProjUsed];   // g[d][j] = d u_j / d x_d
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    float gs = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) gs += (0.125f * mp_w(e & 1, q1[d]) * mp_w(e >> 1, q2[d])) * D[d][e][j];
                    g[d][j] = gs;
                }
            double e6[6], s[6], dd = 0.0;
            e6[0] = (double)g[0][0] + st[kE];
            e6[1] = (double)g[1][1] + st[kE + 1];
            e6[2] = (double)g[2][2] + st[kE + 2];
            e6[3] = ((double)g[2][1] + (double)g[1][2]) + st[kE + 3];
            e6[4] = ((double)g[2][0] + (double)g[0][2]) + st[kE + 4];
            e6[5] = ((double)g[1][0] + (double)g[0][1]) + st[kE + 5];
            cubic_row(rows, spins[v], c);
            cubic_stress(c, a.lam, 0.0, (double)a.C.sgn, 1.0, e6, s);
#pragma unroll
            for (int I = 0; I < 6; ++I) {
                s[I] *= a.C.C44;
                dd += s[I] * e6[I];
            }
            U[0] += 0.5 * dd;
            if (a.sigma)
#pragma unroll
                for (int I = 0; I < 6; ++I) a.sigma[(int64_t)I * a.plane + R.site_off + v] = (float)s[I];
        }
    }
    block_sum_to<1>(a.partials, U, R.node_first + (int)blockIdx.x);
}

__global__ __launch_bounds__(256) void k_mp8_U(double* state, const double* partials, const RepDev* reps,
                                                uint32_t* nonfinite)
{
    const RepDev R = reps[blockIdx.x];
    const int nb = mp8_blocks(R.K);
    double s[1] = {0.0};
    for (int b = threadIdx.x; b < nb; b += 256) s[0] += partials[(int64_t)(R.node_first + b) * 8];
    const double tot = block_total<1>(s);
    if (threadIdx.x == 0) {
        state[(int64_t)blockIdx.x * kStateDoubles + kU] = tot;
        if (!isfinite(tot)) atomicOr(nonfinite, (uint32_t)kNfGlobal);   // a non-finite point stress
    }
}

dim3 mp8_grid(const hmc_ctx_s* c, int (*blocks)(int))
{
    int nb = 1;
    for (const RepDev& R : c->reps) nb = std::max(nb, blocks(R.K));
    return dim3((unsigned)nb, (unsigned)c->n_rep);
}

int step_blocks(int K)
{
    int32_t t[3];
    mp8_tile(K, t);
    const int Kc = K / 2;
    return (Kc + t[0] - 1) / t[0] * ((Kc + t[1] - 1) / t[1]) * ((Kc + t[2] - 1) / t[2]);
}

}  // namespace

// In x, y the fewest tiles whose cells, one more than nodes each way, have a thread each, equally wide.  In z
// the depth whose layers, one more than nodes, cost least: beside 3.5 us a step, a layer took 2.6, 4.05 and 5.6 us with
// one, two and three blocks on every CU (three is what its registers allow; 5.3, less for coarse grains, where lanes
// keep their rows), and beyond, where blocks follow each other, 1.65 us for each block a CU has and 1.7.  The depths it
// picks, and the step there and at others (us, grains of 8 to 17 sites): 64^3 1 (8.5; 10.8 at 2), 96^3 3 (13.8; 16.3
// at 4), 128^3 3 (19.4; 20.9 at 2, 26.9 at 5), 160^3 5 (26.3; 31.0 at 2, 30.1 at 4), 176^3 7 (35.8; 43.5 at 4, 46.3 at
// 10), 200^3 7 (48.7; 52.9 at 4, 50.0 at 10), 224^3 9 (46; 54 at 4, 57 at 13), 256^3 15 (68; 69 at 7, 90 at 14), 280^3
// 18 (83; 91 at 7, 94 at 14), 300^3 6 (99; 94 at 10, 118 at 30), 320^3 27 (115; 121 at 10, 125 at 18).
void mp8_tile(int K, int32_t tile[3])
{
    const int Kc = K / 2;
    int nx = Kc, ny = Kc;
    for (int tx = 1; tx <= Kc && tx < kMp8Threads / 2; ++tx) {
        const int ty = std::min(Kc, kMp8Threads / (tx + 1) - 1);
        const int mx = (Kc + tx - 1) / tx, my = (Kc + ty - 1) / ty;
        if (mx * my <= nx * ny) nx = mx, ny = my;   // of equal counts the widest in x
    }
    tile[0] = (Kc + nx - 1) / nx;
    tile[1] = (Kc + ny - 1) / ny;
    const int tiles = (Kc + tile[0] - 1) / tile[0] * ((Kc + tile[1] - 1) / tile[1]);
    double best = 0.0;
    for (int tz = 1; tz <= std::min(Kc, 32); ++tz) {
        const int blocks = tiles * ((Kc + tz - 1) / tz);
        const double per_cu = blocks / 256.0, three = blocks > kMp8KeepBlocks ? 5.3 : 5.6;
        const double layer = per_cu <= 1 ? 2.6 : per_cu <= 2 ? 4.05 : per_cu <= 3 ? three : 1.65 * per_cu + 1.7;
        const double cost = 3.5 + (tz + 1) * layer;
        if (tz == 1 || cost < best) best = cost, tile[2] = tz;
    }
}

hipError_t launch_mp8_steps(hmc_ctx_s* c, int n_steps)
{
    if (n_steps <= 0) return hipSuccess;
    const int64_t per = (int64_t)c->n_rep * kSumSlots;
    const dim3 grid = mp8_grid(c, step_blocks);
    const bool keep = (int64_t)grid.x * grid.y > kMp8KeepBlocks;
    hipError_t e = seq_begin(c, c->stream);
    for (int i = 0; i < n_steps && e == hipSuccess; ++i) {
        Mp8StepArgs a;
        a.spins = c->d.spins;
        a.C = cubic_tab(c);
        a.uin = c->d.u[i & 1];
        a.uout = c->d.u[1 - (i & 1)];
        a.w = c->d.w;
        a.sums_in = i > 0 ? c->d.sums + ((i - 1) % 3) * per : nullptr;
        a.sums_out = c->d.sums + (i % 3) * per;
        a.sums_clear = c->d.sums + ((i + 1) % 3) * per;
        a.st_in = i > 0 ? c->d.seq_state + (int64_t)((i - 1) & 1) * c->n_rep * kSeqState : c->d.state + kE;
        a.st_in_stride = i > 0 ? kSeqState : kStateDoubles;
        a.st_out = c->d.seq_state + (int64_t)(i & 1) * c->n_rep * kSeqState;
        a.reps = c->d.reps;
        a.plane = c->total_sites;
        a.order = c->block_order;
        const int tok = prof_begin(c, kProfRefreshStep);
        if (keep)
            hipLaunchKernelGGL(k_mp8_step<true>, grid, dim3(kMp8Threads), 0, c->stream, a);
        else
            hipLaunchKernelGGL(k_mp8_step<false>, grid, dim3(kMp8Threads), 0, c->stream, a);
        prof_end(c, tok);
        e = hipGetLastError();
    }
    if (e == hipSuccess && (n_steps & 1)) {
        const int tok = prof_begin(c, kProfRefreshOther);
        hipLaunchKernelGGL(k_mp8_back, mp8_grid(c, mp8_blocks), dim3(256), 0, c->stream, (const float*)c->d.u[1],
                           c->d.u[0], (const RepDev*)c->d.reps, c->total_sites);
        prof_end(c, tok);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = seq_end(c, c->stream, n_steps);
    return e;
}

hipError_t launch_mp8_final(hmc_ctx_s* c, bool write_sigma)
{
    Mp8FinalArgs a;
    a.spins = c->d.spins;
    a.C = cubic_tab(c);
    a.lam = cubic_lam(c);
    a.u = c->d.u[0];
    a.sigma = write_sigma ? c->d.sigma : nullptr;
    a.partials = c->d.partials;
    a.state = c->d.state;
    a.reps = c->d.reps;
    a.plane = c->total_sites;
    const int tok = prof_begin(c, kProfRefreshOther);
    hipLaunchKernelGGL(k_mp8_final, mp8_grid(c, mp8_blocks), dim3(256), 0, c->stream, a);
    hipLaunchKernelGGL(k_mp8_U, dim3(c->n_rep), dim3(256), 0, c->stream, c->d.state, (const double*)c->d.partials,
                       (const RepDev*)c->d.reps, c->d.counters + kNonFinite);
    prof_end(c, tok);
    return hipGetLastError();
}

}  // namespace hmc
