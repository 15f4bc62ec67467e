// hmc_potts.hip -- colour-pass kernels of the Potts sweep (Sec. 3 Eqs. H_1 and metrop_1,
// Sec. 6 checkerboard with deferred updates) and small utility kernels.
//
// Four sites of the active colour class per thread.  Every trial draws its two Philox
// words and forms the trial state; the real flips (new state differs) are compacted per
// wavefront, count the change of unlike neighbour bonds and either decide at once (elastic
// term off: exact integer threshold table) or go to a compacted list for the zone-solve
// kernel (elastic term on).  Because no two sites of one class are neighbours, the
// decide-at-once path may write spins in place: every read of the pass touches other
// classes only.
#include "hmc_internal.h"

namespace hmc {

// ------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): ten rounds; in each, the first and
// third words are multiplied by fixed odd constants, the high halves are mixed with the
// other two words and the key, and the key is advanced by the golden-ratio Weyl steps.
// ------------------------------------------------------------------------------------
// a ^ b ^ k in one instruction (gfx950's three-input bitwise op with truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t k)
{
    return __builtin_amdgcn_bitop3_b32(a, b, k, 0x96);
}

// The first two words for the counter (c0, c1, 0, 0), c1 and the key the same in every lane: of the first two
// rounds the compiler takes what c0 does not reach on the scalar unit.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1, uint32_t& v0,
                                              uint32_t& v1)
{
    uint32_t c2 = 0, c3 = 0;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32 x 32 -> 64-bit product gives both halves (a single v_mad_u64_u32)
        const uint64_t pa = (uint64_t)0xD2511F53u * c0;
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = r < 2 ? (uint32_t)(pb >> 32) ^ (c1 ^ k0) : xor3((uint32_t)(pb >> 32), c1, k0);
        const uint32_t n2 = r < 3 ? (uint32_t)(pa >> 32) ^ (c3 ^ k1) : xor3((uint32_t)(pa >> 32), c3, k1);
        c0 = n0;
        c1 = (uint32_t)pb;
        c2 = n2;
        c3 = (uint32_t)pa;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    v0 = c0;
    v1 = c1;
}

// a in [-K, 2 K) into [0, K).
__device__ __forceinline__ int wrapi(int a, int K)
{
    const uint32_t m = min((uint32_t)a, (uint32_t)(a + K));
    return (int)min(m, m - (uint32_t)K);
}

struct PassArgs {
    int16_t* spins;                 // all replicas, end to end
    const RepDev* reps;
    const int32_t* pass_rep;        // chunk -> replica
    int single;                     // one replica: no table to read first
    int rep_blocks;                 // k_potts_pair: blocks of each replica
    const uint64_t* thr;            // per replica: 64 integer thresholds indexed by gb + M
    TrialEntry* list;
    uint32_t* list_count;
    hmc_trial_record* rec;          // indexed by site_off + site, or null
    unsigned long long* stats;
    int64_t* sweep;                 // Philox counter word 1 (low 32 bits); the second slot is k_potts_pair's
    const float* Stab;              // compliance tables (lower-bound screen)
    const float* sigma;             // stress planes of `plane` floats (lower-bound screen)
    int64_t plane;
    int colour;
    int screen;
    int order;                      // logical block order (hmc_set_block_order)
};

// Point-zone energy 1/2 sigma.(S_old - S_new) sigma of the trial site: a lower bound of the
// zone energy change for every zone size.
__device__ __forceinline__ double point_zone_energy(const float* __restrict__ So, const float* __restrict__ Sn,
                                                    const float s[6])
{
    double d = 0.0;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = i; j < 6; ++j) {
            const int k = sym_index(i, j);
            const double w = (i == j ? 0.5 : 1.0) * (double)s[i] * (double)s[j];
            d += w * ((double)So[k] - (double)Sn[k]);
        }
    return d;
}

// Offset of neighbour slot k.  6: -x,+x,-y,+y,-z,+z.  26: (dz,dy,dx) lexicographic over
// {-1,0,1}^3 without the centre (n = k or k + 1 past the centre; n / 3 = 11 n >> 5 for n < 32).
template <int M>
__device__ __forceinline__ void slot_offset(int k, int& dx, int& dy, int& dz)
{
    if (M == 6) {
        dx = (k == 0) ? -1 : (k == 1 ? 1 : 0);
        dy = (k == 2) ? -1 : (k == 3 ? 1 : 0);
        dz = (k == 4) ? -1 : (k == 5 ? 1 : 0);
    } else {
        const int n = k + (k >= 13), row = (11 * n) >> 5, layer = (11 * row) >> 5;
        dx = n - 3 * row - 1;
        dy = row - 3 * layer - 1;
        dz = layer - 1;
    }
}

// Active index t of a colour class, kept as (i, j, k): i counts the class's sites along x
// (K/2 of them), j along y (K/2 for 26 neighbours, K for 6), k along z.  One division pair
// places a thread's first site; its later sites, 256 indices apart, are reached by adding the
// per-block constants 256 / (K/2) and 256 % (K/2) with carries, so the per-site cost is a
// few adds instead of two integer divisions.
struct ActiveWalk {
    uint32_t i, j, k;
};

__device__ __forceinline__ ActiveWalk walk_start(uint32_t t, uint32_t Kh, uint32_t NJ)
{
    ActiveWalk w;
    const uint32_t row = t / Kh;
    w.i = t - row * Kh;
    w.k = row / NJ;
    w.j = row - w.k * NJ;
    return w;
}

__device__ __forceinline__ void walk_advance(ActiveWalk& w, uint32_t Kh, uint32_t NJ, uint32_t di, uint32_t dr)
{
    w.i += di;
    uint32_t rows = dr;
    if (w.i >= Kh) {
        w.i -= Kh;
        rows += 1;
    }
    w.j += rows;
    if (w.j >= NJ) {
        const uint32_t c = w.j / NJ;
        w.k += c;
        w.j -= c * NJ;
    }
}

template <int M>
__device__ __forceinline__ void walk_site(const ActiveWalk& w, int colour, int& x, int& y, int& z)
{
    if (M == 26) {
        x = 2 * (int)w.i + (colour & 1);
        y = 2 * (int)w.j + ((colour >> 1) & 1);
        z = 2 * (int)w.k + ((colour >> 2) & 1);
    } else {
        y = (int)w.j;
        z = (int)w.k;
        x = 2 * (int)w.i + ((y + z + colour) & 1);
    }
}

// Linear site index; every factor fits 24 bits for K <= 1024, so full-rate 24-bit multiplies.
__device__ __forceinline__ uint32_t site_of(int x, int y, int z, int K, int KK)
{
    return (uint32_t)x + __umul24((uint32_t)K, (uint32_t)y) + __umul24((uint32_t)KK, (uint32_t)z);
}

// Site (x + dx, y + dy, z + dz) of the periodic lattice; POW2: K = 2^lg.
template <bool POW2>
__device__ __forceinline__ uint32_t neighbour_site(int x, int y, int z, int K, int KK, int lg)
{
    if (POW2) {
        const int Km = K - 1;
        return (uint32_t)(x & Km) | ((uint32_t)(y & Km) << lg) | ((uint32_t)(z & Km) << (2 * lg));
    }
    return site_of(wrapi(x, K), wrapi(y, K), wrapi(z, K), K, KK);
}

// For each half of a: 1 if it differs from that of b.
__device__ __forceinline__ uint32_t halves_differ(uint32_t a, uint32_t b)
{
    uint32_t r;
    const uint32_t t = a ^ b;
    asm("v_pk_min_u16 %0, %1, %2 op_sel_hi:[1,0]" : "=v"(r) : "v"(t), "v"(1u));
    return r;
}

// Change of the unlike neighbours of (x, y, z) from state q_old to q_new.  EARLY: the reads round the corner of a
// lattice row go out with the others rather than after them.  Nine reads of eight bytes instead of 26 of two: a pass of
// 512^3 93 -> 72 us, of 200^3 10.75 -> 9.7, ten 60^3 unchanged at 4.1.
template <int M, bool EARLY>
__device__ __forceinline__ int unlike_change(const int16_t* spins, int x, int y, int z, int K, int KK, int q_old,
                                             int q_new)
{
    // byte offsets of the three x, y and z planes around the site (2 bytes per spin;
    // 2 K^3 <= 2^31 for K <= 1024): each neighbour is one add and a load off the
    // replica's spin base
    const uint32_t K2 = 2u * (uint32_t)K, KK2 = 2u * (uint32_t)KK;
    const uint32_t xs[3] = {2u * (uint32_t)wrapi(x - 1, K), 2u * (uint32_t)x, 2u * (uint32_t)wrapi(x + 1, K)};
    const uint32_t ys[3] = {(uint32_t)__umul24((uint32_t)wrapi(y - 1, K), K2), (uint32_t)__umul24((uint32_t)y, K2),
                            (uint32_t)__umul24((uint32_t)wrapi(y + 1, K), K2)};
    const uint32_t zs[3] = {(uint32_t)__umul24((uint32_t)wrapi(z - 1, K), KK2), (uint32_t)__umul24((uint32_t)z, KK2),
                            (uint32_t)__umul24((uint32_t)wrapi(z + 1, K), KK2)};
    const char* sb = reinterpret_cast<const char*>(spins);
    int gb = 0;
    if (M == 26 && K >= 4) {
        // the neighbours lie in nine rows of three, each read as the four sites from `first` on and shifted so that
        // x - 1, x and x + 1 follow from the lowest bits on; at a row's ends the one round the corner is read too
        const int first = min(max(x - 1, 0), K - 4);
        uint64_t v[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) __builtin_memcpy(&v[k], sb + (2u * (uint32_t)first + ys[k % 3] + zs[k / 3]), 8);
        const bool end = x == 0 || x == K - 1;
        uint32_t far[9];
        auto read_far = [&]() {
            const uint32_t round = x == 0 ? 2u * (uint32_t)(K - 1) : 0u;
#pragma unroll
            for (int k = 0; k < 9; ++k)
                far[k] = *reinterpret_cast<const unsigned short*>(sb + (round + ys[k % 3] + zs[k / 3]));
        };
        if (EARLY && end) read_far();
        if (end) {
            if (!EARLY) read_far();
#pragma unroll
            for (int k = 0; k < 9; ++k) v[k] = x == 0 ? v[k] << 16 | far[k] : v[k] >> 32 | (uint64_t)far[k] << 32;
        } else if (x == K - 2) {
#pragma unroll
            for (int k = 0; k < 9; ++k) v[k] >>= 16;
        }
        // unlike neighbours, counted in both halves of a word
        const uint32_t oo = (uint32_t)q_old * 0x10001u, nn = (uint32_t)q_new * 0x10001u;
        uint32_t un = 0, uo = 0, left = 0;
        auto count = [&](uint32_t pair) {
            un += halves_differ(pair, nn);
            uo += halves_differ(pair, oo);
        };
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            count((uint32_t)v[k]);
            if (k % 2 == 0)
                left = (uint32_t)(v[k] >> 32);
            else
                count(__builtin_amdgcn_perm((uint32_t)(v[k] >> 32), left, 0x05040100u));   // two rows' x + 1
        }
        count(__builtin_amdgcn_perm(oo, left, 0x05040100u));
        // less the site's own state, counted with its row and here: unlike the new one, like the old
        gb = (int)(un & 0xffffu) + (int)(un >> 16) - (int)(uo & 0xffffu) - (int)(uo >> 16) - 2;
        return gb;
    }
    if (M == 26) {   // K = 2: the seven other sites, a site that differs in n coordinates being 2^n of the slots
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            const uint32_t at = 2u * (uint32_t)((x ^ (k & 1)) | (y ^ ((k >> 1) & 1)) << 1 | (z ^ (k >> 2)) << 2);
            const uint32_t qn = *reinterpret_cast<const unsigned short*>(sb + at);
            gb += ((int)(qn != (uint32_t)q_new) - (int)(qn != (uint32_t)q_old)) << __builtin_popcount(k);
        }
        return gb;
    }
#pragma unroll
    for (int k = 0; k < M; ++k) {
        int dx, dy, dz;
        slot_offset<M>(k, dx, dy, dz);
        const uint32_t qn = *reinterpret_cast<const unsigned short*>(sb + (xs[dx + 1] + ys[dy + 1] + zs[dz + 1]));
        gb += (int)(qn != (uint32_t)q_new) - (int)(qn != (uint32_t)q_old);
    }
    return gb;
}

// A chunk of kPassSites = 4 x 256 active sites belongs to one replica.  With SPT = 4 one
// block covers a chunk and each thread takes four sites, 256 apart; with SPT = 1 four blocks
// share a chunk, one site per thread (the same sites and draws, a quarter each).  Lattices
// with few chunks per pass (128^3 with 8 colours has 256) take SPT = 1 at zero load: four
// times the wavefronts to hide the chain of dependent reads of a site.  Phase 1 draws every trial and
// keeps only the real flips (q_new != q_old), which each wavefront compacts through LDS; phase
// 2 -- the 26 neighbour reads, the decision or the screen -- then takes the block's real flips
// as one list, 256 at a time, so that it runs once per 64 real flips of the block instead of
// once per site slot (inside grains most proposals are no-ops, and a single real flip would
// otherwise hold a whole wavefront): on large lattices a block of 1024 sites usually has fewer
// than 64, and three of its four wavefronts skip phase 2.  A colour pass has tens of
// thousands of blocks on large lattices, so the block appends its elastic trials with one
// atomic on the list counter and adds its statistics to one of the spread counter copies.
static_assert(kPassSites == 4 * 256, "a chunk is four sites per thread of a 256-thread block");
// Bound at 512^3 by VALU work (117 operations a site, 35 of them Philox), the vector cache (the neighbours of the real
// flips) and reading the whole lattice once a pass (the proposals reach nearly every line: 283 MB), each 70 to 80 % of
// the time; on small lattices by its chain of dependent reads.  Power-of-two sites by bit fields, what the first
// Philox rounds owe to the sweep and the key on the scalar unit, counts from ballots instead of shuffles, the
// thresholds read with the spins (95.5 -> 93 us a pass) and the neighbours by rows of three (93 -> 72) took 256^3
// from 19.0 to 15.5 us and, with 6 neighbours, 512^3 from 216 to 190.
// SCREEN: the lower-bound screen's FP64 path is compiled in only where it is used, since it
// more than doubles the kernel's registers (126 against 48 VGPRs: 4 against 8 wavefronts per
// SIMD, which hide the chain of dependent reads of every site).
// NP2: every replica proposes a neighbour's spin and has a power-of-two edge, known at compile
// time (the common case), so the proposal and the wrap need no uniform branches.
template <int M, bool SCREEN, int SPT, bool NP2>
__global__ __launch_bounds__(256) void k_potts_pass(PassArgs a)
{
    static_assert(SPT == 1 || SPT == 4, "one or four sites per thread");
    constexpr int SUB = kPassSites / (256 * SPT);    // blocks per chunk
    __shared__ uint32_t s_item[4][SPT * 64][3];      // per wavefront: coords, q_old | q_new << 16, r1
    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);   // neighbouring rows share an L2
    const int chunk = lb / SUB, sub = lb % SUB;
    const int r = a.single ? 0 : a.pass_rep[chunk];
    const RepDev R = a.reps[r];
    const uint32_t first =
        (uint32_t)(chunk - R.pass_first) * (uint32_t)kPassSites + (uint32_t)sub * 256u + threadIdx.x;
    const uint32_t n_active = (uint32_t)(R.n3 / (M == 26 ? 8 : 2));
    const bool elastic = R.elastic != 0;
    int16_t* spins = a.spins + R.site_off;
    const int K = R.K, KK = K * K, Km = K - 1;
    const bool pow2 = NP2 || (K & Km) == 0;
    const bool nbr_prop = NP2 || R.proposal == 0;
    const uint32_t sweep = (uint32_t)(*a.sweep);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const unsigned long long below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    uint32_t n_wave = 0;
    const uint32_t Kh = (uint32_t)R.Kh, NJ = (M == 26) ? Kh : (uint32_t)K;
    const int lg = 31 - __builtin_clz((unsigned)K);   // NP2: K = 2^lg
    const uint32_t di = NP2 ? 0u : 256u % Kh, dr = NP2 ? 0u : 256u / Kh;
    ActiveWalk walk{0u, 0u, 0u};
    if (!NP2) walk = walk_start(first, Kh, NJ);
    // the zero-load decisions' thresholds, read with the spins and put down with the lists
    __shared__ uint64_t s_thr[64];
    uint64_t thr = 0;
    if (!elastic && threadIdx.x < 64) thr = a.thr[(int64_t)r * 64 + threadIdx.x];

    // ---- phase 1: draws, proposals; real flips to the wavefront's list ----
    // In three stages, so that all of a thread's spin reads are in flight together: the sites
    // and their draws (arithmetic only), then every own and proposed-neighbour spin read, then
    // the decisions and the list appends.
    uint32_t site[SPT], packed[SPT], nbr[SPT], r0[SPT], r1[SPT];
    bool ok[SPT];
#pragma unroll
    for (int it = 0; it < SPT; ++it) {
        const uint32_t t = first + (uint32_t)it * 256u;
        ok[it] = t < n_active;
        if (NP2)   // the class's (i, j, k) are bit fields of the index
            walk = {t & (Kh - 1), (t >> (lg - 1)) & (NJ - 1), t >> (M == 26 ? 2 * lg - 2 : 2 * lg - 1)};
        else if (it > 0)
            walk_advance(walk, Kh, NJ, di, dr);
        int x, y, z;
        walk_site<M>(walk, a.colour, x, y, z);
        site[it] = NP2 ? (uint32_t)x | ((uint32_t)y << lg) | ((uint32_t)z << (2 * lg)) : site_of(x, y, z, K, KK);
        packed[it] = (uint32_t)x | ((uint32_t)y << 10) | ((uint32_t)z << 20);
        philox4x32_10(site[it], sweep, R.key0, R.key1, r0[it], r1[it]);
        nbr[it] = site[it];
        if (nbr_prop) {
            const int k = (int)__umulhi(r0[it], (uint32_t)M);
            int dx, dy, dz;
            slot_offset<M>(k, dx, dy, dz);
            if (NP2)
                nbr[it] = neighbour_site<true>(x + dx, y + dy, z + dz, K, KK, lg);
            else if (pow2)   // uniform branch: a power-of-two edge wraps by a mask
                nbr[it] = site_of((x + dx) & Km, (y + dy) & Km, (z + dz) & Km, K, KK);
            else
                nbr[it] = neighbour_site<false>(x + dx, y + dy, z + dz, K, KK, lg);
        }
    }
    int q_old[SPT], q_nb[SPT];
    const char* sb = reinterpret_cast<const char*>(spins);
#pragma unroll
    for (int it = 0; it < SPT; ++it) {
        q_old[it] = 0;
        q_nb[it] = 0;
        if (ok[it]) {
            q_old[it] = *reinterpret_cast<const int16_t*>(sb + 2u * site[it]);
            q_nb[it] = *reinterpret_cast<const int16_t*>(sb + 2u * nbr[it]);
        }
    }
#pragma unroll
    for (int it = 0; it < SPT; ++it) {
        bool real = false;
        uint32_t qq = 0;
        if (ok[it]) {
            int q_new = q_nb[it];
            if (!nbr_prop) {
                const uint32_t step = __umulhi(r0[it], (uint32_t)(R.Q - 1));
                q_new = (int)(((uint32_t)q_old[it] + 1u + step) % (uint32_t)R.Q);
            }
            real = (q_new != q_old[it]);
            qq = (uint32_t)q_old[it] | ((uint32_t)q_new << 16);
            if (!real && a.rec) {
                hmc_trial_record rc;
                rc.q_new = q_new;
                rc.gb = 0;
                rc.dPi = 0.0f;
                rc.r1 = r1[it];
                rc.flags = 0;
                rc.reserved = 0;
                a.rec[R.site_off + site[it]] = rc;
            }
        }
        const unsigned long long m = __ballot(real);
        if (real) {
            const uint32_t j = n_wave + (uint32_t)__popcll(m & below);
            s_item[wid][j][0] = packed[it];
            s_item[wid][j][1] = qq;
            s_item[wid][j][2] = r1[it];
        }
        n_wave += (uint32_t)__popcll(m);
    }
    __shared__ uint32_t s_nw[4];
    if (lane == 0) s_nw[wid] = n_wave;
    if (!elastic && threadIdx.x < 64) s_thr[threadIdx.x] = thr;
    __syncthreads();
    // the four wavefronts' lists, read as one list of the block's real flips
    const uint32_t c0 = s_nw[0], c1 = c0 + s_nw[1], c2 = c1 + s_nw[2], n_block = c2 + s_nw[3];

    // ---- phase 2: the block's real flips, 256 at a time (wavefronts past the end skip it) ----
    TrialEntry ent[SPT];
    bool solve[SPT], other[SPT];   // to the list; screened or (zero load) accepted
#pragma unroll
    for (int it = 0; it < SPT; ++it) {
        const uint32_t j = (uint32_t)(it * 256) + threadIdx.x;
        solve[it] = other[it] = false;
        if (j < n_block) {
            const int wv = (j >= c0) + (j >= c1) + (j >= c2);
            const uint32_t jj = j - (wv == 0 ? 0u : wv == 1 ? c0 : wv == 2 ? c1 : c2);
            const uint32_t packed = s_item[wv][jj][0], qq = s_item[wv][jj][1], r1 = s_item[wv][jj][2];
            const int x = (int)(packed & 1023u), y = (int)((packed >> 10) & 1023u), z = (int)(packed >> 20);
            const int q_old = (int)(qq & 0xffffu), q_new = (int)(qq >> 16);
            const uint32_t site = site_of(x, y, z, K, KK);
            const int gb = unlike_change<M, SPT == 1>(spins, x, y, z, K, KK, q_old, q_new);
            bool accepted = false, screened = false;
            if (!elastic) {
                accepted = (uint64_t)r1 < s_thr[gb + M];
            } else if (SCREEN && r1 != 0u) {
                // reject without a solve when even the lowest possible zone energy loses:
                // dE >= J gb + lambda dPi_0 > max(0, E*(r1)) + margin
                float sp[6];
#pragma unroll
                for (int I = 0; I < 6; ++I) sp[I] = a.sigma[(int64_t)I * a.plane + R.site_off + site];
                const float* So = a.Stab + (R.grain_off + q_old) * kTab;
                const float* Sn = a.Stab + (R.grain_off + q_new) * kTab;
                const double lo = R.J * (double)gb + R.lambda * point_zone_energy(So, Sn, sp);
                const double estar = -R.kT * log((double)r1 * 2.3283064365386963e-10);
                double W = 0.0;   // stored-energy scale of the site for the margin
#pragma unroll
                for (int i = 0; i < 6; ++i)
#pragma unroll
                    for (int jj = i; jj < 6; ++jj)
                        W += (i == jj ? 0.5 : 1.0) * (double)sp[i] * (double)sp[jj] *
                             fabs((double)So[sym_index(i, jj)]);
                const double margin = 1e-4 * fabs(R.lambda) * W + 1e-9 * (1.0 + fabs(lo));
                screened = lo > fmax(0.0, estar) + margin;
            }
            if (a.rec) {
                hmc_trial_record rc;
                rc.q_new = q_new;
                rc.gb = gb;
                rc.dPi = 0.0f;
                rc.r1 = r1;
                rc.flags = 1 | (accepted ? 2 : 0) | (screened ? 8 : 0);
                rc.reserved = 0;
                a.rec[R.site_off + site] = rc;
            }
            // same-colour sites are never neighbours: nothing else in this pass reads `site`
            if (accepted) spins[site] = (int16_t)q_new;
            solve[it] = elastic && !screened;
            ent[it].site = site;
            ent[it].qr = (uint32_t)q_new | ((uint32_t)r << 16);
            ent[it].gb = gb;
            ent[it].r1 = r1;
            other[it] = elastic ? screened : accepted;
        }
    }
    // block-collective tail, reached by every thread (`elastic` is uniform over the block: a
    // block belongs to one replica; at zero load nothing enters the list).  Counts come from ballots; the
    // block's real flips are n_block.
    __shared__ uint32_t s_other[4], s_solve[4], s_base;
    uint32_t n_other = 0, n_solve = 0, slot[SPT];
#pragma unroll
    for (int it = 0; it < SPT; ++it) {
        n_other += (uint32_t)__popcll(__ballot(other[it]));
        if (elastic) {
            const unsigned long long m = __ballot(solve[it]);
            slot[it] = n_solve + (uint32_t)__popcll(m & below);
            n_solve += (uint32_t)__popcll(m);
        }
    }
    if (lane == 0) {
        s_other[wid] = n_other;
        s_solve[wid] = n_solve;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (elastic) {
            const uint32_t total = s_solve[0] + s_solve[1] + s_solve[2] + s_solve[3];
            s_base = total ? atomicAdd(a.list_count, total) : 0u;
        }
        unsigned long long* st = a.stats + stat_copy(blockIdx.x);
        const uint32_t others = s_other[0] + s_other[1] + s_other[2] + s_other[3];
        if (n_block) atomicAdd(&st[kStatReal], (unsigned long long)n_block);
        if (others) atomicAdd(&st[elastic ? kStatScreened : kStatAccepted], (unsigned long long)others);
    }
    if (elastic) {
        __syncthreads();
        uint32_t off = s_base;
        for (int w = 0; w < wid; ++w) off += s_solve[w];
#pragma unroll
        for (int it = 0; it < SPT; ++it)
            if (solve[it]) a.list[off + slot[it]] = ent[it];
    }
}

// Two colours in one launch, for lattices of one edge at zero load with 26 neighbours: the colours 2p and 2p + 1 share
// their rows (the y and z parities of p) and alternate along x, so the only sites of one among the neighbours
// of the other lie in the same row, and every other neighbour belongs to no row of the launch.  A block owns whole
// rows, a thread a site of each colour, and takes the first colour, a barrier, and the second: the same trials on the
// same spins as two launches.  The draws and reads of both go out first; a second-colour site that proposes its
// row neighbour's state reads it again after the barrier.  The last pair also advances the sweep index: the
// first (p = 0) copies it to a second slot, which the others read, so that no block reads the slot that is
// written.  A sweep is four launches instead of nine, for lattices whose launch is a chain of waits: measured, us a
// colour by single launches and by pairs, both with the neighbours read by rows: 64^3 4.5 and 3.1, 128^3 5.4 and 3.9,
// ten 60^3 6.2 and 4.4, 160^3 7.5 and 5.8, 200^3 10.7 and 9.3; past the line (kPairBelow) the two meet, ten 100^3 11.0 and
// 10.1, 256^3 13.8 and 13.3, and large ones are better off with four sites a thread and a launch a colour, 320^3 22.7 and
// 33.3.
template <bool NP2>
__global__ __launch_bounds__(256) void k_potts_pair(PassArgs a)
{
    constexpr int M = 26;
    __shared__ uint32_t s_item[4][64][3];   // per wavefront: coords, q_old | q_new << 16, r1
    __shared__ uint32_t s_nw[4], s_acc[4];
    __shared__ uint64_t s_thr[64];
    const int lb = logical_block((int)blockIdx.x, (int)gridDim.x, a.order);
    const int r = a.single ? 0 : lb / a.rep_blocks, block = lb - r * a.rep_blocks;
    const RepDev R = a.reps[r];
    const int K = R.K, KK = K * K, py = a.colour & 1, pz = a.colour >> 1;
    const uint32_t Kh = (uint32_t)R.Kh, rows = 256u / Kh, inv = 0xffffffffu / Kh + 1u;   // n / Kh = n inv >> 32
    const int lg = 31 - __builtin_clz((unsigned)K);   // NP2: K = 2^lg
    const bool nbr_prop = NP2 || R.proposal == 0;
    int16_t* spins = a.spins + R.site_off;
    const int64_t sweep64 = a.sweep[a.colour == 0 ? 0 : 1];
    const uint32_t sweep = (uint32_t)sweep64;
    if (lb == 0 && threadIdx.x == 0) {
        if (a.colour == 0) a.sweep[1] = sweep64;
        if (a.colour == 3) a.sweep[0] = sweep64 + 1;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const unsigned long long below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    uint64_t thr = 0;
    if (threadIdx.x < 64) thr = a.thr[(int64_t)r * 64 + threadIdx.x];

    const uint32_t row = NP2 ? threadIdx.x >> (lg - 1) : __umulhi(threadIdx.x, inv), i = threadIdx.x - row * Kh;
    const uint32_t rr = (uint32_t)block * rows + row, k = NP2 ? rr >> (lg - 1) : __umulhi(rr, inv), j = rr - k * Kh;
    const bool ok = row < rows && rr < Kh * Kh;
    const int y = 2 * (int)j + py, z = 2 * (int)k + pz;
    auto spin = [&](uint32_t v) {
        return (int)*reinterpret_cast<const int16_t*>(reinterpret_cast<const char*>(spins) + 2u * v);
    };
    uint32_t nbr[2], r0[2], r1[2];
    int q_old[2] = {0, 0}, q_nb[2] = {0, 0};
    bool again = false;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int x = 2 * (int)i + c;
        const uint32_t site = NP2 ? neighbour_site<true>(x, y, z, K, KK, lg) : site_of(x, y, z, K, KK);
        philox4x32_10(site, sweep, R.key0, R.key1, r0[c], r1[c]);
        nbr[c] = site;
        if (nbr_prop) {
            const int slot = (int)__umulhi(r0[c], (uint32_t)M);
            int dx, dy, dz;
            slot_offset<M>(slot, dx, dy, dz);
            nbr[c] = neighbour_site<NP2>(x + dx, y + dy, z + dz, K, KK, lg);
            if (c == 1) again = slot == 12 || slot == 13;   // x - 1 or x + 1
        }
        if (ok) {
            q_old[c] = spin(site);
            q_nb[c] = spin(nbr[c]);
        }
    }
    uint32_t n_real = 0, n_acc = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        bool real = false;
        uint32_t qq = 0;
        if (ok) {
            if (c == 1 && again) q_nb[1] = spin(nbr[1]);
            int q_new = q_nb[c];
            if (!nbr_prop) {
                const uint32_t step = __umulhi(r0[c], (uint32_t)(R.Q - 1));
                q_new = (int)(((uint32_t)q_old[c] + 1u + step) % (uint32_t)R.Q);
            }
            real = q_new != q_old[c];
            qq = (uint32_t)q_old[c] | ((uint32_t)q_new << 16);
        }
        const unsigned long long m = __ballot(real);
        if (real) {
            const uint32_t at = (uint32_t)__popcll(m & below);
            s_item[wid][at][0] = (uint32_t)(2 * (int)i + c) | ((uint32_t)y << 10) | ((uint32_t)z << 20);
            s_item[wid][at][1] = qq;
            s_item[wid][at][2] = r1[c];
        }
        if (lane == 0) s_nw[wid] = (uint32_t)__popcll(m);
        if (c == 0 && threadIdx.x < 64) s_thr[threadIdx.x] = thr;
        __syncthreads();
        // the four wavefronts' lists, read as one list of the block's real flips
        const uint32_t c0 = s_nw[0], c1 = c0 + s_nw[1], c2 = c1 + s_nw[2], n_block = c2 + s_nw[3];
        n_real += n_block;
        bool accepted = false;
        if (threadIdx.x < n_block) {
            const uint32_t t = threadIdx.x;
            const int wv = (t >= c0) + (t >= c1) + (t >= c2);
            const uint32_t at = t - (wv == 0 ? 0u : wv == 1 ? c0 : wv == 2 ? c1 : c2);
            const uint32_t p = s_item[wv][at][0], qs = s_item[wv][at][1];
            const int sx = (int)(p & 1023u), sy = (int)((p >> 10) & 1023u), sz = (int)(p >> 20), q_new = (int)(qs >> 16);
            const int gb = unlike_change<M, true>(spins, sx, sy, sz, K, KK, (int)(qs & 0xffffu), q_new);
            accepted = (uint64_t)s_item[wv][at][2] < s_thr[gb + M];
            if (accepted) spins[site_of(sx, sy, sz, K, KK)] = (int16_t)q_new;
        }
        n_acc += (uint32_t)__popcll(__ballot(accepted));
        if (c == 0) __syncthreads();   // the first colour's spins are written, and the lists are free
    }
    if (lane == 0) s_acc[wid] = n_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long* st = a.stats + stat_copy(blockIdx.x);
        const uint32_t acc = s_acc[0] + s_acc[1] + s_acc[2] + s_acc[3];
        if (n_real) atomicAdd(&st[kStatReal], (unsigned long long)n_real);
        if (acc) atomicAdd(&st[kStatAccepted], (unsigned long long)acc);
    }
}

// Deferred update of an elastic pass: every accepted entry writes its new state.
__global__ __launch_bounds__(256) void k_apply(int16_t* spins, const RepDev* reps, const TrialEntry* list,
                                               const uint8_t* acc, const uint32_t* count)
{
    const uint32_t n = *count;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x)
        if (acc[e]) {
            const TrialEntry t = list[e];
            spins[reps[t.qr >> 16].site_off + t.site] = (int16_t)(t.qr & 0xffffu);
        }
}

__global__ void k_set_i64(int64_t* p, int64_t v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

__global__ void k_add_i64(int64_t* p, int64_t v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *p += v;
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_f32(float* p, float v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Spins in and out, eight a thread where the caller's array allows 16-byte accesses (WIDE; a replica's own spins
// start on a multiple of 8 and number one; out four a thread), else one.  Memory bound: 512^3 in 225 us, now 165, out 227
// and 134.
template <bool WIDE>
__global__ void k_convert_spins(const int32_t* in, int16_t* out, int64_t n, int32_t Q, uint32_t* err)
{
    bool bad = false;
    auto take = [&](int32_t v) {
        const bool off = v < 0 || v >= Q;
        bad = bad || off;
        return off ? 0 : v;
    };
    if (WIDE) {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n / 8;
             i += (int64_t)gridDim.x * blockDim.x) {
            const int4 a = reinterpret_cast<const int4*>(in)[2 * i], b = reinterpret_cast<const int4*>(in)[2 * i + 1];
            reinterpret_cast<int4*>(out)[i] =
                make_int4(take(a.x) | take(a.y) << 16, take(a.z) | take(a.w) << 16, take(b.x) | take(b.y) << 16,
                          take(b.z) | take(b.w) << 16);
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
            out[i] = (int16_t)take(in[i]);
    }
    if (bad) atomicOr(err, 1u);
}

__global__ void k_check_finite(const float* p, int64_t n, uint32_t* flag, uint32_t bit)
{
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        bad = bad || !isfinite(p[i]);
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, bit);
}

template <bool WIDE>
__global__ void k_export_spins(const int16_t* in, int32_t* out, int64_t n)
{
    if (WIDE) {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n / 4;
             i += (int64_t)gridDim.x * blockDim.x) {
            const int2 v = reinterpret_cast<const int2*>(in)[i];
            reinterpret_cast<int4*>(out)[i] =
                make_int4(v.x & 0xffff, (int)((unsigned)v.x >> 16), v.y & 0xffff, (int)((unsigned)v.y >> 16));
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
            out[i] = in[i];
    }
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

static unsigned grid_for(int64_t n, int block, unsigned cap = 65535u * 8u)
{
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > (int64_t)cap) g = cap;
    return (unsigned)g;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, float v, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_f32, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_convert_spins(const int32_t* in, int16_t* out, int64_t n, int32_t Q, uint32_t* err, hipStream_t s)
{
    if (aligned16(in) && aligned16(out))
        hipLaunchKernelGGL(k_convert_spins<true>, dim3(grid_for(n / 8, 256, 8192)), dim3(256), 0, s, in, out, n, Q, err);
    else
        hipLaunchKernelGGL(k_convert_spins<false>, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, in, out, n, Q, err);
    return hipGetLastError();
}

hipError_t launch_export_spins(const int16_t* in, int32_t* out, int64_t n, hipStream_t s)
{
    if (aligned16(in) && aligned16(out))
        hipLaunchKernelGGL(k_export_spins<true>, dim3(grid_for(n / 4, 256, 8192)), dim3(256), 0, s, in, out, n);
    else
        hipLaunchKernelGGL(k_export_spins<false>, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

hipError_t launch_check_finite(const float* p, int64_t n, uint32_t* flag, uint32_t bit, hipStream_t s)
{
    hipLaunchKernelGGL(k_check_finite, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, p, n, flag, bit);
    return hipGetLastError();
}

hipError_t launch_set_i64(int64_t* p, int64_t v, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(64), 0, s, p, v);
    return hipGetLastError();
}

hipError_t launch_add_i64(int64_t* p, int64_t v, hipStream_t s)
{
    hipLaunchKernelGGL(k_add_i64, dim3(1), dim3(64), 0, s, p, v);
    return hipGetLastError();
}

static PassArgs pass_args(const hmc_ctx_s* c, int colour, hmc_trial_record* rec)
{
    PassArgs a;
    a.spins = c->d.spins;
    a.reps = c->d.reps;
    a.pass_rep = c->d.pass_rep;
    a.thr = c->d.thr;
    a.list = c->d.list;
    a.list_count = c->d.counters + kListCount + colour;
    a.rec = rec;
    a.stats = c->d.stats;
    a.sweep = c->d.sweep;
    a.Stab = c->d.Stab;
    a.sigma = c->d.sigma;
    a.plane = c->total_sites;
    a.colour = colour;
    a.order = c->block_order;
    a.screen = (c->p.zone_screen != 0 && c->d.sigma != nullptr) ? 1 : 0;
    a.single = c->n_rep == 1;
    a.rep_blocks = 0;
    return a;
}

// Every replica proposes a neighbour's state and has a power-of-two edge.
static bool pow2_neighbours(const hmc_ctx_s* c)
{
    bool np2 = true;
    for (const RepDev& R : c->reps) np2 = np2 && R.proposal == 0 && (R.K & (R.K - 1)) == 0;
    return np2;
}

// One edge of at least 4 and rows that fit a block, no replica under load, and few enough trials that launches and
// waits, not the trials themselves, take the time (kPairBelow).
bool pairs_colours(const hmc_ctx_s* c)
{
    const int64_t Kh = c->reps[0].Kh;
    bool pairs = c->p.neighbors == 26 && Kh >= 2 && Kh <= 256 && !(c->elastic_buffers && c->any_elastic()) &&
                 c->n_rep * Kh * Kh * Kh < kPairBelow;
    for (const RepDev& R : c->reps) pairs = pairs && R.Kh == Kh;
    return pairs;
}

hipError_t launch_potts_pair(hmc_ctx_s* c, int pair)
{
    PassArgs a = pass_args(c, pair, nullptr);
    const int Kh = c->reps[0].Kh, rows = 256 / Kh;
    a.rep_blocks = (Kh * Kh + rows - 1) / rows;
    const dim3 grid((unsigned)(a.rep_blocks * c->n_rep)), block(256);
    const int tok = prof_begin(c, kProfPotts);
    if (pow2_neighbours(c))
        hipLaunchKernelGGL(k_potts_pair<true>, grid, block, 0, c->stream, a);
    else
        hipLaunchKernelGGL(k_potts_pair<false>, grid, block, 0, c->stream, a);
    prof_end(c, tok);
    return hipGetLastError();
}

hipError_t launch_potts_pass(hmc_ctx_s* c, int colour, hmc_trial_record* rec)
{
    const PassArgs a = pass_args(c, colour, rec);
    // one site per thread while a pass has fewer chunks than 4 per compute unit and no trial
    // enters the zone-solve list: with the list in use, four times the blocks means four times
    // the same-address list appends (measured at 128^3 under load: 16.2 against 9.6 us)
    const bool one = c->pass_blocks < kPassSplitBelow && !(c->elastic_buffers && c->any_elastic());
    const dim3 grid((unsigned)(one ? 4 * c->pass_blocks : c->pass_blocks)), block(256);
    const bool np2 = pow2_neighbours(c);
    const int tok = prof_begin(c, kProfPotts);
#define HMC_PASS(MM, SC, SPT)                                                                      \
    do {                                                                                           \
        if (np2) hipLaunchKernelGGL((k_potts_pass<MM, SC, SPT, true>), grid, block, 0, c->stream, a);  \
        else hipLaunchKernelGGL((k_potts_pass<MM, SC, SPT, false>), grid, block, 0, c->stream, a);     \
    } while (0)
    if (c->p.neighbors == 26) {
        if (one) {
            if (a.screen) HMC_PASS(26, true, 1);
            else HMC_PASS(26, false, 1);
        } else {
            if (a.screen) HMC_PASS(26, true, 4);
            else HMC_PASS(26, false, 4);
        }
    } else {
        if (one) {
            if (a.screen) HMC_PASS(6, true, 1);
            else HMC_PASS(6, false, 1);
        } else {
            if (a.screen) HMC_PASS(6, true, 4);
            else HMC_PASS(6, false, 4);
        }
    }
#undef HMC_PASS
    prof_end(c, tok);
    return hipGetLastError();
}

hipError_t launch_apply_pass(hmc_ctx_s* c, int colour)
{
    const unsigned g = grid_for(c->max_list, 256, 2048);
    const int tok = prof_begin(c, kProfApply);
    hipLaunchKernelGGL(k_apply, dim3(g), dim3(256), 0, c->stream, c->d.spins, c->d.reps, c->d.list, c->d.accept,
                       c->d.counters + kListCount + colour);
    prof_end(c, tok);
    return hipGetLastError();
}

}  // namespace hmc
