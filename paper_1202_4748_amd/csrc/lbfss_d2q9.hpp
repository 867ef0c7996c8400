// The paper's own model (Sec. III A): fluctuating non-ideal D2Q9 lattice
// Boltzmann with the Ginzburg-Landau thermodynamics in a modified equilibrium
// (the pressure tensor of Eq. (press-th) imposed on the equilibrium's second
// moment, Eq. (holdych-cond)), BGK relaxation (Eq. (lbe)) and noise with the
// local-sound-speed covariance of Eq. (lbnoise), drawn through its Cholesky
// factor.
//
// Layout: populations [9][L^2] (site = x + L y), stored as deviations from
// the rest state of density rho_c, whose equilibrium puts all mass at rest
// (p0(rho_c) = 0): d_0 = f_0 - rho_c, d_i = f_i otherwise.  Moments are
// taken in the weight-orthogonal basis 1, c_x, c_y, 3c^2 - 2, c_x^2 - c_y^2,
// c_x c_y, (3c^2 - 4) c_x, (3c^2 - 4) c_y, 9c^4 - 15c^2 + 2 and handled as
// deviations from the rest state's moments (rho_c, 0, 0, -2 rho_c, 0, 0, 0, 0,
// 2 rho_c).  Velocity order: 0 (0,0); 1 (1,0) 2 (-1,0) 3 (0,1) 4 (0,-1);
// 5 (1,1) 6 (-1,-1) 7 (1,-1) 8 (-1,1).
#pragma once

#include <algorithm>

#include "lbfss_fft.hpp"
#include "lbfss_fused.hpp"

namespace lbfss {

constexpr int Q2 = 9;

struct D2Desc {
    int32_t L, pad;
    float a, b, kappa, rho_c;
    float gamma;      // 1 - 1/tau
    float nu;         // (tau - 1/2) / 3
    float noise_amp;  // sqrt(3 kT (1/tau)(2 - 1/tau)); the noise scale is sqrt(rho) times this
    uint32_t key0, key1;
};

__host__ __device__ constexpr int c2x(int i) { return i == 1 || i == 5 || i == 7 ? 1 : (i == 2 || i == 6 || i == 8 ? -1 : 0); }
__host__ __device__ constexpr int c2y(int i) { return i == 3 || i == 5 || i == 8 ? 1 : (i == 4 || i == 6 || i == 7 ? -1 : 0); }
__host__ __device__ constexpr float w2(int i) { return i == 0 ? 4.0f / 9.0f : (i < 5 ? 1.0f / 9.0f : 1.0f / 36.0f); }

// e_a(c_i) and the norms N_a = sum_i w_i e_a^2
__host__ __device__ constexpr float e2(int a, int i) {
    const int cx = c2x(i), cy = c2y(i), cc = cx * cx + cy * cy;
    return a == 0 ? 1.0f
         : a == 1 ? (float)cx
         : a == 2 ? (float)cy
         : a == 3 ? (float)(3 * cc - 2)
         : a == 4 ? (float)(cx * cx - cy * cy)
         : a == 5 ? (float)(cx * cy)
         : a == 6 ? (float)((3 * cc - 4) * cx)
         : a == 7 ? (float)((3 * cc - 4) * cy)
                  : (float)(9 * cc * cc - 15 * cc + 2);
}
__host__ __device__ constexpr float n2(int a) {
    return a == 0 ? 1.0f : a <= 2 ? 1.0f / 3.0f : a == 3 ? 4.0f : a == 4 ? 4.0f / 9.0f : a == 5 ? 1.0f / 9.0f
         : a <= 7 ? 2.0f / 3.0f : 16.0f;
}

__device__ __forceinline__ int wrap2(int v, int L) { return v < 0 ? v + L : (v >= L ? v - L : v); }

// Pulled deviations of site (x, y): d_i(r - c_i).  The three source columns
// x - c_x and the three source rows y - c_y are wrapped once; each pull is
// then a 32-bit in-plane offset from the population's (uniform) base.
// MUL24: the rows' offsets by the full-rate 24-bit multiply (L <= 2048), for
// the halo of the one-step kernel's large launches (1000^2 16.4 -> 16.05 us a
// step, 400 x 100^2 81.9 -> 80.9); the kernels of several steps lose by it
// (512^2 5.62 -> 5.75).
template <bool MUL24 = false>
__device__ __forceinline__ void pull2(const float *__restrict__ pop, int L, int x, int y, float (&d)[Q2]) {
    const uint32_t N = (uint32_t)L * (uint32_t)L;
    const uint32_t col[3] = {(uint32_t)wrap2(x + 1, L), (uint32_t)x, (uint32_t)wrap2(x - 1, L)};  // c_x = -1, 0, 1
    auto mul = [](int v, int w) { return MUL24 ? (uint32_t)__umul24(v, w) : (uint32_t)v * (uint32_t)w; };
    const uint32_t row[3] = {mul(wrap2(y + 1, L), L), mul(y, L), mul(wrap2(y - 1, L), L)};  // c_y = -1, 0, 1
#pragma unroll
    for (int i = 0; i < Q2; ++i) d[i] = pop[(size_t)i * N + (col[c2x(i) + 1] + row[c2y(i) + 1])];
}

// The same pulls where y is wave-uniform: the three source rows are scalar
// bases and a lane adds one of three 32-bit column offsets, no 64-bit or
// quarter-rate integer arithmetic per lane.
__device__ __forceinline__ void pull2_row(const float *__restrict__ pop, int L, int x, int y, float (&d)[Q2]) {
    const uint32_t N = (uint32_t)L * (uint32_t)L;
    uint32_t col[3] = {4u * (uint32_t)wrap2(x + 1, L), 4u * (uint32_t)x, 4u * (uint32_t)wrap2(x - 1, L)};
    const uint32_t row[3] = {(uint32_t)wrap2(y + 1, L) * (uint32_t)L, (uint32_t)y * (uint32_t)L,
                             (uint32_t)wrap2(y - 1, L) * (uint32_t)L};
    asm("" : "+v"(col[0]), "+v"(col[1]), "+v"(col[2]));  // keeps the offsets in 32-bit registers
#pragma unroll
    for (int i = 0; i < Q2; ++i) d[i] = ldb(pop + (size_t)i * N + row[c2y(i) + 1], col[c2x(i) + 1]);
}

__device__ __forceinline__ float drho2(const float (&d)[Q2]) {
    return ((d[0] + (d[1] + d[2])) + (d[3] + d[4])) + ((d[5] + d[6]) + (d[7] + d[8]));
}

// Opposite velocities come in pairs (q, q + 1) for q = 1, 3, 5, 7, and each
// basis vector is even or odd under c -> -c (odd: a = 1, 2, 6, 7), so the
// transforms work on pair sums and differences (checked at compile time).
__host__ __device__ constexpr bool k2_odd(int a) { return a == 1 || a == 2 || a == 6 || a == 7; }
__host__ __device__ constexpr bool k2_pairs_ok() {
    for (int k = 0; k < 4; ++k) {
        const int q = 2 * k + 1, p = q + 1;
        if (c2x(p) != -c2x(q) || c2y(p) != -c2y(q) || w2(p) != w2(q)) return false;
        for (int a = 0; a < Q2; ++a)
            if (e2(a, p) != (k2_odd(a) ? -e2(a, q) : e2(a, q))) return false;
    }
    for (int a = 0; a < Q2; ++a)
        if (k2_odd(a) && e2(a, 0) != 0.0f) return false;
    return true;
}
static_assert(k2_pairs_ok(), "opposite velocity pairs and basis parities");

// The six collision normals of (site, step): Philox calls 0 and 1.
struct K2Normals {
    float g[6];
};
__device__ __forceinline__ K2Normals k2_normals(const D2Desc &D, uint32_t s, uint64_t t) {
    const Words4 w0 = philox4x32_10(s, (uint32_t)t, 0u, (uint32_t)(t >> 32), D.key0, D.key1);
    const Words4 w1 = philox4x32_10(s, (uint32_t)t, 1u, (uint32_t)(t >> 32), D.key0, D.key1);
    const float r0 = bm_radius(uniform01(w0.v[0])), a0 = uniform01(w0.v[1]);
    const float r1 = bm_radius(uniform01(w0.v[2])), a1 = uniform01(w0.v[3]);
    const float r2 = bm_radius(uniform01(w1.v[0])), a2 = uniform01(w1.v[1]);
    return K2Normals{{r0 * cos_rev(a0), r0 * sin_rev(a0), r1 * cos_rev(a1), r1 * sin_rev(a1), r2 * cos_rev(a2),
                      r2 * sin_rev(a2)}};
}

// The collision of one site: d holds its nine pulled deviations and
// receives the post-collision ones (stored unshifted: the next step pulls);
// at(dx, dy) is the density deviation of a neighbour (the same sum drho2 of
// its pulled values); normals() gives its collision normals.
// Moments, equilibrium, relaxation, noise, back-transform.  Returns false
// where rho or the noise covariance leaves its domain.
template <typename F, typename G>
__device__ __forceinline__ bool k2_collide_site(const D2Desc &D, float (&d)[Q2], F &&at, G &&normals) {
    // moment deviations, from the rest value and the pair sums (even
    // moments) or differences (odd moments)
    float ps[4], pd[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ps[k] = d[2 * k + 1] + d[2 * k + 2];
        pd[k] = d[2 * k + 1] - d[2 * k + 2];
    }
    float m[Q2];
#pragma unroll
    for (int a = 0; a < Q2; ++a) {
        float v = 0.0f;
        if (e2(a, 0) != 0.0f) v += e2(a, 0) * d[0];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (e2(a, 2 * k + 1) != 0.0f) v += e2(a, 2 * k + 1) * (k2_odd(a) ? pd[k] : ps[k]);
        m[a] = v;
    }
    const float dr = drho2(d);  // the same sum as the density array
    const float rho = D.rho_c + dr;
    // isotropic stencils on the densities of the neighbours
    float gx = 0.0f, gy = 0.0f, lap = 0.0f;
#pragma unroll
    for (int i = 1; i < Q2; ++i) {
        const float v = at(c2x(i), c2y(i));
        gx += 3.0f * w2(i) * (float)c2x(i) * v;
        gy += 3.0f * w2(i) * (float)c2y(i) * v;
        lap += 6.0f * w2(i) * (v - dr);
    }
    // thermodynamics of the Landau potential in d = rho - rho_c
    const float d2 = dr * dr;
    const float p0 = rho * (D.a * dr + D.b * d2 * dr) - (0.5f * D.a * d2 + 0.25f * D.b * d2 * d2);
    const float cs2 = rho * (D.a + 3.0f * D.b * d2);
    // equilibrium moments (deviations from the rest state)
    const float inv_rho = __builtin_amdgcn_rcpf(rho);  // hardware reciprocal, 1 ulp
    const float ux = m[1] * inv_rho, uy = m[2] * inv_rho;
    const float g2 = gx * gx + gy * gy, ug = ux * gx + uy * gy;
    const float S = p0 - D.kappa * rho * lap;
    const float iso = S - 0.5f * D.kappa * g2;
    const float Pxx = iso + D.kappa * gx * gx + rho * ux * ux + D.nu * (2.0f * ux * gx + ug);
    const float Pyy = iso + D.kappa * gy * gy + rho * uy * uy + D.nu * (2.0f * uy * gy + ug);
    const float Pxy = D.kappa * gx * gy + rho * ux * uy + D.nu * (ux * gy + uy * gx);
    float meq[Q2];
    meq[3] = 3.0f * (Pxx + Pyy) - 2.0f * dr;
    meq[4] = Pxx - Pyy;
    meq[5] = Pxy;
    meq[6] = 0.0f;
    meq[7] = 0.0f;
    meq[8] = 2.0f * dr - 6.0f * S - 3.0f * D.kappa * g2;
#pragma unroll
    for (int a = 3; a < Q2; ++a) m[a] = meq[a] + D.gamma * (m[a] - meq[a]);
    // noise, Eq. (lbnoise), through the Cholesky factor of its c_s^2 block
    bool bad = !(rho > 0.0f);
    if (D.noise_amp > 0.0f) {
        const float A = 4.0f * (2.0f - 3.0f * cs2), C = 12.0f * (cs2 - 1.0f / 3.0f),
                    B = 16.0f * (1.25f - 0.75f * cs2);
        // the factor scales normals only: hardware square roots and
        // reciprocal (1 ulp) serve it
        const float L33 = __builtin_amdgcn_sqrtf(A), L83 = C * __builtin_amdgcn_rcpf(L33), R = B - L83 * L83;
        bad |= !(A > 0.0f) || !(R > 0.0f);
        const float L88 = __builtin_amdgcn_sqrtf(R);
        const float sig = D.noise_amp * __builtin_amdgcn_sqrtf(rho);
        const K2Normals n = normals();
        const float g0 = n.g[0], g1 = n.g[1], g2n = n.g[2], g3 = n.g[3], g4 = n.g[4], g5 = n.g[5];
        m[3] += sig * L33 * g0;
        m[4] += sig * (2.0f / 3.0f) * g1;
        m[5] += sig * (1.0f / 3.0f) * g2n;
        m[6] += sig * 0.816496580927726f * g3;  // sqrt(2/3)
        m[7] += sig * 0.816496580927726f * g4;
        m[8] += sig * (L83 * g0 + L88 * g5);
    }
    // back to populations: the rest one, then an even and an odd part per pair
    float mn[Q2];
#pragma unroll
    for (int a = 0; a < Q2; ++a) mn[a] = m[a] * (1.0f / n2(a));
    {
        float v = 0.0f;
#pragma unroll
        for (int a = 0; a < Q2; ++a)
            if (e2(a, 0) != 0.0f) v += e2(a, 0) * mn[a];
        d[0] = w2(0) * v;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int q = 2 * k + 1;
        float ev = 0.0f, od = 0.0f;
#pragma unroll
        for (int a = 0; a < Q2; ++a) {
            if (e2(a, q) == 0.0f) continue;
            if (k2_odd(a)) od += e2(a, q) * mn[a];
            else ev += e2(a, q) * mn[a];
        }
        d[q] = w2(q) * (ev + od);
        d[q + 1] = w2(q) * (ev - od);
    }
    return !bad;
}

// One step on a K2TX x K2TY tile per workgroup (tiles at the edges of the
// lattice are partial, so any L works): every site pulls its nine values,
// the densities of the tile and of a one-site halo (pulled by the first
// threads) go to LDS, and after one barrier each site collides with the
// stencils read there.  The densities are drho2 of the same pulled values
// wherever they are formed, so the result does not depend on the tiling.
// Tiles are numbered x fastest and dealt to the XCDs in contiguous runs
// (xcd_tile), so the halo pulls of a tile find its neighbours' rows in the
// same L2.  64 x 4 tiles: 3% faster than 32 x 8 at 2048^2, 16 x 16 12% slower.
// A batch of replicas (one L, own parameters and seeds) is one launch: the
// tiles of replica r follow those of replica r - 1, each replica's
// populations a [9][L^2] block after the previous one's.
// BATCH = false (one replica, the latency-bound small lattices): the
// descriptor comes with the launch, no replica arithmetic, no descriptor load.
// ROWS: a wave is one row of the tile, so its pulls and stores are scalar row
// bases plus 32-bit lane offsets (64 x 256^2: 70.2 -> 68.3 us a step, 48 x 256^2
// 43.2 -> 41.2, 1800^2 44.1 -> 43.0, 400 x 100^2 85.9 -> 80.9), for launches
// with work enough to hide the scalar chain that forms them (k2_row_bases).
// NT: stores that do not stay in the caches (k2_store_nt).
constexpr int K2TX = 64, K2TY = 4;
// Where the two copies of a batch exceed the 256 MB cache behind the L2s, no
// line that is written is read again before it is evicted, and writing around
// the caches leaves them to the reads: 64 x 256^2 69.7 -> 65.9 us, 128 x 256^2
// 131.9 -> 127.4, 16 x 512^2 71.3 -> 66.4, 4 x 1024^2 72.7 -> 68.6.  Below that
// size it costs (56 x 256^2 47.4 -> 59.4), as it does for rows that are not
// whole 128-byte lines (400 x 100^2 79.1 -> 84.2) and for 2048^2 (69.7 -> 70.4).
inline bool k2_store_nt(int L, int nrep) {
    return L % 32 == 0 && L <= 1024 && nrep > 1 && (int64_t)nrep * L * L * (2 * Q2 * 4) > ((int64_t)256 << 20);
}
// The scalar row bases are a chain ahead of the first load, 0.3 us of a launch
// whose workgroups all start at once: 7 x 256^2 8.32 -> 8.84 us, 20 x 128^2
// 6.80 -> 7.24, 40 x 100^2 8.50 -> 8.74, 14 x 200^2 11.5 -> 11.7, 768^2 10.9 ->
// 11.2, 850^2 12.8 -> 13.1 with them; 9 x 256^2 11.3 -> 11.1, 36 x 128^2 11.2 ->
// 10.95, 16 x 200^2 12.9 -> 12.6, 900^2 14.4 -> 14.3, 1200^2 21.9 -> 21.5.  So
// from nine full tiles a CU in a batch, twelve of one lattice.
inline bool k2_row_bases(int L, int nrep) {
    return (int64_t)nrep * L * L >= (int64_t)(nrep > 1 ? 9 : 12) * 256 * K2TX * K2TY;
}
template <bool BATCH, bool ROWS, bool NT>
__global__ void __launch_bounds__(K2TX * K2TY)
k2_step_tiled(D2Desc D0, const D2Desc *__restrict__ descs, int tiles_per_rep, const float *__restrict__ pop_all,
              float *__restrict__ pop_out_all, uint64_t t, int *__restrict__ err) {
    constexpr int EX = K2TX + 2;
    static_assert(2 * (K2TX + 2) + 2 * K2TY <= K2TX * K2TY, "one halo site per thread");
    __shared__ float s_rho[EX * (K2TY + 2)];
    const int gtile = xcd_tile(blockIdx.x, gridDim.x);
    const int rep = BATCH ? gtile / tiles_per_rep : 0, tile = gtile - rep * tiles_per_rep;
    const D2Desc D = BATCH ? descs[rep] : D0;
    const int L = D.L;
    const int64_t N = (int64_t)L * L;
    const float *pop = pop_all + (int64_t)rep * Q2 * N;
    float *pop_out = pop_out_all + (int64_t)rep * Q2 * N;
    const int ntx = (L + K2TX - 1) / K2TX;
    const int x0 = (tile % ntx) * K2TX, y0 = (tile / ntx) * K2TY;
    const int nx = min(K2TX, L - x0), ny = min(K2TY, L - y0);
    static_assert(K2TX == 64, "a wave per row");
    const int tid = threadIdx.x, ix = tid % K2TX;
    const int iy = ROWS ? __builtin_amdgcn_readfirstlane(tid / K2TX) : tid / K2TX;
    const bool inner = ix < nx && iy < ny;
    const int r_in = (iy + 1) * EX + ix + 1;
    float d[Q2];
    if (inner) {
        if constexpr (ROWS) pull2_row(pop, L, x0 + ix, y0 + iy, d);
        else pull2(pop, L, x0 + ix, y0 + iy, d);
        s_rho[r_in] = drho2(d);
    }
    // halo: the rows above and below the tile, then the columns beside it
    const int ew = nx + 2;
    if (tid < 2 * ew + 2 * ny) {
        int hx = 0, hy = 0;
        if (tid < ew) {
            hx = tid;
        } else if (tid < 2 * ew) {
            hy = ny + 1;
            hx = tid - ew;
        } else {
            const int h = tid - 2 * ew;
            hy = 1 + (h >> 1);
            hx = (h & 1) ? nx + 1 : 0;
        }
        float h[Q2];
        pull2<ROWS>(pop, L, wrap2(x0 - 1 + hx, L), wrap2(y0 - 1 + hy, L), h);
        s_rho[hy * EX + hx] = drho2(h);
    }
    __syncthreads();
    if (!inner) return;
    const uint32_t s = (uint32_t)(x0 + ix) + (uint32_t)L * (uint32_t)(y0 + iy);
    const bool ok = k2_collide_site(
        D, d, [&](int dx, int dy) { return s_rho[r_in + dy * EX + dx]; }, [&] { return k2_normals(D, s, t); });
    if constexpr (ROWS) {
        float *out = pop_out + (uint32_t)(y0 + iy) * (uint32_t)L;
        uint32_t col = 4u * (uint32_t)(x0 + ix);
        asm("" : "+v"(col));
#pragma unroll
        for (int i = 0; i < Q2; ++i) {
            if constexpr (NT) stb(out + (size_t)i * N, col, d[i]);
            else *(float *)((char *)(out + (size_t)i * N) + col) = d[i];
        }
    } else {
        static_assert(!NT, "such launches stay in the caches");
#pragma unroll
        for (int i = 0; i < Q2; ++i) pop_out[i * N + s] = d[i];
    }
    if (!ok) *err = 1;
}

// K steps in one launch, for lattices that leave most of the chip idle: a
// step on its own is then one chain of launch, loads and collision, 4.0 us at
// 256^2 (256 workgroups, one wave per SIMD) of which the arithmetic is a
// quarter.  A workgroup owns a 16 x 16 tile; step k collides the tile with a
// rim of 2 (K - 1 - k) sites around it, whose neighbours' post-collision
// populations of the step before lie in LDS (a step needs the pulls, one site
// away, of the sites it collides and of their neighbours, for the density).
// The first step pulls from memory, the last stores the tile.  Rims are
// computed by every workgroup that needs them, from the same values in the
// same order, so the result does not depend on K.  Positions wrap, so a tile
// may stick out of the lattice or be wider than it.  The rims cost 1.6 times
// the collisions at K = 3; what is left at 256^2 is the chain of three
// collisions, about 1.5 us each, and one launch: 4.0 -> 2.39 us a step.
constexpr int K2F_T = 16;
template <int K>
struct K2Fused {
    static constexpr int C0 = K2F_T + 4 * (K - 1);  // edge of the first step's collided square
    static constexpr int E0 = C0 + 2;               // edge of its density square
    static constexpr int NT = (E0 * E0 + 63) / 64 * 64;
};

// v in [-2 K, L + 16 + 2 K) to [0, L); rL = 1 / L to an ulp
__device__ __forceinline__ int k2_wrap(int v, int L, float rL) {
    return v - L * (int)floorf(((float)v + 0.5f) * rL);
}

template <int K>
__global__ void __launch_bounds__(K2Fused<K>::NT)
k2_steps_fused(const D2Desc *__restrict__ descs, int tiles_per_rep, const float *__restrict__ pop_all,
               float *__restrict__ pop_out_all, uint64_t t, int *__restrict__ err) {
    constexpr int C0 = K2Fused<K>::C0, E0 = K2Fused<K>::E0;
    __shared__ float s_pop[Q2][C0 * C0];
    __shared__ float s_rho[E0 * E0];
    const int gtile = xcd_tile(blockIdx.x, gridDim.x);
    const int rep = gtile / tiles_per_rep, tile = gtile - rep * tiles_per_rep;
    const D2Desc D = descs[rep];
    const int L = D.L, ntx = (L + K2F_T - 1) / K2F_T, x0 = (tile % ntx) * K2F_T, y0 = (tile / ntx) * K2F_T;
    const int64_t N = (int64_t)L * L;
    const float *pop = pop_all + (int64_t)rep * Q2 * N;
    float *pop_out = pop_out_all + (int64_t)rep * Q2 * N;
    const float rL = __builtin_amdgcn_rcpf((float)L);
    const int tid = threadIdx.x;
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // this thread's site of the step's density square (edge E), one site
        // wider on each side than the square collided (edge C)
        const int C = K2F_T + 4 * (K - 1 - k), E = C + 2, rim = 2 * (K - 1 - k) + 1;
        const int ey = tid / E, ex = tid - ey * E;
        const bool on = ey < E, in = on && ex >= 1 && ex <= C && ey >= 1 && ey <= C;
        const int x = k2_wrap(x0 - rim + ex, L, rL), y = k2_wrap(y0 - rim + ey, L, rL);
        const uint32_t site = (uint32_t)(x + L * y);
        float d[Q2];
        K2Normals n;
        if (k == 0) {
            if (on) pull2(pop, L, x, y, d);
            n = k2_normals(D, site, t);  // while the pulls are on their way
        } else if (on) {
            const int c = (ey + 1) * (C + 4) + ex + 1;  // the site in the square the step before collided
#pragma unroll
            for (int i = 0; i < Q2; ++i) d[i] = s_pop[i][c - c2y(i) * (C + 4) - c2x(i)];
        }
        if (on) s_rho[tid] = drho2(d);
        __syncthreads();
        if (in) {
            const float *r = s_rho + tid;
            ok &= k2_collide_site(
                D, d, [&](int dx, int dy) { return r[dy * E + dx]; },
                [&] { return k == 0 ? n : k2_normals(D, site, t + (uint64_t)k); });
            if (k + 1 < K) {
                const int c = (ey - 1) * C + ex - 1;
#pragma unroll
                for (int i = 0; i < Q2; ++i) s_pop[i][c] = d[i];
            } else if (x0 + ex - 1 < L && y0 + ey - 1 < L) {
#pragma unroll
                for (int i = 0; i < Q2; ++i) pop_out[i * N + site] = d[i];
            }
        }
        if (k + 1 < K) __syncthreads();
    }
    if (!ok) *err = 1;
}

// Initial state: rho = rho_c + sigma0 g (generator domain 1, call 0), u = 0,
// the equilibrium of that density (gradients of the density array).
__global__ void __launch_bounds__(kBlock)
k2_init_density(D2Desc D, float sigma0, float *__restrict__ drho) {
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= (int64_t)D.L * D.L) return;
    const Words4 w = philox4x32_10((uint32_t)s, 0u, 1u << 16, 0u, D.key0, D.key1);
    drho[s] = sigma0 * (bm_radius(uniform01(w.v[0])) * cos_rev(uniform01(w.v[1])));
}

__global__ void __launch_bounds__(kBlock)
k2_init_populations(D2Desc D, const float *__restrict__ drho, float *__restrict__ pop) {
    const int L = D.L;
    const int64_t N = (int64_t)L * L;
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= N) return;
    const int x = (int)(s % L), y = (int)(s / L);
    const float dr = drho[s], rho = D.rho_c + dr;
    float gx = 0.0f, gy = 0.0f, lap = 0.0f;
#pragma unroll
    for (int i = 1; i < Q2; ++i) {
        const float v = drho[wrap2(x + c2x(i), L) + (int64_t)L * wrap2(y + c2y(i), L)];
        gx += 3.0f * w2(i) * (float)c2x(i) * v;
        gy += 3.0f * w2(i) * (float)c2y(i) * v;
        lap += 6.0f * w2(i) * (v - dr);
    }
    const float d2 = dr * dr;
    const float p0 = rho * (D.a * dr + D.b * d2 * dr) - (0.5f * D.a * d2 + 0.25f * D.b * d2 * d2);
    const float g2 = gx * gx + gy * gy;
    const float S = p0 - D.kappa * rho * lap, iso = S - 0.5f * D.kappa * g2;
    float m[Q2] = {dr, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    const float Pxx = iso + D.kappa * gx * gx, Pyy = iso + D.kappa * gy * gy;
    m[3] = 3.0f * (Pxx + Pyy) - 2.0f * dr;
    m[4] = Pxx - Pyy;
    m[5] = D.kappa * gx * gy;
    m[8] = 2.0f * dr - 6.0f * S - 3.0f * D.kappa * g2;
    // the state is read by pulling, f_i(r) = buffer_i(r - c_i)
#pragma unroll
    for (int i = 0; i < Q2; ++i) {
        float v = 0.0f;
#pragma unroll
        for (int a = 0; a < Q2; ++a)
            if (e2(a, i) != 0.0f) v += e2(a, i) * (m[a] * (1.0f / n2(a)));
        pop[i * N + wrap2(x - c2x(i), L) + (int64_t)L * wrap2(y - c2y(i), L)] = w2(i) * v;
    }
}

// Export: rho, j and the populations f_i in FP64 of the state at step t
// (post-streaming: f_i(r) = buffer_i(r - c_i)).
__global__ void __launch_bounds__(kBlock)
k2_export(D2Desc D, const float *__restrict__ pop, double *__restrict__ rho, double *__restrict__ j,
          double *__restrict__ f) {
    const int L = D.L;
    const int64_t N = (int64_t)L * L;
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= N) return;
    const int x = (int)(s % L), y = (int)(s / L);
    double r = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 0; i < Q2; ++i) {
        const int xs = wrap2(x - c2x(i), L), ys = wrap2(y - c2y(i), L);
        const double v = (double)pop[i * N + xs + (int64_t)L * ys] + (i == 0 ? (double)D.rho_c : 0.0);
        r += v;
        jx += c2x(i) * v;
        jy += c2y(i) * v;
        if (f) f[i * N + s] = v;
    }
    if (rho) rho[s] = r;
    if (j) {
        j[s] = jx;
        j[N + s] = jy;
    }
}

// Import: the state f_i(r) at step t into the buffer, buffer_i(r - c_i) = f_i(r).
__global__ void __launch_bounds__(kBlock)
k2_import(D2Desc D, const double *__restrict__ f, float *__restrict__ pop) {
    const int L = D.L;
    const int64_t N = (int64_t)L * L;
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= N) return;
    const int x = (int)(s % L), y = (int)(s / L);
#pragma unroll
    for (int i = 0; i < Q2; ++i) {
        const int xs = wrap2(x - c2x(i), L), ys = wrap2(y - c2y(i), L);
        pop[i * N + xs + (int64_t)L * ys] = (float)(f[i * N + s] - (i == 0 ? (double)D.rho_c : 0.0));
    }
}

// ---------------------------------------------------------------------------
// Sampling: the spectra of density and momentum.  The fields are real, so
// their transforms are kept for kx = 0..L/2 only (Lh columns); the other modes
// are mirrored when the spectra are read.
//   k2_spec_rows   a few rows a workgroup: density and momentum summed straight
//                  from the pulled populations, the row transforms (even L: the
//                  even and odd sites of a row as the real and imaginary part
//                  of a line of L/2 points), X[3][y][kx]
//   k2_spec_cols   a few columns a workgroup: the column transforms, the
//                  spectra added to the accumulators [5][kx][ky]
// Per sample, against transforms of all columns (powers of two) or direct ones
// (other L): 64 replicas of 256^2 400 -> 196 us, 2048^2 497 -> 300, 256^2
// 23 -> 16, 376^2 310 -> 37, 32 replicas of 200^2 1190 -> 57.  Large launches
// are bound by LDS round trips and by memory in about equal parts (2048^2:
// 521 MB a sample at 1.7 TB/s), one lattice of 256^2 by the chain of passes.
// ---------------------------------------------------------------------------
constexpr int kTwLds = 512;  // longest twiddle table copied to LDS

// Accumulators of one replica: [5][Lh][L] spectra S, J_x, J_y, J_par, J_perp
// of mode (kx, ky), then [2][Lh] J_par, J_perp of the modes (-kx, L/2) of even
// L: the direction of k folds L/2 to +L/2 on both sides, so they are not the
// mirror images of (kx, L/2).
__host__ __device__ constexpr int64_t k2_acc_len(int L) { return (int64_t)5 * (L / 2 + 1) * L + 2 * (L / 2 + 1); }

template <int NT, int U>
__global__ void __launch_bounds__(NT)
k2_spec_rows(int L, FftPlan p, int rows, const float *__restrict__ pop_all, const double2 *__restrict__ tw,
             double2 *__restrict__ X_all) {
    __shared__ double2 S[U * NT + U * NT / 8 + 64];
    __shared__ double2 s_tw[NT <= kTwLds ? kTwLds : 1];
    const int64_t N = (int64_t)L * L;
    const int Lh = L / 2 + 1, n = p.n, stride = fft_stride(n), y0 = blockIdx.x * rows;
    const float *pop = pop_all + (int64_t)blockIdx.y * Q2 * N;
    double2 *X = X_all + (int64_t)blockIdx.y * 3 * L * Lh;
    const bool even = L % 2 == 0, in_lds = NT <= kTwLds && L <= kTwLds;
    if (in_lds)
        for (int k = threadIdx.x; k < L; k += NT) s_tw[k] = tw[k];
    const float r_L = 1.0f / (float)L, r_Lh = 1.0f / (float)Lh;
    for (int i = threadIdx.x; i < rows * L; i += NT) {
        const int row = div_small(i, r_L), x = i - row * L, y = y0 + row;
        double v[3] = {0.0, 0.0, 0.0};
        if (y < L) {
            float d[Q2];
            pull2(pop, L, x, y, d);
#pragma unroll
            for (int q = 0; q < Q2; ++q) {
                v[0] += (double)d[q];
                v[1] += c2x(q) * (double)d[q];
                v[2] += c2y(q) * (double)d[q];
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double2 *ln = S + (3 * row + c) * stride;
            if (!even) ln[fft_slot(x)] = make_double2(v[c], 0.0);
            else if (x & 1) ln[fft_slot(x >> 1)].y = v[c];
            else ln[fft_slot(x >> 1)].x = v[c];
        }
    }
    __syncthreads();
    const double2 *t = in_lds ? s_tw : tw;
    fft_lines<NT, U>(S, 3 * rows, p, t);
    for (int i = threadIdx.x; i < 3 * rows * Lh; i += NT) {
        const int line = div_small(i, r_Lh), k = i - line * Lh, row = line / 3, c = line - 3 * row, y = y0 + row;
        if (y >= L) continue;
        const double2 *ln = S + line * stride;
        double2 X1;
        if (even) {  // X_k = E_k + w^k O_k, E and O the transforms of the even and odd sites
            const double2 a = ln[fft_slot(k == n ? 0 : k)], b = ln[fft_slot(k == 0 ? 0 : n - k)];
            const double2 E = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
            const double2 O = make_double2(0.5 * (a.y + b.y), 0.5 * (b.x - a.x));
            X1 = cadd(E, cmul(O, t[k]));
        } else {
            X1 = ln[fft_slot(k)];
        }
        X[((int64_t)c * L + y) * Lh + k] = X1;
    }
}

// The spectra of mode (kx, ky) from its transformed channels (density, jx,
// jy): |rho_k|^2, |jx_k|^2, |jy_k|^2 and the projections of j_k on k
// (longitudinal) and across it (transverse), each divided by N; k = 0 has no
// direction (0).
__device__ __forceinline__ void k2_spec_add(double *__restrict__ acc, int L, int ky, int kx, double2 r, double2 jx,
                                            double2 jy) {
    const int Lh = L / 2 + 1;
    const int64_t A = (int64_t)Lh * L, o = (int64_t)kx * L + ky;
    const double inv = 1.0 / ((double)L * (double)L);
    const int mx = kx, my = ky <= L / 2 ? ky : ky - L;
    const double kn = sqrt((double)mx * mx + (double)my * my);
    const double hx = kn > 0 ? mx / kn : 0.0, hy = kn > 0 ? my / kn : 0.0;
    auto norm = [&](double re, double im) { return (re * re + im * im) * inv; };
    acc[o] += norm(r.x, r.y);
    acc[A + o] += norm(jx.x, jx.y);
    acc[2 * A + o] += norm(jy.x, jy.y);
    acc[3 * A + o] += norm(hx * jx.x + hy * jy.x, hx * jx.y + hy * jy.y);
    acc[4 * A + o] += norm(-hy * jx.x + hx * jy.x, -hy * jx.y + hx * jy.y);
    if (2 * ky == L) {  // (-kx, L/2): its j is the conjugate of j at (kx, -L/2) = (kx, L/2)
        acc[5 * A + kx] += norm(-hx * jx.x + hy * jy.x, -hx * jx.y + hy * jy.y);
        acc[5 * A + Lh + kx] += norm(hy * jx.x + hx * jy.x, hy * jx.y + hx * jy.y);
    }
}

// PAR: the three channels of the columns side by side (3 cols L <= U NT), the
// shorter chain, for launches that leave CUs idle; else one after the other,
// the transformed values waiting in registers (cols L <= U NT): more adjacent
// columns a workgroup, so each row is read as cols consecutive values.
template <int NT, int U, bool PAR>
__global__ void __launch_bounds__(NT)
k2_spec_cols(int L, FftPlan p, int cols, const double2 *__restrict__ X_all, const double2 *__restrict__ tw,
             double *__restrict__ acc_all) {
    __shared__ double2 S[U * NT + U * NT / 8 + 64];
    __shared__ double2 s_tw[NT <= kTwLds ? kTwLds : 1];
    const int Lh = L / 2 + 1, stride = fft_stride(L), kx0 = blockIdx.x * cols;
    const double2 *X = X_all + (int64_t)blockIdx.y * 3 * L * Lh;
    double *acc = acc_all + (int64_t)blockIdx.y * k2_acc_len(L);
    const bool in_lds = NT <= kTwLds && L <= kTwLds;
    if (in_lds)
        for (int k = threadIdx.x; k < L; k += NT) s_tw[k] = tw[k];
    const double2 *t = in_lds ? s_tw : tw;
    const float r_c = 1.0f / (float)cols, r_L = 1.0f / (float)L;
    auto load = [&](int c0, int nc) {  // channels c0 .. c0 + nc - 1
        for (int i = threadIdx.x; i < nc * L * cols; i += NT) {
            const int cy = div_small(i, r_c), c = i - cy * cols, ch = div_small(cy, r_L), y = cy - ch * L;
            S[(ch * cols + c) * stride + fft_slot(y)] =
                kx0 + c < Lh ? X[((int64_t)(c0 + ch) * L + y) * Lh + kx0 + c] : make_double2(0.0, 0.0);
        }
        __syncthreads();
    };
    if constexpr (PAR) {
        load(0, 3);
        fft_lines<NT, U>(S, 3 * cols, p, t);
        for (int i = threadIdx.x; i < cols * L; i += NT) {
            const int c = div_small(i, r_L), ky = i - c * L, e = fft_slot(ky);
            if (kx0 + c < Lh)
                k2_spec_add(acc, L, ky, kx0 + c, S[c * stride + e], S[(cols + c) * stride + e],
                            S[(2 * cols + c) * stride + e]);
        }
    } else {
        double2 v[3][U];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            load(ch, 1);
            fft_lines<NT, U>(S, cols, p, t);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = threadIdx.x + u * NT, c = div_small(i, r_L);
                if (i < cols * L) v[ch][u] = S[c * stride + fft_slot(i - c * L)];
            }
            __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * NT, c = div_small(i, r_L), ky = i - c * L;
            if (i < cols * L && kx0 + c < Lh) k2_spec_add(acc, L, ky, kx0 + c, v[0][u], v[1][u], v[2][u]);
        }
    }
}

// The spectra [5][ky][kx] of all modes from the accumulators of one replica:
// modes with kx > L/2 from their mirror images.  32 x 32 modes a workgroup,
// transposed through LDS.
__global__ void __launch_bounds__(kBlock)
k2_spec_full(int L, const double *__restrict__ acc, double *__restrict__ out) {
    __shared__ double T[32][33];
    const int Lh = L / 2 + 1, c = blockIdx.z, a = threadIdx.x & 31, b = threadIdx.x >> 5;
    const int x0 = blockIdx.x * 32, y0 = blockIdx.y * 32;
    const int64_t A = (int64_t)Lh * L;
    for (int k = b; k < 32; k += kBlock / 32) {
        const int kx = x0 + k, ky = y0 + a;
        if (kx >= L || ky >= L) continue;
        int64_t src;
        if (kx < Lh) src = c * A + (int64_t)kx * L + ky;
        else if (c >= 3 && 2 * ky == L) src = 5 * A + (c - 3) * Lh + (L - kx);
        else src = c * A + (int64_t)(L - kx) * L + (ky == 0 ? 0 : L - ky);
        T[k][a] = acc[src];
    }
    __syncthreads();
    for (int k = b; k < 32; k += kBlock / 32) {
        const int kx = x0 + a, ky = y0 + k;
        if (kx < L && ky < L) out[(int64_t)c * L * L + (int64_t)ky * L + kx] = T[a][k];
    }
}

// The launches of a sample of R replicas: as many rows or columns a workgroup
// as its 4 points a thread hold, 256 threads where the lines are short.
struct K2SpecPlan {
    FftPlan row, col;
    int row_nt, rows, col_nt, cols;
    bool par;
};

inline K2SpecPlan k2_spec_plan(int L, int R) {
    K2SpecPlan s{};
    s.row = L % 2 == 0 ? fft_plan(L / 2, 2) : fft_plan(L, 1);
    s.col = fft_plan(L, 1);
    const int n = s.row.n, Lh = L / 2 + 1;
    s.row_nt = 3 * n <= 1024 ? 256 : (3 * n <= 2048 ? 512 : 1024);
    s.rows = std::max(1, std::min(4 * s.row_nt / (3 * n), 8));
    while (s.rows > 1 && (int64_t)R * ((L + s.rows - 1) / s.rows) < 256) --s.rows;
    // three channels side by side while the columns would not fill the chip
    s.par = 3 * L <= 4096 && (int64_t)R * Lh <= 1024;
    s.col_nt = s.par ? (3 * L <= 1024 ? 256 : (3 * L <= 2048 ? 512 : 1024)) : (L <= 256 ? 256 : (L <= 512 ? 512 : 1024));
    s.cols = s.par ? 1 : std::max(1, std::min(4 * s.col_nt / L, 8));
    return s;
}

inline void launch_k2_spectra(const K2SpecPlan &s, int L, int R, const float *pop, const double2 *tw, double2 *X,
                              double *acc, hipStream_t stream) {
    const dim3 gr((unsigned)((L + s.rows - 1) / s.rows), (unsigned)R);
    const dim3 gc((unsigned)((L / 2 + s.cols) / s.cols), (unsigned)R);
#define LBFSS_ROWS(NT_, U_) \
    hipLaunchKernelGGL((k2_spec_rows<NT_, U_>), gr, dim3(NT_), 0, stream, L, s.row, s.rows, pop, tw, X)
#define LBFSS_COLS(NT_, PAR_)                                                                             \
    hipLaunchKernelGGL((k2_spec_cols<NT_, 4, PAR_>), gc, dim3(NT_), 0, stream, L, s.col, s.cols,          \
                       (const double2 *)X, tw, acc)
    if (s.row_nt == 256) LBFSS_ROWS(256, 4);
    else if (s.row_nt == 512) LBFSS_ROWS(512, 4);
    else if (3 * s.row.n <= 4096) LBFSS_ROWS(1024, 4);
    else LBFSS_ROWS(1024, 8);  // odd L from 1367
    if (s.par) {
        if (s.col_nt == 256) LBFSS_COLS(256, true);
        else if (s.col_nt == 512) LBFSS_COLS(512, true);
        else LBFSS_COLS(1024, true);
    } else {
        if (s.col_nt == 256) LBFSS_COLS(256, false);
        else if (s.col_nt == 512) LBFSS_COLS(512, false);
        else LBFSS_COLS(1024, false);
    }
#undef LBFSS_ROWS
#undef LBFSS_COLS
}

}  // namespace lbfss
