// Block step: one workgroup owns a block of TX x TY x TZ sites, all planes at
// once, instead of marching through z.  Two uses:
//
// DENS = false: the whole step in one launch, for lattices that do not fill
// the chip with marching workgroups.  Every thread pulls the populations of
// its own site (kept in registers) and those of its share of the block's halo
// (for the density only), so each load is on the way before the first is
// waited for; the normals are drawn meanwhile.  Densities, then the chemical
// potential on the block and a one-site halo go through LDS (the paper's
// model, EQ, needs a one-site density halo and no potential), then force,
// collision, store.  What bounds it is the chain launch -> loads -> potential
// -> collision: a marching workgroup walks that chain once per plane, tz + 4
// times (16^3 FP32: 54 us a step marching, 9.1 us with the halo in a loop,
// 7.2 us with all loads first; 64^3: 62 -> 15.7 us).
//
// DENS = true: the collide pass of the split plan.  The density of every site
// comes from the pass before; potential, force and collision are one launch
// (96^3 FP32: 47.5 -> 41 us a step against separate potential and collide
// passes, which also wrote and read the potential; 250^3: 859 us, the
// marching kernel with per-site loads 1183 us).  Memory-bound: 240 bytes a
// site, at 96^3 5.0 TB/s.
//
// Positions past the lattice's edge are wrapped, so a block that sticks out
// (or is wider than the lattice) holds densities of periodic images there,
// which are the halo its last sites need; those positions are not collided.
// The arithmetic is the same function calls as in the marching kernels.
#pragma once

#include "lbfss_fused.hpp"
#include "lbfss_meq.hpp"

namespace lbfss {

// v in [-2, L + 35] to [0, L); rL = 1 / L to an ulp: (v + 1/2) / L stays at
// least 1 / (2 L) from an integer, far more than its rounding error
__device__ __forceinline__ int wrap_far(int v, int L, float rL) {
    return v - L * (int)floorf(((float)v + 0.5f) * rL);
}

// The 19 pulled values of site (x, y, z): every load is a scalar base (the
// population's) plus a 32-bit byte offset (L <= 1024: 4 GiB a population).
// MUL24: the row and plane offsets by the full-rate multiply (factors below
// 2^24, products modulo 2^32).  A site of the FP32 force model's blocks pulls
// up to six times and waits on these chains (16^3: 7.5 -> 7.2 us a step, 32^3
// 8.1 -> 7.7, 64^3 15.9 -> 15.7); the other forms schedule worse with
// it (FP16 64^3 13.5 -> 14.0, equilibrium model 13.2 -> 13.7).
template <bool MUL24, typename T>
__device__ __forceinline__ void pull_site(const T *base, uint32_t N, int L, int x, int y, int z, float (&r)[Q]) {
    constexpr uint32_t S = sizeof(T);
    const uint32_t row = (uint32_t)L * S, plane = (uint32_t)L * row;
    const uint32_t x0 = x * S, xm = wrap_dec(x, L) * S, xp = wrap_inc(x, L) * S;
    auto mul = [](uint32_t v, uint32_t w) -> uint32_t { return MUL24 ? (uint32_t)__umul24(v, w) : v * w; };
    const uint32_t y0 = mul(y, row), ym = mul(wrap_dec(y, L), row), yp = mul(wrap_inc(y, L), row);
    const uint32_t z0 = mul(z, plane), zm = mul(wrap_dec(z, L), plane), zp = mul(wrap_inc(z, L), plane);
#pragma unroll
    for (int q = 0; q < Q; ++q) {  // source x - c_q
        const int cx = cx_of(q), cy = cy_of(q), cz = cz_of(q);
        const uint32_t off = (cx > 0 ? xm : (cx < 0 ? xp : x0)) +
                             ((cy > 0 ? ym : (cy < 0 ? yp : y0)) + (cz > 0 ? zm : (cz < 0 ? zp : z0)));
        r[q] = ldb(base + (size_t)q * N, off);
    }
}

template <typename T, int TX, int TY, int TZ, int NT, bool EQ, bool DENS, bool SNAP>
__global__ void __launch_bounds__(NT)
k_block(const RepDesc *__restrict__ desc, const FusedTile *__restrict__ tiles, const T *__restrict__ pop,
        T *__restrict__ pop_out, const float *__restrict__ drho, const uint64_t *__restrict__ step, int koff,
        int *__restrict__ err, float *__restrict__ snap, int64_t total) {
    static_assert(!(EQ && DENS), "the paper's model has a collide pass of its own");
    constexpr int NS = TX * TY * TZ;
    static_assert(NS <= NT, "one site per thread");
    constexpr int H = EQ ? 1 : 2;
    constexpr bool kMul24 = sizeof(T) == 4 && !EQ && !DENS;
    constexpr int EX = TX + 2 * H, EY = TY + 2 * H, EZ = TZ + 2 * H, EP = EX * EY, NE = EP * EZ;
    constexpr int MX = TX + 2, MY = TY + 2, MZ = TZ + 2, MP = MX * MY;
    constexpr int RING = EP - TX * TY;          // halo positions of a plane of the block
    constexpr int NH = 2 * H * EP + TZ * RING;  // halo positions
    // values a thread loads for the densities: halo sites, or stored densities
    constexpr int KH = ((DENS ? NE : NH) + NT - 1) / NT;
    // four threads per site: each draws one Philox call of the site's four
    // (16^3: 7.5 -> 7.2 us a step against all four in the site's own thread)
    constexpr bool SPREAD = !EQ && NT == 4 * NS;
    __shared__ float s_rho[NE];
    __shared__ float s_mu[EQ ? 1 : MP * MZ];
    __shared__ float s_noise[SPREAD ? 16 * NS : 1];

    const FusedTile tl = tiles[xcd_tile(blockIdx.x, gridDim.x)];
    if (tl.nz == 0) return;              // padding of a batch's table (whole workgroup)
    const RepDesc d = desc[tl.rep];      // a copy: its loads go out here, not behind the barriers
    const int L = d.L;
    const float rL = __builtin_amdgcn_rcpf((float)L);
    const uint32_t N = (uint32_t)d.N;
    const T *base = pop + Q * d.site_off;
    const uint64_t t = *step + (uint64_t)koff;
    const int tid = threadIdx.x;
    auto site_of = [&](int i, int &x, int &y, int &z) {  // site i of the block
        x = wrap_far(tl.x0 + i % TX, L, rL);
        y = wrap_far(tl.y0 + (i / TX) % TY, L, rL);
        z = wrap_far(tl.z0 + i / (TX * TY), L, rL);
        return (uint32_t)(x + L * (y + L * z));
    };
    // extended position of halo site h: the H planes below and above the
    // block, then per plane of the block the rows and the columns around it
    auto halo_at = [&](int h, int &ex, int &ey, int &ez) {
        if (h < 2 * H * EP) {
            const int p = h / EP, k = h - p * EP;
            ez = p < H ? p : TZ + p;
            ey = k / EX;
            ex = k - ey * EX;
        } else {
            const int g = h - 2 * H * EP, p = g / RING, k = g - p * RING;
            ez = H + p;
            if (k < 2 * H * EX) {
                const int row = k / EX;
                ey = row < H ? row : TY + row;
                ex = k - row * EX;
            } else {
                const int c = k - 2 * H * EX, col = c % (2 * H);
                ey = H + c / (2 * H);
                ex = col < H ? col : TX + col;
            }
        }
    };
    const int ix = tid % TX, iy = (tid / TX) % TY, iz = tid / (TX * TY);
    const bool own = NS == NT || tid < NS;
    const int r_in = ((iz + H) * EY + (iy + H)) * EX + (ix + H);
    int x, y, z;
    const uint32_t s = site_of(own ? tid : 0, x, y, z);
    float f[Q];
    if (own) pull_site<kMul24>(base, N, L, x, y, z, f);
    // the threads past the last position load it again
    float hv[KH][DENS ? 1 : Q];
    int hs[KH];
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        int ex, ey, ez;
        if constexpr (DENS) {
            const int h = min(tid + k * NT, NE - 1);
            ez = h / EP;
            ey = (h - ez * EP) / EX;
            ex = h - ez * EP - ey * EX;
        } else {
            halo_at(min(tid + k * NT, NH - 1), ex, ey, ez);
        }
        hs[k] = (ez * EY + ey) * EX + ex;
        const int hx = wrap_far(tl.x0 - H + ex, L, rL), hy = wrap_far(tl.y0 - H + ey, L, rL),
                  hz = wrap_far(tl.z0 - H + ez, L, rL);
        if constexpr (DENS) hv[k][0] = drho[d.site_off + (uint32_t)(hx + L * (hy + L * hz))];
        else pull_site<kMul24>(base, N, L, hx, hy, hz, hv[k]);
    }
    // the normals, while the loads are on their way
    float gn[16];
    if constexpr (SPREAD) {
        int nx, ny, nz;
        const int i = tid % NS, call = tid / NS;
        const SiteNoise noise{site_of(i, nx, ny, nz), (uint32_t)t, (uint32_t)(t >> 32), d.key0, d.key1};
        float v[4];
        noise(call, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) s_noise[(4 * call + k) * NS + i] = v[k];
    } else if constexpr (!EQ) {
        const SiteNoise noise{s, (uint32_t)t, (uint32_t)(t >> 32), d.key0, d.key1};
#pragma unroll
        for (int call = 0; call < 4; ++call) {
            float v[4];
            noise(call, v);
#pragma unroll
            for (int k = 0; k < 4; ++k) gn[4 * call + k] = v[k];
        }
    }
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        if constexpr (DENS) s_rho[hs[k]] = hv[k][0];
        else s_rho[hs[k]] = drho_of(hv[k]);
    }
    if (!DENS && own) s_rho[r_in] = drho_of(f);
    __syncthreads();
    if constexpr (!EQ) {
        for (int m = tid; m < MP * MZ; m += NT) {
            const int mz = m / MP, my = (m - mz * MP) / MX, mx = m - mz * MP - my * MX;
            const float *c = &s_rho[((mz + 1) * EY + (my + 1)) * EX + (mx + 1)];
            s_mu[m] = chem_potential(
                d, *c, lap18(*c, [&](int dx, int dy, int dz) { return c[(dz * EY + dy) * EX + dx]; }));
        }
        __syncthreads();
    }
    if (!own || ix >= tl.nx || iy >= tl.ny || iz >= tl.nz) return;
    if constexpr (SNAP) write_snapshot(snap, total, d.site_off + (int64_t)s, f);
    const float *rc = &s_rho[r_in];
    bool bad;
    if constexpr (EQ) {
        bad = !meq_collide_site(
            d, f, *rc, [&](int dx, int dy, int dz) { return rc[(dz * EY + dy) * EX + dx]; }, s, t, meq_nu(d));
    } else {
        float Fx = 0.f, Fy = 0.f, Fz = 0.f;
        if (!(d.flags & 1)) {
            // F = -rho grad(mu) + c_s^2 grad(drho) = grad of psi(y) = drho(y)/3 - rho(x) mu(y)
            const float *mc = &s_mu[((iz + 1) * MY + (iy + 1)) * MX + (ix + 1)];
            const float rho_x = d.rho_c + *rc;
            const Grad18 gr = grad18([&](int dx, int dy, int dz) {
                return (1.0f / 3.0f) * rc[(dz * EY + dy) * EX + dx] - rho_x * mc[(dz * MY + dy) * MX + dx];
            });
            Fx = gr.gx;
            Fy = gr.gy;
            Fz = gr.gz;
        }
        const float rho = collide_site(d, f, Fx, Fy, Fz, [&](int call, float (&n)[4]) {
#pragma unroll
            for (int k = 0; k < 4; ++k) n[k] = SPREAD ? s_noise[(4 * call + k) * NS + tid] : gn[4 * call + k];
        });
        bad = !(rho > 0.0f && rho < 1e30f);  // Sec. III B: rho must stay positive
    }
    T *out = pop_out + Q * d.site_off;
#pragma unroll
    for (int q = 0; q < Q; ++q) Store<T>::st(out + (size_t)q * N, s, f[q]);
    if (bad) *err = 1;
}

// Tiles of a rows, staged or fused plan that run as blocks: shallow ones, of
// which a marching workgroup would spend most planes on the halo.
inline bool block_tile(bool eq, int tx, int ty, int tz) {
    if (eq) return tx == 32 && ty == 8 && tz <= 2;
    return (tx == 16 && ty == 8 && (tz == 1 || tz == 4)) || (tx == 32 && ty == 8 && tz == 4);
}
// Blocks of the split plan's collide pass: 32-wide rows (16 x 8 x 4 takes 979
// us a step at 250^3 FP32), 4 x 4 of them, which need the fewest halo rows of
// the density: FP16 100^3 41.5 against 45.4 us on 8 x 2 rows, 250^3 537 against
// 549; FP32 50^3 14.6 against 14.95, 178^3 306 against 317.  On large FP32
// lattices the y neighbours' rows in the L2 count for more: 198^3 424 on 8 x 2
// against 425, 226^3 628 against 635, 250^3 844 against 853.
constexpr int kSplitTX = 32;
inline bool split_flat(bool fp16, int64_t sites) { return !fp16 && sites >= 190 * 190 * 190; }

struct BlockArgs {
    const RepDesc *desc;
    const FusedTile *tiles;
    int n_tiles;
    const uint64_t *step;
    int koff;
    int *err;
    float *snap;  // where the step also writes the sample snapshot of its input state, or null
    int64_t total;
    hipStream_t stream;
};

template <int TX, int TY, int TZ, int NT, bool EQ, bool DENS, typename T>
void launch_block_shape(const BlockArgs &a, const T *in, T *out, const float *drho) {
    if (a.snap)
        hipLaunchKernelGGL((k_block<T, TX, TY, TZ, NT, EQ, DENS, true>), dim3(a.n_tiles), dim3(NT), 0, a.stream,
                           a.desc, a.tiles, in, out, drho, a.step, a.koff, a.err, a.snap, a.total);
    else
        hipLaunchKernelGGL((k_block<T, TX, TY, TZ, NT, EQ, DENS, false>), dim3(a.n_tiles), dim3(NT), 0, a.stream,
                           a.desc, a.tiles, in, out, drho, a.step, a.koff, a.err, a.snap, a.total);
}

// the force model's step on tiles (tx, ty, tz) that block_tile accepts
template <typename T>
void launch_block(const BlockArgs &a, int tx, int tz, const T *in, T *out) {
    if (tx == 32) launch_block_shape<32, 8, 4, 1024, false, false>(a, in, out, nullptr);
    else if (tz == 4) launch_block_shape<16, 8, 4, 512, false, false>(a, in, out, nullptr);
    else launch_block_shape<16, 8, 1, 512, false, false>(a, in, out, nullptr);
}

// the paper's model
inline void launch_block_eq(const BlockArgs &a, int tz, const float *in, float *out) {
    if (tz == 2) launch_block_shape<32, 8, 2, 512, true, false>(a, in, out, nullptr);
    else launch_block_shape<32, 8, 1, 256, true, false>(a, in, out, nullptr);
}

// the collide pass of the split plan
template <typename T>
void launch_block_split(const BlockArgs &a, const T *in, T *out, const float *drho) {
    if (split_flat(sizeof(T) == 2, a.total)) launch_block_shape<kSplitTX, 8, 2, 512, false, true>(a, in, out, drho);
    else launch_block_shape<kSplitTX, 4, 4, 512, false, true>(a, in, out, drho);
}

}  // namespace lbfss
