// Several steps of a two-dimensional FP32 domain in one launch (gfx950).
#include "pflb_device.hpp"
#include "pflb_internal.hpp"

namespace pflb {

// Small and ensemble domains step faster than one launch per step lets them: a 64x64 domain
// waits for launches (3.7 us a step whatever it computes), and 16 of 256x256 move their
// whole state through HBM for each step.  Here a workgroup takes T = 3 steps of its tile at
// once: it collides the tile and the 2 (T - 1) sites around it, keeps the post-collision
// populations in LDS, streams them there, and collides two sites less on each side at each
// further step.  The sites around the tile are computed again by their own workgroups: that
// is the price (32x16: 1.43 collisions per site and step, 8x8: 2.4), so the tile grows with
// the domain (see plan_of).  T is odd, so that the state ends in the buffer that single
// steps would leave it in.  The arithmetic of a site is the single-step kernels', in the
// same order, and so are the results, bit for bit (tests/test_gpu_fused2d.py).  Bound by the
// collision's vector instructions on large domains, by the launch and the chain of gather,
// barrier and collision on small ones.  Measured against single steps, us a step, same GPU:
// 64x64 3.73 -> 2.28, 256x256 5.25 -> 3.06, 256x1024 with walls 10.6 -> 6.5, 16 domains of
// 256x256 37.6 -> 22.9, 4096x2048 259 -> 171.  (T = 2: 256x1024 6.8, 16 domains 25.5; T = 4
// and 5: 64x64 2.13 and 2.18, but 256x1024 8.5 and more.)

// post-collision pairs of one position into the workgroup's LDS populations
template <int NPOS>
struct LdsWriter {
    float2* p;
    template <int I>
    __device__ __forceinline__ void put(float h, float g) { p[I * NPOS] = make_float2(h, g); }
    __device__ __forceinline__ void finish() {}
};

template <class L, int WALLS, int T, int OX, int OZ, int NT, bool BATCHED>
__global__ void __launch_bounds__(NT)
k_step_fused(Geom G, Model m, int ntx, int nblk, const char* __restrict__ src,
             char* __restrict__ dst, StepTable<BATCHED> tab) {
    static_assert(!L::USES_Y, "tiles of a two-dimensional lattice");
    if constexpr (BATCHED) {
        const StepEnt& e = tab.bt.e[blockIdx.y];
        m = e.m;
        src = e.src;
        dst = e.dst;
    }
    constexpr int Q = L::Q;
    constexpr int C0 = 2 * (T - 1);                   // sites collided beyond the tile at first
    constexpr int BX = OX + 2 * C0, NPOS = BX * (OZ + 2 * C0);
    __shared__ float2 spop[Q * NPOS];
    __shared__ float sphi[(BX + 2) * (OZ + 2 * C0 + 2)];
    const int t = xcd_tile(blockIdx.x, nblk);
    const int x0 = (t % ntx) * OX, z0 = (t / ntx) * OZ;

    static_for<0, T>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int C = 2 * (T - 1 - k);            // sites collided beyond the tile
        constexpr int CX = OX + 2 * C, CZ = OZ + 2 * C, FX = CX + 2;
        constexpr int NC = CX * CZ, NF = NC + 2 * FX + 2 * CZ;
        constexpr int NS = (NF + NT - 1) / NT;
        // position id of this step: the NC sites it collides, row by row, then the ring
        // of sites around them whose phi they need; px, pz count from the ring's corner
        auto place = [&](int id, int& px, int& pz) {
            pz = id / CX + 1;
            px = id - (pz - 1) * CX + 1;
            const int r = id - NC;
            if (r >= 0) {
                const int q = r - 2 * FX;
                px = q < 0 ? (r < FX ? r : r - FX) : (q & 1) * (FX - 1);
                pz = q < 0 ? (r < FX ? 0 : CZ + 1) : 1 + (q >> 1);
            }
        };
        float h[NS][Q], lo[NS];
        GMom g[NS];
        static_for<0, NS>([&](auto J) {
            constexpr int j = decltype(J)::value;
            constexpr bool RING = j * NT >= NC;       // sites whose phi alone is needed
            int px, pz;
            place(min((int)threadIdx.x + j * NT, NF - 1), px, pz);
            const int at = pz * FX + px;
            int vx = x0 - C - 1 + px, vz = z0 - C - 1 + pz;
            if constexpr (k == 0) {
                // wrap or clamp (periodic axes have at least OX + 2 T or OZ + 2 T sites)
                vx = G.wx ? min(max(vx, 0), G.nx - 1)
                          : (vx < 0 ? vx + G.nx : (vx >= G.nx ? vx - G.nx : vx));
                vz = G.wz ? min(max(vz, 0), G.nz - 1)
                          : (vz < 0 ? vz + G.nz : (vz >= G.nz ? vz - G.nz : vz));
                const Col c = make_col(G, vx, 0);
                const ZRow r = make_zrow(G, vz);
                if constexpr (RING) {
                    float f[Q];
                    sphi[at] = (float)pull_site_h<L, StoreF32, WALLS>(src, G, c, r, Codec{}, f);
                } else {
                    sphi[at] = split_hi_lo(pull_site_m<L, WALLS>(src, G, c, r, h[j], g[j]), lo[j]);
                }
            } else {
                uint32_t solid = 0u;
                if constexpr ((WALLS & WALLS_XY) != 0) {
                    vx = min(max(vx, 0), G.nx - 1);
                    solid |= (vx == 0 ? 1u : 0u) | (vx == G.nx - 1 ? 2u : 0u);
                }
                if constexpr ((WALLS & WALLS_Z) != 0) {
                    vz = min(max(vz, 0), G.nz - 1);
                    solid |= (vz == 0 ? 16u : 0u) | (vz == G.nz - 1 ? 32u : 0u);
                }
                const int pos = (vz - z0 + C0) * BX + (vx - x0 + C0);
                PhiAcc acc;
                if constexpr (!RING) g[j] = GMom{};
                static_for<0, Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    using U = Up<L, i, WALLS>;
                    int from = i * NPOS + pos - L::cx(i) - L::cz(i) * BX;
                    if constexpr (U::MAYFLIP) {
                        bool bb = false;
                        if constexpr (U::test_xy) bb = bb || (solid & U::need_xy) != 0u;
                        if constexpr (U::test_z) bb = bb || (solid & U::need_z) != 0u;
                        from = bb ? opp(i) * NPOS + pos : from;
                    }
                    if constexpr (RING) {
                        acc.r += (double)spop[from].x;
                    } else {
                        const float2 v = spop[from];
                        acc.r += (double)v.x;
                        h[j][i] = v.x;
                        add_moment<L, i>(g[j], v.y);
                    }
                });
                if constexpr (RING) sphi[at] = (float)acc.value();
                else sphi[at] = split_hi_lo(acc.value(), lo[j]);
            }
        });
        lds_barrier();
        static_for<0, (NC + NT - 1) / NT>([&](auto J) {
            constexpr int j = decltype(J)::value;
            const int id = (int)threadIdx.x + j * NT;
            int px, pz;
            place(id, px, pz);
            const int vx = x0 - C - 1 + px, vz = z0 - C - 1 + pz;
            bool on = id < NC;
            if constexpr (k == T - 1) {
                on = on && vx < G.nx && vz < G.nz;
            } else {
                if constexpr ((WALLS & WALLS_XY) != 0) on = on && (unsigned)vx < (unsigned)G.nx;
                if constexpr ((WALLS & WALLS_Z) != 0) on = on && (unsigned)vz < (unsigned)G.nz;
            }
            if (on) {
                const int at = pz * FX + px;
                float pn[Q];
                static_for<0, Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    pn[i] = sphi[at + L::cx(i) + L::cz(i) * FX];
                });
                const Macro a = macros<L>(m, pn, g[j]);
                if constexpr (k == T - 1) {
                    SiteWriter32<L, WALLS> out{dst, (uint32_t)vz * (uint32_t)G.nx + (uint32_t)vx, G.S};
                    collide_stream<L>(m, a, lo[j], h[j], g[j], out);
                } else {
                    LdsWriter<NPOS> out{spop + (vz - z0 + C0) * BX + (vx - x0 + C0)};
                    collide_stream<L>(m, a, lo[j], h[j], g[j], out);
                }
            }
        });
        if constexpr (k < T - 1) lds_barrier();
    });
}

template <int WALLS, int T, int OX, int OZ, int NT>
static hipError_t launch_fused(const Launch& a, const char* s, char* d, const StepBatch* bt, int n) {
    const int ntx = (a.G.nx + OX - 1) / OX;
    const int nblk = ntx * ((a.G.nz + OZ - 1) / OZ);
    if (bt) {
        StepTable<true> tab;
        tab.bt = *bt;
        hipLaunchKernelGGL((k_step_fused<LatD2Q9, WALLS, T, OX, OZ, NT, true>), dim3(nblk, n),
                           dim3(NT), 0, a.stream, a.G, a.m, ntx, nblk, s, d, tab);
    } else {
        hipLaunchKernelGGL((k_step_fused<LatD2Q9, WALLS, T, OX, OZ, NT, false>), dim3(nblk),
                           dim3(NT), 0, a.stream, a.G, a.m, ntx, nblk, s, d, StepTable<false>{});
    }
    return hipGetLastError();
}

constexpr int FUSED_T = 3;
static_assert(FUSED_T % 2 == 1, "a launch leaves the state in the buffer its steps would");

// The tiles there are: sizes and threads.  The sites a tile collides (with those around it)
// are near a multiple of the threads, so that few waves run part empty.
#define PFLB_FUSED(X)                              \
    X(0, 8, 8, 320)   /* 256, 144, 64 sites */     \
    X(1, 16, 16, 576) /* 576, 400, 256 */          \
    X(2, 32, 16, 512) /* 960, 720, 512 */

// Which of them a domain takes, -1 for none.  While the tiles leave CUs idle, small tiles
// win (each step's latency counts, not the repeated work); from there on the repeated work
// counts.  Measured, us a step with each tile: 64x64 2.3, 2.8, 3.7; 128x128 (256 tiles of
// 8x8) 2.4, 2.8, 3.7; 256x256 (1024; 256 of 16x16) 4.0, 3.1, 3.8; 256x1024 11.8, 9.9, 6.5.
static int plan_of(const Launch& a, int n) {
    const auto tiles = [&](long ox, long oz) {
        return (a.G.nx + ox - 1) / ox * ((a.G.nz + oz - 1) / oz) * n;
    };
    const int k = tiles(8, 8) <= 512 ? 0 : (tiles(16, 16) <= 256 ? 1 : 2);
    // the kernel wraps a position of a periodic axis once
    const int ox = k == 0 ? 8 : (k == 1 ? 16 : 32), oz = k == 0 ? 8 : 16;
    const bool fits = (a.G.wx || a.G.nx >= ox + 2 * FUSED_T) && (a.G.wz || a.G.nz >= oz + 2 * FUSED_T);
    return fits ? k : -1;
}

int fused_steps(const Launch& a, int n, int left) {
    return a.fuse && left >= FUSED_T && plan_of(a, n) >= 0 ? FUSED_T : 1;
}

template <int WALLS>
static hipError_t fused_w(const Launch& a, const char* s, char* d, const StepBatch* bt, int n) {
    switch (plan_of(a, n)) {
#define X(K, OX, OZ, NT) \
    case K: return launch_fused<WALLS, FUSED_T, OX, OZ, NT>(a, s, d, bt, n);
        PFLB_FUSED(X)
#undef X
    }
    return hipErrorInvalidValue;
}

hipError_t launch_step_fused(const Launch& a, const void* src, void* dst, const StepBatch* bt,
                             int n) {
    if (!a.fuse || n < 1 || n > BATCH_MAX) return hipErrorInvalidValue;
    const char* s = static_cast<const char*>(src);
    char* d = static_cast<char*>(dst);
    switch ((a.G.wx ? WALLS_XY : 0) | (a.G.wz ? WALLS_Z : 0)) {
        case WALLS_XYZ: return fused_w<WALLS_XYZ>(a, s, d, bt, n);
        case WALLS_XY: return fused_w<WALLS_XY>(a, s, d, bt, n);
        case WALLS_Z: return fused_w<WALLS_Z>(a, s, d, bt, n);
        default: return fused_w<WALLS_NONE>(a, s, d, bt, n);
    }
}

}  // namespace pflb
