// In-place storage of the FP32 populations: one state buffer instead of two (half the
// footprint of the pull storage, so about twice the sites per GPU).
//
// Scheme (the "AA" pattern of in-place lattice Boltzmann streaming): two layouts of the
// same Q arrays of h followed by Q arrays of g, each array of stride S floats.
//   layout 0  f_i(x) is in slot (x, i);
//   layout 1  f_i(x) is in slot (x - c_i, opp(i)), or in slot (x, i) where x - c_i lies
//             beyond a wall (halfway bounce-back, Section 2's walls).
// A step from layout 0 reads a site's own slots and writes its post-collision f*_i into
// slot (x, opp(i)); the next step's reader x + c_i then finds it in slot
// ((x + c_i) - c_i, opp(i)): layout 1.  A step from layout 1 reads as layout 1 says and
// writes f*_i into slot (x + c_i, i), or into slot (x, opp(i)) where x + c_i lies beyond a
// wall: layout 0 again.  In either step the slots a site writes are exactly those it
// read, so sites never touch each other's slots and one buffer suffices.
//
// The price is phi: the collision needs phi at the neighbours (central differences,
// Eqs. 2-4 and 9), which other workgroups overwrite in place during the same launch.
// Each step therefore runs two kernels: k_ip_phi writes the phi field (reading only the
// h arrays, 76 B per D3Q19 site, writing 4 B), then k_ip_step collides every site with
// its neighbours' phi from that field (152 B read, 152 B written per site).  That is
// about 1.26x the bytes of the fused pull step, at half its state footprint.
#include "pflb_internal.hpp"

namespace pflb {
namespace {

// Addresses.  As in the pull kernels, a site's neighbours are 32-bit site offsets of its column
// and plane (Col, ZRow), the wall tests are compiled for the walls a domain has (WALLS), and an
// access is a uniform base plus a 32-bit byte offset where they fit (else WALLS has ADDR64).
// Deriving every neighbour by itself, with the wrap's divisions and branches, was more than
// half of the 2000 to 2800 instructions a wave spent on a site and bound the step's second
// kernel: 172 us on 128^3, now 126 (5.1 TB/s), and the first's 31 are the read of the h arrays.

// slot (site, i) of set k (0: h, 1: g), and with FLIP of (site, flip ? opp(i) : i)
template <class L, int I, int WALLS, bool FLIP = false>
__device__ __forceinline__ float* ip_slot(char* __restrict__ b, const Geom& G, int k,
                                          uint32_t site, bool flip = false) {
    char* set = b + (size_t)k * L::Q * G.S * 4;
    if constexpr (!FLIP || I == 0) {
        return reinterpret_cast<float*>(set + (size_t)I * G.S * 4 + elem_off<WALLS, 4>(site));
    } else {
        uint32_t off;
        const char* base = slot_addr<L, I, WALLS, 4>(set, G.S, site, flip, off);
        return reinterpret_cast<float*>(const_cast<char*>(base) + off);
    }
}

// the slots of set 0 and 1 where layout LY holds f_I of the site (c, r)
template <class L, int I, int LY, int WALLS, class F>
__device__ __forceinline__ void ip_source(char* __restrict__ b, const Geom& G, const Col& c,
                                          const ZRow& r, F&& f) {
    if constexpr (LY == 0 || I == 0) {
        const uint32_t s = c.base + r.base;
        f(ip_slot<L, I, WALLS>(b, G, 0, s), ip_slot<L, I, WALLS>(b, G, 1, s));
    } else {
        // (x - c_I, opp(I)), or (x, I) where x - c_I lies beyond a wall
        uint32_t t;
        bool flip;
        upstream<L, I, WALLS>(c, r, t, flip);
        f(ip_slot<L, opp(I), WALLS, true>(b, G, 0, t, flip),
          ip_slot<L, opp(I), WALLS, true>(b, G, 1, t, flip));
    }
}

// neighbour x + (dx, dy, dz) with the periodic wrap; false where it lies beyond a wall
__device__ __forceinline__ bool ip_neighbour(const Geom& G, int x, int y, int z, int dx, int dy,
                                             int dz, size_t& t) {
    int v[3] = {x + dx, y + dy, z + dz};
    const int n[3] = {G.nx, G.ny, G.nz};
    const int w[3] = {G.wx, G.wy, G.wz};
    for (int a = 0; a < 3; ++a) {
        if (v[a] < 0 || v[a] >= n[a]) {
            if (w[a]) return false;
            v[a] = v[a] < 0 ? v[a] + n[a] : v[a] - n[a];
        }
    }
    t = site_of(G, v[0], v[1], v[2]);
    return true;
}

// f_i(x) for all i from layout LY; returns phi = sum h in float64, in index order (the
// sum the pull kernels form)
template <class L, int LY, int WALLS>
__device__ __forceinline__ double ip_load(const Geom& G, const char* __restrict__ b, const Col& c,
                                          const ZRow& r, float (&h)[L::Q], float (&g)[L::Q]) {
    double phi = 0.0;
    static_for<0, L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        ip_source<L, i, LY, WALLS>(const_cast<char*>(b), G, c, r, [&](float* ph, float* pg) {
            h[i] = *ph;
            g[i] = *pg;
        });
        phi += (double)h[i];
    });
    return phi;
}

template <class L, int LY, int WALLS>
__device__ __forceinline__ double ip_phi(const Geom& G, const char* __restrict__ b, const Col& c,
                                         const ZRow& r) {
    double phi = 0.0;
    static_for<0, L::Q>([&](auto I) {
        ip_source<L, decltype(I)::value, LY, WALLS>(
            const_cast<char*>(b), G, c, r, [&](float* ph, float*) { phi += (double)*ph; });
    });
    return phi;
}

// phi(x + c_k) for all k from the phi field, as phi_stencil: beyond a wall the adjacent site's,
// axis by axis
template <class L, int WALLS>
__device__ __forceinline__ void ip_stencil(const Geom& G, const Model& m,
                                           const float* __restrict__ phi, const Col& c,
                                           const ZRow& r, int x, int y, int z, float (&pn)[L::Q]) {
    const uint32_t xm = c.solid & 1u ? 0u : c.dxm, xp = c.solid & 2u ? 0u : c.dxp;
    const uint32_t ym = c.solid & 4u ? 0u : c.dym, yp = c.solid & 8u ? 0u : c.dyp;
    const uint32_t zm = r.solid & 16u ? 0u : r.dzm, zp = r.solid & 32u ? 0u : r.dzp;
    static_for<0, L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int ex = L::cx(i), ey = L::cy(i), ez = L::cz(i);
        uint32_t t = c.base + r.base;
        if constexpr (ex != 0) t += ex > 0 ? xp : xm;
        if constexpr (ey != 0) t += ey > 0 ? yp : ym;
        if constexpr (ez != 0) t += ez > 0 ? zp : zm;
        pn[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(phi) +
                                                elem_off<WALLS, 4>(t));
    });
    if (m.wetting)
        static_for<0, L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            pn[i] = wet_ghost(G, m, x + L::cx(i), y + L::cy(i), z + L::cz(i), pn[i]);
        });
}

// Writer of a site's post-collision pairs for a step from layout LY.  (From layout 1 the
// neighbour is derived afresh, with branches, for each population: the collision between two
// of them is then compiled by itself, as it always was, and rounds the same.  Offsets there
// as well measured 122 us, and another rounding.)
template <class L, int LY, int WALLS>
struct IpWriter {
    char* __restrict__ b;
    const Geom& G;
    const Col& c;
    const ZRow& r;
    int x, y, z;
    template <int I>
    __device__ __forceinline__ void put(float hv, float gv) {
        if constexpr (LY == 0 || I == 0) {
            const uint32_t s = c.base + r.base;
            *ip_slot<L, opp(I), WALLS>(b, G, 0, s) = hv;
            *ip_slot<L, opp(I), WALLS>(b, G, 1, s) = gv;
        } else {
            // (x + c_I, I), or (x, opp(I)) where x + c_I lies beyond a wall
            int dir = opp(I);
            size_t t = c.base + r.base;
            size_t d;
            if (ip_neighbour(G, x, y, z, L::cx(I), L::cy(I), L::cz(I), d)) {
                dir = I;
                t = d;
            }
            *reinterpret_cast<float*>(b + ((size_t)dir * G.S + t) * 4) = hv;
            *reinterpret_cast<float*>(b + ((size_t)(L::Q + dir) * G.S + t) * 4) = gv;
        }
    }
    __device__ __forceinline__ void finish() {}
    __device__ __forceinline__ void shift_h_total(double) {}
};

template <class L, int LY, int WALLS>
__global__ void __launch_bounds__(256)
k_ip_phi(Geom G, uint32_t N, const char* __restrict__ b, float* __restrict__ phi) {
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    if (s >= N) return;
    int x, y, z;
    site_coords(G, s, x, y, z);
    phi[s] = (float)ip_phi<L, LY, WALLS>(G, b, make_col(G, x, y), make_zrow(G, z));
}

template <class L, int LY, int WALLS>
__global__ void __launch_bounds__(256)
k_ip_step(Geom G, Model m, uint32_t N, char* __restrict__ b, const float* __restrict__ phi) {
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    if (s >= N) return;
    int x, y, z;
    site_coords(G, s, x, y, z);
    const Col c = make_col(G, x, y);
    const ZRow r = make_zrow(G, z);
    float h[L::Q], g[L::Q];
    float lo;
    const float hi = split_hi_lo(ip_load<L, LY, WALLS>(G, b, c, r, h, g), lo);
    float pn[L::Q];
    ip_stencil<L, WALLS>(G, m, phi, c, r, x, y, z, pn);
    pn[0] = hi;      // the same float the phi kernel wrote (the same sum, rounded once)
    const GMom gm = g_moments<L>(g);
    const Macro a = macros<L>(m, pn, gm);
    IpWriter<L, LY, WALLS> out{b, G, c, r, x, y, z};
    if (m.moving) {
        // moving walls: the momentum correction of the populations sent into them
        const uint32_t solid = c.solid | r.solid;
        WallWriter<L, IpWriter<L, LY, WALLS>> wout{out, m, solid, 6.0f * a.phi, 6.0f * a.rho,
                                                   solid != 0u};
        collide_stream<L>(m, a, lo, h, gm, wout);
    } else {
        collide_stream<L>(m, a, lo, h, gm, out);
    }
}

// state upload: pre-collision populations (h, g: Q arrays of N) into layout 0
template <class L>
__global__ void __launch_bounds__(256)
k_ip_set(Geom G, uint32_t N, const float* __restrict__ h, const float* __restrict__ g,
         char* __restrict__ b) {
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    if (s >= N) return;
    static_for<0, L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        *ip_slot<L, i, ADDR64>(b, G, 0, s) = h[(size_t)i * N + s];
        *ip_slot<L, i, ADDR64>(b, G, 1, s) = g[(size_t)i * N + s];
    });
}

template <class L, int LY, int WALLS>
__global__ void __launch_bounds__(256)
k_ip_get(Geom G, uint32_t N, const char* __restrict__ b, float* __restrict__ h,
         float* __restrict__ g) {
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    if (s >= N) return;
    int x, y, z;
    site_coords(G, s, x, y, z);
    float fh[L::Q], fg[L::Q];
    ip_load<L, LY, WALLS>(G, b, make_col(G, x, y), make_zrow(G, z), fh, fg);
    static_for<0, L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        h[(size_t)i * N + s] = fh[i];
        g[(size_t)i * N + s] = fg[i];
    });
}

// P, J and u (each may be NULL) from the state and its phi field
template <class L, int LY, int WALLS>
__global__ void __launch_bounds__(256)
k_ip_macro(Geom G, Model m, uint32_t N, const char* __restrict__ b, const float* __restrict__ phi,
           float* __restrict__ P, float* __restrict__ J, float* __restrict__ U) {
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    if (s >= N) return;
    int x, y, z;
    site_coords(G, s, x, y, z);
    float pn[L::Q], hv[L::Q], gv[L::Q];
    const Col col = make_col(G, x, y);
    const ZRow row = make_zrow(G, z);
    ip_stencil<L, WALLS>(G, m, phi, col, row, x, y, z, pn);
    ip_load<L, LY, WALLS>(G, b, col, row, hv, gv);
    const Macro a = macros<L>(m, pn, g_moments<L>(gv));
    if (P) P[s] = a.P;
    const float jv[3] = {a.jx, a.jy, a.jz};
    const float uv[3] = {a.ux, a.uy, a.uz};
    for (int c = 0; c < L::D; ++c) {
        if (J) J[(size_t)c * N + s] = jv[user_axis<L>(c)];
        if (U) U[(size_t)c * N + s] = uv[user_axis<L>(c)];
    }
}

inline dim3 grid_of(uint32_t N) { return dim3((N + 255u) / 256u); }

// calls f with the wall set to compile for (several share a variant) and the layout
template <class F>
hipError_t for_walls(const Launch& a, int layout, F&& f) {
    const auto with = [&](auto w) {
        return layout ? f(w, std::integral_constant<int, 1>{}) : f(w, std::integral_constant<int, 0>{});
    };
    if (a.wide) return with(std::integral_constant<int, WALLS_XYZ | ADDR64>{});
    if (a.G.wx || a.G.wy) return with(std::integral_constant<int, WALLS_XYZ>{});
    if (a.G.wz) return with(std::integral_constant<int, WALLS_Z>{});
    return with(std::integral_constant<int, WALLS_NONE>{});
}

template <class L>
hipError_t step_t(const Launch& a, void* b, int layout, float* phi) {
    const uint32_t N = (uint32_t)a.G.nx * a.G.ny * a.G.nz;
    return for_walls(a, layout, [&](auto w, auto ly) {
        hipLaunchKernelGGL((k_ip_phi<L, ly, w>), grid_of(N), dim3(256), 0, a.stream, a.G, N,
                           static_cast<const char*>(b), phi);
        hipLaunchKernelGGL((k_ip_step<L, ly, w>), grid_of(N), dim3(256), 0, a.stream, a.G, a.m, N,
                           static_cast<char*>(b), static_cast<const float*>(phi));
        return hipGetLastError();
    });
}

template <class L>
hipError_t get_t(const Launch& a, uint32_t N, const void* b, int layout, float* h, float* g) {
    return for_walls(a, layout, [&](auto w, auto ly) {
        hipLaunchKernelGGL((k_ip_get<L, ly, w>), grid_of(N), dim3(256), 0, a.stream, a.G, N,
                           static_cast<const char*>(b), h, g);
        return hipGetLastError();
    });
}

template <class L>
hipError_t read_t(const Launch& a, uint32_t N, const void* b, int layout, float* phi, float* P,
                  float* J, float* U) {
    return for_walls(a, layout, [&](auto w, auto ly) {
        const char* c = static_cast<const char*>(b);
        hipLaunchKernelGGL((k_ip_phi<L, ly, w>), grid_of(N), dim3(256), 0, a.stream, a.G, N, c, phi);
        if (P || J || U)
            hipLaunchKernelGGL((k_ip_macro<L, ly, w>), grid_of(N), dim3(256), 0, a.stream, a.G, a.m,
                               N, c, static_cast<const float*>(phi), P, J, U);
        return hipGetLastError();
    });
}

}  // namespace

hipError_t launch_step_inplace(const Launch& a, void* b, int layout, float* phi) {
    return a.q == 19 ? step_t<LatD3Q19>(a, b, layout, phi) : step_t<LatD2Q9>(a, b, layout, phi);
}

hipError_t launch_set_state_inplace(const Launch& a, uint32_t N, const float* h, const float* g,
                                    void* b) {
    char* c = static_cast<char*>(b);
    if (a.q == 19)
        hipLaunchKernelGGL((k_ip_set<LatD3Q19>), grid_of(N), dim3(256), 0, a.stream, a.G, N, h, g, c);
    else
        hipLaunchKernelGGL((k_ip_set<LatD2Q9>), grid_of(N), dim3(256), 0, a.stream, a.G, N, h, g, c);
    return hipGetLastError();
}

hipError_t launch_get_state_inplace(const Launch& a, uint32_t N, const void* b, int layout,
                                    float* h, float* g) {
    return a.q == 19 ? get_t<LatD3Q19>(a, N, b, layout, h, g) : get_t<LatD2Q9>(a, N, b, layout, h, g);
}

hipError_t launch_read_inplace(const Launch& a, uint32_t N, const void* b, int layout, float* phi,
                               float* P, float* J, float* U) {
    return a.q == 19 ? read_t<LatD3Q19>(a, N, b, layout, phi, P, J, U)
                     : read_t<LatD2Q9>(a, N, b, layout, phi, P, J, U);
}

}  // namespace pflb
