// Kernel parameters from the host state of a handle, and the dispatch from
// its run-time lattice, precision and x boundary to the compiled variants.
#pragma once

#include "engine.hpp"
#include "kernels.hpp"

namespace lbe {

// the grid of a node launch
inline Grid make_grid(const Engine& e) {
    Grid g;
    g.nx = (uint32_t)e.nx;
    g.ny = (uint32_t)e.ny;
    g.nz = (uint32_t)e.nz;
    g.N = (uint32_t)e.N;
    g.S = (uint32_t)e.S;
    g.nblocks = (uint32_t)((e.N + BX - 1) / BX);
    g.bpr = e.nx % BX == 0 ? (uint32_t)(e.nx / BX) : 0u;
    return g;
}

template <class L, class T>
Params<L, T> make_params(const Engine& e) {
    Params<L, T> p;
    for (int k = 0; k < L::Q; ++k) {
        const double r = L::conserved(k) ? 0.0 : e.s[k] / (double)TAB<L>.norm[k];
        p.rate[k] = (T)r;
    }
    for (int a = 0; a < 3; ++a) p.G[a] = (T)(3.0 * e.rho0 * (a < L::D ? e.g[a] : 0.0));
    p.drho = (T)(e.xbc == XBC_PRESSURE ? e.drho : 0.0);
    for (int i = 0; i < L::Q; ++i) {
        double eg = 0;
        for (int a = 0; a < L::D; ++a) eg += L::E[i][a] * e.g[a];
        p.force[i] = (T)(3.0 * L::W[i] * e.rho0 * eg);
        p.seam[i] = (T)(L::W[i] * (e.xbc == XBC_PRESSURE ? e.drho : 0.0));
    }
    p.rho0 = (T)e.rho0;
    p.inv_rho0 = (T)(1.0 / e.rho0);
    p.c0 = 1.0 - e.b;
    p.rho0_d = e.rho0;
    p.wall_scale = e.wall_decay == 1.0 ? 1.0 : e.wall_scale;
    p.c1d = e.two_node ? e.d_lkc1d : nullptr;
    return p;
}

// runtime -> compile-time dispatch over lattice, precision and x boundary
template <class F>
hipError_t dispatch(const Engine& e, F&& f) {
    auto by_xbc = [&](auto lat, auto prec) -> hipError_t {
        using L = decltype(lat);
        using T = decltype(prec);
        switch (e.xbc) {
            case XBC_PRESSURE: return f(L{}, T{}, std::integral_constant<int, XBC_PRESSURE>{});
            case XBC_OUTFLOW: return f(L{}, T{}, std::integral_constant<int, XBC_OUTFLOW>{});
            default: return f(L{}, T{}, std::integral_constant<int, XBC_PERIODIC>{});
        }
    };
    if (e.lattice == 0)
        return e.precision == 0 ? by_xbc(D2Q9{}, double{}) : by_xbc(D2Q9{}, float{});
    if (e.lattice == 2)
        return e.precision == 0 ? by_xbc(D3Q15{}, double{}) : by_xbc(D3Q15{}, float{});
    return e.precision == 0 ? by_xbc(D3Q19{}, double{}) : by_xbc(D3Q19{}, float{});
}

}  // namespace lbe
