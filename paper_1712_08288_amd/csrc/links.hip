// The link tables on the device: the caller's gamma and phi in link order,
// checked, and the coefficients of Eq. (213) made from them.  Both kernels move
// a link's data once and are bound by it; on the host the same work and its
// transfers were most of an update (gradient of 24 steps at 256x256x48 FP32
// through the autograd function, new link fractions each time: 12.6 -> 5.7 ms).
#include "engine.hpp"
#include "kernels.hpp"
#include "link_rule.hpp"
#include "params.hpp"

namespace lbe {

// One thread per link: its gamma and phi from the caller's order (perm) into q
// and wall_u (q_in or wall_in null: the values they had).  bad[0], bad[1]: the first link whose gamma is outside (0, 1] or
// whose l(gamma) is outside the band of Eq. (212).
template <int D>
__global__ void __launch_bounds__(BX)
k_take_links(const double* __restrict__ q_in, const double* __restrict__ wall_in,
             const int32_t* __restrict__ perm, const double* __restrict__ q_old,
             const double* __restrict__ wall_old, int rule, uint32_t L, double* __restrict__ q,
             double* __restrict__ wall_u, uint32_t* __restrict__ bad) {
    const uint32_t k = blockIdx.x * BX + threadIdx.x;
    if (k >= L) return;
    const size_t pk = (size_t)(uint32_t)perm[k];
    const double g = q_in ? q_in[pk] : q_old[k];
    q[k] = g;
    for (int a = 0; a < D; ++a)
        wall_u[(size_t)k * D + a] = wall_in ? wall_in[pk * D + a] : wall_old[(size_t)k * D + a];
    if (!(g > 0.0 && g <= 1.0)) {
        atomicMin(&bad[0], k);
        return;
    }
    if (!l_convex(rule, g)) atomicMin(&bad[1], k);
}

// Coefficients of Eq. (213) for every link and their gamma derivatives along
// l = l(gamma), in double; bound by the tables written (88 bytes a link in
// FP32 handles).  Rounded operation by operation, as written.
template <class L, class T>
__global__ void __launch_bounds__(BX)
k_link_coefficients(const double* __restrict__ q, const double* __restrict__ wall_u,
                    const uint8_t* __restrict__ lkdir, const uint8_t* __restrict__ ibar_link,
                    int rule, double b, double rho0, int two_node, uint32_t n_links,
                    LinkCoefT<T>* __restrict__ coef, LinkDeriv* __restrict__ der,
                    double* __restrict__ c4v, double* __restrict__ c1d, double* __restrict__ d1d) {
#pragma clang fp contract(off)
    const uint32_t k = blockIdx.x * BX + threadIdx.x;
    if (k >= n_links) return;
    const double g = q[k];
    const double l = l_of(rule, g), lp = dl_of(rule, g);
    const double den = 1.0 + l;
    const double c1 = b * (1.0 + l - 2.0 * g) / den;
    const double c2 = b * l / den;
    const double c3 = b * (2.0 * g - l) / den;
    const double c4 = b * 2.0 / den;
    double ephi = 0.0, w = 0.0;
    const int dir = lkdir[k];
    unroll<L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (i == dir) {
            w = L::W[i];
            for (int a = 0; a < L::D; ++a)
                ephi += (double)L::E[i][a] * wall_u[(size_t)k * L::D + a];
        }
    });
    const double unit = 3.0 * w * rho0 * ephi;
    const double den2 = den * den;
    const double d1 = b * ((lp - 2.0) * den - (1.0 + l - 2.0 * g) * lp) / den2;
    const double d2 = b * lp / den2;
    const double d3 = b * ((2.0 - lp) * den - (2.0 * g - l) * lp) / den2;
    const double d4 = -2.0 * b * lp / den2;
    // Eq. (211): the c1 term multiplies f_ibar(x_f, t+1) = f'_ibar(x_f + e_i, t)
    // and is added at the next pull, unless x_f + e_i is solid
    const bool defer = two_node && !ibar_link[k];
    coef[k] = LinkCoefT<T>{(T)(defer ? 0.0 : c1), (T)c2, (T)c3, (T)(c4 * unit)};
    der[k] = LinkDeriv{defer ? 0.0 : d1, d2, d3, d4 * unit};
    c1d[k] = defer ? c1 : 0.0;
    d1d[k] = defer ? d1 : 0.0;
    c4v[k] = c4;
}

hipError_t launch_take_links(Engine& e, const double* q, const double* wall_u, uint32_t* bad) {
    if (!e.n_links) return hipSuccess;
    auto kern = e.D == 2 ? k_take_links<2> : k_take_links<3>;
    hipLaunchKernelGGL(kern, dim3((unsigned)link_blocks(e)), dim3(BX), 0, e.stream, q, wall_u, e.d_perm,
                       e.d_q, e.d_wall_u, e.l_rule, (uint32_t)e.n_links, e.d_q_next,
                       e.d_wall_u_next, bad);
    return hipGetLastError();
}

hipError_t launch_link_coefficients(Engine& e) {
    if (!e.n_links) return hipSuccess;
    auto go = [&](auto lat, auto* coef) -> hipError_t {
        using L = decltype(lat);
        using T = std::conditional_t<std::is_same<decltype(coef), LinkCoefT<float>*>::value, float, double>;
        hipLaunchKernelGGL((k_link_coefficients<L, T>), dim3((unsigned)link_blocks(e)), dim3(BX), 0,
                           e.stream, e.d_q, e.d_wall_u, e.d_lkdir, e.d_lkibar, e.l_rule, e.b, e.rho0,
                           e.two_node ? 1 : 0, (uint32_t)e.n_links, coef, e.d_lkderiv, e.d_lkc4,
                           e.d_lkc1d, e.d_lkd1d);
        return hipGetLastError();
    };
    auto by_lattice = [&](auto* coef) -> hipError_t {
        if (e.lattice == 0) return go(D2Q9{}, coef);
        if (e.lattice == 2) return go(D3Q15{}, coef);
        return go(D3Q19{}, coef);
    };
    return e.precision == 1 ? by_lattice(e.d_lkcoef_f) : by_lattice(e.d_lkcoef);
}

}  // namespace lbe
