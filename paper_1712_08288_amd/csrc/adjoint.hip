// Link kernels of the reverse sweep and its launches (the node kernel and the
// arithmetic of a reverse step: adjoint.hpp).
#include "adjoint.hpp"

namespace lbe {

// The pending reverse steps on records: step j's a_k run at ak[j L1], the
// link runs of its record at lk[j] and its wall-data factor ws[j], in the
// order the steps were taken.
template <class T>
struct AkBatch {
    const T* lk[kAkBatch];
    double ws[kAkBatch];
    int count;
};

// Their terms added to the two sums of every link, step by step in that
// order (the same additions, in the same order, as one step at a time):
// one thread per link, the sums and the coefficient derivatives read once.
// tq (Eq. (211) runs, else null): the pre-pass's gq term of each step, in
// the layout of ak.
template <class T>
__global__ void __launch_bounds__(BX)
k_link_sums(const double* __restrict__ ak, const double* __restrict__ tq, AkBatch<T> b,
            LinkGrad lg, uint32_t L) {
    const uint32_t k = blockIdx.x * BX + threadIdx.x;
    if (k >= L) return;
    const double d1 = lg.deriv[k].d1, d2 = lg.deriv[k].d2, d3 = lg.deriv[k].d3;
    double gq = lg.g[k], gs = lg.g[lg.L1 + k];
    for (int j = 0; j < b.count; ++j) {
        // Eq. (211): the pre-pass's term of step j comes first, as when the
        // pre-pass added it itself
        if (tq) gq += tq[(size_t)j * lg.L1 + k];
        const double a = ak[(size_t)j * lg.L1 + k];
        const T* __restrict__ lk = b.lk[j];
        gq += a * (d1 * (double)lk[k] + d2 * (double)lk[lg.L1 + k] +
                   d3 * (double)lk[2 * lg.L1 + k]);
        gs += a * b.ws[j];
    }
    lg.g[k] = gq;
    lg.g[lg.L1 + k] = gs;
}

// The gradients of every link from its two sums, in the caller's link
// order: dq[perm k] = gq_k + dwall_k gs_k and
// dphi[perm k][a] = c4_k 3 w_i rho0 e_ia gs_k (either output may be null).
template <class L>
__global__ void __launch_bounds__(BX)
k_link_finish(const double* __restrict__ gq, const double* __restrict__ gs,
              const LinkDeriv* __restrict__ deriv, const double* __restrict__ lkc4,
              const uint8_t* __restrict__ lkdir, const int32_t* __restrict__ perm,
              double rho0, uint32_t n_links, double* __restrict__ dq,
              double* __restrict__ dphi) {
    const uint32_t k = blockIdx.x * BX + threadIdx.x;
    if (k >= n_links) return;
    const size_t pk = (size_t)(uint32_t)perm[k];
    if (dq) dq[pk] = gq[k] + deriv[k].dwall * gs[k];
    if (dphi) {
        int e[3] = {0, 0, 0}, ib = 0;
        double w = 0.0;
        dir_data<L>(lkdir[k], e, w, ib);
        const double c = lkc4[k] * 3.0 * w * rho0 * gs[k];
#pragma unroll
        for (int al = 0; al < L::D; ++al) dphi[pk * L::D + al] = c * e[al];
    }
}

// Eq. (211) links k = (x_f, i) with a deferred c1: the link value is
// f_i(x_f, t+1) = (terms at t) + c1 f_ibar(x_f, t+1), so its adjoint a_k also
// reaches f_ibar(x_f, t+1) (whose own adjoint the node x_f + e_i gathers in
// the next kernel) and dJ/dgamma gets a_k dc1 f_ibar(x_f, t+1).  That value
// is pulled from the state at t+1 (A_next), or read from fib_next (the
// link values of the step record of t+1, or of the run's final state).
template <class L, class T, int XB>
__global__ void __launch_bounds__(BX)
k_two_node_pre(const T* __restrict__ A_next, const T* __restrict__ fib_next,
               T* __restrict__ lam_in,
               const int32_t* __restrict__ lknode, const uint8_t* __restrict__ lkdir,
               const int32_t* __restrict__ lktag, const double* __restrict__ c1d,
               const double* __restrict__ d1d, double* __restrict__ gq, int store,
               uint32_t n_links, Grid g, Params<L, T> p, AdjArgs a) {
    const uint32_t k = blockIdx.x * BX + threadIdx.x;
    if (k >= n_links) return;
    const double c = c1d[k];
    if (c == 0.0) {
        if (store) gq[k] = 0.0;
        return;
    }
    const int i = lkdir[k];
    const uint32_t n = (uint32_t)lknode[k];
    int ib = 0, ex = 0;
    unroll<L::Q>([&](auto I) {
        constexpr int ii = decltype(I)::value;
        if (ii == i) {
            ib = TAB<L>.opp[ii];
            ex = L::E[ii][0];
        }
    });
    double ak = (double)ldp<L::Q>(lam_in, i, n);
    if (a.obj_kind == 1 && ex != 0 && lktag[k] == a.obj_tag) ak += -(double)ex * a.w_force;
    T* dst = lam_in + pop_at<L::Q>(ib, n);
    *dst = (T)((double)*dst + c * ak);
    const T fib = fib_next ? fib_next[k] : pull_one<L, T, XB>(A_next, g, p, n, ib);
    // store: the step's run of terms that k_link_sums adds (record sweeps)
    if (store)
        gq[k] = ak * d1d[k] * (double)fib;
    else
        gq[k] += ak * d1d[k] * (double)fib;
}

// The value f_ibar(x_f, t) that the pull of the opposite direction reads at
// each link's node from the state A (for Eq. (211) links the plain pull:
// their opposite direction is no cut link), into out[k].
template <class L, class T, int XB>
__global__ void __launch_bounds__(BX)
k_link_pull(const T* __restrict__ A, const int32_t* __restrict__ lknode,
            const uint8_t* __restrict__ lkdir, uint32_t n_links, Grid g, Params<L, T> p,
            T* __restrict__ out) {
    const uint32_t k = blockIdx.x * BX + threadIdx.x;
    if (k >= n_links) return;
    int ib = 0;
    const int i = lkdir[k];
    unroll<L::Q>([&](auto I) {
        constexpr int ii = decltype(I)::value;
        if (ii == i) ib = TAB<L>.opp[ii];
    });
    out[k] = pull_one<L, T, XB>(A, g, p, (uint32_t)lknode[k], ib);
}

template <class L, class T>
__global__ void __launch_bounds__(BX)
k_adjoint_out(const T* __restrict__ lam, const uint32_t* __restrict__ info,
              uint32_t N, double* __restrict__ out) {
    const uint32_t n = blockIdx.x * BX + threadIdx.x;
    if (n >= N) return;
    const bool fluid = !is_solid(info[n]);
    for (int i = 0; i < L::Q; ++i)
        out[(size_t)i * N + n] = fluid ? (double)ldp<L::Q>(lam, i, n) : 0.0;
}

// ----------------------------------------------------------------------------

static uint32_t wave_blocks(int64_t waves) { return (uint32_t)((waves + BX / 64 - 1) / (BX / 64)); }

int64_t adjoint_blocks(const Engine& e) {
    return std::max<int64_t>(1, (int64_t)wave_blocks(e.n_wact));
}

hipError_t launch_adjoint_step(Engine& e, const Snapshot* fwd, const Snapshot* next,
                               const void* rec, const void* lam_in, void* lam_out,
                               const AdjointObjective& obj) {
    AdjArgs a;
    a.obj_kind = obj.kind;
    a.obj_tag = obj.tag;
    a.w_force = obj.kind == 1 ? obj.weight : 0.0;
    a.w_ux = obj.kind == 2 ? obj.weight * obj.inv_nfluid / e.rho0 : 0.0;
    a.want_ds = e.want_ds ? 1 : 0;
    a.x_in = obj.x_in;
    a.x_out = obj.x_out;
    a.a_in = obj.kind == 3 ? obj.weight * obj.a_in / 3.0 : 0.0;
    a.a_out = obj.kind == 3 ? obj.weight * obj.a_out / 3.0 : 0.0;
    const bool um = rec != nullptr && !a.want_ds;
    if (!um && (!fwd || !next)) return hipErrorInvalidValue;
    const size_t L1 = (size_t)std::max<int64_t>(e.n_links, 1);
    if (um && !e.ak_buf) return hipErrorInvalidValue;
    if (um && e.ak_pending == kAkBatch) {
        const hipError_t fs = launch_link_sums(e);
        if (fs != hipSuccess) return fs;
    }
    const LinkGrad lgr{e.d_lkderiv, um ? e.ak_buf + (size_t)e.ak_pending * L1 : e.d_gq, (uint32_t)L1};
    const AdjointLaunch al{um ? nullptr : fwd, um ? nullptr : next, um ? rec : nullptr,
                           lam_in, lam_out, lgr, a};
    const hipError_t st = e.lattice == 0   ? launch_adjoint_nodes<D2Q9>(e, al)
                          : e.lattice == 2 ? launch_adjoint_nodes<D3Q15>(e, al)
                                           : launch_adjoint_nodes<D3Q19>(e, al);
    if (st != hipSuccess || !um || !e.n_links) return st;
    // a link with no fluid node in an active wave cannot exist, so every
    // a_k of the run was written
    e.ak_rec[e.ak_pending] = rec;
    e.ak_ws[e.ak_pending] = e.wall_scale;
    ++e.ak_pending;
    return hipSuccess;
}

hipError_t launch_link_sums(Engine& e) {
    if (e.ak_pending == 0) return hipSuccess;
    const int count = e.ak_pending;
    e.ak_pending = 0;
    const uint32_t L1 = (uint32_t)std::max<int64_t>(e.n_links, 1);
    const LinkGrad lgr{e.d_lkderiv, e.d_gq, L1};
    const unsigned nb = (unsigned)((e.n_links + BX - 1) / BX);
    auto go = [&](auto prec) -> hipError_t {
        using T = decltype(prec);
        AkBatch<T> b{};
        for (int j = 0; j < count; ++j) {
            b.lk[j] = record_at<T>(e, e.ak_rec[j]).fib;
            b.ws[j] = e.ak_ws[j];
        }
        b.count = count;
        hipLaunchKernelGGL((k_link_sums<T>), dim3(nb), dim3(BX), 0, e.stream, e.ak_buf,
                           e.two_node ? (const double*)e.tq_buf : nullptr, b, lgr,
                           (uint32_t)e.n_links);
        return hipGetLastError();
    };
    return e.precision == 1 ? go(float{}) : go(double{});
}

hipError_t launch_link_gradients(Engine& e, double* dq, double* dphi) {
    if (!e.n_links || (!dq && !dphi)) return hipSuccess;
    auto go = [&](auto lat) {
        using L = decltype(lat);
        hipLaunchKernelGGL((k_link_finish<L>), dim3((unsigned)((e.n_links + BX - 1) / BX)),
                           dim3(BX), 0, e.stream, e.d_gq, e.d_gs, e.d_lkderiv, e.d_lkc4,
                           e.d_lkdir, e.d_perm, e.rho0, (uint32_t)e.n_links, dq, dphi);
        return hipGetLastError();
    };
    if (e.lattice == 0) return go(D2Q9{});
    if (e.lattice == 2) return go(D3Q15{});
    return go(D3Q19{});
}

hipError_t launch_two_node_adjoint(Engine& e, const Snapshot* next, const void* fib_next,
                                   void* lam_in, const AdjointObjective& obj) {
    if (e.n_links == 0) return hipSuccess;
    const Grid g = make_grid(e);
    AdjArgs a;
    a.obj_kind = obj.kind;
    a.obj_tag = obj.tag;
    a.w_force = obj.kind == 1 ? obj.weight : 0.0;
    a.w_ux = 0.0;
    a.want_ds = 0;
    a.x_in = a.x_out = 0u;
    a.a_in = a.a_out = 0.0;
    const unsigned nb = (unsigned)((e.n_links + BX - 1) / BX);
    // on records (fib_next given) the term goes into the step's run of
    // tq_buf, the run the following launch_adjoint_step fills in ak_buf
    const bool store = fib_next != nullptr;
    if (store && !e.tq_buf) return hipErrorInvalidValue;
    if (store && e.ak_pending == kAkBatch) {
        const hipError_t fs = launch_link_sums(e);
        if (fs != hipSuccess) return fs;
    }
    double* gq = store ? e.tq_buf + (size_t)e.ak_pending * (size_t)std::max<int64_t>(e.n_links, 1)
                       : e.d_gq;
    return dispatch(e, [&](auto lat, auto prec, auto xb) -> hipError_t {
        using L = decltype(lat);
        using T = decltype(prec);
        constexpr int XB = decltype(xb)::value;
        hipLaunchKernelGGL((k_two_node_pre<L, T, XB>), dim3(nb), dim3(BX), 0, e.stream,
                           next ? (const T*)next->f : nullptr, (const T*)fib_next,
                           (T*)lam_in, e.d_lknode, e.d_lkdir, e.d_lktag,
                           e.d_lkc1d, e.d_lkd1d, gq, store ? 1 : 0, (uint32_t)e.n_links, g,
                           make_params<L, T>(e), a);
        return hipGetLastError();
    });
}

hipError_t launch_link_pull(Engine& e, const Snapshot& s, void* out) {
    if (e.n_links == 0) return hipSuccess;
    const Grid g = make_grid(e);
    const unsigned nb = (unsigned)((e.n_links + BX - 1) / BX);
    return dispatch(e, [&](auto lat, auto prec, auto xb) -> hipError_t {
        using L = decltype(lat);
        using T = decltype(prec);
        constexpr int XB = decltype(xb)::value;
        hipLaunchKernelGGL((k_link_pull<L, T, XB>), dim3(nb), dim3(BX), 0, e.stream,
                           (const T*)s.f, e.d_lknode, e.d_lkdir, (uint32_t)e.n_links, g,
                           make_params<L, T>(e), (T*)out);
        return hipGetLastError();
    });
}

hipError_t launch_adjoint_out(Engine& e, const void* lam, double* out) {
    const unsigned nb = (unsigned)((e.N + BX - 1) / BX);
    return dispatch(e, [&](auto lat, auto prec, auto) -> hipError_t {
        using L = decltype(lat);
        using T = decltype(prec);
        hipLaunchKernelGGL((k_adjoint_out<L, T>), dim3(nb), dim3(BX), 0, e.stream,
                           (const T*)lam, e.d_info, (uint32_t)e.N, out);
        return hipGetLastError();
    });
}

}  // namespace lbe
