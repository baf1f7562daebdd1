// single.hpp - a cube's solve by one workgroup, for n <= 8: the whole padded
// intermediate fits a CU's LDS and every column of a pass a thread group, so
// the five passes run one after another with workgroup barriers between
// them.  Bound by launches and latency: one launch in place of three (FP64,
// us per solve in a row: n = 4 13.5 -> 4.6, n = 8 13.6 -> 6.8; five launches
// took 20).  At n = 12 the i1 columns take two rounds and one CU needs 16.8
// us, longer than the three launches' 12.6.  Each transform has the plan,
// twiddles and order of operations of its pass kernel, so results are bitwise
// theirs.  A batch whose outputs overlap inputs of other members of the same
// size takes the five passes (feeds_another): workgroups of one launch have
// no order.
#pragma once
#include "passes.hpp"

namespace psp {

template <typename T, int N> struct SingleCfg {
    static constexpr int n = N / 2, K = n + 1, TPC = N / MaxRadix<N, 0>::value();
    static constexpr int THREADS = (N * K * TPC + 63) / 64 * 64;    // the i1 columns (k2, k3), the most of any pass
    static constexpr int C = THREADS / TPC;
    static_assert(THREADS <= 1024, "workgroup");
};

template <typename T, int N>
__global__ void __launch_bounds__((SingleCfg<T, N>::THREADS))
k_single(JobRef jr, Twiddle<T> tw) {
    using V2 = cplx<T>;
    using Cfg = SingleCfg<T, N>;
    using EF = Engine<T, N, Cfg::TPC, false, 0>;
    using EI = Engine<T, N, Cfg::TPC, true, 0>;
    constexpr int n = Cfg::n, K = Cfg::K, C = Cfg::C, PAIRS = n * n / 2, P = ((n + 1 + 15) / 16) * 16;
    __shared__ V2 X[n * n * K], A[n * N * K], xch[C * N], roots[N];
    const Job jb = jr.get();
    const int col = threadIdx.x % C, t = threadIdx.x / C;
    const bool on = t < Cfg::TPC;       // the threads beyond C TPC have no column
    const int i1 = col / K, k3 = col % K;
    const bool lines = on && col < PAIRS, cols = on && col < n * K;

    // every global read at the start: the roots, rho, the multiplier
    for (int e = threadIdx.x; e < N; e += Cfg::THREADS) {
        const double2 w = g_load(&tw.w[e]);
        roots[e] = V2{T(w.x), T(w.y)};
    }
    V2 v[EF::V > EI::V ? EF::V : EI::V];
    const T *ra = (const T *)jb.rho + (size_t)(2 * col) * n, *rb = ra + n;
    EF::for_inputs(v, t, [&](int pos, int r) -> V2 {
        if (r < EF::R(0) / 2 && lines) return V2{g_load(&ra[pos]), g_load(&rb[pos])};
        return c_zero<V2>();
    });
    const bool modes = on && col < N * K;
    double m[EF::V];
    {
        const int k2 = col / K, b = k2 <= n ? k2 : N - k2;
        const double *row = jb.mult + MultAt{true, P, n + 1}(0, b, k3);
        int i = 0;
        EF::for_outputs(v, t, [&](int pos, int, V2 &) {
            const int a = pos <= n ? pos : N - pos;
            m[i++] = modes ? g_load(&row[a]) : 0.0;
        });
    }
    __syncthreads();
    const TableTwiddle<T, N> tab{roots};
    // the line passes form FP64 powers by trees of a root
    const auto line_tw = [&] {
        if constexpr (sizeof(T) == 8) return Twiddle<double>{roots};
        else return TableTwiddle<float, N>{roots};
    }();
    const IdxInter<C> idx{col};
    auto slot = [&](int pos) { return pos * C + col; };

    // H1
    if (on) EF::template compute<0>(v, t, line_tw);
    auto rest = [&](auto engine, const auto &twx) {    // the stages after the first
        using E = decltype(engine);
        static_assert(E::S == 2, "two stages");
        if (on) E::template store_lds<0>(v, xch, t, idx);
        __syncthreads();
        if (on) E::template load_lds<1>(v, xch, t, idx);
        __syncthreads();
        if (on) E::template compute<1>(v, t, twx);
    };
    rest(EF{}, line_tw);
    if (on) EF::for_outputs(v, t, [&](int pos, int, V2 &val) { xch[slot(pos)] = val; });
    __syncthreads();
    for (int it = threadIdx.x; it < PAIRS * K; it += Cfg::THREADS) {
        const int p = it % PAIRS, k = it / PAIRS;
        const V2 z = xch[k * C + p], zc = xch[(k == 0 ? 0 : N - k) * C + p];
        const V2 d = V2{z.x - zc.x, z.y + zc.y};
        X[2 * p * K + k] = V2{T(0.5) * (z.x + zc.x), T(0.5) * (z.y - zc.y)};
        X[(2 * p + 1) * K + k] = V2{T(0.5) * d.y, -T(0.5) * d.x};
    }
    __syncthreads();
    // H2
    if (on) {
        EF::for_inputs(v, t, [&](int pos, int r) -> V2 {
            if (r < EF::R(0) / 2 && cols) return X[(i1 * n + pos) * K + k3];
            return c_zero<V2>();
        });
        EF::template compute<0>(v, t, tab);
    }
    rest(EF{}, tab);
    if (cols) EF::for_outputs(v, t, [&](int pos, int, V2 &val) { A[(i1 * N + pos) * K + k3] = val; });
    __syncthreads();
    // H3, column (k2, k3)
    if (on) {
        EF::for_inputs(v, t, [&](int pos, int r) -> V2 {
            if (r < EF::R(0) / 2 && modes) return A[pos * N * K + col];
            return c_zero<V2>();
        });
        EF::template compute<0>(v, t, tab);
    }
    rest(EF{}, tab);
    if (on) {
        int i = 0;
        EF::for_outputs(v, t, [&](int, int, V2 &val) { val = scale_mode(val, m[i++]); });
        EI::template compute<0>(v, t, tab);
    }
    rest(EI{}, tab);
    if (modes)
        EI::for_outputs(v, t, [&](int pos, int r, V2 &val) {
            if (r < EI::R(EI::S - 1) / 2) A[pos * N * K + col] = val;
        });
    __syncthreads();
    // H4
    if (on) {
        EI::for_inputs(v, t, [&](int pos, int) -> V2 { return cols ? A[(i1 * N + pos) * K + k3] : c_zero<V2>(); });
        EI::template compute<0>(v, t, tab);
    }
    rest(EI{}, tab);
    if (cols)
        EI::for_outputs(v, t, [&](int pos, int r, V2 &val) {
            if (r < EI::R(EI::S - 1) / 2) X[(i1 * n + pos) * K + k3] = val;
        });
    __syncthreads();
    // H5
    for (int it = threadIdx.x; it < PAIRS * K; it += Cfg::THREADS) {
        const int p = it % PAIRS, k = it / PAIRS;
        V2 a = X[2 * p * K + k], b = X[(2 * p + 1) * K + k];
        if (k == 0 || k == n) {
            a.y = 0;
            b.y = 0;
        }
        xch[k * C + p] = V2{a.x - b.y, a.y + b.x};
        if (k != 0 && k != n) xch[(N - k) * C + p] = V2{a.x + b.y, b.x - a.y};
    }
    __syncthreads();
    if (on) EI::template load_lds<0>(v, xch, t, idx);
    __syncthreads();
    if (on) EI::template compute<0>(v, t, line_tw);
    rest(EI{}, line_tw);
    if (lines) {
        T *ua = (T *)jb.u + (size_t)(2 * col) * n, *ub = ua + n;
        EI::for_outputs(v, t, [&](int pos, int r, V2 &val) {
            if (r < EI::R(EI::S - 1) / 2) {
                g_store(&ua[pos], val.x);
                g_store(&ub[pos], val.y);
            }
        });
    }
}

}  // namespace psp
