// fused.hpp - a cube's solve in three launches instead of five, for the
// sizes whose tiles fit a workgroup's LDS.
//
// The i2 transform of length N = R M (R the first radix of its plan, M the
// product of the others) splits into a radix-R stage over the rows i2 = j +
// s M, s < R (Stockham's first stage, which needs no twiddles), and M-point
// transforms over j for each residue r = k2 mod R.  The inverse, which runs
// the radices in reverse, splits the same way: M-point transforms for each
// residue, then one radix-R stage over the residues.  So
//   F1 k_f_fwd : H1 and the radix-R stage of H2 (a workgroup transforms the
//                R/2 nonzero rows of J consecutive j along i3, then combines
//                them per k3);
//   F2 k_f_mid : the M-point transforms, H3, the inverse M-point transforms
//                (a workgroup holds all i1 and j of one residue r and k3);
//   F3 k_f_inv : the radix-R stage of H4 and H5.
// The i3 half spectra never go to memory: the solve moves 19 instead of 27
// real arrays of n^3 values.  Every butterfly has the inputs, twiddles and
// order of operations of the five-pass kernels, so results are bitwise
// theirs.  These sizes are bound by launches (three empty ones in a row take
// 7.5 us) and by the chain of latencies inside each kernel (times of both
// routes at every length beside fused_length).  Large ones are bound by F2
// (39 of 72 us at n = 128 FP64), whose exchanges go through LDS; k_f_midw,
// which does two of six in registers, took it from 59 us.
//
// A holds R (n + 1) blocks [r][k3] of n rows i1 of M columns j (block pitch
// FusedGeo::BLK): F2 reads and writes whole blocks, F1 and F3 touch J
// consecutive columns of one row of every block.
#pragma once
#include "passes.hpp"
#include "single.hpp"

namespace psp {

template <int N, int PY> struct FusedGeo {
    static constexpr int n = N / 2, R = Plan<N, PY>::r[0], M = N / R;
    // block pitch in elements: from 4 KB on an odd number of 128-byte lines,
    // so that the same row of successive blocks does not fall on one memory
    // channel
    template <typename T> static constexpr size_t blk() {
        const size_t e = sizeof(cplx<T>), lines = (n * M * e + 127) / 128;
        return n * M * e < 4096 ? n * M : (lines | 1) * 128 / e;
    }
};

// Stages 1.. of the length-N transform of plan PV (INV: stages 0..S-2 of the
// inverse) as an M-point Stockham transform on sub-positions p of the
// positions r + R p of one residue r.
template <int N, int PV, bool INV> struct SubSeq {
    using P = Plan<N, PV>;
    static constexpr int S = P::S - 1, R0 = P::r[0], M = N / R0;
    __host__ __device__ static constexpr int radix(int s) { return INV ? P::r[P::S - 1 - s] : P::r[s + 1]; }
    __host__ __device__ static constexpr int ns(int s) {
        int p = 1;
        for (int i = 0; i < s; ++i) p *= radix(i);
        return p;
    }
    // twiddle and DFT of butterfly g (of M / radix) of residue r
    template <int s, typename C, typename TW>
    __device__ __forceinline__ static void butterfly(C *w, int g, int r, const TW &tw) {
        constexpr int rad = radix(s), nm = ns(s);
        if constexpr (!INV) {
            constexpr int stride = N / (R0 * nm * rad);
            tw.template apply<rad, false>(w, (r + R0 * (g % nm)) * stride);
        } else if constexpr (nm > 1) {
            constexpr int stride = N / (nm * rad);
            tw.template apply<rad, true>(w, (g % nm) * stride);
        }
        DFT<rad, INV, C>::run(w);
    }
    template <int s> __device__ __forceinline__ static int in_pos(int g, int q) { return g + q * (M / radix(s)); }
    template <int s> __device__ __forceinline__ static int out_pos(int g, int q) {
        constexpr int rad = radix(s), nm = ns(s);
        return (g / nm) * nm * rad + g % nm + q * nm;
    }
};

// Tile of the fused kernels: J columns per workgroup of F1 and F3, KU bins
// per thread and round of F3, NB blocks per workgroup of F2.
template <typename T, int N> struct FusedCfg {
    static constexpr int J = N == 36 ? 2 : N == 108 ? 6 : N == 144 ? 12 : N == 256 ? 8 : N == 192 ? (sizeof(T) == 8 ? 12 : 8) : 4;
    static constexpr int KU = N == 144 || N == 256 ? 1 : N == 192 ? 2 : 3;
    // J of F1 and of F3, KU of F3, with several solves per launch: there are
    // workgroups enough for wider rows of A (us per solve of a batch against
    // the tiles of one solve, when chosen: n = 64 7.34 -> 7.16, FP32 4.69 ->
    // 4.38; n = 128 FP32 40.1 -> 37.9; n = 72, which has only these, 15.7 -> 15.0)
    static constexpr int J1M = N == 128 ? 8 : N == 256 && sizeof(T) == 4 ? 16 : J;
    static constexpr int J3M = N == 128 ? 8 : N == 192 && sizeof(T) == 8 ? 4 : J;
    static constexpr int KUM = N == 128 ? 2 : N == 192 && sizeof(T) == 8 ? 3 : KU;
    static constexpr int NB = N <= 32 ? 4 : N == 36 ? 2 : 1;
    // the 17 MB of A of one solve at n = 64 FP64 written and read past the
    // caches: three launches 2.5 us faster (26.7 -> 24.2 when chosen; other
    // sizes and several solves in one launch lose by it, n = 128 74 -> 84 us)
    static constexpr bool NT = N == 128 && sizeof(T) == 8;
    // whether the plans fit k_f_midw
    static constexpr bool W = N == 128 || N == 192 || N == 256;
};

// consecutive work items on one XCD (workgroups go to the 8 XCDs in turn):
// neighbours share lines of A or a plane of the multiplier in that XCD's L2
__device__ __forceinline__ int xcd_item(int g, int blocks) { return (g % 8) * (blocks / 8) + g / 8; }
inline int xcd_blocks(int items) { return (items + 7) / 8 * 8; }

// the two halves of a pair of lanes exchange a value
__device__ __forceinline__ double lane_xor1(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_xor1(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));
}

// lines of F1 and F3: J consecutive j, their R/2 nonzero (kept) rows, two
// adjacent rows per complex line
template <typename T, int N, int PZ, int PY, int J> struct FusedLines {
    using G = FusedGeo<N, PY>;
    static constexpr int TPC = N / MaxRadix<N, PZ>::value();
    static constexpr int Q = J * G::R / 4;
    static constexpr int THREADS = TPC * Q;
    static constexpr int LINE = N + N / 8;
    static constexpr int GROUPS = G::M / J;
    static_assert(J % 2 == 0 && G::M % J == 0 && G::R % 2 == 0 && THREADS % J == 0 && THREADS % 2 == 0, "tile");
    static_assert(THREADS <= 1024, "workgroup");
};

// The line transforms' twiddles in F1 and F3: the values the five-pass line
// kernels use (FP64: power trees of a root; FP32: the rounded roots, or the
// rounded trees, equal to them), the roots read from a copy in LDS that is
// fetched along with the inputs.  A tree's root read from global memory at
// each stage put a cache miss between the stages of these short kernels.
template <typename T, int N> struct FusedTw {
    using Elem = double2;
    using Src = Twiddle<double>;
};
template <int N> struct FusedTw<float, N> {
    using Elem = float2;
    using Src = TableTwiddle<float, N>;
};
template <typename T, int N, int THREADS> struct FusedTwFetch {
    static constexpr int K = (N + THREADS - 1) / THREADS;
    double2 w[K];
    __device__ __forceinline__ explicit FusedTwFetch(const Twiddle<T> &tw) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = (int)threadIdx.x + k * THREADS;
            if (N % THREADS == 0 || e < N) w[k] = g_load(&tw.w[e]);
        }
    }
    // stores the roots; the caller's next barrier publishes them
    __device__ __forceinline__ typename FusedTw<T, N>::Src commit(typename FusedTw<T, N>::Elem *buf) const {
        using E = typename FusedTw<T, N>::Elem;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = (int)threadIdx.x + k * THREADS;
            if (N % THREADS == 0 || e < N) buf[e] = E{T(w[k].x), T(w[k].y)};
        }
        return typename FusedTw<T, N>::Src{buf};
    }
};

// ------------------------------------------------------------------- F1
template <typename T, int N, int PZ, int PY, int J, int CP>
__global__ void __launch_bounds__((FusedLines<T, N, PZ, PY, J>::THREADS))
k_f_fwd(JobRef jr, Twiddle<T> tw) {
    using C = cplx<T>;
    using G = FusedGeo<N, PY>;
    using F = FusedLines<T, N, PZ, PY, J>;
    using E = Engine<T, N, F::TPC, false, PZ>;
    constexpr int n = N / 2, R = G::R, M = G::M;
    constexpr size_t BLK = G::template blk<T>();
    __shared__ C lds[F::Q * F::LINE + N];
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (item >= n * F::GROUPS) return;              // uniform over the workgroup
    const FusedTwFetch<T, N, F::THREADS> twf(tw);
    const Job jb = jr.get();
    const int i1 = item / F::GROUPS, j0 = (item % F::GROUPS) * J;
    const int t = threadIdx.x % F::TPC, q = threadIdx.x / F::TPC;
    const int row = j0 + 2 * (q % (J / 2)) + (q / (J / 2)) * M;   // i2 of the pair's first line
    const T *ra = (const T *)jb.rho + ((size_t)i1 * n + row) * n;
    const T *rb = ra + n;
    C v[E::V];
    E::for_inputs(v, t, [&](int pos, int r) -> C {
        if (r < E::R(0) / 2) return C{g_load(&ra[pos]), g_load(&rb[pos])};
        return c_zero<C>();
    });
    const auto twx = twf.commit(lds + F::Q * F::LINE);   // published by the first exchange
    IdxLine idx{q * F::LINE};
    E::template run_from<0>(v, lds, t, idx, twx);
    E::for_outputs(v, t, [&](int pos, int, C &val) { lds[idx(pos)] = val; });
    __syncthreads();
    const int j = threadIdx.x % J;                  // THREADS is a multiple of J
    C *dst = (C *)jb.A + (size_t)i1 * M + j0 + j;
    for (int k = threadIdx.x / J; k <= n; k += F::THREADS / J) {
        C w[R];
#pragma unroll
        for (int s = 0; s < R / 2; ++s) {
            IdxLine ix{(s * (J / 2) + j / 2) * F::LINE};
            const C z = lds[ix(k)], zc = lds[ix(k == 0 ? 0 : N - k)];
            if (j & 1)
                w[s] = C{T(0.5) * (z.y + zc.y), -T(0.5) * (z.x - zc.x)};
            else
                w[s] = C{T(0.5) * (z.x + zc.x), T(0.5) * (z.y - zc.y)};
        }
#pragma unroll
        for (int s = R / 2; s < R; ++s) w[s] = c_zero<C>();
        DFT<R, false, C>::run(w);
#pragma unroll
        for (int r = 0; r < R; ++r) a_store<CP>(&dst[(size_t)(r * (n + 1) + k) * BLK], w[r]);
    }
}

// ------------------------------------------------------------------- F2
// NB blocks per workgroup: W = NB M columns (r, k3, k2 = r + R p) of i1
// transforms, TPC threads each (consecutive threads along i1, so that the
// multiplier, whose rows |k1| of one (|k2|, k3) are contiguous for these
// sizes, is read coalesced).  LDS holds a column contiguously with a pad
// slot per 8 positions and an odd pitch: conflict-free both along a column
// (i1 stages) and across columns (M-point stages).
template <typename T, int N, int PY, int PX, int NB> struct FusedMid {
    using G = FusedGeo<N, PY>;
    static constexpr int W = NB * G::M;
    static constexpr int TPC = N / MaxRadix<N, PX>::value(), THREADS = TPC * W;
    // pitch of a column in the i1 exchange buffer and in the M-point stages'
    // (which uses the same memory)
    static constexpr int LINE = (N * 9 / 8) | 1;
    static constexpr int MLINE = (N / 2 * 9 / 8) | 1;
    static constexpr int ELEMS = W * LINE;
    static constexpr int BLOCKS = G::R * (N / 2 + 1);
    static_assert(THREADS <= 1024, "workgroup");
};

template <typename T, int N, int PY, int PX, int NB, int CP>
__global__ void __launch_bounds__((FusedMid<T, N, PY, PX, NB>::THREADS))
k_f_mid(JobRef jr, Twiddle<T> tw) {
    using C = cplx<T>;
    using G = FusedGeo<N, PY>;
    using F = FusedMid<T, N, PY, PX, NB>;
    using SF = SubSeq<N, PY, false>;
    using SI = SubSeq<N, PY, true>;
    using EF = Engine<T, N, F::TPC, false, PX>;
    using EI = Engine<T, N, F::TPC, true, PX>;
    constexpr int n = N / 2, R = G::R, M = G::M, TH = F::THREADS, P = ((n + 1 + 15) / 16) * 16;
    constexpr size_t BLK = G::template blk<T>();
    __shared__ C lds[F::ELEMS + N];
    const int wg = xcd_item(blockIdx.x, gridDim.x);
    if (wg * NB >= F::BLOCKS) return;               // uniform over the workgroup
    const auto twf = tw_fetch<T, N, TH, true>(tw);
    const Job jb = jr.get();
    C *A = (C *)jb.A;

    // block b of the workgroup: residue and k3 (all residues of one k3 are
    // neighbours: they read the same plane of the multiplier)
    auto block_r = [&](int b) { return (wg * NB + b) % R; };
    auto block_k3 = [&](int b) { return (wg * NB + b) / R; };
    auto block_on = [&](int b) { return NB == 1 || wg * NB + b < F::BLOCKS; };
    auto block_at = [&](int b) { return A + (size_t)(block_r(b) * (n + 1) + block_k3(b)) * BLK; };
    auto slot = [&](int col, int pos) { return col * F::MLINE + pos + (pos >> 3); };

    // the items of an M-point stage of radix rad: butterfly g of row i1 of block b
    auto items = [&](auto rad, auto &&f) {
        constexpr int per = M / decltype(rad)::value, IT = n * NB * per, BP = (IT + TH - 1) / TH;
#pragma unroll
        for (int i = 0; i < BP; ++i) {
            const int it = (int)threadIdx.x + i * TH;
            const int g = it % per, row = (it / per) % n, b = it / (per * n);
            if (IT % TH == 0 || it < IT) f(i, g, row, b);
        }
    };
    constexpr int VM = [] {
        int m = 0;
        for (int s = 0; s < SF::S; ++s) {
            const int a = (n * NB * (M / SF::radix(s)) + TH - 1) / TH * SF::radix(s);
            m = a > m ? a : m;
        }
        return m;
    }();
    TableTwiddle<T, N> twx;
    {
        C w[VM];
        // forward M-point transforms; the first stage reads the block
        items(std::integral_constant<int, SF::radix(0)>{}, [&](int i, int g, int row, int b) {
            constexpr int rad = SF::radix(0);
            const C *src = block_at(b) + (size_t)row * M;
#pragma unroll
            for (int q = 0; q < rad; ++q)
                w[i * rad + q] = block_on(b) ? a_load<CP>(&src[SF::template in_pos<0>(g, q)]) : c_zero<C>();
        });
        twx = tw_commit<T, N, TH, true>(tw, twf, lds + F::ELEMS);
        auto stage = [&](auto sc) {
            constexpr int s = decltype(sc)::value, rad = SF::radix(s);
            items(std::integral_constant<int, rad>{}, [&](int i, int g, int row, int b) {
                if constexpr (s > 0) {
#pragma unroll
                    for (int q = 0; q < rad; ++q) w[i * rad + q] = lds[slot(b * M + SF::template in_pos<s>(g, q), row)];
                }
                SF::template butterfly<s>(w + i * rad, g, block_r(b), twx);
            });
            if constexpr (s > 0) __syncthreads();
            items(std::integral_constant<int, rad>{}, [&](int i, int g, int row, int b) {
#pragma unroll
                for (int q = 0; q < rad; ++q) lds[slot(b * M + SF::template out_pos<s>(g, q), row)] = w[i * rad + q];
            });
            __syncthreads();
        };
        stage(std::integral_constant<int, 0>{});
        if constexpr (SF::S > 1) stage(std::integral_constant<int, 1>{});
        if constexpr (SF::S > 2) stage(std::integral_constant<int, 2>{});
        static_assert(SF::S >= 1 && SF::S <= 3, "stages");
    }
    // i1: forward, multiply, inverse, cropped
    {
        const int t = threadIdx.x % F::TPC, col = threadIdx.x / F::TPC;
        const int b = col / M, r = block_r(b), c3 = block_k3(b);
        const int k2 = r + R * (col % M), bk = k2 <= n ? k2 : N - k2;
        C v[EF::V];
        EF::for_inputs(v, t, [&](int pos, int leg) -> C {
            if (leg < EF::R(0) / 2) return lds[slot(col, pos)];
            return c_zero<C>();
        });
        __syncthreads();
        const IdxLine idx{col * F::LINE};
        EF::template run_from<0>(v, lds, t, idx, twx);
        const double *mrow = jb.mult + ((size_t)bk * P + c3) * (n + 1);
        EF::for_outputs(v, t, [&](int pos, int leg, C &val) {
            constexpr int RL = EF::R(EF::S - 1);
            const int a = (RL % 2 == 0) ? (leg < RL / 2 ? pos : N - pos) : (pos <= n ? pos : N - pos);
            val = scale_mode(val, block_on(b) ? g_load(&mrow[a]) : 0.0);
        });
        EI::template run_from<0>(v, lds, t, idx, twx);
        EI::for_outputs(v, t, [&](int pos, int leg, C &val) {
            if (leg < EI::R(EI::S - 1) / 2) lds[slot(col, pos)] = val;
        });
        __syncthreads();
    }
    // inverse M-point transforms; the last stage writes the block
    {
        C w[VM];
        auto stage = [&](auto sc) {
            constexpr int s = decltype(sc)::value, rad = SI::radix(s);
            items(std::integral_constant<int, rad>{}, [&](int i, int g, int row, int b) {
#pragma unroll
                for (int q = 0; q < rad; ++q) w[i * rad + q] = lds[slot(b * M + SI::template in_pos<s>(g, q), row)];
                SI::template butterfly<s>(w + i * rad, g, block_r(b), twx);
            });
            if constexpr (s + 1 < SI::S) __syncthreads();
            items(std::integral_constant<int, rad>{}, [&](int i, int g, int row, int b) {
                if constexpr (s + 1 < SI::S) {
#pragma unroll
                    for (int q = 0; q < rad; ++q) lds[slot(b * M + SI::template out_pos<s>(g, q), row)] = w[i * rad + q];
                } else if (block_on(b)) {
                    C *dst = block_at(b) + (size_t)row * M;
#pragma unroll
                    for (int q = 0; q < rad; ++q) a_store<CP>(&dst[SI::template out_pos<s>(g, q)], w[i * rad + q]);
                }
            });
            if constexpr (s + 1 < SI::S) __syncthreads();
        };
        stage(std::integral_constant<int, 0>{});
        if constexpr (SI::S > 1) stage(std::integral_constant<int, 1>{});
        if constexpr (SI::S > 2) stage(std::integral_constant<int, 2>{});
    }
}

// F2 for i2 plans {R, A, 4} and i1 plans {16, B}, one block per workgroup.
// The threads of the radix-4 M-point stage and of the i1 transform's first
// stage are matched so that the data pass between them in registers: thread
// (t, h, c) does the radix-4 butterflies c of the rows t + (h + 4 e) N/16 (e =
// 0, 1), whose outputs are the columns c + A q, and then transforms column c
// + A h, whose first-stage legs are the rows t + l N/16 of all four h.  With h
// in lane bits 4 and 5 that is a swap of register with lane bits.  The
// threads t of a column are lanes of one wave, so the i1 exchange needs no
// workgroup barrier.  At N = 192 only 12 of a column's 16 lanes hold rows (the
// second i1 stage has 16 butterflies and uses all); five waves per SIMD, for a
// third workgroup per CU, spill 62 registers there (25 -> 39 us).  k_f_mid moved every value through LDS six times between
// twelve barriers, this moves it four times between five.
template <typename T, int N, int PY, int PX> struct FusedMidW {
    using G = FusedGeo<N, PY>;
    static constexpr int NT = N / 16, TPC = NT <= 8 ? 8 : 16;   // threads t that hold rows; lanes of a column
    static constexpr int A4 = G::M / 4, THREADS = G::M * TPC;
    // Pitches that keep the lanes served together on different banks.  The i1
    // exchange (scalars in FP64, values in FP32): a pad slot per 16 positions,
    // and columns of lane groups h and h + 1 offset by half the banks.  The
    // M-point exchange (values): four neighbouring columns by two or four
    // rows, whether the columns are adjacent or A apart.  With a pad slot per
    // 8 positions and odd pitches in both, n = 128 FP64 took 42.1 us alone and
    // 35.4 several per launch, now 39.4 and 30.9.
    static constexpr int ELINE = N + N / 16, EH = N == 192 ? 8 : 16;
    static constexpr int ES = (G::M * ELINE + 3 * EH) / (sizeof(T) == 8 ? 2 : 1) + 1;
    static constexpr int MLINE = N / 2 + (N == 192 ? 6 : 4), MA = N == 192 ? 0 : 4;
    static_assert(N / 2 % 16 == 0, "pitch");
    static constexpr int MS = G::M * MLINE + 3 * MA;
    static constexpr int ELEMS = ES > MS ? ES : MS;
    static constexpr int BLOCKS = G::R * (N / 2 + 1);
    static_assert(Plan<N, PY>::S == 3 && Plan<N, PY>::r[2] == 4 && Plan<N, PX>::S == 2 && Plan<N, PX>::r[0] == 16 &&
                      NT <= 16 && THREADS % 64 == 0,
                  "plans");
};
struct IdxWave {    // one pad slot per 16 positions, components and values alike
    int base;
    __device__ __forceinline__ int operator()(int pos) const { return base + pos + (pos >> 4); }
    __device__ __forceinline__ int scalar(int pos) const { return base + pos + (pos >> 4); }
    template <int> static constexpr bool blocked() { return false; }
};
// orders a wave's LDS accesses (which execute in order) for the compiler
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename T, int N, int PY, int PX, int CP>
__global__ void __launch_bounds__((FusedMidW<T, N, PY, PX>::THREADS), 4)
k_f_midw(JobRef jr, Twiddle<T> tw) {
    using C = cplx<T>;
    using G = FusedGeo<N, PY>;
    using F = FusedMidW<T, N, PY, PX>;
    using SF = SubSeq<N, PY, false>;
    using SI = SubSeq<N, PY, true>;
    using EF = Engine<T, N, F::TPC, false, PX>;
    using EI = Engine<T, N, F::TPC, true, PX>;
    constexpr int n = N / 2, R = G::R, M = G::M, A4 = F::A4, TH = F::THREADS, TPC = F::TPC, NT = F::NT;
    constexpr int P = ((n + 1 + 15) / 16) * 16;
    constexpr size_t BLK = G::template blk<T>();
    __shared__ C lds[F::ELEMS + N];
    const int wg = xcd_item(blockIdx.x, gridDim.x);
    if (wg >= F::BLOCKS) return;                    // uniform over the workgroup
    const auto twf = tw_fetch<T, N, TH, true>(tw);
    const Job jb = jr.get();
    const int res = wg % R, k3 = wg / R;
    C *block = (C *)jb.A + (size_t)(res * (n + 1) + k3) * BLK;
    const int lane = threadIdx.x & 63, h = lane >> 4, u = (threadIdx.x >> 6) * 16 + (lane & 15);
    const int t = u % TPC, c = u / TPC;
    const bool on = NT == TPC || t < NT;
    auto slot = [&](int col, int pos) { return col * F::MLINE + (col / (M / 4)) * F::MA + pos; };

    // radix-A stage: butterfly g of row `row`, IA per thread
    constexpr int RA = SF::radix(0), PA = M / RA, IA = n * PA / TH;
    static_assert(n * PA % TH == 0 && SI::radix(1) == RA && SI::radix(0) == 4, "items");
    C v[16];
#pragma unroll
    for (int i = 0; i < IA; ++i) {
        const int it = (int)threadIdx.x + i * TH, g = it % PA, row = it / PA;
#pragma unroll
        for (int q = 0; q < RA; ++q) v[i * RA + q] = a_load<CP>(&block[(size_t)row * M + SF::template in_pos<0>(g, q)]);
    }
    const TableTwiddle<T, N> twx = tw_commit<T, N, TH, true>(tw, twf, lds + F::ELEMS);
#pragma unroll
    for (int i = 0; i < IA; ++i) {
        const int it = (int)threadIdx.x + i * TH, g = it % PA, row = it / PA;
        SF::template butterfly<0>(v + i * RA, g, res, twx);
#pragma unroll
        for (int q = 0; q < RA; ++q) lds[slot(SF::template out_pos<0>(g, q), row)] = v[i * RA + q];
    }
    __syncthreads();
    // radix-4 stage, then to the i1 column c + A4 h
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[4 * e + q] = c_zero<C>();
            if (on) v[4 * e + q] = lds[slot(SF::template in_pos<1>(c, q), t + (h + 4 * e) * NT)];
        }
    __syncthreads();                                // the buffer becomes the i1 exchange's
#pragma unroll
    for (int e = 0; e < 2; ++e) SF::template butterfly<1>(v + 4 * e, c, res, twx);
    lane_exchange<4, 8>(v);
#pragma unroll
    for (int l = 8; l < 16; ++l) v[l] = c_zero<C>();
    const int col = c + A4 * h, k2 = res + R * col, bk = k2 <= n ? k2 : N - k2;
    const IdxWave idx{col * F::ELINE + F::EH * h};
    T *ls = reinterpret_cast<T *>(lds);
    auto exchange = [&](auto engine) {
        using E = decltype(engine);
        if constexpr (sizeof(T) == 8) {
            E::template store_comp<0, 0>(v, ls, t, idx);
            wave_sync();
            E::template load_comp<1, 0>(v, ls, t, idx);
            wave_sync();
            E::template store_comp<0, 1>(v, ls, t, idx);
            wave_sync();
            E::template load_comp<1, 1>(v, ls, t, idx);
        } else {
            E::template store_lds<0>(v, lds, t, idx);
            wave_sync();
            E::template load_lds<1>(v, lds, t, idx);
        }
        wave_sync();
    };
    EF::template compute<0>(v, t, twx);
    exchange(EF{});
    EF::template compute<1>(v, t, twx);
    const double *mrow = jb.mult + ((size_t)bk * P + k3) * (n + 1);
    EF::for_outputs(v, t, [&](int pos, int leg, C &val) {
        constexpr int RL = EF::R(EF::S - 1);
        val = scale_mode(val, g_load(&mrow[leg < RL / 2 ? pos : N - pos]));
    });
    EI::template compute<0>(v, t, twx);
    exchange(EI{});
    EI::template compute<1>(v, t, twx);
    // legs below 8 are the rows t + l N/16 kept
    lane_exchange<4, 8>(v);
#pragma unroll
    for (int e = 0; e < 2; ++e) SI::template butterfly<0>(v + 4 * e, c, res, twx);
    __syncthreads();                                // every wave is done with its i1 exchange
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (on) lds[slot(SI::template out_pos<0>(c, q), t + (h + 4 * e) * NT)] = v[4 * e + q];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IA; ++i) {
        const int it = (int)threadIdx.x + i * TH, g = it % PA, row = it / PA;
#pragma unroll
        for (int q = 0; q < RA; ++q) v[i * RA + q] = lds[slot(SI::template in_pos<1>(g, q), row)];
        SI::template butterfly<1>(v + i * RA, g, res, twx);
#pragma unroll
        for (int q = 0; q < RA; ++q) a_store<CP>(&block[(size_t)row * M + SI::template out_pos<1>(g, q)], v[i * RA + q]);
    }
}

// ------------------------------------------------------------------- F3
template <typename T, int N, int PZ, int PY, int J, int KU, int CP>
__global__ void __launch_bounds__((FusedLines<T, N, PZ, PY, J>::THREADS))
k_f_inv(JobRef jr, Twiddle<T> tw) {
    using C = cplx<T>;
    using G = FusedGeo<N, PY>;
    using F = FusedLines<T, N, PZ, PY, J>;
    using E = Engine<T, N, F::TPC, true, PZ>;
    constexpr int n = N / 2, R = G::R, M = G::M;
    constexpr size_t BLK = G::template blk<T>();
    __shared__ C lds[F::Q * F::LINE + N];
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (item >= n * F::GROUPS) return;              // uniform over the workgroup
    const FusedTwFetch<T, N, F::THREADS> twf(tw);
    const Job jb = jr.get();
    const int i1 = item / F::GROUPS, j0 = (item % F::GROUPS) * J;
    const int j = threadIdx.x % J;                  // THREADS is a multiple of J
    const C *src = (const C *)jb.A + (size_t)i1 * M + j0 + j;
    // the radix-R stage's twiddles W^(j r) are the same for every k3
    C p[R];
#pragma unroll
    for (int r = 1; r < R; ++r) {
        const double2 e = g_load(&tw.w[(j0 + j) * r]);
        p[r] = C{T(e.x), -T(e.y)};
    }
    // KU bins per thread and round, all loads of a round in flight at once
    constexpr int KT = F::THREADS / J;
    for (int k0 = threadIdx.x / J; k0 <= n; k0 += KU * KT) {
        C w[KU][R];
#pragma unroll
        for (int i = 0; i < KU; ++i)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (k0 + i * KT <= n) w[i][r] = a_load<CP>(&src[(size_t)(r * (n + 1) + k0 + i * KT) * BLK]);
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int k = k0 + i * KT;
            if (k > n) continue;
#pragma unroll
            for (int r = 1; r < R; ++r)
                w[i][r] = C{fmadd(w[i][r].x, p[r].x, -(w[i][r].y * p[r].y)), fmadd(w[i][r].x, p[r].y, w[i][r].y * p[r].x)};
            DFT<R, true, C>::run(w[i]);
            const bool real_bin = k == 0 || k == n;
#pragma unroll
            for (int s = 0; s < R / 2; ++s) {
                // rows j (A, even lane) and j + 1 (B, odd lane): Z[k] = A + i B
                // from the even lane, Z[N-k] = conj A + i conj B from the odd one
                C own = w[i][s];
                if (real_bin) own.y = 0;
                const C other{lane_xor1(own.x), lane_xor1(own.y)};
                IdxLine ix{(s * (J / 2) + j / 2) * F::LINE};
                if (!(j & 1))
                    lds[ix(k)] = C{own.x - other.y, own.y + other.x};
                else if (!real_bin)
                    lds[ix(N - k)] = C{other.x + own.y, own.x - other.y};
            }
        }
    }
    const auto twx = twf.commit(lds + F::Q * F::LINE);
    __syncthreads();
    const int t = threadIdx.x % F::TPC, q = threadIdx.x / F::TPC;
    const int row = j0 + 2 * (q % (J / 2)) + (q / (J / 2)) * M;
    IdxLine idx{q * F::LINE};
    C v[E::V];
    E::template load_lds<0>(v, lds, t, idx);
    __syncthreads();
    E::template run_from<0>(v, lds, t, idx, twx);
    T *ua = (T *)jb.u + ((size_t)i1 * n + row) * n;
    T *ub = ua + n;
    E::for_outputs(v, t, [&](int pos, int r, C &val) {
        if (r < E::R(E::S - 1) / 2) {
            s_store<(CP >= 1 ? 1 : 0)>(&ua[pos], val.x);
            s_store<(CP >= 1 ? 1 : 0)>(&ub[pos], val.y);
        }
    });
}

// ------------------------------------------------------------ launch
template <typename T, int N> hipError_t fused_solve(const Job &one, const Job *table, int count, const void *tw64,
                                                    hipStream_t st) {
    const Twiddle<T> tw = twiddle_of<T>(tw64);
    const JobRef jr{one, table};
    if constexpr (N <= SINGLE_MAX) {
        hipLaunchKernelGGL((k_single<T, N>), dim3(1, count), dim3(SingleCfg<T, N>::THREADS), 0, st, jr, tw);
    } else {
        using Cfg = FusedCfg<T, N>;
        constexpr int n = N / 2, PZ = fused_plan(N, 0), PY = fused_plan(N, 1), PX = fused_plan(N, 2);
        using G = FusedGeo<N, PY>;
        static_assert((size_t)G::R * (n + 1) * G::template blk<T>() <=
                          a_plane(n, n, (n / LayoutTile<T>::W + 1) * LayoutTile<T>::W, sizeof(cplx<T>)) * n,
                      "the blocks fit the intermediate A");
        auto launch = [&](auto many) {
            constexpr bool MANY = decltype(many)::value, NT = Cfg::NT && !MANY;
            constexpr int CW = NT ? 1 : 0, CP = NT ? 2 : 0, J1 = MANY ? Cfg::J1M : Cfg::J, J3 = MANY ? Cfg::J3M : Cfg::J,
                          KU = MANY ? Cfg::KUM : Cfg::KU;
            using F1 = FusedLines<T, N, PZ, PY, J1>;
            using F3 = FusedLines<T, N, PZ, PY, J3>;
            hipLaunchKernelGGL((k_f_fwd<T, N, PZ, PY, J1, CW>), dim3(xcd_blocks(n * F1::GROUPS), count),
                               dim3(F1::THREADS), 0, st, jr, tw);
            if constexpr (Cfg::W) {
                using F2 = FusedMidW<T, N, PY, PX>;
                hipLaunchKernelGGL((k_f_midw<T, N, PY, PX, CP>), dim3(xcd_blocks(F2::BLOCKS), count), dim3(F2::THREADS),
                                   0, st, jr, tw);
            } else {
                using F2 = FusedMid<T, N, PY, PX, Cfg::NB>;
                hipLaunchKernelGGL((k_f_mid<T, N, PY, PX, Cfg::NB, CP>),
                                   dim3(xcd_blocks(ceil_div(F2::BLOCKS, Cfg::NB)), count), dim3(F2::THREADS), 0, st, jr,
                                   tw);
            }
            hipLaunchKernelGGL((k_f_inv<T, N, PZ, PY, J3, KU, CP>), dim3(xcd_blocks(n * F3::GROUPS), count),
                               dim3(F3::THREADS), 0, st, jr, tw);
        };
        // (lengths whose single solves take five passes have no kernels for them)
        if (count > 1)
            launch(Const<1>{});
        else if constexpr (fused_count(N, sizeof(T) == 8, 1))
            launch(Const<0>{});
        else
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace psp
