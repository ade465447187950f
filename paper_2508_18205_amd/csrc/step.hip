// The hot path: one fused kernel per half step of the stabilised leapfrog
// (Kolar-Pozun & Kosec, arXiv 2508.18205, Section 5, eq. 19; 3D with the full
// discrete curl), plus the step loop (sources, receivers, energy of eq. 20,
// checkpoints, HIP-graph replay) and the FP64 reductions.
//
// Per node i the H update is
//   H_i <- H_i + a (-curl_D E)_i + a gamma (D^hv H)_i          a = dt / mu0
// and the E update
//   E_i <- mask_i [ E_i + kappa_i ((curl_D H_new)_i + gamma (D^hv E)_i) ]
// with kappa_i = dt / (eps0 eps_r,i) and mask = the PEC projector.  All
// operators are applied in difference form sum_s w_s (f_s - f_ref) with the
// reference slot left out (the weights sum to zero), which keeps the FP32
// sums free of the cancellation of sum_s w_s f_s.
//
// One wavefront owns one 64-node tile; its lanes stream the tile's packed
// indices and weights with 16-byte loads and gather field values through the
// L2 (nodes are Morton ordered, tiles are mapped XCD-contiguously).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.h"
#include "fields.h"
#include "wpack.h"

namespace {

// Kernel arguments are read by cache line, each first touch waited for, so
// what every kernel needs at its start comes first and what few need last.
template <typename TS, typename TW>
struct SA {
    static constexpr bool kAux = false;
    static constexpr bool kStream = true;   // staged kernels: weights and positions loaded non-temporally
    const TS* E;          // E^n
    const TS* H;          // H update: H^n ; E update: H^{n+1}
    const int32_t* hoff;  // LDS staging: halo lists
    const int32_t* hpool;
    const uint4* lidx;    // LDS staging: [tiles][Q8][64] x 8 u16 halo positions
    const int4* idx;      // collocated: union chunks ; two-set: curl chunks
    const TW* wc;
    const TW* wh;
    int64_t N, tiles;
    TS* out;              // H^{n+1} or E^{n+1}
    int C4, V4, S4, Q8, hmax;
    int xcd;
    // TEz: the 2D kernels with the fields' roles exchanged.  te = 1: the
    // vector kernel updates (Ex, Ey) from Hz with factor -kappa_i and the wall
    // mask; nomask = 1: the scalar kernel updates Hz (no wall mask)
    int te, nomask;
    double a;             // H update: dt / mu0 ; E update: dt / eps0
    double g;             // gamma
    const void* eps_r;    // per-node eps_r (double for FP64 fields, else float) or null
    const uint8_t* emask;
    const int4* idx_h;    // two-set: hv chunks
    const int32_t* pref;  // two-set: curl reference node
    double dt, eps0;
    const double* wnrm;   // [N][dim] unit wall normals (TEz and 3D curved walls; emask bit 3)
};

// a run's receivers and soft sources, folded into the half-step kernels: the H
// update also records E^n at the n_rcv receivers, the E update adds the terms
// of n_src sources.  Steps without them take the kernels without them (looking
// for none cost the staged kernels 0.2 us each).
template <typename TS, typename TW>
struct SX : SA<TS, TW> {
    static constexpr bool kAux = true;
    int n_rcv, n_src, FE, comp;
    const int32_t* rcv;
    void* trace;          // [n_rcv] row of the traces (TC)
    const int32_t* src;
    const void* samp;     // [n_src] amplitudes, [n_src] waveform row (TC)
    const void* swave;
};

// The same arguments for an operator that stays in the memory-side cache from
// one half step to the next: its loads are ordinary ones, which are kept there.
// Non-temporal loads are the better ones for what streams from HBM.
template <typename B>
struct Cached : B {
    static constexpr bool kStream = false;
    explicit Cached(const B& b) : B(b) {}
};

// Receivers: the H update of step n + 1 reads E^{n+1} anyway, so the lanes of
// its tiles (g: tile * 64 + lane) also write the trace row of step n, at their
// end (a kernel of its own per step took 3.6 us on the 40k-node dispersion set,
// 200 receivers; done first, it held every load back by 0.4 us).
template <typename TS, typename TW, typename A>
__device__ __forceinline__ void record_receivers(const A& a, int64_t g) {
    if constexpr (A::kAux) {
        using TC = typename Store<TS>::C;
        for (int64_t r = g; r < a.n_rcv; r += a.tiles * RBFFD_TILE)
            ((TC*)a.trace)[r] = Store<TS>::ld1(a.E, (int64_t)a.rcv[r] * a.FE + a.comp);
    }
}

// Soft sources: E at node i after the bracket gains amp * wave for every
// source on it, in source order, the product rounded before the sum and each
// sum rounded to the storage type as a store would; PEC nodes stay 0.
template <typename TC>
__device__ __forceinline__ TC source_term(const void* amp, const void* wave, int s) {
#pragma clang fp contract(off)
    return ((const TC*)amp)[s] * ((const TC*)wave)[s];
}
template <typename TS, typename TW, typename A>
__device__ __forceinline__ typename Store<TS>::C sourced(const A& a, int64_t i, bool free_, typename Store<TS>::C v) {
    using TC = typename Store<TS>::C;
    if (!free_) return (TC)0;
    if constexpr (A::kAux)
        for (int s = 0; s < a.n_src; ++s)
            if (a.src[s] == (int32_t)i)
                v = Store<TS>::rnd(Store<TS>::rnd(v) + source_term<TC>(a.samp, a.swave, s));
    return v;
}
// 3D: the source acts on Ez; on a curved wall (mask bit 3) E is already
// projected on the normal n, so adding v n_z n keeps (E + v e_z) projected
template <typename TS, typename TW, typename A>
__device__ __forceinline__ void sourced3(const A& a, int64_t i, uint8_t m, typename Store<TS>::C& x,
                                         typename Store<TS>::C& y, typename Store<TS>::C& z) {
    using S = Store<TS>;
    using TC = typename S::C;
    if constexpr (A::kAux)
        for (int s = 0; s < a.n_src; ++s) {
            if (a.src[s] != (int32_t)i) continue;
            const TC v = source_term<TC>(a.samp, a.swave, s);
            if (m & 8) {
                const double* n = a.wnrm + 3 * i;
                x = S::rnd(S::rnd(x) + v * (TC)n[2] * (TC)n[0]);
                y = S::rnd(S::rnd(y) + v * (TC)n[2] * (TC)n[1]);
                z = S::rnd(S::rnd(z) + v * (TC)n[2] * (TC)n[2]);
            } else {
                z = (m & 4) ? S::rnd(S::rnd(z) + v) : (TC)0;
            }
        }
}

template <typename TC>
__device__ __forceinline__ TC* lds_base() {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    return reinterpret_cast<TC*>(smem_raw);
}

// PEC on the in-plane E of the TEz polarisation: bit 0 / 1 of the mask keeps
// Ex / Ey (walls normal to an axis); bit 3 marks a curved-wall node with unit
// normal n = wn[i], where only the normal component survives: E <- (E . n) n
// The same for the 3D E: bits 0..2 keep Ex, Ey, Ez (faces normal to an axis),
// bit 3 projects on the unit normal wn[i] (curved wall)
template <typename TC>
__device__ __forceinline__ void wall3(uint8_t m, const double* wn, int64_t i, TC& x, TC& y, TC& z) {
    if (m & 8) {
        const TC nx = (TC)wn[3 * i], ny = (TC)wn[3 * i + 1], nz = (TC)wn[3 * i + 2];
        const TC en = x * nx + y * ny + z * nz;
        x = en * nx;
        y = en * ny;
        z = en * nz;
    } else {
        x = (m & 1) ? x : (TC)0;
        y = (m & 2) ? y : (TC)0;
        z = (m & 4) ? z : (TC)0;
    }
}

template <typename TC>
__device__ __forceinline__ void te_wall(uint8_t m, const double* wn, int64_t i, TC& x, TC& y) {
    if (m & 8) {
        const TC nx = (TC)wn[2 * i], ny = (TC)wn[2 * i + 1];
        const TC en = x * nx + y * ny;
        x = en * nx;
        y = en * ny;
    } else {
        x = (m & 1) ? x : (TC)0;
        y = (m & 2) ? y : (TC)0;
    }
}

template <typename TS, typename TW>
__device__ __forceinline__ int64_t tile_of(const SA<TS, TW>& a) {
    const int wpb = blockDim.x >> 6;
    const int blk = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    return (int64_t)blk * wpb + (threadIdx.x >> 6);
}

template <typename TS, typename TW>
__device__ __forceinline__ typename Store<TS>::C kappa_of(const SA<TS, TW>& a, int64_t i) {
    using TC = typename Store<TS>::C;
    if (!a.eps_r) return (TC)a.a;
    if (sizeof(TC) == 8) return (TC)(a.dt / (a.eps0 * ((const double*)a.eps_r)[i]));
    return (TC)(a.dt / (a.eps0 * (double)((const float*)a.eps_r)[i]));
}

// ---- 2D TMz, collocated ----------------------------------------------------
template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(512) void k_h2(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    using WV = typename WF<TW>::V;
    const int64_t tile = tile_of(a);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC dx = 0, dy = 0, vx = 0, vy = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int qb = min(a.C4, a.V4);
    int q = 0;
    for (; q < qb; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        WV wx[4], wy[4], wh[4];
        WF<TW>::ldp(pc + (q * 2 + 0) * WF<TW>::CH, wx);
        WF<TW>::ldp(pc + (q * 2 + 1) * WF<TW>::CH, wy);
        WF<TW>::ldp(ph + q * WF<TW>::CH, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = idx4(j, u);
            const TC de = S::ld1(a.E, jj) - e0;
            dx += (TC)wx[u] * de;
            dy += (TC)wy[u] * de;
            TC hx, hy;
            S::ld2(a.H, jj, hx, hy);
            vx += (TC)wh[u] * (hx - hx0);
            vy += (TC)wh[u] * (hy - hy0);
        }
    }
    for (; q < a.C4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        WV wx[4], wy[4];
        WF<TW>::ldp(pc + (q * 2 + 0) * WF<TW>::CH, wx);
        WF<TW>::ldp(pc + (q * 2 + 1) * WF<TW>::CH, wy);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const TC de = S::ld1(a.E, idx4(j, u)) - e0;
            dx += (TC)wx[u] * de;
            dy += (TC)wy[u] * de;
        }
    }
    for (; q < a.V4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        WV wh[4];
        WF<TW>::ldp(ph + q * WF<TW>::CH, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy;
            S::ld2(a.H, idx4(j, u), hx, hy);
            vx += (TC)wh[u] * (hx - hx0);
            vy += (TC)wh[u] * (hy - hy0);
        }
    }
    record_receivers<TS, TW>(a, i);
    if (i < a.N) {
        const TC G = (TC)a.g;
        if (!a.te) {
            const TC F = (TC)a.a;
            S::st2(a.out, i, hx0 + F * (-dy + G * vx), hy0 + F * (dx + G * vy));
        } else {
            // TEz (Ex, Ey) <- E + kappa (D^dy Hz + gamma HV, -D^dx Hz + gamma HV),
            // written as E - kappa (-D^dy Hz - gamma HV, D^dx Hz - gamma HV) with
            // the host's gamma negated; then the wall mask
            const TC F = -kappa_of(a, i);
            TC ex = hx0 + F * (-dy + G * vx), ey = hy0 + F * (dx + G * vy);
            te_wall(a.emask[i], a.wnrm, i, ex, ey);
            S::st2(a.out, i, ex, ey);
        }
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(512) void k_e2(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    using WV = typename WF<TW>::V;
    const int64_t tile = tile_of(a);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC cu = 0, ve = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int qb = min(a.C4, a.V4);
    int q = 0;
    for (; q < qb; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        WV wx[4], wy[4], wh[4];
        WF<TW>::ldp(pc + (q * 2 + 0) * WF<TW>::CH, wx);
        WF<TW>::ldp(pc + (q * 2 + 1) * WF<TW>::CH, wy);
        WF<TW>::ldp(ph + q * WF<TW>::CH, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = idx4(j, u);
            TC hx, hy;
            S::ld2(a.H, jj, hx, hy);
            cu += (TC)wx[u] * (hy - hy0) - (TC)wy[u] * (hx - hx0);
            ve += (TC)wh[u] * (S::ld1(a.E, jj) - e0);
        }
    }
    for (; q < a.C4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        WV wx[4], wy[4];
        WF<TW>::ldp(pc + (q * 2 + 0) * WF<TW>::CH, wx);
        WF<TW>::ldp(pc + (q * 2 + 1) * WF<TW>::CH, wy);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy;
            S::ld2(a.H, idx4(j, u), hx, hy);
            cu += (TC)wx[u] * (hy - hy0) - (TC)wy[u] * (hx - hx0);
        }
    }
    for (; q < a.V4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        WV wh[4];
        WF<TW>::ldp(ph + q * WF<TW>::CH, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) ve += (TC)wh[u] * (S::ld1(a.E, idx4(j, u)) - e0);
    }
    if (i < a.N) {
        const TC k = kappa_of(a, i);
        const TC v = sourced<TS, TW>(a, i, a.nomask || (a.emask[i] & 1), e0 + k * (cu + (TC)a.g * ve));
        S::st1(a.out, i, v);
    }
}

// ---- 2D TMz, two node sets ---------------------------------------------------
// H update: curl of E from the E set (reference = nearest E node), HV of H on
// the H set.  E update: curl of H from the H set, HV of E on the E set.
template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(512) void k_h2x(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    const int64_t tile = tile_of(a);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, a.pref[ic]);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC dx = 0, dy = 0, vx = 0, vy = 0;
    const int4* pi = a.idx + tile * a.C4 * RBFFD_TILE + lane;
    const int4* pj = a.idx_h + tile * a.V4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    for (int q = 0; q < a.C4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4];
        ldw4p(pc + (q * 2 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 2 + 1) * RBFFD_TILE * 4, wy);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const TC de = S::ld1(a.E, idx4(j, u)) - e0;
            dx += (TC)wx[u] * de;
            dy += (TC)wy[u] * de;
        }
    }
    for (int q = 0; q < a.V4; ++q) {
        const int4 j = pj[q * RBFFD_TILE];
        TW wh[4];
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy;
            S::ld2(a.H, idx4(j, u), hx, hy);
            vx += (TC)wh[u] * (hx - hx0);
            vy += (TC)wh[u] * (hy - hy0);
        }
    }
    record_receivers<TS, TW>(a, i);
    if (i < a.N) {
        const TC G = (TC)a.g;
        if (!a.te) {
            const TC F = (TC)a.a;
            S::st2(a.out, i, hx0 + F * (-dy + G * vx), hy0 + F * (dx + G * vy));
        } else {
            // TEz (Ex, Ey) <- E + kappa (D^dy Hz + gamma HV, -D^dx Hz + gamma HV),
            // written as E - kappa (-D^dy Hz - gamma HV, D^dx Hz - gamma HV) with
            // the host's gamma negated; then the wall mask
            const TC F = -kappa_of(a, i);
            TC ex = hx0 + F * (-dy + G * vx), ey = hy0 + F * (dx + G * vy);
            te_wall(a.emask[i], a.wnrm, i, ex, ey);
            S::st2(a.out, i, ex, ey);
        }
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(512) void k_e2x(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    const int64_t tile = tile_of(a);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, a.pref[ic], hx0, hy0);
    TC cu = 0, ve = 0;
    const int4* pi = a.idx + tile * a.C4 * RBFFD_TILE + lane;
    const int4* pj = a.idx_h + tile * a.V4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    for (int q = 0; q < a.C4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4];
        ldw4p(pc + (q * 2 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 2 + 1) * RBFFD_TILE * 4, wy);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy;
            S::ld2(a.H, idx4(j, u), hx, hy);
            cu += (TC)wx[u] * (hy - hy0) - (TC)wy[u] * (hx - hx0);
        }
    }
    for (int q = 0; q < a.V4; ++q) {
        const int4 j = pj[q * RBFFD_TILE];
        TW wh[4];
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) ve += (TC)wh[u] * (S::ld1(a.E, idx4(j, u)) - e0);
    }
    if (i < a.N) {
        const TC k = kappa_of(a, i);
        const TC v = sourced<TS, TW>(a, i, a.nomask || (a.emask[i] & 1), e0 + k * (cu + (TC)a.g * ve));
        S::st1(a.out, i, v);
    }
}

// ---- 2D, two node sets, small node sets ---------------------------------------
// As k_h2x / k_e2x with one 64-node tile per workgroup: its four wavefronts
// each sum every fourth curl chunk and every fourth hyperviscosity chunk, and
// the partial sums meet in LDS in a fixed order (the small-set scheme of
// k_h2s / k_e2s below, for the staggered variant).
template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(256) void k_h2xs(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    __shared__ TC part[3][4][RBFFD_TILE];
    const int64_t tile = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, a.pref[ic]);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC dx = 0, dy = 0, vx = 0, vy = 0;
    const int4* pi = a.idx + tile * a.C4 * RBFFD_TILE + lane;
    const int4* pj = a.idx_h + tile * a.V4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    for (int q = r; q < a.C4; q += 4) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4];
        ldw4p(pc + (q * 2 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 2 + 1) * RBFFD_TILE * 4, wy);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const TC de = S::ld1(a.E, idx4(j, u)) - e0;
            dx += (TC)wx[u] * de;
            dy += (TC)wy[u] * de;
        }
    }
    for (int q = r; q < a.V4; q += 4) {
        const int4 j = pj[q * RBFFD_TILE];
        TW wh[4];
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy;
            S::ld2(a.H, idx4(j, u), hx, hy);
            vx += (TC)wh[u] * (hx - hx0);
            vy += (TC)wh[u] * (hy - hy0);
        }
    }
    if (r > 0) {
        part[r - 1][0][lane] = dx;
        part[r - 1][1][lane] = dy;
        part[r - 1][2][lane] = vx;
        part[r - 1][3][lane] = vy;
    }
    __syncthreads();
    if (r == 0) record_receivers<TS, TW>(a, i);
    if (r > 0 || i >= a.N) return;
    dx = ((dx + part[0][0][lane]) + part[1][0][lane]) + part[2][0][lane];
    dy = ((dy + part[0][1][lane]) + part[1][1][lane]) + part[2][1][lane];
    vx = ((vx + part[0][2][lane]) + part[1][2][lane]) + part[2][2][lane];
    vy = ((vy + part[0][3][lane]) + part[1][3][lane]) + part[2][3][lane];
    const TC G = (TC)a.g;
    if (!a.te) {
        const TC F = (TC)a.a;
        S::st2(a.out, i, hx0 + F * (-dy + G * vx), hy0 + F * (dx + G * vy));
    } else {
        const TC F = -kappa_of(a, i);
        TC ex = hx0 + F * (-dy + G * vx), ey = hy0 + F * (dx + G * vy);
        te_wall(a.emask[i], a.wnrm, i, ex, ey);
        S::st2(a.out, i, ex, ey);
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(256) void k_e2xs(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    __shared__ TC part[3][2][RBFFD_TILE];
    const int64_t tile = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, a.pref[ic], hx0, hy0);
    TC cu = 0, ve = 0;
    const int4* pi = a.idx + tile * a.C4 * RBFFD_TILE + lane;
    const int4* pj = a.idx_h + tile * a.V4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    for (int q = r; q < a.C4; q += 4) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4];
        ldw4p(pc + (q * 2 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 2 + 1) * RBFFD_TILE * 4, wy);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy;
            S::ld2(a.H, idx4(j, u), hx, hy);
            cu += (TC)wx[u] * (hy - hy0) - (TC)wy[u] * (hx - hx0);
        }
    }
    for (int q = r; q < a.V4; q += 4) {
        const int4 j = pj[q * RBFFD_TILE];
        TW wh[4];
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) ve += (TC)wh[u] * (S::ld1(a.E, idx4(j, u)) - e0);
    }
    if (r > 0) {
        part[r - 1][0][lane] = cu;
        part[r - 1][1][lane] = ve;
    }
    __syncthreads();
    if (r > 0 || i >= a.N) return;
    cu = ((cu + part[0][0][lane]) + part[1][0][lane]) + part[2][0][lane];
    ve = ((ve + part[0][1][lane]) + part[1][1][lane]) + part[2][1][lane];
    const TC k = kappa_of(a, i);
    const TC v = sourced<TS, TW>(a, i, a.nomask || (a.emask[i] & 1), e0 + k * (cu + (TC)a.g * ve));
    S::st1(a.out, i, v);
}

// ---- 2D, collocated, small node sets ----------------------------------------
// One 64-node tile per workgroup; its four wavefronts each sum every fourth
// slot chunk of the tile's nodes (every load is still one contiguous run per
// wavefront) and the partial sums meet in LDS in a fixed order.  The chain
// of dependent loads per node is four times shorter, for launches too small
// to fill the chip.  Same terms as k_h2 / k_e2; only the order of the partial
// sums differs.
template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(256) void k_h2s(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    using WV = typename WF<TW>::V;
    __shared__ TC part[3][4][RBFFD_TILE];
    const int64_t tile = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC dx = 0, dy = 0, vx = 0, vy = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int qm = max(a.C4, a.V4);
    for (int q = r; q < qm; q += 4) {
        const int4 j = pi[q * RBFFD_TILE];
        if (q < a.C4) {
            WV wx[4], wy[4];
            WF<TW>::ldp(pc + (q * 2 + 0) * WF<TW>::CH, wx);
            WF<TW>::ldp(pc + (q * 2 + 1) * WF<TW>::CH, wy);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const TC de = S::ld1(a.E, idx4(j, u)) - e0;
                dx += (TC)wx[u] * de;
                dy += (TC)wy[u] * de;
            }
        }
        if (q < a.V4) {
            WV wh[4];
            WF<TW>::ldp(ph + q * WF<TW>::CH, wh);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                TC hx, hy;
                S::ld2(a.H, idx4(j, u), hx, hy);
                vx += (TC)wh[u] * (hx - hx0);
                vy += (TC)wh[u] * (hy - hy0);
            }
        }
    }
    if (r > 0) {
        part[r - 1][0][lane] = dx;
        part[r - 1][1][lane] = dy;
        part[r - 1][2][lane] = vx;
        part[r - 1][3][lane] = vy;
    }
    __syncthreads();
    if (r == 0) record_receivers<TS, TW>(a, i);
    if (r > 0 || i >= a.N) return;
    dx = ((dx + part[0][0][lane]) + part[1][0][lane]) + part[2][0][lane];
    dy = ((dy + part[0][1][lane]) + part[1][1][lane]) + part[2][1][lane];
    vx = ((vx + part[0][2][lane]) + part[1][2][lane]) + part[2][2][lane];
    vy = ((vy + part[0][3][lane]) + part[1][3][lane]) + part[2][3][lane];
    const TC G = (TC)a.g;
    if (!a.te) {
        const TC F = (TC)a.a;
        S::st2(a.out, i, hx0 + F * (-dy + G * vx), hy0 + F * (dx + G * vy));
    } else {
        const TC F = -kappa_of(a, i);
        TC ex = hx0 + F * (-dy + G * vx), ey = hy0 + F * (dx + G * vy);
        te_wall(a.emask[i], a.wnrm, i, ex, ey);
        S::st2(a.out, i, ex, ey);
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(256) void k_e2s(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    using WV = typename WF<TW>::V;
    __shared__ TC part[3][2][RBFFD_TILE];
    const int64_t tile = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC cu = 0, ve = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int qm = max(a.C4, a.V4);
    for (int q = r; q < qm; q += 4) {
        const int4 j = pi[q * RBFFD_TILE];
        if (q < a.C4) {
            WV wx[4], wy[4];
            WF<TW>::ldp(pc + (q * 2 + 0) * WF<TW>::CH, wx);
            WF<TW>::ldp(pc + (q * 2 + 1) * WF<TW>::CH, wy);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                TC hx, hy;
                S::ld2(a.H, idx4(j, u), hx, hy);
                cu += (TC)wx[u] * (hy - hy0) - (TC)wy[u] * (hx - hx0);
            }
        }
        if (q < a.V4) {
            WV wh[4];
            WF<TW>::ldp(ph + q * WF<TW>::CH, wh);
#pragma unroll
            for (int u = 0; u < 4; ++u) ve += (TC)wh[u] * (S::ld1(a.E, idx4(j, u)) - e0);
        }
    }
    if (r > 0) {
        part[r - 1][0][lane] = cu;
        part[r - 1][1][lane] = ve;
    }
    __syncthreads();
    if (r > 0 || i >= a.N) return;
    cu = ((cu + part[0][0][lane]) + part[1][0][lane]) + part[2][0][lane];
    ve = ((ve + part[0][1][lane]) + part[1][1][lane]) + part[2][1][lane];
    const TC k = kappa_of(a, i);
    const TC v = sourced<TS, TW>(a, i, a.nomask || (a.emask[i] & 1), e0 + k * (cu + (TC)a.g * ve));
    S::st1(a.out, i, v);
}

// ---- 3D, collocated: E and H stored as (x, y, z, pad) -------------------------
template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(512) void k_h3(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    const int64_t tile = tile_of(a);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC ex0, ey0, ez0, hx0, hy0, hz0;
    S::ld3(a.E, ic, ex0, ey0, ez0);
    S::ld3(a.H, ic, hx0, hy0, hz0);
    // d_a E_c accumulators for the curl
    TC xEy = 0, xEz = 0, yEx = 0, yEz = 0, zEx = 0, zEy = 0, vx = 0, vy = 0, vz = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 3 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const int qb = min(a.C4, a.V4);
    int q = 0;
    for (; q < qb; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4], wz[4], wh[4];
        ldw4p(pc + (q * 3 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 3 + 1) * RBFFD_TILE * 4, wy);
        ldw4p(pc + (q * 3 + 2) * RBFFD_TILE * 4, wz);
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = idx4(j, u);
            TC ex, ey, ez, hx, hy, hz;
            S::ld3(a.E, jj, ex, ey, ez);
            S::ld3(a.H, jj, hx, hy, hz);
            ex -= ex0; ey -= ey0; ez -= ez0;
            xEy += (TC)wx[u] * ey; xEz += (TC)wx[u] * ez;
            yEx += (TC)wy[u] * ex; yEz += (TC)wy[u] * ez;
            zEx += (TC)wz[u] * ex; zEy += (TC)wz[u] * ey;
            vx += (TC)wh[u] * (hx - hx0);
            vy += (TC)wh[u] * (hy - hy0);
            vz += (TC)wh[u] * (hz - hz0);
        }
    }
    for (; q < a.C4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4], wz[4];
        ldw4p(pc + (q * 3 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 3 + 1) * RBFFD_TILE * 4, wy);
        ldw4p(pc + (q * 3 + 2) * RBFFD_TILE * 4, wz);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC ex, ey, ez;
            S::ld3(a.E, idx4(j, u), ex, ey, ez);
            ex -= ex0; ey -= ey0; ez -= ez0;
            xEy += (TC)wx[u] * ey; xEz += (TC)wx[u] * ez;
            yEx += (TC)wy[u] * ex; yEz += (TC)wy[u] * ez;
            zEx += (TC)wz[u] * ex; zEy += (TC)wz[u] * ey;
        }
    }
    for (; q < a.V4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wh[4];
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy, hz;
            S::ld3(a.H, idx4(j, u), hx, hy, hz);
            vx += (TC)wh[u] * (hx - hx0);
            vy += (TC)wh[u] * (hy - hy0);
            vz += (TC)wh[u] * (hz - hz0);
        }
    }
    record_receivers<TS, TW>(a, i);
    if (i < a.N) {
        const TC F = (TC)a.a, G = (TC)a.g;
        // H <- H - a (curl E - gamma D^hv H)
        S::st3(a.out, i, hx0 - F * ((yEz - zEy) - G * vx), hy0 - F * ((zEx - xEz) - G * vy),
               hz0 - F * ((xEy - yEx) - G * vz));
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(512) void k_e3(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    const int64_t tile = tile_of(a);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC ex0, ey0, ez0, hx0, hy0, hz0;
    S::ld3(a.E, ic, ex0, ey0, ez0);
    S::ld3(a.H, ic, hx0, hy0, hz0);
    TC xHy = 0, xHz = 0, yHx = 0, yHz = 0, zHx = 0, zHy = 0, vx = 0, vy = 0, vz = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 3 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const int qb = min(a.C4, a.V4);
    int q = 0;
    for (; q < qb; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4], wz[4], wh[4];
        ldw4p(pc + (q * 3 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 3 + 1) * RBFFD_TILE * 4, wy);
        ldw4p(pc + (q * 3 + 2) * RBFFD_TILE * 4, wz);
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = idx4(j, u);
            TC ex, ey, ez, hx, hy, hz;
            S::ld3(a.H, jj, hx, hy, hz);
            S::ld3(a.E, jj, ex, ey, ez);
            hx -= hx0; hy -= hy0; hz -= hz0;
            xHy += (TC)wx[u] * hy; xHz += (TC)wx[u] * hz;
            yHx += (TC)wy[u] * hx; yHz += (TC)wy[u] * hz;
            zHx += (TC)wz[u] * hx; zHy += (TC)wz[u] * hy;
            vx += (TC)wh[u] * (ex - ex0);
            vy += (TC)wh[u] * (ey - ey0);
            vz += (TC)wh[u] * (ez - ez0);
        }
    }
    for (; q < a.C4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wx[4], wy[4], wz[4];
        ldw4p(pc + (q * 3 + 0) * RBFFD_TILE * 4, wx);
        ldw4p(pc + (q * 3 + 1) * RBFFD_TILE * 4, wy);
        ldw4p(pc + (q * 3 + 2) * RBFFD_TILE * 4, wz);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC hx, hy, hz;
            S::ld3(a.H, idx4(j, u), hx, hy, hz);
            hx -= hx0; hy -= hy0; hz -= hz0;
            xHy += (TC)wx[u] * hy; xHz += (TC)wx[u] * hz;
            yHx += (TC)wy[u] * hx; yHz += (TC)wy[u] * hz;
            zHx += (TC)wz[u] * hx; zHy += (TC)wz[u] * hy;
        }
    }
    for (; q < a.V4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        TW wh[4];
        ldw4p(ph + q * RBFFD_TILE * 4, wh);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC ex, ey, ez;
            S::ld3(a.E, idx4(j, u), ex, ey, ez);
            vx += (TC)wh[u] * (ex - ex0);
            vy += (TC)wh[u] * (ey - ey0);
            vz += (TC)wh[u] * (ez - ez0);
        }
    }
    if (i < a.N) {
        const TC k = kappa_of(a, i), G = (TC)a.g;
        TC nx = ex0 + k * ((yHz - zHy) + G * vx);
        TC ny = ey0 + k * ((zHx - xHz) + G * vy);
        TC nz = ez0 + k * ((xHy - yHx) + G * vz);
        const uint8_t m = a.emask[i];
        wall3(m, a.wnrm, i, nx, ny, nz);
        sourced3<TS, TW>(a, i, m, nx, ny, nz);
        S::st3(a.out, i, nx, ny, nz);
    }
}

// ---- 3D, small node sets ------------------------------------------------------
// As k_h2s / k_e2s with eight wavefronts per 64-node tile: launches too small to
// fill the chip are bound by the chain of dependent loads (stencil indices, then
// the values they name), so the tile's slot chunks are dealt out to the
// wavefronts, curl chunks first, and a wavefront requests the indices of the
// chunks it holds, then all they name, before it uses any.  The staged kernels
// take 45 us per step on a 13.5k-node box (27 or 14 workgroups on 256 CUs),
// these 15.0 in FP64 and 14.4 in FP32.
constexpr int kSplit3 = 8;

// curl sums (x, y, z of the field C) and hyperviscosity sums (of the field V)
// of the tile's nodes, complete in every lane of wavefront 0.
//
// FP64: a wavefront multiplies its chunks by their weights, and the partial
// sums meet in LDS, the first six wavefronts each adding up one of the six.
// One chunk at a time: two spill (46.8 against 26.6 us per step, 30k nodes);
// sixteen wavefronts per tile, 53.7 against 47.9 us at 64k nodes.
template <typename TS, typename TW>
__device__ __forceinline__ void small_sums3(const SA<TS, TW>& a, const TS* C, const TS* V, int64_t tile, int r, int lane,
                                            const double (&c0)[3], const double (&v0)[3], double (&sum)[6]) {
    using S = Store<TS>;
    __shared__ double part[kSplit3][6][RBFFD_TILE];
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 3 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int total = a.C4 + a.V4;
#pragma unroll
    for (int k = 0; k < 6; ++k) sum[k] = 0;
    for (int g = r; g < total; g += kSplit3) {
        double f[3];
        if (g < a.C4) {
            const int4 j = pi[g * RBFFD_TILE];
            TW w[3][4];
#pragma unroll
            for (int k = 0; k < 3; ++k) ldw4p(pc + (g * 3 + k) * WF<TW>::CH, w[k]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                S::ld3(C, idx4(j, u), f[0], f[1], f[2]);
                const double x = f[0] - c0[0], y = f[1] - c0[1], z = f[2] - c0[2];
                sum[0] += w[1][u] * z - w[2][u] * y;
                sum[1] += w[2][u] * x - w[0][u] * z;
                sum[2] += w[0][u] * y - w[1][u] * x;
            }
        } else {
            const int4 j = pi[(g - a.C4) * RBFFD_TILE];
            TW w[4];
            ldw4p(ph + (g - a.C4) * WF<TW>::CH, w);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                S::ld3(V, idx4(j, u), f[0], f[1], f[2]);
#pragma unroll
                for (int k = 0; k < 3; ++k) sum[3 + k] += w[u] * (f[k] - v0[k]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) part[r][k][lane] = sum[k];
    __syncthreads();
    if (r < 6) {
        double v = part[0][r][lane];
#pragma unroll
        for (int q = 1; q < kSplit3; ++q) v += part[q][r][lane];
        part[0][r][lane] = v;   // read and written by this wavefront only
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 6; ++k) sum[k] = part[0][k][lane];
}

// FP32: the wavefronts only fetch, into LDS ([slot][component][lane]); six of
// them then each sum one or two of the nine sums over all slots, in slot order
// and in the arithmetic of the staged kernels, so that FP32 results do not
// depend on which of the two runs.  Their weights, nine chunks at a time in
// registers, are requested before the values.  A tile of n = 35, n_hv = 71 takes
// 83 KB of LDS, so a CU holds one workgroup; keeping only the slots in use (80
// KB, two per CU) needs a test per slot: 16.3 against 14.4 us per step at 13.5k
// nodes.
constexpr int kAhead3 = 9;
inline size_t small3_lds(const OpBlock& o) { return (size_t)(o.C4 + o.V4) * 4 * 3 * RBFFD_TILE * sizeof(float); }
template <typename TS, typename TW>
__device__ __forceinline__ void small_sums3(const SA<TS, TW>& a, const TS* C, const TS* V, int64_t tile, int r, int lane,
                                            const float (&c0)[3], const float (&v0)[3], float (&sum)[6]) {
    using S = Store<TS>;
    float* sv = lds_base<float>() + lane;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const int total = a.C4 + a.V4;
    // wavefronts 0..2 sum the curl products of the x, y, z weights, 3..5 the
    // hyperviscosity of component r - 3
    const bool curl = r < 3;
    const int n4 = r < 6 ? (curl ? a.C4 : a.V4) : 0;
    const TW* pw = curl ? a.wc + (tile * a.C4 * 3 + r) * WF<TW>::CH + lane * WF<TW>::LS
                        : a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int64_t ws = (curl ? 3 : 1) * WF<TW>::CH;
    TW w[kAhead3][4];
#pragma unroll
    for (int i = 0; i < kAhead3; ++i)
        if (i < n4) ldw4p(pw + i * ws, w[i]);
    for (int g0 = r; g0 < total; g0 += 2 * kSplit3) {
        int4 j[2];
        float f[2][4][3];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int g = g0 + kSplit3 * t;
            if (g < total) j[t] = pi[(g < a.C4 ? g : g - a.C4) * RBFFD_TILE];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int g = g0 + kSplit3 * t;
            if (g >= total) continue;
            const TS* F = g < a.C4 ? C : V;
#pragma unroll
            for (int u = 0; u < 4; ++u) S::ld3(F, idx4(j[t], u), f[t][u][0], f[t][u][1], f[t][u][2]);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int g = g0 + kSplit3 * t;
            if (g >= total) continue;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    sv[((g * 4 + u) * 3 + k) * RBFFD_TILE] = f[t][u][k] - (g < a.C4 ? c0[k] : v0[k]);
        }
    }
    __syncthreads();
    // components that the x, y, z weights multiply: (y, z), (x, z), (x, y)
    const int kp = r == 0 ? 1 : 0, kq = r == 2 ? 1 : 2;
    float p = 0, q = 0;
    for (int b = 0; b < n4; b += kAhead3) {
#pragma unroll
        for (int i = 0; i < kAhead3; ++i) {
            if (b + i >= n4) break;
            const float* s = sv + (curl ? b + i : a.C4 + b + i) * 12 * RBFFD_TILE;
            if (curl) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    p += (float)w[i][u] * s[(u * 3 + kp) * RBFFD_TILE];
                    q += (float)w[i][u] * s[(u * 3 + kq) * RBFFD_TILE];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) p += (float)w[i][u] * s[(u * 3 + r - 3) * RBFFD_TILE];
            }
            if (b + i + kAhead3 < n4) ldw4p(pw + (b + i + kAhead3) * ws, w[i]);
        }
    }
    __syncthreads();   // the sums take the place of the values
    if (curl) {
        sv[(2 * r) * RBFFD_TILE] = p;
        sv[(2 * r + 1) * RBFFD_TILE] = q;
    } else if (r < 6) {
        sv[(3 + r) * RBFFD_TILE] = p;
    }
    __syncthreads();
    // (x f_y, x f_z, y f_x, y f_z, z f_x, z f_y), v
    float c[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) c[k] = sv[k * RBFFD_TILE];
    sum[0] = c[3] - c[5];
    sum[1] = c[4] - c[1];
    sum[2] = c[0] - c[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) sum[3 + k] = c[6 + k];
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(64 * kSplit3) void k_h3s(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    const int64_t tile = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC e0[3], h0[3], s[6];
    S::ld3(a.E, ic, e0[0], e0[1], e0[2]);
    S::ld3(a.H, ic, h0[0], h0[1], h0[2]);
    small_sums3<TS, TW>(a, a.E, a.H, tile, r, lane, e0, h0, s);
    if (r == 0) record_receivers<TS, TW>(a, i);
    if (r > 0 || i >= a.N) return;
    const TC F = (TC)a.a, G = (TC)a.g;
    S::st3(a.out, i, h0[0] - F * (s[0] - G * s[3]), h0[1] - F * (s[1] - G * s[4]), h0[2] - F * (s[2] - G * s[5]));
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(64 * kSplit3) void k_e3s(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    const int64_t tile = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC e0[3], h0[3], s[6];
    S::ld3(a.E, ic, e0[0], e0[1], e0[2]);
    S::ld3(a.H, ic, h0[0], h0[1], h0[2]);
    small_sums3<TS, TW>(a, a.H, a.E, tile, r, lane, h0, e0, s);
    if (r > 0 || i >= a.N) return;
    const TC k = kappa_of(a, i), G = (TC)a.g;
    TC x = e0[0] + k * (s[0] + G * s[3]), y = e0[1] + k * (s[1] + G * s[4]), z = e0[2] + k * (s[2] + G * s[5]);
    const uint8_t m = a.emask[i];
    wall3(m, a.wnrm, i, x, y, z);
    sourced3<TS, TW>(a, i, m, x, y, z);
    S::st3(a.out, i, x, y, z);
}

// ---- LDS-staged variants ------------------------------------------------------
// A workgroup owns 256 consecutive nodes in 2D, in 3D 1024 with FP32 weights
// and 512 with FP64 (4, 16 or 8 wavefront tiles).  It first copies
// the field values of every node its stencils touch (the sorted halo list)
// into LDS with one coalesced pass, then each node sums over its slots with
// 16-bit halo positions (8 per 16-byte load) instead of 32-bit global indices
// and global gathers.  Same arithmetic and summation order as the global
// variants.
__device__ __forceinline__ int pos4(const uint4& v, int half, int u) {
    const uint32_t w = half ? (u < 2 ? v.z : v.w) : (u < 2 ? v.x : v.y);
    return (int)((u & 1) ? (w >> 16) : (w & 0xFFFFu));
}

template <typename TW>
__device__ __forceinline__ void copy4(TW (&d)[4], const TW (&s)[4]) {
    d[0] = s[0];
    d[1] = s[1];
    d[2] = s[2];
    d[3] = s[3];
}
// streamed (non-temporal) or cached loads of a chunk's weights and positions
template <bool STREAM, typename TW, typename WV>
__device__ __forceinline__ void ldw(const TW* p, WV (&w)[4]) {
    if constexpr (STREAM) WF<TW>::ld(p, w);
    else WF<TW>::ldp(p, w);
}
template <bool STREAM>
__device__ __forceinline__ uint4 ldpos(const uint4* p) {
    if constexpr (STREAM) return ldu4s(p);
    else return *p;
}
// weights of chunk q of a 2D block (left unchanged past the chunk counts)
template <bool STREAM, typename TW, typename WV = typename WF<TW>::V>
__device__ __forceinline__ void load2(const TW* pc, const TW* ph, int q, int C4, int V4, WV (&x)[4], WV (&y)[4],
                                      WV (&h)[4]) {
    if (q < C4) {
        ldw<STREAM>(pc + (q * 2 + 0) * WF<TW>::CH, x);
        ldw<STREAM>(pc + (q * 2 + 1) * WF<TW>::CH, y);
    }
    if (q < V4) ldw<STREAM>(ph + q * WF<TW>::CH, h);
}

// weights of chunk q of a 3D block (left unchanged past the chunk counts)
template <bool STREAM, typename TW>
__device__ __forceinline__ void load3(const TW* pc, const TW* ph, int q, int C4, int V4, TW (&x)[4], TW (&y)[4],
                                      TW (&z)[4], TW (&h)[4]) {
    if (q < C4) {
        ldw<STREAM>(pc + (q * 3 + 0) * RBFFD_TILE * 4, x);
        ldw<STREAM>(pc + (q * 3 + 1) * RBFFD_TILE * 4, y);
        ldw<STREAM>(pc + (q * 3 + 2) * RBFFD_TILE * 4, z);
    }
    if (q < V4) ldw<STREAM>(ph + q * RBFFD_TILE * 4, h);
}

// 3-vector LDS entries, packed (12 B in FP32) so that more workgroups fit
template <typename TC>
__device__ __forceinline__ void st_lds3(TC* p, const TC (&v)[3]) {
    p[0] = v[0];
    p[1] = v[1];
    p[2] = v[2];
}
template <typename TC>
__device__ __forceinline__ void ld_lds3(const TC* p, TC (&v)[3]) {
    v[0] = p[0];
    v[1] = p[1];
    v[2] = p[2];
}

// one 16-byte (FP32) or two 16-byte (FP64) LDS accesses per 3-vector entry
__device__ __forceinline__ void st_lds4(float* p, const float (&v)[3]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], 0.0f);
}
__device__ __forceinline__ void st_lds4(double* p, const double (&v)[3]) {
    reinterpret_cast<double2*>(p)[0] = make_double2(v[0], v[1]);
    reinterpret_cast<double2*>(p)[1] = make_double2(v[2], 0.0);
}
__device__ __forceinline__ void ld_lds4(const float* p, float (&v)[3]) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
}
__device__ __forceinline__ void ld_lds4(const double* p, double (&v)[3]) {
    const double2 a = reinterpret_cast<const double2*>(p)[0];
    const double2 b = reinterpret_cast<const double2*>(p)[1];
    v[0] = a.x;
    v[1] = a.y;
    v[2] = b.x;
}

__device__ __forceinline__ void ld_lds2(const float* p, float& x, float& y) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    x = t.x;
    y = t.y;
}
__device__ __forceinline__ void ld_lds2(const double* p, double& x, double& y) {
    const double2 t = *reinterpret_cast<const double2*>(p);
    x = t.x;
    y = t.y;
}
__device__ __forceinline__ void st_lds2(float* p, float x, float y) { *reinterpret_cast<float2*>(p) = make_float2(x, y); }
__device__ __forceinline__ void st_lds2(double* p, double x, double y) {
    *reinterpret_cast<double2*>(p) = make_double2(x, y);
}

// Halo staging with several loads in flight per thread: each round takes up
// to SB list entries per thread, loads all their list values, then all their
// field values, then stores them (a plain loop waits for each load in turn).
// ld(j) returns the staged value of source node j, st(k, v) stores entry k.
template <int SB, typename V, typename LD, typename ST>
__device__ __forceinline__ void stage_rounds(const int32_t* list, int hc, LD ld, ST st) {
    const int nt = (int)blockDim.x, t = (int)threadIdx.x;
    for (int base = 0; base < hc; base += SB * nt) {
        int j[SB];
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int k = base + b * nt + t;
            j[b] = k < hc ? list[k] : -1;
        }
        V v[SB];
#pragma unroll
        for (int b = 0; b < SB; ++b)
            if (j[b] >= 0) v[b] = ld(j[b]);
#pragma unroll
        for (int b = 0; b < SB; ++b)
            if (j[b] >= 0) st(base + b * nt + t, v[b]);
    }
}

template <typename TC>
struct Val3 {
    TC x, y, z;
};
template <typename TC>
struct Val6 {
    TC v[6];
};

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(256) void k_h2l(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    using WV = typename WF<TW>::V;
    TC* sE = lds_base<TC>();
    TC* sH = sE + ((a.hmax + 3) & ~3);                 // pairs (Hx, Hy)
    const int wg = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int h0 = a.hoff[wg], hc = a.hoff[wg + 1] - h0;
    stage_rounds<4, Val3<TC>>(
        a.hpool + h0, hc,
        [&](int j) {
            Val3<TC> v;
            v.x = S::ld1(a.E, j);
            S::ld2(a.H, j, v.y, v.z);
            return v;
        },
        [&](int k, const Val3<TC>& v) {
            sE[k] = v.x;
            st_lds2(sH + 2 * k, v.y, v.z);
        });
    __syncthreads();
    const int64_t tile = (int64_t)wg * (RBFFD_WGT / RBFFD_TILE) + (threadIdx.x >> 6);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC dx = 0, dy = 0, vx = 0, vy = 0;
    const uint4* pl = a.lidx + tile * a.Q8 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int qm = max(a.C4, a.V4);
    // chunk q + 1 is loaded while chunk q is summed
    uint4 li = ldpos<A::kStream>(pl);
    WV nx[4] = {0, 0, 0, 0}, ny[4] = {0, 0, 0, 0}, nh[4] = {0, 0, 0, 0};
    load2<A::kStream>(pc, ph, 0, a.C4, a.V4, nx, ny, nh);
    for (int q = 0; q < qm; ++q) {
        const uint4 lc = li;
        WV wx[4], wy[4], wh[4];
        copy4(wx, nx); copy4(wy, ny); copy4(wh, nh);
        if (q + 1 < qm) {
            if (((q + 1) & 1) == 0) li = ldpos<A::kStream>(pl + ((q + 1) >> 1) * RBFFD_TILE);
            load2<A::kStream>(pc, ph, q + 1, a.C4, a.V4, nx, ny, nh);
        }
        const int hf = q & 1;
        if (q < a.C4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const TC de = sE[pos4(lc, hf, u)] - e0;
                dx += (TC)wx[u] * de;
                dy += (TC)wy[u] * de;
            }
        }
        if (q < a.V4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                TC hx, hy;
                ld_lds2(sH + 2 * pos4(lc, hf, u), hx, hy);
                vx += (TC)wh[u] * (hx - hx0);
                vy += (TC)wh[u] * (hy - hy0);
            }
        }
    }
    record_receivers<TS, TW>(a, i);
    if (i < a.N) {
        const TC G = (TC)a.g;
        if (!a.te) {
            const TC F = (TC)a.a;
            S::st2(a.out, i, hx0 + F * (-dy + G * vx), hy0 + F * (dx + G * vy));
        } else {
            // TEz (Ex, Ey) <- E + kappa (D^dy Hz + gamma HV, -D^dx Hz + gamma HV),
            // written as E - kappa (-D^dy Hz - gamma HV, D^dx Hz - gamma HV) with
            // the host's gamma negated; then the wall mask
            const TC F = -kappa_of(a, i);
            TC ex = hx0 + F * (-dy + G * vx), ey = hy0 + F * (dx + G * vy);
            te_wall(a.emask[i], a.wnrm, i, ex, ey);
            S::st2(a.out, i, ex, ey);
        }
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(256) void k_e2l(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    using WV = typename WF<TW>::V;
    TC* sE = lds_base<TC>();
    TC* sH = sE + ((a.hmax + 3) & ~3);
    const int wg = tile_back(a.xcd);
    const int h0 = a.hoff[wg], hc = a.hoff[wg + 1] - h0;
    stage_rounds<4, Val3<TC>>(
        a.hpool + h0, hc,
        [&](int j) {
            Val3<TC> v;
            v.x = S::ld1(a.E, j);
            S::ld2(a.H, j, v.y, v.z);
            return v;
        },
        [&](int k, const Val3<TC>& v) {
            sE[k] = v.x;
            st_lds2(sH + 2 * k, v.y, v.z);
        });
    __syncthreads();
    const int64_t tile = (int64_t)wg * (RBFFD_WGT / RBFFD_TILE) + (threadIdx.x >> 6);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const TC e0 = S::ld1(a.E, ic);
    TC hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    TC cu = 0, ve = 0;
    const uint4* pl = a.lidx + tile * a.Q8 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 2 * WF<TW>::CH + lane * WF<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * WF<TW>::CH + lane * WF<TW>::LS;
    const int qm = max(a.C4, a.V4);
    uint4 li = ldpos<A::kStream>(pl);
    WV nx[4] = {0, 0, 0, 0}, ny[4] = {0, 0, 0, 0}, nh[4] = {0, 0, 0, 0};
    load2<A::kStream>(pc, ph, 0, a.C4, a.V4, nx, ny, nh);
    for (int q = 0; q < qm; ++q) {
        const uint4 lc = li;
        WV wx[4], wy[4], wh[4];
        copy4(wx, nx); copy4(wy, ny); copy4(wh, nh);
        if (q + 1 < qm) {
            if (((q + 1) & 1) == 0) li = ldpos<A::kStream>(pl + ((q + 1) >> 1) * RBFFD_TILE);
            load2<A::kStream>(pc, ph, q + 1, a.C4, a.V4, nx, ny, nh);
        }
        const int hf = q & 1;
        if (q < a.C4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                TC hx, hy;
                ld_lds2(sH + 2 * pos4(lc, hf, u), hx, hy);
                cu += (TC)wx[u] * (hy - hy0) - (TC)wy[u] * (hx - hx0);
            }
        }
        if (q < a.V4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) ve += (TC)wh[u] * (sE[pos4(lc, hf, u)] - e0);
        }
    }
    if (i < a.N) {
        const TC k = kappa_of(a, i);
        const TC v = sourced<TS, TW>(a, i, a.nomask || (a.emask[i] & 1), e0 + k * (cu + (TC)a.g * ve));
        S::st1(a.out, i, v);
    }
}

// ---- 2D, a whole step in one kernel -------------------------------------------
// The half steps of a large set are bound by reading the operator, twice per step.
// Here a workgroup keeps its tile's weights and positions (up to 160 registers a
// lane) from the H update to the E update.  Between the two it publishes the tile's
// H and waits for the tiles that its halo touches.  Tiles are dispatched in strips
// (OpBlock::ord), so these run at about the same time; a workgroup that has waited
// its patience out computes the missing H by itself from E^n and H^n, which
// nobody writes meanwhile, to the same bits: it never depends on another's progress.
// The sums are those of the staged kernels, in their order.
// us per step, two halves / whole, 2D FP32: 40k nodes (n 25) 11.5 / 10.2, 90k 18.3 /
// 14.1, 360k 48.5 / 37.4, 1M 133 / 101 (n 25, alpha 3: 176 / 146), 4M 491 / 397.  What is
// left at 1M: 14 us of waiting (taken out in a copy: 94, of 104 to 108 then), the sums
// 13 us not hidden by other workgroups' loads, 80 for the loads (420 MB, floor 64).
// Tried: hv weights in LDS for four workgroups a CU 117, all LDS reads of a chunk
// before its sums 122 (spills), 8 neighbouring tiles per XCD 110, two workgroups a CU 127.
// Beside other work on the GPU a workgroup may wait for one that cannot start.  Next
// to a stream of 8192^2 bf16 products: 360k 1585 / 804, 1M 1633 / 848.  Next to one of
// 256 MB copies, with the copies that end meanwhile per ms: 40k 33.6 (8.4) / 27.2 (8.8),
// 194k 57.8 (5.2) / 70.2 (5.0), 360k 96.9 (4.8) / 105 (5.6), 1M 224 (3.6) / 267 (5.1),
// alpha 3 293 (3.4) / 292 (6.7): the copies get more of the chip, and sets that just
// fill it lose a fifth.  Two runs at once on one 1M plan, per step of both: 255 / 191.
template <typename B>
struct Whole : B {   // a: the factor of the E update, out: E^{n+1}
    static constexpr bool kStream = B::kStream;
    explicit Whole(const B& b) : B(b) {}
    uint64_t* Hn;         // H^{n+1}: pairs, read and written past the L2s, which the XCDs do not share
    uint64_t* flags;      // [nwg] tag of the tile's latest H
    uint64_t tag;         // this run and step
    const int4* ord;      // what each workgroup does (OpBlock)
    int32_t* late;        // H tiles computed by workgroups that had waited (OpBlock)
    double aH;
    int32_t patience;     // ticks of 10 ns
};

__device__ __forceinline__ uint64_t pair_bits(float x, float y) {
    return (uint64_t)__float_as_uint(y) << 32 | __float_as_uint(x);
}

// Stores of this wavefront have reached the point that all XCDs see.  H and the flags
// are handed over by relaxed agent-scope atomics alone (an agent-scope release or
// acquire would write back or invalidate the XCD's L2, where the operator lies), which
// rests on the following of gfx950: such loads and stores carry sc1 and pass the L2s in
// both directions, stores count in vmcnt until that point has them, and a load issued
// after the flag's value was used (a barrier lies between them) reads later.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "k_step2 hands H over between workgroups in a way that is shown for gfx950 only"
#endif
__device__ __forceinline__ void stores_done() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    asm volatile("" ::: "memory");
}

__global__ __launch_bounds__(256) void k_no_steps(uint64_t* flags, int n) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < n) flags[t] = 0;
}

// H update of one tile from global memory, slots in the same order
template <typename A>
__device__ __forceinline__ void whole_h_late(const A& a, int64_t wg) {
    const int64_t tile = wg * (RBFFD_WGT / RBFFD_TILE) + (threadIdx.x >> 6);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const float e0 = a.E[ic];
    float hx0, hy0;
    Store<float>::ld2(a.H, ic, hx0, hy0);
    float dx = 0, dy = 0, vx = 0, vy = 0;
    const int4* pi = a.idx + tile * a.S4 * RBFFD_TILE + lane;
    const float* pc = a.wc + tile * a.C4 * 2 * WF<float>::CH + lane * WF<float>::LS;
    const float* ph = a.wh + tile * a.V4 * WF<float>::CH + lane * WF<float>::LS;
    for (int q = 0; q < a.S4; ++q) {
        const int4 j = pi[q * RBFFD_TILE];
        float wx[4], wy[4], wh[4];
        load2<false>(pc, ph, q, a.C4, a.V4, wx, wy, wh);
        if (q < a.C4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float de = a.E[idx4(j, u)] - e0;
                dx += wx[u] * de;
                dy += wy[u] * de;
            }
        }
        if (q < a.V4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float hx, hy;
                Store<float>::ld2(a.H, idx4(j, u), hx, hy);
                vx += wh[u] * (hx - hx0);
                vy += wh[u] * (hy - hy0);
            }
        }
    }
    if (i < a.N) {
        const float F = (float)a.aH, G = (float)a.g;
        __hip_atomic_store(a.Hn + i, pair_bits(hx0 + F * (-dy + G * vx), hy0 + F * (dx + G * vy)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
}

// QC, QV: most chunks of curl and hyperviscosity weights
template <int QC, int QV, typename A>
__global__ __launch_bounds__(256, QV <= 8 ? 3 : 2) void k_step2(A a) {
    using S = Store<float>;
    constexpr int QM = QC > QV ? QC : QV, QP = (QM + 1) / 2;
    __shared__ int want;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    float* sE = lds_base<float>();
    float* sH = sE + ((a.hmax + 3) & ~3);
    const int4 jb = a.ord[blockIdx.x];
    const int wg = jb.x, job = jb.y, hc = jb.w;
    const int32_t* list = a.hpool + jb.z;
    const int64_t tile0 = (int64_t)wg * (RBFFD_WGT / RBFFD_TILE) + wave;
    const bool in = tile0 < a.tiles;
    const int64_t tile = in ? tile0 : a.tiles - 1;
    const uint4* pl = a.lidx + tile * a.Q8 * RBFFD_TILE;
    const float* pc = a.wc + tile * a.C4 * 2 * WF<float>::CH;
    const float* ph = a.wh + tile * a.V4 * WF<float>::CH;
    uint4 li[QP];
    float wx[QC][4], wy[QC][4], wh[QV][4];
    auto load = [&] {
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            if ((q & 1) == 0 && q / 2 < a.Q8) li[q / 2] = ldpos<A::kStream>(pl + q / 2 * RBFFD_TILE + lane);
            if (q < QC && q < a.C4) {
                ldw<A::kStream>(pc + (q * 2 + 0) * WF<float>::CH + lane * 4, wx[q < QC ? q : 0]);
                ldw<A::kStream>(pc + (q * 2 + 1) * WF<float>::CH + lane * 4, wy[q < QC ? q : 0]);
            }
            if (q < QV && q < a.V4) ldw<A::kStream>(ph + q * WF<float>::CH + lane * 4, wh[q < QV ? q : 0]);
        }
    };
    load();
    stage_rounds<2, Val3<float>>(
        list, hc,
        [&](int j) {
            Val3<float> v;
            v.x = S::ld1(a.E, j);
            S::ld2(a.H, j, v.y, v.z);
            return v;
        },
        [&](int k, const Val3<float>& v) {
            sE[k] = v.x;
            st_lds2(sH + 2 * k, v.y, v.z);
        });
    const int64_t i = in ? tile * RBFFD_TILE + lane : a.N;
    const int64_t ic = i < a.N ? i : a.N - 1;
    const float e0 = S::ld1(a.E, ic);
    float hx0, hy0;
    S::ld2(a.H, ic, hx0, hy0);
    __syncthreads();
    const float G = (float)a.g;
    if (!(job & kOnlyE)) {
        float dx = 0, dy = 0, vx = 0, vy = 0;
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            if (q < QC && q < a.C4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float de = sE[pos4(li[q / 2], q & 1, u)] - e0;
                    dx += wx[q < QC ? q : 0][u] * de;
                    dy += wy[q < QC ? q : 0][u] * de;
                }
            }
            if (q < QV && q < a.V4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    float hx, hy;
                    ld_lds2(sH + 2 * pos4(li[q / 2], q & 1, u), hx, hy);
                    vx += wh[q < QV ? q : 0][u] * (hx - hx0);
                    vy += wh[q < QV ? q : 0][u] * (hy - hy0);
                }
            }
        }
        const float F = (float)a.aH;
        hx0 = hx0 + F * (-dy + G * vx);
        hy0 = hy0 + F * (dx + G * vy);
        if (i < a.N) __hip_atomic_store(a.Hn + i, pair_bits(hx0, hy0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stores_done();
        __syncthreads();
        if (threadIdx.x == 0) __hip_atomic_store(a.flags + wg, a.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (in) record_receivers<float, float>(a, i);
        if (job & kOnlyH) return;
    }
    // H of the halo's tiles, as long as the patience lasts; then what is missing is
    // computed here as well, so that no order of dispatch can keep a workgroup waiting
    const uint64_t t0 = wall_clock64();
    bool ok;
    for (;;) {
        ok = true;
        for (int k = (int)threadIdx.x; k < hc; k += 256)
            ok &= __hip_atomic_load(a.flags + list[k] / RBFFD_WGT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.tag;
        if (__all(ok) || wall_clock64() - t0 > (uint64_t)a.patience) break;
        __builtin_amdgcn_s_sleep(1);
    }
    if (__syncthreads_or(!ok)) {
        // ascending, each once: a run RBFFD_STEP_RUNS later may overwrite flags
        for (int last = -1;;) {
            if (threadIdx.x == 0) want = INT32_MAX;
            __syncthreads();
            for (int k = (int)threadIdx.x; k < hc; k += 256) {
                const int t = list[k] / RBFFD_WGT;
                if (__hip_atomic_load(a.flags + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.tag && t > last)
                    atomicMin(&want, t);
            }
            __syncthreads();
            const int t = want;
            if (t == INT32_MAX) break;
            last = t;
            whole_h_late(a, t);
            stores_done();
            __syncthreads();
            if (threadIdx.x == 0) {
                __hip_atomic_store(a.flags + t, a.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                atomicAdd(a.late, 1);
                stores_done();
            }
            __syncthreads();
        }
        load();
    }
    stage_rounds<2, uint64_t>(
        list, hc, [&](int j) { return __hip_atomic_load(a.Hn + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
        [&](int k, uint64_t v) { st_lds2(sH + 2 * k, __uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32))); });
    if (job & kOnlyE) {
        const uint64_t v = __hip_atomic_load(a.Hn + ic, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        hx0 = __uint_as_float((uint32_t)v);
        hy0 = __uint_as_float((uint32_t)(v >> 32));
    }
    __syncthreads();
    float cu = 0, ve = 0;
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        if (q < QC && q < a.C4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float hx, hy;
                ld_lds2(sH + 2 * pos4(li[q / 2], q & 1, u), hx, hy);
                cu += wx[q < QC ? q : 0][u] * (hy - hy0) - wy[q < QC ? q : 0][u] * (hx - hx0);
            }
        }
        if (q < QV && q < a.V4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) ve += wh[q < QV ? q : 0][u] * (sE[pos4(li[q / 2], q & 1, u)] - e0);
        }
    }
    if (i < a.N) {
        const float k = kappa_of(a, i);
        S::st1(a.out, i, sourced<float, float>(a, i, a.nomask || (a.emask[i] & 1), e0 + k * (cu + G * ve)));
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(RBFFD_WGT_3D_F32) void k_h3l(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    TC* sE = lds_base<TC>();                           // 3 values per entry
    TC* sH = sE + 3 * (int64_t)a.hmax;
    const int wg = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int h0 = a.hoff[wg], hc = a.hoff[wg + 1] - h0;
    stage_rounds<4, Val6<TC>>(
        a.hpool + h0, hc,
        [&](int j) {
            Val6<TC> v;
            S::ld3(a.E, j, v.v[0], v.v[1], v.v[2]);
            S::ld3(a.H, j, v.v[3], v.v[4], v.v[5]);
            return v;
        },
        [&](int k, const Val6<TC>& v) {
            const TC e[3] = {v.v[0], v.v[1], v.v[2]}, hh[3] = {v.v[3], v.v[4], v.v[5]};
            st_lds3(sE + 3 * k, e);
            st_lds3(sH + 3 * k, hh);
        });
    __syncthreads();
    const int64_t tile = (int64_t)wg * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC ex0, ey0, ez0, hx0, hy0, hz0;
    S::ld3(a.E, ic, ex0, ey0, ez0);
    S::ld3(a.H, ic, hx0, hy0, hz0);
    TC xEy = 0, xEz = 0, yEx = 0, yEz = 0, zEx = 0, zEy = 0, vx = 0, vy = 0, vz = 0;
    const uint4* pl = a.lidx + tile * a.Q8 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 3 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const int qm = max(a.C4, a.V4);
    // chunk q + 1 is loaded while chunk q is summed
    uint4 li = ldpos<A::kStream>(pl);
    TW nx[4] = {0, 0, 0, 0}, ny[4] = {0, 0, 0, 0}, nz[4] = {0, 0, 0, 0}, nh[4] = {0, 0, 0, 0};
    load3<A::kStream>(pc, ph, 0, a.C4, a.V4, nx, ny, nz, nh);
    for (int q = 0; q < qm; ++q) {
        const uint4 lc = li;
        TW wx[4], wy[4], wz[4], wh[4];
        copy4(wx, nx); copy4(wy, ny); copy4(wz, nz); copy4(wh, nh);
        if (q + 1 < qm) {
            if (((q + 1) & 1) == 0) li = ldpos<A::kStream>(pl + ((q + 1) >> 1) * RBFFD_TILE);
            load3<A::kStream>(pc, ph, q + 1, a.C4, a.V4, nx, ny, nz, nh);
        }
        const int hf = q & 1;
        if (q < a.C4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = pos4(lc, hf, u);
                TC v[3];
                ld_lds3(sE + 3 * k, v);
                const TC ex = v[0] - ex0, ey = v[1] - ey0, ez = v[2] - ez0;
                xEy += (TC)wx[u] * ey; xEz += (TC)wx[u] * ez;
                yEx += (TC)wy[u] * ex; yEz += (TC)wy[u] * ez;
                zEx += (TC)wz[u] * ex; zEy += (TC)wz[u] * ey;
            }
        }
        if (q < a.V4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                TC v[3];
                ld_lds3(sH + 3 * pos4(lc, hf, u), v);
                vx += (TC)wh[u] * (v[0] - hx0);
                vy += (TC)wh[u] * (v[1] - hy0);
                vz += (TC)wh[u] * (v[2] - hz0);
            }
        }
    }
    record_receivers<TS, TW>(a, i);
    if (i < a.N) {
        const TC F = (TC)a.a, G = (TC)a.g;
        S::st3(a.out, i, hx0 - F * ((yEz - zEy) - G * vx), hy0 - F * ((zEx - xEz) - G * vy),
               hz0 - F * ((xEy - yEx) - G * vz));
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(RBFFD_WGT_3D_F32) void k_e3l(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    TC* sE = lds_base<TC>();
    TC* sH = sE + 3 * (int64_t)a.hmax;
    const int wg = tile_back(a.xcd);
    const int h0 = a.hoff[wg], hc = a.hoff[wg + 1] - h0;
    stage_rounds<4, Val6<TC>>(
        a.hpool + h0, hc,
        [&](int j) {
            Val6<TC> v;
            S::ld3(a.E, j, v.v[0], v.v[1], v.v[2]);
            S::ld3(a.H, j, v.v[3], v.v[4], v.v[5]);
            return v;
        },
        [&](int k, const Val6<TC>& v) {
            const TC e[3] = {v.v[0], v.v[1], v.v[2]}, hh[3] = {v.v[3], v.v[4], v.v[5]};
            st_lds3(sE + 3 * k, e);
            st_lds3(sH + 3 * k, hh);
        });
    __syncthreads();
    const int64_t tile = (int64_t)wg * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (tile >= a.tiles) return;
    const int lane = threadIdx.x & 63;
    const int64_t i = tile * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC ex0, ey0, ez0, hx0, hy0, hz0;
    S::ld3(a.E, ic, ex0, ey0, ez0);
    S::ld3(a.H, ic, hx0, hy0, hz0);
    TC xHy = 0, xHz = 0, yHx = 0, yHz = 0, zHx = 0, zHy = 0, vx = 0, vy = 0, vz = 0;
    const uint4* pl = a.lidx + tile * a.Q8 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tile * a.C4 * 3 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tile * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const int qm = max(a.C4, a.V4);
    uint4 li = ldpos<A::kStream>(pl);
    TW nx[4] = {0, 0, 0, 0}, ny[4] = {0, 0, 0, 0}, nz[4] = {0, 0, 0, 0}, nh[4] = {0, 0, 0, 0};
    load3<A::kStream>(pc, ph, 0, a.C4, a.V4, nx, ny, nz, nh);
    for (int q = 0; q < qm; ++q) {
        const uint4 lc = li;
        TW wx[4], wy[4], wz[4], wh[4];
        copy4(wx, nx); copy4(wy, ny); copy4(wz, nz); copy4(wh, nh);
        if (q + 1 < qm) {
            if (((q + 1) & 1) == 0) li = ldpos<A::kStream>(pl + ((q + 1) >> 1) * RBFFD_TILE);
            load3<A::kStream>(pc, ph, q + 1, a.C4, a.V4, nx, ny, nz, nh);
        }
        const int hf = q & 1;
        if (q < a.C4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = pos4(lc, hf, u);
                TC v[3];
                ld_lds3(sH + 3 * k, v);
                const TC hx = v[0] - hx0, hy = v[1] - hy0, hz = v[2] - hz0;
                xHy += (TC)wx[u] * hy; xHz += (TC)wx[u] * hz;
                yHx += (TC)wy[u] * hx; yHz += (TC)wy[u] * hz;
                zHx += (TC)wz[u] * hx; zHy += (TC)wz[u] * hy;
            }
        }
        if (q < a.V4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                TC v[3];
                ld_lds3(sE + 3 * pos4(lc, hf, u), v);
                vx += (TC)wh[u] * (v[0] - ex0);
                vy += (TC)wh[u] * (v[1] - ey0);
                vz += (TC)wh[u] * (v[2] - ez0);
            }
        }
    }
    if (i < a.N) {
        const TC k = kappa_of(a, i), G = (TC)a.g;
        TC nx = ex0 + k * ((yHz - zHy) + G * vx);
        TC ny = ey0 + k * ((zHx - xHz) + G * vy);
        TC nz = ez0 + k * ((xHy - yHx) + G * vz);
        const uint8_t m = a.emask[i];
        wall3(m, a.wnrm, i, nx, ny, nz);
        sourced3<TS, TW>(a, i, m, nx, ny, nz);
        S::st3(a.out, i, nx, ny, nz);
    }
}

// ---- 3D, two-phase staging ----------------------------------------------------
// When the halo values of both operands do not fit the LDS budget together
// (FP64), the operand of the curl is staged and summed first, then the same
// LDS holds the operand of the hyperviscosity term.  Every accumulator runs
// over the slots in the same order as in the kernels above, so the results
// are the same.  Workgroups keep their idle wavefronts (a partial last
// workgroup) through both barriers.
template <typename TS>
__device__ __forceinline__ void stage_vec3(const TS* F, const int32_t* list, int hc,
                                           typename Store<TS>::C* s) {
    using S = Store<TS>;
    using TC = typename S::C;
    stage_rounds<4, Val3<TC>>(
        list, hc,
        [&](int j) {
            Val3<TC> v;
            S::ld3(F, j, v.x, v.y, v.z);
            return v;
        },
        [&](int k, const Val3<TC>& v) {
            const TC w[3] = {v.x, v.y, v.z};
            st_lds3(s + 3 * k, w);
        });
}

// curl sums over the curl slots: d_x, d_y, d_z of the staged 3-vector field
// (reference values f0) into the six accumulators c[0..5] =
// (x f_y, x f_z, y f_x, y f_z, z f_x, z f_y)
template <bool STREAM, typename TC, typename TW>
__device__ __forceinline__ void curl_sums3(const TC* sF, const uint4* pl, const TW* pc, int C4, const TC (&f0)[3],
                                           TC (&c)[6]) {
    uint4 li = ldpos<STREAM>(pl);
    TW nx[4] = {0, 0, 0, 0}, ny[4] = {0, 0, 0, 0}, nz[4] = {0, 0, 0, 0}, nh[4];
    load3<STREAM>(pc, (const TW*)nullptr, 0, C4, 0, nx, ny, nz, nh);
    for (int q = 0; q < C4; ++q) {
        const uint4 lc = li;
        TW wx[4], wy[4], wz[4];
        copy4(wx, nx); copy4(wy, ny); copy4(wz, nz);
        if (q + 1 < C4) {
            if (((q + 1) & 1) == 0) li = ldpos<STREAM>(pl + ((q + 1) >> 1) * RBFFD_TILE);
            load3<STREAM>(pc, (const TW*)nullptr, q + 1, C4, 0, nx, ny, nz, nh);
        }
        const int hf = q & 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC v[3];
            ld_lds3(sF + 3 * pos4(lc, hf, u), v);
            const TC fx = v[0] - f0[0], fy = v[1] - f0[1], fz = v[2] - f0[2];
            c[0] += (TC)wx[u] * fy; c[1] += (TC)wx[u] * fz;
            c[2] += (TC)wy[u] * fx; c[3] += (TC)wy[u] * fz;
            c[4] += (TC)wz[u] * fx; c[5] += (TC)wz[u] * fy;
        }
    }
}

// hyperviscosity sums over the HV slots of the staged 3-vector field
template <bool STREAM, typename TC, typename TW>
__device__ __forceinline__ void hv_sums3(const TC* sF, const uint4* pl, const TW* ph, int V4, const TC (&f0)[3],
                                         TC (&v3)[3]) {
    uint4 li = ldpos<STREAM>(pl);
    TW nx[4], ny[4], nz[4], nh[4] = {0, 0, 0, 0};
    load3<STREAM>((const TW*)nullptr, ph, 0, 0, V4, nx, ny, nz, nh);
    for (int q = 0; q < V4; ++q) {
        const uint4 lc = li;
        TW wh[4];
        copy4(wh, nh);
        if (q + 1 < V4) {
            if (((q + 1) & 1) == 0) li = ldpos<STREAM>(pl + ((q + 1) >> 1) * RBFFD_TILE);
            load3<STREAM>((const TW*)nullptr, ph, q + 1, 0, V4, nx, ny, nz, nh);
        }
        const int hf = q & 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            TC v[3];
            ld_lds3(sF + 3 * pos4(lc, hf, u), v);
            v3[0] += (TC)wh[u] * (v[0] - f0[0]);
            v3[1] += (TC)wh[u] * (v[1] - f0[1]);
            v3[2] += (TC)wh[u] * (v[2] - f0[2]);
        }
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(RBFFD_WGT_3D_F32) void k_h3p(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    TC* sF = lds_base<TC>();
    const int wg = a.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int h0 = a.hoff[wg], hc = a.hoff[wg + 1] - h0;
    const int64_t tile = (int64_t)wg * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const bool live = tile < a.tiles;
    const int64_t tl = live ? tile : a.tiles - 1;
    const int lane = threadIdx.x & 63;
    const int64_t i = tl * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC e0[3], h0v[3];
    S::ld3(a.E, ic, e0[0], e0[1], e0[2]);
    S::ld3(a.H, ic, h0v[0], h0v[1], h0v[2]);
    TC c[6] = {0, 0, 0, 0, 0, 0}, v[3] = {0, 0, 0};
    const uint4* pl = a.lidx + tl * a.Q8 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tl * a.C4 * 3 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tl * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    stage_vec3<TS>(a.E, a.hpool + h0, hc, sF);
    __syncthreads();
    if (live) curl_sums3<A::kStream, TC, TW>(sF, pl, pc, a.C4, e0, c);
    __syncthreads();
    stage_vec3<TS>(a.H, a.hpool + h0, hc, sF);
    __syncthreads();
    if (live) hv_sums3<A::kStream, TC, TW>(sF, pl, ph, a.V4, h0v, v);
    if (live) record_receivers<TS, TW>(a, i);
    if (live && i < a.N) {
        const TC F = (TC)a.a, G = (TC)a.g;
        // c = (xEy, xEz, yEx, yEz, zEx, zEy)
        S::st3(a.out, i, h0v[0] - F * ((c[3] - c[5]) - G * v[0]), h0v[1] - F * ((c[4] - c[1]) - G * v[1]),
               h0v[2] - F * ((c[0] - c[2]) - G * v[2]));
    }
}

template <typename TS, typename TW, typename A>
__global__ __launch_bounds__(RBFFD_WGT_3D_F32) void k_e3p(A a) {
    using S = Store<TS>;
    using TC = typename S::C;
    TC* sF = lds_base<TC>();
    const int wg = tile_back(a.xcd);
    const int h0 = a.hoff[wg], hc = a.hoff[wg + 1] - h0;
    const int64_t tile = (int64_t)wg * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const bool live = tile < a.tiles;
    const int64_t tl = live ? tile : a.tiles - 1;
    const int lane = threadIdx.x & 63;
    const int64_t i = tl * RBFFD_TILE + lane;
    const int64_t ic = i < a.N ? i : a.N - 1;
    TC e0[3], h0v[3];
    S::ld3(a.E, ic, e0[0], e0[1], e0[2]);
    S::ld3(a.H, ic, h0v[0], h0v[1], h0v[2]);
    TC c[6] = {0, 0, 0, 0, 0, 0}, v[3] = {0, 0, 0};
    const uint4* pl = a.lidx + tl * a.Q8 * RBFFD_TILE + lane;
    const TW* pc = a.wc + tl * a.C4 * 3 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    const TW* ph = a.wh + tl * a.V4 * RBFFD_TILE * 4 + lane * WChunk<TW>::LS;
    stage_vec3<TS>(a.H, a.hpool + h0, hc, sF);
    __syncthreads();
    if (live) curl_sums3<A::kStream, TC, TW>(sF, pl, pc, a.C4, h0v, c);
    __syncthreads();
    stage_vec3<TS>(a.E, a.hpool + h0, hc, sF);
    __syncthreads();
    if (live) hv_sums3<A::kStream, TC, TW>(sF, pl, ph, a.V4, e0, v);
    if (live && i < a.N) {
        const TC k = kappa_of(a, i), G = (TC)a.g;
        // c = (xHy, xHz, yHx, yHz, zHx, zHy)
        TC nx = e0[0] + k * ((c[3] - c[5]) + G * v[0]);
        TC ny = e0[1] + k * ((c[4] - c[1]) + G * v[1]);
        TC nz = e0[2] + k * ((c[0] - c[2]) + G * v[2]);
        const uint8_t m = a.emask[i];
        wall3(m, a.wnrm, i, nx, ny, nz);
        sourced3<TS, TW>(a, i, m, nx, ny, nz);
        S::st3(a.out, i, nx, ny, nz);
    }
}

// ---- auxiliaries of a run -----------------------------------------------------
// More sources than the E update looks through per node (kMaxFoldedSources):
// E[node] += amp * wave in source order after the bracket, one thread.
constexpr int kMaxFoldedSources = 16;
template <typename TS>
__global__ void k_source(TS* E, int FE, int comp, const uint8_t* emask, const double* wn, int S, const int32_t* node,
                         const void* amp, const void* wave) {
    using St = Store<TS>;
    using TC = typename St::C;
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    for (int s = 0; s < S; ++s) {
        const int64_t i = node[s];
        const int64_t e = i * FE + comp;
        const TC v = source_term<TC>(amp, wave, s);
        if (emask[i] & 8) {
            // curved 3D wall: E is already projected on the normal n, so adding
            // the projected source v n_comp n keeps (E + v e_comp) projected
            const double* n = wn + 3 * i;
            for (int c = 0; c < 3; ++c)
                St::st1(E, i * FE + c, St::ld1(E, i * FE + c) + v * (TC)n[comp] * (TC)n[c]);
            continue;
        }
        const TC cur = St::ld1(E, e);
        St::st1(E, e, ((emask[i] >> comp) & 1) ? cur + v : (TC)0);
    }
}

// the trace row of a run's last step (the earlier ones: record_receivers)
template <typename TS>
__global__ void k_receivers(const TS* E, int FE, int comp, int R, const int32_t* node, void* trace) {
    using St = Store<TS>;
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < R) ((typename St::C*)trace)[r] = St::ld1(E, (int64_t)node[r] * FE + comp);
}

// checkpoint: (E, H) into one slot, E first, in units of U
template <typename U>
__global__ __launch_bounds__(256) void k_ckpt(const U* E, int64_t e, const U* H, int64_t h, U* slot) {
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < e + h; g += (int64_t)gridDim.x * blockDim.x)
        slot[g] = g < e ? E[g] : H[g - e];
}

// ---- FP64 reductions --------------------------------------------------------

template <typename TS>
__global__ __launch_bounds__(256) void k_energy1(const TS* E, int64_t NE, int FE, int fe, const TS* Ha, const TS* Hb,
                                                 int64_t NH, int FH, int fh, double wE, double wH, double* part) {
    using St = Store<TS>;
    __shared__ double sh[256];
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < NE; i += stride)
        for (int c = 0; c < fe; ++c) {
            const double v = (double)St::ld1(E, i * FE + c);
            acc += wE * v * v;
        }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < NH; i += stride)
        for (int c = 0; c < fh; ++c) {
            const double v = 0.5 * ((double)St::ld1(Ha, i * FH + c) + (double)St::ld1(Hb, i * FH + c));
            acc += wH * v * v;
        }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void k_reduce2(const double* part, int nparts, double* out) {
    __shared__ double sh[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) acc += part[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sh[0];
}

template <typename TS>
__global__ __launch_bounds__(256) void k_compare1(const TS* F, int64_t N, int FS, int nc, const double* ref,
                                                  double* part) {
    using St = Store<TS>;
    __shared__ double sh[3][256];
    double se[4] = {0, 0, 0, 0}, sr[4] = {0, 0, 0, 0}, mx[4] = {0, 0, 0, 0};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride)
        for (int c = 0; c < nc; ++c) {
            const double f = (double)St::ld1(F, i * FS + c), r = ref[i * nc + c];
            const double e = f - r;
            se[c] += e * e;
            sr[c] += r * r;
            mx[c] = fmax(mx[c], fabs(e));
        }
    for (int c = 0; c < nc; ++c) {
        sh[0][threadIdx.x] = se[c];
        sh[1][threadIdx.x] = sr[c];
        sh[2][threadIdx.x] = mx[c];
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if (threadIdx.x < s) {
                sh[0][threadIdx.x] += sh[0][threadIdx.x + s];
                sh[1][threadIdx.x] += sh[1][threadIdx.x + s];
                sh[2][threadIdx.x] = fmax(sh[2][threadIdx.x], sh[2][threadIdx.x + s]);
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            part[(blockIdx.x * nc + c) * 3 + 0] = sh[0][0];
            part[(blockIdx.x * nc + c) * 3 + 1] = sh[1][0];
            part[(blockIdx.x * nc + c) * 3 + 2] = sh[2][0];
        }
        __syncthreads();
    }
}

__global__ void k_compare2(const double* part, int nb, int nc, double* out) {
    const int c = threadIdx.x;
    if (c >= nc) return;
    double se = 0, sr = 0, mx = 0;
    for (int b = 0; b < nb; ++b) {
        se += part[(b * nc + c) * 3 + 0];
        sr += part[(b * nc + c) * 3 + 1];
        mx = fmax(mx, part[(b * nc + c) * 3 + 2]);
    }
    out[c * 3 + 0] = se;
    out[c * 3 + 1] = sr;
    out[c * 3 + 2] = mx;
}

}  // namespace

// ---------------------------------------------------------------------------
// Host side: launching one half step of either kind
// ---------------------------------------------------------------------------
namespace {

template <typename TS, typename TW>
void fill_sa(const rbffd_plan* p, const OpBlock& o, SA<TS, TW>& a, bool hupd) {
    a.idx = (const int4*)o.pidx;
    a.idx_h = (const int4*)o.pidx_h;
    a.pref = o.pref;
    a.wc = (const TW*)o.pwc;
    a.wh = (const TW*)o.pwh;
    a.N = o.Nt;
    a.tiles = o.tiles;
    a.C4 = o.C4;
    a.V4 = o.V4;
    a.S4 = o.S4;
    a.xcd = p->var.xcd;
    a.g = p->gamma;
    a.dt = p->dt;
    a.eps0 = p->p.eps0;
    a.a = hupd ? p->dt / p->p.mu0 : p->dt / p->p.eps0;
    a.emask = p->E.emask;
    a.wnrm = p->E.nrm;
    a.lidx = (const uint4*)o.lidx;
    a.hpool = o.hpool;
    a.hoff = o.hoff;
    a.Q8 = o.Q8;
    a.hmax = o.hmax;
}

// whether the plan's variant takes the small-set kernels; a 3D FP32 tile whose
// values do not fit a CU's LDS takes the staged ones
bool small_set(const rbffd_plan* p, const OpBlock& o) {
    if (p->var.lds != 3) return false;
    return p->dim == 2 || p->p.fdtype == RBFFD_F64 || small3_lds(o) <= RBFFD_LDS_CU;
}

// weights and positions of a staged operator
int64_t node_bytes(const rbffd_plan* p, const OpBlock& o) {
    return (int64_t)(o.C4 * p->dim + o.V4) * chunk_bytes(p->p.wdtype) + o.Q8 * 16;
}
int64_t operator_bytes(const rbffd_plan* p, const OpBlock& o) { return o.tiles * RBFFD_TILE * node_bytes(p, o); }

// whether the operator of a staged half step (weights and positions) streams from
// memory rather than staying in cache (RBFFD_CACHED_BYTES)
bool streams(const rbffd_plan* p, const OpBlock& o) {
    const int64_t node = node_bytes(p, o), bytes = operator_bytes(p, o);
    if (p->dim == 2 && p->p.fdtype != RBFFD_F64 && o.Nt < RBFFD_CACHED_F32) return true;
    if (p->dim == 2 && node <= RBFFD_BAND_NODE && bytes > RBFFD_BAND_LO && bytes < RBFFD_BAND_HI) return true;
    return bytes > RBFFD_CACHED_BYTES;
}

// what a run folds into one half step (null pointers: nothing)
struct HalfAux {
    const int32_t* rcv = nullptr;   // H update
    void* trace = nullptr;
    const int32_t* src = nullptr;   // E update
    const void* samp = nullptr;
    const void* swave = nullptr;
    int n_rcv = 0, n_src = 0;
};

// kernel K with the auxiliaries of a run when this half step has any; staged
// kernels also by whether the operator streams or stays cached
#define RBFFD_LAUNCH_HALF(K, grid, block, lds)                                                              \
    do {                                                                                                    \
        if (aux) hipLaunchKernelGGL((K<TS, TW, SX<TS, TW>>), grid, block, lds, st, a);                       \
        else hipLaunchKernelGGL((K<TS, TW, SA<TS, TW>>), grid, block, lds, st, (const SA<TS, TW>&)a);        \
    } while (0)

#define RBFFD_LAUNCH_STAGED(K, grid, block, lds)                                                            \
    do {                                                                                                    \
        using SAt = SA<TS, TW>;                                                                             \
        using SXt = SX<TS, TW>;                                                                             \
        if (stream) RBFFD_LAUNCH_HALF(K, grid, block, lds);                                                 \
        else if (aux) hipLaunchKernelGGL((K<TS, TW, Cached<SXt>>), grid, block, lds, st, Cached<SXt>(a));     \
        else hipLaunchKernelGGL((K<TS, TW, Cached<SAt>>), grid, block, lds, st, Cached<SAt>((const SAt&)a));  \
    } while (0)

template <typename TS, typename TW>
void launch_half(const rbffd_plan* p, bool hupd, const void* E, const void* H, void* out, const void* eps_r,
                 const HalfAux& x, hipStream_t st) {
    // compressed (W22) weights exist only for the 2D collocated kernels
    constexpr bool kW22 = std::is_same<TW, w22>::value;
    const OpBlock& o = hupd ? p->opH : p->opE;
    SX<TS, TW> a{};
    fill_sa<TS, TW>(p, o, a, hupd);
    a.E = (const TS*)E;
    a.H = (const TS*)H;
    a.out = (TS*)out;
    a.eps_r = hupd ? nullptr : eps_r;
    a.FE = p->FE;
    a.comp = p->dim == 2 ? 0 : 2;
    a.n_rcv = x.n_rcv;
    a.rcv = x.rcv;
    a.trace = x.trace;
    a.n_src = x.n_src;
    a.src = x.src;
    a.samp = x.samp;
    a.swave = x.swave;
    const bool aux = (hupd ? x.n_rcv : x.n_src) > 0;
    if (p->p.pol == RBFFD_POL_TE) {
        // TEz: the Hz update runs the scalar (E-update) kernel on (Hz, E) and
        // the E update the vector (H-update) kernel on (Hz_new, E); the
        // scalar kernel's factor is -dt/mu0, both take -gamma
        a.E = (const TS*)H;
        a.H = (const TS*)E;
        a.g = -p->gamma;
        a.a = hupd ? -p->dt / p->p.mu0 : p->dt / p->p.eps0;
        a.nomask = hupd ? 1 : 0;
        a.te = hupd ? 0 : 1;
        hupd = !hupd;
    }
    if (small_set(p, o)) {
        const dim3 grid((unsigned)o.tiles), block(p->dim == 2 ? 256 : 64 * kSplit3);
        if (p->dim == 2 && p->collocated) {
            if (hupd) RBFFD_LAUNCH_HALF(k_h2s, grid, block, 0);
            else RBFFD_LAUNCH_HALF(k_e2s, grid, block, 0);
            return;
        }
        if constexpr (!kW22) {   // compressed weights: 2D collocated plans only
            if (p->dim == 2) {
                if (hupd) RBFFD_LAUNCH_HALF(k_h2xs, grid, block, 0);
                else RBFFD_LAUNCH_HALF(k_e2xs, grid, block, 0);
            } else {
                const size_t lds = std::is_same<TS, double>::value ? 0 : small3_lds(o);
                if (hupd) RBFFD_LAUNCH_HALF(k_h3s, grid, block, lds);
                else RBFFD_LAUNCH_HALF(k_e3s, grid, block, lds);
            }
        }
        return;
    }
    if (p->collocated && o.hmax > 0 && p->var.lds) {
        using TC = typename Store<TS>::C;
        const bool stream = streams(p, o);
        const dim3 grid((unsigned)o.nwg), block(o.wgt);
        if (p->dim == 2) {
            const size_t lds = (size_t)(((o.hmax + 3) & ~3) + 2 * o.hmax) * sizeof(TC);
            if (hupd) RBFFD_LAUNCH_STAGED(k_h2l, grid, block, lds);
            else RBFFD_LAUNCH_STAGED(k_e2l, grid, block, lds);
            return;
        }
        if constexpr (kW22) {
            // compressed weights: 2D collocated plans only (refused at plan creation otherwise)
            return;
        } else if (o.stage == 1 && p->var.lds != 2) {
            const size_t lds = (size_t)6 * o.hmax * sizeof(TC);
            if (hupd) RBFFD_LAUNCH_STAGED(k_h3l, grid, block, lds);
            else RBFFD_LAUNCH_STAGED(k_e3l, grid, block, lds);
        } else {
            const size_t lds = (size_t)3 * o.hmax * sizeof(TC);
            if (hupd) RBFFD_LAUNCH_STAGED(k_h3p, grid, block, lds);
            else RBFFD_LAUNCH_STAGED(k_e3p, grid, block, lds);
        }
        return;
    }
    const int wpb = p->var.block / 64;
    const dim3 grid((unsigned)cdiv(o.tiles, wpb)), block(p->var.block);
    if (p->dim == 2 && p->collocated) {
        if (hupd) RBFFD_LAUNCH_HALF(k_h2, grid, block, 0);
        else RBFFD_LAUNCH_HALF(k_e2, grid, block, 0);
        return;
    }
    if constexpr (!kW22) {
        if (p->dim == 2) {
            if (hupd) RBFFD_LAUNCH_HALF(k_h2x, grid, block, 0);
            else RBFFD_LAUNCH_HALF(k_e2x, grid, block, 0);
        } else {
            if (hupd) RBFFD_LAUNCH_HALF(k_h3, grid, block, 0);
            else RBFFD_LAUNCH_HALF(k_e3, grid, block, 0);
        }
    }
}

#undef RBFFD_LAUNCH_HALF
#undef RBFFD_LAUNCH_STAGED

void half(const rbffd_plan* p, bool hupd, const void* E, const void* H, void* out, const void* eps_r, hipStream_t st,
          const HalfAux& x = HalfAux()) {
    switch (p->p.fdtype) {
        case RBFFD_F64: launch_half<double, double>(p, hupd, E, H, out, eps_r, x, st); break;
        case RBFFD_F32:
            if (p->p.wdtype == RBFFD_W22) launch_half<float, w22>(p, hupd, E, H, out, eps_r, x, st);
            else launch_half<float, float>(p, hupd, E, H, out, eps_r, x, st);
            break;
        default: launch_half<bf16s, float>(p, hupd, E, H, out, eps_r, x, st); break;
    }
}

// ---- whole steps (k_step2) -----------------------------------------------------
using WA = SA<float, float>;
using WX = SX<float, float>;

int32_t* late_count(const OpBlock& o) { return (int32_t*)(o.ord + 2 * o.nwg) + 1; }

size_t whole_lds(const OpBlock& o) { return (size_t)(((o.hmax + 3) & ~3) + 2 * o.hmax) * sizeof(float); }

bool narrow(const OpBlock& o) { return o.C4 <= 6 && o.V4 <= 8; }   // three workgroups per CU, else two

// Whether a run's steps are whole ones: staged 2D FP32 TMz plans whose weights fit
// the registers, and either all workgroups run at once (room) or there are enough
// for the last, part-filled round not to matter: 977 narrow tiles (room 768)
// n 12 whole 29.4, halves 26.7 us; 625 wide ones (room 512) 32.9 / 30.2; 1407 narrow
// 34.6 / 36.5, 977 wide equal.  Too many tiles that come twice (periodic sets, very
// wide ones) cost what the rest gains.
bool whole_steps(const rbffd_plan* p) {
    const OpBlock& o = p->opH;
    if (!can_step_whole(p) || p->var.lds != 1 || !o.hmax || !o.ord || o.C4 > 8 || o.V4 > 16) return false;
    int per = 0, dev = 0, cus = 0;
    const void* k = narrow(o) ? (const void*)k_step2<6, 8, Whole<WX>> : (const void*)k_step2<8, 16, Whole<WX>>;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, RBFFD_WGT, whole_lds(o)) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const int64_t room = (int64_t)per * cus;
    if (room <= 0) return false;
    return o.nwg + o.split <= room || (o.nwg >= room * 7 / 4 && o.split <= o.nwg / 4);
}

template <typename A>
void launch_whole(const rbffd_plan* p, const Whole<A>& a, hipStream_t st) {
    const OpBlock& o = p->opH;
    const dim3 grid((unsigned)(o.nwg + o.split)), block(RBFFD_WGT);
    if (narrow(o)) hipLaunchKernelGGL((k_step2<6, 8, Whole<A>>), grid, block, whole_lds(o), st, a);
    else hipLaunchKernelGGL((k_step2<8, 16, Whole<A>>), grid, block, whole_lds(o), st, a);
}

// one step of a run from (E, H) into (Eout, Hout); tag: the run and the step
void whole_step(const rbffd_plan* p, const void* E, const void* H, void* Eout, void* Hout, const void* eps_r,
                const HalfAux& x, uint64_t tag, uint64_t* flags, hipStream_t st) {
    const OpBlock& o = p->opH;
    WX a{};
    fill_sa<float, float>(p, o, a, false);
    a.E = (const float*)E;
    a.H = (const float*)H;
    a.out = (float*)Eout;
    a.eps_r = eps_r;
    a.FE = p->FE;
    a.n_rcv = x.n_rcv;
    a.rcv = x.rcv;
    a.trace = x.trace;
    a.n_src = x.n_src;
    a.src = x.src;
    a.samp = x.samp;
    a.swave = x.swave;
    auto go = [&](auto w) {
        w.Hn = (uint64_t*)Hout;
        w.flags = flags;
        w.tag = tag;
        w.ord = o.ord;
        w.late = late_count(o);
        w.patience = p->patience;
        w.aH = p->dt / p->p.mu0;
        launch_whole(p, w, st);
    };
    const bool aux = x.n_rcv > 0 || x.n_src > 0;
    // below the L2s' size the next step finds the operator there: 65k nodes (n 25, 26
    // MB) 11.7 -> 10.6 us, 90k (35 MB) 15.5 -> 15.7
    const bool l2 = operator_bytes(p, o) <= ((int64_t)32 << 20);
    if (streams(p, o) && !l2) {
        if (aux) go(Whole<WX>(a));
        else go(Whole<WA>(a));
    } else {
        if (aux) go(Whole<Cached<WX>>(Cached<WX>(a)));
        else go(Whole<Cached<WA>>(Cached<WA>(a)));
    }
}

template <typename TS>
void launch_energy(const rbffd_plan* p, const void* E, const void* Ha, const void* Hb, double* out, RunWS& w,
                   hipStream_t st) {
    const double wE = std::pow(p->E.h, p->dim);
    const double hh = p->collocated ? p->E.h : p->H.h;
    const double wH = p->eta0 * p->eta0 * std::pow(hh, p->dim);
    const int64_t nmax = std::max(p->E.N, p->H.N);
    const int nb = (int)std::min<int64_t>(RED_BLOCKS, cdiv(nmax, 256));
    hipLaunchKernelGGL(k_energy1<TS>, dim3(nb), dim3(256), 0, st, (const TS*)E, p->E.N, p->FE, p->fe_comp,
                       (const TS*)Ha, (const TS*)Hb, p->H.N, p->FH, p->fh_comp, wE, wH, w.part);
    hipLaunchKernelGGL(k_reduce2, dim3(1), dim3(256), 0, st, w.part, nb, out);
}

void energy(const rbffd_plan* p, const void* E, const void* Ha, const void* Hb, double* out, RunWS& w,
            hipStream_t st) {
    switch (p->p.fdtype) {
        case RBFFD_F64: launch_energy<double>(p, E, Ha, Hb, out, w, st); break;
        case RBFFD_F32: launch_energy<float>(p, E, Ha, Hb, out, w, st); break;
        default: launch_energy<bf16s>(p, E, Ha, Hb, out, w, st); break;
    }
}

int check_fields(const rbffd_plan* p, const rbffd_fields* f) {
    if (!f) return set_err(p, RBFFD_EINVAL, "null fields");
    if (!p->ready) return set_err(p, RBFFD_ESTATE, "rbffd_weights has not run");
    if (f->cur != 0 && f->cur != 1) return set_err(p, RBFFD_EINVAL, "fields.cur must be 0 or 1");
    for (int b = 0; b < 2; ++b)
        if (!f->E[b] || !f->H[b]) return set_err(p, RBFFD_EINVAL, "null field buffer");
    if (f->E[0] == f->E[1] || f->H[0] == f->H[1]) return set_err(p, RBFFD_EINVAL, "ping-pong buffers must differ");
    return RBFFD_OK;
}

}  // namespace

// K-field batch (batched.hip)
int batched_step(const rbffd_plan* p, rbffd_fields* f, int32_t nsteps, hipStream_t st);

extern "C" int rbffd_step(const rbffd_plan* p, rbffd_fields* f, int32_t nsteps, void* stream) {
    if (!p) return RBFFD_EINVAL;
    int rc = check_fields(p, f);
    if (rc) return rc;
    if (nsteps < 0) return set_err(p, RBFFD_EINVAL, "nsteps < 0");
    hipStream_t st = (hipStream_t)stream;
    if (p->K > 1) return batched_step(p, f, nsteps, st);
    for (int s = 0; s < nsteps; ++s) {
        const int c = f->cur, o = 1 - c;
        half(p, true, f->E[c], f->H[c], f->H[o], nullptr, st);
        half(p, false, f->E[c], f->H[o], f->E[o], f->eps_r, st);
        f->cur = o;
    }
    HIPCHK(p, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_half(const rbffd_plan* p, const rbffd_fields* f, int32_t which, void* stream) {
    if (!p) return RBFFD_EINVAL;
    int rc = check_fields(p, f);
    if (rc) return rc;
    if (p->K > 1) return set_err(p, RBFFD_ENOTSUP, "rbffd_half is for single-field plans");
    if (which != 0 && which != 1) return set_err(p, RBFFD_EINVAL, "which must be 0 (H) or 1 (E)");
    const int c = f->cur, o = 1 - c;
    if (which == 0) half(p, true, f->E[c], f->H[c], f->H[o], nullptr, (hipStream_t)stream);
    else half(p, false, f->E[c], f->H[o], f->E[o], f->eps_r, (hipStream_t)stream);
    HIPCHK(p, hipGetLastError());
    return RBFFD_OK;
}

namespace {
template <typename TS>
void launch_sources(const rbffd_plan* p, void* E, int n_src, const int32_t* node, const void* amp, const void* wave,
                    hipStream_t st) {
    hipLaunchKernelGGL(k_source<TS>, dim3(1), dim3(64), 0, st, (TS*)E, p->FE, p->dim == 2 ? 0 : 2, p->E.emask, p->E.nrm,
                       n_src, node, amp, wave);
}
void sources(const rbffd_plan* p, void* E, int n_src, const int32_t* node, const void* amp, const void* wave, hipStream_t st) {
    switch (p->p.fdtype) {
        case RBFFD_F64: launch_sources<double>(p, E, n_src, node, amp, wave, st); break;
        case RBFFD_F32: launch_sources<float>(p, E, n_src, node, amp, wave, st); break;
        default: launch_sources<bf16s>(p, E, n_src, node, amp, wave, st);
    }
}
// sources that the E update looks through by itself
void fold_sources(HalfAux& x, int n_src, const int32_t* node, const void* amp, const void* wave) {
    if (n_src <= 0 || n_src > kMaxFoldedSources) return;
    x.n_src = n_src;
    x.src = node;
    x.samp = amp;
    x.swave = wave;
}
template <typename TS>
void launch_receivers(const rbffd_plan* p, const void* E, const rbffd_run_args* a, void* trace, hipStream_t st) {
    hipLaunchKernelGGL(k_receivers<TS>, dim3((unsigned)cdiv(a->n_rcv, 64)), dim3(64), 0, st, (const TS*)E, p->FE,
                       p->dim == 2 ? 0 : 2, a->n_rcv, a->rcv_node, trace);
}
template <typename U>
void launch_ckpt(const void* E, int64_t eb, const void* H, int64_t hb, void* slot, hipStream_t st) {
    const int64_t e = eb / (int64_t)sizeof(U), h = hb / (int64_t)sizeof(U);
    hipLaunchKernelGGL(k_ckpt<U>, dim3((unsigned)std::min<int64_t>(2048, cdiv(e + h, 256))), dim3(256), 0, st,
                       (const U*)E, e, (const U*)H, h, (U*)slot);
}
// (E, H) into one checkpoint slot, in the widest unit that every address and
// length is a multiple of (a slot's H part starts e_bytes into it)
void checkpoint(const void* E, int64_t eb, const void* H, int64_t hb, void* slot, hipStream_t st) {
    const uint64_t m = (uint64_t)E | (uint64_t)H | (uint64_t)slot | (uint64_t)eb | (uint64_t)hb;
    if (m % 16 == 0) launch_ckpt<uint4>(E, eb, H, hb, slot, st);
    else if (m % 8 == 0) launch_ckpt<uint2>(E, eb, H, hb, slot, st);
    else if (m % 4 == 0) launch_ckpt<uint32_t>(E, eb, H, hb, slot, st);
    else launch_ckpt<uint16_t>(E, eb, H, hb, slot, st);
}

// One full step n (buffers c -> o) with what is due in it: the checkpoint
// before it, the energy sample between its halves; receivers and sources are
// part of the half-step kernels.  tag: whole steps (the run's first tag), 0: halves;
// the sample reads only what a whole step leaves alone (E^n) or has written (H^{n+1}).
void full_step(const rbffd_plan* p, const rbffd_fields* f, int c, int n, const rbffd_run_args* a, RunWS& w, uint64_t tag,
               uint64_t* flags, hipStream_t st) {
    const int o = 1 - c;
    const int64_t tb = p->p.fdtype == RBFFD_F64 ? 8 : 4;   // traces, amplitudes, waveforms
    if (a->ckpt && n % a->ckpt_every == 0) {
        const int64_t eb = p->E.N * p->FE * (int64_t)field_elem_bytes(p->p.fdtype);
        const int64_t hb = p->H.N * p->FH * (int64_t)field_elem_bytes(p->p.fdtype);
        checkpoint(f->E[c], eb, f->H[c], hb, (char*)a->ckpt + (int64_t)(n / a->ckpt_every) * (eb + hb), st);
    }
    HalfAux x;
    if (a->n_rcv > 0 && n > 0) {
        x.n_rcv = a->n_rcv;
        x.rcv = a->rcv_node;
        x.trace = (char*)a->traces + (int64_t)(n - 1) * a->n_rcv * tb;
    }
    const void* wave = (const char*)a->src_wave + ((int64_t)n + a->step0) * a->n_src * tb;
    fold_sources(x, a->n_src, a->src_node, a->src_amp, wave);
    if (tag) whole_step(p, f->E[c], f->H[c], f->E[o], f->H[o], f->eps_r, x, tag + n, flags, st);
    else half(p, true, f->E[c], f->H[c], f->H[o], nullptr, st, x);
    if (a->energy_out && a->energy_every > 0 && n % a->energy_every == 0)
        energy(p, f->E[c], f->H[c], f->H[o], a->energy_out + n / a->energy_every, w, st);
    if (!tag) half(p, false, f->E[c], f->H[o], f->E[o], f->eps_r, st, x);
    if (a->n_src > kMaxFoldedSources) sources(p, f->E[o], a->n_src, a->src_node, a->src_amp, wave, st);
    if (a->n_rcv > 0 && n == a->T - 1) {
        void* row = (char*)a->traces + (int64_t)n * a->n_rcv * tb;
        switch (p->p.fdtype) {
            case RBFFD_F64: launch_receivers<double>(p, f->E[o], a, row, st); break;
            case RBFFD_F32: launch_receivers<float>(p, f->E[o], a, row, st); break;
            default: launch_receivers<bf16s>(p, f->E[o], a, row, st);
        }
    }
}

// steps from n to the next one with a sample or checkpoint due (or to T)
int plain_steps(const rbffd_run_args* a, int n) {
    int e = a->T;
    if (a->ckpt) e = std::min(e, (int)cdiv(n, a->ckpt_every) * a->ckpt_every);
    if (a->energy_out && a->energy_every > 0) e = std::min(e, (int)cdiv(n, a->energy_every) * a->energy_every);
    return e - n;
}
}  // namespace

int plain_step_into(const rbffd_plan* p, const void* E, const void* H, void* Eout, void* Hout, const void* eps_r, int n_src,
                    const int32_t* src_node, const void* src_amp, const void* wave, hipStream_t st) {
    HalfAux x;
    fold_sources(x, n_src, src_node, src_amp, wave);
    half(p, true, E, H, Hout, nullptr, st);
    half(p, false, E, Hout, Eout, eps_r, st, x);
    if (n_src > kMaxFoldedSources) sources(p, Eout, n_src, src_node, src_amp, wave, st);
    HIPCHK(p, hipGetLastError());
    return RBFFD_OK;
}

int batched_run(const rbffd_plan* p, rbffd_fields* f, const rbffd_run_args* a, void* ws, hipStream_t st);

extern "C" int rbffd_run(const rbffd_plan* p, rbffd_fields* f, const rbffd_run_args* a, void* ws, void* stream) {
    if (!p || !a) return RBFFD_EINVAL;
    int rc = check_fields(p, f);
    if (rc) return rc;
    if (!ws) return set_err(p, RBFFD_EINVAL, "run needs the workspace");
    if (a->T < 0) return set_err(p, RBFFD_EINVAL, "T < 0");
    hipStream_t st = (hipStream_t)stream;
    if (p->K > 1) return batched_run(p, f, a, ws, st);
    if (p->p.pol == RBFFD_POL_TE && (a->n_src > 0 || a->n_rcv > 0))
        return set_err(p, RBFFD_ENOTSUP, "sources and receivers are implemented for TMz");
    if (a->n_src > 0 && (!a->src_node || !a->src_amp || !a->src_wave))
        return set_err(p, RBFFD_EINVAL, "sources need node, amplitude and waveform arrays");
    if (a->n_rcv > 0 && (!a->rcv_node || !a->traces)) return set_err(p, RBFFD_EINVAL, "receivers need nodes and traces");
    if (a->ckpt && a->ckpt_every <= 0) return set_err(p, RBFFD_EINVAL, "ckpt_every must be positive");
    if (a->energy_out && a->energy_every < 0) return set_err(p, RBFFD_EINVAL, "energy_every < 0");
    RunWS w = run_ws(ws);
    // runs in flight together (streams, replayed captures) have flags of their own; where
    // more than RBFFD_STEP_RUNS meet, the tags differ: flags that a later run overwrote
    // count as missing, and a workgroup computes more, not wrongly
    const uint32_t run = a->T > 0 && whole_steps(p) ? ++p->whole_runs : 0;
    const uint64_t tag = run ? (uint64_t)run << 32 | 1 : 0;
    uint64_t* flags = run ? p->opH.flags + run % RBFFD_STEP_RUNS * p->opH.nwg : nullptr;
    const bool graphs = !tag && a->use_graph && a->n_src <= 0 && a->n_rcv <= 0 && p->opE.tiles <= RBFFD_GRAPH_TILES;
    if (tag)
        hipLaunchKernelGGL(k_no_steps, dim3((unsigned)cdiv(p->opH.nwg, 256)), dim3(256), 0, st, flags, (int)p->opH.nwg);
    int c = f->cur;
    for (int n = 0; n < a->T;) {
        const int plain = graphs ? plain_steps(a, n) : 0;
        // the steps that fill no graph go first: the GPU is at them during the capture
        if (plain >= RBFFD_GRAPH_MIN_STEPS && plain % RBFFD_GRAPH_STEPS == 0) {
            int done = 0;
            rc = replay_steps(
                p, plain, c, st,
                [&](int b, hipStream_t cs) {
                    half(p, true, f->E[b], f->H[b], f->H[1 - b], nullptr, cs);
                    half(p, false, f->E[b], f->H[1 - b], f->E[1 - b], f->eps_r, cs);
                },
                &done);
            if (rc) return rc;
            n += done;   // even: the buffers are back at c
            if (done > 0) continue;
        }
        full_step(p, f, c, n, a, w, tag, flags, st);
        c = 1 - c;
        ++n;
    }
    f->cur = (a->T % 2) ? 1 - f->cur : f->cur;
    HIPCHK(p, hipGetLastError());
    if (a->energy_out && a->energy_every > 0 && a->unstable_threshold > 0 && a->T > 0) {
        const int ne = (a->T - 1) / a->energy_every + 1;
        std::vector<double> e(ne);
        HIPCHK(p, hipMemcpyAsync(e.data(), a->energy_out, ne * 8, hipMemcpyDeviceToHost, st));
        HIPCHK(p, hipStreamSynchronize(st));
        for (int k = 0; k < ne; ++k)
            if (!std::isfinite(e[k]) || e[k] > a->unstable_threshold * e[0])
                return set_err(p, RBFFD_EUNSTABLE, "energy sample " + std::to_string(k) + " = " + std::to_string(e[k]) +
                                                       " exceeds the threshold");
    }
    return RBFFD_OK;
}

extern "C" int rbffd_whole_steps(const rbffd_plan* p, int64_t* out, void* stream) {
    if (!p || !out) return RBFFD_EINVAL;
    if (!p->ready) return set_err(p, RBFFD_ESTATE, "rbffd_weights has not run");
    const OpBlock& o = p->opH;
    int32_t late = 0;
    if (o.ord && o.hmax) {
        hipStream_t st = (hipStream_t)stream;
        HIPCHK(p, hipMemcpyAsync(&late, late_count(o), 4, hipMemcpyDeviceToHost, st));
        HIPCHK(p, hipStreamSynchronize(st));
    }
    out[0] = whole_steps(p);
    out[1] = o.nwg;
    out[2] = o.split;
    out[3] = late;
    return RBFFD_OK;
}

extern "C" int rbffd_set_patience(rbffd_plan* p, int32_t ticks) {
    if (!p) return RBFFD_EINVAL;
    if (ticks < 0) return set_err(p, RBFFD_EINVAL, "patience < 0");
    p->patience = ticks;
    return RBFFD_OK;
}

extern "C" int rbffd_energy(const rbffd_plan* p, const void* E, const void* Ha, const void* Hb, double* out, void* ws,
                            void* stream) {
    if (!p || !E || !Ha || !Hb || !out || !ws) return RBFFD_EINVAL;
    if (!p->ready) return set_err(p, RBFFD_ESTATE, "rbffd_weights has not run");
    if (p->K > 1) return set_err(p, RBFFD_ENOTSUP, "energy of a K-field batch: use rbffd_compare per field");
    RunWS w = run_ws(ws);
    energy(p, E, Ha, Hb, out, w, (hipStream_t)stream);
    HIPCHK(p, hipGetLastError());
    return RBFFD_OK;
}

// ---- energy without a workspace ------------------------------------------------
// rbffd_energy_static runs the same two kernels as rbffd_energy, with the
// per-block FP64 partial sums in this file-scope device array instead of the
// caller's workspace.  Every device holds its own copy at its own address;
// host code uses only that address (looked up once per device), never the
// array's name.  The reduction writes partial b for every block b < nb before
// the second kernel reads partials 0 .. nb - 1, so nothing must start at zero;
// calls that overlap on one device share the array and race.
namespace {
constexpr int kStaticParts = RED_BLOCKS;   // 8 KB of partial sums per device
static __device__ __align__(256) double energy_scratch[kStaticParts];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

int scratch_for(const rbffd_plan* p, hipStream_t st, double** out) {
    int dev = -1;
    if (st) {
        HIPCHK(p, hipStreamGetDevice(st, &dev));
    } else {
        HIPCHK(p, hipGetDevice(&dev));
    }
    if (dev < 0 || dev >= kMaxDevices) return set_err(p, RBFFD_ESIZE, "device ordinal beyond 63");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        int cur = -1;
        HIPCHK(p, hipGetDevice(&cur));
        if (cur != dev) HIPCHK(p, hipSetDevice(dev));
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(energy_scratch));
        if (cur != dev) HIPCHK(p, hipSetDevice(cur));
        if (e != hipSuccess || !ptr)
            return set_err(p, RBFFD_EHIP, std::string("hipGetSymbolAddress(energy_scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[dev] = (double*)ptr;
    }
    *out = g_scratch_ptr[dev];
    return RBFFD_OK;
}
}  // namespace

extern "C" int rbffd_energy_static(const rbffd_plan* p, const void* E, const void* Ha, const void* Hb, double* out,
                                   void* stream) {
    if (!p || !E || !Ha || !Hb || !out) return RBFFD_EINVAL;
    if (!p->ready) return set_err(p, RBFFD_ESTATE, "rbffd_weights has not run");
    if (p->K > 1) return set_err(p, RBFFD_ENOTSUP, "energy of a K-field batch: use rbffd_compare per field");
    const int64_t nmax = std::max(p->E.N, p->H.N);
    if (std::min<int64_t>(RED_BLOCKS, cdiv(nmax, 256)) > kStaticParts)
        return set_err(p, RBFFD_ESIZE, "more reduction blocks than the static scratch holds");
    hipStream_t st = (hipStream_t)stream;
    double* parts = nullptr;
    int rc = scratch_for(p, st, &parts);
    if (rc) return rc;
    RunWS w{};
    w.part = parts;
    energy(p, E, Ha, Hb, out, w, st);
    HIPCHK(p, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_compare(const rbffd_plan* p, int32_t which, const void* F, const double* ref, double* out,
                             void* ws, void* stream) {
    if (!p || !F || !ref || !out || !ws) return RBFFD_EINVAL;
    if (!p->ready) return set_err(p, RBFFD_ESTATE, "rbffd_weights has not run");
    hipStream_t st = (hipStream_t)stream;
    RunWS w = run_ws(ws);
    const bool isE = which == 0;
    const int64_t N = (isE ? p->E.N : p->H.N) * (p->K > 1 ? 1 : 1);
    int FS = isE ? p->FE : p->FH;
    int nc = isE ? p->fe_comp : p->fh_comp;
    int64_t rows = N;
    if (p->K > 1) {
        // batch layout [N][F][K]: compare every (node, comp, k) value as its own row
        rows = N * nc * p->K;
        FS = 1;
        nc = 1;
    }
    const int nb = (int)std::min<int64_t>(RED_BLOCKS, cdiv(rows, 256));
    switch (p->p.fdtype) {
        case RBFFD_F64:
            hipLaunchKernelGGL(k_compare1<double>, dim3(nb), dim3(256), 0, st, (const double*)F, rows, FS, nc, ref, w.part);
            break;
        case RBFFD_F32:
            hipLaunchKernelGGL(k_compare1<float>, dim3(nb), dim3(256), 0, st, (const float*)F, rows, FS, nc, ref, w.part);
            break;
        default:
            hipLaunchKernelGGL(k_compare1<bf16s>, dim3(nb), dim3(256), 0, st, (const bf16s*)F, rows, FS, nc, ref, w.part);
    }
    hipLaunchKernelGGL(k_compare2, dim3(1), dim3(64), 0, st, w.part, nb, nc, out);
    HIPCHK(p, hipGetLastError());
    return RBFFD_OK;
}

// ---------------------------------------------------------------------------
// Launch tuning: workgroup size and the XCD remap, timed on the device
// ---------------------------------------------------------------------------
extern "C" int rbffd_autotune(rbffd_plan* p, rbffd_fields* f, int32_t reps, void* stream) {
    if (!p) return RBFFD_EINVAL;
    int rc = check_fields(p, f);
    if (rc) return rc;
    if (reps < 1) reps = 1;
    hipStream_t st = (hipStream_t)stream;
    // candidate launch variants: single field -- workgroup size x XCD remap
    // for the global-gather kernels, plus the LDS-staged kernels (fixed
    // shape) with and without the remap; K-field batch -- workgroup size x
    // resident workgroups per CU for the global kernels, plus the staged one
    std::vector<Variant> cand;
    const bool staged = p->collocated && p->opH.hmax > 0;
    for (int b : {64, 128, 256, 512}) {
        if (p->K > 1) {
            if (b > 256) continue;
            for (int pe : {4, 8, 16}) cand.push_back(Variant{b, 1, pe, 0});
        } else {
            for (int x : {0, 1}) cand.push_back(Variant{b, x, 8, 0});
        }
    }
    if (staged) {
        if (p->K > 1) {
            // staged batch: 4-field (persist < 8), 8-field or 16-field slices,
            // one item per workgroup or persistent with staging wavefronts
            for (int l : {1, 2})
                for (int pe : {4, 8, 16}) cand.push_back(Variant{256, 1, pe, l});
        } else {
            for (int x : {0, 1}) cand.push_back(Variant{256, x, 8, 1});
            // 3D with both operands fitting: also the one-operand-at-a-time kernels
            if (p->dim == 3 && p->opH.stage == 1) cand.push_back(Variant{256, 1, 8, 2});
        }
    }
    if (p->K == 1) {
        // several wavefronts per 64-node tile (small node sets)
        for (int x : {0, 1}) cand.push_back(Variant{256, x, 8, 3});
    }
    Variant best = p->var;
    float best_ms = 1e30f;
    hipEvent_t e0, e1;
    HIPCHK(p, hipEventCreate(&e0));
    HIPCHK(p, hipEventCreate(&e1));
    for (const Variant& v : cand) {
        p->var = v;
        rc = rbffd_step(p, f, 2, stream);   // warm
        if (rc) break;
        HIPCHK(p, hipEventRecord(e0, st));
        rc = rbffd_step(p, f, reps, stream);
        if (rc) break;
        HIPCHK(p, hipEventRecord(e1, st));
        HIPCHK(p, hipEventSynchronize(e1));
        float ms = 0;
        HIPCHK(p, hipEventElapsedTime(&ms, e0, e1));
        if (ms < best_ms) {
            best_ms = ms;
            best = v;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    p->var = best;
    return rc;
}
