// multi_impl.hpp -- several time steps per launch for small domains (AA
// scheme, compact layout), the populations of a tile held in LDS.
//
// A per-step kernel on a domain of a few thousand nodes costs 4 to 7 us, most
// of it launch, memory latency and the end-of-kernel write-back; the node
// update itself is a chain of 1 to 2 us.  Here a block loads a tile and a halo
// of `steps` nodes once, runs the AA pair (pull, local) in place in LDS with a
// barrier per step, and writes the tile once.  Step s updates the box without
// its s outer layers, so the halo's redundant updates replace all exchange
// between blocks: no grid-wide wait, any number of blocks.  Blocks read one
// population copy and write the other (neighbours still read the first); two
// launches bring the state back.  A domain of one node per thread of a block
// stays in one block for any number of steps, in place.
//
// What bounds it: the dependent chain of a node update and the barrier behind it.
// D3Q19 FP64 IR, 128 x 128 x 4, tile 8 x 8 x 4: a launch of 4 steps takes 19.4 us,
// with 992 vector instructions a wave and the vector unit 26% busy; the box of
// 1024 nodes loads 4 and updates 2 nodes per node of the tile.
// Per step, single steps -> here: that duct 6.7 -> 4.6 us, the 4 x 64 D2Q9
// channel 3.6 -> 0.55 (one block), an 80 x 80 D2Q9 PR cell 3.8 -> 2.0, 400 x 400
// D2Q9 IR 5.8 -> 3.4, 63 x 63 x 4 D3Q27 FP32 PR 5.4 -> 4.0.
//
// Places in LDS are byte addresses formed without branches: own slot plus the
// neighbour's offset under the neighbour's fluid bit.
#pragma once

#include <algorithm>
#include <type_traits>

#include "step_impl.hpp"

namespace lbm {

// Most threads per block, so that the kernel keeps its values in registers:
// 1024 threads leave 128 registers a lane, 768 leave 168, 512 leave 256.  FP64
// needs more in three dimensions and for the operators with a per-node solve.
// A tile of more nodes than threads is walked in rounds; a whole-domain box
// (BOX) holds at most one node per thread.
template <int LAT, int OP, int PREC, bool BOX> constexpr int multi_threads()
{
    const bool solve = op_base(OP) == OP_PRI || op_base(OP) == OP_IRHB;
    const bool pri = op_base(OP) == OP_PRI;
    if (PREC != PREC_F64 && BOX) return LAT == 2 ? (pri ? 512 : 768) : LAT == 1 && pri ? 768 : 1024;
    if (PREC != PREC_F64) return LAT == 2 && (pri || (PREC == PREC_F16 && op_base(OP) == OP_PR)) ? 768 : 1024;
    if (BOX) return LAT != 0 ? 512 : solve ? 768 : 1024;
    return LAT == 2 || (LAT == 1 && op_base(OP) != OP_IR) || solve ? 768 : 1024;
}

// t / n for 0 <= t < 2^13, n >= 1 (a box holds at most 7123 nodes: 160 KB of
// LDS, 23 bytes a node for D2Q9 FP16), inv_n within an ulp of 1 / n: (t + 1/2) / n
// is at least 1 / (2 n) away from an integer, and its rounding below t 2^-22 / n.
__device__ __forceinline__ int small_div(int t, float inv_n) { return (int)(((float)t + 0.5f) * inv_n); }

// Directions whose component along an axis is s (bit i: direction i).
template <int LAT> constexpr uint32_t dirs_with(int axis, int s)
{
    using L = Lattice<LAT>;
    uint32_t m = 0;
    for (int i = 0; i < L::Q; ++i) {
        const int c = axis == 0 ? L::cx[i] : axis == 1 ? L::cy[i] : L::cz[i];
        if (c == s) m |= 1u << i;
    }
    return m;
}

// BOX: one block holds the whole domain, one thread per node, any number of
// steps; else a block holds a tile and its halo, and the nodes of each step
// are dealt to the threads anew.
template <int LAT, int OP, int PREC, bool BOX>
__global__ __launch_bounds__((multi_threads<LAT, OP, PREC, BOX>())) void k_multi(const MultiArgs a)
{
    using L = Lattice<LAT>;
    constexpr int Q = L::Q;
    using S = typename Store<PREC>::S;
    using C = typename Store<PREC>::C;
    using T = typename Store<PREC>::T;

    const int b = blockIdx.x;
    const int tile = BOX ? b : (b & 7) * a.tiles_per_xcd + (b >> 3);
    if (tile >= a.ntiles) return;  // whole block leaves together

    extern __shared__ double multi_lds[];
    const int nbox = a.nbox;  // nodes of the box
    const int M = a.M;        // the same, rounded up to a multiple of 4: stride of the LDS arrays
    S* const pop = (S*)multi_lds;
    T* const tau = (T*)(pop + (size_t)Q * M);
    uint32_t* const nbm = (uint32_t*)(tau + (has_tau(OP) ? M : 0));
    uint32_t* const slot = nbm + M;
    uint8_t* const flag = (uint8_t*)(slot + (a.all_fluid ? 0 : M));

    const int ttx = tile % a.ntx;
    const int tr = tile / a.ntx;
    const int tty = tr % a.nty, ttz = tr / a.nty;
    // global coordinates of the box's first node, extents of the box
    const int x0 = ttx * a.c[0] - a.h[0], y0 = tty * a.c[1] - a.h[1], z0 = ttz * a.c[2] - a.h[2];
    const int ex = a.e[0], ey = a.e[1], ez = a.e[2], exy = ex * ey;
    const float inv_x = __builtin_amdgcn_rcpf((float)ex), inv_xy = __builtin_amdgcn_rcpf((float)exy);

    const Coll<C>& cp = [&]() -> const Coll<C>& {
        if constexpr (PREC == PREC_F64) return a.cd;
        else return a.cf;
    }();
    // bring the constants' lines of the argument block into the scalar cache
    // with the loads below, not in front of the first step (0.7 us a launch)
    asm volatile("" ::"s"(cp.rho0), "s"(cp.g[0]), "s"(cp.ir_a), "s"(cp.axis), "s"(cp.hb_c));

    // global coordinate of box coordinate g, or -1 beyond a wall
    auto wrap = [](int g, int n, int per) -> int {
        if (g >= 0 && g < n) return g;
        if (!per) return -1;
        while (g < 0) g += n;
        while (g >= n) g -= n;
        return g;
    };
    // load the box: every population of every fluid node, and (no solids in
    // the domain) the fluid neighbours, bit i for direction i, bit 0 the node
    const S* A = (const S*)a.src;
    for (int j = threadIdx.x; j < nbox; j += blockDim.x) {
        const int lz = small_div(j, inv_xy), r = j - lz * exy;
        const int ly = small_div(r, inv_x), lx = r - ly * ex;
        const int gx = wrap(x0 + lx, a.n[0], a.per[0]), gy = wrap(y0 + ly, a.n[1], a.per[1]),
                  gz = wrap(z0 + lz, a.n[2], a.per[2]);
        bool fluid = (gx | gy | gz) >= 0;
        const int row = gy + a.n[1] * gz;
        uint32_t k = (uint32_t)(gx + a.n[0] * row);
        if (a.all_fluid) {
            uint32_t m = (1u << Q) - 1u;
            if (!a.per[0]) m &= ~((gx == 0 ? dirs_with<LAT>(0, -1) : 0u) | (gx == a.n[0] - 1 ? dirs_with<LAT>(0, 1) : 0u));
            if (!a.per[1]) m &= ~((gy == 0 ? dirs_with<LAT>(1, -1) : 0u) | (gy == a.n[1] - 1 ? dirs_with<LAT>(1, 1) : 0u));
            if (!a.per[2]) m &= ~((gz == 0 ? dirs_with<LAT>(2, -1) : 0u) | (gz == a.n[2] - 1 ? dirs_with<LAT>(2, 1) : 0u));
            nbm[j] = fluid ? m : 0u;
        } else {
            if (fluid) {
                const int w = row * a.W + (gx >> 6);
                const uint64_t bits = a.bits[w];
                fluid = (bits >> (gx & 63)) & 1;
                k = a.wbase[w] + (uint32_t)__popcll(bits & ((1ull << (gx & 63)) - 1ull));
            }
            flag[j] = fluid;
            slot[j] = k;
        }
        if (fluid) {
#pragma unroll
            for (int i = 0; i < Q; ++i) pop[i * M + j] = A[(int64_t)i * a.s_src + k];
            if constexpr (has_tau(OP)) tau[j] = ((const T*)a.tau_src)[k];
        }
    }
    // offset of the neighbour one node back / forward along an axis; along an
    // axis the box spans it wraps inside (behind a wall its value is not used)
    auto offs = [](int l, int e, int h, int stride, int (&o)[3]) {
        o[0] = (h == 0 && l == 0) ? (e - 1) * stride : -stride;
        o[1] = 0;
        o[2] = (h == 0 && l == e - 1) ? (1 - e) * stride : stride;
    };
    if (!a.all_fluid) {
        __syncthreads();
        for (int j = threadIdx.x; j < nbox; j += blockDim.x) {
            const int lz = small_div(j, inv_xy), r = j - lz * exy;
            const int ly = small_div(r, inv_x), lx = r - ly * ex;
            uint32_t m = 0;
            // nodes on the rim of a haloed axis have no neighbours in the box
            // and are never updated
            const bool rim = (a.h[0] && (lx == 0 || lx == ex - 1)) || (a.h[1] && (ly == 0 || ly == ey - 1)) ||
                             (a.h[2] && (lz == 0 || lz == ez - 1));
            if (!rim && flag[j]) {
                int ox[3], oy[3], oz[3];
                offs(lx, ex, a.h[0], 1, ox);
                offs(ly, ey, a.h[1], ex, oy);
                offs(lz, ez, a.h[2], exy, oz);
                m = 1u;
#pragma unroll
                for (int i = 1; i < Q; ++i)
                    m |= (uint32_t)flag[j + ox[L::cx[i] + 1] + oy[L::cy[i] + 1] + oz[L::cz[i] + 1]] << i;
                // a wall lies behind the end of a spanned, non-periodic axis
                if (!a.h[0] && !a.per[0])
                    m &= ~((lx == 0 ? dirs_with<LAT>(0, -1) : 0u) | (lx == ex - 1 ? dirs_with<LAT>(0, 1) : 0u));
                if (!a.h[1] && !a.per[1])
                    m &= ~((ly == 0 ? dirs_with<LAT>(1, -1) : 0u) | (ly == ey - 1 ? dirs_with<LAT>(1, 1) : 0u));
                if (!a.h[2] && !a.per[2])
                    m &= ~((lz == 0 ? dirs_with<LAT>(2, -1) : 0u) | (lz == ez - 1 ? dirs_with<LAT>(2, 1) : 0u));
            }
            nbm[j] = m;
        }
    }

    // LDS byte addresses of the populations
    constexpr int SZ = (int)sizeof(S);
    using LdsPtr = __attribute__((address_space(3))) S*;
    const int lds0 = (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) double*)multi_lds;
    auto get = [](int at) -> S { return *(LdsPtr)(uintptr_t)(uint32_t)at; };
    auto put = [](int at, S v) { *(LdsPtr)(uintptr_t)(uint32_t)at = v; };
    // hold the Q places through the collision, or form them again after it
    // where the registers are short (FP64, 3-D, tau field or per-node solve)
    constexpr bool KEEP = !(PREC == PREC_F64 && L::D == 3 && op_base(OP) != OP_IR);
    // Place of the population a node pulls along i, which is also where the
    // one it sends along opp(i) goes: the neighbour's slot opp(i) if that node
    // is fluid, else the node's own slot i (as for every i in the local phase).
    auto pull_places = [&](int lx, int ly, int lz, int j, uint32_t m, int (&at)[Q]) {
        int ox[3], oy[3], oz[3];
        offs(lx, ex, a.h[0], SZ, ox);
        offs(ly, ey, a.h[1], SZ * ex, oy);
        offs(lz, ez, a.h[2], SZ * exy, oz);
        const int own = lds0 + SZ * j;
        at[0] = own;
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const int o = opp(i);
            const int d = ox[L::cx[o] + 1] + oy[L::cy[o] + 1] + oz[L::cz[o] + 1] + (o - i) * SZ * M;
            const int fl = (int)(m << (31 - o)) >> 31;  // all ones: fluid
            at[i] = i * SZ * M + own + (fl & d);
        }
    };
    // One node's step: s odd pulls from and sends to the neighbours, s even
    // stays on the node; the last (even) step writes to global memory.  box
    // coordinates (lx, ly, lz), box index j, neighbour flags m.
    auto update = [&](int s, int lx, int ly, int lz, int j, uint32_t m) {
        int at[Q];
        auto places = [&](int j, uint32_t m) {
            if (s & 1) {
                pull_places(lx, ly, lz, j, m, at);
            } else {
#pragma unroll
                for (int i = 0; i < Q; ++i) at[i] = lds0 + SZ * (i * M + j);
            }
        };
        places(j, m);
        C h[Q];
        Moments<C> mo;
        Pre<C> pr;
        bool used_fb = false;
        C tau_prev = C(0);
        if constexpr (has_tau(OP)) tau_prev = (C)tau[j];
#pragma unroll
        for (int i = 0; i < Q; ++i) h[i] = decode<PREC>(get(at[i]), L::w[i], a.h16_scale);
        collide_node<LAT, OP, PREC>(h, tau_prev, 0, a.cd, cp, mo, pr, used_fb);
        if (s < a.steps) {
            if constexpr (!KEEP) {
                asm volatile("" : "+v"(j), "+v"(m));  // hides their history from the optimiser
                places(j, m);
            }
#pragma unroll
            for (int i = 0; i < Q; ++i) put(at[opp(i)], encode<PREC>(h[i], L::w[i], a.h16_inv));
            if constexpr (has_tau(OP)) tau[j] = (T)pr.tau_p;
        } else {
            const int X = x0 + lx, Y = y0 + ly, Z = z0 + lz;
            if (X < a.n[0] && Y < a.n[1] && Z < a.n[2]) {  // the last tiles reach past the domain
                const uint32_t k = a.all_fluid ? (uint32_t)(X + a.n[0] * (Y + a.n[1] * Z)) : slot[j];
                S* const B = (S*)a.dst;
#pragma unroll
                for (int i = 0; i < Q; ++i) B[(int64_t)opp(i) * a.s_dst + k] = encode<PREC>(h[i], L::w[i], a.h16_inv);
                if constexpr (has_tau(OP)) ((T*)a.tau_dst)[k] = (T)pr.tau_p;
            }
        }
    };

    if constexpr (BOX) {
        __syncthreads();
        const int j = threadIdx.x;
        const uint32_t m = j < nbox ? nbm[j] : 0u;
        const int lz = small_div(j, inv_xy), r = j - lz * exy;
        const int ly = small_div(r, inv_x), lx = r - ly * ex;
        for (int s = 1; s <= a.steps; ++s) {
            if (m & 1u) update(s, lx, ly, lz, j, m);
            __syncthreads();
        }
        return;
    }
    for (int s = 1; s <= a.steps; ++s) {
        __syncthreads();
        // nodes of this step: the box without its s outer layers on haloed axes
        const int gx = a.h[0] ? s : 0, gy = a.h[1] ? s : 0, gz = a.h[2] ? s : 0;
        const int mx = ex - 2 * gx, mxy = mx * (ey - 2 * gy), todo = mxy * (ez - 2 * gz);
        const float ix = __builtin_amdgcn_rcpf((float)mx), ixy = __builtin_amdgcn_rcpf((float)mxy);
        for (int t = threadIdx.x; t < todo; t += blockDim.x) {
            int lz = small_div(t, ixy);
            const int r = t - __mul24(lz, mxy);
            int ly = small_div(r, ix);
            const int lx = r - __mul24(ly, mx) + gx;
            ly += gy;
            lz += gz;
            const int j = lx + __mul24(ly, ex) + __mul24(lz, exy);
            const uint32_t m = nbm[j];
            if (m & 1u) update(s, lx, ly, lz, j, m);
        }
    }
}

// max_box non-NULL: report the most nodes a whole-domain box may hold, launch nothing
template <int LAT, int OP, int PREC>
static hipError_t go_multi(const MultiArgs& a, size_t lds, hipStream_t s, int* max_box)
{
    constexpr int box = multi_threads<LAT, OP, PREC, true>(), most = multi_threads<LAT, OP, PREC, false>();
    if (max_box) {
        *max_box = box;
        return hipSuccess;
    }
    const int threads = std::min((a.nbox + 63) / 64 * 64, most);
    if (a.ntiles == 1) {
        if (a.nbox > box) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_multi<LAT, OP, PREC, true>), dim3(1), dim3((unsigned)(a.nbox + 63) / 64 * 64), lds, s, a);
    } else {
        hipLaunchKernelGGL((k_multi<LAT, OP, PREC, false>), dim3(8u * (unsigned)a.tiles_per_xcd),
                           dim3((unsigned)threads), lds, s, a);
    }
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_multi_lattice(int op, int prec, const MultiArgs& a, size_t lds, hipStream_t s, int* max_box)
{
    auto by_prec = [&](auto O) {
        constexpr int OV = decltype(O)::value;
        switch (prec) {
        case PREC_F64: return go_multi<LAT, OV, PREC_F64>(a, lds, s, max_box);
        case PREC_F32: return go_multi<LAT, OV, PREC_F32>(a, lds, s, max_box);
        case PREC_F16: return go_multi<LAT, OV, PREC_F16>(a, lds, s, max_box);
        default: return (hipError_t)hipErrorInvalidValue;
        }
    };
    switch (op) {
    case OP_PR: return by_prec(std::integral_constant<int, OP_PR>{});
    case OP_IR: return by_prec(std::integral_constant<int, OP_IR>{});
    case OP_PRI: return by_prec(std::integral_constant<int, OP_PRI>{});
    case OP_IRHB: return by_prec(std::integral_constant<int, OP_IRHB>{});
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
