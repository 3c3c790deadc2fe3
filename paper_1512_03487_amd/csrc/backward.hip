// Link gradient and su(3) force of the hopping term (the adjoint HMC's fermion force needs,
// Section 4).
//
// For L = Re <g, c H psi> the complex gradient dL/dRe U + i dL/dIm U of link U_mu(x) is
//   G_mu(x) = c sum_{s, spin} { [(1 + EF gamma_mu) g(x)] psi(x+mu)^dagger
//                             + psi(x) [(1 - EF gamma_mu) g(x+mu)]^dagger },
// EF = -1 for H and +1 for H^dagger. Because (1 + e gamma) v = [h; e A^dagger h] with
// h = v_up + e A v_dn, a spin trace of [(1 + e gamma) v] w^dagger equals the two-spin sum
// h(v) h(w)^dagger of the projected half-spinors (with the same e), so each term is a sum of two
// 3x3 outer products of half-spinors. One thread per (4D site, mu), one mu per wavefront; the
// fifth coordinate is summed inside the thread; no atomics, so results are bitwise reproducible.
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace gridmi {

// Records come through the wavefront's LDS slot (coalesced chunk loads, then each lane reads its
// own record back); the four records of a step are all requested before the first is staged.
template <int MU, int EF, class SP, typename C>
__device__ __forceinline__ void grad_mu(const void *chi, const void *psi, int x4, int xp, int Ls, chunk_t *lds,
                                        Cx<C> G[3][3]) {
    Cx<C> p[4][3], hg[2][3], hp[2][3];
    for (int s = 0; s < Ls; ++s) {
        Fetch<SP> f0, f1, f2, f3;
        fetch<SP>(chi, nullptr, x4 * Ls + s, f0);
        fetch<SP>(psi, nullptr, xp * Ls + s, f1);
        fetch<SP>(psi, nullptr, x4 * Ls + s, f2);
        fetch<SP>(chi, nullptr, xp * Ls + s, f3);
        // [(1 + EF gamma) g(x)] psi(x+mu)^dagger
        stage<SP>(f0, lds, p);
        project<MU, EF>(p, hg);
        stage<SP>(f1, lds, p);
        project<MU, EF>(p, hp);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) G[a][b] = cmac(G[a][b], hg[k][a], cconj(hp[k][b]));
        // psi(x) [(1 - EF gamma) g(x+mu)]^dagger
        stage<SP>(f2, lds, p);
        project<MU, -EF>(p, hp);
        stage<SP>(f3, lds, p);
        project<MU, -EF>(p, hg);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) G[a][b] = cmac(G[a][b], hp[k][a], cconj(hg[k][b]));
    }
}

// G <- coef G of link LINK, or its force TA(coef G U^dagger). A macro: as a function, inlined after the
// kernel's sums had been scheduled, it cost k_link_grad 3 to 6% in FP32 (6 x 14 x 20 x 2 x 8 16.3 -> 17.3 us).
#define GRIDMI_GRAD_FINISH(LINK)                                                                                      \
    const C c = static_cast<C>(coef);                                                                                 \
_Pragma("unroll")                                                                                                     \
    for (int k = 0; k < 9; ++k) G[k / 3][k % 3] = cscale(c, G[k / 3][k % 3]);                                         \
    if (force_mode) {                                                                                                 \
        /* F = TA(G U^dagger), TA(A) = (A - A^dagger)/2 - tr(A - A^dagger)/6 */                                       \
        Cx<C> u[3][3], m[3][3];                                                                                       \
        if constexpr (sizeof(C) == 8)                                                                                 \
            LkF64<3>::load(U, LINK, u);                                                                               \
        else                                                                                                          \
            LkF32<3>::load(U, LINK, u);                                                                               \
_Pragma("unroll")                                                                                                     \
        for (int a = 0; a < 3; ++a)                                                                                   \
_Pragma("unroll")                                                                                                     \
            for (int b = 0; b < 3; ++b) {                                                                             \
                Cx<C> s = cmul(G[a][0], cconj(u[b][0]));                                                              \
                s = cmac(s, G[a][1], cconj(u[b][1]));                                                                 \
                s = cmac(s, G[a][2], cconj(u[b][2]));                                                                 \
                m[a][b] = s;                                                                                          \
            }                                                                                                         \
        /* tr(A - A^dagger) = 2 i Im tr A */                                                                          \
        const C imtr = m[0][0].i + m[1][1].i + m[2][2].i;                                                             \
_Pragma("unroll")                                                                                                     \
        for (int a = 0; a < 3; ++a)                                                                                   \
_Pragma("unroll")                                                                                                     \
            for (int b = 0; b < 3; ++b) {                                                                             \
                Cx<C> f = {C(0.5) * (m[a][b].r - m[b][a].r), C(0.5) * (m[a][b].i + m[b][a].i)};                       \
                if (a == b) f.i -= imtr / C(3);                                                                       \
                G[a][b] = f;                                                                                          \
            }                                                                                                         \
    }

template <class SP, bool DAG>
__global__ void __launch_bounds__(256)
k_link_grad(const void *__restrict__ U, const void *__restrict__ chi, const void *__restrict__ psi, void *__restrict__ Gout,
            GeomDev g, double coef, int force_mode) {
    using C = typename SP::C;
    __shared__ chunk_t sm[4][64 * stage_pitch<SP>()];
    chunk_t *lds = sm[threadIdx.x >> 6];
    // A block covers 64 consecutive sites; wavefront mu computes their direction-mu links, so
    // the direction is uniform across a wavefront (no divergent switch) and the four wavefronts
    // reading chi(x) and psi(x) share them through the CU's L1.
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int mu = threadIdx.x >> 6;
    const int x4r = lb * 64 + (threadIdx.x & 63);
    const bool live = x4r < g.vol;
    const int x4 = live ? x4r : g.vol - 1;   // idle lanes take part in the wave's gathers
    const int t = x4 * 4 + mu;               // link index: site-major, direction fastest
    int nb[8];
    neighbours(g, x4, nb);
    Cx<C> G[3][3];
#pragma unroll
    for (int k = 0; k < 9; ++k) G[k / 3][k % 3] = {C(0), C(0)};
    constexpr int EF = DAG ? +1 : -1;
    switch (mu) {
        case 0: grad_mu<0, EF, SP, C>(chi, psi, x4, nb[0], g.Ls, lds, G); break;
        case 1: grad_mu<1, EF, SP, C>(chi, psi, x4, nb[2], g.Ls, lds, G); break;
        case 2: grad_mu<2, EF, SP, C>(chi, psi, x4, nb[4], g.Ls, lds, G); break;
        default: grad_mu<3, EF, SP, C>(chi, psi, x4, nb[6], g.Ls, lds, G); break;
    }
    GRIDMI_GRAD_FINISH(static_cast<size_t>(t))
    if (!live) return;
    Cx<C> *q = static_cast<Cx<C> *>(Gout) + static_cast<size_t>(t) * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) q[k] = G[k / 3][k % 3];
}

// The same sums on a tile of 4 x 4 x 2 x 2 sites, for lattices it divides: per s the tile's records of
// both fields and those of its +x, +y, +z and +t faces (64 + 96 of each) go through LDS, loaded an s
// ahead, and the four wavefronts (one per mu) read the records of their two sites there. What bounds
// k_link_grad is the 128-byte lines a CU requests: ten records per site and s, in lines of which a pass over
// one s uses three quarters; a tile requests five. k_link_grad against this kernel: 16^4 x 8 FP64 136 ->
// 69 us, FP32 65 -> 43, 16^4 x 16 358 -> 138 and 126 -> 78 us, 24^4 x 4 465 -> 224 and 199 -> 110 us (the
// bytes it cannot do without take 47 us at 16^4 x 8 in FP64); with the gradients stored by their lanes
// 24^4 x 4 took 234 and 120 us.
constexpr int kGtSites = 64, kGtRecs = 160;

template <class SP, bool DAG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_link_grad_tile(const void *__restrict__ U, const void *__restrict__ chi, const void *__restrict__ psi,
                 void *__restrict__ Gout, GeomDev g, double coef, int force_mode) {
    using C = typename SP::C;
    // record pitch in LDS: 208 bytes FP64, 104 FP32 (16- and 8-byte reads of a wavefront on all banks)
    constexpr int CH = SP::kChunks, PITCH = CH * 16 + 2 * sizeof(C);
    constexpr int NLD = (kGtRecs * CH + 255) / 256;      // chunks of one field per thread
    constexpr int EF = DAG ? +1 : -1;
    extern __shared__ chunk_t grad_smem[];               // chi's records, then psi's
    char *grad_lds = reinterpret_cast<char *>(grad_smem);
    const int tid = threadIdx.x, mu = tid >> 6, lane = tid & 63;
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2], Lt = g.L[3], Ls = g.Ls;
    int lb = xcd_block(blockIdx.x, gridDim.x);
    const int x0 = lb % (Lx / 4) * 4;
    lb /= Lx / 4;
    const int y0 = lb % (Ly / 4) * 4;
    lb /= Ly / 4;
    const int z0 = lb % (Lz / 2) * 2, t0 = lb / (Lz / 2) * 2;
    auto site = [&](int x, int y, int z, int t) { return ((t * Lz + z) * Ly + y) * Lx + x; };
    // 4D site of LDS record r: the tile's (x fastest), then the +x, +y, +z and +t faces
    auto record_site = [&](int r) {
        int x = r & 3, y = (r >> 2) & 3, z = (r >> 4) & 1, t = (r >> 5) & 1;
        if (r >= 128) {
            t = 2;
        } else if (r >= 96) {
            t = (r >> 4) & 1;
            z = 2;
        } else if (r >= 64) {
            z = (r >> 2) & 1;
            t = (r >> 3) & 1;
            if (r >= 80) {
                y = 4;
            } else {
                y = r & 3;
                z = (r >> 2) & 1;
                x = 4;
            }
        }
        x = x0 + x == Lx ? 0 : x0 + x;
        y = y0 + y == Ly ? 0 : y0 + y;
        z = z0 + z == Lz ? 0 : z0 + z;
        t = t0 + t == Lt ? 0 : t0 + t;
        return site(x, y, z, t);
    };
    const int cx = lane & 3, cy = (lane >> 2) & 3, cz = (lane >> 4) & 1, ct = lane >> 5;
    const int nb = mu == 0   ? (cx < 3 ? lane + 1 : 64 + cy + 4 * cz + 8 * ct)
                   : mu == 1 ? (cy < 3 ? lane + 4 : 80 + cx + 4 * cz + 8 * ct)
                   : mu == 2 ? (cz < 1 ? lane + 16 : 96 + cx + 4 * cy + 16 * ct)
                             : (ct < 1 ? lane + 32 : 128 + cx + 4 * cy + 16 * cz);
    unsigned off[NLD];   // chunk offset of this thread's loads, s = 0
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
        const int c = min(k * 256 + tid, kGtRecs * CH - 1), r = c / CH;
        off[k] = static_cast<unsigned>(record_site(r)) * Ls * CH + (c - r * CH);
    }
    const chunk_t *pc = static_cast<const chunk_t *>(chi), *pp = static_cast<const chunk_t *>(psi);
    chunk_t wc[NLD], wp[NLD];
    auto issue = [&](int s) {
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            unsigned o = off[k];
            __asm__("" : "+v"(o));   // else a 64-bit address per load stays live
            wc[k] = (pc + s * CH)[o];
            wp[k] = (pp + s * CH)[o];
        }
    };
    // spin K of the projected record r of a field (project(), one spin at a time: 12 registers live
    // in place of 48)
    auto half = [&](auto m, auto e, auto kk, int field, int r, Cx<C> h[3]) {
        constexpr int MU = decltype(m)::value, K = decltype(kk)::value, B = MU < 2 ? 3 - K : 2 + K;
        constexpr int E = (MU == 1 && K == 0) || (MU == 2 && K == 1) ? -decltype(e)::value : decltype(e)::value;
        const Cx<C> *v = reinterpret_cast<const Cx<C> *>(grad_lds + (field * kGtRecs + r) * PITCH);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const Cx<C> p = v[K * 3 + a], b = v[B * 3 + a];
            if (MU == 0 || MU == 2)   // p - i E b
                h[a] = {E > 0 ? p.r + b.i : p.r - b.i, E > 0 ? p.i - b.r : p.i + b.r};
            else                      // p + E b
                h[a] = {E > 0 ? p.r + b.r : p.r - b.r, E > 0 ? p.i + b.i : p.i - b.i};
        }
    };
    Cx<C> G[3][3];
#pragma unroll
    for (int k = 0; k < 9; ++k) G[k / 3][k % 3] = {C(0), C(0)};
    auto add = [&](auto m) {
        // [(1 + EF gamma) g(x)] psi(x+mu)^dagger (field 0, 1), then psi(x) [(1 - EF gamma) g(x+mu)]^dagger
        auto term = [&](auto e, auto kk, int field) {
            Cx<C> a[3], b[3];
            half(m, e, kk, field, lane, a);
            half(m, e, kk, 1 - field, nb, b);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) G[i][j] = cmac(G[i][j], a[i], cconj(b[j]));
            __builtin_amdgcn_sched_barrier(0);
        };
        term(std::integral_constant<int, EF>{}, std::integral_constant<int, 0>{}, 0);
        term(std::integral_constant<int, EF>{}, std::integral_constant<int, 1>{}, 0);
        term(std::integral_constant<int, -EF>{}, std::integral_constant<int, 0>{}, 1);
        term(std::integral_constant<int, -EF>{}, std::integral_constant<int, 1>{}, 1);
    };
    auto put = [&](int o, chunk_t v) {
        typedef unsigned int u2v __attribute__((ext_vector_type(2)));
        if constexpr (PITCH % 16 == 0) {
            *reinterpret_cast<chunk_t *>(grad_lds + o) = v;
        } else {
            u2v *d = reinterpret_cast<u2v *>(grad_lds + o);
            d[0] = u2v{v.x, v.y};
            d[1] = u2v{v.z, v.w};
        }
    };
    issue(0);
#pragma unroll 1
    for (int s = 0; s < Ls; ++s) {
        if (s > 0) __syncthreads();   // the records of s - 1 have been read
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            const int c = k * 256 + tid, r = c / CH;
            if (c < kGtRecs * CH) {
                put(r * PITCH + (c - r * CH) * 16, wc[k]);
                put((kGtRecs + r) * PITCH + (c - r * CH) * 16, wp[k]);
            }
        }
        __syncthreads();
        if (s + 1 < Ls) issue(s + 1);
        if (mu == 0) add(std::integral_constant<int, 0>{});
        else if (mu == 1) add(std::integral_constant<int, 1>{});
        else if (mu == 2) add(std::integral_constant<int, 2>{});
        else add(std::integral_constant<int, 3>{});
    }
    const size_t link = static_cast<size_t>(site(x0 + cx, y0 + cy, z0 + cz, t0 + ct)) * 4 + mu;
    [&] { GRIDMI_GRAD_FINISH(link) }();   // as a function here: 8^4 x 16 FP32 26.6 -> 26.2 us
    // Stored through LDS, the four sites of a row contiguous: a lane's own 144 bytes at 576-byte pitch
    // would cost a request to the L2 per 16 of them.
    __syncthreads();
    Cx<C> *gl = reinterpret_cast<Cx<C> *>(grad_lds);
#pragma unroll
    for (int k = 0; k < 9; ++k) gl[(lane * 4 + mu) * 9 + k] = G[k / 3][k % 3];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int e = k * 256 + tid, row = e / 144;
        static_cast<Cx<C> *>(Gout)[static_cast<size_t>(site(x0, y0 + (row & 3), z0 + ((row >> 2) & 1), t0 + (row >> 3))) * 36 +
                                   (e - row * 144)] = gl[e];
    }
}

// The tile divides the lattice and a field's chunks have 32-bit offsets. It is the faster kernel for short
// sums too: Ls = 1, 24^4 FP64 116 (k_link_grad) against 95 us, FP32 51 against 36, 16^4 28 against 19 and 13.5
// both; Ls = 2, 24^4 238 against 123 and 78 against 53.
static bool grad_tile_applies(const GeomDev &g) {
    return g.L[0] % 4 == 0 && g.L[1] % 4 == 0 && g.L[2] % 2 == 0 && g.L[3] % 2 == 0 &&
           static_cast<double>(g.n5) * 12 < 4294967296.0;
}

template <class SP, bool DAG>
static void launch_grad(const LinkGradArgs &a) {
    const dim3 block(256);
    if (grad_tile_applies(a.g)) {
        const size_t lds = 2 * kGtRecs * (SP::kChunks * 16 + 2 * sizeof(typename SP::C));
        hipLaunchKernelGGL((k_link_grad_tile<SP, DAG>), dim3(a.g.vol / kGtSites), block, lds, a.stream, a.U, a.chi, a.psi,
                           a.G, a.g, a.coef, a.force_mode);
        return;
    }
    hipLaunchKernelGGL((k_link_grad<SP, DAG>), dim3((a.g.vol + 63) / 64), block, 0, a.stream, a.U, a.chi, a.psi, a.G,
                       a.g, a.coef, a.force_mode);
}

hipError_t launch_link_grad(const LinkGradArgs &a) {
    if (a.g.vol == 0) return hipSuccess;
    if (a.prec == GRID_F64)
        a.dag ? launch_grad<SpF64, true>(a) : launch_grad<SpF64, false>(a);
    else if (a.prec == GRID_F32)
        a.dag ? launch_grad<SpF32, true>(a) : launch_grad<SpF32, false>(a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace gridmi
