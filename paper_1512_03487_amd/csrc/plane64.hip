// Plane walk of the hopping operator on 5D FP64 fields (gfx950): H and the domain-wall M.
//
// As k_dhop_plane, a block owns a 4 x 4 tile of (x, y) columns at one z with all their s (16 Ls threads, a
// multiple of 64) and walks slices of t: own records, the tile's faces and the links go through LDS, the z
// neighbours are read straight from memory, psi(x, t + 1) is the next slice's own record, the backward
// t-hop is carried in registers, and the finished records leave through LDS. A block takes 37 (Ls = 4) to
// 111 KB of LDS, so a SIMD holds one wavefront, and its registers hold the next slice's own records, faces
// and links while this slice's hops run.
//
// Why. The direction-parallel kernel spends 5100 vector instructions per 64 sites (eight wavefronts
// decode every site, 12 of 16 lanes reduce), 69 % of its time at 16^4 x 8, and requests 14 lines of 128 bytes
// per site; here it is one site per lane and about eight lines. 16^4 x 8 M 103 -> 82 us
// from memory (91 -> 83 in cache), 20^4 x 8 251 -> 182, 24^4 x 8 532 -> 397 in cache; domain-wall force at
// 16^4 x 8 177 -> 160 us.
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace gridmi {

constexpr int kP6Cols = 16, kP6Halo = 16, kP6Slots = 4 * kP6Cols + kP6Cols + 8;

static size_t plane64_lds_bytes(int Ls) {
    return (kP6Cols + kP6Halo) * static_cast<size_t>(Ls) * 192 + kP6Slots * 144;
}

// acc (spins 2 hf, 2 hf + 1) += f * that half of the record at rec
__device__ __forceinline__ void half_axpy64(Cx<double> acc[4][3], const chunk_t *rec, int hf, double f) {
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const chunk_t v = rec[hf * 6 + j];
        Cx<double> h, &o = acc[2 * hf + j / 3][j % 3];
        __builtin_memcpy(&h, &v, 16);
        o = {o.r + f * h.r, o.i + f * h.i};
    }
}

template <class LK, bool DAG, int KIND, int FUSE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1)))
k_dhop_plane64(const void *__restrict__ U, const void *__restrict__ psi, void *out, GeomDev g, int nseg, double diag,
               double mf, FuseDev fz) {
    using SP = SpF64;
    using R = Cx<double>[4][3];
    constexpr int CH = 12, NC = kP6Cols, NH = kP6Halo, NL = LK::kBytes / 16;
    extern __shared__ chunk_t p64_lds[];
    const int Ls = g.Ls, NT = NC * Ls;
    chunk_t *rec = p64_lds;                                                    // own records, then the halo's
    double2 *lks = reinterpret_cast<double2 *>(rec + (NC + NH) * Ls * CH);     // links of the slice, nine to a slot
    const int td = threadIdx.x;
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2], Lt = g.L[3];
    const int ntx = Lx / 4, nty = Ly / 4, ntile = ntx * nty * Lz;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int seg = lb / ntile, tile = lb - seg * ntile;
    const int x0 = tile % ntx * 4, y0 = tile / ntx % nty * 4, z = tile / (ntx * nty);
    const int c = td / Ls, s = td - c * Ls, cx = c & 3, cy = c >> 2;
    const int V3 = Lx * Ly * Lz, nq = V3 * Ls, plane = Lx * Ly;
    const int col = z * plane + (y0 + cy) * Lx + x0 + cx, q = col * Ls + s;
    const int zpo = (z == Lz - 1 ? 1 - Lz : 1) * plane * Ls, zmo = (z == 0 ? Lz - 1 : -1) * plane * Ls;
    const int t0 = seg * Lt / nseg, T = (seg + 1) * Lt / nseg - t0;
    constexpr int EF = DAG ? +1 : -1;

    // byte offsets, within a slice, of the stores (chunk j 64 + lane of the wavefront's records) and of the halo chunks
    unsigned og[CH], hg[CH], ug;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
        const int i = j * 64 + (td & 63), r = (td & ~63) + i / CH, row = r / (4 * Ls);
        og[j] = (((z * plane + (y0 + row) * Lx + x0) * Ls + (r - row * (4 * Ls))) * CH + i % CH) * 16u;
        const int h = j * NT + td, hc = h / (Ls * CH), off = h - hc * (Ls * CH);   // NH = NC: h < NH Ls CH
        int hx, hy;
        if (hc < 8) {
            hx = hc < 4 ? (x0 == 0 ? Lx - 1 : x0 - 1) : (x0 + 4 == Lx ? 0 : x0 + 4);
            hy = y0 + (hc & 3);
        } else {
            hy = hc < 12 ? (y0 == 0 ? Ly - 1 : y0 - 1) : (y0 + 4 == Ly ? 0 : y0 + 4);
            hx = x0 + (hc & 3);
        }
        hg[j] = static_cast<unsigned>((z * plane + hy * Lx + hx) * Ls * CH + off) * 16u;
    }
    // Link slots: the columns' four links (4 c + mu), U_z(x - z), U_x at the -x face, U_y at the -y face. With
    // fewer than kP6Slots threads (Ls = 4) a thread loads two.
    auto link_index = [&](int i) -> int {
        int lx = x0, ly = y0, lz = z, mu = 0;
        if (i < 5 * NC) {
            const int cc = i < 4 * NC ? i >> 2 : i - 4 * NC;
            mu = i < 4 * NC ? i & 3 : 2;
            lx += cc & 3;
            ly += cc >> 2;
            if (i >= 4 * NC) lz = z == 0 ? Lz - 1 : z - 1;
        } else if (i < 5 * NC + 4) {
            lx = x0 == 0 ? Lx - 1 : x0 - 1;
            ly += i - 5 * NC;
        } else {
            mu = 1;
            ly = y0 == 0 ? Ly - 1 : y0 - 1;
            lx += (i - 5 * NC - 4) & 3;
        }
        return (lz * plane + ly * Lx + lx) * 4 + mu;
    };
    ug = link_index(td < kP6Slots ? td : 0);
    const int nxp = cx < 3 ? td + Ls : (NC + 4 + cy) * Ls + s, nxm = cx > 0 ? td - Ls : (NC + cy) * Ls + s;
    const int nyp = cy < 3 ? td + 4 * Ls : (NC + 12 + cx) * Ls + s, nym = cy > 0 ? td - 4 * Ls : (NC + 8 + cx) * Ls + s;
    const int lxm = cx > 0 ? (c - 1) * 4 : 5 * NC + cy, lym = cy > 0 ? (c - 4) * 4 + 1 : 5 * NC + 4 + cx;
    const int rsp = s == Ls - 1 ? td - (Ls - 1) : td + 1, rsm = s == 0 ? td + Ls - 1 : td - 1;

    auto slice = [](int tt) {   // hidden from the loop optimiser (no address per load kept)
        __asm__("" : "+s"(tt));
        return tt;
    };
    auto load16 = [](const char *b, unsigned off) {
        __asm__("" : "+v"(off));
        return *reinterpret_cast<const chunk_t *>(b + off);
    };
    auto psi_at = [&](int tt) { return static_cast<const char *>(psi) + static_cast<size_t>(slice(tt)) * nq * 192; };
    auto direct = [&](int tt, unsigned n, Cx<double> p[4][3]) {
        const char *b = psi_at(tt);
        const unsigned o = n * 192u;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const chunk_t v = load16(b + j * 16, o);
            __builtin_memcpy(&p[j / 3][j % 3], &v, 16);
        }
    };
    auto staged = [&](int r, Cx<double> p[4][3]) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const chunk_t v = rec[r * CH + j];
            __builtin_memcpy(&p[j / 3][j % 3], &v, 16);
        }
    };
    auto link_of = [&](const double2 *l, Cx<double> u[3][3]) {
#pragma unroll
        for (int k = 0; k < 9; ++k) u[k / 3][k % 3] = {l[k].x, l[k].y};
    };
    // The two hops of a direction are added to each other first (two), then to the sum, x, y, z, t, as in
    // the direction-parallel kernel, and the diagonal part comes last: the same chain of roundings.
    R A, P, two;
    Cx<double> u[3][3], chi_b[2][3];
    auto clear = [](Cx<double> a[4][3]) {
#pragma unroll
        for (int j = 0; j < 12; ++j) a[j / 3][j % 3] = {0.0, 0.0};
    };
    auto pair_done = [&]() {
#pragma unroll
        for (int j = 0; j < 12; ++j) A[j / 3][j % 3] = cadd(A[j / 3][j % 3], two[j / 3][j % 3]);
        clear(two);
        pin(A);
        __builtin_amdgcn_sched_barrier(0);
    };
    double n2 = 0.0;
    auto finish = [&](int tt) {
        if constexpr (FUSE == kFuseAxpy) {
            // r - alpha op psi; r may alias out: a wavefront reads its records before it stores them
            R rv;
            SP::load(fz.r, nullptr, static_cast<size_t>(tt) * nq + q, rv);
            const double al = fz.scal[fz.num] / fz.scal[fz.den];
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                const Cx<double> a = A[j / 3][j % 3], b = rv[j / 3][j % 3];
                A[j / 3][j % 3] = {b.r - al * a.r, b.i - al * a.i};
            }
        }
        n2 += wave_store<SP, FUSE != kFuseNone>(rec + (td & ~63) * CH, nullptr,
                                                static_cast<char *>(out) + static_cast<size_t>(slice(tt)) * nq * 192, og,
                                                nullptr, A);
    };
    R Pn;
    chunk_t wh[CH];
    double2 wl[NL];
    auto issue = [&](int tt) {   // faces and the link of a slice
        const char *b = psi_at(tt);
#pragma unroll
        for (int j = 0; j < CH; ++j) wh[j] = load16(b, hg[j]);
        const double2 *l = reinterpret_cast<const double2 *>(static_cast<const char *>(U) +
                                                             static_cast<size_t>(slice(tt)) * V3 * (4 * LK::kBytes)) +
                           static_cast<size_t>(ug) * NL;
        if (td < kP6Slots)
#pragma unroll
            for (int k = 0; k < NL; ++k) wl[k] = l[k];
    };
    auto put_link = [&](double2 *d, const void *src, size_t i) {
        Cx<double> w[3][3];
        LK::load(src, i, w);
#pragma unroll
        for (int k = 0; k < 9; ++k) d[k] = make_double2(w[k / 3][k % 3].r, w[k / 3][k % 3].i);
    };
    {
        // the backward t-hop of slice t0
        const int tm = t0 == 0 ? Lt - 1 : t0 - 1;
        Cx<double> hb[2][3];
        direct(tm, q, P);
        LK::load(U, (static_cast<size_t>(tm) * V3 + col) * 4 + 3, u);
        direct(t0, q, Pn);
        issue(t0);
        project<3, -EF>(P, hb);
        su3_adj_mul(u, hb, chi_b);
    }
#pragma unroll 1
    for (int k = 0; k < T; ++k) {
        const int tt = t0 + k;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            chunk_t v;
            __builtin_memcpy(&v, &Pn[j / 3][j % 3], 16);
            rec[td * CH + j] = v;
        }
#pragma unroll
        for (int j = 0; j < CH; ++j) rec[(CH + j) * NT + td] = wh[j];
        if (td < kP6Slots) put_link(lks + td * 9, wl, 0);
        if (NT < kP6Slots && td + NT < kP6Slots)
            put_link(lks + (td + NT) * 9, U, static_cast<size_t>(tt) * V3 * 4 + link_index(td + NT));
        __syncthreads();
        R p, zp, zm;
        direct(tt, q + zpo, zp);   // in flight, as the next slice's loads are, during the x and y hops
        direct(tt + 1 == Lt ? 0 : tt + 1, q, Pn);
        if (k + 1 < T) issue(tt + 1);
        clear(A);
        clear(two);
        auto hop = [&](auto mu, auto fwd, int r, int l) {
            constexpr int MU = decltype(mu)::value;
            constexpr bool F = decltype(fwd)::value;
            staged(r, p);
            link_of(lks + l * 9, u);
            hop_term<MU, F ? EF : -EF, !F>(two, p, u);
            pin(two);
            __builtin_amdgcn_sched_barrier(0);
        };
        hop(std::integral_constant<int, 0>{}, std::true_type{}, nxp, c * 4);
        hop(std::integral_constant<int, 0>{}, std::false_type{}, nxm, lxm);
        pair_done();
        direct(tt, q + zmo, zm);
        hop(std::integral_constant<int, 1>{}, std::true_type{}, nyp, c * 4 + 1);
        hop(std::integral_constant<int, 1>{}, std::false_type{}, nym, lym);
        pair_done();
        link_of(lks + (c * 4 + 2) * 9, u);
        hop_term<2, EF, false>(two, zp, u);
        pin(two);
        __builtin_amdgcn_sched_barrier(0);
        link_of(lks + (4 * NC + c) * 9, u);
        hop_term<2, -EF, true>(two, zm, u);
        pair_done();
        // t: forward with psi(x, t + 1), the next slice's own record; the same link and psi(x, t) give the
        // next slice's backward hop
        link_of(lks + (c * 4 + 3) * 9, u);
        hop_term<3, EF, false>(two, Pn, u);
        reconstruct_add<3, -EF>(two, chi_b);
        pair_done();
        staged(td, P);
        {
            Cx<double> hb[2][3];
            project<3, -EF>(P, hb);
            su3_adj_mul(u, hb, chi_b);
        }
        if constexpr (KIND == GRID_DWF) {
            constexpr int hup = DAG ? 0 : 1;
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                Cx<double> &a = A[j / 3][j % 3];
                // diag psi rounded, then - H psi / 2, as the direction-parallel kernel's multiply-adds are formed
                a = {__builtin_fma(-0.5, a.r, diag * P[j / 3][j % 3].r), __builtin_fma(-0.5, a.i, diag * P[j / 3][j % 3].i)};
            }
            half_axpy64(A, rec + rsp * CH, hup, s == Ls - 1 ? mf : -1.0);
            half_axpy64(A, rec + rsm * CH, 1 - hup, s == 0 ? mf : -1.0);
        }
        pin(A);
        __syncthreads();   // what the slice read is free: the stores and the next slice go there
        finish(tt);
    }
    if constexpr (FUSE != kFuseNone) {
        n2 = wave_sum64(n2);
        __shared__ double fred[4];
        if ((td & 63) == 0) fred[td >> 6] = n2;
        __syncthreads();
        if (td == 0) {
            double v = 0.0;
            for (int w = 0; w < NT / 64; ++w) v += fred[w];
            fz.part[blockIdx.x] = v;
        }
    }
}

// Blocks along t: the count with the least (slices of the longest + 1) x rounds of the blocks that the CUs'
// LDS holds at a time. Measured, nseg = 1 / 2 / 4 / 8: 16^4 x 8 93 / 83 / 83 / 89 us, 16^4 x 16 162 / 171 / 180 /
// 200, 24^4 x 8 424 / 441 / 397 / 413, 24^4 x 4 205 / 227 / 231 / 222 us.
static int plane64_nseg(const GeomDev &g, double *even) {
    const long slots = 256 * (163840 / static_cast<long>(plane64_lds_bytes(g.Ls)));
    const long tiles = static_cast<long>(g.vol / g.L[3]) / kP6Cols;
    long best = 0;
    int nseg = 1;
    for (int n = 1; n <= g.L[3]; n = next_walk_count(g.L[3], n)) {
        const long T = (g.L[3] + n - 1) / n, rounds = (tiles * n + slots - 1) / slots, cost = (T + 1) * rounds;
        if (n == 1 || cost < best) {
            best = cost;
            nseg = n;
            *even = static_cast<double>(tiles) * g.L[3] / slots / (T * rounds);
        }
    }
    return nseg;
}

// From 500000 sites on, where the blocks keep the CUs evenly busy (mean over largest number of slices of a
// slot at least 0.93); smaller fields lie in the caches, which the direction-parallel kernel's many
// wavefronts use better. Direction-parallel against this kernel: 16^4 x 8 91 / 83 us, 16^4 x 16 182 / 162, 16^4 x 12
// 133 / 131, 24^4 x 8 532 / 397, 24^4 x 12 786 / 755, 24^4 x 4 265 / 205, 32^2 x 16^2 x 8 424 / 310; 16^2 x 12 x 18 x 12
// (0.90) 114 / 120, 20 x 16 x 18 x 14 x 8 (0.70) 105 / 111, 16^4 x 4 (262144) 44 / 50, 12^4 x 12 (248832) 44 / 85.
bool plane64_applies(const DhopArgs &a) {
    double even = 0.0;
    return !a.custom && (a.kind == GRID_HOP || a.kind == GRID_DWF) && a.prec == GRID_F64 && a.g.L[0] % 4 == 0 &&
           a.g.L[1] % 4 == 0 && (a.g.Ls == 4 || a.g.Ls == 8 || a.g.Ls == 12 || a.g.Ls == 16) && a.g.n5 >= 500000 &&
           offsets32(a.g.n5 / a.g.L[3], 192) && plane64_nseg(a.g, &even) > 0 && even >= 0.93;
}

long plane64_blocks(const DhopArgs &a) {
    double even;
    return static_cast<long>(a.g.vol / a.g.L[3]) / kP6Cols * plane64_nseg(a.g, &even);
}

template <class LK>
static hipError_t launch_plane64_t(const DhopArgs &a) {
    const dim3 grid(static_cast<unsigned>(plane64_blocks(a))), block(kP6Cols * a.g.Ls);
    const size_t lds = plane64_lds_bytes(a.g.Ls);
    double even;
    const int nseg = plane64_nseg(a.g, &even);
#define GRIDMI_LAUNCH(DAG, KIND, FUSE)                                                                                \
    hipLaunchKernelGGL((k_dhop_plane64<LK, DAG, KIND, FUSE>), grid, block, lds, a.stream, a.U, a.psi, a.out, a.g, nseg, \
                       a.diag, a.mf, a.fz)
    if (a.fuse != kFuseNone) {
        switch (a.kind * 4 + a.fuse * 2 + (a.dag ? 1 : 0)) {
            case GRID_DWF * 4 + kFuseNorm * 2 + 0: GRIDMI_LAUNCH(false, GRID_DWF, kFuseNorm); break;
            case GRID_DWF * 4 + kFuseAxpy * 2 + 1: GRIDMI_LAUNCH(true, GRID_DWF, kFuseAxpy); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (a.kind * 2 + (a.dag ? 1 : 0)) {
        case GRID_HOP * 2 + 0: GRIDMI_LAUNCH(false, GRID_HOP, kFuseNone); break;
        case GRID_HOP * 2 + 1: GRIDMI_LAUNCH(true, GRID_HOP, kFuseNone); break;
        case GRID_DWF * 2 + 0: GRIDMI_LAUNCH(false, GRID_DWF, kFuseNone); break;
        case GRID_DWF * 2 + 1: GRIDMI_LAUNCH(true, GRID_DWF, kFuseNone); break;
        default: return hipErrorInvalidValue;
    }
#undef GRIDMI_LAUNCH
    return hipGetLastError();
}

hipError_t launch_plane64(const DhopArgs &a) {
    return a.link_fmt == GRID_L18 ? launch_plane64_t<LkF64<3>>(a) : launch_plane64_t<LkF64<2>>(a);
}

}  // namespace gridmi
