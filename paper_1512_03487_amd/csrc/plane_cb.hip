// Plane walk of the hopping operator on checkerboard fields, Ls = 16 (the even-odd form; FP32 and
// FP16 storage, gfx950): out (parity cb) = Diag(y) + beta H psi, psi of parity 1 - cb.
//
// A block owns a tile of 16 (xh, y) columns at one z with all their s (256 threads, a column a DPP
// row) and walks T slices, as k_dhop_plane does on full fields. A column's own record is at the other
// parity's physical x, 2 xh + 1 - b with b = (cb + y + z + t) & 1 for an output at 2 xh + b, so
//  * it is the t-neighbour of out(t - 1) and out(t + 1): the forward t-hop of the slice before and the
//    backward one of the slice after take it from registers;
//  * it is the +x neighbour of out(t) where b = 0 and the -x neighbour where b = 1; the other one is
//    the own record of column xh - 1 or xh + 1: one x halo column per row, on the side b names;
//  * all eight links of an output are distinct from its neighbours' (four at the output's site, four
//    at the input sites), so they go through LDS once for the 16 s that share them.
// A site fetches 4.75 records per slice in place of eight, and y: what S and (d - S)^-1 move along the
// fifth dimension goes across the DPP row (column_m5inv_row: four steps of doubling in place of 96
// LDS reads). The time goes with the 128-byte lines requested. Checkerboard column walk against this kernel,
// 16^4 x 16 in cache, FP16 storage: (d - S)^-1 H 45.7 -> 27.7 us, M with |out|^2 34.6 -> 30 us, M^dagger with
// r - alpha (...) 38 -> 32 us; FP32 H 48 -> 33 us, with y 57 -> 40 us. From memory H and with y: 16^4 x 16 FP32 52 -> 38,
// 64 -> 47 us, FP16 storage 31 -> 25, 39 -> 28; 24^4 x 16 FP32 278 -> 187, 313 -> 235, FP16 storage 147 -> 109, 192 -> 130. The
// even-odd domain-wall solve at 16^4 x 16: 50.1 -> 40.4 ms.
// Tried and not kept: four wavefronts per SIMD (24 to 48 registers spilled: 38 against 28 us).
#include <math.h>

#include <type_traits>

#include "device.h"
#include "launch.h"

namespace gridmi {

constexpr int kPcLs = 16, kPcCols = 16, kPcThreads = kPcLs * kPcCols;

struct PlaneCbDev {
    int ltx;   // log2 of the tile's xh extent (2: 4 x 4 columns, 1: 2 x 8); y extent 16 >> ltx
    int nseg;  // blocks along t: block i walks slices [i Lt / nseg, (i + 1) Lt / nseg)
};

// Halo columns: one per row (the x neighbour b names), then the -y and the +y face. Link slots: 8 c + m,
// m = 0..3 U_m at the output's site, 4 U_x, 5 U_y, 7 U_t at the column's input site, 6 U_z(x - z); then
// U_x at the -x face and U_y at the -y face.
constexpr int kPcHaloMax = 12, kPcSlotsMax = 8 * kPcCols + 10;
template <class SL>
constexpr size_t plane_cb_lds_bytes() {
    return (kPcCols + kPcHaloMax) * kPcLs * (SL::kChunks * 16 + (SL::kScaled ? 4 : 0)) + kPcSlotsMax * 72;
}

// The policy of the records in LDS: chi = B psi in FP32 for the Moebius operator without dag.
template <class SP, bool DAG, int KIND>
using PcLds = std::conditional_t<(KIND == kMobHop || KIND == kMobDiag || KIND == kMobHopInv) && !DAG, SpF32, SP>;

template <class SP, class LK, bool DAG, int KIND, int FUSE>
__global__ void __launch_bounds__(kPcThreads) __attribute__((amdgpu_waves_per_eu(3)))
k_dhop_plane_cb(const void *__restrict__ U, const void *__restrict__ psi, const float *__restrict__ psi_scale,
                const void *__restrict__ yv, const float *__restrict__ y_scale, void *out, float *out_scale, GeomDev g,
                PlaneCbDev pd, int cbp, double diag, double mf, double beta, double cs, double b5, double c5, FuseDev fz) {
    constexpr bool MOB = KIND == kMobHop || KIND == kMobDiag || KIND == kMobHopInv;
    constexpr bool MOBF = MOB && !DAG;
    constexpr bool MOBA = MOB && DAG;
    constexpr bool INV = KIND == kHopInv || KIND == kMobHopInv;
    constexpr bool HASY = KIND == GRID_DWF || KIND == kMobDiag;
    using SL = PcLds<SP, DAG, KIND>;
    constexpr bool SC = SL::kScaled;
    constexpr int CH = SL::kChunks;
    constexpr int Ls = kPcLs, NC = kPcCols;
    extern __shared__ chunk_t plane_cb_lds[];
    chunk_t *rec = plane_cb_lds;                                                   // own records, then the halo's
    float2 *lks = reinterpret_cast<float2 *>(rec + (NC + kPcHaloMax) * Ls * CH);   // links, FP32, nine to a slot
    [[maybe_unused]] float *rsc = reinterpret_cast<float *>(lks + kPcSlotsMax * 9);   // scales
    const int td = threadIdx.x;
    const int ltx = pd.ltx, TX = 1 << ltx, TY = NC >> ltx, NH = TY + 2 * TX, NS = 8 * NC + TY + TX;
    const int Lx = g.L[0], Lxh = Lx / 2, Ly = g.L[1], Lz = g.L[2], Lt = g.L[3];
    const int ntx = Lxh >> ltx, nty = Ly / TY, ntile = ntx * nty * Lz;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int seg = lb / ntile, tile = lb - seg * ntile;
    const int x0 = (tile % ntx) << ltx, y0 = (tile / ntx) % nty * TY, z = tile / (ntx * nty);
    const int c = td / Ls, s = td & (Ls - 1), cx = c & (TX - 1), cy = c >> ltx;
    const int V3 = Lx * Ly * Lz, nq = V3 / 2 * Ls, plane = Lxh * Ly;
    const int q = (z * plane + (y0 + cy) * Lxh + x0 + cx) * Ls + s;
    const int zpo = (z == Lz - 1 ? 1 - Lz : 1) * plane * Ls, zmo = (z == 0 ? Lz - 1 : -1) * plane * Ls;
    const int t0 = seg * Lt / pd.nseg, T = (seg + 1) * Lt / pd.nseg - t0;
    constexpr int EF = DAG ? +1 : -1;
    // FP32 records are stored through LDS (wave_store; 16^4 x 16 H 36 -> 33 us, 24^4 x 16 204 -> 184), for which
    // out(t - 1) is finished before slice t's records go there; FP16-storage ones, at half the pitch, are
    // as fast stored by their lane (28 against 29 us), and their LDS writes need not wait.
    constexpr bool STAGE = !SP::kScaled;
    // out = diag y - cs S y + beta H psi. y's part comes after the hops: before them, as diag y / beta and larger
    // than they are, it has each of them rounded at its size (domain wall in FP32, beta = -1/4: error 7.8e-8 of the
    // result; 5.1e-8 so, the column walk's). YEND: it is added to the finished sum. In FP32 that exposes the load
    // of y (46 -> 52 us at 16^4 x 16, and spills where it is issued before the t-hop): there it joins beta times
    // the seven hops of the slice, and the last hop is added times beta (47 us).
    constexpr bool YEND = HASY && (MOBA || !STAGE), YMID = HASY && !YEND;
    // wall factors of s + 1 and s - 1
    const float wp = (s == Ls - 1) ? static_cast<float>(-mf) : 1.0f, wm = (s == 0) ? static_cast<float>(-mf) : 1.0f;
    const float bt = static_cast<float>(beta);
    [[maybe_unused]] const float dg = static_cast<float>(diag), csm = -static_cast<float>(cs);
    [[maybe_unused]] const float mb5 = static_cast<float>(b5), mc5 = static_cast<float>(c5);

    // Byte offsets, within a slice, of this thread's stores: chunks j 64 + lane of the wavefront's records
    constexpr int CM = SP::kChunks;
    [[maybe_unused]] unsigned og[CM];
#pragma unroll
    for (int j = 0; j < CM; ++j) {
        const int i = j * 64 + (td & 63), r = (td & ~63) + i / CM, rc = r / Ls;
        og[j] = static_cast<unsigned>(((z * plane + (y0 + (rc >> ltx)) * Lxh + x0 + (rc & (TX - 1))) * Ls + (r & (Ls - 1))) * CM +
                                      i % CM) * 16u;
    }
    // This thread's halo record (b = 0 and b = 1 slices) and link.
    int hq0 = q, hq1 = q, hb0 = 0;
    {
        const int hc = c;
        if (hc < TY) {
            const int row = z * plane + (y0 + hc) * Lxh;
            hq0 = (row + (x0 == 0 ? Lxh - 1 : x0 - 1)) * Ls + s;
            hq1 = (row + (x0 + TX == Lxh ? 0 : x0 + TX)) * Ls + s;
            hb0 = cbp + y0 + hc + z;
        } else if (hc < NH) {
            const int hy = hc < TY + TX ? (y0 == 0 ? Ly - 1 : y0 - 1) : (y0 + TY == Ly ? 0 : y0 + TY);
            hq0 = hq1 = (z * plane + hy * Lxh + x0 + ((hc - TY) & (TX - 1))) * Ls + s;
        }
    }
    int ug, ub;   // link (2 xh, y, z) of the slot and the parity of its x at t = 0
    {
        int lxh = x0, ly = y0, lz = z, mu = 0;
        ub = cbp + z + 1;
        if (td < 8 * NC) {
            const int cc = td >> 3, m = td & 7;
            lxh += cc & (TX - 1);
            ly += cc >> ltx;
            mu = m < 4 ? m : m == 7 ? 3 : m - 4;
            ub += ly + (m < 4 || m == 6 ? 1 : 0);
            if (m == 6) lz = z == 0 ? Lz - 1 : z - 1;
        } else if (td < 8 * NC + TY) {
            lxh = x0 == 0 ? Lxh - 1 : x0 - 1;
            ly += td - 8 * NC;
            ub += ly;
        } else {
            mu = 1;
            ub += y0 + 1;
            ly = y0 == 0 ? Ly - 1 : y0 - 1;
            lxh += (td - 8 * NC - TY) & (TX - 1);
        }
        ug = ((lz * Ly + ly) * Lx + 2 * lxh) * 4 + mu;
    }
    // LDS slots of the neighbours
    const int b0 = cbp + y0 + cy + z;
    const int nxp1 = cx < TX - 1 ? td + Ls : (NC + cy) * Ls + s;   // b = 1: +x
    const int nxm0 = cx > 0 ? td - Ls : (NC + cy) * Ls + s;        // b = 0: -x
    const int nyp = cy < TY - 1 ? td + TX * Ls : (NC + TY + TX + cx) * Ls + s;
    const int nym = cy > 0 ? td - TX * Ls : (NC + TY + cx) * Ls + s;
    const int lxm0 = cx > 0 ? (c - 1) * 8 + 4 : 8 * NC + cy;
    const int lym = cy > 0 ? (c - TX) * 8 + 5 : 8 * NC + TY + cx;

    // Hidden from the loop optimiser: it would keep a 64-bit address per load across the loop.
    auto slice = [](int tt) {
        __asm__("" : "+s"(tt));
        return tt;
    };
    auto link = [&](int slot) {
        __asm__("" : "+v"(slot));
        return lks + slot * 9;
    };
    auto direct = [&](const void *f, const float *fs, int tt, unsigned n, Rec<SP> &r) {
        const char *b = static_cast<const char *>(f) + static_cast<size_t>(slice(tt)) * nq * (CM * 16);
        unsigned o = n * (CM * 16u);
        __asm__("" : "+v"(o));
        uint4 w[CM];
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            const chunk_t v = *reinterpret_cast<const chunk_t *>(b + o + j * 16);
            w[j] = make_uint4(v.x, v.y, v.z, v.w);
        }
        float sc = 1.0f;
        if constexpr (SP::kScaled) {
            const char *sb = reinterpret_cast<const char *>(fs) + static_cast<size_t>(slice(tt)) * nq * 4;
            unsigned so = n * 4u;
            __asm__("" : "+v"(so));
            sc = *reinterpret_cast<const float *>(sb + so);
        }
        r.set(w, sc);
    };
    auto hopped = [&](const Rec<SP> &r, Rec<SL> &h) {
        if constexpr (MOBF) {
#pragma unroll
            for (int j = 0; j < 12; ++j) h.p[j / 3][j % 3] = {0.f, 0.f};
            column_shift_axpy<false>(r, h.p, mc5 * wp, mc5 * wm);
            r.axpy(h.p, mb5);
        } else {
            h = r;
        }
    };
    auto put = [&](int r, const Rec<SL> &x) {
        if constexpr (SC) {
#pragma unroll
            for (int j = 0; j < CH; ++j)
                rec[r * CH + j] = chunk_t{x.w[4 * j], x.w[4 * j + 1], x.w[4 * j + 2], x.w[4 * j + 3]};
            rsc[r] = x.s;
        } else {
            float4 *d = reinterpret_cast<float4 *>(rec + r * CH);
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const Cx<float> a = x.p[(2 * j) / 3][(2 * j) % 3], e = x.p[(2 * j + 1) / 3][(2 * j + 1) % 3];
                d[j] = make_float4(a.r, a.i, e.r, e.i);
            }
        }
    };
    Cx<float> A[4][3], hb[2][3];
    float hs;
    Rec<SL> p;
    MatRow u, utf, utb;
    auto staged = [&](int r) {
        __asm__("" : "+v"(r));
        uint4 w[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const chunk_t v = rec[r * CH + k];
            w[k] = make_uint4(v.x, v.y, v.z, v.w);
        }
        p.set(w, SC ? rsc[r] : 1.0f);
    };
    [[maybe_unused]] double n2 = 0.0;   // fused epilogue: this thread's |out|^2
    auto scale_sum = [&]() {
#pragma unroll
        for (int j = 0; j < 12; ++j) A[j / 3][j % 3] = {bt * A[j / 3][j % 3].r, bt * A[j / 3][j % 3].i};
    };
    // the forward t-hop of the slice before, with psi(x, tt) in p
    auto last_hop = [&]() {
        if constexpr (YMID) {
            Cx<float> h[2][3], chi[2][3];
            p.template proj<3, EF>(h);
            su3_mfma<false>(utf, h, chi);
            reconstruct_fma<3, EF, true>(A, chi, bt);
            pin(A);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            hop_mfma<3, EF, false, SL>(A, p, utf);
        }
    };
    // out(tt) from the finished sum (and with YEND y)
    auto finish = [&](int tt, [[maybe_unused]] const Rec<SP> &raw) {
        if constexpr (!YMID) scale_sum();
        if constexpr (MOBA) {
            // h = A: v = c5 h - cs y, out = diag y + b5 h + S^dagger v (no y for kMobHop and kMobHopInv)
            Rec<SpF32> v;
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                Cx<float> &a = A[j / 3][j % 3];
                v.p[j / 3][j % 3] = {mc5 * a.r, mc5 * a.i};
                a = {mb5 * a.r, mb5 * a.i};
            }
            if constexpr (HASY) {
                raw.axpy(v.p, csm);
                raw.axpy(A, dg);
            }
            column_shift_axpy<true>(v, A, wp, wm);
        } else if constexpr (YEND) {
            raw.axpy(A, dg);
            column_shift_axpy<DAG>(raw, A, csm * wp, csm * wm);
        }
        if constexpr (INV) column_m5inv_row<DAG>(A, s, static_cast<float>(1.0 / diag), static_cast<float>(mf));
        const size_t o = static_cast<size_t>(tt) * nq + q;
        if constexpr (FUSE == kFuseAxpy) {
            // r - alpha op psi; r may alias out: the thread reads its record before storing it
            Cx<float> rv[4][3];
            SP::load(fz.r, fz.r_scale, o, rv);
            const float al = static_cast<float>(fz.scal[fz.num] / fz.scal[fz.den]);
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                const Cx<float> a = A[j / 3][j % 3], e = rv[j / 3][j % 3];
                A[j / 3][j % 3] = {e.r - al * a.r, e.i - al * a.i};
            }
        }
        if constexpr (STAGE)   // the wavefront's part of the LDS is free: own records go there after this
            n2 += wave_store<SP, FUSE != kFuseNone>(rec + (td & ~63) * CH, nullptr,
                                                    static_cast<char *>(out) + static_cast<size_t>(slice(tt)) * nq * (CM * 16),
                                                    og, nullptr, A);
        else if constexpr (FUSE == kFuseNone)
            SP::store(out, out_scale, o, A);
        else
            n2 += SP::store_n2(out, out_scale, o, A);
    };
    {
        // the backward t-hop of slice t0: the column's record and its U_t at t0 - 1
        const int tm = t0 == 0 ? Lt - 1 : t0 - 1;
        Rec<SP> r;
        direct(psi, psi_scale, tm, q, r);
        hopped(r, p);
        p.template proj<3, -EF>(hb);
        hs = p.scale();
        Cx<float> w[3][3];
        const int x = 2 * (x0 + cx) + ((b0 + t0) & 1);
        LK::load(U, (static_cast<size_t>(tm) * V3 + (z * Ly + y0 + cy) * Lx + x) * 4 + 3, w);
        const int i = min(td & 3, 2);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float r0 = w[k][0].r, r1 = w[k][1].r, r2 = w[k][2].r, i0 = w[k][0].i, i1 = w[k][1].i, i2 = w[k][2].i;
            utb.r[k] = i == 0 ? r0 : i == 1 ? r1 : r2;
            utb.i[k] = i == 0 ? i0 : i == 1 ? i1 : i2;
        }
        utf = utb;
    }
#pragma unroll 1
    for (int k = 0; k < T; ++k) {
        const int tt = t0 + k;
        const int b = (b0 + tt) & 1;
        Rec<SP> own, hr, yr;
        alignas(16) char wl[LK::kBytes];
        auto others = [&]() {   // halo record and link
            if (c < NH) direct(psi, psi_scale, tt, (hb0 + tt) & 1 ? hq1 : hq0, hr);
            const char *l = static_cast<const char *>(U) + static_cast<size_t>(slice(tt)) * V3 * (4 * LK::kBytes) +
                            static_cast<size_t>(ug + ((ub + tt) & 1) * 4) * LK::kBytes;
            constexpr int al = LK::kBytes % 16 == 0 ? 16 : LK::kBytes % 8 == 0 ? 8 : 4;
            if (td < NS) __builtin_memcpy(wl, __builtin_assume_aligned(l, al), sizeof(wl));
        };
        auto put_all = [&]() {
            put(td, p);
            if (c < NH) {
                Rec<SL> hp;
                hopped(hr, hp);
                put(NC * Ls + td, hp);
            }
            if (td < NS) {
                Cx<float> wu[3][3];
                LK::load(wl, 0, wu);
                float2 *d = lks + td * 9;
#pragma unroll
                for (int e = 0; e < 9; ++e) d[e] = make_float2(wu[e / 3][e % 3].r, wu[e / 3][e % 3].i);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        direct(psi, psi_scale, tt, q, own);
        if constexpr (!STAGE) others();
        hopped(own, p);
        if constexpr (!STAGE) {
            put_all();
            if constexpr (YEND)
                if (k > 0) direct(yv, y_scale, tt - 1, q, yr);
        }
        // finish out(tt - 1) with psi(x, tt) and start the sum of out(tt)
        if (k > 0) {
            last_hop();
            if constexpr (YEND && STAGE) direct(yv, y_scale, tt - 1, q, yr);
            finish(tt - 1, yr);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (STAGE) others();   // not in registers beside the t-hop's
        {
            Cx<float> chi[2][3];
            su3_mfma<true>(utb, hb, chi);
#pragma unroll
            for (int j = 0; j < 12; ++j) A[j / 3][j % 3] = {0.f, 0.f};
            reconstruct_fma<3, -EF, SC>(A, chi, hs);
            p.renew();
            p.template proj<3, -EF>(hb);
            hs = p.scale();
        }
        if constexpr (STAGE) put_all();
        __syncthreads();
        Rec<SP> rz;
        direct(psi, psi_scale, tt, q + zpo, rz);   // in flight during the x hops
        staged(b ? nxp1 : td);
        mat_row<false>(link(c * 8), u);
        hop_mfma<0, EF, false, SL>(A, p, u);
        staged(b ? td : nxm0);
        mat_row<true>(link(b ? c * 8 + 4 : lxm0), u);
        hop_mfma<0, -EF, true, SL>(A, p, u);
        mat_row<false>(link(c * 8 + 2), u);
        {
            Rec<SL> pz;
            hopped(rz, pz);
            hop_mfma<2, EF, false, SL>(A, pz, u);
        }
        direct(psi, psi_scale, tt, q + zmo, rz);   // in flight during the y hops
        staged(nyp);
        mat_row<false>(link(c * 8 + 1), u);
        hop_mfma<1, EF, false, SL>(A, p, u);
        staged(nym);
        mat_row<true>(link(lym), u);
        hop_mfma<1, -EF, true, SL>(A, p, u);
        // in flight during the last z hop (issued before the y hops it spills: 60 us)
        if constexpr (YMID) direct(yv, y_scale, tt, q, yr);
        mat_row<true>(link(c * 8 + 6), u);
        {
            Rec<SL> pz;
            hopped(rz, pz);
            hop_mfma<2, -EF, true, SL>(A, pz, u);
        }
        if constexpr (YMID) {
            scale_sum();
            yr.axpy(A, dg);
            column_shift_axpy<DAG>(yr, A, csm * wp, csm * wm);
        }
        // U_t at the output's site (forward t-hop of out(tt)) and at the input's (backward one of out(tt + 1))
        mat_row<false>(link(c * 8 + 3), utf);
        mat_row<true>(link(c * 8 + 7), utb);
        __syncthreads();   // the next slice overwrites what was read here
    }
    {
        const int tl = t0 + T - 1;
        Rec<SP> r;
        direct(psi, psi_scale, tl == Lt - 1 ? 0 : tl + 1, q, r);
        hopped(r, p);
        Rec<SP> yr;
        if constexpr (YEND) direct(yv, y_scale, tl, q, yr);
        last_hop();
        finish(tl, yr);
    }
    if constexpr (FUSE != kFuseNone) {
        n2 = wave_sum64(n2);
        __shared__ double fred[4];
        if ((td & 63) == 0) fred[td >> 6] = n2;
        __syncthreads();
        if (td == 0) fz.part[blockIdx.x] = (fred[0] + fred[1]) + (fred[2] + fred[3]);
    }
}

// Tile 4 x 4, or 2 x 8 where only that divides (xh, y). Blocks along t: the count with the least (slices
// of the longest + 0.5) x (1.5 + m), m blocks on a CU (a walk's start and end cost about half a slice;
// one block's slice takes, with m of them on a CU, about as long as 1.5 + m), or beyond the three that
// fit a CU x (1 + 1.5 m), and no less than 6.5: a fourth block on a few CUs waits for a slot on each of them.
// Measured, nseg = 2 / 3 / 4 / 6 / 8 / 12 / 16: FP32 H 16^4 40 / 40 / 32 / 35 / 39 / 43 / 43 us, 24^4 206 / 186 / 189 / 180 / 183 /
// 198 / 209 us; FP16 storage 16^4 32 / 33 / 25 / 26 / 25 / 30 / 28 us; a fourth block on few: nseg = 2 / 4 / 5 / 7 / 14 at 16^3 x 14
// FP32 36 / 31 / 32 / 36 / 38, FP16 storage 29 / 25 / 26 / 25 / 26 (7 would be 3.5 a CU); 6 / 11 / 22 at 12 x 8 x 12 x 22 FP32
// 22 / 18 / 20, FP16 storage 18.1 / 15.1 / 15.9 (22: 3.1).
static PlaneCbDev plane_cb_dev(const GeomDev &g) {
    PlaneCbDev d{};
    d.ltx = (g.L[0] % 8 == 0 && g.L[1] % 4 == 0) ? 2 : (g.L[0] % 4 == 0 && g.L[1] % 8 == 0) ? 1 : 0;
    const long tiles = static_cast<long>(g.vol / g.L[3]) / 2 / kPcCols;
    double best = 0.0;
    for (int n = 1; n <= g.L[3]; n = next_walk_count(g.L[3], n)) {
        const double m = tiles * n / 256.0, t = (g.L[3] + n - 1) / n + 0.5;
        const double cost = t * (m <= 3.0 ? 1.5 + ceil(m) : fmax(6.5, 1.0 + 1.5 * m));
        if (n == 1 || cost < best) {
            best = cost;
            d.nseg = n;
        }
    }
    return d;
}

// Below these sizes (full lattice) the checkerboard column walk is as fast: FP32 8^3 x 16 x 16 (131072
// sites) 10.4 us both, 12 x 8 x 12^2 x 16 (221184) 12.3 here against 12.8, 16 x 8 x 16^2 x 16 (524288) 22 against
// 26; FP16 storage 12 x 8 x 12^2 x 16 11.3 us both, 16 x 8 x 16^2 x 16 15 both for H, 17 against 18 with y.
bool plane_cb_applies(const DhopArgs &a) {
    const int least = a.prec == GRID_F16S ? 400000 : 200000;
    return a.custom && a.cb >= 0 && a.kind != GRID_WILSON && (a.prec == GRID_F32 || a.prec == GRID_F16S) &&
           a.g.Ls == kPcLs && a.g.n5 >= least && plane_cb_dev(a.g).ltx != 0 && offsets32(a.g.n5 / a.g.L[3], 48);
}

long plane_cb_blocks(const DhopArgs &a) {
    return static_cast<long>(a.g.vol / a.g.L[3]) / 2 / kPcCols * plane_cb_dev(a.g).nseg;
}

template <class SP, class LK>
static hipError_t launch_plane_cb_t(const DhopArgs &a) {
    const PlaneCbDev d = plane_cb_dev(a.g);
    const dim3 grid(static_cast<unsigned>(plane_cb_blocks(a))), block(kPcThreads);
    hipStream_t st = a.stream;
#define GRIDMI_LAUNCH(DAG, KIND, FUSE)                                                                       \
    hipLaunchKernelGGL((k_dhop_plane_cb<SP, LK, DAG, KIND, FUSE>), grid, block,                              \
                       (plane_cb_lds_bytes<PcLds<SP, DAG, KIND>>()), st, a.U, a.psi, a.psi_scale, a.y, a.y_scale, \
                       a.out, a.out_scale, a.g, d, a.cb, a.diag, a.mf, a.beta, a.cs, a.b5, a.c5, a.fz)
    if (a.fuse != kFuseNone) {
        switch (a.kind * 4 + a.fuse * 2 + (a.dag ? 1 : 0)) {
            case GRID_DWF * 4 + kFuseNorm * 2 + 0: GRIDMI_LAUNCH(false, GRID_DWF, kFuseNorm); break;
            case kMobDiag * 4 + kFuseNorm * 2 + 0: GRIDMI_LAUNCH(false, kMobDiag, kFuseNorm); break;
            case GRID_DWF * 4 + kFuseAxpy * 2 + 1: GRIDMI_LAUNCH(true, GRID_DWF, kFuseAxpy); break;
            case kMobDiag * 4 + kFuseAxpy * 2 + 1: GRIDMI_LAUNCH(true, kMobDiag, kFuseAxpy); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (a.kind * 2 + (a.dag ? 1 : 0)) {
        case GRID_HOP * 2 + 0: GRIDMI_LAUNCH(false, GRID_HOP, kFuseNone); break;
        case GRID_HOP * 2 + 1: GRIDMI_LAUNCH(true, GRID_HOP, kFuseNone); break;
        case GRID_DWF * 2 + 0: GRIDMI_LAUNCH(false, GRID_DWF, kFuseNone); break;
        case GRID_DWF * 2 + 1: GRIDMI_LAUNCH(true, GRID_DWF, kFuseNone); break;
        case kMobHop * 2 + 0: GRIDMI_LAUNCH(false, kMobHop, kFuseNone); break;
        case kMobHop * 2 + 1: GRIDMI_LAUNCH(true, kMobHop, kFuseNone); break;
        case kMobDiag * 2 + 0: GRIDMI_LAUNCH(false, kMobDiag, kFuseNone); break;
        case kMobDiag * 2 + 1: GRIDMI_LAUNCH(true, kMobDiag, kFuseNone); break;
        case kHopInv * 2 + 0: GRIDMI_LAUNCH(false, kHopInv, kFuseNone); break;
        case kHopInv * 2 + 1: GRIDMI_LAUNCH(true, kHopInv, kFuseNone); break;
        case kMobHopInv * 2 + 0: GRIDMI_LAUNCH(false, kMobHopInv, kFuseNone); break;
        case kMobHopInv * 2 + 1: GRIDMI_LAUNCH(true, kMobHopInv, kFuseNone); break;
        default: return hipErrorInvalidValue;
    }
#undef GRIDMI_LAUNCH
    return hipGetLastError();
}

hipError_t launch_plane_cb(const DhopArgs &a) {
    switch (a.prec * 2 + a.link_fmt) {
        case GRID_F32 * 2 + GRID_L18: return launch_plane_cb_t<SpF32, LkF32<3>>(a);
        case GRID_F32 * 2 + GRID_L12: return launch_plane_cb_t<SpF32, LkF32<2>>(a);
        case GRID_F16S * 2 + GRID_L18: return launch_plane_cb_t<SpF16S, LkF16<3>>(a);
        case GRID_F16S * 2 + GRID_L12: return launch_plane_cb_t<SpF16S, LkF16<2>>(a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace gridmi
