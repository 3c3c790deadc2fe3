// Plane walk of the hopping operator on 5D fields (FP32 and FP16 storage, gfx950).
//
// A block owns a TX x TY tile of (x, y) columns at one z with all their s (one thread per 5D
// column, s fastest, TX TY Ls <= 384 threads) and walks T time slices. Per slice its own records,
// the tile's four faces and every link the slice's hops use go through LDS, so the four x and y
// hops, the fifth-dimension hop and the diagonal read LDS; the two z neighbours are read straight
// from memory; psi(x, t + 1) is the next slice's own record and the backward t-hop is carried in
// registers, as in the column walks. The finished records of a slice leave through LDS (wave_store)
// before the next slice's take their place there.
//
// Why. The column walks are bound by the number of 128-byte lines a site requests times their latency (a CU
// kept about 56 vector-L1 misses in flight in each of them and in a plain copy): 6.9 lines in the same-step walk,
// which fetches a record for each of its uses, and 3.75 here (FP32, 24^4 x 12; FP16 storage 3.9 and 2.1); and stores
// of 16 bytes per lane at the record's pitch send 24 million requests to the L2 there, more than the 14.9 million
// reads, against 6 million through LDS. Same-step walk / this kernel without / with the stores through LDS:
// 24^4 x 12 FP32 376 / 335 / 272 us from memory, in cache 320 -> 279, FP16 storage 190 -> 185 (now 177); 16^4 x 16
// FP32 105 / 72 / 60 us, FP16 storage 59 / 48 / 46; 16^4 x 8 FP32 40 -> 31 us. Moebius: B is applied once to each of the
// four records a site loads instead of to all eight it hops; M at 16^4 x 16 from memory, column walk / this kernel:
// FP32 108 / 74 us, FP16 storage 91 / 57 (its stores through LDS or by their lanes: the same within 1 % at 16^4,
// 24^4, 12^3 x 24 and 20 x 16 x 24 x 14).
// What bounds it now is the bytes that cross the fabric: 24^4 x 12 FP32 reads 1426 MB and writes 385 in 270 us,
// 6.7 TB/s, where a large copy reaches 5.4, and the mean latency of a read is 844 cycles, 447 to 477 in the kernels
// bound by requests. 2.98 times the compulsory bytes are read: a step of the blocks an XCD holds moves as
// much as its L2, so the z neighbours are mostly fetched again.
// Tried and not kept: the next slice's loads in registers during the hops (345 against 325 us in
// FP32, registers spill), streaming stores (580 us), tiles of two z planes (a quarter fewer requests, but
// one block per CU: 352 against 307 us); tiles ordered over 2 x 2 x 2 XCD domains (+- 2 %, in the first version of
// this kernel, which its stores bound: no finding about the present one).
//
// The SU(3) products run on the matrix cores: the four lanes of a v_mfma_f32_4x4x1 block are four s
// of one 4D site and share its link (su3_mfma), which needs Ls to be a multiple of four. A lane then
// holds one row of a link, 24 bytes from LDS in place of 72, and the kernel fits more wavefronts.
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace gridmi {

struct PlaneDev {
    int tx, ty;          // tile extents (powers of two)
    int ltx, lty;        // their logarithms
    int nseg;            // blocks along t: block i walks slices [i Lt / nseg, (i + 1) Lt / nseg)
};

// Halo columns of a tile: the -x, +x faces (ty each), then -y, +y (tx each).
// Link slots of a slice: the tile's own columns' four links (4 c + mu), U_z(x - z) of every column,
// U_x(x - x) at the -x face and U_y(x - y) at the -y face.

static size_t plane_lds_bytes(const PlaneDev &d, int Ls, int chunks, bool scaled) {
    const size_t nc = static_cast<size_t>(d.tx) * d.ty, nh = 2 * (d.tx + d.ty);
    const size_t slots = 5 * nc + d.tx + d.ty;
    return (nc + nh) * Ls * (chunks * 16 + (scaled ? 4 : 0)) + ((slots * 72 + 15) & ~size_t(15));
}

// Registers: three wavefronts per SIMD, two for the Moebius operators with FP32 records in LDS, of
// which two blocks fit a CU in any case (their 17 to 31 spilled registers at three).
template <class SP, class LK, bool DAG, int KIND, int FUSE>
__global__ void __launch_bounds__(384)
__attribute__((amdgpu_waves_per_eu(KIND == GRID_MOBIUS && !(SP::kScaled && DAG) ? 2 : 3)))
k_dhop_plane(const void *__restrict__ U, const void *__restrict__ psi, const float *__restrict__ psi_scale, void *out,
             float *out_scale, GeomDev g, PlaneDev pd, double diag, double mf, double cs, double b5, double c5,
             FuseDev fz) {
    static_assert(KIND == GRID_HOP || KIND == GRID_DWF || KIND == GRID_MOBIUS, "plain operators only");
    // Moebius (Ls = 16). M psi hops chi = B psi, B = b5 + c5 S: every record becomes chi where it is
    // loaded (a column is a DPP row), LDS holds chi in FP32, and out adds diag psi - cs S psi (diag =
    // 1 + (4 - M5) b5, cs = 1 - (4 - M5) c5). M^dagger psi hops psi, forms w = (4 - M5) psi - H^dagger
    // psi / 2 (diag = 4 - M5) and ends with b5 w + psi + S^dagger (c5 w - psi).
    constexpr bool MOBF = KIND == GRID_MOBIUS && !DAG;
    constexpr bool MOBA = KIND == GRID_MOBIUS && DAG;
    using SL = std::conditional_t<MOBF, SpF32, SP>;   // records in LDS
    constexpr bool SC = SL::kScaled;
    constexpr int CH = SL::kChunks;
    constexpr int KH = CH;   // halo chunks per thread (no more halo columns than own ones)
    extern __shared__ chunk_t plane_lds[];
    const int Ls = g.Ls, TX = pd.tx, TY = pd.ty, NC = TX * TY, NH = 2 * (TX + TY), NT = NC * Ls;
    const int NS = 5 * NC + TX + TY;
    chunk_t *rec = plane_lds;                                             // own records, then the halo's
    float2 *lks = reinterpret_cast<float2 *>(rec + (NC + NH) * Ls * CH);  // links, FP32, nine to a slot
    float *rsc = reinterpret_cast<float *>(rec + (NC + NH) * Ls * CH + (NS * 72 + 15) / 16);   // scales
    const int td = threadIdx.x;   // NT threads, a multiple of 64
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2], Lt = g.L[3];
    const int ntx = Lx >> pd.ltx, nty = Ly >> pd.lty, ntile = ntx * nty * Lz;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int seg = lb / ntile, tile = lb - seg * ntile;
    const int x0 = (tile % ntx) << pd.ltx, y0 = ((tile / ntx) % nty) << pd.lty, z = tile / (ntx * nty);
    const int c = td / Ls, s = td - c * Ls, cx = c & (TX - 1), cy = c >> pd.ltx;
    const int V3 = Lx * Ly * Lz, nq = V3 * Ls, plane = Lx * Ly;
    const int col = z * plane + (y0 + cy) * Lx + x0 + cx;
    const int zpo = (z == Lz - 1 ? 1 - Lz : 1) * plane * Ls, zmo = (z == 0 ? Lz - 1 : -1) * plane * Ls;
    const int q = col * Ls + s;
    const int t0 = seg * Lt / pd.nseg, T = (seg + 1) * Lt / pd.nseg - t0;
    constexpr int EF = DAG ? +1 : -1;
    // H and the domain-wall M: out = beta (H psi + (diag psi - S psi) / beta), beta = 1 for H and -1/2 for M
    const float bt = KIND == GRID_HOP ? 1.0f : -0.5f;
    const float dgb = static_cast<float>(diag) / bt;
    const float fpb = -((s == Ls - 1) ? static_cast<float>(-mf) : 1.0f) / bt;
    const float fmb = -((s == 0) ? static_cast<float>(-mf) : 1.0f) / bt;
    [[maybe_unused]] const float wp = (s == Ls - 1) ? static_cast<float>(-mf) : 1.0f;
    [[maybe_unused]] const float wm = (s == 0) ? static_cast<float>(-mf) : 1.0f;
    [[maybe_unused]] const float mb5 = static_cast<float>(b5), mc5 = static_cast<float>(c5);

    // Byte offsets, within a time slice, of this thread's stores (chunks j 64 + lane of the wavefront's
    // 64 records) and loads: halo chunks j NT + td, halo scales, one link. Its own record it loads whole
    // (and for MOBF a halo record).
    constexpr int CM = SP::kChunks;
    [[maybe_unused]] unsigned og[CM], hg[KH], hso = 0, ug, hq = 0;
#pragma unroll
    for (int j = 0; j < CM; ++j) {
        const int i = j * 64 + (td & 63), r = (td & ~63) + i / CM, row = r / (TX * Ls);
        og[j] = ((((z * Ly + y0 + row) * Lx + x0) * Ls + (r - row * (TX * Ls))) * CM + i % CM) * 16u;
    }
    auto halo_col = [&](int hc) -> int {   // first record of a halo column
        int hx, hy;
        if (hc < 2 * TY) {
            hx = hc < TY ? (x0 == 0 ? Lx - 1 : x0 - 1) : (x0 + TX == Lx ? 0 : x0 + TX);
            hy = y0 + (hc & (TY - 1));
        } else {
            hy = hc < 2 * TY + TX ? (y0 == 0 ? Ly - 1 : y0 - 1) : (y0 + TY == Ly ? 0 : y0 + TY);
            hx = x0 + ((hc - 2 * TY) & (TX - 1));
        }
        return ((z * Ly + hy) * Lx + hx) * Ls;
    };
    const int nhc = NH * Ls * CH;
#pragma unroll
    for (int j = 0; j < KH; ++j) {
        const int h = j * NT + td, hc = h / (Ls * CH), off = h - hc * (Ls * CH);
        hg[j] = h < nhc ? (halo_col(hc) * CH + off) * 16u : static_cast<unsigned>(q) * (CH * 16u);
    }
    if constexpr (MOBF) {
        const int hc = td / Ls;
        hq = td < NH * Ls ? halo_col(hc) + (td - hc * Ls) : q;
    }
    if constexpr (SC) {
        const int hc = td / Ls;
        hso = td < NH * Ls ? (halo_col(hc) + (td - hc * Ls)) * 4u : q * 4u;
    }
    {
        int lx = x0, ly = y0, lz = z, mu = 0;
        const int cc = td < 4 * NC ? td >> 2 : td - 4 * NC;
        if (td < 5 * NC) {
            mu = td < 4 * NC ? td & 3 : 2;
            lx = x0 + (cc & (TX - 1));
            ly = y0 + (cc >> pd.ltx);
            if (td >= 4 * NC) lz = z == 0 ? Lz - 1 : z - 1;
        } else if (td < 5 * NC + TY) {
            lx = x0 == 0 ? Lx - 1 : x0 - 1;
            ly = y0 + td - 5 * NC;
        } else if (td < NS) {
            mu = 1;
            ly = y0 == 0 ? Ly - 1 : y0 - 1;
            lx = x0 + td - 5 * NC - TY;
        }
        ug = ((lz * Ly + ly) * Lx + lx) * 4 + mu;
    }
    // LDS slots of the neighbours: records, and the backward hops' links
    const int nxp = cx < TX - 1 ? td + Ls : (NC + TY + cy) * Ls + s;
    const int nxm = cx > 0 ? td - Ls : (NC + cy) * Ls + s;
    const int nyp = cy < TY - 1 ? td + TX * Ls : (NC + 2 * TY + TX + cx) * Ls + s;
    const int nym = cy > 0 ? td - TX * Ls : (NC + 2 * TY + cx) * Ls + s;
    const int lxm = cx > 0 ? (c - 1) * 4 : 5 * NC + cy;
    const int lym = cy > 0 ? (c - TX) * 4 + 1 : 5 * NC + TY + cx;
    const int rsp = s == Ls - 1 ? td - (Ls - 1) : td + 1, rsm = s == 0 ? td + Ls - 1 : td - 1;

    // The slice index and the offsets are hidden from the loop optimiser at each use (empty asm, no
    // instruction): it would otherwise keep a 64-bit address per load across the loop instead of
    // forming the scalar-base, 32-bit-offset loads.
    auto slice = [](int tt) {
        __asm__("" : "+s"(tt));
        return tt;
    };
    auto load16 = [](const char *b, unsigned off) {
        __asm__("" : "+v"(off));
        return *reinterpret_cast<const chunk_t *>(b + off);
    };
    Cx<float> A[4][3], hb[2][3];
    float hs;
    Rec<SL> p;
    MatRow u, utf, utb;
    // record n of a slice, straight from memory
    auto direct = [&](int tt, unsigned n, Rec<SP> &r) {
        const char *b = static_cast<const char *>(psi) + static_cast<size_t>(slice(tt)) * nq * (CM * 16);
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
            const char *sb = reinterpret_cast<const char *>(psi_scale) + static_cast<size_t>(slice(tt)) * nq * 4;
            unsigned so = n * 4u;
            __asm__("" : "+v"(so));
            sc = *reinterpret_cast<const float *>(sb + so);
        }
        r.set(w, sc);
    };
    // the record the hops use: chi = B psi for M, else psi itself
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
    [[maybe_unused]] Rec<SP> raw;   // Moebius: psi(x, tt - 1) until out(tt - 1) is finished
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
                const Cx<float> a = x.p[(2 * j) / 3][(2 * j) % 3], b = x.p[(2 * j + 1) / 3][(2 * j + 1) % 3];
                d[j] = make_float4(a.r, a.i, b.r, b.i);
            }
        }
    };
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
    // out(tt) from the finished sum
    auto finish = [&](int tt) {
#pragma unroll
        for (int j = 0; j < 12; ++j) A[j / 3][j % 3] = {bt * A[j / 3][j % 3].r, bt * A[j / 3][j % 3].i};
        if constexpr (MOBA) {
            // A = -H^dagger psi / 2: w = (4 - M5) psi + A, v = c5 w - psi, out = b5 w + psi + S^dagger v
            raw.axpy(A, static_cast<float>(diag));
            Rec<SpF32> v;
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                Cx<float> &w = A[j / 3][j % 3];
                const Cx<float> c = raw.at(j);
                v.p[j / 3][j % 3] = {mc5 * w.r - c.r, mc5 * w.i - c.i};
                w = {mb5 * w.r + c.r, mb5 * w.i + c.i};
            }
            column_shift_axpy<true>(v, A, wp, wm);
        }
        if constexpr (MOBF) {
            // after the hops: added before them, the larger diag psi has every hop rounded at its size (b5 = 1.5,
            // c5 = 0.5: error 8.9e-8 of the result, here 7.0e-8, the column walk's)
            const float fs = -static_cast<float>(cs);
            raw.axpy(A, static_cast<float>(diag));
            column_shift_axpy<false>(raw, A, fs * wp, fs * wm);
        }
        const size_t o = static_cast<size_t>(tt) * nq + q;
        if constexpr (FUSE == kFuseAxpy) {
            // r - alpha op psi; r may alias out: the thread reads its record before storing it
            Cx<float> rv[4][3];
            SP::load(fz.r, fz.r_scale, o, rv);
            const float al = static_cast<float>(fz.scal[fz.num] / fz.scal[fz.den]);
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                const Cx<float> a = A[j / 3][j % 3], b = rv[j / 3][j % 3];
                A[j / 3][j % 3] = {b.r - al * a.r, b.i - al * a.i};
            }
        }
        chunk_t *wl = rec + (td & ~63) * CH;   // free here: own records go to LDS after this
        n2 += wave_store<SP, FUSE != kFuseNone>(wl, SC ? rsc + (td & ~63) : reinterpret_cast<float *>(wl + 64 * CM),
                                                static_cast<char *>(out) + static_cast<size_t>(slice(tt)) * nq * (CM * 16),
                                                og, SP::kScaled ? out_scale + o : nullptr, A);
    };
    {
        // the backward t-hop of slice t0: U_t(x, t0 - 1) and h(psi(x, t0 - 1))
        const int tm = t0 == 0 ? Lt - 1 : t0 - 1;
        Rec<SP> r;
        direct(tm, q, r);
        hopped(r, p);
        p.template proj<3, -EF>(hb);
        hs = p.scale();
        Cx<float> w[3][3];
        LK::load(U, (static_cast<size_t>(tm) * V3 + col) * 4 + 3, w);
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
        // finishes out(tt - 1) with psi(x, tt) (p) and starts the sum of out(tt)
        auto t_hops = [&](const Rec<SP> &centre) {
            if (k > 0) {
                hop_mfma<3, EF, false, SL>(A, p, utf);
                finish(tt - 1);
            }
            Cx<float> chi[2][3];
            su3_mfma<true>(utb, hb, chi);
#pragma unroll
            for (int j = 0; j < 12; ++j) A[j / 3][j % 3] = {0.f, 0.f};
            reconstruct_fma<3, -EF, SC>(A, chi, hs);
            p.renew();
            p.template proj<3, -EF>(hb);
            hs = p.scale();
            if constexpr (KIND == GRID_DWF) centre.axpy(A, dgb);
            if constexpr (MOBF || MOBA) raw = centre;
        };
        // Own record first: the t-hops need no other load.
        alignas(16) char wl[LK::kBytes];
        auto link_load = [&]() {
            const char *l = static_cast<const char *>(U) + static_cast<size_t>(slice(tt)) * V3 * (4 * LK::kBytes) +
                            static_cast<size_t>(ug) * LK::kBytes;
            constexpr int al = LK::kBytes % 16 == 0 ? 16 : LK::kBytes % 8 == 0 ? 8 : 4;
            __builtin_memcpy(wl, __builtin_assume_aligned(l, al), sizeof(wl));
        };
        auto link_put = [&]() {
            if (td < NS) {
                Cx<float> wu[3][3];
                LK::load(wl, 0, wu);
                float2 *d = lks + td * 9;
#pragma unroll
                for (int e = 0; e < 9; ++e) d[e] = make_float2(wu[e / 3][e % 3].r, wu[e / 3][e % 3].i);
            }
        };
        if constexpr (MOBF) {
            Rec<SP> own, hr;
            direct(tt, q, own);
            direct(tt, hq, hr);
            link_load();
            hopped(own, p);
            t_hops(own);
            put(td, p);
            // a halo record's s is td mod 16, this thread's own
            Rec<SL> hp;
            hopped(hr, hp);
            if (td < NH * Ls) put(NT + td, hp);
            link_put();
        } else {
            const char *b = static_cast<const char *>(psi) + static_cast<size_t>(slice(tt)) * nq * (CH * 16);
            chunk_t wh[KH];
            float sh = 1.f;
            direct(tt, q, p);
#pragma unroll
            for (int j = 0; j < KH; ++j) wh[j] = load16(b, hg[j]);
            if (SC) link_load();
            if constexpr (SC) {
                const char *sb = reinterpret_cast<const char *>(psi_scale) + static_cast<size_t>(slice(tt)) * nq * 4;
                sh = *reinterpret_cast<const float *>(sb + hso);
            }
            t_hops(p);
            __builtin_amdgcn_sched_barrier(0);
            if (!SC) link_load();   // FP32: not in registers beside the t-hops' (18 spilled)
            put(td, p);
#pragma unroll
            for (int j = 0; j < KH; ++j)
                if (j * NT + td < nhc) rec[(CH + j) * NT + td] = wh[j];
            if constexpr (SC)
                if (td < NH * Ls) rsc[NT + td] = sh;
            link_put();
        }
        __syncthreads();
        Rec<SP> rz;
        direct(tt, q + zpo, rz);   // in flight during the x hops
        if constexpr (KIND == GRID_DWF) {
            // - P_- psi~_{s+1} - P_+ psi~_{s-1} (M; P_+ and P_- exchanged for M^dagger)
            constexpr int hup = DAG ? 0 : 1;
            half_axpy<SP>(A, rec + rsp * CH, rsc + rsp, hup, fpb);
            half_axpy<SP>(A, rec + rsm * CH, rsc + rsm, 1 - hup, fmb);
        }
        staged(nxp);
        mat_row<false>(lks + (c * 4) * 9, u);
        hop_mfma<0, EF, false, SL>(A, p, u);
        staged(nxm);
        mat_row<true>(lks + lxm * 9, u);
        hop_mfma<0, -EF, true, SL>(A, p, u);
        mat_row<false>(lks + (c * 4 + 2) * 9, u);
        {
            Rec<SL> pz;
            hopped(rz, pz);
            hop_mfma<2, EF, false, SL>(A, pz, u);
        }
        direct(tt, q + zmo, rz);   // in flight during the y hops
        staged(nyp);
        mat_row<false>(lks + (c * 4 + 1) * 9, u);
        hop_mfma<1, EF, false, SL>(A, p, u);
        staged(nym);
        mat_row<true>(lks + lym * 9, u);
        hop_mfma<1, -EF, true, SL>(A, p, u);
        mat_row<true>(lks + (4 * NC + c) * 9, u);
        {
            Rec<SL> pz;
            hopped(rz, pz);
            hop_mfma<2, -EF, true, SL>(A, pz, u);
        }
        // U_t(x, tt): the forward t-hop of out(tt) and the backward one of out(tt + 1)
        mat_row<false>(lks + (c * 4 + 3) * 9, utf);
        mat_row<true>(lks + (c * 4 + 3) * 9, utb);
        __syncthreads();   // the next slice overwrites what was read here
    }
    {
        const int tl = t0 + T - 1;
        Rec<SP> r;
        direct(tl == Lt - 1 ? 0 : tl + 1, q, r);
        hopped(r, p);
        hop_mfma<3, EF, false, SL>(A, p, utf);
        finish(tl);
    }
    if constexpr (FUSE != kFuseNone) {
        n2 = wave_sum64(n2);
        __shared__ double fred[6];
        if ((td & 63) == 0) fred[td >> 6] = n2;
        __syncthreads();
        if (td == 0) {
            double v = 0.0;
            for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) v += fred[w];
            fz.part[blockIdx.x] = v;
        }
    }
}

// Tile: 4 x 4 columns for Ls = 12 to 24, 8 x 4 (or 4 x 8) for Ls = 8, so that a block has 192 to
// 384 threads, the halo no more columns than the tile and a slice's links no more than the threads.
// (Ls = 28 would leave one block to a CU in FP32.)
static bool plane_tile(const GeomDev &g, PlaneDev *d) {
    if (g.Ls % 4 == 0 && g.Ls >= 12 && g.Ls <= 24) {
        d->ltx = d->lty = 2;
    } else if (g.Ls == 8) {
        d->ltx = g.L[0] % 8 == 0 ? 3 : 2;
        d->lty = 5 - d->ltx;
    } else {
        return false;
    }
    d->tx = 1 << d->ltx;
    d->ty = 1 << d->lty;
    return g.L[0] % d->tx == 0 && g.L[1] % d->ty == 0;
}

// Blocks along t: the count with the least (T + start) x the sum over rounds of (a + blocks of the round on a
// CU), T slices the longest walk. A walk's start and end cost FP32 records 1.2 slices, codes 0.4, and a slice of one
// block takes, with m blocks on its CU, about as long as a + m (latency, then throughput; a = 2, for the five or
// six wavefronts of Ls = 20 and 24 0.25, and for codes 1). Walks are of at most 8 slices, in FP32 of 13 where all
// blocks run in one round (longer ones lose the reuse between neighbouring blocks: 24^4 x 16 T = 6 / 8 / 12
// 355 / 390 / 384 us); a count that does not divide Lt has to be a tenth better.
// Measured, T = 1 / 2 / 3 / 4 / 6 / 8 / 12: 24^4 x 12 FP32 362 / 297 / 270 / 274 / 273 / 288 / 286 us, FP16 storage
// 223 / 187 / 179 / 182 / 178 / 185 / 182; T = 1 / 2 / 4 / 8: 16^4 x 16 FP32 90 / 77 / 69 / 64, 16^4 x 12 FP16 storage
// 42 / 39 / 37 / 43; 16^3 x 13 x 24 FP32 T = 1 / 2 / 4 / 7 / 13 138 / 115 / 114 / 98 / 88 (the column walk 126), 20 x 12 x 21 x 5 x 12
// FP16 storage T = 1 / 2 / 5 25 / 21 / 28 (column walk 21.5), 8 x 24 x 19 x 14 x 12 T = 2 / 7 34 / 38 (35). Over 220 shapes
// with every count timed the choice is 0.9 % from the best.
static PlaneDev plane_dev(const GeomDev &g, bool scaled) {
    PlaneDev d{};
    if (!plane_tile(g, &d)) return d;
    const int waves = (d.tx * d.ty * g.Ls + 63) / 64;
    const long granules = (static_cast<long>(plane_lds_bytes(d, g.Ls, scaled ? 3 : 6, scaled)) + 1279) / 1280;
    const long by_lds = 128 / granules;   // 160 KB in granules of 1280 bytes
    const long per_cu = by_lds < 12 / waves ? by_lds : 12 / waves;   // three wavefronts per SIMD
    const long tiles = static_cast<long>(g.vol / g.L[3]) / (d.tx * d.ty);
    const double start = scaled ? 0.4 : 1.2, a = scaled ? 1.0 : g.Ls > 16 ? 0.25 : 2.0;
    double best = 0.0;
    for (int len = 1; len <= (scaled ? 8 : 13) && len <= g.L[3]; ++len) {
        const int n = (g.L[3] + len - 1) / len, T = (g.L[3] + n - 1) / n;
        const long m = (tiles * n + 255) / 256, rem = m % per_cu;
        if (T > 8 && m > per_cu) continue;
        const double cost = (T + start) * ((m / per_cu) * (a + per_cu) + (rem ? a + rem : 0.0)) * (g.L[3] % n ? 1.1 : 1.0);
        if (d.nseg == 0 || cost < best) {
            best = cost;
            d.nseg = n;
        }
    }
    return d;
}

// Below these sizes the column walk is faster (its wavefronts wait for nothing but their own loads):
// FP32 8^3 x 32 x 8 (131072 sites) 14.8 against 16.1 us here, 12^3 x 8 x 16 (221184) 25.7 against 21.7;
// FP16 storage 12^4 x 12 (248832) 17.9 against 20.6 us, 12^4 x 16 (331776) 23.2 against 21.8.
// Ls = 20 and 24 in FP32 only: 16^4 x 20 120.6 against 100.1 us here, 16^4 x 24 147.1 against 113.0, 12^4 x 24
// 49.6 against 43.8, 12^2 x 13 x 9 x 24 (404352 sites) 42.9 against 41.0, 12^2 x 10 x 8 x 20 (230400) 52.9 against 59.1
// (M^dagger M); FP16 storage, whose larger blocks leave a CU with
// fewer wavefronts than the column walk's, 16^4 x 20 78.8 against 89.3 us, 16^4 x 24 94.7 against 92.7, 12^4 x 24
// 33.4 against 37.9.
bool plane_applies(const DhopArgs &a) {
    PlaneDev d;
    const int least = a.prec == GRID_F16S ? 300000 : a.g.Ls > 16 ? 400000 : 160000;
    if (a.g.Ls > 16 && a.prec != GRID_F32) return false;
    const bool kind = a.kind == GRID_HOP || a.kind == GRID_DWF || (a.kind == GRID_MOBIUS && a.g.Ls == 16);
    return !a.custom && kind && (a.prec == GRID_F32 || a.prec == GRID_F16S) && a.g.n5 >= least && plane_tile(a.g, &d) &&
           offsets32(a.g.n5 / a.g.L[3], 96);
}

// Whether the block's records lie in LDS as FP16 codes and scales.
static bool plane_scaled(const DhopArgs &a) { return a.prec == GRID_F16S && !(a.kind == GRID_MOBIUS && !a.dag); }

long plane_blocks(const DhopArgs &a) {
    const PlaneDev d = plane_dev(a.g, plane_scaled(a));
    return static_cast<long>(a.g.vol / a.g.L[3]) / (d.tx * d.ty) * d.nseg;
}

template <class SP, class LK>
static hipError_t launch_plane_t(const DhopArgs &a) {
    const bool scaled = plane_scaled(a);
    const PlaneDev d = plane_dev(a.g, scaled);
    const dim3 grid(static_cast<unsigned>(plane_blocks(a))), block(d.tx * d.ty * a.g.Ls);
    const size_t lds = plane_lds_bytes(d, a.g.Ls, scaled ? 3 : 6, scaled);
    hipStream_t st = a.stream;
#define GRIDMI_LAUNCH(DAG, KIND, FUSE)                                                                          \
    hipLaunchKernelGGL((k_dhop_plane<SP, LK, DAG, KIND, FUSE>), grid, block, lds, st, a.U, a.psi, a.psi_scale, a.out, \
                       a.out_scale, a.g, d, a.diag, a.mf, a.cs, a.b5, a.c5, a.fz)
    if (a.fuse != kFuseNone) {
        switch (a.kind * 4 + a.fuse * 2 + (a.dag ? 1 : 0)) {
            case GRID_DWF * 4 + kFuseNorm * 2 + 0: GRIDMI_LAUNCH(false, GRID_DWF, kFuseNorm); break;
            case GRID_DWF * 4 + kFuseAxpy * 2 + 1: GRIDMI_LAUNCH(true, GRID_DWF, kFuseAxpy); break;
            case GRID_MOBIUS * 4 + kFuseNorm * 2 + 0: GRIDMI_LAUNCH(false, GRID_MOBIUS, kFuseNorm); break;
            case GRID_MOBIUS * 4 + kFuseAxpy * 2 + 1: GRIDMI_LAUNCH(true, GRID_MOBIUS, kFuseAxpy); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (a.kind * 2 + (a.dag ? 1 : 0)) {
        case GRID_HOP * 2 + 0: GRIDMI_LAUNCH(false, GRID_HOP, kFuseNone); break;
        case GRID_HOP * 2 + 1: GRIDMI_LAUNCH(true, GRID_HOP, kFuseNone); break;
        case GRID_DWF * 2 + 0: GRIDMI_LAUNCH(false, GRID_DWF, kFuseNone); break;
        case GRID_DWF * 2 + 1: GRIDMI_LAUNCH(true, GRID_DWF, kFuseNone); break;
        case GRID_MOBIUS * 2 + 0: GRIDMI_LAUNCH(false, GRID_MOBIUS, kFuseNone); break;
        case GRID_MOBIUS * 2 + 1: GRIDMI_LAUNCH(true, GRID_MOBIUS, kFuseNone); break;
        default: return hipErrorInvalidValue;
    }
#undef GRIDMI_LAUNCH
    return hipGetLastError();
}

hipError_t launch_plane(const DhopArgs &a) {
    switch (a.prec * 2 + a.link_fmt) {
        case GRID_F32 * 2 + GRID_L18: return launch_plane_t<SpF32, LkF32<3>>(a);
        case GRID_F32 * 2 + GRID_L12: return launch_plane_t<SpF32, LkF32<2>>(a);
        case GRID_F16S * 2 + GRID_L18: return launch_plane_t<SpF16S, LkF16<3>>(a);
        case GRID_F16S * 2 + GRID_L12: return launch_plane_t<SpF16S, LkF16<2>>(a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace gridmi
