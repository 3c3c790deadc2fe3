// Tiled time-walk schedule of the hopping operator on 4D fields (gfx950).
//
// Why a third schedule. The column walk fetches each spinor record once per use (eight times)
// and each link once per lane, so it requests several times the compulsory bytes per site. Here
// neighbour reuse happens in LDS instead (Grid's observation, Section 3, that a neighbour spinor
// is used eight times, turned into on-chip reuse). It serves 4D fields in FP16 storage and large
// ones in FP32, where it is the fastest schedule measured.
//
// A block owns a TX x TY x TZ tile of (x, y, z) columns, one thread per column (a wavefront per
// z-plane of the tile), and walks T time slices. Per slice every thread writes its own record
// psi(x, t) to LDS, and the halo faces of slice t (loaded with coalesced 16-byte pieces during the
// previous slice) go beside it; the six spatial hops read LDS. The forward time neighbour
// psi(x, t + 1) is the thread's next centre and stays in registers; the backward time hop
// U_t(x, t-1)^dagger h(psi(x, t-1)) is formed one step ahead from the record and link already in
// hand and carried, as in the column walk. Links: the tile's own, four per site, are contiguous rows
// of memory and go to LDS as stored, with the links of the -x, -y and -z faces beside them; forward
// and backward hops decode theirs from there.
//
// What bounds it: vector instructions (1290 per slice of a wavefront, 36 of 55 us at 32^4) beside the
// 41 us its bytes take. A wavefront that staged one direction's 64 links at a time, seven times per
// slice, touched the same cache lines (24-byte links of four directions at 96-byte pitch) each time:
// 12-real 32^4 70 -> 62 us from memory, 58 -> 55 in cache, 18-real 72 -> 56, 24^4 x 18-real 30 -> 26; before
// that the records' conversion and scaling ahead of the projection, and a last round of blocks a third
// full: 75.5 -> 70 us, 18-real 79 -> 72. FP32: 32^4 143 (direction-parallel) -> 108 us from memory, whose
// bytes take 99 us, with 12-real links 126 -> 90.
//
// Per site: 8 x (12 + 132) + 7 x 24 = 1320 flops, the convention of the flop counts quoted for
// this operator.
#include <math.h>

#include <type_traits>

#include "device.h"
#include "launch.h"

namespace gridmi {

template <int TX, int TY, int TZ>
struct TileShape {
    static constexpr int N = TX * TY * TZ;                 // interior columns = threads
    static constexpr int HX = TY * TZ, HY = TX * TZ, HZ = TX * TY;
    static constexpr int NH = 2 * (HX + HY + HZ);         // halo records (faces only)
    // halo slots after the interior: -x, +x, -y, +y, -z, +z faces
    static constexpr int XM = 0, XP = HX, YM = 2 * HX, YP = 2 * HX + HY, ZM = 2 * (HX + HY), ZP = ZM + HZ;
};

struct TileDev {
    int ntx, nty, ntz;   // tiles per direction
    int nseg;            // blocks along t: block i walks slices [i Lt / nseg, (i + 1) Lt / nseg)
};

// Record of LDS slot `slot` (16-byte chunks at the record pitch), undecoded.
template <class SP>
__device__ __forceinline__ void lds_record(const chunk_t *base, const float *sbase, int slot, Rec<SP> &p) {
    constexpr int CH = SP::kChunks;
    uint4 w[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        const chunk_t v = base[slot * CH + k];
        w[k] = make_uint4(v.x, v.y, v.z, v.w);
    }
    p.set(w, SP::kScaled ? sbase[slot] : 1.0f);
}

// Global chunk offset (relative to the start of a time slice) of chunk c of the tile's loads:
// c < N CH are the interior rows (row-major z, y, x, then chunk), the rest the halo faces.
template <int TX, int TY, int TZ, int CH>
__device__ __forceinline__ int tile_chunk_offset(const GeomDev &g, int x0, int y0, int z0, int c) {
    using S = TileShape<TX, TY, TZ>;
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2];
    int x, y, z, j;
    if (c < S::N * CH) {
        const int row = c / (TX * CH), off = c - row * (TX * CH);
        const int ry = row % TY, rz = row / TY;
        const int rx = off / CH;
        j = off - rx * CH;
        x = x0 + rx;
        y = y0 + ry;
        z = z0 + rz;
    } else {
        c -= S::N * CH;
        const int r = c / CH;
        j = c - r * CH;
        const int xm = x0 == 0 ? Lx - 1 : x0 - 1, xp = x0 + TX == Lx ? 0 : x0 + TX;
        const int ym = y0 == 0 ? Ly - 1 : y0 - 1, yp = y0 + TY == Ly ? 0 : y0 + TY;
        const int zm = z0 == 0 ? Lz - 1 : z0 - 1, zp = z0 + TZ == Lz ? 0 : z0 + TZ;
        if (r < S::YM) {                 // x faces: index over (y, z)
            const int i = r < S::XP ? r : r - S::XP;
            x = r < S::XP ? xm : xp;
            y = y0 + i % TY;
            z = z0 + i / TY;
        } else if (r < S::ZM) {          // y faces: index over (x, z)
            const int i = r < S::YP ? r - S::YM : r - S::YP;
            y = r < S::YP ? ym : yp;
            x = x0 + i % TX;
            z = z0 + i / TX;
        } else {                         // z faces: index over (x, y)
            const int i = r < S::ZP ? r - S::ZM : r - S::ZP;
            z = r < S::ZP ? zm : zp;
            x = x0 + i % TX;
            y = y0 + i / TX;
        }
    }
    return ((z * Ly + y) * Lx + x) * CH + j;
}

// Links of a tile in LDS: a site's four links as stored and eight bytes of padding (the reads of a
// wavefront, one link per lane at this pitch, then spread over all banks), the face links after them. The
// pitch leaves a link aligned to its unit of eight or four bytes, not to the 16 that a 12-real FP32 link is
// read by from memory: get() reads units (16-byte reads there are undefined, and where the hardware allows
// them slower: 32^4 98 to 102 us, in units 89 to 92).
template <class LK>
struct LinkTile {
    static constexpr int LB = LK::kBytes;
    static constexpr int kPitch = 4 * LB + 8;
    static constexpr int kChunks = 4 * LB / 16;         // 16-byte chunks per site = chunks per lane
    static constexpr int kUnit = LB % 8 == 0 ? 8 : 4;   // a face link is copied in these
    static constexpr int kUnits = LB / kUnit;
    typedef unsigned int u2v __attribute__((ext_vector_type(2)));
    using T = std::conditional_t<kUnit == 8, u2v, uint32_t>;
    static_assert(kPitch % kUnit == 0 && LB % kUnit == 0 && kUnit % sizeof(T) == 0, "links aligned to their unit");
    // the link at sl + at (a multiple of kUnit)
    __device__ __forceinline__ static void get(const char *sl, int at, Cx<typename LK::C> u[3][3]) {
        if constexpr (LK::kAlign <= kUnit) {
            LK::load(sl + at, 0, u);
        } else {
            alignas(LK::kAlign) char w[LB];
#pragma unroll
            for (int k = 0; k < kUnits; ++k) {
                const T v = reinterpret_cast<const T *>(sl + at)[k];
                __builtin_memcpy(w + k * kUnit, &v, kUnit);
            }
            LK::load(w, 0, u);
        }
    }
};

template <class SP, class LK, bool DAG, int KIND, int FUSE, int TX, int TY, int TZ>
__global__ void __launch_bounds__(TX * TY * TZ) __attribute__((amdgpu_waves_per_eu(SP::kScaled ? 2 : 1)))
k_dhop_tile(const void *__restrict__ U, const void *__restrict__ psi, const float *__restrict__ psi_scale, void *out,
            float *out_scale, GeomDev g, TileDev td, double diag, FuseDev fz) {
    using C = typename SP::C;
    using S = TileShape<TX, TY, TZ>;
    using LT = LinkTile<LK>;
    using LU = typename LT::T;
    static_assert(TX * TY == 64, "one wavefront per z-plane of the tile");
    constexpr int N = S::N, CH = SP::kChunks, NU = LT::kUnits, NL = LT::kChunks;
    constexpr int KH = (S::NH * CH + N - 1) / N;         // halo chunks per thread
    __shared__ chunk_t sb[(N + S::NH) * CH];             // interior, then halo records of slice t
    __shared__ float sbs[SP::kScaled ? N + S::NH : 1];   // FP16 storage: their scales
    constexpr int NF = S::HX + S::HY + S::HZ;            // links of the -x, -y and -z faces
    __shared__ __align__(16) char sl[N * LT::kPitch + NF * LT::LB];

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int ntiles = td.ntx * td.nty * td.ntz;
    const int seg = lb / ntiles, tile = lb - seg * ntiles;
    const int x0 = (tile % td.ntx) * TX, y0 = ((tile / td.ntx) % td.nty) * TY, z0 = (tile / (td.ntx * td.nty)) * TZ;
    const int cx = tid % TX, cy = (tid / TX) % TY, cz = tid / (TX * TY);
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2], Lt = g.L[3];
    const int V3 = Lx * Ly * Lz;
    const int x = x0 + cx, y = y0 + cy, z = z0 + cz;
    const int col = (z * Ly + y) * Lx + x;
    const int t0 = seg * Lt / td.nseg, T = (seg + 1) * Lt / td.nseg - t0;
    constexpr int EF = DAG ? +1 : -1;

    // halo chunk offsets of this thread's loads (slice-relative, fixed along the walk)
    int hoff[KH];
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        const int c = N * CH + k * N + tid;
        hoff[k] = c < (N + S::NH) * CH ? tile_chunk_offset<TX, TY, TZ, CH>(g, x0, y0, z0, c) : -1;
    }
    int hrec = -1;   // FP16 storage: this thread's halo scale
    if constexpr (SP::kScaled) {
        static_assert(!SP::kScaled || S::NH <= N, "one halo scale per thread");
        if (tid < S::NH) hrec = tile_chunk_offset<TX, TY, TZ, 1>(g, x0, y0, z0, N + tid);
    }
    // neighbour slots (LDS): interior slot or halo slot (>= N)
    const int own = tid;
    const int nxp = cx < TX - 1 ? own + 1 : N + S::XP + cy + TY * cz;
    const int nxm = cx > 0 ? own - 1 : N + S::XM + cy + TY * cz;
    const int nyp = cy < TY - 1 ? own + TX : N + S::YP + cx + TX * cz;
    const int nym = cy > 0 ? own - TX : N + S::YM + cx + TX * cz;
    const int nzp = cz < TZ - 1 ? own + TX * TY : N + S::ZP + cx + TX * cy;
    const int nzm = cz > 0 ? own - TX * TY : N + S::ZM + cx + TX * cy;
    // links: a wavefront loads the four links of its z-plane's 64 sites, rows of TX sites contiguous in
    // memory, and threads below NF one link of a -x, -y or -z face each
    unsigned lofs[NL], lfof = 0;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int u = k * 64 + lane, row = u / (TX * NL), off = u - row * (TX * NL);
        lofs[k] = static_cast<unsigned>(((z * Ly + y0 + row) * Lx + x0) * NL + off) * 16u;
    }
    if (tid < NF) {
        int fx = x0, fy = y0, fz0 = z0, mu;
        if (tid < S::HX) {
            fx = x0 == 0 ? Lx - 1 : x0 - 1;
            fy += tid % TY;
            fz0 += tid / TY;
            mu = 0;
        } else if (tid < S::HX + S::HY) {
            const int i = tid - S::HX;
            fy = y0 == 0 ? Ly - 1 : y0 - 1;
            fx += i % TX;
            fz0 += i / TX;
            mu = 1;
        } else {
            const int i = tid - S::HX - S::HY;
            fz0 = z0 == 0 ? Lz - 1 : z0 - 1;
            fx += i % TX;
            fy += i / TX;
            mu = 2;
        }
        lfof = static_cast<unsigned>(((fz0 * Ly + fy) * Lx + fx) * 4 + mu) * LT::LB;
    }
    // stores: byte offsets, within a slice, of chunks k 64 + lane of the wavefront's records
    [[maybe_unused]] unsigned oofs[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        const int i = k * 64 + lane, r = i / CH;
        oofs[k] = static_cast<unsigned>(((z * Ly + y0 + r / TX) * Lx + x0 + r % TX) * CH + i % CH) * 16u;
    }
    // LDS byte offsets of the links: own site, and the backward hops'
    constexpr int FB = N * LT::kPitch;
    const int lown = tid * LT::kPitch;
    const int lxm = cx > 0 ? lown - LT::kPitch : FB + (cy + TY * cz) * LT::LB;
    const int lym = cy > 0 ? lown - TX * LT::kPitch + LT::LB : FB + (S::HX + cx + TX * cz) * LT::LB;
    const int lzm = cz > 0 ? lown - TX * TY * LT::kPitch + 2 * LT::LB : FB + (S::HX + S::HY + cx + TX * cy) * LT::LB;
    const char *ub = static_cast<const char *>(U);
    chunk_t lw[NL];
    LU lf[NU];
    auto issue_links = [&](int t) {
        const char *tb = ub + static_cast<size_t>(t) * V3 * (4 * LT::LB);
#pragma unroll
        for (int k = 0; k < NL; ++k) lw[k] = *reinterpret_cast<const chunk_t *>(tb + lofs[k]);
        if (tid < NF)
#pragma unroll
            for (int k = 0; k < NU; ++k) lf[k] = *reinterpret_cast<const LU *>(tb + lfof + k * LT::kUnit);
    };
    auto put_links = [&]() {
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            typedef unsigned int u2v __attribute__((ext_vector_type(2)));
            const int u = k * 64 + lane;
            u2v *d = reinterpret_cast<u2v *>(sl + wv * (64 * LT::kPitch) + u * 16 + (u / NL) * 8);
            // a chunk of a site starts 16 (u mod NL) bytes into it
            d[0] = u2v{lw[k].x, lw[k].y};
            d[1] = u2v{lw[k].z, lw[k].w};
        }
        if (tid < NF)
#pragma unroll
            for (int k = 0; k < NU; ++k) *reinterpret_cast<LU *>(sl + FB + tid * LT::LB + k * LT::kUnit) = lf[k];
    };

    const chunk_t *src = reinterpret_cast<const chunk_t *>(psi);
    chunk_t wh[KH];
    float shv = 1.0f;
    auto issue_halo = [&](int t) {
        const size_t cbase = static_cast<size_t>(t) * V3 * CH;
#pragma unroll
        for (int j = 0; j < KH; ++j)
            if (hoff[j] >= 0) wh[j] = src[cbase + hoff[j]];
        if constexpr (SP::kScaled)
            if (hrec >= 0) shv = psi_scale[static_cast<size_t>(t) * V3 + hrec];
    };
    // raw record (chunks + scale) of this thread's column at slice tt
    auto own_raw = [&](int tt, uint4 w[CH], float &sc) {
        const size_t r = static_cast<size_t>(tt) * V3 + col;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const chunk_t v = src[r * CH + j];
            w[j] = make_uint4(v.x, v.y, v.z, v.w);
        }
        sc = SP::kScaled ? psi_scale[r] : 1.0f;
    };
    Cx<C> chi_b[2][3], u[3][3];
    C chi_s;   // chi_b is the transported half-spinor over the record's scale
    Rec<SP> p;
    uint4 Pw[CH];      // centre record psi(x, t), raw
    float Ps = 1.0f;
    {
        // prologue: the backward time hop of slice t0, U_t(x, t0 - 1)^dagger h(psi(x, t0 - 1)),
        // the centre record psi(x, t0) and slice t0's halo
        const int tm = t0 == 0 ? Lt - 1 : t0 - 1;
        uint4 w[CH];
        float sc;
        own_raw(tm, w, sc);
        own_raw(t0, Pw, Ps);
        issue_halo(t0);
        issue_links(t0);
        LK::load(U, (static_cast<size_t>(tm) * V3 + col) * 4 + 3, u);
        Cx<C> hb[2][3];
        p.set(w, sc);
        p.template proj<3, -EF>(hb);
        su3_adj_mul(u, hb, chi_b);
        chi_s = p.scale();
    }
    [[maybe_unused]] double n2 = 0.0;
#pragma unroll 1
    for (int k = 0; k < T; ++k) {
        const int t = t0 + k;
        const int tn = t == Lt - 1 ? 0 : t + 1;
        // stage this thread's centre record and its share of the halo of slice t
#pragma unroll
        for (int j = 0; j < CH; ++j) sb[tid * CH + j] = chunk_t{Pw[j].x, Pw[j].y, Pw[j].z, Pw[j].w};
        if constexpr (SP::kScaled) sbs[tid] = Ps;
#pragma unroll
        for (int j = 0; j < KH; ++j)
            if (hoff[j] >= 0) sb[(CH + j) * N + tid] = wh[j];
        if constexpr (SP::kScaled)
            if (hrec >= 0) sbs[N + tid] = shv;
        put_links();
        __syncthreads();
        // the forward time neighbour psi(x, t + 1) (the next centre) and the next halo
        uint4 Qw[CH];
        float Qs = 1.0f;
        own_raw(tn, Qw, Qs);
        if (k + 1 < T) {
            issue_halo(tn);
            issue_links(tn);
        }
        auto rec = [&](int slot, Rec<SP> &q) { lds_record<SP>(sb, sbs, slot, q); };
        // FP32: the two hops of a direction are added to each other first, then to the sum, which keeps the
        // chain of roundings as short as the direction-parallel kernel's (error at 32^4 7.4e-8 of the
        // result; one chain of eight 7.8e-8)
        constexpr bool PAIR = !SP::kScaled;
        Cx<C> acc[4][3];
        [[maybe_unused]] Cx<C> two[4][3];
        Cx<C>(&sum)[4][3] = PAIR ? two : acc;
        auto clear = [](Cx<C> a[4][3]) {
#pragma unroll
            for (int j = 0; j < 12; ++j) a[j / 3][j % 3] = {C(0), C(0)};
        };
        auto pair_done = [&]() {
            if constexpr (PAIR) {
#pragma unroll
                for (int j = 0; j < 12; ++j) acc[j / 3][j % 3] = cadd(acc[j / 3][j % 3], two[j / 3][j % 3]);
                clear(two);
            }
        };
        clear(acc);
        if constexpr (PAIR)
            clear(two);
        else
            reconstruct_fma<3, -EF, SP::kScaled>(acc, chi_b, chi_s);
        rec(nxp, p);
        LT::get(sl, lown, u);
        hop_rec<0, EF, false, SP>(sum, p, u);
        rec(nxm, p);
        LT::get(sl, lxm, u);
        hop_rec<0, -EF, true, SP>(sum, p, u);
        pair_done();
        rec(nyp, p);
        LT::get(sl, lown + LT::LB, u);
        hop_rec<1, EF, false, SP>(sum, p, u);
        rec(nym, p);
        LT::get(sl, lym, u);
        hop_rec<1, -EF, true, SP>(sum, p, u);
        pair_done();
        rec(nzp, p);
        LT::get(sl, lown + 2 * LT::LB, u);
        hop_rec<2, EF, false, SP>(sum, p, u);
        rec(nzm, p);
        LT::get(sl, lzm, u);
        hop_rec<2, -EF, true, SP>(sum, p, u);
        pair_done();
        // forward time hop psi(x, t + 1) with U_t(x, t); the same link carries the backward time
        // hop of slice t + 1, U_t(x, t)^dagger h(psi(x, t))
        LT::get(sl, lown + 3 * LT::LB, u);
        p.set(Qw, Qs);
        if constexpr (PAIR) reconstruct_fma<3, -EF, SP::kScaled>(two, chi_b, chi_s);
        hop_rec<3, EF, false, SP>(sum, p, u);
        pair_done();
        rec(own, p);   // the centre psi(x, t), as staged
        if constexpr (KIND != GRID_HOP) {
            // D = (4 + m) - H/2
            const C dg = static_cast<C>(diag);
#pragma unroll
            for (int j = 0; j < 12; ++j) acc[j / 3][j % 3] = {C(-0.5) * acc[j / 3][j % 3].r, C(-0.5) * acc[j / 3][j % 3].i};
            p.axpy(acc, dg);
        }
        {
            Cx<C> h[2][3];
            p.renew();
            p.template proj<3, -EF>(h);
            su3_adj_mul(u, h, chi_b);
            chi_s = p.scale();
        }
        const size_t q = static_cast<size_t>(t) * V3 + col;
        if constexpr (FUSE == kFuseAxpy) {
            // r - alpha op psi; r may alias out: this thread reads its own record before storing it
            Cx<C> rv[4][3];
            SP::load(fz.r, fz.r_scale, q, rv);
            const C al = static_cast<C>(fz.scal[fz.num] / fz.scal[fz.den]);
#pragma unroll
            for (int j = 0; j < 12; ++j) {
                const Cx<C> a = acc[j / 3][j % 3], b = rv[j / 3][j % 3];
                acc[j / 3][j % 3] = {b.r - al * a.r, b.i - al * a.i};
            }
        }
        if constexpr (SP::kScaled) {
            if constexpr (FUSE == kFuseNone)
                SP::store(out, out_scale, q, acc);
            else
                n2 += SP::store_n2(out, out_scale, q, acc);
        }
#pragma unroll
        for (int j = 0; j < CH; ++j) Pw[j] = Qw[j];
        Ps = Qs;
        __syncthreads();   // the next slice overwrites the records read here
        // FP32: stored through the wavefront's part of the records (110.5 -> 106.6 us at 32^4); FP16 storage,
        // at half the pitch, is as fast stored by its lane (61.7 against 62.1 us)
        if constexpr (!SP::kScaled)
            n2 += wave_store<SP, FUSE != kFuseNone>(sb + (tid & ~63) * CH, nullptr,
                                                    static_cast<char *>(out) + static_cast<size_t>(t) * V3 * (CH * 16), oofs,
                                                    nullptr, acc);
    }
    if constexpr (FUSE != kFuseNone) {
        n2 = wave_sum64(n2);
        constexpr int NW = N / 64;
        __shared__ double fred[NW];
        if ((tid & 63) == 0) fred[tid >> 6] = n2;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += fred[w];
            fz.part[blockIdx.x] = s;
        }
    }
}

// Tiles: 8 x 8 x 4 (256 threads) for FP16 storage, 8 x 8 x 2 for FP32, whose links and records fill the
// LDS (76 KB; 8 x 8 x 4 takes 134 KB, with 12-real links 104, and one block per CU: 32^4 18-real 115 against 108 us,
// 12-real 100 against 90, 32^3 x 16 63 and 54 against 59 and 50). Two blocks fit a CU. Blocks along t: the count with
// the least (slices of the longest + start) x the sum over the rounds of blocks a CU runs at a time, 2.5 for two
// and `alone` for one; start and alone as measured, FP32's longer prefetch weighing more. 12-real links: FP16 storage,
// nseg = 1 / 2 / 4 / 6 / 8 / 12 / 16, 32^4 116 / 64 / 55 / 62 / 59 / 65 / 62 us, 24^4 87 / 47 / 28 / 30 / 25 / 26 / 29; FP32 32^4,
// nseg = 1 / 2 / 4 / 6 / 8 / 16, 138 / 90 / 99 / 111 / 112 / 131 us, 18-real 143 / 108 / 121 / 128 / 130 / 158. FP16 storage, two
// blocks of one slice against one of two: 16 x 24 x 12 x 28 nseg 28 / 14 10.6 / 11.7 us, 16^2 x 20 x 24 nseg 24 / 12
// 10.6 / 11.5; three of one against two of two: 24^2 x 20 x 16 nseg 16 / 8 17.3 / 18.8 us.
constexpr int kTX = 8, kTY = 8;
template <class SP>
constexpr int kTZ = SP::kScaled ? 4 : 2;

static int tile_z(const DhopArgs &a) { return a.prec == GRID_F16S ? kTZ<SpF16S> : kTZ<SpF32>; }

// share: the slices of an evenly spread lattice over those the model charges (at least one).
static TileDev tile_dev(const DhopArgs &a, double *share = nullptr) {
    const GeomDev &g = a.g;
    const double start = a.prec == GRID_F16S ? 0.4 : 0.7, alone = a.prec == GRID_F16S ? 1.5 : 1.8;
    TileDev td;
    td.ntx = g.L[0] / kTX;
    td.nty = g.L[1] / kTY;
    td.ntz = g.L[2] / tile_z(a);
    const long ntiles = static_cast<long>(td.ntx) * td.nty * td.ntz;
    double best = 0.0;
    for (int n = 1; n <= g.L[3]; n = next_walk_count(g.L[3], n)) {
        const long m = (ntiles * n + 255) / 256, rem = m % 2;
        const double cost = ((g.L[3] + n - 1) / n + start) * ((m / 2) * 2.5 + (rem ? alone : 0.0));
        if (n == 1 || cost < best) {
            best = cost;
            td.nseg = n;
        }
    }
    if (share) *share = static_cast<double>(ntiles) * g.L[3] / 256.0 * 1.25 / best;
    return td;
}

// 4D fields the tile divides. FP16 storage: all (32^4: 55 us, the column walk 93, the direction-parallel kernel
// 132), but with 12-real links not those of 2 to 2.83 slices of a block per CU, where two blocks on a CU take a
// third round for a part of one: H here / column walk 16 x 8 x 28 x 38 (2.1) 16.2 / 15.3 us, 24 x 16 x 20^2 (2.3) 16.8 /
// 15.4, 24^3 x 13 (2.7) 18.6 / 16.8, 24^2 x 20 x 16 (2.8) 18.4 / 16.4, D 18.6 / 16.9, and beside that range 16^3 x 28 (1.75)
// 11.9 / 12.1, 24^2 x 36 x 9 (2.85) 17.3 / 19.0, 24^3 x 15 (3.2) 19.4 / 21.1; nor, for the same reason, those of 4 to 5
// in time slices of up to 15000 sites (larger ones slow the column walk): 8 x 24 x 36 x 38 (4.01) 23.9 / 22.1, 24 x 16
// x 24 x 31 (4.4) 24.7 / 23.3, 32 x 24 x 12 x 34 (4.8) 25.0 / 24.0, 24 x 32 x 16 x 26 (4.9) 24.8 / 24.5, D 25.0 / 24.4, beside them
// 40 x 16^2 x 24 (3.75) 20.0 / 20.7, 24 x 16 x 32 x 27 (5.06) 24.8 / 27.4, 48 x 16 x 36 x 10 (4.2, 27648 sites) 24.6 / 27.9;
// with 18-real links 24^3 x 13 19.4 / 21.8.
// FP32: from 500000 sites on (24^4, 331776 sites, which the caches hold, 12-real 35.4 us here, 34.7
// direct) where the blocks keep the CUs evenly busy: a share of at least 0.78 (18-real) or 0.70 (12-real).
// Direction-parallel / tile from memory, H with 18-real and 12-real links, by share: 56 x 32 x 24^2 (0.91) 137 / 125,
// 126 / 104 us, 32 x 24 x 28 x 26 (0.88) 78 / 65, 69 / 55, 40^2 x 24^2 (0.82) 123 / 117, 110 / 100, 32^2 x 20 x 28 (0.82) 80 / 69,
// 71 / 58, 32^2 x 24^2 (0.81) 82 / 83, 71 / 70 (D 12-real 76 / 71), 24^2 x 32 x 30 (0.79) 73 / 67, 66 / 57, 16 x 48 x 30 x 28
// (0.77) 87 / 89, 78 / 76, 48 x 16 x 30 x 27 (0.74) 87 / 88, 77 / 76, 56 x 48 x 26 x 9 (0.70) 93 / 95, 82 / 82.
bool tile_applies(const DhopArgs &a) {
    if (a.custom || a.g.Ls != 1 || (a.kind != GRID_HOP && a.kind != GRID_WILSON)) return false;
    if (a.prec != GRID_F16S && a.prec != GRID_F32) return false;
    if (a.g.L[0] % kTX || a.g.L[1] % kTY || a.g.L[2] % tile_z(a) || !offsets32(a.g.vol / a.g.L[3], 288)) return false;
    if (a.prec == GRID_F16S) {
        const double per_cu = static_cast<double>(a.g.vol) / (kTX * kTY * kTZ<SpF16S> * 256.0);
        const bool third_round =
            (per_cu > 2.0 && per_cu < 2.83) || (per_cu > 4.0 && per_cu < 5.0 && a.g.vol / a.g.L[3] <= 15000);
        return a.link_fmt == GRID_L18 || !third_round;
    }
    if (a.g.n5 < 500000) return false;
    double share;
    tile_dev(a, &share);
    return share >= (a.link_fmt == GRID_L12 ? 0.70 : 0.78);
}

long tile_blocks(const DhopArgs &a) {
    const TileDev td = tile_dev(a);
    return static_cast<long>(td.ntx) * td.nty * td.ntz * td.nseg;
}

template <class SP, class LK>
static hipError_t launch_tile_t(const DhopArgs &a) {
    const TileDev td = tile_dev(a);
    const dim3 grid(static_cast<unsigned>(tile_blocks(a))), block(kTX * kTY * kTZ<SP>);
    hipStream_t st = a.stream;
#define GRIDMI_LAUNCH(DAG, KIND, FUSE)                                                                          \
    hipLaunchKernelGGL((k_dhop_tile<SP, LK, DAG, KIND, FUSE, kTX, kTY, kTZ<SP>>), grid, block, 0, st, a.U, a.psi,      \
                       a.psi_scale, a.out, a.out_scale, a.g, td, a.diag, a.fz)
    if (a.fuse != kFuseNone) {
        switch (a.kind * 4 + a.fuse * 2 + (a.dag ? 1 : 0)) {
            case GRID_WILSON * 4 + kFuseNorm * 2 + 0: GRIDMI_LAUNCH(false, GRID_WILSON, kFuseNorm); break;
            case GRID_WILSON * 4 + kFuseAxpy * 2 + 1: GRIDMI_LAUNCH(true, GRID_WILSON, kFuseAxpy); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (a.kind * 2 + (a.dag ? 1 : 0)) {
        case GRID_HOP * 2 + 0: GRIDMI_LAUNCH(false, GRID_HOP, kFuseNone); break;
        case GRID_HOP * 2 + 1: GRIDMI_LAUNCH(true, GRID_HOP, kFuseNone); break;
        case GRID_WILSON * 2 + 0: GRIDMI_LAUNCH(false, GRID_WILSON, kFuseNone); break;
        case GRID_WILSON * 2 + 1: GRIDMI_LAUNCH(true, GRID_WILSON, kFuseNone); break;
        default: return hipErrorInvalidValue;
    }
#undef GRIDMI_LAUNCH
    return hipGetLastError();
}

hipError_t launch_tile(const DhopArgs &a) {
    switch (a.prec * 2 + a.link_fmt) {
        case GRID_F32 * 2 + GRID_L18: return launch_tile_t<SpF32, LkF32<3>>(a);
        case GRID_F32 * 2 + GRID_L12: return launch_tile_t<SpF32, LkF32<2>>(a);
        case GRID_F16S * 2 + GRID_L18: return launch_tile_t<SpF16S, LkF16<3>>(a);
        case GRID_F16S * 2 + GRID_L12: return launch_tile_t<SpF16S, LkF16<2>>(a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace gridmi
