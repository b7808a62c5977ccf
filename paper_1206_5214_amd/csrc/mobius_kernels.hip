// mobius_kernels.hip -- HIP kernels for gfx950 (MI355X) of the red/black
// Moebius domain-wall operator (Brower, Neff, Orginos, Sec. 3 and Sec. 4.1).
//
// Thread mapping of the site kernels: one lane per (4d site, s).  A 64-lane
// wavefront holds floor(64 / Ls) whole 4d sites, their Ls slices in
// consecutive lanes, so that
//  * every lane of a site reads the same eight links (one cache line serves
//    all Ls lanes: the links are read from HBM once per 4d site and reused
//    across the fifth dimension),
//  * the b5/c5 coupling between s-1, s, s+1 (the "vector gather" of Sec. 4.1)
//    is a cross-lane shuffle inside the wavefront,
//  * the Ls-direction solves I^-1 (closed-form elimination, Sec. 3) run in the
//    same wavefront through LDS, one lane per colour-spin component.
// Packed layouts are described in mobius_internal.h.
#include "mobius_device.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <mutex>

namespace mobius {
namespace {

int sites_per_wave(int Ls) { return 64 / Ls; }

// most workgroups of a launch in the y direction
[[maybe_unused]] constexpr int MAX_GRID_Y = 65535;

// dynamic LDS of one block for the staged links: [8][sites per block][record]
template <int P>
size_t link_lds_bytes(int spw, bool rows)
{
    // FP16: the dot2 operand form, or the matrix-core rows (pf 3)
    return (size_t)8 * WAVES * spw * (P == MOBIUS_F16 ? (rows ? LINKROW_REC : LINKH2_REC) : Link<P>::REC);
}

// ---------------------------------------------------------------------------
// hop kernel: out = epilogue( -1/2 sum_mu [...] )  on every s-slice


// Order in which a lane visits its eight directions (index d of the neighbour
// and link records: 0..3 forward x, y, z, t; 4..7 backward).  A neighbour
// spinor is read by eight sites; the reader one t-slice earlier starts a slice
// time before the readers in the spinor's own slice, the one a t-slice later a
// slice time after them.  With t- first and t+ last the reads fall close
// together, while the line is still in the XCD's L2 (at 24^3 x 64, Ls = 12 the
// L2 turns over about every 5 us and a wavefront lives 10 to 19 us): the FP64
// hop reads 3.04 GB from memory instead of 4.48.  The pairs -mu, +mu in between
// are close because the two reads of one wavefront overlap in the L1.
// Against x+ y+ z+ t+ x- y- z- t-, D_pre and D_pre^+ there: FP64 2090 and 2265
// to 2010 and 2215 us, FP16 600 and 650 to 565 and 607 us; FP64 hop at
// 16^3 x 32, Ls = 16: 160 to 147 us (the reverse order: 166 us).  The order in
// between (y- y+ z- z+ or z- z+ y- y+ in pairs, or as here) is within 0.5 %.
// Lattices whose fields stay in the caches gain nothing: D_pre and D_pre^+ there are
// equal to 2 %, a hop by itself 2 to 7 % slower in FP32 and FP16 (16^3 x 32, Ls = 5,
// FP16 adjoint hop 17.9 to 19.2 us; 16^4, Ls = 8, FP32 left form 18.4 to 19.5 us).
__device__ constexpr int HOP_DIR[8] = {7, 4, 0, 5, 6, 1, 2, 3};

// What follows the hopping sum r = -1/2 H (B in) at one lane (Epilogue): the
// s-direction operators, x - r, the norm and the store.  WAVE_ONLY: this
// wavefront runs it by itself (its I^-1 buffer is the first of the workgroup's).
// lds_shared: the I^-1 buffer overlays LDS that the other wavefronts may still
// read.
template <int P, bool DAG, int EPI, bool WAVE_ONLY>
__device__ __forceinline__ void hop_epilogue(const HopParams &hp, const SiteMap &m,
                                             cx<typename Spin<P>::T> acc[12], int r, int64_t lb, int m5_off,
                                             bool lds_shared)
{
    using S = Spin<P>;
    using T = typename S::T;
    extern __shared__ u32x4 dyn_lds[];
    const int Ls = hp.Ls;
    const uint32_t i5 = (uint32_t)m.i, s5 = (uint32_t)m.s;
    const Lay lay{(uint32_t)Ls, (uint32_t)hp.N5};
    const int64_t fbytes = S::bytes(hp.N5);
    const Buf bout(hp.out + r * hp.fstride, fbytes);
    const char *xr = hp.x ? hp.x + r * hp.fstride : nullptr;
    const char *yr = hp.y ? hp.y + r * hp.fstride : nullptr;
    // coefficients of the epilogue, converted here so that none of them is
    // held in a register across the direction loop
    const Coef<T> k = make_coef<T>(hp.c);
    if constexpr (DAG && (EPI & EPI_NOBOUT) == 0) {  // B^+ on the output
        if (!k.ls)
            mix_s(acc, k.b5, k.c5, k.mf, m, Ls, true);
        else
            mix_s(acc, mix_w(k, false, m, Ls, true), k.mf, m, Ls, true);
    }
    if constexpr ((EPI & EPI_M5ADD) != 0) {
        cx<T> yv[12];
        S::load(Buf(yr, fbytes), lay, i5, s5, yv);
        mix_s(yv, mix_w(k, true, m, Ls, DAG), k.mf, m, Ls, DAG);  // I y = M+ y + M- C5 y
        // (I y rounded before the sum in every variant, which contracting the
        // products into it would leave to the compiler)
#pragma unroll
        for (int c = 0; c < 12; ++c) pin(yv[c]);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = acc[c] + yv[c];
    }
    if constexpr ((EPI & EPI_M5SUB) != 0) {
        cx<T> yv[12];
        S::load(Buf(yr, fbytes), lay, i5, s5, yv);
        mix_s(yv, mix_w(k, true, m, Ls, DAG), k.mf, m, Ls, DAG);  // I y (I^+ y)
#pragma unroll
        for (int c = 0; c < 12; ++c) pin(yv[c]);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = yv[c] - acc[c];
    }
    if constexpr ((EPI & EPI_PRESUB) != 0) {
        cx<T> xv[12];
        S::load(Buf(xr, fbytes), lay, i5, s5, xv);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = xv[c] - acc[c];
    }
    if constexpr ((EPI & EPI_M5INV) != 0) {
        // the buffer lives in the dynamic LDS; where it overlays the staged
        // links, every wave of the block must be past its direction loop
        if (!WAVE_ONLY && lds_shared) __syncthreads();
        M5Lds<T> &lds = *reinterpret_cast<M5Lds<T> *>(reinterpret_cast<char *>(dyn_lds) + m5_off);
        m5inv_lanes<WAVE_ONLY>(acc, k, m, Ls, DAG, lds);
    }
    if constexpr ((EPI & EPI_BMIX) != 0)  // B r (B^+ r in the adjoint hop)
        mix_s(acc, mix_w(k, false, m, Ls, DAG), k.mf, m, Ls, DAG);
    if constexpr ((EPI & EPI_POSTSUB) != 0) {
        cx<T> xv[12];
        S::load(Buf(xr, fbytes), lay, i5, s5, xv);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = xv[c] - acc[c];
    }
    if constexpr ((EPI & EPI_NORM) != 0) {
        // |stored value|^2, from the encoded registers
        double n = 0;
        if (m.site_ok) n = S::store_norm2(bout, lay, i5, s5, acc);
        if constexpr (WAVE_ONLY) {
            n = wave_sum(n);
            if (m.lane == 0) hp.partials[r * hp.pstride + lb] = n;
        } else {
            block_sum_store(n, hp.partials + r * hp.pstride, lb);
        }
    } else {
        if (m.site_ok) S::store(bout, lay, i5, s5, acc);
    }
}

// PF: software pipelining of the direction loop.  0: operands of direction d
// are loaded in segment d; 1: the neighbour spinor of direction d+1 is loaded
// while direction d computes; 2: its link as well.  The eight neighbour
// indices are always loaded up front.
// The block takes the right-hand sides r0, r0 + rstep, ... (one staging of the
// links for all of them).
template <int P, bool DAG, int EPI, int PF>
__device__ __forceinline__ void hop_block(const HopParams &hp, int64_t lb, int r0, int rstep)
{
    using S = Spin<P>;
    using T = typename S::T;
    const SiteMap m = site_map_lb(hp.Ls, hp.spw, hp.Vh, lb);
    const Coef<T> k = make_coef<T>(hp.c);
    const int Ls = hp.Ls;
    const uint32_t Vh = (uint32_t)hp.Vh;
    const uint32_t i = (uint32_t)m.i, s5 = (uint32_t)m.s;
    const Lay lay{(uint32_t)Ls, (uint32_t)hp.N5};
    const int64_t fbytes = S::bytes(hp.N5);
    const Buf blink(hp.links, (int64_t)8 * hp.Vh * Link<P>::REC);
    const Buf bnbr(hp.nbr, 8 * hp.Vh * 4);

    if (hp.active) {  // a system group whose systems have all converged: nothing to stage
        bool any = false;
        for (int r = r0; r < hp.nrhs; r += rstep) any = any || hp.active[r];
        if (!any) return;
    }

    extern __shared__ u32x4 dyn_lds[];
    LinkSource<P> ls;
    ls.glob = &blink;
    ls.lds = nullptr;
    ls.Vh = Vh;
    ls.i = i;
    ls.sites_blk = (uint32_t)(WAVES * hp.spw);
    // lanes without a site (idle tail lanes of a wavefront) read record 0
    ls.sib = m.site_ok ? (uint32_t)(m.wave * hp.spw + m.g) : 0u;
    if (hp.stage_links && P == MOBIUS_F16) {
        // one thread per (direction, site): the record expanded to the dot2 operand form
        constexpr uint32_t REC = Link<P>::REC;
        const uint32_t i0 = (uint32_t)(lb * WAVES * hp.spw);
        const uint32_t nsites = min(ls.sites_blk, Vh - i0);
        for (uint32_t c = threadIdx.x; c < 8u * nsites; c += BLOCK) {
            const uint32_t d = c / nsites, j = c - d * nsites;
            u32x4 q[3];
#pragma unroll
            for (int w = 0; w < 3; ++w)
                q[w] = hp.nt ? blink.ld16_nt((i0 + j) * REC + 16u * w, d * Vh * REC)
                             : blink.ld16((i0 + j) * REC + 16u * w, d * Vh * REC);
            half2v u[9];
            Link<MOBIUS_F16>::raw_from_words(q, u);
            constexpr uint32_t W = (PF == 3 ? LINKROW_REC : LINKH2_REC) / 16;
            u32x4 *dst = dyn_lds + (size_t)(d * ls.sites_blk + j) * W;
            if (d < 4)
                stage_link_f16<true, PF == 3>(u, dst);
            else
                stage_link_f16<false, PF == 3>(u, dst);
        }
        ls.lds = reinterpret_cast<const char *>(dyn_lds);
    } else if (hp.stage_links) {
        constexpr uint32_t REC = Link<P>::REC;
        const uint32_t i0 = (uint32_t)(lb * WAVES * hp.spw);
        const uint32_t nsites = min(ls.sites_blk, Vh - i0);
        const uint32_t cpd = nsites * REC / 16u;  // 16-byte words per direction
        for (uint32_t c = threadIdx.x; c < 8u * cpd; c += BLOCK) {
            const uint32_t d = c / cpd, q = c - d * cpd;
            const u32x4 v = hp.nt ? blink.ld16_nt(i0 * REC + q * 16u, d * Vh * REC)
                                  : blink.ld16(i0 * REC + q * 16u, d * Vh * REC);
            dyn_lds[(d * ls.sites_blk * REC) / 16u + q] = v;
        }
        ls.lds = reinterpret_cast<const char *>(dyn_lds);
    }

    uint32_t jn[8];
    {
        const u32x4 n0 = bnbr.ld16(i * 32u, 0u), n1 = bnbr.ld16(i * 32u + 16u, 0u);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            jn[d] = n0[d];
            jn[4 + d] = n1[d];
        }
    }

    if (hp.stage_links) __syncthreads();

    for (int r = r0; r < hp.nrhs; r += rstep) {
    if (hp.active && !hp.active[r]) continue;
    const Buf bin(hp.in + r * hp.fstride, fbytes);

    cx<T> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = {0, 0};
    // B = b5 + c5 C5 applied to the neighbours here (forward hop), unless the
    // input already holds B in (written so by an EPI_BMIX epilogue)
    constexpr bool MIXIN = !DAG && (EPI & EPI_PREMIXED) == 0;

    // B weights of this lane (per-slice b5(s), c5(s) when the operator has them)
    const MixW<T> wB = mix_w(k, false, m, Ls, false);
    if constexpr (P == MOBIUS_F16) {
        // forward block: B mixing weights of this lane (norms folded in per direction)
        const float wu = MIXIN ? (float)wB.bu * (m.s == 0 ? -(float)k.mf : 1.f) : 0.f;
        const float wl = MIXIN ? (float)wB.bl * (m.s == Ls - 1 ? -(float)k.mf : 1.f) : 0.f;
        // PF 3: the colour multiply on the matrix cores, links and neighbour
        // spinors prefetched one direction ahead
        constexpr bool MF = PF == 3;
        const int quad = m.lane & 3;
        // (its spinors two directions ahead: the registers the colour
        // multiply frees hold one more direction in flight)
        RawH nx, nx2;
        LinkH2 unx;
        LinkRows rnx;
        load_raw_f16(bin, lay, jn[HOP_DIR[0]], s5, nx);
        if constexpr (MF) {
            load_raw_f16(bin, lay, jn[HOP_DIR[1]], s5, nx2);
            ls.get_rows(HOP_DIR[0], quad, rnx);
        } else if constexpr (PF >= 2) {
            ls.template get_h2<(HOP_DIR[0] < 4)>(HOP_DIR[0], unx);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int d = HOP_DIR[q], d1 = HOP_DIR[q < 7 ? q + 1 : 7], d2 = HOP_DIR[q < 6 ? q + 2 : 7];
            const RawH o = nx;
            if constexpr (MF) {
                nx = nx2;
                if (q < 6) load_raw_f16(bin, lay, jn[d2], s5, nx2);
            } else {
                if (q < 7) load_raw_f16(bin, lay, jn[d1], s5, nx);
            }
            LinkH2 u;
            LinkRows ur;
            if constexpr (MF) {
                ur = rnx;
                if (q < 7) ls.get_rows(d1, quad, rnx);
            } else if constexpr (PF >= 2) {
                u = unx;
                if (q < 7 && d1 < 4)
                    ls.template get_h2<true>(d1, unx);
                else if (q < 7)
                    ls.template get_h2<false>(d1, unx);
            } else {
                if (d < 4)
                    ls.template get_h2<true>(d, u);
                else
                    ls.template get_h2<false>(d, u);
            }
            constexpr int SF = DAG ? +1 : -1;
            half2v hh[6];
#define MOBIUS_DIR(MU, SG)                                                                         \
    {                                                                                              \
        const float sc = half_spinor_f16<MU, SG, MIXIN>(o, (float)wB.a, wu, wl, m, hh);            \
        cx<float> w[2][3];                                                                         \
        if constexpr (MF)                                                                          \
            link_mult_mfma(hh, ur, w);                                                             \
        else                                                                                       \
            link_mult_h2(hh, u, w);                                                                \
        spin_accumulate_f16<MU, SG>(w, -0.5f * sc, acc);                                           \
    }                                                                                              \
    break
            switch (d) {
            case 0: MOBIUS_DIR(0, SF);
            case 1: MOBIUS_DIR(1, SF);
            case 2: MOBIUS_DIR(2, SF);
            case 3: MOBIUS_DIR(3, SF);
            case 4: MOBIUS_DIR(0, -SF);
            case 5: MOBIUS_DIR(1, -SF);
            case 6: MOBIUS_DIR(2, -SF);
            default: MOBIUS_DIR(3, -SF);
            }
#undef MOBIUS_DIR
#pragma unroll
            for (int c = 0; c < 12; ++c) pin(acc[c]);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
    cx<T> nxt[12], unx[9];
    if constexpr (PF >= 1) S::load(bin, lay, jn[HOP_DIR[0]], s5, nxt);
    if constexpr (PF >= 2) ls.get(HOP_DIR[0], unx);

#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int d = HOP_DIR[q], d1 = HOP_DIR[q < 7 ? q + 1 : 7];
        cx<T> chi[12], u[9];
        if constexpr (PF >= 1) {
#pragma unroll
            for (int c = 0; c < 12; ++c) chi[c] = nxt[c];
            if (q < 7) S::load(bin, lay, jn[d1], s5, nxt);
        } else {
            S::load(bin, lay, jn[d], s5, chi);
        }
        if constexpr (PF >= 2) {
#pragma unroll
            for (int e = 0; e < 9; ++e) u[e] = unx[e];
            if (q < 7) ls.get(d1, unx);
        } else {
            ls.get(d, u);
        }
        if constexpr (MIXIN) {
            // B = b5 + c5 C5 on the input: gather s-1, s, s+1 of the neighbour
            mix_s(chi, wB, k.mf, m, Ls, false);
        }
        constexpr int SF = DAG ? +1 : -1;  // forward projector (1 -+ g_mu)
        switch (d) {
        case 0: hop_dir<P, 0, true, SF>(chi, u, acc); break;
        case 1: hop_dir<P, 1, true, SF>(chi, u, acc); break;
        case 2: hop_dir<P, 2, true, SF>(chi, u, acc); break;
        case 3: hop_dir<P, 3, true, SF>(chi, u, acc); break;
        case 4: hop_dir<P, 0, false, -SF>(chi, u, acc); break;
        case 5: hop_dir<P, 1, false, -SF>(chi, u, acc); break;
        case 6: hop_dir<P, 2, false, -SF>(chi, u, acc); break;
        default: hop_dir<P, 3, false, -SF>(chi, u, acc); break;
        }
        // the accumulator is complete here; nothing of direction d+1 beyond
        // its prefetched loads moves above this point
#pragma unroll
        for (int c = 0; c < 12; ++c) pin(acc[c]);
        __builtin_amdgcn_sched_barrier(0);
    }
    }
    // the -1/2 of the hopping term (the FP16 loop folds it into each
    // direction's scale, a power of two, so the result is the same)
    if constexpr (P != MOBIUS_F16) {
        const T mhalf = (T)-0.5;
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = mhalf * acc[c];
    }

    hop_epilogue<P, DAG, EPI, false>(hp, m, acc, r, lb, hp.m5_off, hp.m5_off == 0 && hp.stage_links);
    }  // rhs
}

// The hop with its directions split over the four wavefronts of a workgroup
// (PF 4): small lattices, where a hop lasts as long as one wavefront's chain
// of eight directions.  Every wavefront of block lb covers the same 64 / Ls
// sites; wavefront w forms the colour products of directions HOP_DIR[2w] and
// [2w + 1] (both neighbours and links loaded before either is used), hands them
// over in LDS, and the first one adds all eight in the order of the unsplit
// loop -- the same bits -- and runs the epilogue.

// LDS of one wavefront: first its staged FP16 link rows, then its products
template <int P>
constexpr int split_lds_wave(int spw)
{
    // 12 products and (FP16) two scales per lane; 2 spw link records
    const int prod = 64 * (12 * (int)sizeof(cx<typename Spin<P>::T>) + (P == MOBIUS_F16 ? 8 : 0));
    const int rows = P == MOBIUS_F16 ? 2 * spw * LINKROW_REC : 0;
    return prod > rows ? prod : rows;
}

// colour products w and scales sc (FP16) of directions HOP_DIR[2 PART] and [2 PART + 1]
template <int P, bool DAG, int EPI, int PART>
__device__ __forceinline__ void hop_two_dirs(const HopParams &hp, const SiteMap &m, int r, char *lds,
                                             cx<typename Spin<P>::T> w[2][2][3], float sc[2])
{
    using S = Spin<P>;
    using T = typename S::T;
    constexpr int D0 = HOP_DIR[2 * PART], D1 = HOP_DIR[2 * PART + 1];
    constexpr int SF = DAG ? +1 : -1;  // forward projector (1 -+ g_mu)
    constexpr int S0 = D0 < 4 ? SF : -SF, S1 = D1 < 4 ? SF : -SF;
    constexpr bool MIXIN = !DAG && (EPI & EPI_PREMIXED) == 0;
    const int Ls = hp.Ls;
    const uint32_t Vh = (uint32_t)hp.Vh, i = (uint32_t)m.i, s5 = (uint32_t)m.s;
    const Lay lay{(uint32_t)Ls, (uint32_t)hp.N5};
    const Buf bnbr(hp.nbr, 8 * hp.Vh * 4), blink(hp.links, (int64_t)8 * hp.Vh * Link<P>::REC);
    const Buf bin(hp.in + r * hp.fstride, S::bytes(hp.N5));
    const uint32_t j0 = bnbr.ld4(i * 32u + 4u * D0, 0u);
    const uint32_t j1 = bnbr.ld4(i * 32u + 4u * D1, 0u);
    const Coef<T> k = make_coef<T>(hp.c);
    const MixW<T> wB = mix_w(k, false, m, Ls, false);
    if constexpr (P == MOBIUS_F16) {
        // the unsplit loop's choice: matrix cores where whole 4-lane groups share a site
        const bool mf = hp.split_mfma;
        constexpr uint32_t REC = Link<P>::REC;
        LinkH2 u0, u1;
        if (mf) {  // one lane per link record
            const uint32_t spw = (uint32_t)hp.spw, i0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)i);
            const uint32_t lane = (uint32_t)m.lane, dd = lane / spw, j = lane - dd * spw;
            if (dd < 2 && i0 + j < Vh) {
                half2v u[9];
                u32x4 *dst = reinterpret_cast<u32x4 *>(lds + lane * LINKROW_REC);
                Link<P>::raw_load(blink, (i0 + j) * REC + (dd ? D1 : D0) * Vh * REC, 0u, u);
                if (dd == 0)
                    stage_link_f16<(D0 < 4), true>(u, dst);
                else
                    stage_link_f16<(D1 < 4), true>(u, dst);
            }
        } else {
            const LinkSource<P> ls{&blink, nullptr, Vh, i, 0u, 0u};
            ls.template get_h2<(D0 < 4)>(D0, u0);
            ls.template get_h2<(D1 < 4)>(D1, u1);
        }
        RawH o0, o1;
        load_raw_f16(bin, lay, j0, s5, o0);
        load_raw_f16(bin, lay, j1, s5, o1);
        const float wu = MIXIN ? (float)wB.bu * (m.s == 0 ? -(float)k.mf : 1.f) : 0.f;
        const float wl = MIXIN ? (float)wB.bl * (m.s == Ls - 1 ? -(float)k.mf : 1.f) : 0.f;
        half2v h0[6], h1[6];
        sc[0] = half_spinor_f16<(D0 & 3), S0, MIXIN>(o0, (float)wB.a, wu, wl, m, h0);
        sc[1] = half_spinor_f16<(D1 & 3), S1, MIXIN>(o1, (float)wB.a, wu, wl, m, h1);
        if (mf) {
            lds_sync<true>();
            LinkSource<P> ls{&blink, lds, Vh, i, m.site_ok ? (uint32_t)m.g : 0u, (uint32_t)hp.spw};
            LinkRows x;
            ls.get_rows(0, m.lane & 3, x);
            link_mult_mfma(h0, x, w[0]);
            ls.get_rows(1, m.lane & 3, x);
            link_mult_mfma(h1, x, w[1]);
            lds_sync<true>();  // (the products take the rows' place)
        } else {
            link_mult_h2(h0, u0, w[0]);
            link_mult_h2(h1, u1, w[1]);
        }
    } else {
        cx<T> c0[12], c1[12], u0[9], u1[9];
        load_link<P>(blink, Vh, D0, i, u0);
        load_link<P>(blink, Vh, D1, i, u1);
        S::load(bin, lay, j0, s5, c0);
        S::load(bin, lay, j1, s5, c1);
        if constexpr (MIXIN) mix_s(c0, wB, k.mf, m, Ls, false);
        hop_dir_w<P, (D0 & 3), (D0 < 4), S0>(c0, u0, w[0]);
        if constexpr (MIXIN) mix_s(c1, wB, k.mf, m, Ls, false);
        hop_dir_w<P, (D1 & 3), (D1 < 4), S1>(c1, u1, w[1]);
    }
}

// acc += the products of direction D
template <int P, bool DAG, int D>
__device__ __forceinline__ void split_accumulate(const cx<typename Spin<P>::T> w[2][3], float sc,
                                                 cx<typename Spin<P>::T> acc[12])
{
    constexpr int SF = DAG ? +1 : -1, SG = D < 4 ? SF : -SF;
    if constexpr (P == MOBIUS_F16)
        spin_accumulate_f16<(D & 3), SG>(w, -0.5f * sc, acc);
    else
        spin_accumulate<typename Spin<P>::T, (D & 3), SG>(w, acc);
}

template <int P, bool DAG, int EPI>
__device__ __forceinline__ void hop_split(const HopParams &hp, int64_t lb, int r)
{
    using T = typename Spin<P>::T;
    if (hp.active && !hp.active[r]) return;
    const SiteMap m = site_map_first(hp.Ls, hp.spw, hp.Vh, lb * hp.spw);
    extern __shared__ u32x4 dyn_lds[];
    const int stride = split_lds_wave<P>(hp.spw);
    const int wv = __builtin_amdgcn_readfirstlane(m.wave);
    char *mine = reinterpret_cast<char *>(dyn_lds) + wv * stride;
    cx<T> w[2][2][3];
    float sc[2] = {0.f, 0.f};
    switch (wv) {
    case 0: hop_two_dirs<P, DAG, EPI, 0>(hp, m, r, mine, w, sc); break;
    case 1: hop_two_dirs<P, DAG, EPI, 1>(hp, m, r, mine, w, sc); break;
    case 2: hop_two_dirs<P, DAG, EPI, 2>(hp, m, r, mine, w, sc); break;
    default: hop_two_dirs<P, DAG, EPI, 3>(hp, m, r, mine, w, sc); break;
    }
    if (wv > 0) {
        cx<T> *p = reinterpret_cast<cx<T> *>(mine);
#pragma unroll
        for (int e = 0; e < 12; ++e) p[e * 64 + m.lane] = w[e / 6][(e / 3) % 2][e % 3];
        if constexpr (P == MOBIUS_F16) {
            float *q = reinterpret_cast<float *>(p + 12 * 64);
            q[m.lane] = sc[0];
            q[64 + m.lane] = sc[1];
        }
    }
    __syncthreads();
    if (wv > 0) return;
    cx<T> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = {0, 0};
    split_accumulate<P, DAG, HOP_DIR[0]>(w[0], sc[0], acc);
    split_accumulate<P, DAG, HOP_DIR[1]>(w[1], sc[1], acc);
#define MOBIUS_PART(Q)                                                                             \
    {                                                                                              \
        const cx<T> *p = reinterpret_cast<const cx<T> *>(reinterpret_cast<const char *>(dyn_lds) + (Q) * stride); \
        _Pragma("unroll") for (int e = 0; e < 12; ++e) w[e / 6][(e / 3) % 2][e % 3] = p[e * 64 + m.lane]; \
        if constexpr (P == MOBIUS_F16) {                                                           \
            const float *q = reinterpret_cast<const float *>(p + 12 * 64);                         \
            sc[0] = q[m.lane];                                                                     \
            sc[1] = q[64 + m.lane];                                                                \
        }                                                                                          \
        split_accumulate<P, DAG, HOP_DIR[2 * (Q)]>(w[0], sc[0], acc);                              \
        split_accumulate<P, DAG, HOP_DIR[2 * (Q) + 1]>(w[1], sc[1], acc);                          \
    }
    MOBIUS_PART(1)
    MOBIUS_PART(2)
    MOBIUS_PART(3)
#undef MOBIUS_PART
    // rounded here as in the loop: the last FP16 product must not be contracted into
    // the epilogue's subtraction.  FP64, whose bits do not depend on it: the epilogues
    // that mix a second field in s need fewer registers (D_DW on 8^3 x 16, Ls = 8, 26.6
    // to 17.3 us), the others are up to 5 % slower.
    if constexpr (P != MOBIUS_F64 || (EPI & (EPI_M5ADD | EPI_M5SUB)) != 0) {
#pragma unroll
        for (int c = 0; c < 12; ++c) pin(acc[c]);
    }
    if constexpr (P != MOBIUS_F16) {
        const T mhalf = (T)-0.5;
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = mhalf * acc[c];
    }
    lds_sync<true>();
    hop_epilogue<P, DAG, EPI, true>(hp, m, acc, r, lb, 0, false);
}

// Wavefronts per SIMD a hop kernel is held to.  The binary16 matrix-core loop
// to four (128 VGPRs): its adjoint hop with the I^-+ epilogue needs 130 on its
// own and then runs three (the cap costs it one spilled dword pair; the FP16
// solve runs about 1 % faster).  FP32: four without a prefetched neighbour
// (D_pre at 24^3 x 64, Ls = 12: 900 to 877 us), three with one (its mixing hops
// with an epilogue need 172 and would run two: 955 to 905 us, 20 spilled bytes).
// The FP64 hop spills under a three-wave cap and keeps two (821 against 923 us).
constexpr int hop_waves(int P, int PF)
{
    return P == MOBIUS_F16 && PF == 3 ? 4 : P == MOBIUS_F32 && PF < 3 ? (PF == 0 ? 4 : 3) : 1;
}

template <int P, bool DAG, int EPI, int PF>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(hop_waves(P, PF))))
void hop_kernel(HopParams hp)
{
    if constexpr (PF == 4) {
        // (the grid has a row per right-hand side, so one pass; written as a loop it
        // compiles to fewer instructions: D_pre at 4^4, FP16, 12.0 against 12.6 us)
        for (int r = blockIdx.y; r < hp.nrhs; r += gridDim.y) {
            hop_split<P, DAG, EPI>(hp, logical_block(hp.remap), r);
            if (r + (int)gridDim.y < hp.nrhs) __syncthreads();
        }
    } else {
        hop_block<P, DAG, EPI, PF>(hp, logical_block(hp.remap), blockIdx.y, gridDim.y);
    }
}

// Persistent launch over a batch of lattices of uneven size: a fixed grid
// walks the concatenated block lists of all groups (group j owns work items
// [prefix[j], prefix[j+1]), its site blocks once per split right-hand side); every
// workgroup exits after its last item.
template <int P, bool DAG, int EPI, int PF>
__global__ __launch_bounds__(BLOCK) void hop_batch_kernel(const HopParams *groups, int ngroups,
                                                          const int64_t *prefix)
{
    const int64_t total = prefix[ngroups];
    int j = 0;
    // XCD-contiguous order (as the single-lattice launch with remap on) over
    // the n = min(grid, items) workgroups that have work, so that every XCD
    // takes an eighth of the items and each its own contiguous range
    const int64_t n = total < (int64_t)gridDim.x ? total : (int64_t)gridDim.x;
    const int64_t b = blockIdx.x;
    if (b >= n) return;
    const int64_t q = n / NUM_XCD, rem = n % NUM_XCD, x = b % NUM_XCD;
    for (int64_t w = x * q + (x < rem ? x : rem) + b / NUM_XCD; w < total; w += n) {
        while (w >= prefix[j + 1]) ++j;
        const HopParams &hp = groups[j];
        const int64_t i = w - prefix[j], r0 = i / hp.nblocks;
        hop_block<P, DAG, EPI, PF>(hp, i - r0 * hp.nblocks, (int)r0, hp.split);
        __syncthreads();  // LDS of this item is dead before the next item stages
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launch of the hop kernels.  Their instantiations are most of this file's
// compile time, so each storage precision, single and batched launch is a
// compilation unit of its own (MOBIUS_HOP_PREC, MOBIUS_HOP_BATCH; build.py),
// reached through run_hop<P> and run_hop_batch<P>.
#ifdef MOBIUS_HOP_PREC
namespace {

template <int P, bool DAG, int EPI>
void hop_launch(const HopParams &hp0, hipStream_t st)
{
    HopParams hp = hp0;
    const size_t links = hp.stage_links ? link_lds_bytes<P>(hp.spw, hp.pf == 3) : 0;
    const int split = std::min(hp.split, MAX_GRID_Y);
    size_t dyn = links;
    if constexpr ((EPI & EPI_M5INV) != 0) {
        hp.m5_off = split < hp.nrhs ? (int)links : 0;
        dyn = std::max(links, (size_t)hp.m5_off + sizeof(M5Lds<typename Spin<P>::T>));
    }
    // split directions: each wavefront's products; the one I^-1 buffer in use goes over them
    if (hp.pf == 4) dyn = (size_t)WAVES * split_lds_wave<P>(hp.spw);
    const dim3 grid((unsigned)hp.nblocks, (unsigned)split), blk(BLOCK);
    switch (hp.pf) {
    case 0: hipLaunchKernelGGL((hop_kernel<P, DAG, EPI, 0>), grid, blk, dyn, st, hp); break;
    case 1: hipLaunchKernelGGL((hop_kernel<P, DAG, EPI, 1>), grid, blk, dyn, st, hp); break;
    case 4: hipLaunchKernelGGL((hop_kernel<P, DAG, EPI, 4>), grid, blk, dyn, st, hp); break;
    case 3:
        if constexpr (P == MOBIUS_F16) {
            hipLaunchKernelGGL((hop_kernel<P, DAG, EPI, 3>), grid, blk, dyn, st, hp);
            break;
        }
        [[fallthrough]];
    default: hipLaunchKernelGGL((hop_kernel<P, DAG, EPI, 2>), grid, blk, dyn, st, hp); break;
    }
}

template <int P, bool DAG, int EPI>
void hop_batch_launch(const HopParams *groups, int n, const int64_t *prefix, size_t dyn, int grid,
                      int pf, hipStream_t st)
{
    switch (pf) {
    case 0: hipLaunchKernelGGL((hop_batch_kernel<P, DAG, EPI, 0>), dim3(grid), dim3(BLOCK), dyn, st, groups, n, prefix); break;
    case 1: hipLaunchKernelGGL((hop_batch_kernel<P, DAG, EPI, 1>), dim3(grid), dim3(BLOCK), dyn, st, groups, n, prefix); break;
    case 3:
        if constexpr (P == MOBIUS_F16) {
            hipLaunchKernelGGL((hop_batch_kernel<P, DAG, EPI, 3>), dim3(grid), dim3(BLOCK), dyn, st, groups, n, prefix);
            break;
        }
        [[fallthrough]];
    default: hipLaunchKernelGGL((hop_batch_kernel<P, DAG, EPI, 2>), dim3(grid), dim3(BLOCK), dyn, st, groups, n, prefix); break;
    }
}

// Calls F<P, DAG, EPI>() for the runtime (dag, epi); false if unsupported.
template <int P, template <int, bool, int> class F, class... A>
bool dispatch_hop(int dag, int epi, A &&...args)
{
#define MOBIUS_EPI_CASES(P, D)                                                                     \
    switch (epi) {                                                                                 \
    case 0: F<P, D, 0>::run(args...); return true;                                                 \
    case EPI_M5INV: F<P, D, EPI_M5INV>::run(args...); return true;                                 \
    case EPI_M5INV | EPI_POSTSUB: F<P, D, EPI_M5INV | EPI_POSTSUB>::run(args...); return true;     \
    case EPI_POSTSUB: F<P, D, EPI_POSTSUB>::run(args...); return true;                             \
    case EPI_M5INV | EPI_POSTSUB | EPI_NORM:                                                       \
        F<P, D, EPI_M5INV | EPI_POSTSUB | EPI_NORM>::run(args...);                                 \
        return true;                                                                               \
    case EPI_PRESUB | EPI_M5INV: F<P, D, EPI_PRESUB | EPI_M5INV>::run(args...); return true;       \
    case EPI_POSTSUB | EPI_NORM: F<P, D, EPI_POSTSUB | EPI_NORM>::run(args...); return true;       \
    case EPI_M5ADD: F<P, D, EPI_M5ADD>::run(args...); return true;                                 \
    case EPI_M5ADD | EPI_PRESUB: F<P, D, EPI_M5ADD | EPI_PRESUB>::run(args...); return true;       \
    case EPI_M5ADD | EPI_PRESUB | EPI_NORM:                                                        \
        F<P, D, EPI_M5ADD | EPI_PRESUB | EPI_NORM>::run(args...);                                  \
        return true;                                                                               \
    case EPI_M5INV | EPI_BMIX:                                                                     \
        if constexpr (!D) F<P, D, EPI_M5INV | EPI_BMIX>::run(args...);                             \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_M5INV | EPI_POSTSUB | EPI_NORM:                                        \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_M5INV | EPI_POSTSUB | EPI_NORM>::run(args...); \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_M5INV | EPI_POSTSUB:                                                   \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_M5INV | EPI_POSTSUB>::run(args...);           \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_POSTSUB | EPI_NORM:                                                    \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_POSTSUB | EPI_NORM>::run(args...);            \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_POSTSUB:                                                               \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_POSTSUB>::run(args...);                       \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_BMIX:                                                                  \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_BMIX>::run(args...);                          \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_M5INV | EPI_BMIX:                                                      \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_M5INV | EPI_BMIX>::run(args...);              \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_M5INV | EPI_BMIX | EPI_POSTSUB:                                        \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_M5INV | EPI_BMIX | EPI_POSTSUB>::run(args...); \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_M5INV | EPI_BMIX | EPI_POSTSUB | EPI_NORM:                             \
        if constexpr (!D)                                                                          \
            F<P, D, EPI_PREMIXED | EPI_M5INV | EPI_BMIX | EPI_POSTSUB | EPI_NORM>::run(args...);   \
        return !D;                                                                                 \
    case EPI_NOBOUT:                                                                               \
        if constexpr (D) F<P, D, EPI_NOBOUT>::run(args...);                                        \
        return D;                                                                                  \
    case EPI_PREMIXED | EPI_M5SUB:                                                                 \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_M5SUB>::run(args...);                         \
        return !D;                                                                                 \
    case EPI_PREMIXED | EPI_M5SUB | EPI_NORM:                                                      \
        if constexpr (!D) F<P, D, EPI_PREMIXED | EPI_M5SUB | EPI_NORM>::run(args...);              \
        return !D;                                                                                 \
    case EPI_M5SUB:                                                                                \
        if constexpr (D) F<P, D, EPI_M5SUB>::run(args...);                                         \
        return D;                                                                                  \
    case EPI_M5SUB | EPI_NORM:                                                                     \
        if constexpr (D) F<P, D, EPI_M5SUB | EPI_NORM>::run(args...);                              \
        return D;                                                                                  \
    case EPI_NOBOUT | EPI_M5INV | EPI_BMIX:                                                        \
        if constexpr (D) F<P, D, EPI_NOBOUT | EPI_M5INV | EPI_BMIX>::run(args...);                 \
        return D;                                                                                  \
    case EPI_NOBOUT | EPI_POSTSUB:                                                                 \
        if constexpr (D) F<P, D, EPI_NOBOUT | EPI_POSTSUB>::run(args...);                          \
        return D;                                                                                  \
    case EPI_NOBOUT | EPI_POSTSUB | EPI_NORM:                                                      \
        if constexpr (D) F<P, D, EPI_NOBOUT | EPI_POSTSUB | EPI_NORM>::run(args...);               \
        return D;                                                                                  \
    }                                                                                              \
    return false;
    if (dag) {
        MOBIUS_EPI_CASES(P, true)
    } else {
        MOBIUS_EPI_CASES(P, false)
    }
#undef MOBIUS_EPI_CASES
    return false;
}

template <int P, bool D, int E>
struct RunHop {
    static void run(const HopParams &hp, hipStream_t st) { hop_launch<P, D, E>(hp, st); }
};
template <int P, bool D, int E>
struct RunHopBatch {
    static void run(const HopParams *g, int n, const int64_t *prefix, size_t dyn, int grid, int pf,
                    hipStream_t st)
    {
        hop_batch_launch<P, D, E>(g, n, prefix, dyn, grid, pf, st);
    }
};

}  // namespace

#if MOBIUS_HOP_BATCH
template <>
bool run_hop_batch<MOBIUS_HOP_PREC>(int dag, int epi, const HopParams *groups, int n, const int64_t *prefix,
                                    size_t dyn, int grid, int pf, hipStream_t st)
{
    return dispatch_hop<MOBIUS_HOP_PREC, RunHopBatch>(dag, epi, groups, n, prefix, dyn, grid, pf, st);
}
#else
template <>
bool run_hop<MOBIUS_HOP_PREC>(int dag, int epi, const HopParams &hp, hipStream_t st)
{
    return dispatch_hop<MOBIUS_HOP_PREC, RunHop>(dag, epi, hp, st);
}
#endif

#else  // !MOBIUS_HOP_PREC: everything else

namespace {

// A wavefront's whole sites of a field in records (one stretch of memory) to and
// from the chunks of each lane's 5d site, through the wavefront's own LDS.  The
// s-direction operators only stream their field: where a site's chunk of Ls * 16
// bytes is no whole number of 128-byte lines (Ls = 4, 12, 20, 28), one access per
// chunk touches half lines, and the stores, which go past the caches, pay for them.
// Moved as one stretch, every access covers whole lines.  24^3 x 64, Ls = 12, I and
// I^-1: FP32 198 to 172 and 200 to 177 us, FP64 383 to 365 and 400 to 367 us;
// 24^3 x 32, Ls = 4: FP64 63.4 to 50.3 and 65.2 to 55.1 us.  With one site to a
// wavefront (Ls = 36) the pass through LDS costs I^-1 more than it gains (167 to
// 210 us): such sites, whole lines and small fields (m5_launch) are read and written
// directly.
template <int P>
struct RecordTile {
    using T = typename Spin<P>::T;
    static constexpr int CH = 12 * (int)sizeof(cx<T>) / 16;  // 16-byte chunks of a 5d site
    static constexpr int PER = 12 / CH;                      // components of a chunk
    struct Chunk { cx<T> v[PER]; };
    u32x4 *lds;                                              // 64 * CH of them
    uint32_t base, n;                                        // byte offset in the field, chunks
    __device__ __forceinline__ RecordTile(void *buf, const SiteMap &m, int Ls, int spw, int64_t Vh, int64_t lb)
        : lds(static_cast<u32x4 *>(buf))
    {
        const int64_t first = (lb * WAVES + m.wave) * spw, left = Vh - first;
        base = left > 0 ? (uint32_t)(first * Ls) * (CH * 16u) : 0u;
        n = left > 0 ? (uint32_t)((left < spw ? left : spw) * Ls * CH) : 0u;
    }
    // chunk c of this lane (a lane without a site reads the first site's)
    __device__ __forceinline__ uint32_t slot(const SiteMap &m, int Ls, int c) const
    {
        return (uint32_t)(((m.site_ok ? m.g : 0) * CH + c) * Ls + m.s);
    }
    __device__ __forceinline__ void load(const Buf &b, const SiteMap &m, int Ls, cx<T> v[12])
    {
        u32x4 t[CH];
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const uint32_t u = (uint32_t)j * 64u + (uint32_t)m.lane;
            t[j] = b.ld16(u < n ? base + u * 16u : base, 0u);
        }
#pragma unroll
        for (int j = 0; j < CH; ++j) lds[j * 64 + m.lane] = t[j];
        lds_sync<true>();
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const Chunk q = __builtin_bit_cast(Chunk, lds[slot(m, Ls, c)]);
#pragma unroll
            for (int e = 0; e < PER; ++e) v[c * PER + e] = q.v[e];
        }
        lds_sync<true>();
    }
    __device__ __forceinline__ void store(const Buf &b, const SiteMap &m, int Ls, const cx<T> v[12])
    {
        lds_sync<true>();
        if (m.site_ok) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                Chunk q;
#pragma unroll
                for (int e = 0; e < PER; ++e) q.v[e] = v[c * PER + e];
                lds[slot(m, Ls, c)] = __builtin_bit_cast(u32x4, q);
            }
        }
        lds_sync<true>();
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const uint32_t u = (uint32_t)j * 64u + (uint32_t)m.lane;
            if (u < n) b.st16(lds[u], base + u * 16u, 0u);
        }
    }
};

// per-site s-direction operators: kind 0 -> I (or I^+), kind 1 -> I^-1 (or I^-+).
// LINEAR: the field moves through RecordTile.
template <int P, bool DAG, int KIND, bool LINEAR>
__global__ __launch_bounds__(BLOCK) void m5_kernel(const char *in, char *out, int64_t Vh,
                                                   int64_t N5, int Ls, int spw, OpCoeffs c)
{
    using S = Spin<P>;
    using T = typename S::T;
    const SiteMap m = site_map(Ls, spw, Vh);
    const Coef<T> k = make_coef<T>(c);
    const int64_t fbytes = S::bytes(N5);
    const Lay lay{(uint32_t)Ls, (uint32_t)N5};
    __shared__ M5Lds<T> lds;
    cx<T> v[12];
    if constexpr (LINEAR)
        RecordTile<P>(lds.buf[m.wave], m, Ls, spw, Vh, logical_block(0))
            .load(Buf(in, fbytes), m, Ls, v);
    else
        S::load(Buf(in, fbytes), lay, (uint32_t)m.i, (uint32_t)m.s, v);
    if constexpr (KIND == 0)
        mix_s(v, mix_w(k, true, m, Ls, DAG), k.mf, m, Ls, DAG);
    else
        m5inv_lanes(v, k, m, Ls, DAG, lds);
    if constexpr (LINEAR)
        RecordTile<P>(lds.buf[m.wave], m, Ls, spw, Vh, logical_block(0))
            .store(Buf(out, fbytes), m, Ls, v);
    else if (m.site_ok)
        S::store(Buf(out, fbytes), lay, (uint32_t)m.i, (uint32_t)m.s, v);
}

// ---------------------------------------------------------------------------
// geometry, packing

__device__ __forceinline__ void coords_of(int64_t c, const int *L, int x[4])
{
    for (int mu = 0; mu < 4; ++mu) {
        x[mu] = (int)(c % L[mu]);
        c /= L[mu];
    }
}

__device__ __forceinline__ int64_t canon_index(const int x[4], const int *L)
{
    return (((int64_t)x[3] * L[2] + x[2]) * L[1] + x[1]) * L[0] + x[0];
}

struct Dims {
    int L[4];
};

// nbr[p][i][d] = packed index of the d-th neighbour of packed site i of parity p
__global__ void build_nbr_kernel(Dims D, int64_t Vh, const int32_t *canon_of,
                                 const int32_t *packed_of, int32_t *nbr)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * Vh) return;
    const int64_t c = canon_of[t];
    int x[4];
    coords_of(c, D.L, x);
    for (int d = 0; d < 8; ++d) {
        int y[4] = {x[0], x[1], x[2], x[3]};
        const int mu = d & 3;
        const int dir = d < 4 ? 1 : -1;
        y[mu] = (y[mu] + dir + D.L[mu]) % D.L[mu];
        nbr[t * 8 + d] = packed_of[canon_index(y, D.L)];
    }
}

template <int P>
__device__ __forceinline__ void put_link_elem(char *dst, int64_t idx, double re, double im)
{
    if constexpr (P == MOBIUS_F64) {
        reinterpret_cast<double2 *>(dst)[idx] = make_double2(re, im);
    } else if constexpr (P == MOBIUS_F32) {
        reinterpret_cast<float2 *>(dst)[idx] = make_float2((float)re, (float)im);
    } else {
        half2v h;
        h.x = (_Float16)re;
        h.y = (_Float16)im;
        reinterpret_cast<half2v *>(dst)[idx] = h;
    }
}

// record (p, d, i) of the packed links; padding elements are zero
template <int P>
// sf, sb: factors of the time-like forward (d = 3) and backward (d = 7)
// records (e^{+-mu} of a chemical potential; 1 without one)
__global__ void pack_links_kernel(Dims D, int64_t V, int64_t Vh, const int32_t *canon_of,
                                  const double2 *canon, char *packed, double sf, double sb)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * Vh * 8) return;
    const int64_t i = t % Vh;
    const int d = (int)((t / Vh) % 8);
    const int p = (int)(t / (Vh * 8));
    const int64_t c = canon_of[p * Vh + i];
    int x[4];
    coords_of(c, D.L, x);
    const int mu = d & 3;
    if (d >= 4) x[mu] = (x[mu] - 1 + D.L[mu]) % D.L[mu];
    const int64_t src = ((int64_t)mu * V + canon_index(x, D.L)) * 9;
    constexpr int REC = Link<P>::REC;
    constexpr int EB = P == MOBIUS_F64 ? 16 : P == MOBIUS_F32 ? 8 : 4;
    char *rec = packed + (((int64_t)p * 8 + d) * Vh + i) * REC;
    const double f = d == 3 ? sf : d == 7 ? sb : 1.0;
    for (int e = 0; e < REC / EB; ++e) {
        double2 u = e < 9 ? canon[src + e] : make_double2(0.0, 0.0);
        put_link_elem<P>(rec, e, f * u.x, f * u.y);
    }
}

// Walls of the fifth dimension (Sec. 2.2): the chiral shift P_{ss'} =
// delta_{ss'} P- + delta_{s',s+1 mod Ls} P+ puts a 4d field b on slice 0 as
// P- b and on slice Ls-1 as P+ b, and q = (P^+ psi)_0 = P- psi_0 + P+ psi_{Ls-1}
// reads one back.  Canonical layouts, P+ = spins 0, 1 (components 0..5).
__global__ __launch_bounds__(256) void wall_place_kernel(int64_t V, int Ls, int64_t n,
                                                         const double2 *b4, double2 *eta5)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (rhs, s, x)
    if (t >= n) return;
    const int64_t x = t % V, rs = t / V;
    const int s = (int)(rs % Ls);
    const int64_t r = rs / Ls;
    const double2 *src = b4 + (r * V + x) * 12;
    double2 *dst = eta5 + t * 12;
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        const bool take = q < 6 ? s == Ls - 1 : s == 0;
        dst[q] = take ? src[q] : make_double2(0.0, 0.0);
    }
}

__global__ __launch_bounds__(256) void wall_read_kernel(int64_t V, int Ls, int64_t n,
                                                        const double2 *psi5, double2 *q4)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (rhs, x)
    if (t >= n) return;
    const int64_t x = t % V, r = t / V;
    const double2 *lo = psi5 + ((r * Ls + 0) * V + x) * 12;
    const double2 *hi = psi5 + ((r * Ls + Ls - 1) * V + x) * 12;
    double2 *dst = q4 + t * 12;
#pragma unroll
    for (int q = 0; q < 12; ++q) dst[q] = q < 6 ? hi[q] : lo[q];
}

// Bulk reconstruction from the overlap solution (Sec. 2.3): with y the
// Pauli-Villars solution D_DW(1) y = D_DW(m) P psi~,  Omega = P^+ y,
// (P^+ y)_s = P- y_s + P+ y_{s-1 mod Ls}, and Psi_0 = psi, Psi_s = -Omega_s.
__global__ __launch_bounds__(256) void bulk_assemble_kernel(int64_t V, int Ls, int64_t n,
                                                            const double2 *psi4, const double2 *y5,
                                                            double2 *Psi5)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (rhs, s, x)
    if (t >= n) return;
    const int64_t x = t % V, rs = t / V;
    const int s = (int)(rs % Ls);
    const int64_t r = rs / Ls;
    double2 *dst = Psi5 + t * 12;
    if (s == 0) {
        const double2 *src = psi4 + (r * V + x) * 12;
#pragma unroll
        for (int q = 0; q < 12; ++q) dst[q] = src[q];
        return;
    }
    const double2 *ys = y5 + t * 12, *ym = y5 + ((r * Ls + s - 1) * V + x) * 12;
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        const double2 v = q < 6 ? ym[q] : ys[q];  // P+ from s-1, P- from s
        dst[q] = make_double2(-v.x, -v.y);
    }
}

// canonical [s][t][z][y][x][12] complex128 <-> packed halves, blockIdx.y the
// right-hand side.  Memory bound: a lane of the packed side owns one 5d site
// (64 of them in a row of each chunk), while a 5d site is a 192-byte record of
// the canonical side, records of neighbouring lanes far apart.  The two sides
// meet in LDS: on the canonical side twelve lanes move one record, so every
// access covers whole 64-byte sectors.  (One lane per record on both sides
// spread each access over 64 cache lines: at 24^3 x 64, Ls = 12 FP64 pack 969
// and unpack 1666 us, now 764 and 802 us, 5.2 TB/s as a device copy; FP16
// 663 and 1425 us, now 475 and 562 us.)  One wavefront per workgroup: 256
// threads hold 55 KB of LDS and wait for each other (8^3 x 16: 8.1 against
// 6.7 us).  The two parities' workgroups of one stretch of sites follow each
// other on one XCD, whose L2 joins the records' shared lines; the canonical
// field is not read back from there, so unpack stores it non-temporally (FP16
// 629 to 562 us).
constexpr int PACK_BLOCK = 64;

template <typename T>
struct PackLds {
    static constexpr int STRIDE = 13;  // complex per 5d site: 12 and one against bank conflicts
    cx<T> v[PACK_BLOCK * STRIDE];
    int64_t rec[PACK_BLOCK];           // canonical index of each lane's record, -1: none
};

struct PackMap {
    int p;
    uint32_t i, s;  // packed 4d site and slice of this lane
    bool ok;
};

template <typename T>
__device__ __forceinline__ PackMap pack_map(int64_t Vh, int Ls, const int32_t *canon_of, PackLds<T> &lds)
{
    const int64_t lb = logical_block(1);
    PackMap m;
    m.p = (int)(lb & 1);
    const int64_t k5 = (lb >> 1) * PACK_BLOCK + threadIdx.x;
    m.ok = k5 < Vh * Ls;
    m.i = (uint32_t)k5 / (uint32_t)Ls;
    m.s = (uint32_t)k5 - m.i * (uint32_t)Ls;
    const int64_t rec = m.ok ? (int64_t)m.s * 2 * Vh + canon_of[m.p * Vh + m.i] : -1;
    lds.rec[threadIdx.x] = rec;
    return m;
}

template <int P>
__global__ __launch_bounds__(PACK_BLOCK) void pack_spinor_kernel(int64_t Vh, int Ls,
                                                                 const int32_t *canon_of,
                                                                 const double2 *canon, char *even,
                                                                 char *odd)
{
    using S = Spin<P>;
    using T = typename S::T;
    __shared__ PackLds<T> lds;
    const int64_t N5 = Vh * Ls;
    const PackMap m = pack_map(Vh, Ls, canon_of, lds);
    canon += (int64_t)blockIdx.y * 2 * N5 * 12;
    __syncthreads();
    double2 z[12];
#pragma unroll
    for (int j = 0; j < 12; ++j) {  // (all in flight together; lanes past the end read record 0)
        const uint32_t u = (uint32_t)j * PACK_BLOCK + threadIdx.x, r = u / 12u, c = u - r * 12u;
        const int64_t rec = lds.rec[r];
        z[j] = canon[(rec < 0 ? 0 : rec) * 12 + c];
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const uint32_t u = (uint32_t)j * PACK_BLOCK + threadIdx.x, r = u / 12u, c = u - r * 12u;
        lds.v[r * PackLds<T>::STRIDE + c] = {(T)z[j].x, (T)z[j].y};
    }
    __syncthreads();
    if (!m.ok) return;
    cx<T> v[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = lds.v[threadIdx.x * PackLds<T>::STRIDE + c];
    S::store(Buf((m.p == 0 ? even : odd) + blockIdx.y * S::bytes(N5), S::bytes(N5)), Lay{(uint32_t)Ls, (uint32_t)N5}, m.i, m.s, v);
}

template <int P>
__global__ __launch_bounds__(PACK_BLOCK) void unpack_spinor_kernel(int64_t Vh, int Ls,
                                                                   const int32_t *canon_of,
                                                                   const char *even, const char *odd,
                                                                   double2 *canon)
{
    using S = Spin<P>;
    using T = typename S::T;
    __shared__ PackLds<T> lds;
    const int64_t N5 = Vh * Ls;
    const PackMap m = pack_map(Vh, Ls, canon_of, lds);
    canon += (int64_t)blockIdx.y * 2 * N5 * 12;
    if (m.ok) {
        cx<T> v[12];
        S::load(Buf((m.p == 0 ? even : odd) + blockIdx.y * S::bytes(N5), S::bytes(N5)), Lay{(uint32_t)Ls, (uint32_t)N5}, m.i, m.s, v);
#pragma unroll
        for (int c = 0; c < 12; ++c) lds.v[threadIdx.x * PackLds<T>::STRIDE + c] = v[c];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const uint32_t u = (uint32_t)j * PACK_BLOCK + threadIdx.x, r = u / 12u, c = u - r * 12u;
        const int64_t rec = lds.rec[r];
        if (rec >= 0) {
            const cx<T> z = lds.v[r * PackLds<T>::STRIDE + c];
            typedef double f64x2 __attribute__((ext_vector_type(2)));
            __builtin_nontemporal_store(f64x2{(double)z.r, (double)z.i}, reinterpret_cast<f64x2 *>(canon + rec * 12 + c));
        }
    }
}

// ---------------------------------------------------------------------------
// BLAS-1 and reductions (one thread per site5)

constexpr int BLAS_BLOCK = 256;

// A packed field of `n5` 5d sites filled with seeded pseudo-random values in
// [-1, 1) (FP16: binary16 components with site norms in [1, 2)), from a
// 32-bit hash of the word index: launch-parameter timing on data with the
// magnitudes of a Gaussian field rather than on zeros.
__device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

template <int P>
__global__ void fill_random_kernel(char *out, int64_t n5, uint32_t seed)
{
    const int64_t words = Spin<P>::bytes(n5) / 4;
    for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < words;
         w += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t h = mix32((uint32_t)w * 2654435761u ^ seed);
        const float u = (float)(h >> 8) * (1.0f / 8388608.0f) - 1.0f;  // [-1, 1)
        uint32_t v;
        if constexpr (P == MOBIUS_F64) {
            // the high word of a double in [-1, 1) with this word's low 32 bits
            const double d = (double)u;
            const uint64_t b = __builtin_bit_cast(uint64_t, d);
            v = (w & 1) ? (uint32_t)(b >> 32) : h;
        } else if constexpr (P == MOBIUS_F32) {
            v = __builtin_bit_cast(uint32_t, u);
        } else {
            if (w >= 3 * 4 * n5) {  // the site norms
                v = __builtin_bit_cast(uint32_t, 1.5f + 0.5f * u);
            } else {
                const _Float16 a = (_Float16)u, b = (_Float16)(-0.5f * u);
                v = (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
            }
        }
        reinterpret_cast<uint32_t *>(out)[w] = v;
    }
}

__global__ void zero_kernel(uint4 *p, int64_t n16, unsigned char *tail, int64_t ntail)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n16) p[k] = make_uint4(0, 0, 0, 0);
    if (k < ntail) tail[k] = 0;
}

// ---------------------------------------------------------------------------
// batched vector kernels: blockIdx.y selects the system (one lattice and one
// right-hand side); systems whose active flag is zero return at once.

__device__ __forceinline__ bool sys_inactive(const VecSys &v, const int32_t *active)
{
    return v.flag >= 0 && active && active[v.flag] == 0;
}

// 5d site k of a system in the order of the packed records: slice s of site i
struct Slice5 {
    Lay lay;
    uint32_t i, s;
    __device__ __forceinline__ Slice5(const VecSys &v, int64_t k) : lay{(uint32_t)v.Ls, (uint32_t)v.N5}
    {
        i = (uint32_t)k / lay.Ls;
        s = (uint32_t)k - i * lay.Ls;
    }
};

// The CG scalars.  The kernel that needs beta or alpha sums the norm it depends
// on itself, every workgroup the same partial sums in the same order, and its
// first workgroup keeps the scalars: a reduction launch and a scalar launch
// per norm (4.6 us each) were a fifth of an iteration on an 8^3 x 16 lattice.
// Nothing a kernel reads here is written by the same kernel (beta's reads gamma
// and the restart flag, which alpha's writes; alpha's reads gamma_new, which
// beta's writes), so no workgroup waits for another.

// the k-th summand of a sum of partials: `group` consecutive slots, added in
// the order in which a workgroup adds its wavefronts (the split hop leaves one
// slot per wavefront of sites), so that the sum does not depend on the split
__device__ __forceinline__ double summand(const double *part, int64_t k, int group, int64_t n)
{
    if (group == 1) return part[k];
    double t = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) t += k * WAVES + w < n ? part[k * WAVES + w] : 0.0;
    return t;
}

// sum of n partial sums by the whole workgroup (BLAS_BLOCK threads), in every thread
// (with the row sums of wave_sum instead of LDS shuffles, no barrier for up to
// 64 partials, and the r update no longer waiting for its stores: FP16 solve on
// 16^3 x 32, Ls = 16, 536 to 529 ms, 12 columns on 8^3 x 16 367 to 362, FP64 on
// 8^3 x 16 64.1 to 63.2; the same for up to 128 or 256 partials, where every
// wavefront loads them all, is slower again by 0.5 %)
static_assert(BLOCK == BLAS_BLOCK, "the r update runs in the site kernels' workgroups");
__device__ __forceinline__ double block_total(const double *part, int64_t n, int group)
{
    __shared__ double red[BLAS_BLOCK / 64];
    double t = 0;
    if (n <= 64 && group == 1) {  // each wavefront by itself: none waits for another
        const int64_t k = threadIdx.x & 63;
        return wave_sum(k < n ? part[k] : 0.0);
    }
#pragma unroll 4
    for (int64_t k = threadIdx.x; k * group < n; k += BLAS_BLOCK) t += summand(part, k, group, n);
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    t = 0;
#pragma unroll
    for (int w = 0; w < BLAS_BLOCK / 64; ++w) t += red[w];
    return t;
}

// beta = gamma_new / gamma (0 when the system restarts) with gamma_new = the sum
// of v.red
__device__ __forceinline__ double cg_beta(const VecSys &v, const int32_t *restart)
{
    CgScalars &s = *v.cg;
    const double gamma = s.gamma;
    const bool rs = restart[v.flag] != 0;
    const double g = block_total(v.red, v.nred, v.redgroup);
    const double beta = (!rs && gamma > 0) ? g / gamma : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        s.gamma_new = g;
        s.beta = beta;
        if (s.hist && s.nhist < s.hmax) s.hist[2 * s.nhist] = beta;
    }
    return beta;
}

// alpha = gamma_new / |q|^2 with |q|^2 = the sum of v.red; slot: see aring
__device__ __forceinline__ double cg_alpha(const VecSys &v, int32_t *restart, int slot)
{
    CgScalars &s = *v.cg;
    const double g = s.gamma_new;
    const double qq = block_total(v.red, v.nred, v.redgroup);
    const double alpha = qq > 0 ? g / qq : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        s.qq = qq;
        s.alpha = alpha;
        s.gamma = g;
        if (s.hist && s.nhist < s.hmax) s.hist[2 * s.nhist++ + 1] = alpha;
        if (slot >= 0) s.aring[slot] = alpha;
        restart[v.flag] = 0;
    }
    return alpha;
}

// x (PX) += alpha p;  r -= alpha q;  partials of |r|^2.  a = x, b = p, c = r, d = q
// (a null: r and its norm only, x is updated elsewhere).
template <int P, int PX>
__global__ __launch_bounds__(BLAS_BLOCK) void cg_xr_batch(const VecSys *sys, const int32_t *active,
                                                          int32_t *restart, int slot)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using SX = Spin<PX>;
    using T = typename S::T;
    using TX = typename SX::T;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if ((int64_t)blockIdx.x * BLAS_BLOCK >= v.N5) return;
    const bool ok = k < v.N5;
    const int64_t fb = S::bytes(v.N5);
    const Slice5 z(v, ok ? k : v.N5 - 1);
    const Buf bx(v.a, SX::bytes(v.N5)), bp(v.b, fb), br(v.c, fb), bq(v.d, fb);
    cx<T> rv[12], qv[12];
    S::load(br, z.lay, z.i, z.s, rv);
    S::load(bq, z.lay, z.i, z.s, qv);
    const double alpha = cg_alpha(v, restart, slot);
    double n = 0;
    if (ok) {
        const T al = (T)alpha;
        if (v.a) {
            const TX alx = (TX)alpha;
            cx<TX> xv[12];
            cx<T> pv[12];
            SX::load(bx, z.lay, z.i, z.s, xv);
            S::load(bp, z.lay, z.i, z.s, pv);
#pragma unroll
            for (int c = 0; c < 12; ++c) xv[c] = xv[c] + alx * cx<TX>{(TX)pv[c].r, (TX)pv[c].i};
            SX::store(bx, z.lay, z.i, z.s, xv);
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) rv[c] = rv[c] - al * qv[c];
        n = S::store_norm2(br, z.lay, z.i, z.s, rv);
    }
    block_sum_store(n, v.partials, blockIdx.x);
}

// d = s0 * a + s1 * b  (null scalar = 1); optional partials of |d|^2
template <int P, bool NORM>
__global__ __launch_bounds__(BLAS_BLOCK) void axpby_batch(const VecSys *sys, const int32_t *active)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using T = typename S::T;
    if ((int64_t)blockIdx.x * BLAS_BLOCK >= v.N5) return;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double n = 0;
    if (k < v.N5) {
        const T av = v.s0 ? (T)*v.s0 : (T)1, bv = v.s1 ? (T)*v.s1 : (T)1;
        const int64_t fb = S::bytes(v.N5);
        const Slice5 z(v, k);
        cx<T> xv[12], yv[12];
        S::load(Buf(v.a, fb), z.lay, z.i, z.s, xv);
        S::load(Buf(v.b, fb), z.lay, z.i, z.s, yv);
#pragma unroll
        for (int c = 0; c < 12; ++c) xv[c] = av * xv[c] + bv * yv[c];
        if constexpr (NORM)
            n = S::store_norm2(Buf(v.d, fb), z.lay, z.i, z.s, xv);
        else
            S::store(Buf(v.d, fb), z.lay, z.i, z.s, xv);
    }
    if constexpr (NORM) block_sum_store(n, v.partials, blockIdx.x);
}

// partials of |a|^2
template <int P>
__global__ __launch_bounds__(BLAS_BLOCK) void norm2_batch(const VecSys *sys, const int32_t *active)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using T = typename S::T;
    if ((int64_t)blockIdx.x * BLAS_BLOCK >= v.N5) return;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double n = 0;
    if (k < v.N5) {
        const Slice5 z(v, k);
        cx<T> x[12];
        S::load(Buf(v.a, S::bytes(v.N5)), z.lay, z.i, z.s, x);
        n = site_norm2(x);
    }
    block_sum_store(n, v.partials, blockIdx.x);
}

// precision conversion b (PO) = a (PI); accumulate: d (F64) += a (PI)
template <int PI, int PO>
__global__ __launch_bounds__(BLAS_BLOCK) void convert_batch(const VecSys *sys, const int32_t *active)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (k >= v.N5) return;
    const Slice5 z(v, k);
    cx<typename Spin<PI>::T> x[12];
    Spin<PI>::load(Buf(v.a, Spin<PI>::bytes(v.N5)), z.lay, z.i, z.s, x);
    cx<typename Spin<PO>::T> w[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = {(typename Spin<PO>::T)x[c].r, (typename Spin<PO>::T)x[c].i};
    Spin<PO>::store(Buf(v.b, Spin<PO>::bytes(v.N5)), z.lay, z.i, z.s, w);
}

template <int PI>
__global__ __launch_bounds__(BLAS_BLOCK) void accumulate_batch(const VecSys *sys, const int32_t *active)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (k >= v.N5) return;
    const Slice5 z(v, k);
    cx<typename Spin<PI>::T> x[12];
    Spin<PI>::load(Buf(v.a, Spin<PI>::bytes(v.N5)), z.lay, z.i, z.s, x);
    cx<double> h[12];
    const Buf bh(v.d, Spin<MOBIUS_F64>::bytes(v.N5));
    Spin<MOBIUS_F64>::load(bh, z.lay, z.i, z.s, h);
#pragma unroll
    for (int c = 0; c < 12; ++c) h[c] = {h[c].r + (double)x[c].r, h[c].i + (double)x[c].i};
    Spin<MOBIUS_F64>::store(bh, z.lay, z.i, z.s, h);
    // the low-precision correction is consumed: clear it
    cx<typename Spin<PI>::T> zero[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) zero[c] = {0, 0};
    Spin<PI>::store(Buf(v.a, Spin<PI>::bytes(v.N5)), z.lay, z.i, z.s, zero);
}

// x (PX) += alpha p_old;  p = s + beta p_old.  a = s, b = p, c = x, s0 = alpha.
// (The x update of a CG step moved here from the r update: p_old is read anyway.)
template <int P, int PX>
__global__ __launch_bounds__(BLAS_BLOCK) void pupd_x_batch(const VecSys *sys, const int32_t *active,
                                                           const int32_t *restart)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using SX = Spin<PX>;
    using T = typename S::T;
    using TX = typename SX::T;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if ((int64_t)blockIdx.x * BLAS_BLOCK >= v.N5) return;
    const int64_t fb = S::bytes(v.N5);
    const Slice5 z(v, k < v.N5 ? k : v.N5 - 1);
    const Buf bs(v.a, fb), bp(v.b, fb), bx(v.c, SX::bytes(v.N5));
    cx<T> sv[12], pv[12];
    cx<TX> xv[12];
    S::load(bp, z.lay, z.i, z.s, pv);
    SX::load(bx, z.lay, z.i, z.s, xv);
    S::load(bs, z.lay, z.i, z.s, sv);
    const TX al = (TX)*v.s0;
    const T be = (T)cg_beta(v, restart);
    if (k >= v.N5) return;
#pragma unroll
    for (int c = 0; c < 12; ++c) xv[c] = xv[c] + al * cx<TX>{(TX)pv[c].r, (TX)pv[c].i};
    SX::store(bx, z.lay, z.i, z.s, xv);
#pragma unroll
    for (int c = 0; c < 12; ++c) pv[c] = sv[c] + be * pv[c];
    S::store(bp, z.lay, z.i, z.s, pv);
}

// x (PX) += alpha p.  a = p, c = x, s0 = alpha.
template <int P, int PX>
__global__ __launch_bounds__(BLAS_BLOCK) void xflush_batch(const VecSys *sys, const int32_t *active)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using SX = Spin<PX>;
    using TX = typename SX::T;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (k >= v.N5) return;
    const TX al = (TX)*v.s0;
    const Slice5 z(v, k);
    const Buf bx(v.c, SX::bytes(v.N5));
    cx<typename S::T> pv[12];
    cx<TX> xv[12];
    S::load(Buf(v.a, S::bytes(v.N5)), z.lay, z.i, z.s, pv);
    SX::load(bx, z.lay, z.i, z.s, xv);
#pragma unroll
    for (int c = 0; c < 12; ++c) xv[c] = xv[c] + al * cx<TX>{(TX)pv[c].r, (TX)pv[c].i};
    SX::store(bx, z.lay, z.i, z.s, xv);
}

// p[slot] = s + beta p[prev] in a ring of directions (the deferred x update
// keeps one chunk's directions; slot = prev: in place).  a = s, b = p[0], slots
// sstride bytes apart.
template <int P>
__global__ __launch_bounds__(BLAS_BLOCK) void pupd_ring_batch(const VecSys *sys, const int32_t *active,
                                                              const int32_t *restart, int slot,
                                                              int prev)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using T = typename S::T;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if ((int64_t)blockIdx.x * BLAS_BLOCK >= v.N5) return;
    const int64_t fb = S::bytes(v.N5);
    const Slice5 z(v, k < v.N5 ? k : v.N5 - 1);
    cx<T> sv[12], pv[12];  // (in flight while beta is summed)
    S::load(Buf(v.b + prev * v.sstride, fb), z.lay, z.i, z.s, pv);
    S::load(Buf(v.a, fb), z.lay, z.i, z.s, sv);
    const T be = (T)cg_beta(v, restart);
    if (k >= v.N5) return;
#pragma unroll
    for (int c = 0; c < 12; ++c) pv[c] = sv[c] + be * pv[c];
    S::store(Buf(v.b + slot * v.sstride, fb), z.lay, z.i, z.s, pv);
}

// x (PX) += sum_{i < n} alpha_i p[i]: the x update of a chunk in one pass.
// b = p[0], slots sstride bytes apart, s0 = the alphas, c = x.
template <int P, int PX>
__global__ __launch_bounds__(BLAS_BLOCK) void xring_batch(const VecSys *sys, const int32_t *active, int n)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using SX = Spin<PX>;
    using TX = typename SX::T;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (k >= v.N5) return;
    const int64_t fb = S::bytes(v.N5);
    const Slice5 z(v, k);
    cx<TX> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = cx<TX>{0, 0};
#pragma unroll 2
    for (int i = 0; i < n; ++i) {
        const TX al = (TX)v.s0[i];
        cx<typename S::T> pv[12];
        S::load(Buf(v.b + i * v.sstride, fb), z.lay, z.i, z.s, pv);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = acc[c] + al * cx<TX>{(TX)pv[c].r, (TX)pv[c].i};
    }
    const Buf bx(v.c, SX::bytes(v.N5));
    cx<TX> xv[12];
    SX::load(bx, z.lay, z.i, z.s, xv);
#pragma unroll
    for (int c = 0; c < 12; ++c) xv[c] = xv[c] + acc[c];
    SX::store(bx, z.lay, z.i, z.s, xv);
}

// r -= alpha q, |r|^2 per site block, and u = I^-+ r of the stored r, in the
// site-lane mapping of the hop so that the Ls-direction solve stays inside a
// wavefront.  a = r, b = q, c = u; one workgroup per site block.
template <int P>
__global__ __launch_bounds__(BLOCK) void rupd_m5inv_batch(const VecSys *sys, const int32_t *active,
                                                          int32_t *restart, int slot, int mode)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    const int Ls = v.Ls, spw = 64 / Ls;
    const int64_t Vh = v.N5 / Ls;
    const int64_t per_block = (int64_t)spw * WAVES;
    if ((int64_t)blockIdx.x * per_block >= Vh) return;  // uniform in the workgroup
    using S = Spin<P>;
    using T = typename S::T;
    const SiteMap m = site_map_lb(Ls, spw, Vh, blockIdx.x);
    const Coef<T> k = make_coef<T>(*v.coef);
    const uint32_t i5 = (uint32_t)m.i, s5 = (uint32_t)m.s;
    const Lay lay{(uint32_t)Ls, (uint32_t)v.N5};
    const int64_t fb = S::bytes(v.N5);
    const Buf br(v.a, fb);
    cx<T> rv[12], qv[12];
    S::load(br, lay, i5, s5, rv);
    S::load(Buf(v.b, fb), lay, i5, s5, qv);
    const T al = (T)cg_alpha(v, restart, slot);
#pragma unroll
    for (int c = 0; c < 12; ++c) rv[c] = rv[c] - al * qv[c];
    double n = 0;
    if (m.site_ok) n = S::store_norm2_q(br, lay, i5, s5, rv);
    block_sum_store(n, v.partials, blockIdx.x);
    if (mode == 2) return;  // uniform: no solve of the updated residual
    __shared__ M5Lds<T> lds;
    m5inv_lanes(rv, k, m, Ls, mode != 1, lds);
    if (mode == 3) mix_s(rv, k.b5, k.c5, k.mf, m, Ls, true);  // B^+ I^-+ r (left form)
    if (m.site_ok) S::store(Buf(v.c, fb), lay, i5, s5, rv);
}

// partials of Re <a, b>
template <int P>
__global__ __launch_bounds__(BLAS_BLOCK) void dot_batch(const VecSys *sys, const int32_t *active)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active)) return;
    using S = Spin<P>;
    using T = typename S::T;
    if ((int64_t)blockIdx.x * BLAS_BLOCK >= v.N5) return;
    const int64_t k = (int64_t)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double n = 0;
    if (k < v.N5) {
        const int64_t fb = S::bytes(v.N5);
        const Slice5 z(v, k);
        cx<T> x[12], y[12];
        S::load(Buf(v.a, fb), z.lay, z.i, z.s, x);
        S::load(Buf(v.b, fb), z.lay, z.i, z.s, y);
#pragma unroll
        for (int c = 0; c < 12; ++c) n += (double)x[c].r * y[c].r + (double)x[c].i * y[c].i;
    }
    block_sum_store(n, v.partials, blockIdx.x);
}

// One block per system: out[sys * out_stride] = sum of the system's partials
// (fixed order).
__global__ __launch_bounds__(1024) void reduce_batch(const VecSys *sys, const int32_t *active,
                                                     int64_t count_override, double *out,
                                                     int64_t out_stride)
{
    const VecSys v = sys[blockIdx.x];
    if (sys_inactive(v, active)) return;
    __shared__ double sm[1024];
    const int64_t n = count_override > 0 ? count_override : v.nparts;
    double t = 0;
    for (int64_t k = threadIdx.x; k * v.group < n; k += 1024) t += summand(v.partials, k, v.group, n);
    sm[threadIdx.x] = t;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x * out_stride] = sm[0];
}

// First level of a long sum: slot b of out[sys * RED_PARTS + b] = the b-th part
// of the system's partials.
__global__ __launch_bounds__(BLAS_BLOCK) void reduce_parts_batch(const VecSys *sys, const int32_t *active,
                                                                 double *out)
{
    const VecSys v = sys[blockIdx.y];
    if (sys_inactive(v, active) || v.nparts <= RED_DIRECT) return;
    const int64_t n = v.nparts, a = n * blockIdx.x / RED_PARTS, b = n * (blockIdx.x + 1) / RED_PARTS;
    const double t = block_total(v.partials + a, b - a, 1);  // (so long a sum is no split hop's)
    if (threadIdx.x == 0) out[(int64_t)blockIdx.y * RED_PARTS + blockIdx.x] = t;
}

// alpha = 0 for every active system: no x update is pending
__global__ void clear_alpha_batch(CgScalars *sc, int nsys, const int32_t *active)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < nsys && (!active || active[j])) sc[j].alpha = 0.0;
}

}  // namespace

// ---------------------------------------------------------------------------
// Workspace of the allocation-free entry point (mobius_dslash_noalloc): one
// statically sized array per GPU, held until the process ends.  In host code
// `scratch` names a host-side stand-in, not device memory: only the address
// that hipGetSymbolAddress returns for the current device is ever passed to a
// kernel or a copy.
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];
namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    void *ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

void *noalloc_scratch(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_ptr[device];
}

HopTuning &hop_tuning()
{
    static HopTuning t = [] {
        HopTuning d;
        const auto given = [](const char *name, int v) {
            const char *e = std::getenv(name);
            return e ? std::atoi(e) : v;
        };
        d.xcd_remap = given("MOBIUS_XCD_REMAP", d.xcd_remap);
        d.prefetch = given("MOBIUS_PREFETCH", d.prefetch);
        d.stage_links = given("MOBIUS_STAGE_LINKS", d.stage_links);
        d.nt_links = given("MOBIUS_NT_LINKS", d.nt_links);
        // another loop variant than the default was asked for (the block order is the
        // split form's too)
        const HopTuning own;
        if (d.prefetch != own.prefetch || d.stage_links != own.stage_links || d.nt_links != own.nt_links)
            d.split_dirs = 0;
        return d;
    }();
    return t;
}

// ---------------------------------------------------------------------------
// launchers

int64_t site_kernel_blocks(const Geometry &g)
{
    const int spw = sites_per_wave(g.Ls);
    const int64_t per_block = (int64_t)spw * WAVES;
    return (g.Vh + per_block - 1) / per_block;
}

bool hop_splits_dirs(const Geometry &g, int prec, int nrhs, const HopTuning &t)
{
    return t.split_dirs && site_kernel_blocks(g) * nrhs <= SPLIT_BLOCKS[prec];
}

int64_t hop_partials(const Geometry &g, bool split_dirs)
{
    const int spw = sites_per_wave(g.Ls);
    return split_dirs ? (g.Vh + spw - 1) / spw : site_kernel_blocks(g);
}

int64_t blas_blocks(const Geometry &g) { return (g.N5 + BLAS_BLOCK - 1) / BLAS_BLOCK; }

hipError_t launch_build_geometry(const Geometry &g, const int32_t *packed_of, int32_t *nbr,
                                 hipStream_t st)
{
    Dims D{{g.L[0], g.L[1], g.L[2], g.L[3]}};
    const int64_t n = 2 * g.Vh;
    hipLaunchKernelGGL(build_nbr_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, D,
                       g.Vh, g.canon_of, packed_of, nbr);
    return hipGetLastError();
}

hipError_t launch_pack_links(const Geometry &g, int prec, const void *canon, void *packed,
                             hipStream_t st, double sf, double sb)
{
    Dims D{{g.L[0], g.L[1], g.L[2], g.L[3]}};
    const int64_t n = 2 * g.Vh * 8;
    dim3 grid((unsigned)((n + 255) / 256));
    const double2 *c = static_cast<const double2 *>(canon);
    char *o = static_cast<char *>(packed);
    switch (prec) {
    case MOBIUS_F64: hipLaunchKernelGGL(pack_links_kernel<MOBIUS_F64>, grid, dim3(256), 0, st, D, g.V, g.Vh, g.canon_of, c, o, sf, sb); break;
    case MOBIUS_F32: hipLaunchKernelGGL(pack_links_kernel<MOBIUS_F32>, grid, dim3(256), 0, st, D, g.V, g.Vh, g.canon_of, c, o, sf, sb); break;
    case MOBIUS_F16: hipLaunchKernelGGL(pack_links_kernel<MOBIUS_F16>, grid, dim3(256), 0, st, D, g.V, g.Vh, g.canon_of, c, o, sf, sb); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_wall_place(const Geometry &g, const void *b4, void *eta5, int nrhs, hipStream_t st)
{
    const int64_t n = (int64_t)nrhs * g.Ls * g.V;
    hipLaunchKernelGGL(wall_place_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g.V, g.Ls, n,
                       static_cast<const double2 *>(b4), static_cast<double2 *>(eta5));
    return hipGetLastError();
}

hipError_t launch_wall_read(const Geometry &g, const void *psi5, void *q4, int nrhs, hipStream_t st)
{
    const int64_t n = (int64_t)nrhs * g.V;
    hipLaunchKernelGGL(wall_read_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g.V, g.Ls, n,
                       static_cast<const double2 *>(psi5), static_cast<double2 *>(q4));
    return hipGetLastError();
}

hipError_t launch_bulk_assemble(const Geometry &g, const void *psi4, const void *y5, void *Psi5,
                                int nrhs, hipStream_t st)
{
    const int64_t n = (int64_t)nrhs * g.Ls * g.V;
    hipLaunchKernelGGL(bulk_assemble_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g.V,
                       g.Ls, n, static_cast<const double2 *>(psi4), static_cast<const double2 *>(y5),
                       static_cast<double2 *>(Psi5));
    return hipGetLastError();
}

namespace {
// one block per PACK_BLOCK packed 5d sites of a parity, the parities alternating
dim3 pack_grid(const Geometry &g, int nrhs)
{
    return dim3((unsigned)(2 * ((g.N5 + PACK_BLOCK - 1) / PACK_BLOCK)), (unsigned)nrhs);
}
}  // namespace

hipError_t launch_pack_spinor(const Geometry &g, int prec, const void *canon, void *even, void *odd,
                              int nrhs, hipStream_t st)
{
    const dim3 blk(PACK_BLOCK);
    const int64_t fb = field_bytes(g, prec);
    for (int r = 0; r < nrhs; r += MAX_GRID_Y) {
        const dim3 grid = pack_grid(g, std::min(nrhs - r, MAX_GRID_Y));
        const double2 *c = static_cast<const double2 *>(canon) + (int64_t)r * 2 * g.N5 * 12;
        char *e = static_cast<char *>(even) + r * fb, *o = static_cast<char *>(odd) + r * fb;
        switch (prec) {
        case MOBIUS_F64: hipLaunchKernelGGL(pack_spinor_kernel<MOBIUS_F64>, grid, blk, 0, st, g.Vh, g.Ls, g.canon_of, c, e, o); break;
        case MOBIUS_F32: hipLaunchKernelGGL(pack_spinor_kernel<MOBIUS_F32>, grid, blk, 0, st, g.Vh, g.Ls, g.canon_of, c, e, o); break;
        case MOBIUS_F16: hipLaunchKernelGGL(pack_spinor_kernel<MOBIUS_F16>, grid, blk, 0, st, g.Vh, g.Ls, g.canon_of, c, e, o); break;
        default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

hipError_t launch_unpack_spinor(const Geometry &g, int prec, const void *even, const void *odd,
                                void *canon, int nrhs, hipStream_t st)
{
    const dim3 blk(PACK_BLOCK);
    const int64_t fb = field_bytes(g, prec);
    for (int r = 0; r < nrhs; r += MAX_GRID_Y) {
        const dim3 grid = pack_grid(g, std::min(nrhs - r, MAX_GRID_Y));
        double2 *c = static_cast<double2 *>(canon) + (int64_t)r * 2 * g.N5 * 12;
        const char *e = static_cast<const char *>(even) + r * fb, *o = static_cast<const char *>(odd) + r * fb;
        switch (prec) {
        case MOBIUS_F64: hipLaunchKernelGGL(unpack_spinor_kernel<MOBIUS_F64>, grid, blk, 0, st, g.Vh, g.Ls, g.canon_of, e, o, c); break;
        case MOBIUS_F32: hipLaunchKernelGGL(unpack_spinor_kernel<MOBIUS_F32>, grid, blk, 0, st, g.Vh, g.Ls, g.canon_of, e, o, c); break;
        case MOBIUS_F16: hipLaunchKernelGGL(unpack_spinor_kernel<MOBIUS_F16>, grid, blk, 0, st, g.Vh, g.Ls, g.canon_of, e, o, c); break;
        default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

size_t m5_epilogue_lds_bytes(int prec)
{
    return prec == MOBIUS_F64 ? sizeof(M5Lds<double>) : sizeof(M5Lds<float>);
}

size_t hop_link_lds_bytes(int prec, int Ls, bool rows)
{
    const int spw = sites_per_wave(Ls);
    switch (prec) {
    case MOBIUS_F64: return link_lds_bytes<MOBIUS_F64>(spw, false);
    case MOBIUS_F32: return link_lds_bytes<MOBIUS_F32>(spw, false);
    default: return link_lds_bytes<MOBIUS_F16>(spw, rows);
    }
}

namespace {

// Whether the right-hand sides of a launch run side by side, each workgroup
// staging its links for one of them, or take turns in workgroups that stage once.
// Ratios: time taking turns / time side by side, D_{p,1-p} and its adjoint and left
// forms unless D_pre is named.
bool rhs_side_by_side(const Geometry &g, const HopArgs &a, const HopParams &hp)
{
    const int64_t n = a.nrhs, b = site_kernel_blocks(g), cus = 256;
    const auto per_cu = [](int64_t blocks) { return (blocks + cus - 1) / cus; };
    // links of a parity beyond half the 256 MB Infinity Cache come from memory
    // each time (24^3 x 64, Ls = 12, 3 right-hand sides, D_pre: FP64 0.97, FP16 0.97)
    if (8 * g.Vh * link_record_bytes(a.prec) > (int64_t)128 << 20) return false;
    if (!hp.stage_links) return true;  // nothing is staged (FP64, Ls = 4, 16^4, 3: D_pre 1.1)
    // CUs that the sites alone leave idle (128 blocks, 3 to 12: 1.0 to 2.3; 210
    // blocks, 2: 1.0 to 1.2)
    if (b <= 160 || b * n <= 2 * cus) return true;
    // The I^-1 epilogue's buffer takes the links' place in LDS only if they are
    // done with; beside them it may cost a resident workgroup (16^3 x 32, Ls = 8,
    // 3 right-hand sides, D_pre: FP64 1.19, FP16 1.11; at Ls = 12, where FP64 loses
    // none, 0.94).  FP32 and FP16 keep two on a CU, enough for up to 512 blocks
    // (16^4, Ls = 4, 2 to 6, FP32: 0.9).
    const bool inverse = (a.epi & EPI_M5INV) != 0, mixes = !a.dag && !(a.epi & EPI_PREMIXED);
    if (inverse && (a.prec == MOBIUS_F64 || b > 2 * cus)) {
        const int64_t lds = 160 * 1024, resident = a.prec == MOBIUS_F64 ? 2 : 4;
        const int64_t both = hop_link_lds_bytes(a.prec, g.Ls, hp.pf == 3) + m5_epilogue_lds_bytes(a.prec);
        if (lds / both < resident) return true;
    }
    // FP32 and FP16: the sites fill the chip from about 400 blocks (324: 1.0 to 1.3;
    // 432: 0.9 to 1.0, with an epilogue or input mixing 1.0 to 1.1); FP16, whose staging
    // converts the links, then loses by repeating it (683 to 4096 blocks 0.8 to 1.0)
    const int64_t few = inverse || mixes ? 448 : 384;
    if (a.prec == MOBIUS_F16) return b <= few;
    // many slices to a link while the fields stay in the Infinity Cache (Ls = 12, 519
    // blocks, 3: FP64 1.1 to 1.2, FP32 1.1; 16^3 x 32, Ls = 12, FP64: 0.96) or beyond
    // (Ls = 16, 3 to 12: FP64 1.0 to 1.28), or many right-hand sides on several
    // rounds of workgroups (1024 to 1536 blocks, 6 and 12: FP64 1.0 to 1.2; 2 or 3 of
    // them 0.9 to 1.0)
    if (g.Ls >= 10 && 2 * field_bytes(g, a.prec) <= (int64_t)256 << 20) return true;
    if ((g.Ls >= 16 && n >= 3) || (n >= 6 && b >= 1024)) return true;
    if (a.prec == MOBIUS_F32) return b <= few;  // (Ls = 5, 683 blocks: 0.9)
    // FP64, whose workgroups on one CU run one after the other in effect: by the
    // fullest CU (324 blocks, 3: 4 against 6, 1.05 to 1.13; 216 blocks, 3: 3 against 3,
    // 0.85; 432 blocks, 3: 6 against 6, 0.84)
    return 10 * per_cu(b * n) <= 7 * n * per_cu(b);
}

}  // namespace

HopParams make_hop_params(const Geometry &g, const OpCoeffs &c, const void *links,
                          const int32_t *nbr, const HopArgs &a)
{
    HopParams hp{};
    const int64_t lb = (int64_t)8 * g.Vh * link_record_bytes(a.prec);
    hp.links = static_cast<const char *>(links) + (int64_t)a.out_parity * lb;
    hp.nbr = nbr + (int64_t)a.out_parity * 8 * g.Vh;
    hp.in = static_cast<const char *>(a.in);
    hp.out = static_cast<char *>(a.out);
    hp.x = static_cast<const char *>(a.x);
    hp.y = static_cast<const char *>(a.y);
    hp.partials = a.partials;
    hp.active = a.active;
    hp.Vh = g.Vh;
    hp.N5 = g.N5;
    hp.fstride = a.fstride > 0 ? a.fstride : field_bytes(g, a.prec);
    const HopTuning &t = a.tune ? *a.tune : hop_tuning();
    const bool split_dirs = a.allow_split && hop_splits_dirs(g, a.prec, a.nrhs, t);
    hp.nblocks = hop_partials(g, split_dirs);
    hp.pstride = a.pstride > 0 ? a.pstride : hp.nblocks;
    hp.Ls = g.Ls;
    hp.spw = sites_per_wave(g.Ls);
    hp.nrhs = a.nrhs;
    hp.remap = t.xcd_remap;
    hp.stage_links = t.stage_links && hop_link_lds_bytes(a.prec, g.Ls, false) <= 64 * 1024;
    hp.nt = nt_link_loads(t, g, a.prec);
    hp.pf = prefetch_depth(t, a.prec, !a.dag && !(a.epi & EPI_PREMIXED));
    // matrix-core colour multiply: FP16 with staged links and whole 4-lane
    // groups of one site (Ls divisible by 4)
    if (a.prec == MOBIUS_F16 && t.mfma && hp.stage_links && g.Ls % 4 == 0 &&
        hop_link_lds_bytes(a.prec, g.Ls, true) <= 64 * 1024)
        hp.pf = 3;
    hp.split = rhs_side_by_side(g, a, hp) ? a.nrhs : 1;
    if (split_dirs) {
        hp.split_mfma = hp.pf == 3;
        hp.pf = 4;
        hp.stage_links = 0;
        hp.split = a.nrhs;
    }
    hp.c = c;
    return hp;
}

hipError_t launch_hop(const Geometry &g, const OpCoeffs &c, const void *links, const int32_t *nbr,
                      const HopArgs &a, hipStream_t st)
{
    const HopParams hp = make_hop_params(g, c, links, nbr, a);
    const int epi = a.epi & ~EPI_BDAG;
    bool ok = false;
    switch (a.prec) {
    case MOBIUS_F64: ok = run_hop<MOBIUS_F64>(a.dag, epi, hp, st); break;
    case MOBIUS_F32: ok = run_hop<MOBIUS_F32>(a.dag, epi, hp, st); break;
    case MOBIUS_F16: ok = run_hop<MOBIUS_F16>(a.dag, epi, hp, st); break;
    }
    return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_hop_batch(int prec, int dag, int epi, const HopParams *groups_dev, int ngroups,
                            const int64_t *prefix_dev, size_t lds_bytes, int grid, int pf,
                            hipStream_t st)
{
    epi &= ~EPI_BDAG;
    bool ok = false;
    switch (prec) {
    case MOBIUS_F64: ok = run_hop_batch<MOBIUS_F64>(dag, epi, groups_dev, ngroups, prefix_dev, lds_bytes, grid, pf, st); break;
    case MOBIUS_F32: ok = run_hop_batch<MOBIUS_F32>(dag, epi, groups_dev, ngroups, prefix_dev, lds_bytes, grid, pf, st); break;
    case MOBIUS_F16: ok = run_hop_batch<MOBIUS_F16>(dag, epi, groups_dev, ngroups, prefix_dev, lds_bytes, grid, pf, st); break;
    }
    return ok ? hipGetLastError() : hipErrorInvalidValue;
}

namespace {
template <int P>
void m5_launch(int kind, int dag, const char *in, char *out, const Geometry &g, const OpCoeffs &c,
               int64_t blocks, hipStream_t st)
{
    const int spw = sites_per_wave(g.Ls);
    // (see RecordTile)  A field and its result in the L2s' 32 MB are not bound by lines,
    // and the passes through LDS lengthen each wavefront's chain: I^-1 of FP64 on
    // 4 x 10 x 12 x 8, Ls = 4 (1.4 MB) takes 6.3 us as one stretch and 5.1 directly, on
    // 12^4, Ls = 12 (23 MB) 14.3 and 11.5, of FP32 there (11 MB) 7.5 and 6.4.  Fields past
    // them gain by the stretch: FP32, 36 MB, Ls = 12 (16^4) 15.8 and 16.4, Ls = 4
    // (16^2 x 24 x 32) 13.6 and 18.7; FP64, 36 MB, Ls = 4 (16^3 x 24) 15.5 and 16.1.  FP64
    // with a longer Ls has fewer half lines and gains from later on: Ls = 20 at 76 MB
    // 32.8 and 31.8, at 120 MB 47.8 and 48.4; Ls = 12 at 72 MB 31.9 and 31.2, at 108 MB
    // 43.7 and 44.8.
    const int64_t least = (int64_t)(P == MOBIUS_F64 && g.Ls > 4 ? 96 : 32) << 20;
    const bool linear = P != MOBIUS_F16 && g.Ls % 8 == 4 && spw > 1 && field_bytes(g, P) >= least;
    const dim3 grid((unsigned)blocks), blk(BLOCK);
#define MOBIUS_M5(D, K)                                                                             \
    if (linear)                                                                                    \
        hipLaunchKernelGGL((m5_kernel<P, D, K, P != MOBIUS_F16>), grid, blk, 0, st, in, out, g.Vh, g.N5, g.Ls, spw, c); \
    else                                                                                           \
        hipLaunchKernelGGL((m5_kernel<P, D, K, false>), grid, blk, 0, st, in, out, g.Vh, g.N5, g.Ls, spw, c)
    if (kind == 0 && !dag) { MOBIUS_M5(false, 0); }
    if (kind == 0 && dag) { MOBIUS_M5(true, 0); }
    if (kind == 1 && !dag) { MOBIUS_M5(false, 1); }
    if (kind == 1 && dag) { MOBIUS_M5(true, 1); }
#undef MOBIUS_M5
}
}  // namespace

hipError_t launch_m5(const Geometry &g, const OpCoeffs &c, int prec, int kind, int dag,
                     const void *in, void *out, int nrhs, hipStream_t st)
{
    const int64_t blocks = site_kernel_blocks(g);
    const int64_t fb = field_bytes(g, prec);
    for (int r = 0; r < nrhs; ++r) {
        const char *i = static_cast<const char *>(in) + r * fb;
        char *o = static_cast<char *>(out) + r * fb;
        switch (prec) {
        case MOBIUS_F64: m5_launch<MOBIUS_F64>(kind, dag, i, o, g, c, blocks, st); break;
        case MOBIUS_F32: m5_launch<MOBIUS_F32>(kind, dag, i, o, g, c, blocks, st); break;
        case MOBIUS_F16: m5_launch<MOBIUS_F16>(kind, dag, i, o, g, c, blocks, st); break;
        default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

hipError_t launch_fill_random(int prec, void *ptr, int64_t n5, uint32_t seed, hipStream_t st)
{
    const dim3 grid(2048), blk(256);
    char *p = static_cast<char *>(ptr);
    switch (prec) {
    case MOBIUS_F64: hipLaunchKernelGGL(fill_random_kernel<MOBIUS_F64>, grid, blk, 0, st, p, n5, seed); break;
    case MOBIUS_F32: hipLaunchKernelGGL(fill_random_kernel<MOBIUS_F32>, grid, blk, 0, st, p, n5, seed); break;
    case MOBIUS_F16: hipLaunchKernelGGL(fill_random_kernel<MOBIUS_F16>, grid, blk, 0, st, p, n5, seed); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_zero(void *ptr, int64_t bytes, hipStream_t st)
{
    const int64_t n16 = bytes / 16;
    const int64_t ntail = bytes - n16 * 16;
    const int64_t n = n16 > ntail ? n16 : ntail;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       static_cast<uint4 *>(ptr), n16,
                       static_cast<unsigned char *>(ptr) + n16 * 16, ntail);
    return hipGetLastError();
}

hipError_t launch_vec_batch(int kind, int prec, int prec2, const VecSys *sys_dev, int nsys,
                            int64_t max_n5, const int32_t *active, hipStream_t st)
{
    const dim3 grid((unsigned)((max_n5 + BLAS_BLOCK - 1) / BLAS_BLOCK), (unsigned)nsys), blk(BLAS_BLOCK);
#define MOBIUS_L(K) hipLaunchKernelGGL(K, grid, blk, 0, st, sys_dev, active)
#define MOBIUS_P3(KT)                                                                   \
    switch (prec) {                                                                     \
    case MOBIUS_F64: MOBIUS_L((KT<MOBIUS_F64>)); break;                                 \
    case MOBIUS_F32: MOBIUS_L((KT<MOBIUS_F32>)); break;                                 \
    case MOBIUS_F16: MOBIUS_L((KT<MOBIUS_F16>)); break;                                 \
    default: return hipErrorInvalidValue;                                               \
    }
    switch (kind) {
    case VEC_AXPBY:
        switch (prec) {
        case MOBIUS_F64: MOBIUS_L((axpby_batch<MOBIUS_F64, false>)); break;
        case MOBIUS_F32: MOBIUS_L((axpby_batch<MOBIUS_F32, false>)); break;
        case MOBIUS_F16: MOBIUS_L((axpby_batch<MOBIUS_F16, false>)); break;
        default: return hipErrorInvalidValue;
        }
        break;
    case VEC_AXPBY_NORM:
        switch (prec) {
        case MOBIUS_F64: MOBIUS_L((axpby_batch<MOBIUS_F64, true>)); break;
        case MOBIUS_F32: MOBIUS_L((axpby_batch<MOBIUS_F32, true>)); break;
        case MOBIUS_F16: MOBIUS_L((axpby_batch<MOBIUS_F16, true>)); break;
        default: return hipErrorInvalidValue;
        }
        break;
    case VEC_NORM2: MOBIUS_P3(norm2_batch) break;
    case VEC_DOT: MOBIUS_P3(dot_batch) break;
    case VEC_XFLUSH:
        if (prec == MOBIUS_F64 && prec2 == MOBIUS_F64) MOBIUS_L((xflush_batch<MOBIUS_F64, MOBIUS_F64>));
        else if (prec == MOBIUS_F32 && prec2 == MOBIUS_F32) MOBIUS_L((xflush_batch<MOBIUS_F32, MOBIUS_F32>));
        else if (prec == MOBIUS_F16 && prec2 == MOBIUS_F32) MOBIUS_L((xflush_batch<MOBIUS_F16, MOBIUS_F32>));
        else return hipErrorInvalidValue;
        break;
    case VEC_ACCUMULATE: MOBIUS_P3(accumulate_batch) break;
    case VEC_CONVERT:
#define MOBIUS_CV(PI)                                                                   \
    switch (prec2) {                                                                    \
    case MOBIUS_F64: MOBIUS_L((convert_batch<PI, MOBIUS_F64>)); break;                  \
    case MOBIUS_F32: MOBIUS_L((convert_batch<PI, MOBIUS_F32>)); break;                  \
    case MOBIUS_F16: MOBIUS_L((convert_batch<PI, MOBIUS_F16>)); break;                  \
    default: return hipErrorInvalidValue;                                               \
    }
        switch (prec) {
        case MOBIUS_F64: MOBIUS_CV(MOBIUS_F64) break;
        case MOBIUS_F32: MOBIUS_CV(MOBIUS_F32) break;
        case MOBIUS_F16: MOBIUS_CV(MOBIUS_F16) break;
        default: return hipErrorInvalidValue;
        }
#undef MOBIUS_CV
        break;
    default: return hipErrorInvalidValue;
    }
#undef MOBIUS_P3
#undef MOBIUS_L
    return hipGetLastError();
}

hipError_t launch_reduce_batch(const VecSys *sys_dev, int nsys, const int32_t *active,
                               int64_t count_override, double *out, int64_t out_stride,
                               hipStream_t st)
{
    hipLaunchKernelGGL(reduce_batch, dim3(nsys), dim3(1024), 0, st, sys_dev, active, count_override,
                       out, out_stride);
    return hipGetLastError();
}

hipError_t launch_rupd_m5inv_batch(int prec, const VecSys *sys_dev, int nsys, int64_t max_blocks,
                                   const int32_t *active, int32_t *restart, int slot, int mode, hipStream_t st)
{
    if (slot >= RING_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)max_blocks, (unsigned)nsys), blk(BLOCK);
    switch (prec) {
    case MOBIUS_F64: hipLaunchKernelGGL(rupd_m5inv_batch<MOBIUS_F64>, grid, blk, 0, st, sys_dev, active, restart, slot, mode); break;
    case MOBIUS_F32: hipLaunchKernelGGL(rupd_m5inv_batch<MOBIUS_F32>, grid, blk, 0, st, sys_dev, active, restart, slot, mode); break;
    case MOBIUS_F16: hipLaunchKernelGGL(rupd_m5inv_batch<MOBIUS_F16>, grid, blk, 0, st, sys_dev, active, restart, slot, mode); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_reduce_parts(const VecSys *sys_dev, int nsys, const int32_t *active, double *out,
                               hipStream_t st)
{
    hipLaunchKernelGGL(reduce_parts_batch, dim3(RED_PARTS, (unsigned)nsys), dim3(BLAS_BLOCK), 0, st, sys_dev,
                       active, out);
    return hipGetLastError();
}

hipError_t launch_clear_alpha(CgScalars *sc, int nsys, const int32_t *active, hipStream_t st)
{
    hipLaunchKernelGGL(clear_alpha_batch, dim3((nsys + 63) / 64), dim3(64), 0, st, sc, nsys, active);
    return hipGetLastError();
}

hipError_t launch_cg_update(int kind, int prec, int prec2, const VecSys *sys_dev, int nsys, int64_t max_n5,
                            const int32_t *active, int32_t *restart, int slot, int prev, hipStream_t st)
{
    const dim3 grid((unsigned)((max_n5 + BLAS_BLOCK - 1) / BLAS_BLOCK), (unsigned)nsys), blk(BLAS_BLOCK);
    if (slot >= RING_MAX || prev >= RING_MAX) return hipErrorInvalidValue;
#define MOBIUS_PX(K, ...)                                                               \
    if (prec == MOBIUS_F64 && prec2 == MOBIUS_F64)                                      \
        hipLaunchKernelGGL((K<MOBIUS_F64, MOBIUS_F64>), grid, blk, 0, st, __VA_ARGS__); \
    else if (prec == MOBIUS_F32 && prec2 == MOBIUS_F32)                                 \
        hipLaunchKernelGGL((K<MOBIUS_F32, MOBIUS_F32>), grid, blk, 0, st, __VA_ARGS__); \
    else if (prec == MOBIUS_F16 && prec2 == MOBIUS_F32)                                 \
        hipLaunchKernelGGL((K<MOBIUS_F16, MOBIUS_F32>), grid, blk, 0, st, __VA_ARGS__); \
    else                                                                                \
        return hipErrorInvalidValue
    switch (kind) {
    case VEC_CG_XR: MOBIUS_PX(cg_xr_batch, sys_dev, active, restart, slot); break;
    case VEC_PUPD_X: MOBIUS_PX(pupd_x_batch, sys_dev, active, restart); break;
    case VEC_PUPD_RING:
        if (slot < 0 || prev < 0) return hipErrorInvalidValue;
        switch (prec) {
        case MOBIUS_F64: hipLaunchKernelGGL(pupd_ring_batch<MOBIUS_F64>, grid, blk, 0, st, sys_dev, active, restart, slot, prev); break;
        case MOBIUS_F32: hipLaunchKernelGGL(pupd_ring_batch<MOBIUS_F32>, grid, blk, 0, st, sys_dev, active, restart, slot, prev); break;
        case MOBIUS_F16: hipLaunchKernelGGL(pupd_ring_batch<MOBIUS_F16>, grid, blk, 0, st, sys_dev, active, restart, slot, prev); break;
        default: return hipErrorInvalidValue;
        }
        break;
    default: return hipErrorInvalidValue;
    }
#undef MOBIUS_PX
    return hipGetLastError();
}

hipError_t launch_xring(int prec, int prec2, const VecSys *sys_dev, int nsys, int64_t max_n5,
                        const int32_t *active, int n, hipStream_t st)
{
    const dim3 grid((unsigned)((max_n5 + BLAS_BLOCK - 1) / BLAS_BLOCK), (unsigned)nsys), blk(BLAS_BLOCK);
    if (n < 1 || n > RING_MAX || prec2 != MOBIUS_F32) return hipErrorInvalidValue;
    switch (prec) {
    case MOBIUS_F32: hipLaunchKernelGGL((xring_batch<MOBIUS_F32, MOBIUS_F32>), grid, blk, 0, st, sys_dev, active, n); break;
    case MOBIUS_F16: hipLaunchKernelGGL((xring_batch<MOBIUS_F16, MOBIUS_F32>), grid, blk, 0, st, sys_dev, active, n); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#endif  // MOBIUS_HOP_PREC

}  // namespace mobius
