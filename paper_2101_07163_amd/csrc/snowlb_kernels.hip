// snowlb_kernels.hip -- gfx950 kernels of the coupled lattice-Boltzmann ice-growth step
// (Tan et al., arXiv:2101.07163).
//
// k_step fuses, per lattice cell, the three LB updates of one time step:
//   flow   : D2Q9 BGK with the solid drag force and the velocity projection (Sec. 2.2.1),
//   vapour : D2Q5 advection-diffusion-reaction with the depletion source (Sec. 2.2.2),
//   phase  : the capacity-form LB of Eq. (d) with the equilibrium of Eq. (e) (Sec. 2.2.3),
// with an isotropic gradient of Table 1 (Sec. 3.1.1; E4 by default, or E2, E6, E8) and the anisotropy of
// Sec. 2.1.
//
// The step is bound by HBM bandwidth (about 2 flop per byte against a balance of about 20), so the
// kernel is built around memory traffic: every population is read once and written once per step,
// and a 64 x 4 tile's populations are one contiguous run of memory (planes side by side per block,
// see cell_index).  The only neighbour data the step needs -- phi at the eight neighbours
// (gradient) and h_q at x + c_q (the destination term of Eq. (d)) -- is staged in LDS from a
// halo of the 9 h planes (one cell wide, two for E6/E8), so halo re-reads hit LDS/L2 instead of HBM.
//
// Streaming is "push": Eq. (d) evaluates a_s^2 at the source node and needs the destination's own
// pre-collision h_q(x + c_q, t), so each cell writes h'_q(x + c_q) = P_q(x) - B(x) h_q(x + c_q, t),
// with P_q = h*_q / a^2 and B = (1 - a^2)/a^2.  Every (destination, q) pair is written by exactly one
// thread, so there is no race.
//
// The storage formats (FP32, or 16-bit deviations from local references) are described with their
// policies in snowlb_device.h.  Set-up, read-out, population exchange and diagnostics kernels are in
// snowlb_io.hip.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "snowlb_device.h"
#include "snowlb_internal.h"

namespace snowlb {

// The y part of cell_index with a full-rate 24-bit multiply (v_mul_u32_u24): every lattice the host
// accepts has fewer than 2^14 block rows and a block-row stride (64 nbx nq) below 2^24 elements, and its
// offsets below 2^32.
__device__ __forceinline__ uint32_t cell_ypart24(int nbx, int nq, int y) {
    return __umul24((uint32_t)(y >> 2), ((uint32_t)nbx * (uint32_t)nq) << 8) + ((uint32_t)(y & 3) << 6);
}

// i mod n for a staged position, -span < i < n + span: one add or subtract, except on lattices smaller
// than the staged region (a uniform branch, n is the same for the whole workgroup).
__device__ __forceinline__ int wrap_near(int i, int n, int span) {
    if (i < 0) i += n;
    if (i >= n) i -= n;
    if (__builtin_expect(n < span, 0)) i = ((i % n) + n) % n;
    return i;
}

// ---------------------------------------------------------------------------------------------
// the fused step; RAD is the reach of the gradient stencil (1: E2, E4; 2: E6, E8), i.e. the width of
// the halo ring staged in LDS
// Occupancy floor: four waves per SIMD (at most 128 VGPRs) for the one-cell-reach tiles at least
// four rows high, which fit without spilling; the others keep the compiler's own choice.
template <int TY, int RAD>
constexpr int kMinWaves = (RAD == 1 && TY >= 4) ? 4 : 1;

// LOOP: a persistent grid whose workgroups take several tiles (else grid == ntiles).  The scalar arguments come
// first and in this order because the first 14 words are preloaded into scalar registers: with the tile
// computed instead of read from a list, a workgroup then waits for one scalar load (its descriptor) before
// its first vector load, where argument, list and descriptor loads in turn were five (701 x 499 14.2 ->
// 12.5 us, 128^2 without flow 4.0 -> 3.7 us, together with the loads in one block below).
template <int TX, int TY, class S, bool FLOW, bool INOUT, int RAD, bool LOOP>
__global__ void __launch_bounds__(TX * TY) __attribute__((amdgpu_waves_per_eu(kMinWaves<TY, RAD>)))
k_step(const DomDesc* __restrict__ doms, const TileDesc* __restrict__ tiles, int flags, int grid, int ntx, int strip,
       int per, uint32_t m_per, uint32_t m_strip, uint32_t m_last, uint32_t codes, int ntiles) {
    using T = typename S::T;
    constexpr bool REF = S::kLocalRef;
    constexpr int NR = REF ? (FLOW ? 4 : 1) : 1;  // reference planes staged in LDS
    constexpr int NT = TX * TY;
    constexpr int LX = TX + 2 * RAD, LY = TY + 2 * RAD, LN = LX * LY;
    constexpr int RING = LN - NT;
    constexpr int PF = 0, PG = FLOW ? 9 : 0, PH = PG + 5;  // first plane of f, g and h in a copy
    constexpr int NP = (FLOW ? 23 : 14) + (REF ? NR : 0);  // planes per block of a copy (d.nqb)
    constexpr int PR = FLOW ? 23 : 14;                      // first 16-bit reference plane
    constexpr uint32_t ES = sizeof(T);
    // Planes follow each other PB bytes apart, so one scalar base in the middle of GP planes reaches all of them with
    // the 13-bit immediate offsets of the memory instructions; a base per access is two scalar additions each
    // (FP32 inlet instance: 478 scalar instructions, 292 so; 128^2 without flow 3.7 -> 3.6 us).
    constexpr int PB = kBlockCells * ES, GP = 8192 / PB, NG = (NP + GP - 1) / GP;
    __shared__ double s_phi[LN];
    __shared__ float s_phif[REF ? LN : 1];  // phi(t) rounded to FP32: the h references
    __shared__ float s_h[8][LN];            // h_1 .. h_8 (h_0 moves nowhere)
    __shared__ float s_ref[NR][REF ? LN : 1];
    // A wave of a tile at least 64 cells wide lies in one row: its y and everything made of it is uniform, and an
    // access is a scalar base (plane and row) plus one of three lane offsets (x, x + 1, x - 1).
    constexpr bool ROWS = TX % 64 == 0;
    auto uniform = [](int v) { return ROWS ? __builtin_amdgcn_readfirstlane(v) : v; };

    const int tid = threadIdx.x;
    const int tx = tid % TX, ty = uniform(tid / TX);
    const int own = (ty + RAD) * LX + (tx + RAD);
    const int par = flags & 1, npar = 1 - par;

    // XCD-aware order: consecutive workgroup ids are spread over the 8 XCDs; give each
    // XCD a contiguous run of tiles so neighbouring tiles share halo lines in that XCD's L2.  XCD x
    // receives G/8 workgroups, one more for x < G % 8; its runs follow each other in x order, so the
    // mapping is a permutation of the grid for any G.  Every other step (input copy 1) walks each run
    // backwards: a step then starts on the tiles the previous one wrote last, whose populations are
    // still in the last-level cache.
    const int G = grid;
    const int b = blockIdx.x;
    const int xcd = b % 8, kx = b / 8, cnt = G / 8 + (xcd < G % 8 ? 1 : 0);
    const int slot = xcd * (G / 8) + min(xcd, G % 8) + (par ? cnt - 1 - kx : kx);

    // The halo ring: lane tid takes its positions tid, tid + NT, ... (ring_at below).
    constexpr int RROWS = 2 * RAD * TX, SLOTS = (RING + NT - 1) / NT;

    for (int t = slot; !LOOP || t < ntiles; t += G) {
        int dom = 0, x0, y0;
        if (tiles) {
            const TileDesc td = tiles[t];
            dom = td.dom;
            x0 = td.x0;
            y0 = td.y0;
        } else {
            StepGeom geo;
            geo.ntx = ntx;
            geo.strip = strip;
            geo.per = per;
            geo.m_per = m_per;
            geo.m_strip = m_strip;
            geo.m_last = m_last;
            geo.codes = codes;
            int ti, tj;
            geo.tile_at(t, ti, tj);
            x0 = ti * TX;
            y0 = tj * TY;
        }
        const DomDesc& d = doms[dom];
        const int nx = d.nx, ny = d.ny, nbx = d.nbx;
        const GMEM char* pin = (const GMEM char*)d.pop[par];
        GMEM char* pout = (GMEM char*)d.pop[npar];
        const GMEM char* phin = (const GMEM char*)d.phip[par];
        GMEM char* phout = (GMEM char*)d.phip[npar];
        if constexpr (!FLOW && !REF) {  // step of an adjoint tape (bits 2.. of flags)
            const int64_t at = (int64_t)(flags >> 2) * d.slot_stride;
            pin += at;
            pout += at;
            phin += at;
            phout += at;
        }

        const int x = x0 + tx, y = y0 + ty;
        const bool active = (x < nx) && (y < ny);
        // byte offsets into the population buffer of a row and of a position in it (the 16-bit reference planes
        // share its blocks), and into the phi_prev plane
        auto yof = [&](int sy) { return cell_ypart24(nbx, NP, sy) * ES; };
        auto xof = [&](int sx) { return cell_xpart(sx, NP) * ES; };
        auto yof1 = [&](int sy) { return cell_ypart24(nbx, 1, sy) * 4u; };
        auto xof1 = [&](int sx) { return cell_xpart(sx, 1) * 4u; };
        // A row of the input copy: its group bases (the row's own offset in them, or, where a wave spans rows, in the
        // lane's), and the value of plane p at lane offset xo.  The empty asm keeps the compiler from taking
        // the bases apart again.
        struct Row {
            const GMEM char* base[NG];
            uint32_t lane;
            __device__ __forceinline__ T get(int p, uint32_t xo) const {
                return *(const GMEM T*)(base[p / GP] + (lane + xo) + (p % GP - GP / 2) * PB);
            }
        };
        auto row_of = [&](bool rows, uint32_t yo, int first, int last) {  // of the planes first..last
            Row r;
            r.lane = rows ? 0u : yo;
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (g >= first / GP && g <= last / GP) {
                    r.base[g] = pin + (rows ? yo : 0u) + (g * GP + GP / 2) * PB;
                    asm("" : "+s"(r.base[g]));
                }
            return r;
        };
        auto load1 = [&](bool rows, uint32_t yo, uint32_t xo) {  // phi_prev
            return rows ? gld<float>(phin + yo, xo) : gld<float>(phin, yo + xo);
        };
        // closure of a staged position: y periodic; x periodic, or (inlet/outlet) clamped -- the outlet repeats
        // column nx - 1, the inlet ghost is masked where it can occur
        auto cy = [&](int gy) { return wrap_near(gy, ny, LY); };
        auto cx = [&](int gx) { return INOUT ? min(max(gx, 0), nx - 1) : wrap_near(gx, nx, LX); };

        // ---- issue every global load of this tile first: the cell's own h, phi_prev (and 16-bit references), g
        // and f, which are one contiguous run per workgroup, then the halo ring.  The loads are
        // unconditional, so that they form one block and nothing is computed before the last is issued.  The
        // ring before f and g lets the staging start earlier (1024^2 FP32 30.6 instead of 30.8 us) but
        // splits the run, which costs HBM-sized lattices 1.8 % (2048^2 149.5 against 146.7 us); h before g and
        // f, kept apart from them, is worth 2 % on small lattices (256^2 4.7 -> 4.6 us).
        // A lane up to RAD cells outside the domain stages the h of the position its LDS slot stands for, the halo of an
        // active neighbour.  What an idle lane stages further out and its g and f are read by nobody: they
        // come from the last column and row, whose lines the active lanes load anyway (from the position the
        // closure maps the lane to they were lines of the far side: 16001 x 5 with flow 8.4 -> 6.7 us, 65 x 20001
        // 79.8 -> 73.2, habit batch of 400^2 22.0 -> 21.8; a branch around them costs full tiles 2 to 4 %).
        T graw[5], fraw[9], hraw[9], rraw[SLOTS][9];
        T oref[NR], rref[SLOTS][NR];
        float rphi[SLOTS];  // phi_prev of the staged ring positions
        const int px = x - nx, py = y - ny;
        const int osx = px < 0 ? x : (!INOUT && px < RAD ? px : nx - 1), osy = py < 0 ? y : (py < RAD ? py : ny - 1);
        const uint32_t xg = xof(min(x, nx - 1));
        const uint32_t xo = xof(osx), yo = yof(osy), xo1 = xof1(osx), yo1 = yof1(osy);
        const Row own_row = row_of(ROWS, yo, 0, NP - 1);
#pragma unroll
        for (int q = 0; q < 9; ++q) hraw[q] = own_row.get(PH + q, xo);
        const float ophi = load1(ROWS, yo1, xo1);
        if (REF) {
#pragma unroll
            for (int k = 0; k < NR; ++k) oref[k] = own_row.get(PR + k, xo);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 5; ++q) graw[q] = own_row.get(PG + q, xg);
        __builtin_amdgcn_sched_barrier(0);
        if (FLOW) {
#pragma unroll
            for (int q = 0; q < 9; ++q) fraw[q] = own_row.get(PF + q, xg);
        }
        // Ring position r in the staged region.  One cell wide: the rows below and above the tile, corners included,
        // then the columns.  Two cells wide: the four rows of TX cells, aligned like the tile's own (a wave's
        // share lies in one row; returns true), then the four columns of LY cells; all passes over it are
        // loaded here, up front (800^2 E8 16.3 -> 15.2 us).  The aligned form of the narrow ring is slower
        // (701 x 499 12.9 instead of 12.6 us, 1024^2 30.9 instead of 30.7).
        auto ring_at = [&](int r, int& lx, int& ly) {
            if constexpr (RAD == 1) {
                const bool above = r >= LX, column = r >= 2 * LX, right = r >= 2 * LX + TY;
                const int kr = above ? r - LX : r, kc = r - 2 * LX - (right ? TY : 0);
                lx = column ? (right ? LX - 1 : 0) : kr;
                ly = column ? 1 + kc : (above ? LY - 1 : 0);
                return false;
            } else {
                static_assert(RROWS % 64 == 0 && RROWS + 2 * RAD * LY == RING, "ring");
                const int k = uniform(r) / TX, c = r - RROWS, col = c / LY;
                const bool in_rows = uniform(r) < RROWS;
                ly = in_rows ? (k < RAD ? k : k + TY) : c - col * LY;
                lx = in_rows ? RAD + r % TX : (col < RAD ? col : col + TX);
                return ROWS && in_rows;
            }
        };
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) {
            const int r = tid + sl * NT;
            if (r < RING) {
                int lx, ly;
                const bool uni = ring_at(r, lx, ly);  // a uniform row: its offset goes to the scalar bases
                const int sx = cx(x0 + lx - RAD), sy = cy(y0 + ly - RAD);
                const uint32_t ry = yof(sy), ry1 = yof1(sy);
                const uint32_t by = uni ? __builtin_amdgcn_readfirstlane(ry) : 0u;
                const uint32_t by1 = uni ? __builtin_amdgcn_readfirstlane(ry1) : 0u;
                uint32_t rx = xof(sx) + (uni ? 0u : ry);
                asm("" : "+v"(rx));
                const Row row = row_of(true, by, PH, NP - 1);
#pragma unroll
                for (int q = 0; q < 9; ++q) rraw[sl][q] = row.get(PH + q, rx);
                if (REF) {
                    rphi[sl] = gld<float>(phin + by1, xof1(sx) + (uni ? 0u : ry1));
#pragma unroll
                    for (int k = 0; k < NR; ++k) rref[sl][k] = row.get(PR + k, rx);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // Decode h of one staged position and write phi and the 16-bit references to LDS.  phi is
        // summed in FP64: it is close to -1 or 1 in the bulk, and a gradient of FP32 sums would
        // carry cancellation error of order 1e-7 / |grad phi| into the direction of the normal, i.e.
        // into a and N where |grad phi| is small.  h is stored against its holder's phi_prev.
        auto stage = [&](bool ghost, const T raw[9], float href, const T refs[NR], int li, float hh[9]) {
            double p64 = 0.0;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                hh[q] = S::dec(raw[q], W9[q], href);
                p64 += (double)hh[q];
            }
            if (INOUT && ghost) p64 = -1.0;  // inlet ghost: phi = -1 (its h are never used)
            s_phi[li] = p64;
            if (REF) {
                s_phif[li] = (float)p64;
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    const float gv = k == R_U ? d.U_in : k == R_RHO ? d.ref_f : k == R_JX ? d.ref_f * d.u_in : 0.f;
                    s_ref[k][li] = S::from_ref(INOUT && ghost ? S::to_ref(gv) : refs[k]);
                }
            }
        };
        float h[9];
        stage(false, hraw, ophi, oref, own, h);
#pragma unroll
        for (int q = 1; q < 9; ++q) s_h[q - 1][own] = h[q];
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) {
            const int r = tid + sl * NT;
            if (r < RING) {
                int lx, ly;
                ring_at(r, lx, ly);
                const int li = ly * LX + lx;
                float hr[9];
                stage(x0 + lx - RAD < 0, rraw[sl], rphi[sl], rref[sl], li, hr);
#pragma unroll
                for (int q = 1; q < 9; ++q) s_h[q - 1][li] = hr[q];
            }
        }
        __syncthreads();

        if (active) {
            const float phip = ophi;  // phi(t-1) of this cell
            // ---- vapour and flow populations (16-bit: references of their source cells)
            float g[5], f[9];
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                float m = 0.f;
                if (REF) {
                    const int ls = own - CY[q] * LX - CX[q];
                    m = FLOW ? g_ref(s_ref[R_U][ls], s_ref[R_JX][ls], s_ref[R_JY][ls], CX[q], CY[q]) : s_ref[R_U][ls];
                }
                g[q] = S::dec(graw[q], W5[q], m);
            }
            if (FLOW) {
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    float m = 0.f;
                    if (REF) {
                        const int ls = own - CY[q] * LX - CX[q];
                        m = f_ref(s_ref[R_RHO][ls], s_ref[R_JX][ls], s_ref[R_JY][ls], CX[q], CY[q]);
                    }
                    f[q] = f_dev_dec<S>(fraw[q], q, m);  // f_q - w_q
                }
            }
            // FP32 storage closes the zeroth and first moments of each collision exactly (below): the
            // sums of the incoming populations are then taken in FP64, where a sum of a few FP32 values
            // is exact.  In uniform streams every cell rounds the same numbers the same way, so
            // independent roundings of each population add up coherently into a drift of the
            // pressure level and of the species; with the moments closed, the collision changes them
            // by one rounding of a small population only.  16-bit storage rounds every population to
            // 16 bits afterwards anyway and keeps the cheaper FP32 sums.
            constexpr bool EXACT = !REF;
            const double U64 = EXACT ? (((double)g[0] + (double)g[1]) + ((double)g[2] + (double)g[3])) + (double)g[4] : 0.0;
            const float U = EXACT ? (float)U64 : (g[0] + g[1]) + (g[2] + g[3]) + g[4];

            // ---- isotropic gradient (Sec. 3.1.1): sum over the stencil of w(|c|^2) phi(x + c) c with
            // the Table 1 weights (E4: 1/3 on axis neighbours, 1/12 on diagonals; no 1/cs^2), or the
            // central difference (E2: 1/2, 0), in FP64
            const double phi64 = s_phi[own];
            const float phi = (float)phi64;
            const double* P = s_phi + own;
            const double pE = P[1], pW = P[-1], pN = P[LX], pS = P[-LX];
            const double pNE = P[LX + 1], pNW = P[LX - 1], pSW = P[-LX - 1], pSE = P[-LX + 1];
            double gx64 = d.gw[0] * (pE - pW) + d.gw[1] * ((pNE - pNW) + (pSE - pSW));
            double gy64 = d.gw[0] * (pN - pS) + d.gw[1] * ((pNE + pNW) - (pSE + pSW));
            if constexpr (RAD == 2) {
                // E6 / E8: the layers |c|^2 = 4 (2, 0), 5 (2, 1) and (1, 2), and 8 (2, 2)
                auto Q = [&](int i, int j) { return P[j * LX + i]; };
                const double w4 = d.gw[2], w5 = d.gw[3], w8 = d.gw[4];
                gx64 += 2.0 * w4 * (Q(2, 0) - Q(-2, 0)) +
                        w5 * (2.0 * ((Q(2, 1) - Q(-2, 1)) + (Q(2, -1) - Q(-2, -1))) +
                              ((Q(1, 2) - Q(-1, 2)) + (Q(1, -2) - Q(-1, -2)))) +
                        2.0 * w8 * ((Q(2, 2) - Q(-2, 2)) + (Q(2, -2) - Q(-2, -2)));
                gy64 += 2.0 * w4 * (Q(0, 2) - Q(0, -2)) +
                        w5 * (2.0 * ((Q(1, 2) - Q(1, -2)) + (Q(-1, 2) - Q(-1, -2))) +
                              ((Q(2, 1) - Q(2, -1)) + (Q(-2, 1) - Q(-2, -1)))) +
                        2.0 * w8 * ((Q(2, 2) - Q(2, -2)) + (Q(-2, 2) - Q(-2, -2)));
            }
            const bool has_normal = gx64 * gx64 + gy64 * gy64 > d.grad_eps2;
            const float gx = (float)gx64, gy = (float)gy64;

            // ---- anisotropy a = 1 + eps cos(n theta) and flux N = kappa Dphi |g|^2 a da/dg, as
            // polynomials in the unit normal (theta-free, sign-free): with X = gx^2/|g|^2,
            // Y = gy^2/|g|^2, cos 6t = X^3 - 15 X^2 Y + 15 X Y^2 - Y^3,
            // sin 6t = (gx gy/|g|^2)(6 X^2 - 20 X Y + 6 Y^2), and d cos(nt)/dg = n sin(nt)(gy,-gx)/|g|^2.
            float a = 1.f, Nx = 0.f, Ny = 0.f;
            if (has_normal) {
                const float inv = 1.f / (gx * gx + gy * gy);
                const float X = gx * gx * inv, Y = gy * gy * inv, XY = gx * gy * inv;
                float Cn, Sn;
                if (d.n_fold == 6) {
                    Cn = X * X * X - 15.f * X * X * Y + 15.f * X * Y * Y - Y * Y * Y;
                    Sn = XY * (6.f * X * X - 20.f * X * Y + 6.f * Y * Y);
                } else {
                    Cn = X * X - 6.f * X * Y + Y * Y;
                    Sn = XY * 4.f * (X - Y);
                }
                a = 1.f + d.eps * Cn;
                const float c = d.aniso_coef * a * Sn;
                Nx = c * gy;
                Ny = -c * gx;
            }

            // ---- phase field, Eq. (d)/(e): relaxation eta = a^2 Dphi / cs^2 + 1/2, source Q / tau0
            const float a2 = a * a;
            const float ia2 = 1.f / a2;
            const float B = ia2 - 1.f;
            const float ieta = 1.f / (3.f * d.Dphi * a2 + 0.5f);
            const float om = 1.f - phi * phi;
            const float srcQ = (phi - phi * phi * phi + d.lam * U * om * om) * d.inv_tau0;

            // The FP32 lattice weights do not sum to one (float(1/3) + 4 float(1/6) = 1 + 3e-8), which
            // would make every collision a tiny systematic source of mass, vapour and phase.  Each
            // equilibrium and source therefore takes its rest population as the remainder of the moving
            // ones, so that the zeroth moments close exactly in real arithmetic and only unbiased
            // rounding is left.

            // ---- flow: drag and projection, Guo forcing, 2nd-order equilibrium (Sec. 2.2.1), all in
            // deviations from the weights: f holds f_q - w_q, drho = rho - 1, and
            // f_eq,q - w_q = w_q (drho + rho (3 c.u + 4.5 (c.u)^2 - 1.5 u.u))
            float ux = 0.f, uy = 0.f, rho = 0.f, jx = 0.f, jy = 0.f;
            float fs[9];
            if (FLOW) {
                double m64 = 0.0, jx64 = 0.0, jy64 = 0.0;
                float drho;
                if (EXACT) {
#pragma unroll
                    for (int q = 0; q < 9; ++q) m64 += (double)f[q];
                    jx64 = ((double)f[1] - (double)f[3]) + ((double)f[5] - (double)f[6]) + ((double)f[8] - (double)f[7]);
                    jy64 = ((double)f[2] - (double)f[4]) + ((double)f[5] + (double)f[6]) - ((double)f[7] + (double)f[8]);
                    drho = (float)m64;
                    jx = (float)jx64;
                    jy = (float)jy64;
                } else {
                    drho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
                    jx = (f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7]);
                    jy = (f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8]);
                }
                // drag k = h eta_f (1 + phi)^2 (1 - phi) / (4 W0^2) and the projected velocity
                // u = (1 - phi)/2 j / (rho + k/2).  FP32 storage takes this chain in FP64 from the FP64
                // moments: in FP32, rho u differs from j by a few ulps, by the same amount in every cell
                // of a uniform stream, and the momentum closure below would apply that difference as a
                // force on the whole stream at every step
                float k;
                double rho64 = 0.0, k64 = 0.0, ux64 = 0.0, uy64 = 0.0;
                if (EXACT) {
                    rho64 = 1.0 + m64;
                    const double pc64 = fmin(fmax(phi64, -1.0), 1.0);
                    k64 = (double)d.kdrag * (1.0 + pc64) * (1.0 + pc64) * (1.0 - pc64);
                    const double sc64 = 0.5 * (1.0 - pc64) / (rho64 + 0.5 * k64);
                    ux64 = jx64 * sc64;
                    uy64 = jy64 * sc64;
                    rho = (float)rho64;
                    k = (float)k64;
                    ux = (float)ux64;
                    uy = (float)uy64;
                } else {
                    rho = 1.f + drho;
                    const float pc = fminf(fmaxf(phi, -1.f), 1.f);
                    k = d.kdrag * (1.f + pc) * (1.f + pc) * (1.f - pc);
                    const float sc = 0.5f * (1.f - pc) / (rho + 0.5f * k);
                    ux = jx * sc;
                    uy = jy * sc;
                }
                const float uu = ux * ux + uy * uy;
                // BGK relaxation with the Guo term of F = -k u, written as relaxation toward a shifted
                // target: fs_q = f_q - omega (f_q - T_q) with T_q = f_eq,q - w_q + S_q / omega (exact in
                // real arithmetic; the difference f_q - T_q is small near equilibrium, so the update keeps
                // its accuracy in uniform streams).  T_q = w_q (A + Bc c.u + Cc (c.u)^2) with, for
                // G = (tau_f - 1/2) k = guo k / omega,
                //   A = drho - (1.5 rho - 3 G) u.u,  Bc = 3 (rho - G),  Cc = 4.5 rho - 9 G;
                // opposite velocities share w (A + Cc (c.u)^2) and differ in the sign of w Bc c.u; the
                // rest population takes the remainder of the moving ones
                const float omf = d.omega_f, G = d.tauf_m_half * k;
                const float A = drho - (1.5f * rho - 3.f * G) * uu;
                const float Bc = 3.f * (rho - G), Cc = 4.5f * rho - 9.f * G;
                float Tq[9];
                auto pair = [&](int q, int qb, float cu) {  // q along c, qb along -c
                    const float S0 = W9[q] * __builtin_fmaf(Cc * cu, cu, A), D = W9[q] * Bc * cu;
                    Tq[q] = S0 + D;
                    Tq[qb] = S0 - D;
                };
                pair(1, 3, ux);
                pair(2, 4, uy);
                pair(5, 7, ux + uy);
                pair(6, 8, uy - ux);
                Tq[0] = drho - sum8(Tq);
#pragma unroll
                for (int q = 0; q < 9; ++q) fs[q] = __builtin_fmaf(-omf, f[q] - Tq[q], f[q]);
                if (EXACT) {
                    // after collision the first moments are j - omega (j - rho u) + (1 - omega/2) F and the
                    // zeroth is unchanged (Guo forcing, Sec. 2.2.1): fs_1 and fs_2 take the first moments as
                    // remainders, then fs_0 the zeroth, with every sum in FP64
                    const double omd = d.omega_f, gud = d.guo;
                    const double px = jx64 - omd * (jx64 - rho64 * ux64) - gud * k64 * ux64;
                    const double py = jy64 - omd * (jy64 - rho64 * uy64) - gud * k64 * uy64;
                    fs[1] = (float)(px - ((-(double)fs[3] + (double)fs[5]) + ((double)fs[8] - (double)fs[6] - (double)fs[7])));
                    fs[2] = (float)(py - ((-(double)fs[4] + (double)fs[5]) + ((double)fs[6] - (double)fs[7] - (double)fs[8])));
                    double s64 = 0.0;
#pragma unroll
                    for (int q = 1; q < 9; ++q) s64 += (double)fs[q];
                    fs[0] = (float)(m64 - s64);
                }
            }

            // ---- vapour (Sec. 2.2.2): tau_g = 1/2 + (tau_vap - 1/2) q with q = clamp((1 - phi)/2, 0, 1),
            // or q = 1 in both phases for the symmetric (thermal) variant
            const float sq = d.sym ? 1.f : fminf(fmaxf(0.5f * (1.f - phi), 0.f), 1.f);
            const float itg = 1.f / (0.5f + d.tauv_m_half * sq);
            const float srcg = d.half_Lsat * (phi - phip);
            float gs[5];
            {
                // relaxation toward g_eq = w U (1 + 3 c.u) and the source share w srcg, gathered:
                //   gs_q = (1 - itg) g_q + w (itg U - srcg) + 3 w itg U c.u, rest as the remainder
                const float K = itg * U - srcg, G0 = W5[1] * K, G1 = 0.5f * itg * U;  // 3 w = 1/2
                const float Gx = G1 * ux, Gy = G1 * uy, itc = 1.f - itg;
                const float E1 = G0 + Gx, E3 = G0 - Gx, E2 = G0 + Gy, E4 = G0 - Gy;
                gs[1] = __builtin_fmaf(itc, g[1], E1);
                gs[2] = __builtin_fmaf(itc, g[2], E2);
                gs[3] = __builtin_fmaf(itc, g[3], E3);
                gs[4] = __builtin_fmaf(itc, g[4], E4);
                gs[0] = __builtin_fmaf(itc, g[0], K - ((E1 + E2) + (E3 + E4)));
                if (EXACT)  // the zeroth moment after collision is U - src: gs_0 as its remainder
                    gs[0] = (float)((U64 - (double)srcg) - (((double)gs[1] + (double)gs[2]) + ((double)gs[3] + (double)gs[4])));
            }

            // ---- phase field (Eq. d, e): relaxation toward h_eq = w (phi - 3 c.N) plus the source share
            // w srcQ, divided by a^2, gathered into Pq = ia2 (1 - ieta) h_q + ia2 (w K - 3 ieta w c.N)
            // with K = ieta phi + srcQ; opposite velocities share the first term of the bracket and
            // the rest population takes the remainder of the moving ones
            float HP[9];
            const float hc = ia2 * (1.f - ieta);
            {
                const float K = __builtin_fmaf(ieta, phi, srcQ), Ka = ia2 * K, Na = 3.f * ia2 * ieta;
                auto pair = [&](int q, int qb, float cN) {
                    const float S0 = W9[q] * Ka, D = W9[q] * Na * cN;
                    HP[q] = S0 - D;
                    HP[qb] = S0 + D;
                };
                pair(1, 3, Nx);
                pair(2, 4, Ny);
                pair(5, 7, Nx + Ny);
                pair(6, 8, Ny - Nx);
                // from the rounded Ka in every instance (the compiler would fuse its product into the difference
                // in some of them)
                float rest = Ka;
                asm("" : "+v"(rest));
                HP[0] = rest - sum8(HP);
            }

            // ---- destination rows y - 1, y, y + 1 of the output copy, as group bases and lane offsets
            const uint32_t yd[3] = {yof(y > 0 ? y - 1 : ny - 1), yo, yof(y + 1 < ny ? y + 1 : 0)};
            GMEM char* out[3][NG];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    out[k][g] = pout + (ROWS ? yd[k] : 0u) + (g * GP + GP / 2) * PB;
                    asm("" : "+s"(out[k][g]));
                }
            auto store = [&](int p, int dy, uint32_t xd, T v) {  // plane p, row y + dy, lane offset xd
                *(GMEM T*)(out[dy + 1][p / GP] + (ROWS ? xd : yd[dy + 1] + xd) + (p % GP - GP / 2) * PB) = v;
            };
            // ---- references this cell hands to the populations it emits (16-bit storage)
            float rU = 0.f, rR = 0.f, rJx = 0.f, rJy = 0.f;
            if (REF) {
                const T tU = S::to_ref(U);
                store(PR + R_U, 0, xo, tU);
                rU = S::from_ref(tU);
                if (FLOW) {
                    const T tR = S::to_ref(rho), tX = S::to_ref(jx), tY = S::to_ref(jy);
                    store(PR + R_RHO, 0, xo, tR);
                    store(PR + R_JX, 0, xo, tX);
                    store(PR + R_JY, 0, xo, tY);
                    rR = S::from_ref(tR);
                    rJx = S::from_ref(tX);
                    rJy = S::from_ref(tY);
                }
            }

            // ---- push streaming into copy 1 - par.  Population q goes to the lane offset xd of row y + c_y, where
            // h'_q takes h_q of the LDS position li.  On lattices of more than twice the last-level cache (bit 1 of
            // flags) FP32 waves pause 6 x 64 cycles before each direction's stores: all stores in one burst hold up the
            // loads of the CU's other workgroups (64-crystal batch 947 -> 900 us, 3000^2 331 -> 323, 2048^2 151
            // -> 148.5; pauses of 3 or 4 are worth less, 9 no more; without flow and in 16 bits they only cost).
            // Between one and two caches they cost too: 1300^2 (335 MB) 64.9 us, 61.9 without, 65 x 20001 (492 MB) 75.3 and
            // 73.4; from there on they pay (1750^2, 602 MB, 111.1 and 113.2).
            const bool paced = FLOW && !REF && (flags & 2);
            auto push = [&](int q, uint32_t xd, int li) {
                if (paced) __builtin_amdgcn_s_sleep(6);
                const float Pq = __builtin_fmaf(hc, h[q], HP[q]);
                const float hat = q == 0 ? h[0] : s_h[q == 0 ? 0 : q - 1][li];
                const float href = REF ? s_phif[li] : 0.f;  // h references its holder's phi(t)
                store(PH + q, CY[q], xd, S::enc(__builtin_fmaf(-B, hat, Pq), IW9[q], href));
                if (FLOW) {
                    const float fm = REF ? f_ref(rR, rJx, rJy, CX[q], CY[q]) : 0.f;
                    store(PF + q, CY[q], xd, f_dev_enc<S>(fs[q], q, fm));
                }
                if (q < 5) {
                    const float gm = REF ? (FLOW ? g_ref(rU, rJx, rJy, CX[q], CY[q]) : rU) : 0.f;
                    store(PG + q, CY[q], xd, S::enc(gs[q], IW5[q], gm));
                }
            };
            // the directions with the same c_x share a test of the domain's edge and a lane offset (opaque, so
            // that it stays a 32-bit offset of scalar bases in its block)
            auto opaque = [](uint32_t v) {
                asm("" : "+v"(v));
                return v;
            };
            const uint32_t xc = opaque(xo);
            push(0, xc, own);
            push(2, xc, own + LX);
            push(4, xc, own - LX);
            const bool last = x == nx - 1, first = x == 0;
            if (!(INOUT && last)) {
                const uint32_t xe = opaque(xof(last ? 0 : x + 1));
                push(1, xe, own + 1);
                push(5, xe, own + LX + 1);
                push(8, xe, own - LX + 1);
            }
            if (!(INOUT && first)) {
                const uint32_t xw = opaque(xof(first ? nx - 1 : x - 1));
                push(3, xw, own - 1);
                push(6, xw, own + LX - 1);
                push(7, xw, own - LX - 1);
            }
            if constexpr (INOUT) {
                if (last) {
                    // outlet ghost at x = nx is a copy of this column: it streams into (nx-1, y + cy)
                    const uint32_t xl = opaque(xo);
                    push(3, xl, own);
                    push(6, xl, own + LX);
                    push(7, xl, own - LX);
                }
                if (first) {
                    // inlet ghost at x = -1: equilibrium at (rho0, u_in; U_in; phi = -1); its reference values
                    // are the LDS ones of the ghost column
                    const uint32_t xf = opaque(xo);
                    auto inflow = [&](int q) {
                        const int lg = own - CX[q] - CY[q] * LX;  // the ghost source in the LDS halo
                        float gfm = 0.f, ggm = 0.f;
                        if constexpr (REF) {
                            ggm = g_ref(s_ref[R_U][lg], s_ref[R_JX][lg], s_ref[R_JY][lg], CX[q], CY[q]);
                            gfm = f_ref(s_ref[R_RHO][lg], s_ref[R_JX][lg], s_ref[R_JY][lg], CX[q], CY[q]);
                        }
                        store(PH + q, 0, xf, S::enc(-W9[q], IW9[q], REF ? phi : 0.f));
                        store(PF + q, 0, xf, f_dev_enc<S>(d.df_in[q], q, gfm));
                        if (q < 5) store(PG + q, 0, xf, S::enc(d.g_in[q], IW5[q], ggm));
                    };
                    inflow(1);
                    inflow(5);
                    inflow(8);
                }
            }
            gst<float>(phout + (ROWS ? yo1 : 0u), opaque(xo1 + (ROWS ? 0u : yo1)), phi);
        }
        if (!LOOP) break;
        __syncthreads();  // LDS is reused by the next tile
    }
}

// ---------------------------------------------------------------------------------------------
// tile configurations
struct TileCfg {
    int tx, ty;
    const char* name;
};
static constexpr TileCfg kTiles[] = {
    {64, 4, "64x4"}, {64, 8, "64x8"}, {128, 2, "128x2"}, {128, 4, "128x4"}, {64, 2, "64x2"}, {32, 8, "32x8"},
};
static constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
static_assert(kTiles[kTileTwoHigh].tx == 64 && kTiles[kTileTwoHigh].ty == 8 && kTiles[kTileTwoWide].tx == 128 &&
                  kTiles[kTileTwoWide].ty == 4, "the tiles that the default of 16-bit lattices names");

int tile_config_count() { return kNumTiles; }
const char* tile_config_name(int i) { return (i >= 0 && i < kNumTiles) ? kTiles[i].name : "?"; }
int tile_config_tx(int i) { return kTiles[i].tx; }
int tile_config_ty(int i) { return kTiles[i].ty; }

template <int TX, int TY, class S, bool FLOW, bool INOUT, int RAD>
static void* step_fn(bool loop) {
    return loop ? reinterpret_cast<void*>(&k_step<TX, TY, S, FLOW, INOUT, RAD, true>)
                : reinterpret_cast<void*>(&k_step<TX, TY, S, FLOW, INOUT, RAD, false>);
}

template <class S, bool FLOW, bool INOUT, int RAD>
static void* step_fn_tile(int cfg, bool loop) {
    switch (cfg) {
        case 0: return step_fn<64, 4, S, FLOW, INOUT, RAD>(loop);
        case 1: return step_fn<64, 8, S, FLOW, INOUT, RAD>(loop);
        case 2: return step_fn<128, 2, S, FLOW, INOUT, RAD>(loop);
        case 3: return step_fn<128, 4, S, FLOW, INOUT, RAD>(loop);
        case 4: return step_fn<64, 2, S, FLOW, INOUT, RAD>(loop);
        case 5: return step_fn<32, 8, S, FLOW, INOUT, RAD>(loop);
    }
    return nullptr;
}

template <class S, int RAD>
static void* step_fn_store(int cfg, int flow, int inout, bool loop) {
    if (!flow) return step_fn_tile<S, false, false, RAD>(cfg, loop);
    if (!inout) return step_fn_tile<S, true, false, RAD>(cfg, loop);
    return step_fn_tile<S, true, true, RAD>(cfg, loop);
}

template <int RAD>
static void* step_kernel_rad(int cfg, int storage, int flow, int inout, bool loop) {
    switch (storage) {
        case 0: return step_fn_store<StoreF32, RAD>(cfg, flow, inout, loop);
        case 1: return step_fn_store<StoreF16, RAD>(cfg, flow, inout, loop);
        case 2: return step_fn_store<StoreBF16, RAD>(cfg, flow, inout, loop);
    }
    return nullptr;
}

static void* step_kernel(int cfg, int storage, int flow, int inout, int rad, bool loop) {
    if (cfg < 0 || cfg >= kNumTiles) return nullptr;
    if (inout && !flow) return nullptr;
    if (rad == 1) return step_kernel_rad<1>(cfg, storage, flow, inout, loop);
    if (rad == 2) return step_kernel_rad<2>(cfg, storage, flow, inout, loop);
    return nullptr;
}

// Dynamic LDS that limits the waves per CU of an FP32 step whose lattices do not fit in the last-level cache: to 20
// with flow, 16 without.  The registers allow 28 to 32, and lattices in that cache are fastest with them (1024^2
// 30.7 us, 32.4 with 12; 701 x 499 12.6 and 14.5), but from HBM more tiles in flight than the L2 holds (4 MB per
// XCD, 47 KB per tile with flow) evict halo and partly written lines: 2048^2 with flow reads 9 % and writes 4 %
// more than with the limit and takes 159 us instead of 148 to 149 (3000^2 359 and 323; 12 waves 321, but the
// 64-crystal batch 960 instead of 900); without flow 2048^2 96.9, 92.9 with 16, 112.7 with 12.  16-bit storage
// keeps them all (2048^2 FP16 with 128 x 4 tiles 94.5 us, 97.9 with 16 waves, 100.0 with 8; 1024^2 with 64 x 4 tiles
// 21.7, 23.7 with 16).
static int step_lds_pad(int cfg, int flow, int rad) {
    const TileCfg& t = kTiles[cfg];
    const int limit = flow ? 20 : 16, waves = t.tx * t.ty / 64, used = (t.tx + 2 * rad) * (t.ty + 2 * rad) * 40 + 256;
    return std::max(0, std::min(65536, 163840 * waves / limit) - used);
}

// Persistent grid over `ntiles` tiles: one wave of resident workgroups that loops over the tiles, or a workgroup per tile if
// all are resident.
int step_grid(int cfg, int ntiles, int storage, int flow, int inout, int rad) {
    void* fn = step_kernel(cfg, storage, flow, inout, rad, true);
    if (!fn || ntiles <= 0) return 0;
    int per_cu = 0;
    const int nt = kTiles[cfg].tx * kTiles[cfg].ty;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), nt, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    int dev = 0, ncu = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    long g = (long)per_cu * ncu;
    if (g >= ntiles) return ntiles;
    g -= g % 8;  // a multiple of 8 keeps the XCD-contiguous order a permutation
    return (int)(g > 0 ? g : ntiles);
}

hipError_t launch_step(int cfg, int storage, int flow, int inout, int rad, const DomDesc* doms_dev,
                       const TileDesc* tiles_dev, const StepGeom& geom, int hbm, int par, hipStream_t s, int slot) {
    const bool loop = geom.grid < geom.ntiles;
    void* fn = step_kernel(cfg, storage, flow, inout, rad, loop);
    if (!fn) return hipErrorInvalidValue;
    if (geom.ntiles <= 0) return hipSuccess;
    const int nt = kTiles[cfg].tx * kTiles[cfg].ty;
    // The wave limit and the pauses are for workgroups that come and go: a persistent grid is the resident set, whose
    // workgroups neither of them helps (2048^2 FP32 175 us without, 191 with the limit, 184 with the pauses; 1600^2 104,
    // 113, 106).
    const bool thin = storage == 0 && hbm && !loop;
    StepGeom g = geom;
    int flags = par | (thin && hbm > 1 ? 2 : 0) | slot << 2;
    void* args[] = {(void*)&doms_dev, (void*)&tiles_dev, (void*)&flags, (void*)&g.grid, (void*)&g.ntx, (void*)&g.strip,
                    (void*)&g.per, (void*)&g.m_per, (void*)&g.m_strip, (void*)&g.m_last, (void*)&g.codes, (void*)&g.ntiles};
    return hipLaunchKernel(fn, dim3(g.grid), dim3(nt), args, thin ? step_lds_pad(cfg, flow, rad) : 0, s);
}

}  // namespace snowlb
