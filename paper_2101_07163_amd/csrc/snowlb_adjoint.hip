// snowlb_adjoint.hip -- hand-written discrete adjoint of the fused step (no flow, periodic, FP32).
//
// For a loss L(phi_T), the adjoint lambda_t = dL/d(state at t) obeys lambda_t = (dF/ds)^T lambda_{t+1}
// where F is one step of the phase field (Eq. (d)/(e), anisotropy of Sec. 2.1, E4 gradient of
// Table 1) and the vapour ADR solver (Sec. 2.2.2) with u = 0.  Each reverse step is one kernel,
// k_adj, over 64 x 16 or 64 x 8 tiles, in two passes:
//   pass A (per position p of the tile and of its one-cell ring): recompute the forward quantities of
//     p from the stored state at t (phi with its halo for the gradient, a, N, eta, Q, h_eq, h*), take
//     lambda_{t+1} of the populations p emitted (at p + c_q), and form every adjoint that is local to
//     p: lambda_g(p, t) and lambda_phiprev(p, t) completely, and for the h adjoint the per-cell
//     factors A_h = (1 - 1/eta)/a^2, B = (1 - a^2)/a^2, the adjoint of the gradient Gbar(p) and the
//     local part of phibar(p); the explicit dependence on eps is reduced into per-workgroup FP64
//     partials (tile cells only);
//   pass B (per cell x of the tile): lambda_h,q(x, t) = lambda_h,q(x + c_q) A_h(x)   [through h*_q(x)]
//                                     - B(x - c_q) lambda_h,q(x)      [destination term of Eq. (d)]
//                                     + phibar(x) + sum_k W_k c_k . Gbar(x - c_k)   [phi = sum h]
//     with B and Gbar of the neighbours taken from LDS.
// Layout: the state slot holds g_0..4 then h_0..8 in the populations' cell order (14 planes side by
// side per 64 x 4 block); lambda of g_0..4, h_0..8 uses the same order, lambda of phi_prev is a plane
// of its own.
#include <hip/hip_runtime.h>

#include <cstring>
#include <stdint.h>

#include "snowlb_internal.h"

namespace snowlb {

namespace {
__device__ constexpr int AX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int AY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__device__ constexpr float AW9[9] = {4.f / 9.f,  1.f / 9.f,  1.f / 9.f,  1.f / 9.f, 1.f / 9.f,
                                     1.f / 36.f, 1.f / 36.f, 1.f / 36.f, 1.f / 36.f};
__device__ constexpr float AW5[5] = {1.f / 3.f, 1.f / 6.f, 1.f / 6.f, 1.f / 6.f, 1.f / 6.f};

constexpr int ATX = 64, ALX = ATX + 2;  // tiles of 64 x ATY cells, with the one-cell ring ALX wide

// i mod n for any i (one add or subtract in the common case: neighbours and halos of wide lattices)
__device__ __forceinline__ int wrapn(int i, int n) {
    if (i < 0) i += n;
    if (i >= n) i -= n;
    if ((unsigned)i >= (unsigned)n) i = ((i % n) + n) % n;
    return i;
}

// The y part of cell_index with a full-rate 24-bit multiply: the host accepts lattices of at most
// 65536 x 65536 cells, i.e. fewer than 2^14 block rows and a block-row stride (64 nbx nq, nq <= 14)
// below 2^24 elements.
__device__ __forceinline__ uint32_t ypart24(int nbx, int nq, int y) {
    return __umul24((uint32_t)(y >> 2), ((uint32_t)nbx * (uint32_t)nq) << 8) + ((uint32_t)(y & 3) << 6);
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}
}  // namespace

// LDS slots of the one-cell ring around a tile: top row, bottom row, left column, right column.
template <int ATY>
__device__ __forceinline__ int ring_slot(int r) {
    constexpr int ALY = ATY + 2;
    if (r < ALX) return r;
    if (r < 2 * ALX) return (ALY - 1) * ALX + (r - ALX);
    if (r < 2 * ALX + ATY) return (1 + r - 2 * ALX) * ALX;
    return (1 + r - 2 * ALX - ATY) * ALX + ALX - 1;
}
// One reverse step is one kernel over 64 x 16 tiles (1024 lanes, one workgroup per CU) or 64 x 8 tiles (512 lanes,
// two per CU); the one-cell ring is 16 % or 29 % of the tile.  Pass B at a cell gathers B(x - c_q) and
// Gbar(x - c_k) from pass A at its eight neighbours, so each workgroup runs pass A on its tile and
// on the one-cell ring around it (the ring positions recomputed by both neighbouring workgroups
// from the same inputs with the same code, hence bitwise equal), which needs h and phi on a two-cell
// ring.  No intermediate plane goes through memory.
constexpr int L2X = ATX + 4;  // staging region: tile + two rings

// Byte offsets of a lattice position (wrapped into the periodic lattice) and of its eight
// neighbours, as separable x and y parts.
struct Nb {
    uint32_t xp, xE, xW, yp, yN, yS;
    __device__ __forceinline__ uint32_t at() const { return (xp + yp) * 4u; }
    __device__ __forceinline__ uint32_t dest(int q) const {
        return ((AX[q] > 0 ? xE : (AX[q] < 0 ? xW : xp)) + (AY[q] > 0 ? yN : (AY[q] < 0 ? yS : yp))) * 4u;
    }
};
__device__ __forceinline__ Nb nb_of(const AdjDesc& A, int gx, int gy) {
    Nb n;
    // the position wrapped once; its neighbours then step over at most one edge
    const int wx = wrapn(gx, A.nx), wy = wrapn(gy, A.ny);
    n.xp = cell_xpart(wx, kAdjPlanes);
    n.xE = cell_xpart(wx + 1 == A.nx ? 0 : wx + 1, kAdjPlanes);
    n.xW = cell_xpart(wx == 0 ? A.nx - 1 : wx - 1, kAdjPlanes);
    n.yp = ypart24(A.nbx, kAdjPlanes, wy);
    n.yN = ypart24(A.nbx, kAdjPlanes, wy + 1 == A.ny ? 0 : wy + 1);
    n.yS = ypart24(A.nbx, kAdjPlanes, wy == 0 ? A.ny - 1 : wy - 1);
    return n;
}

// Pass A at one position p: recompute the forward quantities of p from the staged h and phi (slot
// c2 of the staging region), then reverse the phase-field collision and push.  Always gives B(p) and
// Gbar(p); with FULL also reverses the vapour collision and push and gives lambda_g(p, t) (lgo),
// lambda_phiprev(p, t) (lppo), A_h(p), the local part of phibar(p) and the eps contribution of p.
template <bool FULL, int L2N>
__device__ __forceinline__ void pass_a(const AdjDesc& A, const double* s_phi, const float (*s_h)[L2N], int c2,
                                       const float g[5], const float lh[9], const float lg[5], float lpp,
                                       float& Bv, float& Gxb, float& Gyb, float& Ah, float& phb, double& deps,
                                       float lgo[5], float& lppo) {
    float h[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) h[q] = s_h[q][c2];
    const float phi = (float)s_phi[c2];
    // U as the forward step forms it in FP32 storage (an exact FP64 sum, rounded once)
    const float U = (float)((((double)g[0] + (double)g[1]) + ((double)g[2] + (double)g[3])) + (double)g[4]);

    // ---- forward recompute (as the step kernel)
    const double* S = s_phi + c2;
    const double gx64 = (1.0 / 3.0) * (S[1] - S[-1]) + (1.0 / 12.0) * ((S[L2X + 1] - S[L2X - 1]) + (S[-L2X + 1] - S[-L2X - 1]));
    const double gy64 = (1.0 / 3.0) * (S[L2X] - S[-L2X]) + (1.0 / 12.0) * ((S[L2X + 1] + S[L2X - 1]) - (S[-L2X + 1] + S[-L2X - 1]));
    const bool on = gx64 * gx64 + gy64 * gy64 > A.grad_eps2;
    const float gx = (float)gx64, gy = (float)gy64;
    float a = 1.f, Cn = 0.f, Sn = 0.f, c = 0.f, iG2 = 0.f;
    if (on) {
        iG2 = 1.f / (gx * gx + gy * gy);
        const float X = gx * gx * iG2, Y = gy * gy * iG2, XY = gx * gy * iG2;
        if (A.n_fold == 6) {
            Cn = X * X * X - 15.f * X * X * Y + 15.f * X * Y * Y - Y * Y * Y;
            Sn = XY * (6.f * X * X - 20.f * X * Y + 6.f * Y * Y);
        } else {
            Cn = X * X - 6.f * X * Y + Y * Y;
            Sn = XY * 4.f * (X - Y);
        }
        a = 1.f + A.eps * Cn;
        c = A.coefN * A.eps * a * Sn;
    }
    const float Nx = c * gy, Ny = -c * gx;
    const float a2 = a * a, ia2 = 1.f / a2, B = ia2 - 1.f;
    const float ie = 1.f / (3.f * A.Dphi * a2 + 0.5f);
    const float om = 1.f - phi * phi;
    const float Q = phi - phi * phi * phi + A.lam * U * om * om;

    // ---- reverse of the phase-field collision and push
    float ia2b = 0.f, Bb = 0.f, ieb = 0.f, Qb = 0.f, pb_ = 0.f, Nxb = 0.f, Nyb = 0.f;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const float Pb = lh[q];                          // lambda_h,q(p + c_q, t + 1)
        const float hold = s_h[q][c2 + AY[q] * L2X + AX[q]];  // h_q(p + c_q, t)
        const float heq = AW9[q] * (phi - 3.f * (AX[q] * Nx + AY[q] * Ny));
        const float hs = h[q] - (h[q] - heq) * ie + AW9[q] * Q * A.inv_tau0;
        Bb -= Pb * hold;
        ia2b += Pb * hs;
        const float hsb = Pb * ia2;
        ieb += hsb * (heq - h[q]);
        const float heqb = hsb * ie;
        Qb += hsb * AW9[q] * A.inv_tau0;
        pb_ += AW9[q] * heqb;
        Nxb -= 3.f * AW9[q] * heqb * AX[q];
        Nyb -= 3.f * AW9[q] * heqb * AY[q];
    }
    pb_ += Qb * (1.f - 3.f * phi * phi - 4.f * A.lam * U * phi * om);
    float Ub = Qb * A.lam * om * om;
    ia2b += Bb;
    const float a2b = -ia2 * ia2 * ia2b + 3.f * A.Dphi * (-ie * ie * ieb);
    float ab = 2.f * a * a2b;
    Gxb = 0.f;
    Gyb = 0.f;
    if (on) {
        const float cb = gy * Nxb - gx * Nyb;  // N = c (gy, -gx)
        Gxb += -c * Nyb;
        Gyb += c * Nxb;
        ab += A.coefN * A.eps * Sn * cb;
        const float Sb = A.coefN * A.eps * a * cb;
        if (FULL) deps = (double)(Cn * ab) + (double)(A.coefN * a * Sn * cb);
        const float Cb = A.eps * ab;
        const float m = (float)A.n_fold;
        Gxb += (Cb * m * Sn * gy - Sb * m * Cn * gy) * iG2;
        Gyb += (-Cb * m * Sn * gx + Sb * m * Cn * gx) * iG2;
    }
    Bv = B;
    if (!FULL) return;

    // ---- reverse of the vapour collision and push
    const float qd = 0.5f * (1.f - phi);
    const bool inside = qd > 0.f && qd < 1.f;
    const float itg = 1.f / (0.5f + A.tauv_m_half * fminf(fmaxf(qd, 0.f), 1.f));
    float itgb = 0.f, srcb = 0.f;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        itgb -= lg[q] * (g[q] - AW5[q] * U);
        Ub += AW5[q] * lg[q] * itg;
        srcb -= AW5[q] * lg[q];
    }
    pb_ += A.half_Lsat * srcb;
    if (inside) pb_ += -0.5f * A.tauv_m_half * (-itg * itg * itgb);
    pb_ += lpp;  // phi_prev(t + 1) = phi(t)
#pragma unroll
    for (int q = 0; q < 5; ++q) lgo[q] = lg[q] * (1.f - itg) + Ub;
    lppo = -A.half_Lsat * srcb;
    Ah = ia2 * (1.f - ie);
    phb = pb_;
}

template <int ATY>
__global__ void __launch_bounds__(ATX * ATY) k_adj(AdjDesc A) {
    constexpr int ANT = ATX * ATY, ALY = ATY + 2, ALN = ALX * ALY, L2Y = ATY + 4, L2N = L2X * L2Y;
    constexpr int RING1 = 2 * ALX + 2 * ATY;  // the one-cell ring
    static_assert(RING1 <= ANT, "one ring position per lane");
    __shared__ double s_phi[L2N];
    __shared__ float s_h[9][L2N];
    __shared__ float s_B[ALN], s_Gx[ALN], s_Gy[ALN];
    __shared__ double s_red[ANT / 64];
    const int tid = threadIdx.x, tx = tid % ATX, ty = tid / ATX;
    const int ntx = (A.nx + ATX - 1) / ATX;
    // tiles in XCD-contiguous order (workgroup ids are dealt round-robin to the 8 XCDs; each XCD gets
    // a contiguous run of tiles, so the halos of neighbouring tiles meet in its L2)
    const int G = gridDim.x, bid = blockIdx.x;
    const int tile = (bid % 8) * (G / 8) + min(bid % 8, G % 8) + bid / 8;
    const int x0 = (tile % ntx) * ATX, y0 = (tile / ntx) * ATY;
    const int x = x0 + tx, y = y0 + ty;
    const bool active = x < A.nx && y < A.ny;
    const uint64_t pb = (uint64_t)kBlockCells * 4;  // bytes between the planes of a block
    const GMEM char* st = (const GMEM char*)A.st;
    const GMEM char* lin = (const GMEM char*)A.lin;
    GMEM char* lout = (GMEM char*)A.lout;
    // this workgroup's eps partial of the later steps, loaded here rather than at the very end
    const double epart = tid == 0 ? A.epart[blockIdx.x] : 0.0;

    // ---- global loads before the barrier: what pass A on the tile needs.  Values used only later
    // (the ring's inputs, lambda_h(t + 1) of the cell itself for pass B) are loaded where they are
    // used, which keeps them out of the registers live across the staging: 105 VGPRs instead of
    // 123, and a backward pass about 9 % shorter.  This lane's own position (wrapped into the
    // lattice for lanes outside it: their slots are halo of active neighbours) ...
    const Nb on = nb_of(A, x, y);
    float g[5], lh[9], lg[5] = {}, lpp = 0.f;
#pragma unroll
    for (int q = 0; q < 5; ++q) g[q] = gld<float>(st + q * pb, on.at());
#pragma unroll
    for (int q = 0; q < 9; ++q) lh[q] = gld<float>(lin + (5 + q) * pb, on.dest(q));
    if (active) {
#pragma unroll
        for (int q = 0; q < 5; ++q) lg[q] = gld<float>(lin + q * pb, on.dest(q));
        lpp = gld<float>((const GMEM char*)A.lppin, (cell_xpart(x, 1) + ypart24(A.nbx, 1, y)) * 4u);
    }
    // ... the position of the one-cell ring this lane recomputes (pass A there needs g and
    // lambda_h(t + 1) only, loaded after the barrier) ...
    const bool has_ring = tid < RING1;
    const int r1 = has_ring ? ring_slot<ATY>(tid) : 0;  // slot in the (ALX x ALY) pass-A region
    const Nb rn = nb_of(A, x0 + r1 % ALX - 1, y0 + r1 / ALX - 1);
    // ... and h(t) with phi(t) = sum h (FP64, as in the forward step) on the tile and two rings
    for (int r = tid; r < L2N; r += ANT) {
        const int lx = r % L2X, ly = r / L2X;
        const uint32_t o =
            (cell_xpart(wrapn(x0 + lx - 2, A.nx), kAdjPlanes) + ypart24(A.nbx, kAdjPlanes, wrapn(y0 + ly - 2, A.ny))) * 4u;
        double p = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const float v = gld<float>(st + (5 + q) * pb, o);
            p += (double)v;
            s_h[q][r] = v;
        }
        s_phi[r] = p;
    }
    __syncthreads();

    // ---- pass A on the tile (every lane, at its wrapped position) and on the ring
    double deps = 0.0;
    float Ah = 0.f, phb = 0.f;
    {
        const int c2 = (ty + 2) * L2X + tx + 2, c1 = (ty + 1) * ALX + tx + 1;
        float lgo[5], lppo = 0.f, Bv, Gx, Gy;
        pass_a<true, L2N>(A, s_phi, s_h, c2, g, lh, lg, lpp, Bv, Gx, Gy, Ah, phb, deps, lgo, lppo);
        s_B[c1] = Bv;
        s_Gx[c1] = Gx;
        s_Gy[c1] = Gy;
        if (active) {
            const uint32_t io = on.at();
#pragma unroll
            for (int q = 0; q < 5; ++q) gst<float>(lout + q * pb, io, lgo[q]);
            gst<float>((GMEM char*)A.lppout, (cell_xpart(x, 1) + ypart24(A.nbx, 1, y)) * 4u, lppo);
        } else {
            deps = 0.0;
        }
    }
    if (has_ring) {
        float rg[5], rlh[9];
#pragma unroll
        for (int q = 0; q < 5; ++q) rg[q] = gld<float>(st + q * pb, rn.at());
#pragma unroll
        for (int q = 0; q < 9; ++q) rlh[q] = gld<float>(lin + (5 + q) * pb, rn.dest(q));
        const int c2 = (r1 / ALX + 1) * L2X + r1 % ALX + 1;
        float Bv, Gx, Gy, ah_, ph_, lgo[5], lppo;
        double de_ = 0.0;
        pass_a<false, L2N>(A, s_phi, s_h, c2, rg, rlh, rg, 0.f, Bv, Gx, Gy, ah_, ph_, de_, lgo, lppo);
        s_B[r1] = Bv;
        s_Gx[r1] = Gx;
        s_Gy[r1] = Gy;
    }
    __syncthreads();

    // ---- pass B: lambda_h,q(x, t) = lambda_h,q(x + c_q) A_h(x) - B(x - c_q) lambda_h,q(x)
    //                                + phibar(x) + sum_k W_k c_k . Gbar(x - c_k)
    if (active) {
        float lo[9];  // lambda_h(t + 1) at the cell itself
#pragma unroll
        for (int q = 0; q < 9; ++q) lo[q] = gld<float>(lin + (5 + q) * pb, on.at());
        const int own = (ty + 1) * ALX + tx + 1;
#pragma unroll
        for (int k = 1; k < 9; ++k) {  // phi(x) entered G(x - c_k) with weight W_k c_k
            const int j = own - AY[k] * ALX - AX[k];
            const float w = (k < 5) ? (1.f / 3.f) : (1.f / 12.f);
            phb += w * (AX[k] * s_Gx[j] + AY[k] * s_Gy[j]);
        }
        const uint32_t io = on.at();
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const float Bu = s_B[own - AY[q] * ALX - AX[q]];
            gst<float>(lout + (5 + q) * pb, io, lh[q] * Ah - Bu * lo[q] + phb);
        }
    }

    // fixed-order workgroup reduction of the eps contribution
    const double w = wave_sum_d(deps);
    if (tid % 64 == 0) s_red[tid / 64] = w;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int k = 0; k < ANT / 64; ++k) t += s_red[k];
        A.epart[blockIdx.x] = epart + t;
    }
}

// lambda_T: dL/dphi_T on every h_q, zero on g and phi_prev
__global__ void __launch_bounds__(256) k_adj_seed(AdjDesc A, const float* __restrict__ dphi) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
    if (x >= A.nx || y >= A.ny) return;
    const int64_t P = kBlockCells, i = cell_index(A.nbx, kAdjPlanes, x, y);
    const float v = dphi[(int64_t)y * A.nx + x];
#pragma unroll
    for (int q = 0; q < 9; ++q) A.lout[(5 + q) * P + i] = v;
#pragma unroll
    for (int q = 0; q < 5; ++q) A.lout[q * P + i] = 0.f;
    A.lppout[cell_index(A.nbx, 1, x, y)] = 0.f;
}

// dL/dU_init(x) = sum_q w_q lambda_g,q(x, 0) (the initial g_q = w_q U_init); per-row FP64 sums
__global__ void __launch_bounds__(256) k_adj_uinit(AdjDesc A, float* __restrict__ dU, double* __restrict__ rows) {
    __shared__ double s_red[4];
    const int y = blockIdx.x, tid = threadIdx.x;
    double acc = 0.0;
    for (int x = tid; x < A.nx; x += 256) {
        const int64_t i = cell_index(A.nbx, kAdjPlanes, x, y);
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 5; ++q) v += AW5[q] * A.lin[q * kBlockCells + i];
        dU[(int64_t)y * A.nx + x] = v;
        acc += v;
    }
    const double w = wave_sum_d(acc);
    if (tid % 64 == 0) s_red[tid / 64] = w;
    __syncthreads();
    if (tid == 0) rows[y] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}

// out[0] = sum of the eps partials, out[1] = sum of the row sums: a wave for each, lane l adding the values l, l + 64,
// ... in order, then a tree over the lanes -- a fixed order (one lane for all values took 43 us at 512^2).
__global__ void __launch_bounds__(128) k_adj_final(const double* __restrict__ epart, int ne,
                                                   const double* __restrict__ rows, int nr, double* __restrict__ out) {
    const int which = threadIdx.x / 64, lane = threadIdx.x % 64;
    const double* v = which == 0 ? epart : rows;
    const int n = which == 0 ? ne : nr;
    double t = 0.0;
#pragma unroll 4
    for (int k = lane; k < n; k += 64) t += v[k];
    t = wave_sum_d(t);
    if (lane == 0) out[which] = t;
}

// Rows of a tile.  64 x 16 tiles run one per CU and have the smaller ring, so they are faster where their rounds
// over the 256 CUs are (nearly) full: 512^2 (256 tiles) 12.0 us a step against 12.3 with 64 x 8 tiles, 1024^2 (1024)
// 42.2 against 42.9.  Where they leave CUs idle the smaller tiles spread further: 256^2 (64 tiles) 9.1 against
// 7.2, 141^2 8.4 against 7.1, 768^2 (576 tiles, the third round a quarter full) 28.9 against 26.0.
static int adj_tiles(const AdjDesc& A, int rows) { return ((A.nx + ATX - 1) / ATX) * ((A.ny + rows - 1) / rows); }
static int adj_rows(const AdjDesc& A) {
    constexpr int kCUs = 256;
    const int64_t t = adj_tiles(A, 16), slots = (t + kCUs - 1) / kCUs * kCUs;
    return 8 * t >= 7 * slots ? 16 : 8;
}
int adj_blocks(const AdjDesc& A) { return adj_tiles(A, adj_rows(A)); }

struct DescriptorPair {
    DomDesc d[2];
};
constexpr int kPairWords = sizeof(DescriptorPair) / 4;
static_assert(kPairWords <= 256 && sizeof(DescriptorPair) % 4 == 0, "a word per lane");
__global__ void __launch_bounds__(256) k_put_descriptors(uint32_t* __restrict__ dst, DescriptorPair pair) {
    if (threadIdx.x < kPairWords) dst[threadIdx.x] = reinterpret_cast<const uint32_t*>(&pair)[threadIdx.x];
}

hipError_t launch_put_descriptors(DomDesc* dst, const DomDesc& a, const DomDesc& b, hipStream_t s) {
    DescriptorPair pair;
    std::memcpy((void*)&pair.d[0], (const void*)&a, sizeof a);
    std::memcpy((void*)&pair.d[1], (const void*)&b, sizeof b);
    hipLaunchKernelGGL(k_put_descriptors, dim3(1), dim3(256), 0, s, reinterpret_cast<uint32_t*>(dst), pair);
    return hipGetLastError();
}

hipError_t launch_adj_seed(const AdjDesc& A, const float* dphi, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_seed, dim3((A.nx + 255) / 256, A.ny), dim3(256), 0, s, A, dphi);
    return hipGetLastError();
}

hipError_t launch_adj_step(const AdjDesc& A, hipStream_t s) {
    if (adj_rows(A) == 16) hipLaunchKernelGGL(k_adj<16>, dim3(adj_blocks(A)), dim3(ATX * 16), 0, s, A);
    else hipLaunchKernelGGL(k_adj<8>, dim3(adj_blocks(A)), dim3(ATX * 8), 0, s, A);
    return hipGetLastError();
}

hipError_t launch_adj_finish(const AdjDesc& A, float* dU, double* rows, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_uinit, dim3(A.ny), dim3(256), 0, s, A, dU, rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_adj_final, dim3(1), dim3(128), 0, s, A.epart, adj_blocks(A), rows, A.ny, out);
    return hipGetLastError();
}

}  // namespace snowlb
