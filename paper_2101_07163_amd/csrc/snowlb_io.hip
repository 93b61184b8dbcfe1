// snowlb_io.hip -- set-up and read-out kernels of libsnowlb (Tan et al., arXiv:2101.07163): the
// initial state, macroscopic field read-out and overwrite, population exchange with a canonical FP32
// layout, FP64 diagnostics and a plain copy that measures the practical HBM ceiling.  None of them is
// on the per-step path: plain per-cell code, laid out so that each is bound by the bytes it has to move.
#include <hip/hip_runtime.h>

#include <mutex>
#include <stdint.h>

#include "snowlb_device.h"
#include "snowlb_internal.h"
#include "snowlb_io.h"

namespace snowlb {

// Every buffer lives in device global memory.  The plane pointers are read from the descriptor,
// so the compiler cannot infer that and would emit flat (generic) accesses, which wait on both the
// memory and the LDS counters; the casts below make them global accesses.
template <class S>
__device__ __forceinline__ const GMEM typename S::T* plane_ptr(const DomDesc& d, int par, int q) {
    return (const GMEM typename S::T*)(d.pop[par]) + (int64_t)q * d.plane;
}
template <class S>
__device__ __forceinline__ GMEM typename S::T* plane_ptr_w(const DomDesc& d, int par, int q) {
    return (GMEM typename S::T*)(d.pop[par]) + (int64_t)q * d.plane;
}
__device__ __forceinline__ GMEM float* phip_ptr(const DomDesc& d, int par) {
    return (GMEM float*)(d.phip[par]);
}

// Reference values (U, rho, jx, jy) of lattice position (gx, gy) with the closure: the inlet ghost
// carries (U_in, rho0, rho0 u_in, 0) rounded to the storage format.  Loaded first, converted where they are used, so
// that loads of several positions are in flight together.
template <class S>
struct StoredRef {
    typename S::T v[4];
    bool inlet;
};
template <class S>
__device__ __forceinline__ StoredRef<S> load_ref(const DomDesc& d, int par, int gx, int gy) {
    StoredRef<S> r{};
    r.inlet = d.inout && gx < 0;
    gx = d.inout ? min(max(gx, 0), d.nx - 1) : wrapi(gx, d.nx);
    const int64_t i = cell_index(d.nbx, d.nqb, gx, wrapi(gy, d.ny));
    const GMEM typename S::T* b = (const GMEM typename S::T*)(d.refs[par]);
    r.v[R_U] = b[i];
    if (d.npop == 23) {
        r.v[R_RHO] = b[d.rplane + i];
        r.v[R_JX] = b[2 * d.rplane + i];
        r.v[R_JY] = b[3 * d.rplane + i];
    }
    return r;
}
template <class S>
__device__ __forceinline__ void ref_value(const DomDesc& d, const StoredRef<S>& t, float r[4]) {
    const bool flow = d.npop == 23;
    r[R_U] = S::from_ref(t.inlet ? S::to_ref(d.U_in) : t.v[R_U]);
    r[R_RHO] = flow ? S::from_ref(t.inlet ? S::to_ref(d.ref_f) : t.v[R_RHO]) : 0.f;
    r[R_JX] = flow ? S::from_ref(t.inlet ? S::to_ref(d.ref_f * d.u_in) : t.v[R_JX]) : 0.f;
    r[R_JY] = flow && !t.inlet ? S::from_ref(t.v[R_JY]) : 0.f;
}

template <class S>
__device__ __forceinline__ void ref_at(const DomDesc& d, int par, int gx, int gy, float r[4]) {
    if constexpr (S::kLocalRef) ref_value<S>(d, load_ref<S>(d, par, gx, gy), r);
    else r[0] = r[1] = r[2] = r[3] = 0.f;
}

// Cell of a lane: a workgroup of 256 lanes takes one 64 x 4 block, whose planes are contiguous in memory, so every
// access of a wave is a run of 64 elements and a workgroup's accesses one range of planes.  (With rows of
// 256 x 1 cells per workgroup each plane is four runs in four blocks: the 2048^2 FP32 initial state from a field of U takes
// 79 us, 72 in blocks.)
__device__ __forceinline__ void lane_cell(int& x, int& y) {
    x = blockIdx.x * kBlockX + threadIdx.x % kBlockX;
    y = blockIdx.y * kBlockY + threadIdx.x / kBlockX;
}
static dim3 block_grid(const DomDesc& d) { return dim3(d.nbx, (d.ny + kBlockY - 1) / kBlockY); }

// The same with each XCD taking a contiguous run of blocks, for canonical rows of another length than whole lines: a block
// then reads three lines a row, and the blocks that share the outer two lie on one L2.  (On eight XCDs they
// fetch them twice: h of 1500 x 1100 FP32 22.9 us, in runs 18.6, in rows of 256 x 1 cells 20.6; 2049 x 2047 FP16 47.9, 36.5,
// 40.2; 3000 x 1500 FP32 57.8, 60.8, 58.0.  With whole lines runs only cost their division: 1024^2 FP16 10.0 and
// 10.4.)
__device__ __forceinline__ void lane_cell_runs(int& x, int& y) {
    const uint32_t G = gridDim.x * gridDim.y, b = blockIdx.y * gridDim.x + blockIdx.x;
    const uint32_t xcd = b % 8, slot = xcd * (G / 8) + min(xcd, G % 8) + b / 8, by = slot / gridDim.x;
    x = (int)(slot - by * gridDim.x) * kBlockX + threadIdx.x % kBlockX;
    y = (int)by * kBlockY + threadIdx.x / kBlockX;
}

// Rows of 256 x 1 cells per workgroup.
__device__ __forceinline__ void lane_cell_rows(int& x, int& y) {
    x = blockIdx.x * kBlockCells + threadIdx.x;
    y = blockIdx.y;
}
static dim3 row_grid(const DomDesc& d) { return dim3((d.nx + kBlockCells - 1) / kBlockCells, d.ny); }

// Decode one population set of an in-domain cell; sets that are not asked for are not loaded.
template <class S>
__device__ __forceinline__ void decode_h(const DomDesc& d, int par, int x, int y, float h[9]) {
    const int64_t i = cell_index(d.nbx, d.nqb, x, y);
    const float hr = S::kLocalRef ? phip_ptr(d, par)[cell_index(d.nbx, 1, x, y)] : 0.f;
#pragma unroll
    for (int q = 0; q < 9; ++q) h[q] = S::dec(plane_ptr<S>(d, par, d.off_h + q)[i], W9[q], hr);
}
// The stored values of N planes from plane `first` on, of one cell.
template <class S, int N>
__device__ __forceinline__ void load_planes(const DomDesc& d, int par, int first, int x, int y, typename S::T raw[N]) {
    const int64_t i = cell_index(d.nbx, d.nqb, x, y);
#pragma unroll
    for (int q = 0; q < N; ++q) raw[q] = plane_ptr<S>(d, par, first + q)[i];
}
// g and f take the references of their source cells from ref(dx, dy, r): of the cell at (x + dx, y + dy).
template <class S, class R>
__device__ __forceinline__ void decode_g(const typename S::T raw[5], const R& ref, float g[5]) {
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        float r[4];
        ref(-CX[q], -CY[q], r);
        g[q] = S::dec(raw[q], W5[q], g_ref(r[R_U], r[R_JX], r[R_JY], CX[q], CY[q]));
    }
}
template <class S, class R>
__device__ __forceinline__ void decode_f(const typename S::T raw[9], const R& ref, float f[9]) {
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        float r[4];
        ref(-CX[q], -CY[q], r);
        f[q] = f_abs_dec<S>(raw[q], q, f_ref(r[R_RHO], r[R_JX], r[R_JY], CX[q], CY[q]));
    }
}

// The references of a block and its one-cell ring in LDS (16-bit storage): each is formed once per position
// instead of once per population that needs it (2048^2 FP16 from the nine sources of each cell: initial
// state 85 us, now 60, read of rho 69 us, of U 44 us; with the ring's loads waiting for the block's 40 and 34 us, together 29
// and 25).  load(gx, gy) gives those of a lattice position in a form that value() turns into floats; every lane of the
// workgroup calls the constructor.
template <class S>
struct BlockRefs {
    static constexpr int LX = kBlockX + 2, LY = kBlockY + 2, N = S::kLocalRef ? LX * LY : 1;
    const float (*s)[N];
    int own;
    // Every lane takes its own cell and the first lanes one position of the ring each.
    template <class L, class V>
    __device__ __forceinline__ BlockRefs(float (*lds)[N], int x0, int y0, const L& load, const V& value) : s(lds) {
        const int tid = threadIdx.x, tx = tid % kBlockX + 1, ty = tid / kBlockX + 1;
        own = ty * LX + tx;
        if constexpr (S::kLocalRef) {
            constexpr int RING = N - kBlockCells;
            const int c = tid - 2 * LX;
            const int rx = tid < 2 * LX ? tid % LX : (c & 1) * (LX - 1), ry = tid < 2 * LX ? tid / LX * (LY - 1) : 1 + c / 2;
            const auto a = load(x0 + tx - 1, y0 + ty - 1);
            auto b = a;
            if (tid < RING) b = load(x0 + rx - 1, y0 + ry - 1);
            float r[4];
            value(a, r);
#pragma unroll
            for (int k = 0; k < 4; ++k) lds[k][own] = r[k];
            if (tid < RING) {
                value(b, r);
#pragma unroll
                for (int k = 0; k < 4; ++k) lds[k][ry * LX + rx] = r[k];
            }
            __syncthreads();
        }
    }
    __device__ __forceinline__ void operator()(int dx, int dy, float r[4]) const {
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = S::kLocalRef ? s[k][own + dy * LX + dx] : 0.f;
    }
};
template <class S>
__device__ __forceinline__ BlockRefs<S> block_refs(const DomDesc& d, int par) {
    __shared__ float lds[4][BlockRefs<S>::N];
    return BlockRefs<S>(lds, blockIdx.x * kBlockX, blockIdx.y * kBlockY,
                        [&](int gx, int gy) { return load_ref<S>(d, par, gx, gy); },
                        [&](const StoredRef<S>& t, float r[4]) { ref_value<S>(d, t, r); });
}

// ---------------------------------------------------------------------------------------------
// initial state: circular tanh seed, equilibrium populations (rest population as remainder)
// Initial phi, x-velocity and U at an in-domain lattice position.
__device__ __forceinline__ void init_at(const DomDesc& d, const InitArgs& a, int x, int y, float& phi0, float& ux,
                                        float& U) {
    const float dx = (float)x - a.sx, dy = (float)y - a.sy;
    const float r = sqrtf(__builtin_fmaf(dy, dy, dx * dx));
    phi0 = tanhf((a.R - r) / (1.41421356237309505f * a.width));
    ux = (d.npop == 23 && d.inout) ? 0.5f * (1.f - phi0) * a.u_in : 0.f;
    U = a.U_init ? a.U_init[(int64_t)y * d.nx + x] : a.U0;
}

// Reference values of the initial state at any lattice position, with the closure of load_ref.
template <class S>
__device__ __forceinline__ void init_ref_at(const DomDesc& d, const InitArgs& a, int gx, int gy, float r[4]) {
    const int sy = wrapi(gy, d.ny);
    if (d.inout) {
        if (gx < 0) {
            r[R_U] = S::from_ref(S::to_ref(d.U_in));
            r[R_RHO] = S::from_ref(S::to_ref(d.ref_f));
            r[R_JX] = S::from_ref(S::to_ref(d.ref_f * d.u_in));
            r[R_JY] = 0.f;
            return;
        }
        if (gx >= d.nx) gx = d.nx - 1;
    } else {
        gx = wrapi(gx, d.nx);
    }
    float phi0, ux, U;
    init_at(d, a, gx, sy, phi0, ux, U);
    r[R_U] = S::from_ref(S::to_ref(U));
    r[R_RHO] = S::from_ref(S::to_ref(d.ref_f));
    r[R_JX] = S::from_ref(S::to_ref(d.ref_f * ux));
    r[R_JY] = 0.f;
}

// Cell (x, y) of the lane; with 16-bit storage the workgroup has the block of 64 x 4 cells at (x0, y0).
template <class S>
__device__ __forceinline__ void init_cell(const DomDesc& d, int par, const InitArgs& a, int x, int y, int x0, int y0) {
    __shared__ float lds[4][BlockRefs<S>::N];
    const BlockRefs<S> refs(
        lds, x0, y0, [](int gx, int gy) { return int2{gx, gy}; },
        [&](int2 at, float r[4]) { init_ref_at<S>(d, a, at.x, at.y, r); });
    if (x >= d.nx || y >= d.ny) return;
    const bool flow = d.npop == 23;
    const float rho0 = d.ref_f;
    float phi0, ux, U;
    init_at(d, a, x, y, phi0, ux, U);
    const int64_t i = cell_index(d.nbx, d.nqb, x, y);
    phip_ptr(d, par)[cell_index(d.nbx, 1, x, y)] = phi0;
    if (S::kLocalRef) {
        GMEM typename S::T* wb = (GMEM typename S::T*)(d.refs[par]);
        const int64_t ir = i;  // the reference planes share the populations' blocks
        wb[ir] = S::to_ref(U);
        if (flow) {
            wb[d.rplane + ir] = S::to_ref(rho0);
            wb[2 * d.rplane + ir] = S::to_ref(rho0 * ux);
            wb[3 * d.rplane + ir] = S::to_ref(0.f);
        }
    }
    float hq[9];
#pragma unroll
    for (int q = 1; q < 9; ++q) hq[q] = W9[q] * phi0;
    hq[0] = phi0 - sum8(hq);
#pragma unroll
    for (int q = 0; q < 9; ++q)
        plane_ptr_w<S>(d, par, d.off_h + q)[i] = S::enc(hq[q], IW9[q], S::kLocalRef ? phi0 : 0.f);
    float dfq[9], gq[5];  // f_eq - w in deviation form
    const float uu = ux * ux, drho0 = rho0 - 1.f;
#pragma unroll
    for (int q = 1; q < 9; ++q) {
        const float cu = CX[q] * ux;
        dfq[q] = W9[q] * (drho0 + rho0 * (3.f * cu + 4.5f * cu * cu - 1.5f * uu));
    }
    dfq[0] = drho0 - sum8(dfq);
#pragma unroll
    for (int q = 1; q < 5; ++q) gq[q] = W5[q] * U * (1.f + 3.f * CX[q] * ux);
    gq[0] = U - ((gq[1] + gq[2]) + (gq[3] + gq[4]));
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        float r[4] = {0.f, 0.f, 0.f, 0.f};
        refs(-CX[q], -CY[q], r);
        if (flow) plane_ptr_w<S>(d, par, q)[i] = f_dev_enc<S>(dfq[q], q, f_ref(r[R_RHO], r[R_JX], r[R_JY], CX[q], CY[q]));
        if (q < 5) plane_ptr_w<S>(d, par, d.off_g + q)[i] = S::enc(gq[q], IW5[q], g_ref(r[R_U], r[R_JX], r[R_JY], CX[q], CY[q]));
    }
}

template <class S, bool ROWS>
__global__ void __launch_bounds__(kBlockCells) k_init(DomDesc d, int par, InitArgs a) {
    static_assert(!(ROWS && S::kLocalRef), "16-bit references are formed by block");
    int x, y;
    if (ROWS) lane_cell_rows(x, y);
    else lane_cell(x, y);
    init_cell<S>(d, par, a, x, y, blockIdx.x * kBlockX, blockIdx.y * kBlockY);
}

// Every lattice of a batch in one launch over its list of 64 x 4 tiles: a launch per lattice leaves most of the chip
// idle while the lattices are small (64 crystals in FP32 612 -> 476 us, 24 of 100^2 to 583^2 153 -> 79, in FP16 211 -> 58,
// seven of 400^2 without flow 47 -> 27).
template <class S>
__global__ void __launch_bounds__(kBlockCells)
    k_init_batch(const DomDesc* __restrict__ doms, const TileDesc* __restrict__ tiles, const InitArgs* __restrict__ args) {
    const TileDesc t = tiles[blockIdx.x];
    const DomDesc d = doms[t.dom];
    init_cell<S>(d, 0, args[t.dom], t.x0 + threadIdx.x % kBlockX, t.y0 + threadIdx.x / kBlockX, t.x0, t.y0);
}

hipError_t launch_init_batch(int storage, const DomDesc* doms, const TileDesc* tiles, int ntiles, const InitArgs* args,
                             hipStream_t s) {
    const dim3 grid(ntiles), lanes(kBlockCells);
    switch (storage) {
        case 0: hipLaunchKernelGGL(k_init_batch<StoreF32>, grid, lanes, 0, s, doms, tiles, args); break;
        case 1: hipLaunchKernelGGL(k_init_batch<StoreF16>, grid, lanes, 0, s, doms, tiles, args); break;
        case 2: hipLaunchKernelGGL(k_init_batch<StoreBF16>, grid, lanes, 0, s, doms, tiles, args); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <class S>
static hipError_t init_s(const DomDesc& d, int par, const InitArgs& a, hipStream_t s) {
    // Blocks, except where they would leave a quarter of their lanes idle: there rows do better in FP32 (2048^2 with flow
    // 71.8 us in blocks, 79.1 in rows, 3000 x 1500 without flow 52.7 and 58.9; 65 x 20001 29.4 and 27.0).
    if constexpr (!S::kLocalRef) {
        const int64_t lanes = (int64_t)d.nbx * kBlockX * ((d.ny + kBlockY - 1) / kBlockY * kBlockY);
        if (4 * (int64_t)d.nx * d.ny <= 3 * lanes) {
            hipLaunchKernelGGL((k_init<S, true>), row_grid(d), dim3(kBlockCells), 0, s, d, par, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_init<S, false>), block_grid(d), dim3(kBlockCells), 0, s, d, par, a);
    return hipGetLastError();
}

hipError_t launch_init(const DomDesc& d, int par, const float* U_init, float U0, float sx, float sy,
                       float R, float w, float u_in, hipStream_t s) {
    const InitArgs a{U_init, U0, sx, sy, R, w, u_in};
    switch (d.storage) {
        case 0: return init_s<StoreF32>(d, par, a, s);
        case 1: return init_s<StoreF16>(d, par, a, s);
        case 2: return init_s<StoreBF16>(d, par, a, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// macroscopic field read-out.  One instance per kind of field, which loads only the populations that field is
// a moment of: a read is bound by those bytes (2048^2 FP32, loading all 23 planes for any field: 75 us each).
enum { READ_PHI, READ_U, READ_RHO, READ_VELOCITY };
template <class S, int KIND>
__global__ void __launch_bounds__(kBlockCells) k_read(DomDesc d, int par, int axis, float* __restrict__ dst) {
    int x, y;
    lane_cell(x, y);
    const bool active = x < d.nx && y < d.ny;
    float phi = 0.f, v = 0.f;
    typename S::T graw[5], fraw[9];  // loaded before the references, which wait for a barrier
    if (KIND == READ_U && active) load_planes<S, 5>(d, par, d.off_g, x, y, graw);
    if ((KIND == READ_RHO || KIND == READ_VELOCITY) && active) load_planes<S, 9>(d, par, 0, x, y, fraw);
    if ((KIND == READ_PHI || KIND == READ_VELOCITY) && active) {
        float h[9];
        decode_h<S>(d, par, x, y, h);
        double p = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q) p += (double)h[q];
        v = phi = (float)p;
    }
    if constexpr (KIND != READ_PHI) {
        const BlockRefs<S> refs = block_refs<S>(d, par);
        if (!active) return;
        if (KIND == READ_U) {
            float g[5];
            decode_g<S>(graw, refs, g);
            v = (g[0] + g[1]) + (g[2] + g[3]) + g[4];
        }
        if (KIND == READ_RHO || KIND == READ_VELOCITY) {
            float f[9];
            decode_f<S>(fraw, refs, f);
            const float rho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
            v = rho;
            if (KIND == READ_VELOCITY) {
                const float jx = (f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7]);
                const float jy = (f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8]);
                const float pc = fminf(fmaxf(phi, -1.f), 1.f);
                const float k = d.kdrag * (1.f + pc) * (1.f + pc) * (1.f - pc);
                const float sc = 0.5f * (1.f - pc) / (rho + 0.5f * k);
                v = (axis == 0 ? jx : jy) * sc;
            }
        }
    }
    if (active) dst[(int64_t)y * d.nx + x] = v;
}

// the density and velocity of a lattice without flow
__global__ void k_fill_zero(float* __restrict__ dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0.f;
}

template <class S>
static hipError_t read_s(const DomDesc& d, int par, int field, float* dst, hipStream_t s) {
    const dim3 grid = block_grid(d), lanes(kBlockCells);
    if (field == 0) hipLaunchKernelGGL((k_read<S, READ_PHI>), grid, lanes, 0, s, d, par, 0, dst);
    else if (field == 1) hipLaunchKernelGGL((k_read<S, READ_U>), grid, lanes, 0, s, d, par, 0, dst);
    else if (d.npop != 23) {
        const int64_t n = (int64_t)d.nx * d.ny;
        hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, n);
    } else if (field == 2) hipLaunchKernelGGL((k_read<S, READ_RHO>), grid, lanes, 0, s, d, par, 0, dst);
    else hipLaunchKernelGGL((k_read<S, READ_VELOCITY>), grid, lanes, 0, s, d, par, field - 3, dst);
    return hipGetLastError();
}

hipError_t launch_read(const DomDesc& d, int par, int field, float* dst, hipStream_t s) {
    switch (d.storage) {
        case 0: return read_s<StoreF32>(d, par, field, dst, s);
        case 1: return read_s<StoreF16>(d, par, field, dst, s);
        case 2: return read_s<StoreBF16>(d, par, field, dst, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// overwrite one macroscopic field (debugging and tests): PHI sets h_q = w_q phi with phi_prev = phi (the
// phase field at rest, no anisotropic flux); U sets g_q = g_eq(U, u) with the velocity u the
// collisions currently see (0 without flow).  16-bit storage encodes h against the new phi_prev and g
// against a U reference reset to 0 (inlet-ghost sources keep the ghost constant), as a population
// write does.  The U case reads only f, h and phi_prev, none of which it writes.
// Rows in FP32, blocks in 16 bits: phi of 65 x 20001 FP32 13.7 and 14.7 us, FP16 13.0 and 11.0; U with flow 27.4 and 30.6,
// FP16 33.3 and 30.4.
template <class S>
__global__ void __launch_bounds__(kBlockCells) k_write_field(DomDesc d, int par, int field,
                                                             const float* __restrict__ src) {
    int x, y;
    if (S::kLocalRef) lane_cell(x, y);
    else lane_cell_rows(x, y);
    if (x >= d.nx || y >= d.ny) return;
    const int64_t i = cell_index(d.nbx, d.nqb, x, y), i1 = cell_index(d.nbx, 1, x, y);
    const float v = src[(int64_t)y * d.nx + x];
    if (field == 0) {
        phip_ptr(d, par)[i1] = v;
        float hq[9];
#pragma unroll
        for (int q = 1; q < 9; ++q) hq[q] = W9[q] * v;
        hq[0] = v - sum8(hq);
#pragma unroll
        for (int q = 0; q < 9; ++q)
            plane_ptr_w<S>(d, par, d.off_h + q)[i] = S::enc(hq[q], IW9[q], S::kLocalRef ? v : 0.f);
        return;
    }
    const bool flow = d.npop == 23;
    float ux = 0.f, uy = 0.f;
    if (flow) {
        float f[9], h[9];
        typename S::T raw[9];
        load_planes<S, 9>(d, par, 0, x, y, raw);
        decode_f<S>(raw, [&](int dx, int dy, float r[4]) { ref_at<S>(d, par, x + dx, y + dy, r); }, f);
        decode_h<S>(d, par, x, y, h);
        double p = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q) p += (double)h[q];
        const float pc = fminf(fmaxf((float)p, -1.f), 1.f);
        const float rho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
        const float k = d.kdrag * (1.f + pc) * (1.f + pc) * (1.f - pc);
        const float sc = 0.5f * (1.f - pc) / (rho + 0.5f * k);
        ux = ((f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7])) * sc;
        uy = ((f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8])) * sc;
    }
    float gq[5];
#pragma unroll
    for (int q = 1; q < 5; ++q) gq[q] = W5[q] * v * (1.f + 3.f * (CX[q] * ux + CY[q] * uy));
    gq[0] = v - ((gq[1] + gq[2]) + (gq[3] + gq[4]));
    if (S::kLocalRef) ((GMEM typename S::T*)(d.refs[par]))[i] = S::to_ref(0.f);
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        float r[4] = {0.f, 0.f, 0.f, 0.f};
        if (S::kLocalRef && d.inout && x - CX[q] < 0) ref_at<S>(d, par, -1, y - CY[q], r);  // ghost constants
        plane_ptr_w<S>(d, par, d.off_g + q)[i] = S::enc(gq[q], IW5[q], g_ref(r[R_U], r[R_JX], r[R_JY], CX[q], CY[q]));
    }
}

template <class S>
static hipError_t write_field_s(const DomDesc& d, int par, int field, const float* src, hipStream_t s) {
    hipLaunchKernelGGL(k_write_field<S>, S::kLocalRef ? block_grid(d) : row_grid(d), dim3(kBlockCells), 0, s, d, par, field, src);
    return hipGetLastError();
}

hipError_t launch_write_field(const DomDesc& d, int par, int field, const float* src, hipStream_t s) {
    switch (d.storage) {
        case 0: return write_field_s<StoreF32>(d, par, field, src, s);
        case 1: return write_field_s<StoreF16>(d, par, field, src, s);
        case 2: return write_field_s<StoreBF16>(d, par, field, src, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// population sets <-> canonical FP32 [q][y][x]
template <class S, int SET>
__global__ void __launch_bounds__(kBlockCells) k_pop_get(DomDesc d, int par, float* __restrict__ canon) {
    int x, y;
    lane_cell(x, y);
    const bool active = x < d.nx && y < d.ny;
    const int64_t n = (int64_t)d.nx * d.ny, c = (int64_t)y * d.nx + x;
    float v[9];
    if constexpr (SET == 0 || SET == 1) {
        typename S::T raw[9];
        if (active) load_planes<S, SET == 0 ? 9 : 5>(d, par, SET == 0 ? 0 : d.off_g, x, y, raw);
        const BlockRefs<S> refs = block_refs<S>(d, par);
        if (!active) return;
        if (SET == 0) decode_f<S>(raw, refs, v);
        else decode_g<S>(raw, refs, v);
    }
    if (!active) return;
    if (SET == 2) decode_h<S>(d, par, x, y, v);
    if (SET == 3) v[0] = phip_ptr(d, par)[cell_index(d.nbx, 1, x, y)];
#pragma unroll
    for (int q = 0; q < (SET == 3 ? 1 : SET == 1 ? 5 : 9); ++q) canon[q * n + c] = v[q];
}

// Writing a set re-encodes it against the references the step will decode it with.  Writing f
// (resp. g) resets the rho, j (resp. U) reference planes to 0 -- any consistent reference is valid;
// populations streamed from the inlet ghost keep the ghost's references.  Writing phi_prev
// re-encodes h.
// The 16-bit value of a population of f or g: its deviation is rounded to FP32 and then to 16 bits.  (Left to itself the
// compiler may fold the conversion into the multiply-add, which rounds once, in some instances and not in others.  It
// does so for h and phi_prev below and in k_write_field in every instance, and their bits have always been those.)
template <class S>
__device__ __forceinline__ typename S::T enc_deviation(float p, float iw, float ref) {
    float e = __builtin_fmaf(p, iw, -ref);
    asm("" : "+v"(e));
    return S::to_ref(e);
}

template <class S, int SET>
__global__ void __launch_bounds__(kBlockCells) k_pop_set(DomDesc d, int par, const float* __restrict__ canon) {
    int x, y;
    if (SET != 3 && d.nx % 32) lane_cell_runs(x, y);
    else lane_cell(x, y);
    if (x >= d.nx || y >= d.ny) return;
    const int64_t n = (int64_t)d.nx * d.ny, c = (int64_t)y * d.nx + x, i = cell_index(d.nbx, d.nqb, x, y);
    const int64_t i1 = cell_index(d.nbx, 1, x, y), ir = i;
    constexpr int NQ = SET == 3 ? 1 : SET == 1 ? 5 : 9;
    float v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = canon[q * n + c];
    GMEM typename S::T* wb = S::kLocalRef ? (GMEM typename S::T*)(d.refs[par]) : nullptr;
    if constexpr (SET == 0 || SET == 1) {
        if (S::kLocalRef) {
            if (SET == 1) wb[ir] = S::to_ref(0.f);
            else for (int k = 1; k < 4; ++k) wb[k * d.rplane + ir] = S::to_ref(0.f);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            float r[4] = {0.f, 0.f, 0.f, 0.f};
            if (S::kLocalRef && d.inout && x - CX[q] < 0) ref_at<S>(d, par, -1, y - CY[q], r);  // ghost constants
            const float m = SET == 0 ? f_ref(r[R_RHO], r[R_JX], r[R_JY], CX[q], CY[q])
                                     : g_ref(r[R_U], r[R_JX], r[R_JY], CX[q], CY[q]);
            typename S::T e;
            if constexpr (S::kLocalRef) e = enc_deviation<S>(v[q], SET == 0 ? IW9[q] : IW5[q < 5 ? q : 0], m);
            else e = SET == 0 ? f_abs_enc<S>(v[q], q, m) : v[q];
            plane_ptr_w<S>(d, par, (SET == 0 ? 0 : d.off_g) + q)[i] = e;
        }
    } else if constexpr (SET == 2) {
        const float ref = S::kLocalRef ? phip_ptr(d, par)[i1] : 0.f;
#pragma unroll
        for (int q = 0; q < 9; ++q) plane_ptr_w<S>(d, par, d.off_h + q)[i] = S::enc(v[q], IW9[q], ref);
    } else {
        const float pnew = v[0];
        if (S::kLocalRef) {
            const float pold = phip_ptr(d, par)[i1];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                GMEM typename S::T* p = plane_ptr_w<S>(d, par, d.off_h + q) + i;
                *p = S::enc(S::dec(*p, W9[q], pold), IW9[q], pnew);
            }
        }
        phip_ptr(d, par)[i1] = pnew;
    }
}

template <class S, int SET>
static void pop_io_set(const DomDesc& d, int par, int to_canon, float* canon, hipStream_t s) {
    const dim3 grid = block_grid(d), lanes(kBlockCells);
    if (to_canon) hipLaunchKernelGGL((k_pop_get<S, SET>), grid, lanes, 0, s, d, par, canon);
    else hipLaunchKernelGGL((k_pop_set<S, SET>), grid, lanes, 0, s, d, par, (const float*)canon);
}

template <class S>
static hipError_t pop_io_s(const DomDesc& d, int par, int set, int to_canon, float* canon, hipStream_t s) {
    switch (set) {
        case 0: pop_io_set<S, 0>(d, par, to_canon, canon, s); break;
        case 1: pop_io_set<S, 1>(d, par, to_canon, canon, s); break;
        case 2: pop_io_set<S, 2>(d, par, to_canon, canon, s); break;
        default: pop_io_set<S, 3>(d, par, to_canon, canon, s);
    }
    return hipGetLastError();
}

hipError_t launch_pop_io(const DomDesc& d, int par, int set, int to_canon, float* canon, hipStream_t s) {
    switch (d.storage) {
        case 0: return pop_io_s<StoreF32>(d, par, set, to_canon, canon, s);
        case 1: return pop_io_s<StoreF16>(d, par, set, to_canon, canon, s);
        case 2: return pop_io_s<StoreBF16>(d, par, set, to_canon, canon, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// FP64 diagnostics: per-thread sums over a fixed set of cells, wave64 shuffle reduction, LDS
// across waves, one partial per workgroup, then a single-workgroup pass in a fixed order.
static constexpr int kDiagThreads = 256;

// Four cells a lane in FP32, one in 16 bits, where a cell is a long chain (its references, then its populations): fewer
// partials cost k_diag_final less, more lanes hide the chain (both kernels, 1024^2 FP32 23.1 us with four, 25.0 with one;
// 701 x 499 without flow 10.4 and 13.8; 128^2 FP16 15.6 and 9.3, 701 x 499 19.7 and 17.6).
int diag_blocks(const DomDesc& d) {
    const long cells = (long)d.nx * d.ny, per = kDiagThreads * (d.storage == 0 ? 4 : 1);
    long b = (cells + per - 1) / per;
    if (b > kDiagMaxBlocks) b = kDiagMaxBlocks;  // larger lattices loop over more cells per thread
    return (int)(b < 1 ? 1 : b);
}

// Scratch of the allocation-free diagnostics (snowlb_diag_noalloc): the per-workgroup partials, at
// most kDiagMaxBlocks x 8 doubles (128 KiB), in a file-scope device array.  Each GPU the library
// runs on holds its own copy until the process ends; host code never passes the array's name to a
// kernel (on the host it is only a stand-in), but the device address that hipGetSymbolAddress
// returns for the current device, looked up once per device and kept.
static __device__ __align__(256) double scratch[kDiagMaxBlocks * 8];

hipError_t diag_scratch(double** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr[dev] = p;
    }
    *out = static_cast<double*>(ptr[dev]);
    return hipSuccess;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

template <class S>
__global__ void __launch_bounds__(kDiagThreads) k_diag(DomDesc d, int par, double* __restrict__ partials) {
    const bool flow = d.npop == 23;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t cells = (int64_t)d.nx * d.ny;
    for (int64_t c = (int64_t)blockIdx.x * kDiagThreads + threadIdx.x; c < cells;
         c += (int64_t)gridDim.x * kDiagThreads) {
        const int y = (int)((uint32_t)c / (uint32_t)d.nx), x = (int)c - y * d.nx;  // cells < 2^31
        float f[9], g[5], h[9];
        decode_h<S>(d, par, x, y, h);
        const auto ref = [&](int dx, int dy, float r[4]) { ref_at<S>(d, par, x + dx, y + dy, r); };
        typename S::T graw[5], fraw[9];
        load_planes<S, 5>(d, par, d.off_g, x, y, graw);
        decode_g<S>(graw, ref, g);
        if (flow) {
            load_planes<S, 9>(d, par, 0, x, y, fraw);
            decode_f<S>(fraw, ref, f);
        }
        double phi = 0, U = 0, rho = 0, jx = 0, jy = 0;
        bool bad = false;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            bad |= !isfinite(h[q]);
            phi += h[q];
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            bad |= !isfinite(g[q]);
            U += g[q];
        }
        if (flow) {
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                bad |= !isfinite(f[q]);
                rho += f[q];
                jx += CX[q] * (double)f[q];
                jy += CY[q] * (double)f[q];
            }
        }
        const float pp = phip_ptr(d, par)[cell_index(d.nbx, 1, x, y)];
        bad |= !isfinite(pp);
        acc[0] += rho; acc[1] += jx; acc[2] += jy; acc[3] += U; acc[4] += phi; acc[5] += pp;
        acc[6] += (phi > 0.0) ? 1.0 : 0.0;
        acc[7] += bad ? 1.0 : 0.0;
    }
    __shared__ double s_part[kDiagThreads / 64][8];
    const int lane = threadIdx.x % 64, wid = threadIdx.x / 64;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double v = wave_sum(acc[k]);
        if (lane == 0) s_part[wid][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        double v = 0;
        for (int w = 0; w < kDiagThreads / 64; ++w) v += s_part[w][threadIdx.x];
        partials[(int64_t)blockIdx.x * 8 + threadIdx.x] = v;
    }
}

__global__ void __launch_bounds__(256) k_diag_final(const double* __restrict__ partials, int nblk, double half_Lsat,
                                                    double* __restrict__ out) {
    // 32 lanes per quantity: lane l of quantity k sums blocks l, l + 32, ... in order, then lane 0
    // adds the 32 lane sums in order.  Fixed order, hence deterministic.  Then the species invariant
    // sum U + (L_sat/2) sum phi_prev (the vapour the depletion source of Sec. 2.2.2 removes is
    // (L_sat/2) times the phase gained).  A lane loads a batch of its partials before it adds the first: the
    // kernel is bound by the latency of those loads (one by one, 2048 blocks took 17 to 20 us: diagnostics of 1024^2
    // FP16 41 us, now 28; 2048^2 FP32 95, now 81).
    constexpr int kBatch = 16;
    __shared__ double s[8][32];
    __shared__ double tot[8];
    const int k = threadIdx.x % 8, l = threadIdx.x / 8;
    double v = 0;
    for (int b = l; b < nblk; b += 32 * kBatch) {
        double p[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) p[i] = b + 32 * i < nblk ? partials[(int64_t)(b + 32 * i) * 8 + k] : 0.0;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) v += p[i];
    }
    s[k][l] = v;
    __syncthreads();
    if (l == 0) {
        double t = 0;
        for (int i = 0; i < 32; ++i) t += s[k][i];
        out[k] = t;
        tot[k] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0) out[8] = __dadd_rn(tot[3], __dmul_rn(half_Lsat, tot[5]));
}

template <class S>
static hipError_t diag_s(const DomDesc& d, int par, double* partials, double* out, double half_Lsat, hipStream_t s) {
    const int nb = diag_blocks(d);
    hipLaunchKernelGGL(k_diag<S>, dim3(nb), dim3(kDiagThreads), 0, s, d, par, partials);
    hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(256), 0, s, partials, nb, half_Lsat, out);
    return hipGetLastError();
}

hipError_t launch_diag(const DomDesc& d, int par, double* partials, double* out, double half_Lsat, hipStream_t s) {
    switch (d.storage) {
        case 0: return diag_s<StoreF32>(d, par, partials, out, half_Lsat, s);
        case 1: return diag_s<StoreF16>(d, par, partials, out, half_Lsat, s);
        case 2: return diag_s<StoreBF16>(d, par, partials, out, half_Lsat, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// plain copy: the practical HBM ceiling (read + write of the same byte count)
__global__ void __launch_bounds__(256) k_copy(float4* __restrict__ dst, const float4* __restrict__ src, int64_t n) {
    // one 16-byte element per lane, one workgroup per 4 KiB chunk, dispatched in address order
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_copy(void* dst, const void* src, int64_t bytes, hipStream_t s) {
    const int64_t n = bytes / 16;
    if (n <= 0) return hipSuccess;
    const int64_t grid = (n + 255) / 256;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy, dim3((unsigned)grid), dim3(256), 0, s, (float4*)dst, (const float4*)src, n);
    return hipGetLastError();
}

}  // namespace snowlb
