// tile2d.hip -- small 2D grids, radius R = 1 or 2: a work-group holds a tile in
// registers and advances it many steps before it returns to memory.
//
// The row pipelines (stream2d_impl.h) carry a pass through a chain of rows, one
// after the other: a short chunk pays the chain's start, a long one leaves CUs
// idle.  Here (paper Sec. 4.1, an xy tile held on chip) lane L of wave w holds
// columns X0 + L*VX .. +VX-1 of rows Y0 + w*K .. +K-1 of a tile of 64*VX x NW*K
// cells; every step all waves update their rows at once: x neighbours from the
// lane's own registers or lane +-1 through DPP, y neighbours from the wave's own
// rows and, for its first and last row, through LDS (one barrier a step, two
// buffers alternating).  After t steps the tile is exact but for R*t cells a side.
//
// Zero rule: a tile that would cross the grid's edge is moved inward to touch
// it; there the zeros that enter through DPP and the LDS rows outside the tile
// are the ghost layer.  Periodic rule: rows and columns are loaded wrapped.
// The points of a cell are taken in the canonical order (the centre, then
// (dy, dx) lexicographic; one multiply, then an FMA chain), so the bits are
// those of every other kernel.
//
// What bounds it: the chain of steps -- one LDS round trip, a barrier and the
// wave's own arithmetic each, 0.45 us for FP64 5 points at one column a
// lane, of which 0.24 is arithmetic; a pass adds 2.3 us.  512^2 FP64, 100 steps:
// 125 us with the row pipeline, 60 us here.  Radius 2, us a step, rows and tiles:
// FP64 9 points 512^2 2.40 and 1.27, 25 points 3.52 and 2.20, FP32 25 points
// 1024^2 5.15 and 2.24.
#include "dev_common.h"
#include "internal.h"

namespace st {
namespace t2d {

constexpr int kNW = 8, kK = 8;  // waves, rows a wave

template <typename TS, int R, bool BOX, int VX, bool PER>
struct Tile {
    using S = Storage<TS>;
    using TC = typename S::TC;
    static constexpr int NW = kNW, K = kK, W = 64 * VX, H = NW * K;
    static_assert(VX >= R && K >= 2 * R, "neighbours in the next lane and the next wave");
    // LDS rows of a buffer: R above the tile, the first and the last R of each
    // wave, R below the tile
    static constexpr int SLOTS = 2 * R * (NW + 1), BUF = SLOTS * W;
    static constexpr int kPoints = BOX ? (2 * R + 1) * (2 * R + 1) : 4 * R + 1;
    static constexpr uint32_t kOut = 0x80000000u;
    static constexpr int32_t kRsrcWord3 = 0x00020000;

    static __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t r, uint32_t o, TC (&v)[VX]) {
        constexpr int kBytes = VX * static_cast<int>(sizeof(TS));
        TS vals[VX];
        if constexpr (kBytes == 16) {
            const u32x4 raw = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
            __builtin_memcpy(vals, &raw, 16);
        } else if constexpr (kBytes == 8) {
            const u32x2 raw = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
            __builtin_memcpy(vals, &raw, 8);
        } else {
            static_assert(kBytes == 4, "4, 8 or 16 bytes a lane");
            const uint32_t raw = __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
            __builtin_memcpy(vals, &raw, 4);
        }
#pragma unroll
        for (int e = 0; e < VX; ++e) v[e] = S::widen(vals[e]);
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t o, const TC (&v)[VX]) {
        constexpr int kBytes = VX * static_cast<int>(sizeof(TS));
        TS vals[VX];
#pragma unroll
        for (int e = 0; e < VX; ++e) vals[e] = S::narrow(v[e]);
        if constexpr (kBytes == 16) {
            u32x4 raw;
            __builtin_memcpy(&raw, vals, 16);
            __builtin_amdgcn_raw_buffer_store_b128(raw, r, o, 0, 0);
        } else if constexpr (kBytes == 8) {
            u32x2 raw;
            __builtin_memcpy(&raw, vals, 8);
            __builtin_amdgcn_raw_buffer_store_b64(raw, r, o, 0, 0);
        } else {
            uint32_t raw;
            __builtin_memcpy(&raw, vals, 4);
            __builtin_amdgcn_raw_buffer_store_b32(raw, r, o, 0, 0);
        }
    }

    // a row with its x neighbours
    struct Row {
        TC v[VX], l[R], r[R];
    };
    static __device__ __forceinline__ Row row(const TC (&v)[VX]) {
        Row q;
#pragma unroll
        for (int e = 0; e < VX; ++e) q.v[e] = v[e];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            q.l[j] = from_lower_z(v[VX - R + j]);
            q.r[j] = from_upper_z(v[j]);
        }
        return q;
    }
    static __device__ __forceinline__ TC at(const Row& q, int x) {
        return x < 0 ? q.l[x < 0 ? R + x : 0] : (x >= VX ? q.r[x >= VX ? x - VX : 0] : q.v[x < 0 ? 0 : (x >= VX ? 0 : x)]);
    }
    // row k of the wave's rows with the R above (a) and below (b)
    static __device__ __forceinline__ const Row& pick(const Row (&q)[K], const Row (&a)[R], const Row (&b)[R], int k) {
        return k < 0 ? a[k < 0 ? R + k : 0] : (k >= K ? b[k >= K ? k - K : 0] : q[k < 0 ? 0 : (k >= K ? 0 : k)]);
    }
    static __device__ __forceinline__ TC next(const TC (&w)[kPoints], const Row (&q)[K], const Row (&a)[R],
                                              const Row (&b)[R], int k, int e) {
        TC acc = w[0] * q[k].v[e];
        int p = 1;
#pragma unroll
        for (int dy = -R; dy <= R; ++dy) {
            const Row& m = pick(q, a, b, k + dy);
#pragma unroll
            for (int dx = -R; dx <= R; ++dx)
                if ((dy != 0 || dx != 0) && (BOX || dy == 0 || dx == 0)) acc = fma_c(w[p++], at(m, e + dx), acc);
        }
        return S::round(acc);
    }

    static __device__ __forceinline__ void step(const TC (&w)[kPoints], TC (&u)[K][VX], TC* buf, int own) {
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                buf[own + (R + j) * W + e] = u[j][e];
                buf[own + (2 * R + j) * W + e] = u[K - R + j][e];
            }
        __syncthreads();
        TC va[R][VX], vb[R][VX];
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                va[j][e] = buf[own + j * W + e];
                vb[j][e] = buf[own + (3 * R + j) * W + e];
            }
        TC n[K][VX];
        Row q[K], a[R], b[R];
#pragma unroll
        for (int k = 0; k < K; ++k) q[k] = row(u[k]);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            a[j] = row(va[j]);
            b[j] = row(vb[j]);
        }
        // the rows between first, then those that wait for LDS
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int k = i < K - 2 * R ? i + R : (i < K - R ? i - (K - 2 * R) : i);
#pragma unroll
            for (int e = 0; e < VX; ++e) n[k][e] = next(w, q, a, b, k, e);
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int e = 0; e < VX; ++e) u[k][e] = n[k][e];
    }

    static __device__ __forceinline__ void run(const Tile2DArgs& a, TC* lds) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
        const uint32_t item = static_cast<uint32_t>(xcd_remap(blockIdx.x, gridDim.x));
        const int32_t ty = static_cast<int32_t>(item / static_cast<uint32_t>(a.tiles_x));
        const int32_t tx = static_cast<int32_t>(item) - ty * a.tiles_x;
        const int32_t nx = a.nx, ny = a.ny;
        const int32_t ox0 = tx > 0 ? tx * a.out_w + a.edge_x : 0, ox1 = tx + 1 < a.tiles_x ? (tx + 1) * a.out_w + a.edge_x : nx;
        const int32_t oy0 = ty > 0 ? ty * a.out_h + a.edge_y : 0, oy1 = ty + 1 < a.tiles_y ? (ty + 1) * a.out_h + a.edge_y : ny;
        int32_t X0 = ox0 - a.hx, Y0 = oy0 - a.hy;
        if (!PER) {
            X0 = X0 < 0 ? 0 : (X0 + W > nx ? nx - W : X0);
            Y0 = Y0 < 0 ? 0 : (Y0 + H > ny ? ny - H : Y0);
        }
        const int32_t xl = X0 + lane * VX, yw = Y0 + wave * K;
        const int32_t x0 = PER ? wrap_idx(xl, nx) : xl;
        const uint32_t bytes = static_cast<uint32_t>(ny) * static_cast<uint32_t>(nx) * sizeof(TS);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.src), 0, bytes, kRsrcWord3);
        uint32_t off[K];
        TC u[K][VX];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t y = PER ? wrap_idx(yw + k, ny) : yw + k;
            off[k] = static_cast<uint32_t>(y * nx + x0) * sizeof(TS);
            ld(rs, off[k], u[k]);
        }
        // the rows outside the tile hold 0
        for (int i = threadIdx.x; i < 2 * R * W; i += 64 * NW) {
            TC* b = lds + (i / (R * W)) * BUF + i % (R * W);
            b[0] = TC(0);
            b[(SLOTS - R) * W] = TC(0);
        }
        TC w[kPoints];
#pragma unroll
        for (int p = 0; p < kPoints; ++p) w[p] = static_cast<TC>(a.w[p]);
        const int own = 2 * R * wave * W + lane * VX;
        int32_t t = a.t;
        for (; t >= 2; t -= 2) {
            step(w, u, lds, own);
            step(w, u, lds + BUF, own);
        }
        if (t > 0) step(w, u, lds, own);
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(a.dst, 0, bytes, kRsrcWord3);
        const bool xown = xl + VX > ox0 && xl < ox1;
#pragma unroll
        for (int k = 0; k < K; ++k) st(rd, xown && yw + k >= oy0 && yw + k < oy1 ? off[k] : kOut, u[k]);
    }
};

// 128 registers a lane: two work-groups a CU
template <typename TS, int R, bool BOX, int VX, bool PER>
__global__ __launch_bounds__(64 * kNW, 4) void tile2d_kernel(const Tile2DArgs a) {
    using P = Tile<TS, R, BOX, VX, PER>;
    __shared__ __align__(16) typename P::TC lds[2 * P::BUF];
    P::run(a, lds);
}

template <typename TS, int R, int VX>
hipError_t go(bool box, bool per, const Tile2DArgs& a, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(a.tiles_x) * static_cast<unsigned>(a.tiles_y)), block(64 * kNW);
    if (box && per) hipLaunchKernelGGL((tile2d_kernel<TS, R, true, VX, true>), grid, block, 0, s, a);
    else if (box) hipLaunchKernelGGL((tile2d_kernel<TS, R, true, VX, false>), grid, block, 0, s, a);
    else if (per) hipLaunchKernelGGL((tile2d_kernel<TS, R, false, VX, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((tile2d_kernel<TS, R, false, VX, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace t2d

int tile2d_rows() { return t2d::kNW * t2d::kK; }
int tile2d_lds_bytes(int dtype, int radius, int vx) {
    return 2 * 2 * radius * (t2d::kNW + 1) * 64 * vx * (dtype == kF64 ? 8 : 4);  // two buffers of Tile::SLOTS rows
}

hipError_t launch_tile2d(int dtype, int radius, int vx, bool box, bool periodic, const Tile2DArgs& a, hipStream_t s) {
    if (radius == 1) {
        if (dtype == kF64 && vx == 1) return t2d::go<double, 1, 1>(box, periodic, a, s);
        if (dtype == kF64 && vx == 2) return t2d::go<double, 1, 2>(box, periodic, a, s);
        if (dtype == kF32 && vx == 1) return t2d::go<float, 1, 1>(box, periodic, a, s);
        if (dtype == kF32 && vx == 2) return t2d::go<float, 1, 2>(box, periodic, a, s);
        if (dtype == kBF16 && vx == 4) return t2d::go<bf16s, 1, 4>(box, periodic, a, s);
    } else if (radius == 2) {
        if (dtype == kF64 && vx == 2) return t2d::go<double, 2, 2>(box, periodic, a, s);
        if (dtype == kF32 && vx == 2) return t2d::go<float, 2, 2>(box, periodic, a, s);
        if (dtype == kBF16 && vx == 4) return t2d::go<bf16s, 2, 4>(box, periodic, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace st
