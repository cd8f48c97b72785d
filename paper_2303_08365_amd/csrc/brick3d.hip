// brick3d.hip -- small 3D grids, 7-point star: a work-group holds a brick in
// registers and advances it several steps before it returns to memory.
//
// The plane pipelines (pipe3d_impl.h, stream3d_impl.h) carry a pass through a
// chain of planes; on a small grid that chain, and with one step per launch the
// launches, take the time.  Here (paper Sec. 4.1, the tile held on chip) wave
// (wy, wz) of 4 x 4 holds rows Y0 + 4 wy .. +3 of planes Z0 + 4 wz .. +3, lane L
// columns X0 + L*VX .. +VX-1: a brick of 64*VX x 16 x 16 cells.  Every step all
// waves update their cells at once: x neighbours through DPP, y and z neighbours
// from the wave's own registers and, across waves, from edge rows in LDS.  After
// t steps the brick is exact but for t cells a side.
//
// LDS holds, per plane, the first and last row of each wave in y, per row the
// first and last plane of each wave in z, and one row of zeros that stands for
// everything outside the brick.  One buffer, two barriers a step: the second
// comes after the step's arithmetic, when every wave has long read its rows.
//
// Zero rule: a brick that would cross the grid's edge is moved inward to touch
// it; there the zeros from DPP and LDS are the ghost layer.  Periodic rule:
// rows, planes and columns are loaded wrapped.  A cell takes its points in the
// canonical order (centre, z-1, y-1, x-1, x+1, y+1, z+1; one multiply, then an
// FMA chain): the bits of every other kernel.
//
// What bounds it: the chain of steps: 1.6 us each for FP32 at one column a lane
// (1.1 arithmetic, 0.4 edge rows through LDS), 2.4 for FP64; a pass adds 4.5 us.
// 89 x 97 x 101 FP32, 10 steps: 75 us in single steps, 35 us here.
#include "dev_common.h"
#include "internal.h"

namespace st {
namespace b3 {

constexpr int kN = 4, kW = 4;       // rows (planes) a wave, waves, in y and in z
constexpr int kEdge = kN * kW;      // rows, planes of a brick

template <typename TS, int VX, bool PER>
struct Brick {
    using S = Storage<TS>;
    using TC = typename S::TC;
    static constexpr int W = 64 * VX;
    static constexpr int kZRows = kEdge * 2 * kW, kZero = 2 * kZRows, kRows = kZero + 1;
    static constexpr int LDS_BYTES = kRows * W * static_cast<int>(sizeof(TC));
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
    static constexpr uint32_t kOut = 0x80000000u;
    static constexpr int32_t kRsrcWord3 = 0x00020000;

    // row `row` of the grid: the range is the row
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int32_t row, int32_t nx) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<TS*>(static_cast<const TS*>(p) + static_cast<int64_t>(row) * nx), 0,
                                                 static_cast<uint32_t>(nx) * sizeof(TS), kRsrcWord3);
    }
    static __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t r, uint32_t o, TC (&v)[VX]) {
        constexpr int kBytes = VX * static_cast<int>(sizeof(TS));
        TS vals[VX];
        if constexpr (kBytes == 8) {
            const u32x2 raw = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
            __builtin_memcpy(vals, &raw, 8);
        } else {
            static_assert(kBytes == 4, "4 or 8 bytes a lane");
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
        if constexpr (kBytes == 8) {
            u32x2 raw;
            __builtin_memcpy(&raw, vals, 8);
            __builtin_amdgcn_raw_buffer_store_b64(raw, r, o, 0, 0);
        } else {
            uint32_t raw;
            __builtin_memcpy(&raw, vals, 4);
            __builtin_amdgcn_raw_buffer_store_b32(raw, r, o, 0, 0);
        }
    }
    static __device__ __forceinline__ void get(const TC* lds, int row, int col, TC (&v)[VX]) {
#pragma unroll
        for (int e = 0; e < VX; ++e) v[e] = lds[row * W + col + e];
    }
    static __device__ __forceinline__ void put(TC* lds, int row, int col, const TC (&v)[VX]) {
#pragma unroll
        for (int e = 0; e < VX; ++e) lds[row * W + col + e] = v[e];
    }

    static __device__ __forceinline__ void step(const TC (&w)[7], TC (&u)[kN][kN][VX], TC* lds, int wy, int wz, int col) {
        // edge rows of the wave: of each plane in y, of each row in z
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int y = ((wz * kN + i) * kW + wy) * 2, z = kZRows + ((wy * kN + i) * kW + wz) * 2;
            put(lds, y, col, u[i][0]);
            put(lds, y + 1, col, u[i][kN - 1]);
            put(lds, z, col, u[0][i]);
            put(lds, z + 1, col, u[kN - 1][i]);
        }
        __syncthreads();
        TC ya[kN][VX], yb[kN][VX], za[kN][VX], zb[kN][VX];
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int y = ((wz * kN + i) * kW + wy) * 2, z = kZRows + ((wy * kN + i) * kW + wz) * 2;
            get(lds, wy > 0 ? y - 1 : kZero, col, ya[i]);
            get(lds, wy < kW - 1 ? y + 2 : kZero, col, yb[i]);
            get(lds, wz > 0 ? z - 1 : kZero, col, za[i]);
            get(lds, wz < kW - 1 ? z + 2 : kZero, col, zb[i]);
        }
        TC n[kN][kN][VX];
#pragma unroll
        for (int z = 0; z < kN; ++z)
#pragma unroll
            for (int y = 0; y < kN; ++y) {
                const TC l = from_lower_z(u[z][y][VX - 1]), r = from_upper_z(u[z][y][0]);
#pragma unroll
                for (int e = 0; e < VX; ++e) {
                    TC acc = w[0] * u[z][y][e];
                    acc = fma_c(w[1], z > 0 ? u[z > 0 ? z - 1 : 0][y][e] : za[y][e], acc);
                    acc = fma_c(w[2], y > 0 ? u[z][y > 0 ? y - 1 : 0][e] : ya[z][e], acc);
                    acc = fma_c(w[3], e > 0 ? u[z][y][e > 0 ? e - 1 : 0] : l, acc);
                    acc = fma_c(w[4], e + 1 < VX ? u[z][y][e + 1 < VX ? e + 1 : 0] : r, acc);
                    acc = fma_c(w[5], y + 1 < kN ? u[z][y + 1 < kN ? y + 1 : 0][e] : yb[z][e], acc);
                    acc = fma_c(w[6], z + 1 < kN ? u[z + 1 < kN ? z + 1 : 0][y][e] : zb[y][e], acc);
                    n[z][y][e] = S::round(acc);
                }
            }
#pragma unroll
        for (int z = 0; z < kN; ++z)
#pragma unroll
            for (int y = 0; y < kN; ++y)
#pragma unroll
                for (int e = 0; e < VX; ++e) u[z][y][e] = n[z][y][e];
        __syncthreads();
    }

    static __device__ __forceinline__ void run(const Brick3DArgs& a, TC* lds) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
        const int wy = wave % kW, wz = wave / kW, col = lane * VX;
        const uint32_t item = static_cast<uint32_t>(xcd_remap(blockIdx.x, gridDim.x));
        const uint32_t tyz = item / static_cast<uint32_t>(a.tiles[2]);
        const int32_t t[3] = {static_cast<int32_t>(tyz / static_cast<uint32_t>(a.tiles[1])),
                              static_cast<int32_t>(tyz % static_cast<uint32_t>(a.tiles[1])),
                              static_cast<int32_t>(item - tyz * a.tiles[2])};
        // owned cells and the brick's first, per axis z, y, x
        int32_t o0[3], o1[3], b0[3];
        const int32_t size[3] = {kEdge, kEdge, W};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            o0[d] = t[d] > 0 ? t[d] * a.own[d] + a.edge[d] : 0;
            o1[d] = t[d] + 1 < a.tiles[d] ? (t[d] + 1) * a.own[d] + a.edge[d] : a.n[d];
            b0[d] = o0[d] - a.halo[d];
            if (!PER) b0[d] = b0[d] < 0 ? 0 : (b0[d] + size[d] > a.n[d] ? a.n[d] - size[d] : b0[d]);
        }
        const int32_t nz = a.n[0], ny = a.n[1], nx = a.n[2];
        const int32_t xl = b0[2] + col, yw = b0[1] + wy * kN, zw = b0[0] + wz * kN;
        const uint32_t xo = static_cast<uint32_t>(PER ? wrap_idx(xl, nx) : xl) * sizeof(TS);
        TC u[kN][kN][VX];
#pragma unroll
        for (int z = 0; z < kN; ++z)
#pragma unroll
            for (int y = 0; y < kN; ++y) {
                const int32_t zz = PER ? wrap_idx(zw + z, nz) : zw + z, yy = PER ? wrap_idx(yw + y, ny) : yw + y;
                ld(rsrc(a.src, zz * ny + yy, nx), xo, u[z][y]);
            }
        for (int i = threadIdx.x; i < W; i += 64 * kW * kW) lds[kZero * W + i] = TC(0);
        TC w[7];
#pragma unroll
        for (int p = 0; p < 7; ++p) w[p] = static_cast<TC>(a.w[p]);
        for (int32_t k = 0; k < a.t; ++k) step(w, u, lds, wy, wz, col);
        const uint32_t so = xl + VX > o0[2] && xl < o1[2] ? xo : kOut;
#pragma unroll
        for (int z = 0; z < kN; ++z)
#pragma unroll
            for (int y = 0; y < kN; ++y)
                if (zw + z >= o0[0] && zw + z < o1[0] && yw + y >= o0[1] && yw + y < o1[1])
                    st(rsrc(a.dst, (zw + z) * ny + yw + y, nx), so, u[z][y]);
    }
};

template <typename TS, int VX, bool PER>
__global__ __launch_bounds__(64 * kW * kW) void brick3d_kernel(const Brick3DArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    using P = Brick<TS, VX, PER>;
    P::run(a, reinterpret_cast<typename P::TC*>(smem));
}

template <typename TS, int VX>
hipError_t go(bool per, const Brick3DArgs& a, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(a.tiles[0]) * static_cast<unsigned>(a.tiles[1]) * static_cast<unsigned>(a.tiles[2]));
    const dim3 block(64 * kW * kW);
    if (per) hipLaunchKernelGGL((brick3d_kernel<TS, VX, true>), grid, block, (Brick<TS, VX, true>::LDS_BYTES), s, a);
    else hipLaunchKernelGGL((brick3d_kernel<TS, VX, false>), grid, block, (Brick<TS, VX, false>::LDS_BYTES), s, a);
    return hipGetLastError();
}

}  // namespace b3

int brick3d_edge() { return b3::kEdge; }
int brick3d_lds_bytes(int dtype, int vx) {
    return dtype == kF64 ? b3::Brick<double, 1, false>::LDS_BYTES * vx : b3::Brick<float, 1, false>::LDS_BYTES * vx;
}

hipError_t launch_brick3d(int dtype, int vx, bool periodic, const Brick3DArgs& a, hipStream_t s) {
    if (dtype == kF64 && vx == 1) return b3::go<double, 1>(periodic, a, s);
    if (dtype == kF32 && vx == 1) return b3::go<float, 1>(periodic, a, s);
    if (dtype == kF32 && vx == 2) return b3::go<float, 2>(periodic, a, s);
    return hipErrorInvalidValue;
}

}  // namespace st
