// naive.hip -- one time step per launch for any point list (ndim 1..3,
// radius <= 4, up to 125 points), one thread per cell.  This is the plain
// form of the sweep (paper Sec. 2.1, Alg. 1: every cell becomes the weighted
// sum of its pattern neighbours from the previous step) and the bitwise
// reference for the fused kernels: it evaluates the canonical point order
// with the same multiply / fma chain and the same ghost-cell zeros.
//
// rows_kernel: a wave takes 64 to 256 cells of one row (1, 2 or 4 a lane), so
// a point's row is wave-uniform.  The row is read through a buffer descriptor
// whose range is the row, empty outside the grid: zero-rule ghost cells load
// as 0 and a point costs one address add, one load and one FMA a cell, the
// rest scalar and shared by the lane's cells.  A batch of 8 to 16 points' loads
// is in flight before the first is used.  Bound by the launch at few cells, by
// the L1's loads at many.  Against index divisions and range tests per lane and
// point, FP64 / FP32: 27 points 256^3 415 / 396 -> 199 / 67 us; 7 points 512^3
// 1263 / 1148 -> 660 / 256 us, 64^3 6.0 -> 4.6 / 4.3 us; 25-point star 200^3
// 207 / 194 -> 118 / 42 us.  naive_kernel, with 64-bit indices, keeps the grids
// beyond rows_kernel's 32-bit rows and launch limits.
#include <type_traits>

#include "dev_common.h"

namespace st {

template <typename TS>
__global__ __launch_bounds__(256) void naive_kernel(const NaiveArgs a) {
    using S = Storage<TS>;
    using TC = typename S::TC;
    const ST_GLOBAL TS* src = gptr<TS>(a.src);
    ST_GLOBAL TS* dst = gptr_mut<TS>(a.dst);
    const int64_t nz = a.n[0], ny = a.n[1], nx = a.n[2];
    const int64_t cells = nz * ny * nx;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < cells;
         i += stride) {
        const int64_t x = i % nx;
        const int64_t y = (i / nx) % ny;
        const int64_t z = i / (nx * ny);
        TC acc = TC(0);
        for (int p = 0; p < a.npoints; ++p) {
            int64_t zz = z + a.off[p][0], yy = y + a.off[p][1], xx = x + a.off[p][2];
            TC v = TC(0);
            const bool out = zz < 0 || zz >= nz || yy < 0 || yy >= ny || xx < 0 || xx >= nx;
            if (a.bc == kPeriodic) {
                zz = wrap_idx(zz, nz);
                yy = wrap_idx(yy, ny);
                xx = wrap_idx(xx, nx);
                v = ld1(src + (zz * ny + yy) * nx + xx);
            } else if (!out) {
                v = ld1(src + (zz * ny + yy) * nx + xx);
            }
            const TC w = static_cast<TC>(a.w[p]);
            acc = (p == 0) ? w * v : fma_c(w, v, acc);
        }
        st1(dst + i, acc);
    }
}

// the last n < kBatch points as one batch
template <int N, typename F>
__device__ __forceinline__ void tail_batch(int n, int p, const F& batch) {
    if constexpr (N > 0) {
        if (n == N) batch(p, std::integral_constant<int, N>{});
        else tail_batch<N - 1>(n, p, batch);
    }
}

// V columns a lane, 64 apart; WX waves of a work-group side by side along x,
// 4 / WX rows.
template <typename TS, bool PER, int V, int WX>
__global__ __launch_bounds__(256) void rows_kernel(const NaiveArgs) {
    using S = Storage<TS>;
    using TC = typename S::TC;
    // the argument block where it lies, in the kernel-argument segment: named
    // as a parameter, its many indexed uses would make a private copy of it
    const auto a = (const __attribute__((address_space(4))) NaiveArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int kBatch = 32 / V < 16 ? 32 / V : 16;  // points whose loads are in flight together
    constexpr int32_t kRsrcWord3 = 0x00020000;         // gfx9: raw 32-bit data
    constexpr uint32_t kE = static_cast<uint32_t>(sizeof(TS));
    const int32_t nz = static_cast<int32_t>(a->n[0]), ny = static_cast<int32_t>(a->n[1]), nx = static_cast<int32_t>(a->n[2]);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int32_t z = static_cast<int32_t>(blockIdx.z);
    const int32_t y = static_cast<int32_t>(blockIdx.y) * (4 / WX) + wave / WX;
    const int32_t x0 = (static_cast<int32_t>(blockIdx.x) * WX + wave % WX) * (64 * V);
    if (y >= ny || x0 >= nx) return;
    const int32_t x = x0 + static_cast<int32_t>(threadIdx.x & 63);
    const uint32_t row_bytes = static_cast<uint32_t>(nx) * kE;
    const auto row_at = [&](int32_t zz, int32_t yy) { return (static_cast<int64_t>(zz) * ny + yy) * nx; };
    const TS* own = static_cast<const TS*>(a->src) + row_at(z, y);
    const auto load = [&](int p, TC (&v)[V]) {
        int32_t zz = z + a->off[p][0], yy = y + a->off[p][1];
        const int32_t dx = a->off[p][2];
        const TS* base;
        uint32_t range = row_bytes;
        if constexpr (PER) {
            zz = zz < 0 ? zz + nz : (zz >= nz ? zz - nz : zz);  // one extent at most (launch_naive checks)
            yy = yy < 0 ? yy + ny : (yy >= ny ? yy - ny : yy);
            base = static_cast<const TS*>(a->src) + row_at(zz, yy);
        } else {
            // outside the grid the range is empty and the address unused
            base = own + a->lin[p];
            if (static_cast<uint32_t>(zz) >= static_cast<uint32_t>(nz) || static_cast<uint32_t>(yy) >= static_cast<uint32_t>(ny))
                range = 0;
        }
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<TS*>(base), 0, range, kRsrcWord3);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            // lanes past the row's end may stay outside, the store drops them
            int32_t xx = x + 64 * k + dx;
            if constexpr (PER) xx = xx < 0 ? xx + nx : (xx >= nx ? xx - nx : xx);
            const uint32_t o = static_cast<uint32_t>(xx) * kE;
            if constexpr (sizeof(TS) == 8) v[k] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
            else if constexpr (sizeof(TS) == 4) v[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
            else v[k] = bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(r, o, 0, 0));
        }
    };
    // N points from p on, straight-line: all loads, then the chain
    TC acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = TC(0);
    const auto batch = [&](int p, auto count) {
        constexpr int N = decltype(count)::value;
        TC v[N][V];
#pragma unroll
        for (int j = 0; j < N; ++j) load(p + j, v[j]);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const TC w = static_cast<TC>(a->w[p + j]);
#pragma unroll
            for (int k = 0; k < V; ++k) acc[k] = p + j == 0 ? w * v[j][k] : fma_c(w, v[j][k], acc[k]);
        }
    };
    int p = 0;
    for (; p + kBatch <= a->npoints; p += kBatch) batch(p, std::integral_constant<int, kBatch>{});
    tail_batch<kBatch - 1>(a->npoints - p, p, batch);
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(static_cast<TS*>(a->dst) + row_at(z, y), 0, row_bytes, kRsrcWord3);
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const TS o = S::narrow(acc[k]);
        const uint32_t so = static_cast<uint32_t>(x + 64 * k) * kE;  // past the row: dropped
        if constexpr (sizeof(TS) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), r, so, 0, 0);
        else if constexpr (sizeof(TS) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o), r, so, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, o), r, so, 0, 0);
    }
}

namespace {
template <typename TS, int V, int WX>
void launch_rows(const NaiveArgs& a, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>((a.n[2] + 64 * V * WX - 1) / (64 * V * WX)),
                    static_cast<unsigned>((a.n[1] + 4 / WX - 1) / (4 / WX)), static_cast<unsigned>(a.n[0]));
    if (a.bc == kPeriodic) hipLaunchKernelGGL((rows_kernel<TS, true, V, WX>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((rows_kernel<TS, false, V, WX>), grid, dim3(256), 0, s, a);
}

// Four columns a lane share a point's scalar work (row address and range: the
// limit with one column, 45 Gcell/s for 27 points at any type) on rows that
// fill them; fewer on short rows, and one on a single row (1D), where the
// waves side by side are what there is to spread.
template <typename TS>
void launch_rows_v(const NaiveArgs& a, hipStream_t s) {
    if (a.n[1] == 1 && a.n[0] == 1) launch_rows<TS, 1, 4>(a, s);
    else if (a.n[2] > 128) launch_rows<TS, 4, 1>(a, s);
    else if (a.n[2] > 64) launch_rows<TS, 2, 1>(a, s);
    else launch_rows<TS, 1, 1>(a, s);
}
}  // namespace

hipError_t launch_naive(int dtype, NaiveArgs& a, hipStream_t s) {
    // rows below 2 GiB (32-bit offsets; a ghost column's offset wraps past
    // them), grid dimensions a launch takes, and offsets that wrap around an
    // extent at most once
    const int64_t esz = dtype == kF64 ? 8 : (dtype == kF32 ? 4 : 2);
    bool once = true;
    for (int p = 0; p < a.npoints; ++p)
        for (int d = 0; d < 3; ++d) once = once && (a.off[p][d] < 0 ? -a.off[p][d] : a.off[p][d]) <= a.n[d];
    for (int p = 0; p < a.npoints; ++p)
        a.lin[p] = (static_cast<int64_t>(a.off[p][0]) * a.n[1] + a.off[p][1]) * a.n[2];
    if (once && a.n[2] * esz < (int64_t(1) << 31) - 1024 && a.n[2] < (int64_t(1) << 30) && a.n[1] <= 4 * 65535 &&
        a.n[0] <= 65535) {
        switch (dtype) {
            case kF64: launch_rows_v<double>(a, s); break;
            case kF32: launch_rows_v<float>(a, s); break;
            case kBF16: launch_rows_v<bf16s>(a, s); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    const int64_t cells = a.n[0] * a.n[1] * a.n[2];
    int64_t blocks = (cells + 255) / 256;
    if (blocks > (int64_t(1) << 20)) blocks = int64_t(1) << 20;
    if (blocks < 1) blocks = 1;
    const dim3 grid(static_cast<unsigned>(blocks)), block(256);
    switch (dtype) {
        case kF64: hipLaunchKernelGGL(naive_kernel<double>, grid, block, 0, s, a); break;
        case kF32: hipLaunchKernelGGL(naive_kernel<float>, grid, block, 0, s, a); break;
        case kBF16: hipLaunchKernelGGL(naive_kernel<bf16s>, grid, block, 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace st
