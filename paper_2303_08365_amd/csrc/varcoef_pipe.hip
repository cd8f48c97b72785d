// varcoef_pipe.hip -- two steps of the variable-coefficient heat operator, or
// of its adjoint, per pass over memory.
//
// Tiling as in the constant-weight pipelines (paper Sec. 4.1: an xy tile held
// on chip while the work-group streams along z, advanced several steps before
// it returns to memory): lane L of wave w holds columns X0 + L*VX .. +VX-1 of
// rows Y0 + w*K .. +K-1.  A cell takes its six faces in the order z-, y-, y+,
// x-, x+, z+ (the order of every kernel of this operator, so all give the same
// bits): the face to plane z+1 comes last, so a step keeps its previous plane
// and that plane's sum short of one face; when plane z arrives, the face
// between the two finishes plane z-1 of the next step and begins plane z's
// sum.  A face's conductivity and difference are formed once and enter both
// cells, with opposite signs.  Step 2's plane follows one plane behind.
//
// The adjoint (lambda^{n+1} -> lambda^n -> lambda^{n-1}) is the same pair of
// steps on lambda; beside each, the sum of dL/dk takes the same faces with the
// differences of the state u^n (u^{n-1}) and of lambda.  dL/dk of plane z gets
// the two steps' terms one after the other, as two passes of one step would.
//
// Ghost layer: u and lambda are 0 there (loads outside the range, the zero that
// enters the wave through DPP, zero LDS rows; planes of step 1 outside the grid
// are set to 0).  k repeats the edge cell: clamped rows and planes, and DPP's old
// operand in x; then k / 2 + k / 2 = k makes the interior formula the edge term.
// In dL/dk the interior formula gives half of a ghost face's -u * lambda, and
// the adjoint adds the other half once per ghost face.
//
// The y neighbours of all fields go through LDS, one barrier per plane, two
// buffers alternating; rows outside the tile are loaded for step 1 and missing
// for step 2, so tiles overlap by one row and two columns a side (whole lanes),
// and edge tiles are moved inward to touch the grid's edge.
//
// What bounds it: the bytes, with the vector units close behind.  A forward
// pair moves 12 bytes a FP32 cell instead of 24 (16 where the state between is
// stored too), an adjoint pair 28 instead of 48; at 256^3 FP32 a pair takes 43
// us (55 with the state between), two single steps 90, and an adjoint pair 94
// instead of 172: 4.4 to 5.0 TB/s, where a copy reaches 5.2 to 5.9 (44 and 57 us
// before planes of k were halved as they arrive, which leaves a face's
// conductivity one addition).  FP64 256^3: 47 us a step instead of 82.  Taking a
// face's conductivity once for both cells brings a step from 25 to 16 operations
// a cell.  8 waves of 4 rows (2 in the
// adjoint, whose fields need the registers) are one work-group a CU: the
// rows re-read in y fall to 1/15 (1/7).
#include "dev_common.h"

namespace st {
namespace vcp {

template <typename T, int VX, int K, int NW, bool ADJ, bool MID>
struct Pipe {
    static_assert(!(ADJ && MID), "the state between two steps is stored by the forward form only");
    static constexpr int W = 64 * VX;
    static constexpr int H = NW * K;
    static constexpr int HX = (2 + VX - 1) / VX * VX;
    static constexpr int OUTW = W - 2 * HX, OUTH = H - 2;
    // LDS rows of a field: slot 0 above the tile, 2w+1 and 2w+2 the first and
    // last row of wave w, 2*NW+1 below the tile, 2*NW+2 a sink
    static constexpr int SLOTS = 2 * NW + 3;
    // fields exchanged: step 1's state and k, step 2's state; adjoint: step 1's u
    // (step 2's comes from memory a second time: a fifth field does not fit)
    static constexpr int NF = ADJ ? 4 : 3;
    static constexpr int FV = 0, FK = 1, FV1 = 2, FU = 3;
    static constexpr int FIELD = SLOTS * W, BUF = NF * FIELD;
    static constexpr int LDS_BYTES = 2 * BUF * static_cast<int>(sizeof(T));
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
    static constexpr uint32_t kOut = 0x80000000u;
    static constexpr int32_t kRsrcWord3 = 0x00020000;
    static constexpr int kNT = 2;

    struct Ctx {
        const T* v;    // u^n (forward) or lambda^{n+1} (adjoint)
        const T* k;
        const T* u;    // adjoint: u^n
        const T* u1;   // adjoint: u^{n-1}
        T* out;
        T* mid;        // MID: u^{n+1}
        T* grad;       // adjoint
        int32_t nz, zs, ze;
        int64_t plane_elems;
        uint32_t plane_bytes;
        uint32_t lo[K];     // the lane's columns in the wave's rows
        uint32_t so[K];     // same for the stores; kOut outside the owned cells
        uint32_t hz, hc;    // the wave's halo row: kOut where outside (zero fields), clamped (k)
        int hslot;          // its LDS slot
        uint32_t ra, rb;    // adjoint: the rows above and below the wave's; kOut where outside
        int lane, wave;
        T alpha;
        int ngy[K], ngx[VX];  // adjoint: ghost faces in y and x
    };

    static __device__ __forceinline__ bool zghost(int32_t z, int32_t nz) {
        return static_cast<uint32_t>(z) >= static_cast<uint32_t>(nz);
    }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane(const Ctx& c, const T* p, int32_t z, bool ok) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p) + static_cast<int64_t>(ok ? z : 0) * c.plane_elems, 0,
                                                 ok ? c.plane_bytes : 0, kRsrcWord3);
    }
    // 0 outside the grid / the nearest plane / empty outside the chunk
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_zero(const Ctx& c, const T* p, int32_t z) {
        return plane(c, p, z, !zghost(z, c.nz));
    }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_clamp(const Ctx& c, const T* p, int32_t z) {
        return plane(c, p, z < 0 ? 0 : (z < c.nz ? z : c.nz - 1), true);
    }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_own(const Ctx& c, T* p, int32_t z) {
        return plane(c, p, z, static_cast<uint32_t>(z - c.zs) < static_cast<uint32_t>(c.ze - c.zs));
    }
    static __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t r, uint32_t o, T (&v)[VX]) {
        constexpr int kBytes = VX * static_cast<int>(sizeof(T));
        if constexpr (kBytes == 16) {
            const u32x4 raw = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
            __builtin_memcpy(v, &raw, 16);
        } else if constexpr (kBytes == 8) {
            const u32x2 raw = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
            __builtin_memcpy(v, &raw, 8);
        } else {
            static_assert(kBytes == 4, "4, 8 or 16 bytes a lane");
            v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
        }
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t o, const T (&v)[VX]) {
        constexpr int kBytes = VX * static_cast<int>(sizeof(T));
        if constexpr (kBytes == 16) {
            u32x4 raw;
            __builtin_memcpy(&raw, v, 16);
            __builtin_amdgcn_raw_buffer_store_b128(raw, r, o, 0, kNT);
        } else if constexpr (kBytes == 8) {
            u32x2 raw;
            __builtin_memcpy(&raw, v, 8);
            __builtin_amdgcn_raw_buffer_store_b64(raw, r, o, 0, kNT);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), r, o, 0, kNT);
        }
    }
    template <int N>
    static __device__ __forceinline__ void copy(T (&d)[N][VX], const T (&s)[N][VX]) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) d[i][e] = s[i][e];
    }

    // (opaque: fused into a face's sum, k itself would have to stay beside it)
    static __device__ __forceinline__ void halve(T (&d)[VX], const T (&s)[VX]) {
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            d[e] = T(0.5) * s[e];
            asm("" : "+v"(d[e]));
        }
    }

    // The planes one iteration takes in: step 1's state and k (and u) of plane
    // z with the wave's halo row, u^{n-1} of plane z-1.
    struct In {
        T v[K][VX], k[K][VX], hv[VX], hk[VX];
        T u[ADJ ? K : 1][VX], hu[VX], u1[ADJ ? K : 1][VX];
    };
    static __device__ __forceinline__ void load(const Ctx& c, int32_t z, In& in) {
        const __amdgpu_buffer_rsrc_t rv = plane_zero(c, c.v, z), rk = plane_clamp(c, c.k, z);
#pragma unroll
        for (int i = 0; i < K; ++i) {
            ld(rv, c.lo[i], in.v[i]);
            ld(rk, c.lo[i], in.k[i]);
        }
        ld(rv, c.hz, in.hv);
        ld(rk, c.hc, in.hk);
        if constexpr (ADJ) {
            const __amdgpu_buffer_rsrc_t ru = plane_zero(c, c.u, z), r1 = plane_zero(c, c.u1, z - 1);
#pragma unroll
            for (int i = 0; i < K; ++i) {
                ld(ru, c.lo[i], in.u[i]);
                ld(r1, c.lo[i], in.u1[i]);
            }
            ld(ru, c.hz, in.hu);
        }
    }

    // One step's standing: its previous plane, that plane's sum short of the
    // z+ face; adjoint: the same for u and dL/dk.
    struct Level {
        T prev[K][VX], acc[K][VX];
        T uprev[ADJ ? K : 1][VX], gacc[ADJ ? K : 1][VX];
    };

    // Plane v (plane z of a step; u beside it) arrives; kz is the conductivity
    // of the faces between it and the previous plane.  out gets the step's
    // result on the previous plane, gout that plane's dL/dk sum.
    static __device__ __forceinline__ void zface(const Ctx& c, Level& s, const T (&v)[K][VX], const T (&u)[ADJ ? K : 1][VX],
                                                 const T (&kz)[K][VX], int ngz, T (&out)[K][VX],
                                                 T (&gout)[ADJ ? K : 1][VX]) {
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                const T d = v[i][e] - s.prev[i][e];
                out[i][e] = fma_c(c.alpha, fma_c(kz[i][e], d, s.acc[i][e]), s.prev[i][e]);
                s.acc[i][e] = fma_c(kz[i][e], -d, T(0));
                if constexpr (ADJ) {
                    // (u_f - u_c) / 2 * (lambda_c - lambda_f), alike from both sides
                    const T du = T(0.5) * (u[i][e] - s.uprev[i][e]);
                    const T g = fma_c(du, -d, s.gacc[i][e]);
                    const int ng = ngz + c.ngy[i] + c.ngx[e];
                    gout[i][e] = ng > 0 ? fma_c(T(-0.5) * static_cast<T>(ng) * s.uprev[i][e], s.prev[i][e], g) : g;
                    s.gacc[i][e] = fma_c(-du, d, T(0));
                }
            }
        copy(s.prev, v);
        if constexpr (ADJ) copy(s.uprev, u);
    }

    // x neighbours across the lane boundary: 0, or the lane's own edge value
    template <bool OWN>
    static __device__ __forceinline__ void sides(const T (&v)[VX], T& l, T& r) {
        if constexpr (OWN) {
            l = from_lower(v[VX - 1], v[0]);
            r = from_upper(v[0], v[VX - 1]);
        } else {
            l = from_lower_z(v[VX - 1]);
            r = from_upper_z(v[0]);
        }
    }
    static __device__ __forceinline__ T at(const T (&v)[VX], T l, T r, int e) {
        return e < 0 ? l : (e >= VX ? r : v[e < 0 ? 0 : (e >= VX ? 0 : e)]);
    }

    // The y and x faces of the level's newest plane (s.prev, s.uprev), with k
    // and the rows above and below.
    static __device__ __forceinline__ void yxfaces(Level& s, const T (&k)[K][VX], const T* lds, int base, int fv, const T* ka,
                                                   const T* kb, const T* ua, const T* ub) {
        T va[VX], vb[VX];
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            va[e] = lds[fv * FIELD + base + e];
            vb[e] = lds[fv * FIELD + base + 3 * W + e];
        }
        // faces below row i - 1: rows 0 .. K
#pragma unroll
        for (int i = 0; i <= K; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                const T v0 = i > 0 ? s.prev[i > 0 ? i - 1 : 0][e] : va[e], v1 = i < K ? s.prev[i < K ? i : 0][e] : vb[e];
                const T k0 = i > 0 ? k[i > 0 ? i - 1 : 0][e] : ka[e], k1 = i < K ? k[i < K ? i : 0][e] : kb[e];
                const T kap = k0 + k1, d = v1 - v0;
                T du = T(0);
                if constexpr (ADJ)
                    du = T(0.5) * ((i < K ? s.uprev[ADJ && i < K ? i : 0][e] : ub[e]) -
                                   (i > 0 ? s.uprev[ADJ && i > 0 ? i - 1 : 0][e] : ua[e]));
                // y+ of the row above comes after its y- (the previous i)
                if (i > 0) {
                    s.acc[i > 0 ? i - 1 : 0][e] = fma_c(kap, d, s.acc[i > 0 ? i - 1 : 0][e]);
                    if constexpr (ADJ) s.gacc[ADJ && i > 0 ? i - 1 : 0][e] = fma_c(du, -d, s.gacc[ADJ && i > 0 ? i - 1 : 0][e]);
                }
                if (i < K) {
                    s.acc[i < K ? i : 0][e] = fma_c(kap, -d, s.acc[i < K ? i : 0][e]);
                    if constexpr (ADJ) s.gacc[ADJ && i < K ? i : 0][e] = fma_c(-du, d, s.gacc[ADJ && i < K ? i : 0][e]);
                }
            }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            T vl, vr, kl, kr, ul = T(0), ur = T(0);
            sides<false>(s.prev[i], vl, vr);
            sides<true>(k[i], kl, kr);
            if constexpr (ADJ) sides<false>(s.uprev[ADJ ? i : 0], ul, ur);
            // faces left of column e: x+ of column e - 1 after its x-
#pragma unroll
            for (int e = 0; e <= VX; ++e) {
                const T kap = at(k[i], kl, kr, e - 1) + at(k[i], kl, kr, e);
                const T d = at(s.prev[i], vl, vr, e) - at(s.prev[i], vl, vr, e - 1);
                T du = T(0);
                if constexpr (ADJ) du = T(0.5) * (at(s.uprev[ADJ ? i : 0], ul, ur, e) - at(s.uprev[ADJ ? i : 0], ul, ur, e - 1));
                if (e > 0) {
                    s.acc[i][e > 0 ? e - 1 : 0] = fma_c(kap, d, s.acc[i][e > 0 ? e - 1 : 0]);
                    if constexpr (ADJ) s.gacc[ADJ ? i : 0][e > 0 ? e - 1 : 0] = fma_c(du, -d, s.gacc[ADJ ? i : 0][e > 0 ? e - 1 : 0]);
                }
                if (e < VX) {
                    s.acc[i][e < VX ? e : 0] = fma_c(kap, -d, s.acc[i][e < VX ? e : 0]);
                    if constexpr (ADJ) s.gacc[ADJ ? i : 0][e < VX ? e : 0] = fma_c(-du, d, s.gacc[ADJ ? i : 0][e < VX ? e : 0]);
                }
            }
        }
    }

    static __device__ __forceinline__ void put(T* row, const T (&v)[VX]) {
#pragma unroll
        for (int e = 0; e < VX; ++e) row[e] = v[e];
    }

    struct State {
        Level s0, s1;
        In in;
        T k[K][VX], kz[K][VX];       // half of the newest plane's k; its faces to the plane before
        T ka[VX], kb[VX];            // half of k above and below the wave's rows, newest plane
        T ghold[ADJ ? K : 1][VX];    // step 1's dL/dk of the plane step 2 finishes next
    };
    enum Phase { kFirst, kStep1, kBoth, kLast };

    // Plane z arrives.  kFirst: it only becomes the previous plane; kStep1: step
    // 2's plane too, whose faces in y and x are not needed; kLast: no plane follows.
    template <Phase PH>
    static __device__ __forceinline__ void iteration(const Ctx& c, int32_t z, T* buf, State& s) {
        const int own = (2 * c.wave) * W + c.lane * VX, hrow = c.hslot * W + c.lane * VX;
        T v[K][VX], k[K][VX], u[ADJ ? K : 1][VX], u1[ADJ ? K : 1][VX], gold[ADJ ? K : 1][VX], ua[VX], ub[VX];
        copy(v, s.in.v);
#pragma unroll
        for (int i = 0; i < K; ++i) halve(k[i], s.in.k[i]);
        if constexpr (ADJ) {
            copy(u, s.in.u);
            copy(u1, s.in.u1);
        }
        if constexpr (PH == kStep1 || PH == kBoth) {
            put(buf + FV * FIELD + hrow, s.in.hv);
            halve(s.in.hk, s.in.hk);
            put(buf + FK * FIELD + hrow, s.in.hk);
            if constexpr (ADJ) put(buf + FU * FIELD + hrow, s.in.hu);
        }
        if constexpr (ADJ && (PH == kBoth || PH == kLast)) {
            const __amdgpu_buffer_rsrc_t r1 = plane_zero(c, c.u1, z - 1), rg = plane_own(c, c.grad, z - 2);
#pragma unroll
            for (int i = 0; i < K; ++i) ld(rg, c.so[i], gold[i]);
            if constexpr (PH == kBoth) {
                ld(r1, c.ra, ua);
                ld(r1, c.rb, ub);
            }
        }
        if constexpr (PH != kLast) load(c, z + 1, s.in);
        if constexpr (PH == kFirst) {
            copy(s.s0.prev, v);
            copy(s.k, k);
            if constexpr (ADJ) copy(s.s0.uprev, u);
            return;
        }
        // step 1: plane z-1 of its result is whole
        T kz[K][VX], w1[K][VX], w2[K][VX], g0[ADJ ? K : 1][VX], g1[ADJ ? K : 1][VX];
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) kz[i][e] = k[i][e] + s.k[i][e];
        zface(c, s.s0, v, u, kz, (z - 1 == 0) + (z == c.nz), w1, g0);
        const bool ghost1 = zghost(z - 1, c.nz);
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) w1[i][e] = ghost1 ? T(0) : w1[i][e];
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PH == kStep1) {
            copy(s.s1.prev, w1);
            if constexpr (ADJ) copy(s.s1.uprev, u1);
        } else {
            if constexpr (MID) {
                const __amdgpu_buffer_rsrc_t r = plane_own(c, c.mid, z - 1);
#pragma unroll
                for (int i = 0; i < K; ++i) st(r, c.so[i], w1[i]);
            }
            // step 2: plane z-1 arrives
            zface(c, s.s1, w1, u1, s.kz, (z - 2 == 0) + (z - 1 == c.nz), w2, g1);
            const __amdgpu_buffer_rsrc_t r = plane_own(c, c.out, z - 2);
#pragma unroll
            for (int i = 0; i < K; ++i) st(r, c.so[i], w2[i]);
            if constexpr (ADJ) {
                const __amdgpu_buffer_rsrc_t rg = plane_own(c, c.grad, z - 2);
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    T g[VX];
#pragma unroll
                    for (int e = 0; e < VX; ++e)
                        g[e] = fma_c(c.alpha, g1[i][e], fma_c(c.alpha, s.ghold[i][e], gold[i][e]));
                    st(rg, c.so[i], g);
                }
                copy(s.ghold, g0);
            }
            if constexpr (PH == kLast) return;
        }
        __builtin_amdgcn_sched_barrier(0);
        // edge rows of every field, one barrier
        put(buf + FV * FIELD + own + W, v[0]);
        put(buf + FV * FIELD + own + 2 * W, v[K - 1]);
        put(buf + FK * FIELD + own + W, k[0]);
        put(buf + FK * FIELD + own + 2 * W, k[K - 1]);
        if constexpr (PH == kBoth) {
            put(buf + FV1 * FIELD + own + W, w1[0]);
            put(buf + FV1 * FIELD + own + 2 * W, w1[K - 1]);
        }
        if constexpr (ADJ) {
            put(buf + FU * FIELD + own + W, u[0]);
            put(buf + FU * FIELD + own + 2 * W, u[K - 1]);
        }
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        T ka[VX], kb[VX];
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            ka[e] = buf[FK * FIELD + own + e];
            kb[e] = buf[FK * FIELD + own + 3 * W + e];
        }
        if constexpr (PH == kBoth) yxfaces(s.s1, s.k, buf, own, FV1, s.ka, s.kb, ua, ub);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ADJ) {
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                ua[e] = buf[FU * FIELD + own + e];
                ub[e] = buf[FU * FIELD + own + 3 * W + e];
            }
        }
        yxfaces(s.s0, k, buf, own, FV, ka, kb, ua, ub);
        // step 2 forms this plane's face conductivities anew one trip later: kept,
        // they would not fit into the registers
        copy(s.k, k);
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) asm volatile("" : "+v"(s.k[i][e]));
        copy(s.kz, kz);
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            s.ka[e] = ka[e];
            s.kb[e] = kb[e];
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    static __device__ __forceinline__ void run(const VarcoefArgs& a, T* lds) {
        Ctx c;
        c.lane = threadIdx.x & 63;
        c.wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
        const uint32_t tiles = static_cast<uint32_t>(a.tiles_x) * a.tiles_y * a.chunks_z;
        const uint32_t item = static_cast<uint32_t>(xcd_remap(blockIdx.x, gridDim.x));
        if (item >= tiles) return;
        const uint32_t txy = item / static_cast<uint32_t>(a.tiles_x);
        const int32_t tx = static_cast<int32_t>(item - txy * a.tiles_x);
        const int32_t ty = static_cast<int32_t>(txy % static_cast<uint32_t>(a.tiles_y));
        const int32_t cz = static_cast<int32_t>(txy / static_cast<uint32_t>(a.tiles_y));
        const int32_t nx = static_cast<int32_t>(a.nx), ny = static_cast<int32_t>(a.ny);
        c.v = static_cast<const T*>(ADJ ? a.lam : a.u);
        c.k = static_cast<const T*>(a.k);
        c.u = static_cast<const T*>(a.u);
        c.u1 = static_cast<const T*>(a.u1);
        c.out = static_cast<T*>(a.out);
        c.mid = static_cast<T*>(a.mid);
        c.grad = static_cast<T*>(a.grad);
        c.nz = static_cast<int32_t>(a.nz);
        c.plane_elems = a.ny * a.nx;
        c.plane_bytes = static_cast<uint32_t>(c.plane_elems * static_cast<int64_t>(sizeof(T)));
        c.alpha = static_cast<T>(a.alpha);
        c.zs = cz * a.chunk_z;
        c.ze = c.zs + a.chunk_z < c.nz ? c.zs + a.chunk_z : c.nz;
        const int32_t ox0 = tx > 0 ? tx * OUTW + a.edge_x : 0, ox1 = tx + 1 < a.tiles_x ? (tx + 1) * OUTW + a.edge_x : nx;
        const int32_t oy0 = ty > 0 ? ty * OUTH + a.edge_y : 0, oy1 = ty + 1 < a.tiles_y ? (ty + 1) * OUTH + a.edge_y : ny;
        int32_t X0 = ox0 - HX, Y0 = oy0 - 1;
        X0 = X0 < 0 ? 0 : (X0 + W > nx ? nx - W : X0);
        Y0 = Y0 < 0 ? 0 : (Y0 + H > ny ? ny - H : Y0);
        const int32_t xl = X0 + c.lane * VX, yw = Y0 + c.wave * K;
        // whole lanes (the adjoint's dL/dk is read, added to and written by
        // exactly one tile: its rows are whole multiples of VX)
        const bool xown = xl + VX > ox0 && xl < ox1;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            c.lo[i] = static_cast<uint32_t>((yw + i) * nx + xl) * sizeof(T);
            c.so[i] = xown && yw + i >= oy0 && yw + i < oy1 ? c.lo[i] : kOut;
            c.ngy[i] = (yw + i == 0) + (yw + i == ny - 1);
        }
#pragma unroll
        for (int e = 0; e < VX; ++e) c.ngx[e] = (xl + e == 0) + (xl + e == nx - 1);
        {
            const bool top = c.wave == 0, bot = c.wave == NW - 1;
            const int32_t hy = top ? Y0 - 1 : Y0 + H;
            const bool in = static_cast<uint32_t>(hy) < static_cast<uint32_t>(ny);
            const int32_t hyc = hy < 0 ? 0 : (hy < ny ? hy : ny - 1);
            c.hz = (top || bot) && in ? static_cast<uint32_t>(hy * nx + xl) * sizeof(T) : kOut;
            c.hc = top || bot ? static_cast<uint32_t>(hyc * nx + xl) * sizeof(T) : kOut;
            if constexpr (ADJ) {
                c.ra = yw > 0 ? static_cast<uint32_t>((yw - 1) * nx + xl) * sizeof(T) : kOut;
                c.rb = yw + K < ny ? static_cast<uint32_t>((yw + K) * nx + xl) * sizeof(T) : kOut;
            }
            c.hslot = top ? 0 : (bot ? 2 * NW + 1 : 2 * NW + 2);
        }
        // step 2's rows outside the tile hold 0 for the whole pass
        for (int i = threadIdx.x; i < 2 * W; i += 64 * NW) {
            T* f = lds + (i / W) * BUF + FV1 * FIELD + i % W;
            f[0] = T(0);
            f[(2 * NW + 1) * W] = T(0);
        }
        State s;
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e) {
                s.s0.prev[i][e] = s.s0.acc[i][e] = s.s1.prev[i][e] = s.s1.acc[i][e] = T(0);
                s.k[i][e] = s.kz[i][e] = T(0);
            }
#pragma unroll
        for (int i = 0; i < (ADJ ? K : 1); ++i)
#pragma unroll
            for (int e = 0; e < VX; ++e)
                s.s0.uprev[i][e] = s.s0.gacc[i][e] = s.s1.uprev[i][e] = s.s1.gacc[i][e] = s.ghold[i][e] = T(0);
#pragma unroll
        for (int e = 0; e < VX; ++e) s.ka[e] = s.kb[e] = T(0);

        // planes zs-2 .. ze+1: plane z finishes plane z-1 of step 1 and plane
        // z-2 of step 2.  The first three and the last do only the part of it
        // that owned planes need.
        T* b0 = lds;
        T* b1 = lds + BUF;
        load(c, c.zs - 2, s.in);
        iteration<kFirst>(c, c.zs - 2, b0, s);
        iteration<kStep1>(c, c.zs - 1, b0, s);
        iteration<kStep1>(c, c.zs, b1, s);
        // two per trip: the planes change registers without being copied.  An odd
        // chunk takes in one plane more, whose stores fall outside the chunk.
        int32_t z = c.zs + 1;
        if constexpr (!ADJ) {
            for (; z <= c.ze; z += 2) {
                iteration<kBoth>(c, z, b0, s);
                iteration<kBoth>(c, z + 1, b1, s);
            }
        } else {
            for (; z <= c.ze; ++z) iteration<kBoth>(c, z, lds + ((z ^ c.zs) & 1 ? 0 : BUF), s);
        }
        iteration<kLast>(c, z, b0, s);
    }
};

// Work-groups of 8 waves a CU holds: by registers, 256 a lane with 16 bytes of a
// row per lane, else 128.
constexpr int wgs_per_cu(int lane_bytes) { return lane_bytes == 16 ? 1 : 2; }

template <typename T, int VX, int K, int NW, bool ADJ, bool MID>
__global__ __launch_bounds__(64 * NW, 2 * wgs_per_cu(VX * static_cast<int>(sizeof(T)))) void varcoef_pipe_kernel(const VarcoefArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    Pipe<T, VX, K, NW, ADJ, MID>::run(a, reinterpret_cast<T*>(smem));
}

constexpr int kNW = 8, kKF = 4, kKA = 2;  // waves; rows a wave, forward and adjoint

template <typename T, int VX, bool ADJ, bool MID>
void go(const VarcoefArgs& a, hipStream_t s) {
    constexpr int K = ADJ ? kKA : kKF;
    using P = Pipe<T, VX, K, kNW, ADJ, MID>;
    const int64_t wgs = static_cast<int64_t>(a.tiles_x) * a.tiles_y * a.chunks_z;
    hipLaunchKernelGGL((varcoef_pipe_kernel<T, VX, K, kNW, ADJ, MID>), dim3(static_cast<unsigned>(wgs)), dim3(64 * kNW),
                       P::LDS_BYTES, s, a);
}

template <typename T, int VX>
void pick(bool adjoint, const VarcoefArgs& a, hipStream_t s) {
    if (adjoint) go<T, VX, true, false>(a, s);
    else if (a.mid) go<T, VX, false, true>(a, s);
    else go<T, VX, false, false>(a, s);
}

}  // namespace vcp

VarcoefPipeShape varcoef_pipe_shape(int dtype, int vx, bool adjoint) {
    const int hx = (2 + vx - 1) / vx * vx, h = vcp::kNW * (adjoint ? vcp::kKA : vcp::kKF);
    const int esz = dtype == kF64 ? 8 : 4, fields = adjoint ? 4 : 3;
    return VarcoefPipeShape{64 * vx, h, 64 * vx - 2 * hx, h - 2, vcp::wgs_per_cu(vx * esz),
                            2 * fields * (2 * vcp::kNW + 3) * 64 * vx * esz};
}

hipError_t launch_varcoef_pipe(int dtype, int vx, bool adjoint, const VarcoefArgs& a, hipStream_t s) {
    const int64_t wgs = static_cast<int64_t>(a.tiles_x) * a.tiles_y * a.chunks_z;
    if (wgs <= 0) return hipSuccess;
    if (wgs >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    if (dtype == kF64 && vx == 2) vcp::pick<double, 2>(adjoint, a, s);
    else if (dtype == kF64 && vx == 1) vcp::pick<double, 1>(adjoint, a, s);
    else if (dtype == kF32 && vx == 4) vcp::pick<float, 4>(adjoint, a, s);
    else if (dtype == kF32 && vx == 1) vcp::pick<float, 1>(adjoint, a, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace st
