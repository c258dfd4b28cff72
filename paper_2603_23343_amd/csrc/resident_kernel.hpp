// resident_kernel.hpp -- Jacobi-PCG with the whole grid held on the chip.
//
// The paper keeps a solve's vectors in the cores' SRAM for all iterations
// (Sec. VII); MI355X has 128 MiB of vector registers and 40 MiB of LDS, so a
// grid of up to ~4 M points fits as well (160^3; flat ones of fewer points may
// not, since only z is split within a thread). One persistent launch runs every
// iteration: a work-group owns a box of the grid, r, p, q and the FP64 x of its
// points live in registers, the current direction p (with a one-point halo)
// in LDS. Per iteration only scalars and the boxes' surfaces leave a CU.
//
// One iteration (the two-kernel form's arithmetic, pcg.hip):
//   p = D^-1 r + beta p on own points and on the halo (each box keeps the
//   residual of its halo points itself, from the neighbours' last q), q = A p,
//   partials of p.q;                                   -- grid sum: alpha
//   x += alpha p, r -= alpha q on own points, partials of r.r;
//                                                      -- grid sum: beta
// The box's surface values of q leave during the first sum and have arrived
// before the second; the neighbours read them while they form their own p. So
// one surface exchange serves an iteration and neither its stores nor its
// loads are waited for alone. Published before the first sum and read after
// it, an iteration on 512 x 112 x 64 took 12.0 us instead of 9.8 (boxes inside
// the grid have six surfaces to send and the others waited for them), at 128^3
// with cell coefficients 10.2 instead of 7.6, at 32^3 3.9 instead of 3.6 (9.7,
// 7.4 and 3.6 with the stores' addresses formed where they are used).
//
// What bounds an iteration: the two grid sums (1.1 us over 8 work-groups, 2.7
// over 256), then, in wide boxes, the stencil's five LDS accesses per point
// (3500 clocks for 32 points per thread, 2560 at the LDS's rate). 512 threads
// with up to 256 registers each hold the most points per CU.
//
// Grid sum: every work-group stores its FP64 partial and the sum's number in
// its own slot (two 8-byte words, each half a double and the number, so a
// word is valid exactly when its number matches) and polls all slots; all
// add the partials in the same order and hold the same bits. Data that
// crosses work-groups is written and read with agent-scope accesses, which go
// past the XCDs' L2s, and a wave waits for its surface stores before its
// work-group's slot is written: no fence, whose L2 write-back costs ~40 ns per
// work-group. The work-groups must run at the same time: at most one per CU is
// launched (the host reserves them, resident.hpp), and every wait is bounded;
// a work-group that waited too long raises a flag and leaves, and the host
// runs the solve in another form instead.
#pragma once

#include "ops.hpp"
#include "resident.hpp"

namespace pcgmi {

namespace resident {

constexpr int RT = 512;     // threads per work-group
constexpr int RW = RT / 64;  // wavefronts
constexpr int AGENT = 16;  // cache policy of a buffer access: agent scope (sc1)

using Words4 = __attribute__((ext_vector_type(4))) uint32_t;
using Words2 = __attribute__((ext_vector_type(2))) uint32_t;
using Buf = __amdgpu_buffer_rsrc_t;

__device__ __forceinline__ Buf make_buf(void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000);
}

// Sum over the wavefront in a fixed order: row shifts and row broadcasts (DPP)
// leave the total in lane 63. An FP64 butterfly over the LDS crossbar takes
// about three times as long, and four of these sit on an iteration's
// critical path.
template <int CTRL, int ROW> __device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW, 0xf, false);
    return v + __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ double wave_total(double v) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add<0x112, 0xf>(v);  // row_shr:2
    v = dpp_add<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add<0x118, 0xf>(v);  // row_shr:8
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31
    return v;                    // lane 63
}

// A value that is the same in every lane, kept in scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

struct SumLds {
    double wave[2][RES_SUMS][RW];  // the work-group's wavefront sums, per set
    double slot[RES_SUMS][RW];     // sums of the slots, per polling wavefront
    int bad;
};

// First part of a grid sum: wavefront sums to LDS. Two sets (of LDS and of
// slots) take turns, so that a work-group may enter the next sum while others
// still read the last one.
template <int NC> __device__ __forceinline__ void sum_local(const double (&v)[NC], SumLds& L, int set) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const double s = wave_total(v[c]);
        if ((threadIdx.x & 63) == 63) L.wave[set][c][threadIdx.x >> 6] = s;
    }
}

// Slots: [set][copy][component][work-group], 16 bytes each.
__device__ __forceinline__ int slot_at(int set, int copy, int c, int rank, int G) {
    return (((set * RES_COPIES + copy) * RES_SUMS + c) * res_slot_pitch(G) + rank) * 16;
}

// The first threads store the work-group's partial in every copy (after a
// __syncthreads that follows sum_local).
template <int NC>
__device__ __forceinline__ void sum_publish(SumLds& L, Buf slots, int set, int rank, int G, uint32_t no) {
    if (G > 1 && threadIdx.x < RES_COPIES) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double s = L.wave[set][c][0];
#pragma unroll
            for (int w = 1; w < RW; ++w) s += L.wave[set][c][w];
            const uint64_t b = __builtin_bit_cast(uint64_t, s);
            __builtin_amdgcn_raw_buffer_store_b128(Words4{no, (uint32_t)(b >> 32), no, (uint32_t)b}, slots,
                                                   slot_at(set, threadIdx.x, c, rank, G), 0, AGENT);
        }
    }
}

// Last part: wait for all slots and add them; false after a timeout.
template <int NC>
__device__ __forceinline__ bool sum_collect(double (&tot)[NC], SumLds& L, Buf slots, int set, int rank, int G,
                                            uint32_t no, long long wait) {
    const int t = threadIdx.x, wid = t >> 6;
    const int nw = (G + 63) >> 6;
    if (G == 1) {  // a lone work-group: its own sums are the totals
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double s = L.wave[set][c][0];
            for (int w = 1; w < RW; ++w) s += L.wave[set][c][w];
            tot[c] = uniform(s);
        }
        return true;
    }
    if (wid < nw) {
        double s[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) s[c] = 0.0;
        if (t < G) {
            Words4 a[NC];
            const long long began = wall_clock64();
            for (;;) {
                bool ok = true;
                __asm__ volatile("" ::: "memory");  // the loads stay in the loop
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    a[c] = __builtin_amdgcn_raw_buffer_load_b128(slots, slot_at(set, rank & (RES_COPIES - 1), c, t, G), 0,
                                                                 AGENT);
#pragma unroll
                for (int c = 0; c < NC; ++c) ok = ok && a[c].x == no && a[c].z == no;
                if (ok) break;
                if (wall_clock64() - began > wait) {
                    L.bad = 1;
                    break;
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
                s[c] = __builtin_bit_cast(double, ((uint64_t)a[c].y << 32) | a[c].w);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double w = wave_total(s[c]);
            if ((t & 63) == 63) L.slot[c][wid] = w;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        double s = L.slot[c][0];
        for (int w = 1; w < nw; ++w) s += L.slot[c][w];
        tot[c] = uniform(s);
    }
    return __builtin_amdgcn_readfirstlane(L.bad) == 0;
}

__device__ __forceinline__ uint32_t word(float v, int) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ uint32_t word(double v, int h) {
    return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> (32 * h));
}
__device__ __forceinline__ float value(Words4 w, int e, float) {
    const uint32_t u = w[e];
    return __builtin_bit_cast(float, u);
}
__device__ __forceinline__ double value(Words4 w, int e, double) {
    return __builtin_bit_cast(double, ((uint64_t)w[2 * e + 1] << 32) | w[2 * e]);
}

// N consecutive values of C to byte offset off of a buffer.
template <typename C, int N> __device__ __forceinline__ void put_run(Buf b, int off, const C (&v)[N]) {
    constexpr int P = (int)sizeof(C) / 4;  // words per value
#pragma unroll
    for (int i = 0; i < N * P / 4; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(Words4{word(v[(4 * i) / P], 0), word(v[(4 * i + 1) / P], 1 % P),
                                                      word(v[(4 * i + 2) / P], 0), word(v[(4 * i + 3) / P], 1 % P)},
                                               b, off + 16 * i, 0, AGENT);
    constexpr int done = (N * P / 4) * 4 / P, left = N * P % 4;  // 0 or 2 words
    if constexpr (left == 2)
        __builtin_amdgcn_raw_buffer_store_b64(Words2{word(v[done], 0), word(v[done + 2 / P - 1], 1 % P)}, b,
                                              off + 16 * (N * P / 4), 0, AGENT);
}
__device__ __forceinline__ void put_one(Buf b, int off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(word(v, 0), b, off, 0, AGENT);
}
__device__ __forceinline__ void put_one(Buf b, int off, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(Words2{word(v, 0), word(v, 1)}, b, off, 0, AGENT);
}

// Element i of an array of T behind a buffer, 0 where ok is false: the offset
// then lies past the buffer's end, which loads as 0 and stores nothing, so a
// run of predicated accesses needs no branches.
template <typename T, int POLICY = 0> __device__ __forceinline__ T get_at(Buf b, int i, bool ok) {
    const int off = ok ? i * (int)sizeof(T) : -1;
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, POLICY));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, POLICY));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(b, off, 0, POLICY));
}
template <typename T, int POLICY = 0> __device__ __forceinline__ void set_at(Buf b, int i, bool ok, T v) {
    const int off = ok ? i * (int)sizeof(T) : -1;
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(Words2, v), b, off, 0, POLICY);
    else if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), b, off, 0, POLICY);
    else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), b, off, 0, POLICY);
}

// A solve with ||r||^2 = rr over n points is scaled by 2^scale_of(rr, n): 0
// while the mean square lies within 2^-60 .. 2^60, else what brings it to about
// 1. The partial sums are FP32 squares, which underflow below 1e-19 and overflow
// above 1e19; within the bounds they stay normal numbers to a relative residual
// of 1e-9. Multiplying by a power of two commutes with every rounding, so a
// scaled solve has the bits of an unscaled one wherever that is in range.
__device__ __forceinline__ int scale_of(double rr, double n) {
    const double ms = rr / n;
    if (!(ms > 0.0) || !isfinite(ms)) return 0;
    const int e = __builtin_amdgcn_readfirstlane(ilogb(ms));
    return abs(e) <= 60 ? 0 : -(e / 2);
}
__device__ __forceinline__ float times_2(float v, int e) { return __builtin_amdgcn_ldexpf(v, e); }
__device__ __forceinline__ double times_2(double v, int e) { return __builtin_amdgcn_ldexp(v, e); }

// The thread's index, formed anew: what is derived from it is computed where
// it is used. Addresses kept over an iteration, or hoisted out of it, are
// spilled, and a reload among the surface stores waits until the stores before
// it have arrived.
__device__ __forceinline__ int fresh_thread() {
    int u = threadIdx.x;
    __asm__ volatile("" : "+v"(u));
    return u;
}

// Face coefficients of a thread's points (variable operator), computed once.
template <typename C, int V, bool VAR> struct Faces {
    C l[V], r[V], d[V], u[V], z[V + 1];
};
template <typename C, int V> struct Faces<C, V, false> {};

// One work-group's part (box `rank`) of a solve. T: storage type, X: the x
// accumulator's type in memory (FP64 registers), V z points per thread, 2^LX x
// 2^LY threads along x and y (the rest along z). False when a wait ran out.
template <typename T, typename X, int V, bool VAR, int LX, int LY>
__device__ __forceinline__ bool solve_box(const ResTask& a, const int rank, unsigned char* dyn, SumLds& L) {
    using C = typename Traits<T>::C;
    using Sh = ResShape<LX, LY, V>;
    constexpr int TX = Sh::TX, TY = Sh::TY, ZR = Sh::ZR, ZP = Sh::ZP, PX = Sh::PX, PP = Sh::PP;
    constexpr int NXF = Sh::NXF, NYF = Sh::NYF, NZF = Sh::NZF, S = Sh::S;
    constexpr int GN = 16 / (int)sizeof(C);            // halo points per group (one 16-byte load)
    constexpr int HG = (S / GN + RT - 1) / RT;         // groups per thread
    static_assert(HG * RT * sizeof(int) <= RES_HALO_LDS);
    constexpr int NB = VAR ? 2 : 1;
    constexpr bool JUDGE = sizeof(X) == 8;
    const ResGeo& g = a.geo;
    const bool judge = JUDGE && a.judge;
    SolveState* const st = a.st;
    double* const hist = a.hist;
    const int G = g.G;
    C* tile = reinterpret_cast<C*>(dyn);               // [ZP + 2][TY + 2][TX + 2]
    double* xlds = reinterpret_cast<double*>(tile + ((PP * (ZP + 2) + 1) & ~1));  // [V][RT] (VAR)
    int* hgi = reinterpret_cast<int*>(xlds + (VAR ? V * RT : 0));  // [HG][RT]

    // Scalars of the recursion: from the solve state when the start was made
    // by other kernels, else (judge) formed here from b.
    double rr0 = 0.0, tol2 = 0.0, dconst = 1.0 / 6.0, rho = 0.0, beta_d = 0.0, rr = 0.0, stag_best = 0.0;
    int maxit = a.maxit, stag = 0, iters = 0, done = 0, stag_at = 0;
    int scale = 0;  // r, p, q and x are 2^scale times the system's; rr, rho, sigma and tol2 4^scale times
    if (!judge) {
        if (st->done != 0 || st->maxit <= 0) {  // the same in every work-group
            if (rank == 0 && threadIdx.x == 0) {
                a.out->used = 0;
                a.out->ticks1 = a.out->ticks2 = 0;
            }
            return true;
        }
        scale = scale_of(st->rr, (double)g.nx * g.ny * g.nz);
        rr0 = uniform(times_2(st->rr0, 2 * scale));
        tol2 = uniform(times_2(st->tol2, 2 * scale));
        dconst = uniform(st->dinv);
        maxit = st->maxit;
        stag = st->stag;
        rho = uniform(times_2(st->rho, 2 * scale));
        beta_d = uniform(st->beta);
        rr = uniform(times_2(st->rr, 2 * scale));
        stag_best = uniform(st->stag_best);
        iters = st->iters;
        stag_at = st->stag_at;
    }
    const int first = iters;
    int seg0 = iters;  // iterations when the residual was last loaded
    const long long t_begin = judge ? wall_clock64() : 0;
    double sigma = 0.0, alpha_d64 = 0.0;

    const int t = threadIdx.x;
    const int tx = t & (TX - 1), ty = (t >> LX) & (TY - 1), tz = t >> (LX + LY);
    const int cx = rank % g.gx, cy = (rank / g.gx) % g.gy, cz = rank / (g.gx * g.gy);
    const int ox = cx * g.bx, oy = cy * g.by, oz = cz * g.bz;
    const int ex = min(g.bx, g.nx - ox), ey = min(g.by, g.ny - oy), ez = min(g.bz, g.nz - oz);
    const int z0 = tz * V;
    const bool act = tx < ex && ty < ey && z0 < ez;
    const int nv = act ? min(V, ez - z0) : 0;
    const bool full = __syncthreads_and(nv == V) != 0;  // no masking needed in this box (also: LDS is free)
    // The thread's first point in the grid, its index and its number of points,
    // formed anew where memory is accessed: offsets and masks kept from the
    // start, or hoisted, would take registers from the iteration.
    struct Own {
        int x, y, z, gi, nv;
    };
    auto own = [&]() {
        const int u = fresh_thread();
        const int ux = u & (TX - 1), uy = (u >> LX) & (TY - 1), uz = (u >> (LX + LY)) * V;
        Own o{ox + ux, oy + uy, oz + uz, 0, 0};
        o.gi = (o.z * g.ny + o.y) * g.nx + o.x;
        o.nv = ux < ex && uy < ey && uz < ez ? min(V, ez - uz) : 0;
        return o;
    };
    const int lb = (z0 + 1) * PP + (ty + 1) * PX + tx + 1;
    // the cell above the thread's last point (the top halo is the tile's last plane)
    const int zt = z0 + nv == ez ? (ZP + 1) * PP + (ty + 1) * PX + tx + 1 : lb + V * PP;
    const bool hxl = cx > 0, hxr = cx + 1 < g.gx, hyl = cy > 0, hyr = cy + 1 < g.gy, hzl = cz > 0, hzr = cz + 1 < g.gz;
    const uint32_t half = (uint32_t)g.G * S * (uint32_t)sizeof(C);
    const Buf slots = make_buf(a.slots, res_slot_bytes(G));
    const Buf surf = make_buf(a.surf, 2 * half);
    // the grid's arrays (resident_plan keeps them below 2 GiB)
    const uint32_t npts = (uint32_t)g.nx * g.ny * g.nz;
    const Buf bbuf = make_buf(const_cast<void*>(a.r), npts * (uint32_t)sizeof(T));
    const Buf r2buf = make_buf(a.r2, judge ? npts * (uint32_t)sizeof(T) : 0u);
    const Buf xbuf = make_buf(a.x, npts * (uint32_t)sizeof(X));
    const Buf dbuf = make_buf(const_cast<void*>(a.dinv), VAR ? npts * (uint32_t)sizeof(T) : 0u);
    const Buf kbuf = make_buf(const_cast<float*>(a.kc), VAR ? npts * 4u : 0u);

    for (int i = t; i < PP * (ZP + 2); i += RT) tile[i] = C(0);
    if (t == 0) L.bad = 0;

    // Halo groups of this thread: GN points along z (x and y faces) or along
    // x (z faces). hl: tile index of the first (-1: none), hz: its step; hs:
    // byte offset of the neighbour's values; hgi: the first point's index in the
    // grid (LDS); rh: the points' residuals.
    // Points of a group outside the box are carried along in halo cells that
    // no point reads (the tile has ZP + 2 planes).
    int hl[HG], hs[HG], hz[HG];
    C rh[HG][GN], dh[VAR ? HG : 1][GN];
#pragma unroll
    for (int m = 0; m < HG; ++m) {
        int j = (t + m * RT) * GN;
        hl[m] = -1;
        hs[m] = 0;
        hz[m] = PP;
#pragma unroll
        for (int e = 0; e < GN; ++e) {
            rh[m][e] = C(0);
            if constexpr (VAR) dh[m][e] = C(0);
        }
        if (j >= S) continue;
        int x, y, z, from, face;  // box coordinates of the first point, neighbour's rank and face
        bool ok;
        int sx = 0;
        if (j < 2 * NXF) {
            const bool hi = j >= NXF;
            j -= hi ? NXF : 0;
            y = j / ZP;
            z = j % ZP;
            x = hi ? ex : -1;
            ok = (hi ? hxr : hxl) && y < ey && z < ez;
            from = rank + (hi ? 1 : -1);
            face = hi ? 0 : NXF;
        } else if (j < 2 * (NXF + NYF)) {
            j -= 2 * NXF;
            const bool hi = j >= NYF;
            j -= hi ? NYF : 0;
            x = j / ZP;
            z = j % ZP;
            y = hi ? ey : -1;
            ok = (hi ? hyr : hyl) && x < ex && z < ez;
            from = rank + (hi ? g.gx : -g.gx);
            face = 2 * NXF + (hi ? 0 : NYF);
        } else {
            j -= 2 * (NXF + NYF);
            const bool hi = j >= NZF;
            j -= hi ? NZF : 0;
            y = j / TX;
            x = j % TX;
            z = hi ? ez : -1;
            ok = (hi ? hzr : hzl) && x < ex && y < ey;
            from = rank + (hi ? g.gx * g.gy : -g.gx * g.gy);
            face = 2 * (NXF + NYF) + (hi ? 0 : NZF);
            sx = 1;
            hz[m] = 1;
        }
        if (ok) {
            hs[m] = (from * S + face + j) * (int)sizeof(C);
            hl[m] = (z == ez ? ZP + 1 : z + 1) * PP + (y + 1) * PX + x + 1;
        }
        hgi[m * RT + t] = ((oz + z) * g.ny + (oy + y)) * g.nx + ox + x;
        if constexpr (VAR)
#pragma unroll
            for (int e = 0; e < GN; ++e) dh[m][e] = to_c(get_at<T>(dbuf, hgi[m * RT + t] + e * (sx ? 1 : g.nx * g.ny), ok));
    }

    // own points
    const int gp = ((oz + z0) * g.ny + (oy + ty)) * g.nx + ox + tx;
    const int gz = g.nx * g.ny;
    C r[V], p[V], q[V], dv[VAR ? V : 1];
    double x[VAR ? 1 : V];
    Faces<C, V, VAR> kf;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        p[v] = q[v] = r[v] = C(0);
        const double xv = times_2((double)to_c(get_at<X>(xbuf, gp + v * gz, v < nv && !judge)), scale);
        if constexpr (VAR) {
            xlds[v * RT + t] = xv;
            dv[v] = to_c(get_at<T>(dbuf, gp + v * gz, v < nv));
        } else {
            x[v] = xv;
        }
        if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (VAR) {
        // k of a cell outside the grid reads 0: the face then takes the inside cell's k
        auto face = [](C a, C b) -> C { return b == C(0) ? a : C(2) * a * b / (a + b); };
        const int gx0 = ox + tx, gy0 = oy + ty, gz0 = oz + z0;
        C k0 = (C)get_at<float>(kbuf, gp, nv > 0);
        kf.z[0] = face(k0, (C)get_at<float>(kbuf, gp - gz, nv > 0 && gz0 > 0));
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const bool in = v < nv;
            const int i = gp + v * gz;
            kf.l[v] = face(k0, (C)get_at<float>(kbuf, i - 1, in && gx0 > 0));
            kf.r[v] = face(k0, (C)get_at<float>(kbuf, i + 1, in && gx0 + 1 < g.nx));
            kf.d[v] = face(k0, (C)get_at<float>(kbuf, i - g.nx, in && gy0 > 0));
            kf.u[v] = face(k0, (C)get_at<float>(kbuf, i + g.nx, in && gy0 + 1 < g.ny));
            const C k1 = (C)get_at<float>(kbuf, i + gz, in && gz0 + v + 1 < g.nz);
            kf.z[v + 1] = face(k0, k1);
            k0 = k1;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();

    // The box's surface values of q: V values along z per thread on the x and
    // y faces (16-byte stores), one on the z faces (qt: the thread's topmost).
    auto publish = [&](const int mine, const C qt) {
        const int u = fresh_thread(), tx = u & (TX - 1), ty = (u >> LX) & (TY - 1), z0 = (u >> (LX + LY)) * V;
        if (tx == 0 && hxl) put_run<C, V>(surf, mine + (ty * ZP + z0) * (int)sizeof(C), q);
        if (tx == ex - 1 && hxr) put_run<C, V>(surf, mine + (NXF + ty * ZP + z0) * (int)sizeof(C), q);
        if (ty == 0 && hyl) put_run<C, V>(surf, mine + (2 * NXF + tx * ZP + z0) * (int)sizeof(C), q);
        if (ty == ey - 1 && hyr) put_run<C, V>(surf, mine + (2 * NXF + NYF + tx * ZP + z0) * (int)sizeof(C), q);
        const int zf = mine + (2 * (NXF + NYF) + ty * TX + tx) * (int)sizeof(C);
        if (z0 == 0 && hzl) put_one(surf, zf, q[0]);
        if (z0 + nv == ez && hzr) put_one(surf, zf + NZF * (int)sizeof(C), qt);
    };

    uint32_t no = a.base;
    bool late = false;  // a wait ran out
    int restarts = 0, total = 0;
    double rr_true = 0.0;
    const bool keeper = rank == 0 && t == 0;
    long long t1 = 0, t2 = 0, mark = 0;
    for (;;) {  // segments: the solve, then its restarts
        {
            const Buf rbuf = restarts ? r2buf : bbuf;
            const Own o = own();
            int gi = o.gi;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                r[v] = to_c(get_at<T, AGENT>(rbuf, gi, v < o.nv));
                gi += gz;
                if (v % 8 == 7) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int m = 0; m < HG; ++m)
#pragma unroll
                for (int e = 0; e < GN; ++e)
                    rh[m][e] = to_c(get_at<T, AGENT>(rbuf, hgi[m * RT + t] + e * (hz[m] == 1 ? 1 : gz), hl[m] >= 0));
        }
        if (judge && restarts == 0) {  // ||b||^2 and r.z of the start r = b
            double sums[NB];
            {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    s0 += (double)r[v] * (double)r[v];
                    if constexpr (VAR) s1 += (double)dv[v] * (double)r[v] * (double)r[v];
                }
                sums[0] = s0;
                if constexpr (VAR) sums[NB - 1] = s1;
            }
            sum_local<NB>(sums, L, 1);
            __syncthreads();
            sum_publish<NB>(L, slots, 1, rank, G, no);
            double tot[NB];
            late = !sum_collect<NB>(tot, L, slots, 1, rank, G, no, a.wait);
            ++no;
            scale = scale_of(tot[0], (double)npts);
            rr0 = rr = uniform(times_2(tot[0], 2 * scale));
            tol2 = uniform(a.rtol2 * rr0);
            rho = VAR ? uniform(times_2(tot[NB - 1], 2 * scale)) : uniform(dconst * rr0);
            if (!isfinite(rr0)) done = 2;
            else if (rr <= (a.step_first ? 0.0 : tol2)) done = 1;
            else if (maxit <= 0) done = 3;
            if (keeper && hist) hist[0] = rr;
        }
        if (late) break;
        if (scale != 0 && restarts == 0) {  // a restart's residual is stored scaled
#pragma unroll
            for (int v = 0; v < V; ++v) r[v] = times_2(r[v], scale);
#pragma unroll
            for (int m = 0; m < HG; ++m)
#pragma unroll
                for (int e = 0; e < GN; ++e) rh[m][e] = times_2(rh[m][e], scale);
        }
        if (a.timing) mark = wall_clock64();  // the phases only: no load, norm or judge of a segment
        while (!done) {
            // ---- direction, q = A p, p.q. The neighbours' last q (zero before
            // the first update) brings the halo's residual up to date.
            Words4 qh[HG];
            const int theirs = (int)(((no - 1) & 1) * half);
#pragma unroll
            for (int m = 0; m < HG; ++m) {
                qh[m] = Words4{0, 0, 0, 0};
                if (hl[m] >= 0 && iters > seg0)
                    qh[m] = __builtin_amdgcn_raw_buffer_load_b128(surf, theirs + hs[m], 0, AGENT);
            }
            const C beta = (C)beta_d;
            const C dc = (C)dconst;
            if (act) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    p[v] = stored<T>((VAR ? dv[VAR ? v : 0] : dc) * r[v] + beta * p[v]);
                    tile[lb + v * PP] = p[v];
                }
            }
            {
                const C alpha = (C)alpha_d64;
#pragma unroll
                for (int m = 0; m < HG; ++m)
                    if (hl[m] >= 0)
#pragma unroll
                        for (int e = 0; e < GN; ++e) {
                            C& c = tile[hl[m] + e * hz[m]];
                            if (iters > seg0) rh[m][e] = stored<T>(rh[m][e] - alpha * value(qh[m], e, C(0)));
                            c = stored<T>((VAR ? dh[VAR ? m : 0][e] : dc) * rh[m][e] + beta * c);
                        }
            }
            __syncthreads();

            C acc = C(0), qt = C(0);
            if (act) {
                const C below = tile[lb - PP], above = tile[zt];
                auto sweep = [&]<bool FULL>() {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const int a = lb + v * PP;
                        const C b = v == 0 ? below : p[v == 0 ? 0 : v - 1];
                        C f = v == V - 1 ? above : p[v == V - 1 ? v : v + 1];
                        if constexpr (!FULL) f = v + 1 == nv ? above : f;
                        C ax;
                        if constexpr (VAR)
                            ax = kf.l[v] * (p[v] - tile[a - 1]) + kf.r[v] * (p[v] - tile[a + 1]) +
                                 kf.d[v] * (p[v] - tile[a - PX]) + kf.u[v] * (p[v] - tile[a + PX]) + kf.z[v] * (p[v] - b) +
                                 kf.z[v + 1] * (p[v] - f);
                        else
                            ax = StencilConst<C>::apply(p[v], tile[a - 1], tile[a + 1], tile[a - PX], tile[a + PX], b, f);
                        if constexpr (!FULL) {
                            ax = v < nv ? ax : C(0);
                            qt = v + 1 == nv ? ax : qt;
                        }
                        q[v] = ax;
                        acc += p[v] * ax;
                        // a few points' LDS reads in flight, not all V of them
                        if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (FULL) qt = q[V - 1];
                };
                if (full) sweep.template operator()<true>();
                else sweep.template operator()<false>();
            }
            {
                const double v1[1] = {(double)acc};
                sum_local<1>(v1, L, 0);
            }
            __syncthreads();
            sum_publish<1>(L, slots, 0, rank, G, no);
            // The surface leaves while the partials travel. Neighbours read it
            // after the next sum, which this work-group enters only when its
            // stores have arrived.
            if (act) publish((int)((no & 1) * half) + rank * S * (int)sizeof(C), qt);
            double tot1[1];
            if (!sum_collect<1>(tot1, L, slots, 0, rank, G, no, a.wait)) {
                late = true;
                break;
            }
            sigma = tot1[0];
            if (!(sigma > 0.0) || !isfinite(sigma)) {  // as FinAlpha
                done = 2;
                if (judge) {  // the sets of slots keep taking turns
                    const double zero[1] = {0.0};
                    sum_local<1>(zero, L, 1);
                    __syncthreads();
                    sum_publish<1>(L, slots, 1, rank, G, no);
                    late = !sum_collect<1>(tot1, L, slots, 1, rank, G, no, a.wait);
                }
                ++no;
                break;
            }
            alpha_d64 = uniform(rho / sigma);
            if (a.timing) {
                const long long now = wall_clock64();
                t1 += now - mark;
                mark = now;
            }

            // ---- update, r.r
            const C alpha = (C)alpha_d64;
            const double alpha_d = (double)alpha;
            double part[NB];
            {
                C a0 = C(0), a1 = C(0);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    r[v] = stored<T>(r[v] - alpha * q[v]);
                    a0 += r[v] * r[v];
                    if constexpr (VAR) a1 += dv[v] * r[v] * r[v];
                }
                part[0] = (double)a0;
                if constexpr (VAR) part[NB - 1] = (double)a1;
            }
            sum_local<NB>(part, L, 1);
            __builtin_amdgcn_s_waitcnt(0);  // this wavefront's surface stores have arrived
            __syncthreads();
            sum_publish<NB>(L, slots, 1, rank, G, no);
            // x while the partials travel
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if constexpr (VAR) xlds[v * RT + t] += alpha_d * (double)p[v];
                else x[v] += alpha_d * (double)p[v];
            }
            double tot2[NB];
            if (!sum_collect<NB>(tot2, L, slots, 1, rank, G, no, a.wait)) {
                late = true;
                break;
            }
            ++no;
            // as FinBeta; the history holds ||r||^2 until the end of the solve
            rr = tot2[0];
            ++iters;
            if (keeper && hist) hist[iters] = rr;
            if (a.timing) {
                const long long now = wall_clock64();
                t2 += now - mark;
                mark = now;
            }
            if (!isfinite(rr)) done = 2;
            else if (rr <= tol2) done = 1;
            else if (iters >= maxit) done = 3;
            else if (stag > 0) {
                const double rel = uniform(sqrt(rr / rr0));
                if (rel < 0.9 * stag_best) {
                    stag_best = rel;
                    stag_at = iters;
                } else if (iters - stag_at >= stag) {
                    done = 4;
                }
            }
            if (done) break;
            const double rho_new = VAR ? tot2[NB - 1] : dconst * rr;
            beta_d = uniform(rho_new / rho);
            rho = uniform(rho_new);
        }
        if (!judge || late) break;

        // ---- the FP64 residual of x, from memory: x goes past the L2s, the
        // work-groups meet, and a rolled loop (no register arrays) forms r =
        // b - A x, its norms and the residual a restart begins with.
        {
            const Own o = own();
            int gi = o.gi;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                double xv;
                if constexpr (VAR) xv = xlds[v * RT + t];
                else xv = x[v];
                set_at<double, AGENT>(xbuf, gi, v < o.nv, xv);
                gi += gz;
                if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        }
        {
            const double zero[1] = {0.0};
            sum_local<1>(zero, L, 0);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            sum_publish<1>(L, slots, 0, rank, G, no);
            double tot[1];
            late = !sum_collect<1>(tot, L, slots, 0, rank, G, no, a.wait);
            if (late) break;
        }
        ++no;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        total += iters;
        constexpr int NS = VAR ? 3 : 2;
        double sums[NS] = {};
        {
            const Own o = own();
            const int jx = o.x, jy = o.y, jz = o.z;
            int gi = o.gi;
#pragma unroll 1
            for (int v = 0; v < o.nv; ++v) {
                const double xc = get_at<double>(xbuf, gi, true);
                auto near = [&](int at, bool ok) { return get_at<double>(xbuf, at, ok); };
                const bool il = jx > 0, ir = jx + 1 < g.nx, id = jy > 0, iu = jy + 1 < g.ny, ib = jz + v > 0,
                           ia = jz + v + 1 < g.nz;
                const double xl = near(gi - 1, il), xr = near(gi + 1, ir), xd = near(gi - g.nx, id),
                             xu = near(gi + g.nx, iu), xb = near(gi - gz, ib), xa = near(gi + gz, ia);
                double ax;
                if constexpr (VAR) {
                    using K = UK<double>;
                    auto k = [&](int at, bool ok) { return (double)get_at<float>(kbuf, at, ok); };
                    ax = StencilVar<double>::apply(K{xc, k(gi, true)}, K{xl, k(gi - 1, il)}, K{xr, k(gi + 1, ir)},
                                                   K{xd, k(gi - g.nx, id)}, K{xu, k(gi + g.nx, iu)},
                                                   K{xb, k(gi - gz, ib)}, K{xa, k(gi + gz, ia)});
                } else {
                    ax = StencilConst<double>::apply(xc, xl, xr, xd, xu, xb, xa);
                }
                const double res = times_2((double)to_c(get_at<T>(bbuf, gi, true)), scale) - ax;
                const T rs = from_c<T>((C)res);
                const double rv = (double)to_c(rs);
                set_at<T, AGENT>(r2buf, gi, true, rs);
                sums[0] += res * res;
                sums[1] += rv * rv;
                if constexpr (VAR) sums[NS - 1] += (double)to_c(get_at<T>(dbuf, gi, true)) * rv * rv;
                gi += gz;
            }
        }
        sum_local<NS>(sums, L, 1);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        sum_publish<NS>(L, slots, 1, rank, G, no);
        double tot[NS];
        late = !sum_collect<NS>(tot, L, slots, 1, rank, G, no, a.wait);
        if (late) break;
        ++no;
        rr_true = tot[0];
        if (done != 1 || rr_true <= tol2 || restarts >= a.max_restarts || total >= a.maxit) break;
        // restart from r = b - A x
        ++restarts;
        rr = tot[1];
        rho = VAR ? tot[NS - 1] : uniform(dconst * rr);
        beta_d = 0.0;
        iters = seg0 = 0;
        maxit = a.maxit - total;
        done = !isfinite(rr) ? 2 : rr <= (a.step_first ? 0.0 : tol2) ? 1 : 0;
        if (keeper && hist) hist[0] = rr;
    }
    if (late) {
        if (t == 0) __hip_atomic_store(&a.out->timeout, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    if (!judge || scale != 0) {  // a judged x is in place, but for its scale
        const Own o = own();
        int ge = o.gi;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            double xv;
            if constexpr (VAR) xv = xlds[v * RT + t];
            else xv = x[v];
            set_at<X>(xbuf, ge, v < o.nv, from_c<X>((typename Traits<X>::C)times_2(xv, -scale)));
            ge += gz;
            if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (rank == 0) {
        __syncthreads();
        if (hist)
            for (int i = (judge ? 0 : first + 1) + t; i <= iters; i += RT) hist[i] = rr0 > 0.0 ? sqrt(hist[i] / rr0) : 0.0;
        if (t == 0) {
            if (!judge) {
                st->rho = times_2(rho, -2 * scale);
                st->alpha = alpha_d64;
                st->beta = beta_d;
                st->sigma = times_2(sigma, -2 * scale);
                st->rr = times_2(rr, -2 * scale);
                st->iters = iters;
                st->done = done;
                st->stag_at = stag_at;
                st->stag_best = stag_best;
            }
            ResOut& o = *a.out;
            o.done = done;
            o.iters = judge ? total : iters;
            o.last_iters = iters;
            o.restarts = restarts;
            o.used = no - a.base;
            o.rr = rr;
            o.rr0 = rr0;
            o.rr_true = rr_true;
            o.ticks1 = t1;
            o.ticks2 = t2;
            o.t_begin = t_begin;
            o.t_done = judge ? wall_clock64() : 0;
        }
    }
    return true;
}

template <typename T, typename X, int V, bool VAR, int LX, int LY>
__global__ void __launch_bounds__(RT, 2) k_pcg_resident(const ResTask a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    __shared__ SumLds L;
    solve_box<T, X, V, VAR, LX, LY>(a, (int)xcd_remap(blockIdx.x, gridDim.x), dyn, L);
}

template <typename T, typename X, int V, bool VAR, int LX, int LY>
hipError_t run_resident(const ResPlan& p, const ResTask& a, hipStream_t s) {
    auto* k = k_pcg_resident<T, X, V, VAR, LX, LY>;
    const size_t lds = ResShape<LX, LY, V>::lds(sizeof(typename Traits<T>::C), VAR);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)p.geo.G), dim3(RT), lds, s, a);
    return hipGetLastError();
}

template <typename T, typename X, bool VAR, int LX, int LY> hipError_t pick_v(const ResPlan& p, const ResTask& a, hipStream_t s) {
    constexpr int most = res_most_v(sizeof(typename Traits<T>::C) == 8, VAR);
    hipError_t e = hipErrorInvalidValue;
    auto one = [&]<int V>() {
        if constexpr (V <= most)
            if (p.V == V) e = run_resident<T, X, V, VAR, LX, LY>(p, a, s);
    };
    [&]<int... V>(std::integer_sequence<int, V...>) {
        (one.template operator()<V>(), ...);
    }(ResVs{});
    return e;
}

template <typename T, typename X, bool VAR> hipError_t pick_shape(const ResPlan& p, const ResTask& a, hipStream_t s) {
    hipError_t e = hipErrorInvalidValue;
    auto one = [&]<int SH>() {
        constexpr int LX = RES_SHAPES[SH][0], LY = RES_SHAPES[SH][1];
        if (p.geo.lx == LX && p.geo.ly == LY) e = pick_v<T, X, VAR, LX, LY>(p, a, s);
    };
    [&]<int... SH>(std::integer_sequence<int, SH...>) {
        (one.template operator()<SH>(), ...);
    }(std::make_integer_sequence<int, RES_NSHAPES>{});
    return e;
}

}  // namespace resident

}  // namespace pcgmi
