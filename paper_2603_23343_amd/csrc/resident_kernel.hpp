// resident_kernel.hpp -- Jacobi-PCG with the whole grid held on the chip.
//
// The paper keeps a solve's vectors in the cores' SRAM for all iterations
// (Sec. VII); MI355X has 128 MiB of vector registers and 40 MiB of LDS, so a
// grid of up to ~4 M points fits as well. One persistent launch runs every
// iteration: a work-group owns a box of the grid, r, p, q and the FP64 x of its
// points live in registers, the current direction p (with a one-point halo)
// in LDS. Per iteration only scalars and the boxes' surfaces leave a CU.
//
// One iteration (the two-kernel form's arithmetic, pcg.hip):
//   p = D^-1 r + beta p on own points and on the halo (each box keeps the
//   residual of its halo points itself), q = A p, partials of p.q; the box's
//   surface values of q are published;                 -- grid sum: alpha
//   x += alpha p, r -= alpha q on own points; the neighbours' q updates the
//   halo's r; partials of r.r;                         -- grid sum: beta
// so one surface exchange serves an iteration and its latency hides behind
// the second sum.
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
// runs the solve with the two-kernel form instead.
#pragma once

#include "ops.hpp"
#include "resident.hpp"

namespace pcgmi {

namespace resident {

constexpr int RT = 512;     // threads per work-group
constexpr int RW = RT / 64;  // wavefronts
// Copies of the slots. Each work-group writes its partial to all of them and
// polls one, so that 256 work-groups do not poll the same 4 KiB: a sum over
// 256 work-groups takes 2.7 us with 8 copies and 3.4 us with one (64
// work-groups: 1.65 and 2.1 us).
constexpr int RES_COPIES = 8;
constexpr long long RES_WAIT_TICKS = 100000000;  // 1 s of the 100 MHz wall clock
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
    double wave[2][RW];  // the work-group's wavefront sums
    double slot[2][RW];  // sums of the slots, per polling wavefront
    int bad;
};

// First part of a grid sum: wavefront sums to LDS.
template <int NC> __device__ __forceinline__ void sum_local(const double (&v)[NC], SumLds& L) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const double s = wave_total(v[c]);
        if ((threadIdx.x & 63) == 63) L.wave[c][threadIdx.x >> 6] = s;
    }
}

// Slots of one sum: [copy][component][work-group], 16 bytes each.
__device__ __forceinline__ int slot_at(int copy, int c, int rank) {
    return ((copy * 2 + c) * RES_MAX_WG + rank) * 16;
}

// The first threads store the work-group's partial in every copy (after a
// __syncthreads that follows sum_local).
template <int NC> __device__ __forceinline__ void sum_publish(SumLds& L, Buf slots, int set, int rank, uint32_t no) {
    if (threadIdx.x < RES_COPIES) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double s = L.wave[c][0];
#pragma unroll
            for (int w = 1; w < RW; ++w) s += L.wave[c][w];
            const uint64_t b = __builtin_bit_cast(uint64_t, s);
            __builtin_amdgcn_raw_buffer_store_b128(Words4{no, (uint32_t)(b >> 32), no, (uint32_t)b}, slots,
                                                   set + slot_at(threadIdx.x, c, rank), 0, AGENT);
        }
    }
}

// Last part: wait for all slots and add them; false after a timeout.
template <int NC>
__device__ __forceinline__ bool sum_collect(double (&tot)[NC], SumLds& L, Buf slots, int set, int rank, int G,
                                            uint32_t no) {
    const int t = threadIdx.x, wid = t >> 6;
    const int nw = (G + 63) >> 6;
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
                    a[c] = __builtin_amdgcn_raw_buffer_load_b128(slots, set + slot_at(rank & (RES_COPIES - 1), c, t), 0,
                                                                 AGENT);
#pragma unroll
                for (int c = 0; c < NC; ++c) ok = ok && a[c].x == no && a[c].z == no;
                if (ok) break;
                if (wall_clock64() - began > RES_WAIT_TICKS) {
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
template <typename T> __device__ __forceinline__ T get_at(Buf b, int i, bool ok) {
    const int off = ok ? i * (int)sizeof(T) : -1;
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(b, off, 0, 0));
}
template <typename T> __device__ __forceinline__ void set_at(Buf b, int i, bool ok, T v) {
    const int off = ok ? i * (int)sizeof(T) : -1;
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(Words2, v), b, off, 0, 0);
    else if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), b, off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), b, off, 0, 0);
}

// Face coefficients of a thread's points (variable operator), computed once.
template <typename C, int V, bool VAR> struct Faces {
    C l[V], r[V], d[V], u[V], z[V + 1];
};
template <typename C, int V> struct Faces<C, V, false> {};

// T: storage type, X: the x accumulator's type in memory (FP64 registers), V
// z points per thread, 2^LX x 2^LY threads along x and y (the rest along z).
template <typename T, typename X, int V, bool VAR, int LX, int LY>
__global__ void __launch_bounds__(RT, 2) k_pcg_resident(const ResGeo g, const T* __restrict__ r0, X* __restrict__ xio,
                                                       const float* __restrict__ kc, const T* __restrict__ dinv_in,
                                                       SolveState* st, double* hist, void* slots_p, void* surf_p,
                                                       uint32_t base, ResOut* out, int timing) {
    using C = typename Traits<T>::C;
    using Sh = ResShape<LX, LY, V>;
    constexpr int TX = Sh::TX, TY = Sh::TY, ZR = Sh::ZR, ZP = Sh::ZP, PX = Sh::PX, PP = Sh::PP;
    constexpr int NXF = Sh::NXF, NYF = Sh::NYF, NZF = Sh::NZF, S = Sh::S;
    constexpr int GN = 16 / (int)sizeof(C);            // halo points per group (one 16-byte load)
    constexpr int HG = (S / GN + RT - 1) / RT;         // groups per thread
    constexpr int NB = VAR ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    __shared__ SumLds L;
    C* tile = reinterpret_cast<C*>(dyn);               // [ZP + 2][TY + 2][TX + 2]
    double* xlds = reinterpret_cast<double*>(tile + ((PP * (ZP + 2) + 1) & ~1));  // [V][RT] (VAR)

    if (st->done != 0 || st->maxit <= 0) return;  // the same in every work-group
    const double rr0 = uniform(st->rr0), tol2 = uniform(st->tol2), dconst = uniform(st->dinv);
    const int maxit = st->maxit, stag = st->stag;
    double rho = uniform(st->rho), beta_d = uniform(st->beta), rr = uniform(st->rr);
    double stag_best = uniform(st->stag_best);
    int iters = st->iters, done = 0, stag_at = st->stag_at;
    double sigma = 0.0, alpha_d64 = 0.0;

    const int t = threadIdx.x;
    const int tx = t & (TX - 1), ty = (t >> LX) & (TY - 1), tz = t >> (LX + LY);
    const int rank = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int cx = rank % g.gx, cy = (rank / g.gx) % g.gy, cz = rank / (g.gx * g.gy);
    const int ox = cx * g.bx, oy = cy * g.by, oz = cz * g.bz;
    const int ex = min(g.bx, g.nx - ox), ey = min(g.by, g.ny - oy), ez = min(g.bz, g.nz - oz);
    const int z0 = tz * V;
    const bool act = tx < ex && ty < ey && z0 < ez;
    const int nv = act ? min(V, ez - z0) : 0;
    const bool full = __syncthreads_and(nv == V) != 0;  // no masking needed in this box
    const int lb = (z0 + 1) * PP + (ty + 1) * PX + tx + 1;
    // the cell above the thread's last point (the top halo is the tile's last plane)
    const int zt = z0 + nv == ez ? (ZP + 1) * PP + (ty + 1) * PX + tx + 1 : lb + V * PP;
    const bool hxl = cx > 0, hxr = cx + 1 < g.gx, hyl = cy > 0, hyr = cy + 1 < g.gy, hzl = cz > 0, hzr = cz + 1 < g.gz;
    const uint32_t half = (uint32_t)g.G * S * (uint32_t)sizeof(C);
    const Buf slots = make_buf(slots_p, RES_SLOT_BYTES);
    const Buf surf = make_buf(surf_p, 2 * half);
    // the grid's arrays (resident_plan keeps them below 2 GiB)
    const uint32_t npts = (uint32_t)g.nx * g.ny * g.nz;
    const Buf rbuf = make_buf(const_cast<T*>(r0), npts * (uint32_t)sizeof(T));
    const Buf xbuf = make_buf(xio, npts * (uint32_t)sizeof(X));
    const Buf dbuf = make_buf(const_cast<T*>(dinv_in), VAR ? npts * (uint32_t)sizeof(T) : 0u);
    const Buf kbuf = make_buf(const_cast<float*>(kc), VAR ? npts * 4u : 0u);

    for (int i = t; i < PP * (ZP + 2); i += RT) tile[i] = C(0);
    if (t == 0) L.bad = 0;

    // Halo groups of this thread: GN points along z (x and y faces) or along
    // x (z faces). hl: tile index of the first (-1: none), hz: its step; hs:
    // byte offset of the neighbour's values; rh: the points' residuals.
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
        int sx = 0, sz = 1;
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
            sz = 0;
            hz[m] = 1;
        }
        if (ok) {
            hs[m] = (from * S + face + j) * (int)sizeof(C);
            hl[m] = (z == ez ? ZP + 1 : z + 1) * PP + (y + 1) * PX + x + 1;
        }
#pragma unroll
        for (int e = 0; e < GN; ++e) {
            const bool in = ok && ((sx && x + e < ex) || (sz && z + e < ez));
            const int gi = ((oz + z + sz * e) * g.ny + (oy + y)) * g.nx + ox + x + sx * e;
            rh[m][e] = to_c(get_at<T>(rbuf, gi, in));
            if constexpr (VAR) dh[m][e] = to_c(get_at<T>(dbuf, gi, in));
        }
    }

    // own points
    const int gp = ((oz + z0) * g.ny + (oy + ty)) * g.nx + ox + tx;
    const int gz = g.nx * g.ny;
    C r[V], p[V], q[V], dv[VAR ? V : 1];
    double x[VAR ? 1 : V];
    Faces<C, V, VAR> kf;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        p[v] = q[v] = C(0);
        r[v] = to_c(get_at<T>(rbuf, gp + v * gz, v < nv));
        const double xv = (double)to_c(get_at<X>(xbuf, gp + v * gz, v < nv));
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

    uint32_t no = base;
    long long t1 = 0, t2 = 0, mark = timing ? wall_clock64() : 0;
    const bool keeper = rank == 0 && t == 0;
    for (;;) {
        // ---- direction, q = A p, p.q
        const C beta = (C)beta_d;
        const C dc = (C)dconst;
        if (act) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                p[v] = stored<T>((VAR ? dv[VAR ? v : 0] : dc) * r[v] + beta * p[v]);
                tile[lb + v * PP] = p[v];
            }
        }
#pragma unroll
        for (int m = 0; m < HG; ++m)
            if (hl[m] >= 0)
#pragma unroll
                for (int e = 0; e < GN; ++e) {
                    C& c = tile[hl[m] + e * hz[m]];
                    c = stored<T>((VAR ? dh[VAR ? m : 0][e] : dc) * rh[m][e] + beta * c);
                }
        __syncthreads();

        const int mine = (int)((no & 1) * half) + rank * S * (int)sizeof(C);
        C acc = C(0);
        if (act) {
            C qt = C(0);
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
            // the box's surface: V values along z per thread on the x and y
            // faces (16-byte stores), one on the z faces
            if (tx == 0 && hxl) put_run<C, V>(surf, mine + (ty * ZP + z0) * (int)sizeof(C), q);
            if (tx == ex - 1 && hxr) put_run<C, V>(surf, mine + (NXF + ty * ZP + z0) * (int)sizeof(C), q);
            if (ty == 0 && hyl) put_run<C, V>(surf, mine + (2 * NXF + tx * ZP + z0) * (int)sizeof(C), q);
            if (ty == ey - 1 && hyr) put_run<C, V>(surf, mine + (2 * NXF + NYF + tx * ZP + z0) * (int)sizeof(C), q);
            const int zf = mine + (2 * (NXF + NYF) + ty * TX + tx) * (int)sizeof(C);
            if (z0 == 0 && hzl) put_one(surf, zf, q[0]);
            if (z0 + nv == ez && hzr) put_one(surf, zf + NZF * (int)sizeof(C), qt);
        }
        {
            const double v1[1] = {(double)acc};
            sum_local<1>(v1, L);
        }
        __builtin_amdgcn_s_waitcnt(0);  // this wavefront's surface stores have arrived
        __syncthreads();
        sum_publish<1>(L, slots, 0, rank, no);
        double tot1[1];
        if (!sum_collect<1>(tot1, L, slots, 0, rank, g.G, no)) break;
        sigma = tot1[0];
        if (!(sigma > 0.0) || !isfinite(sigma)) {  // as FinAlpha
            done = 2;
            break;
        }
        alpha_d64 = uniform(rho / sigma);
        if (timing) {
            const long long now = wall_clock64();
            t1 += now - mark;
            mark = now;
        }

        // ---- update, r.r
        Words4 qh[HG];
        const int theirs = (int)((no & 1) * half);
#pragma unroll
        for (int m = 0; m < HG; ++m) {
            qh[m] = Words4{0, 0, 0, 0};
            if (hl[m] >= 0) qh[m] = __builtin_amdgcn_raw_buffer_load_b128(surf, theirs + hs[m], 0, AGENT);
        }
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
        sum_local<NB>(part, L);
        __syncthreads();
        sum_publish<NB>(L, slots, RES_SLOT_BYTES / 2, rank, no);
        // x and the halo's residual while the partials travel
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if constexpr (VAR) xlds[v * RT + t] += alpha_d * (double)p[v];
            else x[v] += alpha_d * (double)p[v];
        }
#pragma unroll
        for (int m = 0; m < HG; ++m) {
#pragma unroll
            for (int e = 0; e < GN; ++e) rh[m][e] = stored<T>(rh[m][e] - alpha * value(qh[m], e, C(0)));
        }
        double tot2[NB];
        if (!sum_collect<NB>(tot2, L, slots, RES_SLOT_BYTES / 2, rank, g.G, no)) break;
        ++no;
        // as FinBeta; the history holds ||r||^2 until the end of the solve
        rr = tot2[0];
        ++iters;
        if (keeper && hist) hist[iters] = rr;
        if (timing) {
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
    if (L.bad) {
        if (t == 0) __hip_atomic_store(&out->timeout, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    // the offsets are formed again here, not kept in registers since the start
    int ge = gp;
    __asm__ volatile("" : "+v"(ge));
#pragma unroll
    for (int v = 0; v < V; ++v) {
        double xv;
        if constexpr (VAR) xv = xlds[v * RT + t];
        else xv = x[v];
        set_at<X>(xbuf, ge, v < nv, from_c<X>((typename Traits<X>::C)xv));
        ge += gz;
        if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (rank == 0) {
        __syncthreads();
        const int first = st->iters;
        if (hist)
            for (int i = first + 1 + t; i <= iters; i += RT) hist[i] = sqrt(hist[i] / rr0);
        __syncthreads();
        if (t == 0) {
            st->rho = rho;
            st->alpha = alpha_d64;
            st->beta = beta_d;
            st->sigma = sigma;
            st->rr = rr;
            st->iters = iters;
            st->done = done;
            st->stag_at = stag_at;
            st->stag_best = stag_best;
            out->ticks1 = t1;
            out->ticks2 = t2;
        }
    }
}

template <typename T, typename X, int V, bool VAR, int LX, int LY>
hipError_t run_resident(const ResLaunch& a, hipStream_t s) {
    auto* k = k_pcg_resident<T, X, V, VAR, LX, LY>;
    const size_t lds = ResShape<LX, LY, V>::lds(sizeof(typename Traits<T>::C), VAR);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)a.plan.geo.G), dim3(RT), lds, s, a.plan.geo, static_cast<const T*>(a.r),
                       static_cast<X*>(a.x), a.kc, static_cast<const T*>(a.dinv), a.st, a.hist, a.slots, a.surf, a.base,
                       a.out, a.timing);
    return hipGetLastError();
}

template <typename T, typename X, bool VAR, int LX, int LY> hipError_t pick_v(const ResLaunch& a, hipStream_t s) {
    constexpr int most = res_most_v(sizeof(typename Traits<T>::C) == 8, VAR);
    hipError_t e = hipErrorInvalidValue;
    auto one = [&]<int V>() {
        if constexpr (V <= most)
            if (a.plan.V == V) e = run_resident<T, X, V, VAR, LX, LY>(a, s);
    };
    [&]<int... V>(std::integer_sequence<int, V...>) {
        (one.template operator()<V>(), ...);
    }(ResVs{});
    return e;
}

template <typename T, typename X, bool VAR> hipError_t pick_shape(const ResLaunch& a, hipStream_t s) {
    const int lx = a.plan.geo.lx, ly = a.plan.geo.ly;
    if (lx == 5 && ly == 4) return pick_v<T, X, VAR, 5, 4>(a, s);
    if (lx == 4 && ly == 4) return pick_v<T, X, VAR, 4, 4>(a, s);
    if (lx == 3 && ly == 4) return pick_v<T, X, VAR, 3, 4>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace resident

}  // namespace pcgmi
