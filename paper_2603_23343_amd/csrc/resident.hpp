// resident.hpp -- host interface of the on-chip PCG (resident.hip).
#pragma once

#include <utility>

#include "internal.hpp"

namespace pcgmi {

constexpr int RES_MAX_WG = 256;                    // one work-group per CU
constexpr size_t RES_MAX_LDS = (size_t)156 << 10;  // of a CU's 160 KiB

// Compiled work-group shapes (log2 of the threads along x and y; 512 in all)
// and z points per thread.
constexpr int RES_SHAPES[][2] = {{5, 4}, {4, 4}, {3, 4}};
using ResVs = std::integer_sequence<int, 2, 4, 6, 8, 10, 12, 16, 20, 24, 28, 32>;
constexpr int RES_VS[] = {2, 4, 6, 8, 10, 12, 16, 20, 24, 28, 32};
// Points per thread that the 256 registers of a lane hold: r, p, q and x, or
// r, p, q, five face coefficients and D^-1 (x then lies in LDS).
constexpr int res_most_v(bool f64, bool var) { return f64 ? (var ? 8 : 16) : (var ? 16 : 32); }

// Sizes that follow from a shape and the points per thread. A box's six
// faces are stored x-, x+ ([y][z]), y-, y+ ([x][z]), z-, z+ ([y][x]).
template <int LX, int LY, int V> struct ResShape {
    static constexpr int TX = 1 << LX, TY = 1 << LY, TZ = 512 >> (LX + LY);
    static constexpr int ZR = TZ * V;             // planes of the box
    static constexpr int ZP = (ZR + 3) & ~3;      // z pitch of the x and y faces
    static constexpr int PX = TX + 2, PP = PX * (TY + 2);
    static constexpr int NXF = TY * ZP, NYF = TX * ZP, NZF = TX * TY;
    static constexpr int S = 2 * (NXF + NYF + NZF);
    static constexpr size_t lds(size_t cs, bool var) {
        return cs * (((size_t)PP * (ZP + 2) + 1) & ~(size_t)1) + (var ? (size_t)8 * 512 * V : 0);
    }
};

// Boxes of bx x by x bz points (the last along a dimension may be smaller),
// gx x gy x gz of them; 2^lx x 2^ly threads along x and y, the rest along z.
struct ResGeo {
    int nx, ny, nz;
    int lx, ly;
    int bx, by, bz;
    int gx, gy, gz;
    int G;  // work-groups
};

struct ResPlan {
    ResGeo geo;
    int V;  // z points per thread
    int S;  // values of a box's surface
};

struct ResOut {
    int timeout;  // a wait ran out: the solve did not finish (set once, never cleared)
    int pad;
    long long ticks1, ticks2;  // wall-clock ticks (10 ns) of the two phases
};

constexpr size_t RES_HEAD_BYTES = 256;  // ResOut, padded
// Two sums, eight copies of two components per work-group, 16 bytes each.
constexpr uint32_t RES_SLOT_BYTES = 2 * 8 * 2 * RES_MAX_WG * 16;

struct ResLaunch {
    ResPlan plan;
    const void* r;  // start residual
    void* x;        // x accumulator (read and written)
    const float* kc;
    const void* dinv;
    SolveState* st;
    double* hist;
    void* slots;    // RES_SLOT_BYTES
    void* surf;     // 2 * G * S values of the arithmetic type
    uint32_t base;  // number of the first grid sum (never used before on these slots)
    ResOut* out;
    int timing;
};

bool resident_candidate(int nx, int ny, int nz, int dt, bool var, int lx, int ly, int V, int max_wg, ResPlan* out);
// A plan for the grid on at most max_wg work-groups; false if it does not fit.
bool resident_plan(int nx, int ny, int nz, int dt, bool var, int max_wg, ResPlan* out);
hipError_t launch_pcg_resident(int dt, int xdt, const ResLaunch& a, hipStream_t s);
hipError_t launch_resident_f32(const ResLaunch& a, hipStream_t s);
hipError_t launch_resident_f32_var(const ResLaunch& a, hipStream_t s);
hipError_t launch_resident_f64(const ResLaunch& a, hipStream_t s);

// A claim on CUs of a device for the time of a persistent launch: its
// work-groups wait for each other, so two such launches of this process may
// only overlap while both fit. Waits up to wait_s for others to end; ok() is
// false if it ran out (the caller then takes a form that needs no claim).
class CuHold {
public:
    CuHold(int dev, int want, int cap, double wait_s);
    ~CuHold();
    CuHold(const CuHold&) = delete;
    CuHold& operator=(const CuHold&) = delete;
    bool ok() const { return ok_; }

private:
    int dev_, want_;
    bool ok_ = false;
};

}  // namespace pcgmi
