// resident.hpp -- host interface of the on-chip PCG (resident.hip).
#pragma once

#include <array>
#include <chrono>
#include <utility>

#include "internal.hpp"

struct pcg_ctx_s;
struct pcg_batch_s;

namespace pcgmi {

constexpr int RES_MAX_WG = 256;                    // one work-group per CU
constexpr size_t RES_MAX_LDS = (size_t)156 << 10;  // of a CU's 160 KiB

constexpr size_t RES_HALO_LDS = (size_t)4 * 512 * 4;  // grid indices of the halo groups

// Compiled work-group shapes (log2 of the threads along x and y; 512 in all)
// and z points per thread.
constexpr int RES_SHAPES[][2] = {{5, 4}, {4, 4}, {3, 4}};
constexpr int RES_NSHAPES = sizeof RES_SHAPES / sizeof RES_SHAPES[0];
using ResVs = std::integer_sequence<int, 2, 4, 6, 8, 10, 12, 16, 20, 24, 28, 32>;
template <int... V> constexpr std::array<int, sizeof...(V)> res_list(std::integer_sequence<int, V...>) { return {V...}; }
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
        return cs * (((size_t)PP * (ZP + 2) + 1) & ~(size_t)1) + (var ? (size_t)8 * 512 * V : 0) + RES_HALO_LDS;
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
    size_t lds;  // dynamic LDS
};

// Result of a launch (work-group 0), all but the first field.
struct ResOut {
    int timeout;     // a wait ran out: the solve did not finish (the host zeroes it before the next launch)
    int done;        // as SolveState::done
    int iters;       // iterations, restarts included
    int last_iters;  // iterations since the last restart
    int restarts;
    uint32_t used;   // numbers of grid sums used
    double rr, rr0, rr_true;       // recursive ||r||^2, ||b||^2, FP64 ||b - A x||^2 (judge), up to one common factor
    long long ticks1, ticks2;      // wall-clock ticks (10 ns) of the two phases
    long long t_begin, t_done;     // wall clock (judge)
};

// Components of a grid sum at most, and copies of the slots. Each work-group
// writes its partial to every copy and polls one, so that 256 work-groups do
// not poll the same 4 KiB: a sum over 256 work-groups takes 2.7 us with 8
// copies and 3.4 us with one (64 work-groups: 1.65 and 2.1 us).
constexpr int RES_SUMS = 3, RES_COPIES = 8;
constexpr size_t RES_HEAD_BYTES = 256;  // ResOut, padded
static_assert(sizeof(ResOut) <= RES_HEAD_BYTES);
// Slots of a group of G work-groups: two sets, 16 bytes a component, whole
// 128-byte lines.
constexpr int res_slot_pitch(int G) { return (G + 7) & ~7; }
constexpr uint32_t res_slot_bytes(int G) { return 2u * RES_COPIES * RES_SUMS * (uint32_t)res_slot_pitch(G) * 16u; }
constexpr uint32_t RES_SLOT_BYTES = res_slot_bytes(RES_MAX_WG);

// One solve. judge = 0: a start made by other kernels (r, x, st) is iterated
// to its end and x and st are left for others. judge = 1: the solve of A x = b
// from x = 0 (r is b), FP64 judge and restarts included.
struct ResTask {
    ResGeo geo;
    const void* r;
    void* r2;  // judge: the residual that a restart begins with (a vector of the storage type)
    void* x;   // the accumulator, or (judge) the caller's FP64 x
    const float* kc;
    const void* dinv;
    SolveState* st;
    double* hist;   // may be null
    void* slots;    // res_slot_bytes(G), zeroed once
    void* surf;     // 2 * G * S values of the arithmetic type
    ResOut* out;
    double rtol2;   // judge
    uint32_t base;  // number of the first grid sum (never used before on these slots)
    int timing;
    int judge, maxit, max_restarts;
    int step_first;  // judge: a start within the tolerance is iterated all the same (as the streaming batch does)
    long long wait;  // ticks (10 ns) a work-group waits in a grid sum at most
};
constexpr long long RES_WAIT_TICKS = 100000000;  // 1 s

// What a context or a batch knows of its launches: the sums' numbers that are
// used up, whether the slots can be trusted, and when to try again after a
// launch whose work-groups did not come together (another process on the
// device, a stream without all CUs): a hundred times what the attempt lost, so
// that a lasting interference costs a hundredth and a passing one ends.
struct ResSeries {
    uint32_t next = 1;
    bool clean = true;  // false: slots and result must be zeroed first
    long long wait = -1;  // tests: limit of a wait in ticks (-1: the form's own)
    int drop = 0;         // tests: the launch of this number from now counts as late
    std::chrono::steady_clock::time_point again{};

    bool ready() const { return std::chrono::steady_clock::now() >= again; }
    // Zeroing is due: a launch did not end well, or the numbers near their end.
    bool stale() const { return !clean || next > (1u << 30); }
    void zeroed() {
        next = 1;
        clean = true;
    }
    // The end of a launch that began at t0; true if its results count.
    bool ended(bool timeout, uint32_t used, std::chrono::steady_clock::time_point t0) {
        const bool late = timeout || (drop > 0 && --drop == 0);
        if (late) {
            const auto now = std::chrono::steady_clock::now();
            again = now + 100 * (now - t0);
        } else {
            next += used + 1;
            clean = true;
        }
        return !late;
    }
};
// How long a launch waits for its CUs on the host at most (results would
// otherwise depend on what else runs: the other forms sum in another order).
constexpr double RES_HOLD_S = 30.0;
// A batch waits as long as it takes: its streaming kernel needs its
// work-groups together, too, and beside a launch that holds CUs its barriers
// would run out of time. Every claim ends, since every wait of its holder does.
constexpr double RES_HOLD_BATCH_S = 1e8;

// One problem of a batch: its task and its compiled shape.
struct ResBatchTask {
    ResTask task;
    int shape;  // index into RES_SHAPES
    int V;
};
// All problems of a batch in one launch of nwg work-groups: work-group w runs
// the boxes work[first[w]] .. work[first[w + 1] - 1], {problem, rank}, in
// this order, which is the same order of problems for all of them.
hipError_t launch_batch_resident(const ResBatchTask* tasks, const int2* work, const int* first, int nwg, size_t lds,
                                 hipStream_t s);
// Points per thread compiled for batches (the kernel's bodies follow this list).
using ResBatchVs = std::integer_sequence<int, 4, 8, 12, 16, 24, 32>;

bool resident_candidate(int nx, int ny, int nz, int dt, bool var, int lx, int ly, int V, int max_wg, ResPlan* out);
// A plan for the grid on at most max_wg work-groups; false if it does not fit.
bool resident_plan(int nx, int ny, int nz, int dt, bool var, int max_wg, ResPlan* out);
hipError_t launch_pcg_resident(int dt, int xdt, const ResPlan& p, const ResTask& a, hipStream_t s);
hipError_t launch_resident_f32(const ResPlan& p, const ResTask& a, hipStream_t s);
hipError_t launch_resident_f32_var(const ResPlan& p, const ResTask& a, hipStream_t s);
hipError_t launch_resident_f64(const ResPlan& p, const ResTask& a, hipStream_t s);

// For tests of what follows a launch whose work-groups did not come together
// (ResSeries::wait, drop); after a retry the next solve tries again at once.
void resident_limits(pcg_ctx_s* c, long long wait, int drop);
void resident_retry(pcg_ctx_s* c);
void batch_limits(pcg_batch_s* b, long long wait, int drop);
void batch_retry(pcg_batch_s* b);

// A claim on CUs of a device for the time of a persistent launch: its
// work-groups wait for each other, so two such launches of this process may
// only overlap while both fit. Claims are served in the order they come. Waits
// up to wait_s for others to end; ok() is false if it ran out (the caller then
// takes a form that needs no claim).
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
    CuHold *prev_ = nullptr, *next_ = nullptr;  // in the queue of waiting claims
};

}  // namespace pcgmi
