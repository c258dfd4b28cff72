// resident.hip -- plans and launches of the on-chip PCG (resident_kernel.hpp),
// and the reservation of the CUs that its persistent launches need.
#include <chrono>
#include <condition_variable>
#include <mutex>

#include "resident.hpp"

namespace pcgmi {

bool resident_candidate(int nx, int ny, int nz, int dt, bool var, int lx, int ly, int V, int max_wg, ResPlan* out) {
    const int TX = 1 << lx, TY = 1 << ly, TZ = 512 >> (lx + ly);
    auto cut = [](int n, int m, int& b, int& g) {
        g = (n + m - 1) / m;
        b = (n + g - 1) / g;
        g = (n + b - 1) / b;
    };
    ResPlan p{};
    ResGeo& g = p.geo;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.lx = lx;
    g.ly = ly;
    cut(nx, TX, g.bx, g.gx);
    cut(ny, TY, g.by, g.gy);
    cut(nz, TZ * V, g.bz, g.gz);
    if ((int64_t)g.gx * g.gy * g.gz > max_wg) return false;
    g.G = g.gx * g.gy * g.gz;
    const size_t cs = dt == DT_F64 ? 8 : 4;
    p.V = V;
    const int zr = TZ * V, zp = (zr + 3) & ~3;
    p.S = 2 * (TY * zp + TX * zp + TX * TY);
    if ((int64_t)nx * ny * nz > (int64_t)1 << 27) return false;  // 32-bit byte offsets
    const size_t lds = cs * (((size_t)(TX + 2) * (TY + 2) * (zp + 2) + 1) & ~(size_t)1) + (var ? (size_t)8 * 512 * V : 0) + RES_HALO_LDS;
    if (lds > RES_MAX_LDS) return false;
    p.lds = lds;
    *out = p;
    return true;
}

// Microseconds of an iteration as measured, up to a constant: 0.11 per point
// and thread (0.25 with cell coefficients, 0.3 in FP64, 0.55 in FP64 with
// coefficients) and 0.017 per work-group for the two grid sums (64^3: 4.7 us
// with 64 work-groups and 8 points per thread, 7.5 with 256 and 2; 128^3: 9.3
// with 256 and 16, 9.6 with 192 and 24). Shapes come in the order of their
// speed (wide rows first) and the first one wins a tie.
bool resident_plan(int nx, int ny, int nz, int dt, bool var, int max_wg, ResPlan* out) {
    const int most = res_most_v(dt == DT_F64, var);
    const double per_v = dt == DT_F64 ? (var ? 0.55 : 0.3) : (var ? 0.25 : 0.11);
    if (max_wg > RES_MAX_WG) max_wg = RES_MAX_WG;
    bool have = false;
    double best = 0.0;
    for (const auto& sh : RES_SHAPES)
        for (int V : res_list(ResVs{})) {
            ResPlan p;
            if (V > most || !resident_candidate(nx, ny, nz, dt, var, sh[0], sh[1], V, max_wg, &p)) continue;
            const double cost = per_v * p.V + 0.017 * p.geo.G;
            if (!have || cost < best - 1e-9) {
                have = true;
                best = cost;
                *out = p;
            }
        }
    return have;
}

hipError_t launch_pcg_resident(int dt, int xdt, const ResPlan& p, const ResTask& a, hipStream_t s) {
    if (p.geo.G < 1 || p.geo.G > RES_MAX_WG || xdt != DT_F64) return hipErrorInvalidValue;
    const bool var = a.kc != nullptr;
    if (dt == DT_F32) return var ? launch_resident_f32_var(p, a, s) : launch_resident_f32(p, a, s);
    if (dt == DT_F64) return launch_resident_f64(p, a, s);
    return hipErrorInvalidValue;
}

namespace {

constexpr int MAX_DEVICES = 16;

// CUs of each device that persistent launches of this process hold, and the
// claims that wait for some, in the order they came. The queue is served from
// its head only: a batch, which needs every CU, is not passed by solves that
// need a few. A waiting claim is a node of the list itself (no allocation).
struct Held {
    std::mutex m;
    std::condition_variable cv;
    int used[MAX_DEVICES] = {};
    CuHold* head[MAX_DEVICES] = {};
    CuHold* tail[MAX_DEVICES] = {};
};
Held& held() {
    static Held h;
    return h;
}

}  // namespace

CuHold::CuHold(int dev, int want, int cap, double wait_s) : dev_(dev), want_(want) {
    if (dev < 0 || dev >= MAX_DEVICES || want > cap) return;
    Held& h = held();
    {
        std::unique_lock<std::mutex> l(h.m);
        (h.tail[dev] ? h.tail[dev]->next_ : h.head[dev]) = this;
        prev_ = h.tail[dev];
        h.tail[dev] = this;
        ok_ = h.cv.wait_for(l, std::chrono::duration<double>(wait_s),
                            [&] { return h.head[dev] == this && h.used[dev] + want <= cap; });
        (prev_ ? prev_->next_ : h.head[dev]) = next_;
        (next_ ? next_->prev_ : h.tail[dev]) = prev_;
        if (ok_) h.used[dev] += want;
    }
    h.cv.notify_all();  // the next in the queue may fit as well
}

CuHold::~CuHold() {
    if (!ok_) return;
    Held& h = held();
    {
        std::lock_guard<std::mutex> l(h.m);
        h.used[dev_] -= want_;
    }
    h.cv.notify_all();
}

}  // namespace pcgmi
