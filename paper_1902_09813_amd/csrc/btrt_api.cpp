// C ABI of one solver handle (include/btrt.h): a single problem instance on one stream.

#include "btrt.h"
#include "btrt_host.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

using namespace btrth;
using btrtk::kError;
using btrtk::kReducePartials;
using btrtk::kResidual;

struct btrt {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    char* mem = nullptr;
    bool own_mem = false;
    int check_interval = 1000;
    btrtk::LaunchCfg launch{};  // requested launch shape (zero fields: automatic)
    void* wsched = nullptr;     // device wall schedule in force (owned), of wsched_bytes bytes
    size_t wsched_bytes = 0;
    void* wspare = nullptr;     // the schedule before it: the next call of btrt_set_walls fills it if it fits
    size_t wspare_bytes = 0;
    StagingUser staging;
    Instance inst;
};

namespace {

using btrtk::LaunchCfg;

// n steps as launches of the handle's shape; a count that is not a multiple of its steps per
// launch ends with one shorter launch.
int enqueue_steps(btrt* h, const LaunchCfg& want, int64_t n) { return instance_steps(h->inst, want, n, h->stream); }

int enqueue_steps(btrt* h, int64_t n) { return enqueue_steps(h, h->launch, n); }

bool launch_ok(const btrt_launch_t* c)
{
    if (c && c->steps_per_launch == 1 && c->strip_rows != 0 &&
        (c->strip_rows > 16 || (c->strip_rows & (c->strip_rows - 1))))
        return false;  // one step per launch: tile height 1, 2, 4, 8 or 16 rows
    return c && c->steps_per_launch >= 0 && c->steps_per_launch <= btrtk::kMaxFuse && c->strip_rows >= 0 &&
           c->strip_rows <= (1 << 24) &&
           (c->strips_per_group == 0 || c->strips_per_group == 1 || c->strips_per_group == btrtk::kWalkGroup) &&
           (c->tile == 0 || (c->tile == 1 && c->steps_per_launch == 2));
}

LaunchCfg to_cfg(const btrt_launch_t& c) { return LaunchCfg{c.steps_per_launch, c.strip_rows, c.strips_per_group, c.tile}; }

btrt_launch_t to_public(const LaunchCfg& c) { return btrt_launch_t{c.steps, c.rows, c.group, c.tile}; }

int reduce_sync(btrt* h, int mode, double out[kReducePartials])
{
    int rc = instance_reduce_async(h->inst, mode, h->stream);
    if (rc == BTRT_OK) rc = instance_result_async(h->inst, out, h->stream);
    if (rc != BTRT_OK) return rc;
    hipError_t e = hipStreamSynchronize(h->stream);
    return e == hipSuccess ? static_cast<int>(BTRT_OK) : hip_fail(e, "hipStreamSynchronize");
}

// Waits for the handle's stream, frees what the library allocated and deletes the handle.
void release(btrt* h)
{
    if (!h) return;
    DeviceGuard g(h->device);
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    if (h->own_mem && h->mem) (void)hipFree(h->mem);
    if (h->wsched) (void)hipFree(h->wsched);
    if (h->wspare) (void)hipFree(h->wspare);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    delete h;
}

// ---- checkpoint layout ---------------------------------------------------------------------
// [header (kCkHeader bytes)] [f: the planes of the state (9, or 2 or 3 in the moment form), storage format] [phi: one plane] [snapshot: nx*ny FP64]
// [wall entry: one wall-table entry (Instance::wall_entry_slots() values) in the phi type,
//  general node model only]
constexpr char kCkMagic[8] = {'B', 'T', 'R', 'T', 'C', 'K', 'P', '3'};
constexpr int kCkParams = 48;
constexpr size_t kCkHeader = 512;

struct CkHeader {
    char magic[8];
    int32_t nx, ny, precision, pitch;
    int64_t step;
    int64_t f_bytes, phi_bytes, snap_bytes, wall_bytes;
    int32_t wall_mode;  // 0: per-side constants or none; 1: a wall schedule was active
    int32_t pad;
    double params[kCkParams];
};
static_assert(sizeof(CkHeader) <= kCkHeader, "checkpoint header");

template <typename T>
void ck_params_of(const SweepArgs<T>& a, const Instance& I, double p[kCkParams])
{
    int k = 0;
    auto put = [&](double v) { p[k++] = v; };
    for (double v : I.info.K1) put(v);
    for (double v : I.info.K2) put(v);
    put(I.info.k0);
    put(a.ax); put(a.ay); put(a.bx); put(a.by); put(a.fcx); put(a.fcy); put(a.fq);
    put(a.a11); put(a.a12); put(a.a22); put(a.beta);
    put(a.rr); put(a.rp); put(a.dg); put(a.de); put(a.ds); put(a.dpoly);
    put(a.src_amp);
    for (int q = 0; q < 4; ++q) put(a.wall[q]);
    put(a.dev_scale);
    put(I.kind); put(I.kmode() & btrtk::kK1Mask); put(I.perx); put(I.pery); put(I.growth);
    while (k < kCkParams) put(0.0);
}

void ck_params(const Instance& I, double p[kCkParams])
{
    if (I.precision == BTRT_F64)
        ck_params_of(I.a64, I, p);
    else
        ck_params_of(I.a32, I, p);
}

struct CkSizes {
    size_t f, phi, snap, wall, total;
};

CkSizes ck_sizes(const Instance& I)
{
    CkSizes z{};
    const size_t ps = I.precision == BTRT_F64 ? 8 : 4;
    z.f = static_cast<size_t>(I.state_planes()) * static_cast<size_t>(I.plane) * I.state_bytes();
    z.phi = static_cast<size_t>(I.plane) * ps;
    z.snap = static_cast<size_t>(I.nx) * I.ny * 8;
    z.wall = I.gen ? static_cast<size_t>(I.wall_entry_slots()) * ps : 0;
    z.total = kCkHeader + z.f + z.phi + z.snap + z.wall;
    return z;
}

}  // namespace

extern "C" {

int btrt_checkpoint_size(const btrt_t* h, size_t* bytes)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!bytes) return fail(BTRT_E_INVAL, "bytes is NULL");
    *bytes = ck_sizes(h->inst).total;
    return ok();
}

int btrt_checkpoint(btrt_t* h, void* buf, size_t bytes)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    const Instance& I = h->inst;
    const CkSizes z = ck_sizes(I);
    if (!buf || bytes < z.total) return fail(BTRT_E_INVAL, "checkpoint buffer of %zu bytes < %zu", bytes, z.total);
    DeviceGuard g(h->device);
    if (g.status() != hipSuccess) return hip_fail(g.status(), "hipSetDevice");
    CkHeader hd{};
    std::memcpy(hd.magic, kCkMagic, sizeof(kCkMagic));
    hd.nx = I.nx;
    hd.ny = I.ny;
    hd.precision = I.precision;
    hd.pitch = I.pitch;
    hd.step = I.step;
    hd.f_bytes = static_cast<int64_t>(z.f);
    hd.phi_bytes = static_cast<int64_t>(z.phi);
    hd.snap_bytes = static_cast<int64_t>(z.snap);
    hd.wall_bytes = static_cast<int64_t>(z.wall);
    hd.wall_mode = I.wall_limit != INT64_MAX ? 1 : 0;
    ck_params(I, hd.params);
    char* out = static_cast<char*>(buf);
    std::memset(out, 0, kCkHeader);
    std::memcpy(out, &hd, sizeof(hd));
    char* p = out + kCkHeader;
    hipError_t e = hipMemcpyAsync(p, I.mem + I.L.f[I.cur], z.f, hipMemcpyDeviceToHost, h->stream);
    p += z.f;
    if (e == hipSuccess) e = hipMemcpyAsync(p, I.mem + I.L.phi[I.cur], z.phi, hipMemcpyDeviceToHost, h->stream);
    p += z.phi;
    if (e == hipSuccess) e = hipMemcpyAsync(p, I.mem + I.L.snap, z.snap, hipMemcpyDeviceToHost, h->stream);
    p += z.snap;
    if (e == hipSuccess && z.wall) {
        const size_t es = I.precision == BTRT_F64 ? 8 : 4;
        const char* cur = I.wtab + static_cast<size_t>(I.step - I.wall_t0) * I.wall_stride * es;
        e = hipMemcpyAsync(p, cur, z.wall, hipMemcpyDeviceToHost, h->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    return e == hipSuccess ? ok() : hip_fail(e, "checkpoint copy");
}

int btrt_restore(btrt_t* h, const void* buf, size_t bytes)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    Instance& I = h->inst;
    if (!buf || bytes < kCkHeader) return fail(BTRT_E_INVAL, "not a checkpoint (too short)");
    CkHeader hd;
    std::memcpy(&hd, buf, sizeof(hd));
    if (std::memcmp(hd.magic, kCkMagic, sizeof(kCkMagic)) != 0) return fail(BTRT_E_INVAL, "not a checkpoint");
    const CkSizes z = ck_sizes(I);
    if (hd.nx != I.nx || hd.ny != I.ny || hd.precision != I.precision || hd.pitch != I.pitch)
        return fail(BTRT_E_INVAL, "checkpoint of a %d x %d grid (precision %d) restored into a %d x %d grid (%d)",
                    hd.nx, hd.ny, hd.precision, I.nx, I.ny, I.precision);
    const size_t ps = I.precision == BTRT_F64 ? 8 : 4;
    const size_t wall_entry = static_cast<size_t>(I.wall_entry_slots()) * ps;
    const size_t wall = static_cast<size_t>(hd.wall_bytes);
    if (hd.f_bytes != static_cast<int64_t>(z.f) || hd.phi_bytes != static_cast<int64_t>(z.phi) ||
        hd.snap_bytes != static_cast<int64_t>(z.snap) || (wall != 0 && wall != wall_entry) ||
        bytes < kCkHeader + z.f + z.phi + z.snap + wall || hd.step < 0 || (hd.wall_mode == 1 && wall == 0))
        return fail(BTRT_E_INVAL, "checkpoint sizes do not match this handle");
    double params[kCkParams];
    ck_params(I, params);
    for (int k = 0; k < kCkParams; ++k)
        if (std::memcmp(&params[k], &hd.params[k], sizeof(double)) != 0)
            return fail(BTRT_E_INVAL, "checkpoint of a different problem (derived constant %d differs)", k);
    DeviceGuard g(h->device);
    if (g.status() != hipSuccess) return hip_fail(g.status(), "hipSetDevice");
    const char* p = static_cast<const char*>(buf) + kCkHeader;
    // The general node model by the problem itself (a power-law flux, a phi-dependent source or
    // D != phi I; the same on both sides, as the constants match) keeps its one-entry table in
    // the workspace; a checkpoint taken under a wall schedule brings the values then in force,
    // which become a one-entry table of their own (steps wait for btrt_set_walls).
    const bool problem_gen = I.gen_problem;
    void* wmem = nullptr;
    if (hd.wall_mode == 1) {
        if (hipMalloc(&wmem, wall) != hipSuccess) {
            (void)hipGetLastError();
            return fail(BTRT_E_NOMEM, "hipMalloc of %zu bytes for the wall values failed", wall);
        }
    } else if ((wall != 0) != problem_gen) {
        return fail(BTRT_E_INVAL, "checkpoint of a different problem (node model differs)");
    }
    hipError_t e = hipStreamSynchronize(h->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(I.mem + I.L.f[I.cur], p, z.f, hipMemcpyHostToDevice, h->stream);
    p += z.f;
    if (e == hipSuccess) e = hipMemcpyAsync(I.mem + I.L.phi[I.cur], p, z.phi, hipMemcpyHostToDevice, h->stream);
    p += z.phi;
    if (e == hipSuccess) e = hipMemcpyAsync(I.mem + I.L.snap, p, z.snap, hipMemcpyHostToDevice, h->stream);
    p += z.snap;
    if (e == hipSuccess && wall) {
        char* dst = wmem ? static_cast<char*>(wmem) : I.mem + I.L.wall0;
        e = hipMemcpyAsync(dst, p, wall, hipMemcpyHostToDevice, h->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) {
        if (wmem) (void)hipFree(wmem);
        return hip_fail(e, "restore copy");
    }
    I.step = hd.step;
    if (h->wsched) {
        (void)hipFree(h->wsched);  // the stream is idle
        h->wsched = nullptr;
    }
    I.gen = wall != 0;
    I.wtab = wmem ? static_cast<const char*>(wmem) : (wall ? I.mem + I.L.wall0 : nullptr);
    h->wsched = wmem;
    h->wsched_bytes = wmem ? wall : 0;
    I.wall_t0 = hd.step;
    I.wall_stride = 0;
    I.wall_limit = wmem ? hd.step : INT64_MAX;
    return ok();
}

int btrt_validate(const btrt_grid_t* grid, const btrt_flux_t* B, const btrt_diff_t* K, const btrt_dterm_t* D,
                  const btrt_source_t* R, const btrt_bc_t* bc, const btrt_relax_t* relax, btrt_info_t* info)
{
    Resolved r{};
    int rc = validate(grid, B, K, D, R, bc, relax, &r);
    if (rc != BTRT_OK) return rc;
    if (info) fill_info(grid, r, R ? R->kind : BTRT_SRC_NONE, info);
    return ok();
}

size_t btrt_workspace_size(const btrt_grid_t* grid, const btrt_diff_t* K, const btrt_source_t* R)
{
    if (!grid_ok(grid)) return 0;
    return layout_for(grid->nx, grid->ny, grid->precision, R ? R->kind : BTRT_SRC_NONE, K && K->field).total;
}

int btrt_create(const btrt_grid_t* grid, const btrt_flux_t* B, const btrt_diff_t* K, const btrt_dterm_t* D,
                const btrt_source_t* R, const btrt_bc_t* bc, const btrt_relax_t* relax, const double* phi0,
                btrt_t** out)
{
    if (!out) return fail(BTRT_E_INVAL, "out is NULL");
    *out = nullptr;
    Resolved r{};
    int rc = validate(grid, B, K, D, R, bc, relax, &r);
    if (rc != BTRT_OK) return rc;
    rc = validate_phi0(grid, phi0);
    if (rc != BTRT_OK) return rc;
    const size_t need = layout_for(grid->nx, grid->ny, grid->precision, R ? R->kind : BTRT_SRC_NONE, r.afield).total;
    if (grid->workspace && grid->workspace_bytes < need)
        return fail(BTRT_E_NOMEM, "workspace of %zu bytes < %zu needed", grid->workspace_bytes, need);

    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev <= 0) return fail(BTRT_E_DEVICE, "no HIP device available");
    if (grid->device < 0 || grid->device >= ndev)
        return fail(BTRT_E_DEVICE, "device %d not in [0, %d)", grid->device, ndev);

    btrt* h = new (std::nothrow) btrt();
    if (!h) return fail(BTRT_E_NOMEM, "host allocation failed");
    h->device = grid->device;
    h->check_interval = relax->check_interval;
    {
        DeviceGuard g(h->device);
        if (g.status() != hipSuccess) {
            rc = hip_fail(g.status(), "hipSetDevice");
        } else {
            if (grid->stream) {
                h->stream = static_cast<hipStream_t>(grid->stream);
            } else {
                e = hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking);
                if (e != hipSuccess)
                    rc = hip_fail(e, "hipStreamCreate");
                else
                    h->own_stream = true;
            }
            if (rc == BTRT_OK) {
                if (grid->workspace) {
                    h->mem = static_cast<char*>(grid->workspace);
                } else if (hipMalloc(reinterpret_cast<void**>(&h->mem), need) != hipSuccess) {
                    h->mem = nullptr;
                    (void)hipGetLastError();
                    rc = fail(BTRT_E_NOMEM, "hipMalloc of %zu bytes failed", need);
                } else {
                    h->own_mem = true;
                }
            }
            h->inst.device = h->device;
            if (rc == BTRT_OK) rc = instance_setup(h->inst, grid, B, K, R, bc, r, phi0, h->mem, h->stream);
        }
    }
    if (rc != BTRT_OK) {
        const std::string msg = last_error();
        release(h);
        return fail(rc, "%s", msg.c_str());
    }
    *out = h;
    return ok();
}

int btrt_step(btrt_t* h, int64_t n)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (n < 0) return fail(BTRT_E_INVAL, "n = %lld < 0", static_cast<long long>(n));
    DeviceGuard g(h->device);
    if (g.status() != hipSuccess) return hip_fail(g.status(), "hipSetDevice");
    int rc = enqueue_steps(h, n);
    return rc == BTRT_OK ? ok() : rc;
}

int btrt_set_walls(btrt_t* h, const double* values, int64_t steps)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    Instance& I = h->inst;
    if (!values) return fail(BTRT_E_INVAL, "values is NULL");
    if (steps < 1) return fail(BTRT_E_INVAL, "steps = %lld < 1", static_cast<long long>(steps));
    if (I.precision != BTRT_F64 && I.precision != BTRT_F32)
        return fail(BTRT_E_INVAL, "wall schedules need BTRT_F64 or BTRT_F32 storage");
    const int64_t P = I.wall_entry_values(), S = I.wall_entry_slots();
    const bool wall_side[4] = {!I.perx, !I.perx, !I.pery, !I.pery};
    const int64_t sx = 2LL * I.ny + 1, sy = 2LL * I.nx + 1;
    const int64_t side_begin[5] = {0, sx, 2 * sx, 2 * sx + sy, P};
    const bool finite = all_finite(values, static_cast<size_t>(steps) * P);
    for (int64_t k = 0; k < steps && !finite; ++k)  // say where, unless it is a periodic side's entry
        for (int q = 0; q < 4; ++q) {
            if (!wall_side[q]) continue;
            for (int64_t e = side_begin[q]; e < side_begin[q + 1]; ++e)
                if (!std::isfinite(values[k * P + e]))
                    return fail(BTRT_E_INVAL, "non-finite wall value at step %lld, entry %lld",
                                static_cast<long long>(k), static_cast<long long>(e));
        }
    const size_t es = I.precision == BTRT_F64 ? 8 : 4;
    const size_t bytes = static_cast<size_t>(S) * static_cast<size_t>(steps + 1) * es;
    DeviceGuard g(h->device);
    if (g.status() != hipSuccess) return hip_fail(g.status(), "hipSetDevice");
    // The new values go into the table before the one in force, if it is large enough, else into a new one: a
    // call that fails leaves the schedule in force as it is. (What the spare table once fed is ahead of the new
    // values on the stream.)
    const bool reuse = h->wspare && h->wspare_bytes >= bytes;
    if (!reuse) {
        if (h->wspare) {
            (void)hipStreamSynchronize(h->stream);  // a launch may still read it
            (void)hipFree(h->wspare);
            h->wspare = nullptr;
        }
        if (hipMalloc(&h->wspare, bytes) != hipSuccess) {
            h->wspare = nullptr;
            (void)hipGetLastError();
            return fail(BTRT_E_NOMEM, "hipMalloc of %zu bytes for the wall schedule failed", bytes);
        }
        h->wspare_bytes = bytes;
    }
    char* dst = static_cast<char*>(h->wspare);
    // Entry 0: the values the next pull reads (the step that ends at the current count), from
    // the current table, or the per-side constants the populations were initialised with.
    hipError_t e;
    if (I.gen && I.wtab) {
        const char* cur = I.wtab + static_cast<size_t>(I.step - I.wall_t0) * I.wall_stride * es;
        e = hipMemcpyAsync(dst, cur, static_cast<size_t>(S) * es, hipMemcpyDeviceToDevice, h->stream);
    } else {
        e = upload_wall_entry(I, dst, h->stream);
    }
    if (e == hipSuccess) e = upload_wall_values(I, values, static_cast<size_t>(steps), dst + S * es, h->stream);
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(h->stream);
        return hip_fail(e, "wall schedule upload");
    }
    std::swap(h->wsched, h->wspare);
    std::swap(h->wsched_bytes, h->wspare_bytes);
    I.gen = true;
    I.wtab = dst;
    I.wall_t0 = I.step;
    I.wall_limit = I.step + steps;
    I.wall_stride = static_cast<int>(S);
    return ok();
}

int btrt_set_fusion(btrt_t* h, int32_t steps_per_launch)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (steps_per_launch < 1 || steps_per_launch > btrtk::kMaxFuse)
        return fail(BTRT_E_INVAL, "steps_per_launch = %d: must be in [1, %d]", steps_per_launch, btrtk::kMaxFuse);
    h->launch = LaunchCfg{steps_per_launch, 0, 0, 0};
    return ok();
}

int btrt_set_launch(btrt_t* h, const btrt_launch_t* cfg)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!launch_ok(cfg)) return fail(BTRT_E_INVAL, "invalid launch configuration");
    h->launch = to_cfg(*cfg);
    return ok();
}

int btrt_get_launch(btrt_t* h, btrt_launch_t* cfg)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!cfg) return fail(BTRT_E_INVAL, "cfg is NULL");
    DeviceGuard g(h->device);
    *cfg = to_public(instance_resolve(h->inst, h->launch));
    return ok();
}

int btrt_get_sweep(btrt_t* h, btrt_sweep_t* sweep)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!sweep) return fail(BTRT_E_INVAL, "sweep is NULL");
    DeviceGuard g(h->device);
    *sweep = instance_sweep(h->inst, h->launch);
    return ok();
}

int btrt_tune(btrt_t* h, int64_t max_steps, btrt_launch_t* best, int64_t* steps_used)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (max_steps < 0) return fail(BTRT_E_INVAL, "max_steps < 0");
    max_steps = std::min<int64_t>(max_steps, h->inst.wall_limit - h->inst.step);  // stay inside a wall schedule
    DeviceGuard g(h->device);
    // Candidates: the automatic shape (first), one step per launch, the two-step LDS tile, the
    // automatic strip rows of six and seven steps, and strip walkers over steps per launch x strip
    // rows x strips per group.
    const LaunchCfg automatic = instance_resolve(h->inst, LaunchCfg{});
    std::vector<LaunchCfg> cand{automatic, {1, 4, 0, 0}, {1, 8, 0, 0}, {1, 16, 0, 0}, {2, 0, 0, 1}, {6, 0, 0, 0},
                                {7, 0, 0, 0}};
    for (int k = 2; k <= btrtk::kMaxFuse; ++k)
        for (int rows : {8, 16, 32, 64, 128})
            for (int grp : {1, btrtk::kWalkGroup}) cand.push_back(LaunchCfg{k, rows, grp, 0});
    int64_t used = 0;
    // Times `list` (indices into cand): each candidate runs one untimed launch and `reps` timed
    // ones, as far as max_steps allows; adds each one's time per step to ms_per_step and counts
    // its timings in n.
    auto time_list = [&](const std::vector<size_t>& list, int reps, std::vector<double>& ms_per_step,
                         std::vector<int>& n) -> int {
        std::vector<hipEvent_t> ev;
        std::vector<size_t> timed;
        int rc = BTRT_OK;
        for (size_t c : list) {
            const int span = cand[c].fuse > 0 ? cand[c].fuse : cand[c].steps;  // steps of one launch
            const int64_t need = static_cast<int64_t>(1 + reps) * span;
            if (used + need > max_steps) continue;
            hipEvent_t e0 = nullptr, e1 = nullptr;
            if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
                if (e0) (void)hipEventDestroy(e0);
                rc = fail(BTRT_E_DEVICE, "hipEventCreate failed");
                break;
            }
            ev.push_back(e0);
            ev.push_back(e1);
            rc = enqueue_steps(h, cand[c], span);
            if (rc == BTRT_OK && hipEventRecord(e0, h->stream) != hipSuccess) rc = fail(BTRT_E_DEVICE, "hipEventRecord");
            if (rc == BTRT_OK) rc = enqueue_steps(h, cand[c], static_cast<int64_t>(reps) * span);
            if (rc == BTRT_OK && hipEventRecord(e1, h->stream) != hipSuccess) rc = fail(BTRT_E_DEVICE, "hipEventRecord");
            used += need;
            timed.push_back(c);
            if (rc != BTRT_OK) break;
        }
        hipError_t e = hipStreamSynchronize(h->stream);
        if (rc == BTRT_OK && e != hipSuccess) rc = hip_fail(e, "hipStreamSynchronize");
        for (size_t j = 0; j < timed.size() && rc == BTRT_OK; ++j) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, ev[2 * j], ev[2 * j + 1]) != hipSuccess) {
                rc = fail(BTRT_E_DEVICE, "hipEventElapsedTime failed");
                break;
            }
            const LaunchCfg& t = cand[timed[j]];
            ms_per_step[timed[j]] += ms / (reps * (t.fuse > 0 ? t.fuse : t.steps));
            ++n[timed[j]];
        }
        for (hipEvent_t x : ev) (void)hipEventDestroy(x);
        return rc;
    };
    // Pass 1: every candidate, one timed launch, after a few warm-up launches of the automatic
    // shape. It may still run while the GPU clocks rise, which favours the candidates timed last,
    // so pass 2 re-times the kFinal fastest and the automatic shape in turn, twice over, two timed
    // launches each, and keeps the lowest mean.
    constexpr int kFinal = 4;
    const int64_t warm = std::min<int64_t>(max_steps / 10, 8LL * (automatic.fuse > 0 ? automatic.fuse : automatic.steps));
    if (warm > 0) {
        int rc0 = enqueue_steps(h, automatic, warm);
        if (rc0 != BTRT_OK) return rc0;
        used += warm;
    }
    std::vector<double> t1(cand.size(), 0.0), t2(cand.size(), 0.0);
    std::vector<int> n1(cand.size(), 0), n2(cand.size(), 0);
    std::vector<size_t> all(cand.size());
    for (size_t c = 0; c < cand.size(); ++c) all[c] = c;
    int rc = time_list(all, 1, t1, n1);
    std::vector<size_t> ranked;
    for (size_t c = 0; c < cand.size(); ++c)
        if (n1[c] > 0) ranked.push_back(c);
    std::sort(ranked.begin(), ranked.end(), [&](size_t x, size_t y) { return t1[x] < t1[y]; });
    if (ranked.size() > static_cast<size_t>(kFinal)) ranked.resize(kFinal);
    if (n1[0] > 0 && std::find(ranked.begin(), ranked.end(), size_t{0}) == ranked.end()) ranked.push_back(0);
    for (int round = 0; round < 2 && rc == BTRT_OK; ++round) rc = time_list(ranked, 2, t2, n2);
    if (rc != BTRT_OK) return rc;
    LaunchCfg pick = h->launch;
    double best_ms = -1.0;
    for (size_t c : ranked) {
        const double ms = n2[c] > 0 ? t2[c] / n2[c] : t1[c];  // pass 1 only when the steps ran out
        if (best_ms < 0 || ms < best_ms) {
            best_ms = ms;
            // The automatic shape stays automatic: what it resolves to depends on the model in force, which a
            // wall schedule changes.
            pick = c == 0 ? LaunchCfg{} : cand[c];
        }
    }
    h->launch = pick;
    if (best) *best = to_public(instance_resolve(h->inst, pick));
    if (steps_used) *steps_used = used;
    return ok();
}

int btrt_field(btrt_t* h, double* phi_out)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!phi_out) return fail(BTRT_E_INVAL, "phi_out is NULL");
    DeviceGuard g(h->device);
    int rc = instance_gather(h->inst, -1, phi_out, h->stream);
    return rc == BTRT_OK ? ok() : rc;
}

int btrt_populations(btrt_t* h, double* f_out)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!f_out) return fail(BTRT_E_INVAL, "f_out is NULL");
    DeviceGuard g(h->device);
    const size_t nn = static_cast<size_t>(h->inst.nx) * h->inst.ny;
    for (int i = 0; i < 9; ++i) {
        int rc = instance_gather(h->inst, i, f_out + i * nn, h->stream);
        if (rc != BTRT_OK) return rc;
    }
    return ok();
}

int btrt_residual(btrt_t* h, double* out)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!out) return fail(BTRT_E_INVAL, "out is NULL");
    double v[kReducePartials];
    DeviceGuard g(h->device);
    int rc = reduce_sync(h, kResidual, v);
    if (rc != BTRT_OK) return rc;
    if (v[5] > 0) {
        *out = NAN;
        return fail(BTRT_E_UNSTABLE, "phi holds %.0f non-finite values at step %lld", v[5],
                    static_cast<long long>(h->inst.step));
    }
    *out = v[1] > 0 ? v[0] / v[1] : (v[0] > 0 ? INFINITY : 0.0);
    return ok();
}

int btrt_error(btrt_t* h, const double* ref, double out[3])
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!ref || !out) return fail(BTRT_E_INVAL, "NULL argument");
    const size_t nn = static_cast<size_t>(h->inst.nx) * h->inst.ny;
    double v[kReducePartials];
    DeviceGuard g(h->device);
    hipError_t e = hipMemcpyAsync(h->inst.mem + h->inst.L.tmp, ref, nn * sizeof(double), hipMemcpyHostToDevice,
                                  h->stream);
    if (e != hipSuccess) return hip_fail(e, "reference upload");
    int rc = reduce_sync(h, kError, v);
    if (rc != BTRT_OK) return rc;
    if (v[5] > 0) {
        out[0] = out[1] = out[2] = NAN;
        return fail(BTRT_E_UNSTABLE, "phi holds %.0f non-finite values", v[5]);
    }
    out[0] = v[0] / v[1];
    out[1] = v[4];
    out[2] = std::sqrt(v[2] / v[3]);
    return ok();
}

int btrt_solve(btrt_t* h, double tol, int64_t max_steps, int64_t* steps_taken, double* residual)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (max_steps < 0 || !(tol >= 0.0)) return fail(BTRT_E_INVAL, "bad tol or max_steps");
    int64_t done = 0;
    double res = INFINITY;
    int rc = BTRT_OK;
    while (done < max_steps) {
        const int64_t k = std::min<int64_t>(h->check_interval, max_steps - done);
        rc = btrt_step(h, k);
        if (rc != BTRT_OK) break;
        done += k;
        rc = btrt_residual(h, &res);
        if (rc != BTRT_OK || res <= tol) break;
    }
    if (steps_taken) *steps_taken = done;
    if (residual) *residual = res;
    return rc == BTRT_OK ? ok() : rc;
}

int btrt_sync(btrt_t* h)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    DeviceGuard g(h->device);
    hipError_t e = hipStreamSynchronize(h->stream);
    return e == hipSuccess ? ok() : hip_fail(e, "hipStreamSynchronize");
}

int btrt_get_info(const btrt_t* h, btrt_info_t* info)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    if (!info) return fail(BTRT_E_INVAL, "info is NULL");
    *info = h->inst.info;
    info->step = h->inst.step;
    return ok();
}

int btrt_destroy(btrt_t* h)
{
    if (!h) return fail(BTRT_E_STATE, "NULL handle");
    release(h);
    return ok();
}

const char* btrt_strerror(int code)
{
    switch (code) {
        case BTRT_OK: return "ok";
        case BTRT_E_INVAL: return "invalid argument";
        case BTRT_E_NOMEM: return "out of device memory";
        case BTRT_E_DEVICE: return "HIP device error";
        case BTRT_E_UNSTABLE: return "non-finite values in phi (unstable run)";
        case BTRT_E_STATE: return "invalid handle";
        default: return "unknown error code";
    }
}

const char* btrt_last_error(void) { return last_error(); }

}  // extern "C"
