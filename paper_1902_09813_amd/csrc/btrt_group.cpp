// A group of resident problem instances advanced together: one persistent launch per
// (fused) time step walks the tiles of every member. Shared by the batched C ABI and the
// solve server; membership can change between calls.

#include "btrt_host.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace btrth {

using btrtk::BatchEntry;
using btrtk::kReducePartials;
using btrtk::kResidual;

namespace {

size_t entry_bytes(int precision)
{
    return precision == BTRT_F64 ? sizeof(BatchEntry<double>) : sizeof(BatchEntry<float>);
}

void drop_graph(Group& g)
{
    if (g.gexec) (void)hipGraphExecDestroy(g.gexec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
    g.gexec = nullptr;
    g.graph = nullptr;
}

int grid_blocks(const Group& g) { return g.cfg.blocks_per_cu > 0 ? g.ncu * g.cfg.blocks_per_cu : 0; }

constexpr int kDefaultStripRows = 16;
int strip_rows(const btrt_batch_config_t& c) { return c.strip_rows > 0 ? c.strip_rows : kDefaultStripRows; }

// Members in the moment form advance on regions where no strip height is set (kRegions), else in strips.
constexpr int kRegions = -1;

// Rows of a unit of `steps` steps: the configured strip height, or the tiles' own below four steps.
int unit_rows(const Group& g, int p, int steps)
{
    if (p == 1 && steps > 1 && g.cfg.strip_rows == 0) return kRegions;
    return btrtk::batch_walks(steps) ? strip_rows(g.cfg) : btrtk::tile_rows(steps, g.precision == BTRT_F64 ? 8 : 4);
}

// Launches one part: slot picks the unit table (steps, or 0: one step for the members that need one).
hipError_t part_launch(Group& g, int p, int slot, int steps, int flip)
{
    const Group::Part& P = g.part[p];
    const int n = static_cast<int>(P.inst.size());
    const int rows = unit_rows(g, p, steps);
    if (n == 0 || P.total[slot] == 0) return hipSuccess;
    if (p == 1 && rows == kRegions) {
        if (g.precision == BTRT_F64)
            return btrtk::launch_batch_region<double>(static_cast<const BatchEntry<double>*>(P.d_ent), P.d_begin[slot],
                                                      P.d_par, n, P.total[slot], flip, steps, grid_blocks(g),
                                                      P.region[steps], g.stream);
        return btrtk::launch_batch_region<float>(static_cast<const BatchEntry<float>*>(P.d_ent), P.d_begin[slot], P.d_par,
                                                 n, P.total[slot], flip, steps, grid_blocks(g), P.region[steps], g.stream);
    }
    if (p == 1) {
        if (g.precision == BTRT_F64)
            return btrtk::launch_batch_mom<double>(static_cast<const BatchEntry<double>*>(P.d_ent), P.d_begin[slot], P.d_par,
                                                   n, P.total[slot], flip, steps, grid_blocks(g), rows, g.stream);
        return btrtk::launch_batch_mom<float>(static_cast<const BatchEntry<float>*>(P.d_ent), P.d_begin[slot], P.d_par, n,
                                              P.total[slot], flip, steps, grid_blocks(g), rows, g.stream);
    }
    bool k0one = true;
    for (const Instance* I : P.inst) k0one = k0one && I->k0_one;
    if (g.precision == BTRT_F64)
        return btrtk::launch_batch_sweep<double>(static_cast<const BatchEntry<double>*>(P.d_ent), P.d_begin[slot], P.d_par,
                                                 n, P.total[slot], flip, steps, grid_blocks(g), rows, k0one, g.nts,
                                                 g.stream);
    return btrtk::launch_batch_sweep<float>(static_cast<const BatchEntry<float>*>(P.d_ent), P.d_begin[slot], P.d_par, n,
                                            P.total[slot], flip, steps, grid_blocks(g), rows, k0one, g.nts, g.stream);
}

hipError_t raw_launch(Group& g, int steps, int flip)
{
    hipError_t e = part_launch(g, 0, steps, steps, flip);
    return e == hipSuccess ? part_launch(g, 1, steps, steps, flip) : e;
}

btrtk::BatchGrid grid_of(const Instance& I)
{
    return btrtk::BatchGrid{I.nx, I.ny, I.perx != 0, I.pery != 0};
}

btrtk::BatchRegion region_shape(const Group& g, int steps)
{
    std::vector<btrtk::BatchGrid> grids;
    for (const Instance* I : g.part[1].inst) grids.push_back(grid_of(*I));
    const int n = static_cast<int>(grids.size());
    return g.precision == BTRT_F64 ? btrtk::batch_region<double>(grids.data(), n, steps)
                                   : btrtk::batch_region<float>(grids.data(), n, steps);
}

// Offsets of each member's units in part p's concatenated list for `steps` per launch: 64 x rows
// tiles, or walker strips. skip_first: members whose first step is free get no units.
int upload_begin(Group& g, int p, int slot, int steps, int rows, bool skip_first)
{
    Group::Part& P = g.part[p];
    const int n = static_cast<int>(P.inst.size());
    if (n == 0) return BTRT_OK;
    std::vector<int> begin(n + 1);
    if (rows == kRegions) P.region[steps] = region_shape(g, steps);
    const int width = p == 1 ? btrtk::mom_strip_columns(steps)
                             : (btrtk::batch_walks(steps) ? btrtk::batch_strip_columns(steps) : btrtk::kTileWidth);
    int64_t acc = 0;
    for (int i = 0; i < n; ++i) {
        begin[i] = static_cast<int>(acc);
        const Instance& I = *P.inst[i];
        if (rows == kRegions)
            acc += btrtk::batch_regions(grid_of(I), steps, P.region[steps].rows * P.region[steps].waves);
        else if (!(skip_first && I.first_step_free()))
            acc += static_cast<int64_t>((I.nx + width - 1) / width) * ((I.ny + rows - 1) / rows);
    }
    if (acc > INT32_MAX) return fail(BTRT_E_INVAL, "more than 2^31 - 1 tiles in one group");
    begin[n] = static_cast<int>(acc);
    P.total[slot] = static_cast<int>(acc);
    hipError_t e = hipMemcpyAsync(P.d_begin[slot], begin.data(), (n + 1) * sizeof(int), hipMemcpyHostToDevice,
                                  g.stream);
    if (e == hipSuccess) e = hipStreamSynchronize(g.stream);
    return e == hipSuccess ? static_cast<int>(BTRT_OK) : hip_fail(e, "group table upload");
}

// The unit tables of k steps per launch for the configured strip height (built when first needed).
int ensure_table(Group& g, int k)
{
    for (int p = 0; p < 2; ++p) {
        const int rows = unit_rows(g, p, k);
        if (g.part[p].built_rows[k] == rows || g.part[p].inst.empty()) continue;
        int rc = upload_begin(g, p, k, k, rows, false);
        if (rc != BTRT_OK) return rc;
        g.part[p].built_rows[k] = rows;
    }
    return BTRT_OK;
}

void advance(Group& g, int steps, int launches)
{
    if (launches & 1) {
        g.flip ^= 1;
        for (Instance* I : g.inst) I->cur ^= 1;
    }
    for (Instance* I : g.inst) I->step += static_cast<int64_t>(steps) * launches;
}

int launch_once(Group& g, int steps)
{
    int rc = ensure_table(g, steps);
    if (rc != BTRT_OK) return rc;
    hipError_t e = raw_launch(g, steps, g.flip);
    if (e != hipSuccess) return hip_fail(e, "batch sweep launch");
    advance(g, steps, 1);
    return BTRT_OK;
}

// Captures cfg.graph_launches launches (flip 0, 1, 0, ...) into a graph.
int build_graph(Group& g)
{
    drop_graph(g);
    hipError_t e = hipStreamBeginCapture(g.stream, hipStreamCaptureModeRelaxed);
    if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
    hipError_t le = hipSuccess;
    for (int j = 0; j < g.cfg.graph_launches && le == hipSuccess; ++j) le = raw_launch(g, g.cfg.steps_per_launch, j & 1);
    e = hipStreamEndCapture(g.stream, &g.graph);
    if (le != hipSuccess) return hip_fail(le, "batch sweep capture");
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    e = hipGraphInstantiate(&g.gexec, g.graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        drop_graph(g);
        return hip_fail(e, "hipGraphInstantiate");
    }
    g.gcfg = g.cfg;
    return BTRT_OK;
}

template <typename T>
void fill_entries(const Group::Part& P, std::vector<BatchEntry<T>>& ent, bool nts)
{
    ent.resize(P.inst.size());
    for (size_t i = 0; i < P.inst.size(); ++i) {
        const Instance& I = *P.inst[i];
        for (int p = 0; p < 2; ++p) {
            ent[i].a[p] = sweep_args<T>(I, p);
            ent[i].a[p].nts = nts ? 1 : 0;
        }
        ent[i].variant = 2 * (I.mom ? (I.kind != btrtk::kSrcNone ? 1 : 0) : I.kind) + (I.k1_per_node ? 1 : 0);
        ent[i].pad = 0;
    }
}

}  // namespace

bool config_ok(const btrt_batch_config_t* c)
{
    return c && btrtk::batch_steps_ok(c->steps_per_launch) &&
           c->strip_rows >= 0 && c->strip_rows <= 4096 && c->blocks_per_cu >= 0 &&
           c->blocks_per_cu <= 64 && c->graph_launches >= 0 && c->graph_launches <= 4096 &&
           (c->graph_launches == 0 || (c->graph_launches >= 2 && c->graph_launches % 2 == 0));
}

int group_init(Group& g, int device, hipStream_t s, int precision, int capacity)
{
    g.device = device;
    g.stream = s;
    g.precision = precision;
    g.capacity = capacity;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess && prop.multiProcessorCount > 0)
        g.ncu = prop.multiProcessorCount;
    // Per part: entries, unit offsets for 1, 2, 4, 6 and 7 steps and for a first step, parities.
    const size_t ints = align_up(static_cast<size_t>(capacity + 1) * sizeof(int));
    const size_t bytes = 2 * (align_up(capacity * entry_bytes(precision)) + 7 * ints);
    if (hipMalloc(reinterpret_cast<void**>(&g.tables), bytes) != hipSuccess) {
        g.tables = nullptr;
        (void)hipGetLastError();
        return fail(BTRT_E_NOMEM, "hipMalloc of %zu bytes failed", bytes);
    }
    char* t = g.tables;
    for (Group::Part& P : g.part) {
        P.d_ent = t;
        t += align_up(capacity * entry_bytes(precision));
        for (int k : {0, 1, 2, 4, 6, 7}) {
            P.d_begin[k] = reinterpret_cast<int*>(t);
            t += ints;
        }
        P.d_par = reinterpret_cast<int*>(t);
        t += ints;
    }
    if (hipHostMalloc(reinterpret_cast<void**>(&g.h_res),
                      static_cast<size_t>(capacity) * kReducePartials * sizeof(double)) != hipSuccess) {
        g.h_res = nullptr;
        return fail(BTRT_E_NOMEM, "pinned host allocation failed");
    }
    return BTRT_OK;
}

int group_upload(Group& g)
{
    drop_graph(g);
    const int n = static_cast<int>(g.inst.size());
    if (n > g.capacity) return fail(BTRT_E_INVAL, "group of %d exceeds its capacity %d", n, g.capacity);
    g.flip = 0;
    double state = 0;
    for (const Instance* I : g.inst) state += 2.0 * (I->state_planes() + 1.0) * I->plane * (g.precision == BTRT_F64 ? 8 : 4);
    g.nts = state > 256.0 * 1024 * 1024;  // the members' state exceeds the Infinity Cache
    for (int p = 0; p < 2; ++p) {
        Group::Part& P = g.part[p];
        P.inst.clear();
        for (Instance* I : g.inst)
            if ((I->mom ? 1 : 0) == p) P.inst.push_back(I);
        for (int k = 0; k <= btrtk::kBatchMaxSteps; ++k) P.built_rows[k] = P.total[k] = 0;
        if (P.inst.empty()) continue;
        std::vector<int> par(P.inst.size());
        for (size_t i = 0; i < P.inst.size(); ++i) par[i] = P.inst[i]->cur;
        hipError_t e = hipMemcpyAsync(P.d_par, par.data(), par.size() * sizeof(int), hipMemcpyHostToDevice, g.stream);
        if (e == hipSuccess) e = hipStreamSynchronize(g.stream);
        if (e == hipSuccess && g.precision == BTRT_F64) {
            std::vector<BatchEntry<double>> ent;
            fill_entries(P, ent, g.nts);
            e = hipMemcpyAsync(P.d_ent, ent.data(), ent.size() * sizeof(ent[0]), hipMemcpyHostToDevice, g.stream);
            if (e == hipSuccess) e = hipStreamSynchronize(g.stream);
        } else if (e == hipSuccess) {
            std::vector<BatchEntry<float>> ent;
            fill_entries(P, ent, g.nts);
            e = hipMemcpyAsync(P.d_ent, ent.data(), ent.size() * sizeof(ent[0]), hipMemcpyHostToDevice, g.stream);
            if (e == hipSuccess) e = hipStreamSynchronize(g.stream);
        }
        if (e != hipSuccess) return hip_fail(e, "group table upload");
    }
    return BTRT_OK;
}

namespace {

// The first step of members whose planes already hold it changes their count alone; where others
// must take a step with them, those do so in a launch of their own.
int first_step(Group& g)
{
    size_t free_members = 0;
    for (const Instance* I : g.inst) free_members += I->first_step_free() ? 1 : 0;
    if (free_members == 0) return 0;
    if (free_members < g.inst.size()) {
        for (int p = 0; p < 2; ++p) {
            int rc = upload_begin(g, p, 0, 1, unit_rows(g, p, 1), true);
            if (rc != BTRT_OK) return -rc;
        }
        for (int p = 0; p < 2; ++p) {
            hipError_t e = part_launch(g, p, 0, 1, g.flip);
            if (e != hipSuccess) return -hip_fail(e, "batch sweep launch");
        }
        advance(g, 1, 1);  // members passed over hold their state in both buffers
    } else {
        for (Instance* I : g.inst) I->step += 1;
    }
    return 1;
}

}  // namespace

// Steps per launch by the members' states. All in the moment form: the regions' model picks. Else, with
// few nodes, whose rounds are latency-bound, the fully parallel two-step tiles; from kAutoWalkNodes on
// (measured with a served workload) four-step units, which move the state once per four steps.
btrt_batch_config_t group_auto(const Group& g)
{
    constexpr int64_t kAutoWalkNodes = int64_t(1) << 21;
    if (!g.part[0].inst.empty()) {
        int64_t nodes = 0;
        for (const Instance* I : g.inst) nodes += static_cast<int64_t>(I->nx) * I->ny;
        return btrt_batch_config_t{nodes >= kAutoWalkNodes ? 4 : 2, 0, 0, 0};
    }
    btrt_batch_config_t best{2, 0, 0, 0};
    double best_t = 0;
    if (g.part[1].inst.empty()) return best;
    for (int k : {2, 4, 6, 7}) {
        const double t = region_shape(g, k).cost / k;
        if (best_t == 0 || t < best_t) {
            best_t = t;
            best.steps_per_launch = k;
        }
    }
    return best;
}

int group_enqueue(Group& g, int64_t n)
{
    if (g.inst.empty()) return BTRT_OK;
    int64_t left = n;
    if (left > 0) {
        const int done = first_step(g);
        if (done < 0) return -done;
        left -= done;
    }
    const int k = g.cfg.steps_per_launch;
    const int L = g.cfg.graph_launches;
    if (left >= k) {
        int rc = ensure_table(g, k);
        if (rc != BTRT_OK) return rc;
    }
    if (L > 0) {
        const int64_t chunk = static_cast<int64_t>(L) * k;
        if (left >= chunk + (g.flip ? k : 0)) {
            if (g.flip) {  // the graph starts from flip 0
                int rc = launch_once(g, k);
                if (rc != BTRT_OK) return rc;
                left -= k;
            }
            if (!g.gexec || g.gcfg.steps_per_launch != g.cfg.steps_per_launch ||
                g.gcfg.blocks_per_cu != g.cfg.blocks_per_cu || g.gcfg.graph_launches != L ||
                g.gcfg.strip_rows != g.cfg.strip_rows) {
                int rc = build_graph(g);
                if (rc != BTRT_OK) return rc;
            }
            while (left >= chunk) {
                hipError_t e = hipGraphLaunch(g.gexec, g.stream);
                if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
                advance(g, k, L);
                left -= chunk;
            }
        }
    }
    while (left > 0) {
        // Whole launches of k steps, then 2 and 1 for the remainder.
        const int s = left >= k ? k : (left >= 2 ? 2 : 1);
        int rc = launch_once(g, s);
        if (rc != BTRT_OK) return rc;
        left -= s;
    }
    return BTRT_OK;
}

int group_residuals(Group& g, double* out, int* bad)
{
    const int n = static_cast<int>(g.inst.size());
    for (int i = 0; i < n; ++i) {
        int rc = instance_reduce_async(*g.inst[i], kResidual, g.stream);
        if (rc == BTRT_OK) rc = instance_result_async(*g.inst[i], g.h_res + i * kReducePartials, g.stream);
        if (rc != BTRT_OK) return rc;
    }
    hipError_t e = hipStreamSynchronize(g.stream);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    int nb = 0;
    for (int i = 0; i < n; ++i) {
        const double* v = g.h_res + i * kReducePartials;
        if (v[5] > 0) {
            out[i] = NAN;
            ++nb;
        } else {
            out[i] = v[1] > 0 ? v[0] / v[1] : (v[0] > 0 ? INFINITY : 0.0);
        }
    }
    if (bad) *bad = nb;
    return BTRT_OK;
}

int group_tune(Group& g, int64_t max_steps, btrt_batch_config_t* best, int64_t* used_out)
{
    std::vector<btrt_batch_config_t> cand;
    for (int k : {4, 6, 7})
        for (int rows : {0, 16, 32}) cand.push_back({k, 0, 16, rows});
    cand.push_back({4, 0, 0, 32});
    cand.push_back({4, 4, 16, 32});
    for (int gl : {0, 16}) cand.push_back({2, 0, gl, 0});
    cand.push_back({1, 0, 16, 0});
    // A few warm-up steps of the configuration in force, then pass 1: each candidate runs k untimed
    // steps and one timed graph-replay's worth (16 launches of k steps), as far as three quarters
    // of max_steps allow. Pass 1 may run while the GPU clocks still rise, which favours candidates
    // timed late, so pass 2 re-times the kFinal fastest in turn, twice over, within the rest of
    // max_steps, and the lowest mean time per step wins.
    constexpr int kFinal = 3;
    const btrt_batch_config_t keep = g.cfg;
    int64_t used = 0;
    btrt_batch_config_t best_cfg = keep;
    if (!g.inst.empty()) {
        hipEvent_t t0 = nullptr, t1 = nullptr;
        if (hipEventCreate(&t0) != hipSuccess || hipEventCreate(&t1) != hipSuccess) {
            if (t0) (void)hipEventDestroy(t0);
            return fail(BTRT_E_DEVICE, "hipEventCreate");
        }
        int rc = BTRT_OK;
        std::vector<double> ms_sum(cand.size(), 0.0);
        std::vector<int> n(cand.size(), 0);
        // Times candidate c (k untimed steps, or 2 k so that the timed run starts at launch
        // parity 0 where a graph replay starts, then 16 k timed) if it fits within `limit` steps.
        auto time_one = [&](size_t c, int64_t limit) -> int {
            const int k = cand[c].steps_per_launch;
            const int64_t per = 16LL * k;
            const int64_t warm_k = g.flip ? k : 2LL * k;  // each launch flips the parity
            if (used + warm_k + per > limit) return BTRT_OK;
            g.cfg = cand[c];
            int r = group_enqueue(g, warm_k);
            used += warm_k;
            if (r == BTRT_OK) r = ensure_table(g, k);
            if (r == BTRT_OK && cand[c].graph_launches > 0) r = build_graph(g);
            if (r != BTRT_OK) return r;
            (void)hipEventRecord(t0, g.stream);
            r = group_enqueue(g, per);
            (void)hipEventRecord(t1, g.stream);
            (void)hipEventSynchronize(t1);
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, t0, t1);
            used += per;
            if (r == BTRT_OK) {
                ms_sum[c] += ms / per;
                ++n[c];
            }
            return r;
        };
        const int64_t warm = std::min<int64_t>(max_steps / 10, 64) / keep.steps_per_launch * keep.steps_per_launch;
        if (warm > 0) {
            rc = group_enqueue(g, warm);
            used += warm;
        }
        for (size_t c = 0; c < cand.size() && rc == BTRT_OK; ++c) rc = time_one(c, max_steps * 3 / 4);
        std::vector<size_t> ranked;
        for (size_t c = 0; c < cand.size(); ++c)
            if (n[c] > 0) ranked.push_back(c);
        std::sort(ranked.begin(), ranked.end(), [&](size_t x, size_t y) { return ms_sum[x] < ms_sum[y]; });
        if (ranked.size() > static_cast<size_t>(kFinal)) ranked.resize(kFinal);
        std::vector<double> first(ms_sum);
        std::vector<int> n1(n);
        for (size_t c : ranked) {
            ms_sum[c] = 0.0;
            n[c] = 0;
        }
        for (int round = 0; round < 2 && rc == BTRT_OK; ++round)
            for (size_t j = 0; j < ranked.size() && rc == BTRT_OK; ++j) rc = time_one(ranked[j], max_steps);
        (void)hipEventDestroy(t0);
        (void)hipEventDestroy(t1);
        if (rc != BTRT_OK) {
            g.cfg = keep;
            return rc;
        }
        double best_ms = INFINITY;
        for (size_t c : ranked) {
            const double ms = n[c] > 0 ? ms_sum[c] / n[c] : first[c] / n1[c];  // pass 1 only if the steps ran out
            if (ms < best_ms) {
                best_ms = ms;
                best_cfg = cand[c];
            }
        }
    }
    g.cfg = best_cfg;
    if (best) *best = best_cfg;
    if (used_out) *used_out = used;
    return BTRT_OK;
}

void group_free(Group& g)
{
    drop_graph(g);
    if (g.tables) (void)hipFree(g.tables);
    if (g.h_res) (void)hipHostFree(g.h_res);
    g.tables = nullptr;
    g.h_res = nullptr;
    g.inst.clear();
}

}  // namespace btrth
