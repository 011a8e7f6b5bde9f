// Batched solves on the persistent kernels: blocks run as teams of workgroups, every team all
// steps of one replica group of one block inside one launch per class, state and couplings on
// chip (band_persistent_kernel.h, strip_persistent_kernel.h).  The planner decides which
// blocks run this way and where; the others keep the per-step launches.
#include <algorithm>
#include <numeric>
#include <queue>

#include "band_persistent.h"

namespace qh {

// One graph's entry for k_batch_geometry: `units` band blocks, or row tiles of a dense graph, whose
// strips go to off / lo / w / tiles from index `at` on (band blocks: lo and w only).
struct GeomDesc {
    const int32_t *p0, *p1;     // bb_lo, bb_w or t_ptr, t_col
    int32_t units, dense, eb, pad;
    int64_t at;
};

// The blocks' geometry in one buffer, so that the host reads it with one copy.  A row tile that spans
// more tiles than a word has bits gets width 0; gap[b]: stored tiles that are not consecutive.
__global__ __launch_bounds__(256) void k_batch_geometry(const GeomDesc *__restrict__ G, int64_t *__restrict__ off,
                                                        int32_t *__restrict__ lo, int32_t *__restrict__ w,
                                                        uint64_t *__restrict__ tiles, int32_t *__restrict__ gap) {
    const GeomDesc &g = G[blockIdx.x];
    bool gaps = false;
    for (int64_t i = threadIdx.x; i < g.units; i += 256) {
        if (!g.dense) {
            lo[g.at + i] = g.p0[i];
            w[g.at + i] = g.p1[i];
            continue;
        }
        constexpr int S = kTile / kBandRows;
        const int32_t t0 = g.p0[i], t1 = g.p0[i + 1];
        const int32_t c0 = t1 > t0 ? g.p1[t0] : (int32_t)i, nt = t1 > t0 ? g.p1[t1 - 1] - c0 + 1 : 1;
        uint64_t m = 0;
        if (nt <= 64)
            for (int32_t t = t0; t < t1; ++t) m |= 1ull << (g.p1[t] - c0);
        gaps |= nt != t1 - t0;
        for (int s = 0; s < S; ++s) {
            const int64_t e = g.at + i * S + s;
            off[e] = ((int64_t)t0 * kTileElems + s * (kTileElems / S)) * g.eb;
            lo[e] = c0 * kTile;
            w[e] = nt <= 64 ? nt * kTile : 0;
            tiles[e] = m;
        }
    }
    const int any = __syncthreads_or(gaps);
    if (threadIdx.x == 0) gap[blockIdx.x] = any;
}

// Shorter schedules keep the per-step launches: geometry, placement, tables and cooperative launches cost a
// call 90 us (2 blocks) to 500 us (200 uneven ones) that they do not earn back.  us per call of 8 / 16 /
// 32 steps, per-step / teams: 2 blocks of 50-100, R = 16 190 / 268, 244 / 281, 350 / 316; 200 SNP blocks of
// 50-3,000 896 / 995, 1,182 / 1,062, 1,733 / 1,199; 600 blocks of 50-300, R = 64 1,527 / 1,779, 1,819 / 1,867,
// 2,424 / 2,030.
constexpr int kTeamMinSteps = 24;
static_assert(kTeamMinSteps >= kBpMinSteps);

namespace {

struct Geo {
    int b;                      // block
    const int32_t *lo, *w;      // host geometry of its band blocks (strips)
    int64_t at;
    int32_t nblk;
    int32_t below, above;       // most rows a band block reaches past its own
    double quads, stream_us;    // mean width; per-step kernels' time at the chip's memory rate
};

struct Team {
    int g, wpg;                 // class-local graph
    double us;
    std::vector<int> at;        // workgroups
};

// A class of a batch with one kernel variant: teams (one per graph and replica group).
struct ClassPlan {
    double us = 0.0;            // at least: the teams' time + the other blocks' per-step time
    int rt = 0, um = 0;
    std::vector<char> in;       // graphs that run as teams
    std::vector<Team> teams;
};

}  // namespace

// Teams onto workgroups: widest first, then longest, each onto the workgroups that are free
// earliest; it starts when all of them are.  Every workgroup takes its teams in this order, so the
// first unfinished team always has all its workgroups (no two wait for each other).
static double place(std::vector<Team> &teams, int n_cu, int &workers) {
    std::stable_sort(teams.begin(), teams.end(),
                     [](const Team &a, const Team &b) { return a.wpg != b.wpg ? a.wpg > b.wpg : a.us > b.us; });
    std::vector<double> load(n_cu, 0.0);
    std::vector<int> id(n_cu);
    double end = 0.0;
    std::iota(id.begin(), id.end(), 0);
    auto less = [&](int a, int b) { return load[a] != load[b] ? load[a] < load[b] : a < b; };
    size_t i = 0;
    for (; i < teams.size() && teams[i].wpg > 1; ++i) {
        Team &t = teams[i];
        std::nth_element(id.begin(), id.begin() + t.wpg - 1, id.end(), less);
        double start = 0.0;
        for (int k = 0; k < t.wpg; ++k) start = std::max(start, load[id[k]]);
        t.at.assign(id.begin(), id.begin() + t.wpg);
        std::sort(t.at.begin(), t.at.end());
        for (int k : t.at) load[k] = start + t.us;
        end = std::max(end, start + t.us);
    }
    using L = std::pair<double, int>;
    std::priority_queue<L, std::vector<L>, std::greater<L>> heap;
    for (int k = 0; k < n_cu; ++k) heap.push({load[k], k});
    for (; i < teams.size(); ++i) {
        const L l = heap.top();
        heap.pop();
        teams[i].at.assign(1, l.second);
        heap.push({l.first + teams[i].us, l.second});
        end = std::max(end, l.first + teams[i].us);
    }
    workers = 0;
    for (const Team &t : teams) workers = std::max(workers, t.at.back() + 1);
    return end;
}

// The class's graphs as teams of the kernel variant (rt, um): each graph over the fewest
// workgroups that hold it.  all = false leaves out the blocks whose share of the chip takes
// longer than the per-step kernels' memory traffic at 4.5 TB/s (and whatever does not fit): a
// dense block of more than about 3,300 reads has rows of x that leave LDS no room for 32 replicas,
// and with 16 its couplings are held twice.  Measured per step, all blocks per-step / as planned:
// 3,000 uneven blocks (FP8 reads, BF16 SNPs, R = 32) 1,075 / 810 us; 12 F16 read and 12 F16 SNP blocks of
// 50-900 vertices, R = 64: 23.8 / 6.3; 1,500 SNP blocks alone 333 / 113.
static ClassPlan plan_class(const std::vector<Geo> &gs, int dtype, bool strips, int R, int rt, int um, int n_cu,
                            bool all) {
    ClassPlan c;
    c.rt = rt;
    c.um = um;
    c.in.assign(gs.size(), 0);
    const int held = band_held_chunks(dtype, um, strips);
    double rest = 0.0, tail = 0.0, sum = 0.0, longest = 0.0;
    for (size_t i = 0; i < gs.size(); ++i) {
        const Geo &g = gs[i];
        bool fits = false;
        double us = 0.0;
        int wpg = (int)ceil_div(g.nblk, um * kBpWaves);
        for (; g.quads > 0.0 && wpg <= n_cu; ++wpg) {
            const int64_t own = ceil_div(g.nblk, wpg) * kBandRows, all_rows = (int64_t)g.nblk * kBandRows;
            const int64_t rows = std::min(all_rows, own + g.below + g.above);
            if (band_lds_bytes(rows, rt, strips) > kBpLdsLimit) {
                if (own <= kBandRows) break;
                continue;
            }
            fits = true;
            us = band_step_us(g.quads, std::max(0.0, g.quads / 4.0 - held), ceil_div(g.nblk, wpg), wpg, rt, strips);
            break;
        }
        const int groups = R / rt;
        if (fits && (all || us * wpg * groups / n_cu < g.stream_us)) {
            c.in[i] = 1;
            for (int q = 0; q < groups; ++q) c.teams.push_back({(int)i, wpg, us, {}});
            sum += us * wpg * groups;
            longest = std::max(longest, us);
        } else {
            rest += g.stream_us;
            tail = std::max(tail, 3.0 + g.quads * 0.03);
        }
    }
    c.us = std::max(sum / n_cu, longest) + std::max(rest, tail);
    return c;
}

void plan_batch_teams(const qh_graph *const *gs, const std::vector<SolvePlan *> &plans,
                      const std::vector<BlockDesc> &desc, const qh_bsb_opts *o, BatchTeams &bt, hipStream_t st) {
    const int nb = (int)desc.size(), R = o->replicas;
    bt.in.assign(nb, 0);
    int dev = 0, n_cu = 0, coop = 0;
    QH_HIP(hipGetDevice(&dev));
    QH_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    QH_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop || n_cu < 1 || o->steps < kTeamMinSteps || o->steps >= (1 << 30)) return;

    // geometry: dense blocks' strips first (they have tables of their own), then band blocks
    std::vector<GeomDesc> gd(nb);
    int64_t strips = 0, units = 0;
    for (int pass = 0; pass < 2; ++pass)
        for (int b = 0; b < nb; ++b) {
            const qh_graph *g = gs[b];
            const bool dense = g->storage == QH_STORE_DENSE;
            if (dense != (pass == 0)) continue;
            GeomDesc &d = gd[b];
            d = GeomDesc{};
            d.dense = dense;
            d.p0 = dense ? g->t_ptr.p : g->bb_lo.p;
            d.p1 = dense ? g->t_col.p : g->bb_w.p;
            d.units = (int32_t)(dense ? g->n_rt : g->n_bblk);
            d.eb = dense ? (int32_t)dtype_bytes(g->dtype) : 0;
            d.at = units;
            units += dense ? g->n_rt * (kTile / kBandRows) : g->n_bblk;
            if (dense) strips = units;
        }
    if (!units) return;
    DevBuf<GeomDesc> d_gd(nb);
    d_gd.upload(gd.data(), nb, st);
    bt.off.alloc(strips);
    bt.tiles.alloc(strips);
    bt.geo.alloc(2 * units + nb);
    int32_t *lo = bt.geo.p, *wd = lo + units, *gap = wd + units;
    hipLaunchKernelGGL(k_batch_geometry, dim3(nb), dim3(256), 0, st, d_gd.p, bt.off.p, lo, wd, bt.tiles.p, gap);
    QH_CHECK_LAUNCH();
    const std::vector<int32_t> h = download(bt.geo.p, 2 * units + nb, st);

    std::vector<BandTeam> teams;
    std::vector<std::vector<BandJob>> jobs;            // of all launches, by workgroup
    int64_t xch = 0, flags = 0;
    for (int cls = 0; cls < kBatchClasses; ++cls) {
        const bool dense = cls < 4, str = dense && cls > 0;
        std::vector<Geo> geo;
        for (int b = 0; b < nb; ++b) {
            const qh_graph *g = gs[b];
            if (batch_class(g) != cls || gd[b].units == 0 || g->n >= ((int64_t)1 << 26)) continue;
            if (dense && o->field && h[2 * units + b]) continue;   // (a state that may not stay finite)
            Geo e{};
            e.b = b;
            e.at = gd[b].at;
            e.lo = h.data() + e.at;
            e.w = h.data() + units + e.at;
            e.nblk = gd[b].units * (dense ? kTile / kBandRows : 1);
            bool ok = true;
            for (int32_t k = 0; k < e.nblk; ++k) {
                const int32_t own = k * kBandRows;
                ok = ok && (e.w[k] > 0 || !dense);
                e.quads += (double)ceil_div(e.w[k], 4);
                e.below = std::max(e.below, own - e.lo[k]);
                e.above = std::max(e.above, e.lo[k] + e.w[k] - own - kBandRows);
            }
            e.quads = ok ? std::max(e.quads / e.nblk, 1e-9) : 0.0;
            e.stream_us = dense ? ((double)g->n_tiles * kTileElems * dtype_bytes(g->dtype) + (double)g->n * R * 20.0) / 4.5e6
                                : ((double)g->bb_elems * dtype_bytes(g->bb_dtype) + (double)g->n * R * 16.0) / 1.5e6;
            geo.push_back(e);
        }
        if (geo.empty()) continue;
        const int dtype = str ? cls == 1 ? QH_F16 : cls == 2 ? QH_BF16 : QH_FP8_ROWSCALE
                              : cls == 0 ? kBpTiles : cls == 4 ? QH_F32 : cls == 5 ? QH_F16 : QH_BF16;
        ClassPlan best;
        bool any = false;
        for (int rt : {32, 16}) {
            if (R % rt) continue;
            for (int um = 1; um <= (str ? 4 : 8); um *= 2)
                for (int all = 0; all < 2; ++all) {
                    ClassPlan c = plan_class(geo, dtype, str, R, rt, um, n_cu, all != 0);
                    if (!any || c.us < best.us) best = std::move(c);
                    any = true;
                }
        }
        if (best.teams.empty()) continue;
        // the launch's jobs, per workgroup in the placement's order
        BatchTeams::Launch L;
        BandLaunch &bl = L.launch;
        L.us = place(best.teams, n_cu, bl.grid);
        bl.rt = best.rt;
        bl.um = best.um;
        bl.dtype = dtype;
        bl.strips = str;
        std::vector<int> team_of(geo.size(), -1), group(geo.size(), 0);
        std::vector<BandSplit> split(geo.size());
        std::vector<std::vector<BandJob>> wj(bl.grid);
        for (const Team &t : best.teams) {
            const Geo &e = geo[t.g];
            const qh_graph *g = gs[e.b];
            BandSplit &s = split[t.g];
            if (team_of[t.g] < 0) {
                s = split_band(e.lo, e.w, e.nblk, t.wpg);
                bl.lds_bytes = std::max(bl.lds_bytes, band_lds_bytes(s.lds_rows, best.rt, str));
                team_of[t.g] = (int)teams.size();
                BandTeam T{};
                T.bb_off = dense ? bt.off.p + e.at : g->bb_off.p;
                T.bb_lo = lo + e.at;
                T.bb_w = wd + e.at;
                T.bb_val = dense ? g->t_val.p : g->bb_val.p;
                T.scale = g->row_scale.p;
                T.tiles = dense ? bt.tiles.p + e.at : nullptr;
                T.x = plans[e.b]->xa.p;
                T.y = plans[e.b]->y.p;
                T.field = desc[e.b].field;
                T.c0 = desc[e.b].c0;
                T.bscale = dense ? 1.0f : g->bb_scale;
                T.n = (int32_t)g->n;
                teams.push_back(T);
                bt.in[e.b] = 1;
                plans[e.b]->one_rt = best.rt;
                plans[e.b]->one_wpg = t.wpg;
                plans[e.b]->one_lds = band_lds_bytes(s.lds_rows, best.rt, str);
            }
            const int64_t rows = (int64_t)e.nblk * kBandRows;
            for (int w = 0; w < t.wpg; ++w) {
                BandJob J = s.part[w];
                J.team = team_of[t.g];
                J.r0 = group[t.g] * best.rt;
                J.t0 = 0;
                J.flag_off = (int32_t)flags;
                J.xch_rows = (int32_t)rows;
                J.xch_off = xch;
                wj[t.at[w]].push_back(J);
            }
            ++group[t.g];
            if (t.wpg > 1) {
                flags += t.wpg * kBpWaves;
                xch += rows * best.rt * (str ? 1 : 2);
            }
        }
        if (bl.lds_bytes > kBpLdsLimit) fail(QH_EUNSUPPORTED, "a team's rows exceed the LDS");
        L.ptr_at = (int64_t)jobs.size();               // (made into offsets below)
        for (auto &v : wj) jobs.push_back(std::move(v));
        bt.launches.push_back(std::move(L));
    }
    if (bt.launches.empty()) return;
    // one table of jobs and one of pointers: a launch's pointers are grid + 1 entries
    std::vector<BandJob> all;
    std::vector<int32_t> ptr;
    for (auto &L : bt.launches) {
        const int64_t first = L.ptr_at;
        L.ptr_at = (int64_t)ptr.size();
        ptr.push_back((int32_t)all.size());
        for (int w = 0; w < L.launch.grid; ++w) {
            all.insert(all.end(), jobs[first + w].begin(), jobs[first + w].end());
            ptr.push_back((int32_t)all.size());
        }
    }
    alloc_exchange(bt.xch, xch);                       // (the largest first: it may find no room)
    bt.teams.alloc(teams.size());
    bt.teams.upload(teams.data(), teams.size(), st);
    bt.jobs.alloc(all.size());
    bt.jobs.upload(all.data(), all.size(), st);
    bt.ptr.alloc(ptr.size());
    bt.ptr.upload(ptr.data(), ptr.size(), st);
    bt.flags.alloc((size_t)flags + kBpFlagsPad);
    bt.n_flags = flags;
    QH_HIP(hipStreamSynchronize(st));                  // (the uploads read this function's vectors)
}

void run_batch_teams(BatchTeams &bt, const qh_bsb_opts *o, double a0, const float *pump, hipStream_t st) {
    if (bt.launches.empty()) return;
    bt.flags.zero(st);
    for (const BatchTeams::Launch &L : bt.launches) {
        BandPersistArgs a{};
        a.R = o->replicas;
        a.kb = 0;
        a.ke = o->steps;
        a.dt = (float)o->dt;
        a.a0 = (float)a0;
        a.pump = pump;
        a.teams = bt.teams.p;
        a.jobs = bt.jobs.p;
        a.job_ptr = bt.ptr.p + L.ptr_at;
        a.xch = bt.xch.p;
        a.flags = bt.flags.p;
        a.err = bt.flags.p + bt.n_flags + kBpErr;
        // a team may wait for a workgroup that is still busy with its earlier teams; a poll takes 0.1 us
        // or more
        a.max_polls = std::max(kWaitPolls, (int64_t)(L.us * o->steps * 64.0));
        forced_wait_error(a.err, st);
        launch_band(L.launch, a, o->variant == 1, st);
    }
}

}  // namespace qh
