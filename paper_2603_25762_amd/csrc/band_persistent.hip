// Persistent band solve (SNP graphs, FP32 dense graphs): planner and launch (the kernel is in
// band_persistent_kernel.h; the discrete variant's instantiations in
// band_persistent_discrete.hip, so that the two halves compile in parallel).
#include <algorithm>

#include "strip_persistent_kernel.h"

namespace qh {

int32_t force_wait_error = 0;

void forced_wait_error(int *err, hipStream_t st) {
    if (force_wait_error) QH_HIP(hipMemsetAsync(err, 1, sizeof(int), st));
}

int64_t exchange_limit = INT64_MAX;

void alloc_exchange(DevBuf<float> &xch, int64_t floats) {
    if (floats * 4 > exchange_limit) fail(QH_ENOMEM, "exchange buffers of %lld bytes", (long long)floats * 4);
    xch.alloc((size_t)floats);
}

void check_waits(int *err, hipStream_t st) {
    if (!download(err, 1, st)[0]) return;
    QH_HIP(hipMemsetAsync(err, 0, sizeof(int), st));
    QH_HIP(hipStreamSynchronize(st));
    fail(QH_EHIP, "one-launch bSB kernel: a neighbour wait exceeded its poll limit");
}

// Contiguous parts of the band blocks, as even as possible, with the rows each part holds, the
// blocks that reach past its own rows, the blocks its neighbours reach, and the neighbour range
// (made symmetric: "reads from" and "is read by" together).
BandSplit split_band(const int32_t *bb_lo, const int32_t *bb_w, int64_t n_bblk, int wpg) {
    BandSplit s;
    s.wpg = wpg;
    s.part.resize(wpg);
    std::vector<int32_t> owner(n_bblk);
    for (int w = 0; w < wpg; ++w) {
        const int32_t b0 = (int32_t)(n_bblk * w / wpg), b1 = (int32_t)(n_bblk * (w + 1) / wpg);
        BandJob &J = s.part[w];
        J = BandJob{};
        J.w = w;
        J.blk0 = b0;
        J.nblk = b1 - b0;
        s.max_blocks = std::max(s.max_blocks, b1 - b0);
        const int32_t own_lo = b0 * kBandRows, own_hi = b1 * kBandRows;
        J.xlo = own_lo;
        J.xhi = own_hi;
        J.in_a = 0;
        J.in_b = J.nblk;
        for (int32_t b = b0; b < b1; ++b) {
            owner[b] = w;
            const int32_t lo = bb_lo[b], hi = bb_lo[b] + bb_w[b];
            J.xlo = std::min(J.xlo, lo);
            J.xhi = std::max(J.xhi, hi);
            if (lo < own_lo) J.in_a = b - b0 + 1;                      // last block that reaches below
            if (hi > own_hi) J.in_b = std::min(J.in_b, b - b0);        // first block that reaches above
        }
        if (J.in_a >= J.in_b) J.in_a = J.in_b = 0;
        s.lds_rows = std::max<int64_t>(s.lds_rows, J.xhi - J.xlo);
    }
    for (int w = 0; w < wpg; ++w) {
        s.part[w].nbr0 = s.part[w].nbr1 = w;
        s.part[w].pub_a = 0;
        s.part[w].pub_b = s.part[w].nblk;
    }
    for (int w = 0; w < wpg; ++w) {
        BandJob &J = s.part[w];
        const int32_t o0 = owner[J.xlo / kBandRows], o1 = owner[(J.xhi - 1) / kBandRows];
        J.nbr0 = std::min(J.nbr0, o0);
        J.nbr1 = std::max(J.nbr1, o1);
        for (int v = o0; v <= o1; ++v) {
            if (v == w) continue;
            BandJob &V = s.part[v];
            V.nbr0 = std::min(V.nbr0, w);
            V.nbr1 = std::max(V.nbr1, w);
            // rows [xlo, own_lo) and [own_hi, xhi) of w lie in v: the top blocks of a lower
            // neighbour from row xlo on, the bottom blocks of an upper one up to row xhi
            if (v < w) V.pub_b = std::min(V.pub_b, std::max(0, J.xlo / kBandRows - V.blk0));
            else V.pub_a = std::max(V.pub_a, std::min(V.nblk, (J.xhi - 1) / kBandRows + 1 - V.blk0));
        }
    }
    return s;
}

// whole chunks of 16 columns that the kernel variant keeps in registers per block (strip)
int band_held_chunks(int dtype, int um, bool strips) {
    if (strips) return kSpRegs / um / sp_tile_regs(dtype) * (kTile / 16);
    return dtype == kBpTiles ? 32 / um : (dtype == QH_F32 ? 32 : 48) / um - 1;
}

// The 16-row strips of a dense graph as band blocks over whole tiles: their first column, width,
// the byte offset of their part of the first stored tile, and which tiles of the range are
// stored (a row tile without stored tiles: none, over its own rows).  False when a range is
// longer than a word has bits.
static bool strips_of(const qh_graph *g, std::vector<int64_t> &off, std::vector<int32_t> &lo, std::vector<int32_t> &w,
                      std::vector<uint64_t> &tiles, bool &gaps, hipStream_t st) {
    const auto tptr = download(g->t_ptr.p, g->n_rt + 1, st), tcol = download(g->t_col.p, g->n_tiles, st);
    const int64_t eb = dtype_bytes(g->dtype);
    for (int64_t rt = 0; rt < g->n_rt; ++rt) {
        const int32_t t0 = tptr[rt], t1 = tptr[rt + 1];
        const int32_t c0 = t1 > t0 ? tcol[t0] : (int32_t)rt, nt = t1 > t0 ? tcol[t1 - 1] - c0 + 1 : 1;
        if (nt > 64) return false;
        gaps |= nt != t1 - t0;                 // (a row tile without stored tiles multiplies its own rows by 0)
        uint64_t m = 0;
        for (int32_t t = t0; t < t1; ++t) m |= 1ull << (tcol[t] - c0);
        for (int s = 0; s < kTile / kBandRows; ++s) {
            off.push_back(((int64_t)t0 * kTileElems + s * (kTileElems / 4)) * eb);
            lo.push_back(c0 * kTile);
            w.push_back(nt * kTile);
            tiles.push_back(m);
        }
    }
    return true;
}

static int units_variant(int64_t blocks) {
    const int64_t u = ceil_div(blocks, kBpWaves);
    return u <= 1 ? 1 : u <= 2 ? 2 : u <= 4 ? 4 : u <= 8 ? 8 : 0;
}

// Estimated time of a step of one team, us: `blocks` band blocks (strips) per workgroup, `quads` of
// columns each, `past` chunks of 16 columns of a block read from memory.  Fitted to measured
// steps (f16, estimate / measured): 0.9 for a step's barriers and latencies; per band block of
// a SIMD 0.0195 per MFMA and 0.12; 1.8 for the exchange with neighbours; 0.25 per chunk read from
// memory.  2,001 SNPs, R = 128: 3.1 / 3.6; 7,768 SNPs, F32, 36 quads wide, R = 128: 5.7 / 5.3;
// 100,000 SNPs, R = 64: 12.4 / 11.3; 250,000: 27.7 / 26.7.
double band_step_us(double quads, double past, int64_t blocks, int wpg, int rt, bool strips) {
    const double units = std::max(1.0, (double)blocks / 4.0);      // per SIMD
    const double unit = strips ? quads / 16.0 * ((rt / 16) * 0.04 + 0.02) + 0.2 + past * 0.1
                               : quads * (rt / 16) * 0.0195 + 0.12 + past * 0.25;
    return 0.9 + units * unit + (wpg > 1 ? 1.8 : 0.0);
}

// Chooses replicas per group, workgroups per graph and the kernel variant for one graph by the
// estimated time of a step times the passes that the replica groups take.
// The per-step kernels take their state's traffic at 4.6 TB/s and a launch, or the latency of
// walking the band (2,001 SNPs 8.8, 7,768 SNPs 17.2, 250,000 56.6 measured); the plan has to
// beat that by a tenth.  Both sides are estimates, fitted to the shapes above and not timed on the
// graph.  Over 20 more shapes (SNP graphs of 60 to 50,000 SNPs in bands of 14 to 440 columns, read graphs of
// 60 to 12,000 reads, 16 to 2,048 replicas) plan 0 took from the same time as the per-step plans
// (8,000 F16 reads, R = 1,024) to a fifth of it (1,000 SNPs in bands of 440, R = 64).
bool build_band_plan(const qh_graph *g, SolvePlan &p, BandPersist &bp, hipStream_t st) {
    bp.ok = false;
    const int R = p.R;
    const bool tiles = g->storage == QH_STORE_DENSE;
    const int64_t nb = tiles ? g->n_rt * (kTile / kBandRows) : g->n_bblk;
    const bool strips = tiles && g->dtype != QH_F32;
    if (g->l_nnz > 0 || nb == 0 || g->n >= ((int64_t)1 << 26)) return false;
    int n_cu = 0, coop = 0;
    QH_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, g->device));
    QH_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, g->device));
    if (!coop || n_cu < 1) return false;
    const int dtype = strips ? g->dtype : tiles ? kBpTiles : g->bb_dtype;
    std::vector<int64_t> off;
    std::vector<int32_t> lo, wd;
    std::vector<uint64_t> tm;
    if (tiles) {
        bp.gaps = false;
        if (!strips_of(g, off, lo, wd, tm, bp.gaps, st)) return false;
    } else {
        lo = download(g->bb_lo.p, nb, st);
        wd = download(g->bb_w.p, nb, st);
    }
    double quads = 0.0;
    for (int32_t w : wd) quads += ceil_div(w, 4);
    quads /= (double)nb;
    struct Cand { double us; int rt, wpg, um, slots, passes; };
    std::vector<Cand> cands;
    for (int rt : {32, 16}) {
        if (R % rt) continue;
        const int ng = R / rt;
        for (int bpw = 1; bpw <= (strips ? 4 : 8) * kBpWaves; ++bpw) {
            const int wpg = (int)ceil_div(nb, bpw);
            if (wpg > n_cu || (bpw > 1 && (int)ceil_div(nb, bpw - 1) == wpg)) continue;
            const int um = units_variant(ceil_div(nb, wpg));
            const int held = band_held_chunks(dtype, um, strips);
            double past = 0.0;
            for (int32_t w : wd) past += std::max(0, w / 16 - held);
            const int slots = std::min(ng, n_cu / wpg), passes = (int)ceil_div(ng, slots);
            const double us = band_step_us(quads, past / nb, ceil_div(nb, wpg), wpg, rt, strips);
            cands.push_back({us * passes, rt, wpg, um, slots, passes});
        }
    }
    std::sort(cands.begin(), cands.end(), [](const Cand &a, const Cand &b) { return a.us < b.us; });
    const double state_us = (double)g->n * R * 16.0 / 4.6e6;
    double step_us;
    if (strips) step_us = std::max(4.5, 3.0 + quads / 16.0 * 0.2 + state_us);
    else if (tiles) step_us = std::max(4.0, 3.0 + quads * 0.1 + state_us);
    else step_us = std::max({4.0, 1.5 + quads * 0.43, 3.0 + state_us});
    for (const Cand &c : cands) {
        if (c.us > 0.9 * step_us) break;
        BandSplit s = split_band(lo.data(), wd.data(), nb, c.wpg);
        const int64_t lds = band_lds_bytes(s.lds_rows, c.rt, strips);
        if (lds > kBpLdsLimit || units_variant(s.max_blocks) != c.um) continue;
        BandLaunch &bl = bp.launch;
        bl = BandLaunch{};
        bl.rt = c.rt;
        bl.um = c.um;
        bl.grid = c.wpg * c.slots;
        bl.wpg = c.wpg;
        bl.dtype = dtype;
        bl.strips = strips;
        bl.lds_bytes = lds;
        const int64_t rows = nb * kBandRows;
        bl.xch_floats = c.wpg > 1 ? (int64_t)c.slots * 2 * rows * c.rt : 0;
        bl.n_flags = (int64_t)bl.grid * kBpWaves;
        bl.job_ptr.push_back(0);
        for (int sl = 0; sl < c.slots; ++sl)
            for (int w = 0; w < c.wpg; ++w) {
                for (int q = sl, k = 0; q < R / c.rt; q += c.slots, ++k) {
                    BandJob J = s.part[w];
                    J.team = 0;
                    J.r0 = q * c.rt;
                    J.t0 = k;
                    J.flag_off = sl * c.wpg * kBpWaves;
                    J.xch_rows = (int32_t)rows;
                    J.xch_off = (int64_t)sl * 2 * rows * c.rt;
                    bl.jobs.push_back(J);
                }
                bl.job_ptr.push_back((int32_t)bl.jobs.size());
            }
        alloc_exchange(bp.xch, bl.xch_floats);         // (the largest first: it may find no room)
        BandTeam T{};
        if (tiles) {
            bp.off.alloc(nb);
            bp.off.upload(off.data(), nb, st);
            bp.lo.alloc(nb);
            bp.lo.upload(lo.data(), nb, st);
            bp.w.alloc(nb);
            bp.w.upload(wd.data(), nb, st);
            bp.tiles.alloc(nb);
            bp.tiles.upload(tm.data(), nb, st);
        }
        T.bb_off = tiles ? bp.off.p : g->bb_off.p;
        T.bb_lo = tiles ? bp.lo.p : g->bb_lo.p;
        T.bb_w = tiles ? bp.w.p : g->bb_w.p;
        T.bb_val = tiles ? g->t_val.p : g->bb_val.p;
        T.scale = g->row_scale.p;
        T.tiles = bp.tiles.p;
        T.x = p.xa.p;
        T.y = p.y.p;
        T.bscale = tiles ? 1.0f : g->bb_scale;
        T.n = (int32_t)g->n;
        bp.passes = c.passes;
        // A cooperative launch that loads state and couplings starts 18 us (60 reads) to 50 us (250,000
        // SNPs) later than a per-step one; a step then saves 3 to 32 us.  us per range, per-step launches / one
        // launch, at 1, 4 and 8 steps: 2,001 SNPs, R = 64 34 / 58, 59 / 65, 106 / 78; 250,000 SNPs 197 / 244,
        // 365 / 312, 607 / 412; FP32, 8,000 reads, R = 64 39 / 62, 66 / 76, 110 / 95.  16- and 8-bit dense graphs
        // took a cooperative launch before: from two steps on.
        bp.min_steps = strips ? kBpMinSteps : tiles ? 8 : step_us >= 20.0 ? 3 : step_us >= 7.0 ? 4 : 6;
        bp.team.alloc(1);
        bp.team.upload(&T, 1, st);
        bp.jobs.alloc(bl.jobs.size());
        bp.jobs.upload(bl.jobs.data(), bl.jobs.size(), st);
        bp.job_ptr.alloc(bl.job_ptr.size());
        bp.job_ptr.upload(bl.job_ptr.data(), bl.job_ptr.size(), st);
        bp.flags.alloc((size_t)bl.n_flags + kBpFlagsPad);
        bp.failed.take();
        QH_HIP(hipStreamSynchronize(st));
        bp.ok = true;
        return true;
    }
    return false;
}

void launch_band_plain(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st) {
    launch_band_disc<false>(bl, a, st);
}

void launch_band(const BandLaunch &bl, const BandPersistArgs &a, int discrete, hipStream_t st) {
    if (bl.strips) {
        if (discrete) launch_strip_discrete(bl, a, st);
        else launch_strip_plain(bl, a, st);
    } else {
        if (discrete) launch_band_discrete(bl, a, st);
        else launch_band_plain(bl, a, st);
    }
}

}  // namespace qh
