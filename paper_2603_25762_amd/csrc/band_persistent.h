// Persistent band solve (all steps in one cooperative launch): tables shared by
// the host planner, the single-graph solve and the batched solve.
#pragma once

#include "internal.h"

namespace qh {

constexpr int kBpWaves = 8;                  // waves per workgroup (two per SIMD)
constexpr int kBpThreads = 64 * kBpWaves;
constexpr int kBpMinSteps = 2;               // steps of a launch, at least
constexpr int kBpPadRows = 32;               // LDS rows past the last held row (read-ahead, never used)

// DT values of the band kernel: a storage type of band blocks, or the FP32 tiles of a dense graph,
// whose 16-row strips are band blocks over whole tiles
constexpr int kBpTiles = 100;

// One graph of a launch.
struct BandTeam {
    const int64_t *bb_off;
    const int32_t *bb_lo, *bb_w;
    const uint8_t *bb_val;
    float *x, *y;               // [n][R] state, in and out
    const float *field;         // deformation field h [n] (nullptr: none)
    const float *scale;         // FP8 tiles: row scales
    const uint64_t *tiles;      // dense graphs: bit c of a strip's word is set when tile c of its range is stored
    float c0, bscale;
    int32_t n;
};

// One workgroup's share of one replica group of one graph.
struct BandJob {
    int32_t team;
    int32_t r0;                 // first replica
    int32_t blk0, nblk;         // band blocks [blk0, blk0 + nblk) of kBandRows rows
    int32_t in_a, in_b;         // blocks blk0 + [in_a, in_b) read own rows only; the others need neighbours' rows
    int32_t pub_a, pub_b;       // blocks blk0 + [0, pub_a) and blk0 + [pub_b, nblk) are read by neighbours
    int32_t xlo, xhi;           // rows held in LDS: [xlo, xhi), own rows included
    int32_t w, nbr0, nbr1;      // index in the team; neighbours [nbr0, nbr1] (inclusive, self among them)
    int32_t t0;                 // earlier jobs of the same team flags (each counts one call's steps)
    int32_t flag_off;           // team's flags: [workgroup][wave] step counters
    int32_t xch_rows;           // rows of one half of the team's exchange buffer
    int64_t xch_off;            // floats; two halves of [xch_rows][RT]
};

struct BandPersistArgs {
    int32_t R, kb, ke;
    float dt, a0;
    const float *pump;
    const BandTeam *teams;
    const BandJob *jobs;
    const int32_t *job_ptr;     // [grid + 1]
    float *xch;
    int *flags, *err;
    int64_t max_polls;
    // single-graph solves: this call's c0 and field in place of the team's (single = 1)
    int32_t single;
    float c0;
    const float *field;
};

// Host description of a launch: the jobs of every workgroup.
struct BandLaunch {
    int rt = 0;                 // replicas per group (16 or 32)
    int um = 0;                 // band blocks per wave (kernel variant: 1, 2, 4 or 8)
    int grid = 0;
    int wpg = 0;                // workgroups per replica group (single-graph launches)
    int dtype = 0;
    bool strips = false;        // the strip kernel (16/8-bit dense graphs), else the band kernel
    int64_t lds_bytes = 0, xch_floats = 0, n_flags = 0;
    std::vector<BandJob> jobs;  // in launch order of each workgroup (job_ptr)
    std::vector<int32_t> job_ptr;
};

// Partition of one graph's band blocks over `wpg` workgroups.
struct BandSplit {
    int wpg = 0, max_blocks = 0;
    int64_t lds_rows = 0;       // most rows a workgroup holds (without the read-ahead rows)
    std::vector<BandJob> part;  // geometry fields of each workgroup's job
};

// Plan of one graph and replica count (device tables built once).
struct BandPersist {
    bool ok = false;
    BandLaunch launch;
    int passes = 0;             // most jobs of one workgroup
    int min_steps = 0;          // a shorter range is faster in per-step launches
    bool gaps = false;          // dense graphs: some row tile's stored tiles are none, or not consecutive
    DevBuf<BandTeam> team;
    DevBuf<int64_t> off;        // dense graphs: the strips as band blocks
    DevBuf<int32_t> lo, w;
    DevBuf<uint64_t> tiles;
    DevBuf<BandJob> jobs;
    DevBuf<int32_t> job_ptr;
    DevBuf<float> xch;
    DevBuf<int> flags;          // n_flags counters, then the error word
    HostWord failed;            // readout = 0: set by the stream when a wait gave up
    bool fresh = true;          // the error word has not been cleared yet
};
// Polls of a neighbour's flag before a wait gives up.
constexpr int64_t kWaitPolls = (int64_t)1 << 27;
// Set by tests: every launch finds the error word set, as by a wait that gave up.
extern int32_t force_wait_error;
void forced_wait_error(int *err, hipStream_t st);
// Most bytes of exchange buffers (tests lower it).
extern int64_t exchange_limit;
void alloc_exchange(DevBuf<float> &xch, int64_t floats);
constexpr int64_t kBpErr = 32, kBpFlagsPad = 64;       // the error word's place past the flags
// Fails with EHIP when the error word of launches that have ended is set, and clears it.
void check_waits(int *err, hipStream_t st);

constexpr int64_t kBpLdsLimit = 160 * 1024;
constexpr int kSpPadRows = kTile;   // strip kernel: LDS rows past the last held row (read-ahead, never used)
// LDS of a workgroup that holds `rows` rows of rt replicas
inline int64_t band_lds_bytes(int64_t rows, int rt, bool strips) {
    return strips ? (rows + kSpPadRows) * rt * 2 : (rows + kBpPadRows) * rt * 4;
}
int band_held_chunks(int dtype, int um, bool strips);
double band_step_us(double quads, double past, int64_t blocks, int wpg, int rt, bool strips);

BandSplit split_band(const int32_t *bb_lo, const int32_t *bb_w, int64_t n_bblk, int wpg);
bool build_band_plan(const qh_graph *g, SolvePlan &p, BandPersist &bp, hipStream_t st);
// The blocks of a batch that run as teams of the persistent kernels, and their launches.
struct BatchTeams {
    struct Launch {
        BandLaunch launch;      // (jobs and job_ptr unused: the tables below)
        int64_t ptr_at = 0;     // its workgroups' pointers in ptr
        double us = 0.0;        // estimated time of a step of all its teams
    };
    std::vector<char> in;       // blocks
    std::vector<Launch> launches;
    DevBuf<int32_t> geo, ptr;
    DevBuf<int64_t> off;
    DevBuf<uint64_t> tiles;
    DevBuf<BandTeam> teams;
    DevBuf<BandJob> jobs;
    DevBuf<float> xch;
    DevBuf<int> flags;          // n_flags counters, then the error word
    int64_t n_flags = 0;
};
void plan_batch_teams(const qh_graph *const *gs, const std::vector<SolvePlan *> &plans,
                      const std::vector<BlockDesc> &desc, const qh_bsb_opts *o, BatchTeams &bt, hipStream_t st);
void run_batch_teams(BatchTeams &bt, const qh_bsb_opts *o, double a0, const float *pump, hipStream_t st);

void launch_band(const BandLaunch &bl, const BandPersistArgs &a, int discrete, hipStream_t st);
void launch_band_plain(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st);
void launch_band_discrete(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st);
void launch_strip_plain(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st);
void launch_strip_discrete(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st);

}  // namespace qh
