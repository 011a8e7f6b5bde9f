// The persistent band kernel (SNP graphs, and FP32 dense read graphs): all steps of a solve inside
// one launch, the whole state and the couplings on chip.
//
// A workgroup owns consecutive band blocks (16 rows each) of one group of RT replicas.  Its x
// rows, and the neighbours' rows that its blocks reach, sit in LDS; its y and its couplings
// sit in VGPRs (a block's 16 x W couplings are W / 4 MFMA A operands, one 16-bit or 32-bit
// value per lane each).  A step is
//   1. blocks that read own rows only: z = J x (v_mfma_f32_16x16x4f32) and y,
//   2. wait for the neighbours' step, fetch their rows into LDS, the remaining blocks,
//   3. barrier; x and the walls for every block, in registers and LDS; the rows neighbours
//      read go out with device-coherent stores, then the wave's step flag.
// v_mfma_f32_16x16x4f32 adds its four products one by one, each with one rounding (checked on
// the device against a chain of FMAs, subnormal values included: identical bits), so a row's
// sum runs over its columns in the order of the per-step band kernels and the results are
// theirs bit for bit.
//
// What bounds it: the FP32 matrix rate (256 flop per cycle and CU), twice the vector FMA rate
// of the per-step kernel; memory is touched only by the halo rows.  Replica groups that do not
// fit the chip at once run one after another.
//
// Flags count steps.  A workgroup publishes step t into half t % 2 of the exchange buffer only
// after its neighbours' flags reached t, that is after they read half t % 2 for the last time;
// the neighbour lists are symmetric.  A launch runs at least two steps: a workgroup reads its
// neighbours' rows of the initial state from where they write their final one, and only the wait
// of a second step shows that the neighbours are past that read.  Waits are bounded: past
// max_polls a workgroup raises the error word, every wait then returns at its next 1,024th poll,
// and the final x is NaN; the host fails the call, or, where a call returns before its launch has
// ended, the next one on the graph.
#pragma once

#include "band_persistent.h"
#include "formats.h"

namespace qh {

typedef float bp_float4_t __attribute__((ext_vector_type(4)));

// LDS operations of the whole workgroup before it are visible after it (global stores may
// still be in flight).
__device__ inline void bp_barrier() {
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
}

// Tables and arrays are read through their address spaces: constant (scalar loads) for the job
// and graph tables, global for the state, so that pointers taken from a table neither make
// their addresses per-lane values nor turn accesses into flat ones.
#define QH_CONST __attribute__((address_space(4)))
#define QH_GLOBAL __attribute__((address_space(1)))

template <int NB>
struct BpVec {
    float v[NB];
};

template <int NB>
struct BpWord {
    typedef uint32_t type;
};
template <>
struct BpWord<2> {
    typedef uint64_t type;
};
// NB consecutive floats of global memory: plain, and to other workgroups (one device-coherent access)
template <int NB>
__device__ inline BpVec<NB> bp_global(const float *p) {
    typedef typename BpWord<NB>::type word;
    const word u = *(const QH_GLOBAL word *)p;
    BpVec<NB> r;
    __builtin_memcpy(&r, &u, sizeof(u));
    return r;
}
template <int NB>
__device__ inline void bp_global_store(float *p, const BpVec<NB> &r) {
    typedef typename BpWord<NB>::type word;
    word u;
    __builtin_memcpy(&u, &r, sizeof(u));
    *(QH_GLOBAL word *)p = u;
}
template <int NB>
__device__ inline void bp_store(float *p, const BpVec<NB> &r) {
    typedef typename BpWord<NB>::type word;
    word u;
    __builtin_memcpy(&u, &r, sizeof(u));
    __hip_atomic_store((QH_GLOBAL word *)p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int bp_flag(const int *p) {
    return __hip_atomic_load((const QH_GLOBAL int *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int NB>
__device__ inline BpVec<NB> bp_lds(const float *p) {
    BpVec<NB> r;
    __builtin_memcpy(&r, __builtin_assume_aligned(p, 4 * NB), 4 * NB);
    return r;
}
template <int NB>
__device__ inline void bp_lds_store(float *p, const BpVec<NB> &r) {
    __builtin_memcpy(__builtin_assume_aligned(p, 4 * NB), &r, 4 * NB);
}

// Every wave of neighbours [nbr0, nbr1] (but w itself) has published step t - 1, or a wait gave up.
__device__ inline void bp_wait(const BandPersistArgs &a, const int *flags, int nbr0, int nbr1, int w, int t, int lane) {
    const int f0 = nbr0 * kBpWaves, nf = (nbr1 + 1) * kBpWaves - f0;
    int64_t polls = 0;
    for (int f = lane; f - lane < nf; f += 64) {
        while (true) {
            const bool late = f < nf && f / kBpWaves + nbr0 != w && bp_flag(flags + f0 + f) < t;
            if (!__any(late)) break;
            if ((++polls & 1023) == 0 && (polls > a.max_polls || bp_flag(a.err) != 0)) {
                __hip_atomic_fetch_or(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
}

// Neighbours' rows -> LDS: bytes [0, lo_end) and [hi, end) of src to the same offsets of dst, all
// loads in flight at once (device-coherent, straight into LDS; the waves take 1 KB each in turn).
// With the loads through registers, 4 or 8 per thread at a time, a fetch took a memory round trip
// per 16 to 32 KB.  Before / now: 8,000 reads (BF16, R = 256), 2,000 steps 8.3 / 7.85 ms; 1,501 reads
// (F32, R = 64), 250 steps 0.97 / 0.86 ms; a step of 1,500 FP8 read blocks of 50-5,000 689 / 642 us.
__device__ inline void bp_fetch(void *dst, const void *src, int lo_end, int hi, int end, int wave, int lane) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, end, 0x00027000);
    constexpr int kCoherent = 16;                  // sc1: as the loads of device scope
    auto piece = [&](int at, int to) {
        if (at + lane * 16 < to)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)((char *)dst + at), 16,
                                                     lane * 16, at, 0, kCoherent);
    };
    int at = wave * 1024;
    for (; at < lo_end; at += kBpWaves * 1024) piece(at, lo_end);
    // the first piece past the low range goes to the wave whose turn it is
    for (at += hi - (lo_end + 1023) / 1024 * 1024; at < end; at += kBpWaves * 1024) piece(at, end);
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// couplings of one chunk of 16 columns: four MFMA A operands (quads of four columns), two per
// register in 16-bit types
template <int DT>
struct BpChunk {
    static constexpr int kRegs = DT == QH_F32 || DT == kBpTiles ? 4 : 2;
};
template <int DT>
__device__ inline float bp_a(const uint32_t *j, int k) {   // quad k of a chunk, widened exactly
    if constexpr (DT == QH_F32 || DT == kBpTiles) return __uint_as_float(j[k]);
    else if constexpr (DT == QH_F16) return f16_bits_to_f32((uint16_t)(k & 1 ? j[k >> 1] >> 16 : j[k >> 1]));
    else return __uint_as_float(k & 1 ? j[k >> 1] & 0xffff0000u : j[k >> 1] << 16);
}
// A block's couplings as a buffer of W columns: loads past its end return 0, so columns past W
// need no test and no read ever leaves the block.
typedef __amdgpu_buffer_rsrc_t bp_rsrc_t;
template <int DT>
__device__ inline bp_rsrc_t bp_block(const uint8_t *val, const int64_t *bb_off, int blk, int W) {
    constexpr int EB = DT == QH_F32 ? 4 : 2;
    const int64_t off = ((const QH_CONST int64_t *)bb_off)[blk];
    // raw dword buffer of gfx9: stride 0, 32-bit data format
    return __builtin_amdgcn_make_buffer_rsrc((void *)(val + off * EB), 0, W * kBandRows * EB, 0x00027000);
}
// A strip's parts of its stored tiles (tile_bytes apart, part_bytes each) as a buffer; an empty
// one when there are none.  bp_tile_off: byte offset of tile c of the strip's range, past the
// buffer's end, where loads return 0, when that tile is not stored.
__device__ inline bp_rsrc_t bp_strip(const uint8_t *val, int64_t off, uint64_t tiles, int tile_bytes, int part_bytes) {
    const int nt = __builtin_popcountll(tiles);
    return __builtin_amdgcn_make_buffer_rsrc((void *)(val + (nt ? off : 0)), 0,
                                             nt ? (nt - 1) * tile_bytes + part_bytes : 0, 0x00027000);
}
__device__ inline int bp_tile_off(uint64_t tiles, int c, int tile_bytes) {
    return (tiles >> c & 1 ? __builtin_popcountll(tiles & ((1ull << c) - 1)) : 64) * tile_bytes;
}
// chunk c of a block: lane l holds row l % 16 of column l / 16 of each quad, which is element l
// of the quad's 64
template <int DT>
__device__ inline void bp_load_chunk(uint32_t *j, bp_rsrc_t blk, int c, int lane, uint64_t tiles = 0) {
    if constexpr (DT == kBpTiles) {
        // a strip's part of a tile: four chunks, each lane's four quads together
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(
            blk, lane * 16 + bp_tile_off(tiles, c >> 2, kTileElems * 4) + (c & 3) * 1024, 0, 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) j[k] = v[k];
    } else if constexpr (DT == QH_F32) {
#pragma unroll
        for (int k = 0; k < 4; ++k) j[k] = __builtin_amdgcn_raw_buffer_load_b32(blk, lane * 4 + (c * 4 + k) * 256, 0, 0);
    } else {
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            v[k] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(blk, lane * 2 + (c * 4 + k) * 128, 0, 0);
        j[0] = v[0] | v[1] << 16;
        j[1] = v[2] | v[3] << 16;
    }
}

// RT = 16 NB replicas per group; lane l holds rows 4 (l / 16) .. + 3 of a block and replicas
// NB (l % 16) .. + NB - 1 of the group, so that a quad's B operands (four x rows) are one
// contiguous LDS read of 4 NB bytes per lane.
// UM band blocks per wave, kRegs registers of couplings shared out among them; columns past
// what the registers hold are read from memory each step.
template <int DT, int NB, int UM, bool DISC>
__global__ __launch_bounds__(kBpThreads, 2) void k_band_persistent(BandPersistArgs a) {
    extern __shared__ __attribute__((aligned(16))) float bp_x[];
    constexpr int RT = 16 * NB;
    constexpr int CR = BpChunk<DT>::kRegs;
    constexpr int kRegs = CR == 4 ? 128 : 96;
    constexpr bool kWhole = DT == kBpTiles;        // blocks end with a whole chunk
    // whole chunks of 16 columns held per block (and the last, partial one)
    constexpr int MAXC = kRegs / UM / CR - (kWhole ? 0 : 1);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;
    const int64_t R = a.R;
    const int steps = a.ke - a.kb;

    const int job_end = ((const QH_CONST int32_t *)a.job_ptr)[blockIdx.x + 1];
    for (int jb = ((const QH_CONST int32_t *)a.job_ptr)[blockIdx.x]; jb < job_end; ++jb) {
        const QH_CONST BandJob &J = *(const QH_CONST BandJob *)(a.jobs + jb);
        const QH_CONST BandTeam &T = *(const QH_CONST BandTeam *)(a.teams + J.team);
        const float c0 = a.single ? a.c0 : T.c0;
        const float *field = a.single ? a.field : T.field;
        const float bscale = T.bscale;
        const int n = T.n, r0 = J.r0, xlo = J.xlo, nblk = J.nblk;
        const int n_in = J.in_b - J.in_a;
        const bool has_nbr = J.nbr1 > J.nbr0;
        // units [0, ih) of every wave need own rows only
        const int ih = has_nbr ? n_in / kBpWaves : UM;
        // x rows -> LDS (rows past n and the read-ahead rows hold 0)
        bp_barrier();                              // the previous job's last LDS reads are done
        for (int e = tid; e < (J.xhi - xlo + kBpPadRows) * 16; e += kBpThreads) {
            const int row = xlo + (e >> 4);
            BpVec<NB> v{};
            if (row < J.xhi && row < n) v = bp_global<NB>(T.x + (int64_t)row * R + r0 + (e & 15) * NB);
            bp_lds_store<NB>(bp_x + e * NB, v);
        }
        // units of this wave: position i * kBpWaves + wave, blocks with own rows only first
        uint32_t uo[UM];                           // LDS rows of the unit's first column (low half) and own first row
        int uw[UM];                                // columns (0: no unit)
        int upub = 0;                              // bit i: neighbours read unit i's rows
        uint32_t jr[UM][kRegs / UM];
        BpVec<NB> ys[UM][4];
#pragma unroll
        for (int i = 0; i < UM; ++i) {
            const int p = i * kBpWaves + wave;
            const int q = p - n_in;
            const int rel = p < n_in ? J.in_a + p : (q < J.in_a ? q : J.in_b + (q - J.in_a));
            const bool live = p < nblk;
            const int blk = J.blk0 + (live ? rel : 0);
            const int L = ((const QH_CONST int32_t *)T.bb_lo)[blk];
            const int Wb = ((const QH_CONST int32_t *)T.bb_w)[blk];
            const int W = live ? Wb : 0;
            uw[i] = W;
            uo[i] = (uint32_t)(L - xlo) | (uint32_t)(blk * kBandRows - xlo) << 16;
            if (live && (rel < J.pub_a || rel >= J.pub_b)) upub |= 1 << i;
            const uint64_t tiles = kWhole && live ? ((const QH_CONST uint64_t *)T.tiles)[blk] : 0;
            const bp_rsrc_t rsrc = kWhole ? bp_strip(T.bb_val, ((const QH_CONST int64_t *)T.bb_off)[blk], tiles,
                                                     kTileElems * 4, kTileElems)
                                          : bp_block<DT>(T.bb_val, T.bb_off, blk, W);
#pragma unroll
            for (int c = 0; c < kRegs / UM / CR; ++c) {
                bp_load_chunk<DT>(&jr[i][c * CR], rsrc, c < MAXC ? c : W >> 4, lane, tiles);
                if (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (bounds the loads in flight, and their registers)
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int u = blk * kBandRows + 4 * g4 + k;
                ys[i][k] = BpVec<NB>{};
                if (live && u < n) ys[i][k] = bp_global<NB>(T.y + (int64_t)u * R + r0 + l16 * NB);
            }
        }
        float *xch = a.xch + J.xch_off;
        const int64_t half = (int64_t)J.xch_rows * RT;
        int *flags = a.flags + J.flag_off;
        const int t0 = J.t0 * steps;
        bp_barrier();

        float pump = ((const QH_CONST float *)a.pump)[a.kb];
        for (int s = 0; s < steps; ++s) {
            const int t = t0 + s;
            const float coef = a.a0 - pump;
#pragma unroll 1
            for (int ph = 0; ph < 2; ++ph) {
                if (ph == 1 && has_nbr) {
                    // the neighbours' step t - 1 is published: their rows -> LDS
                    bp_wait(a, flags, J.nbr0, J.nbr1, J.w, t, lane);
                    if (s > 0) {                   // (the first step's rows came with the initial state)
                        const int own = (J.blk0 * kBandRows - xlo) * RT * 4;
                        bp_fetch(bp_x, xch + ((t - 1) & 1) * half + (int64_t)xlo * RT, own, own + nblk * kBandRows * RT * 4,
                                 (J.xhi - xlo) * RT * 4, wave, lane);
                    }
                    bp_barrier();
                }
                // The couplings, widths and rows do not change from step to step: without this the
                // compiler widens the couplings and builds masks, conditions and addresses once,
                // ahead of the step loop, and spills them.
#pragma unroll
                for (int i = 0; i < UM; ++i) {
                    __asm__ volatile("" : "+s"(uw[i]), "+s"(uo[i]));
#pragma unroll
                    for (int c = 0; c < kRegs / UM; ++c) __asm__ volatile("" : "+v"(jr[i][c]));
                }
                // x rows of chunk c of unit i
                auto read4 = [&](BpVec<NB> (&bv)[4], int i, int c) {
                    const float *xb = bp_x + (uo[i] & 0xffff) * RT + lane * NB;
#pragma unroll
                    for (int k = 0; k < 4; ++k) bv[k] = bp_lds<NB>(xb + (c * 4 + k) * 4 * RT);
                };
                // each chunk's x rows are read while the previous chunk multiplies, a unit's first
                // ones under the end of the unit before (they may not be read before phase 1 starts
                // when the unit belongs to it)
                BpVec<NB> first[4];
                read4(first, 0, 0);
#pragma unroll
                for (int i = 0; i < UM; ++i) {
                    const int W = uw[i];
                    if (W != 0 && (i < ih) == (ph == 0)) {
                        const int orow = uo[i] >> 16;      // LDS row of the unit's first own row
                        bp_float4_t acc[NB];
#pragma unroll
                        for (int b = 0; b < NB; ++b) acc[b] = bp_float4_t{0.f, 0.f, 0.f, 0.f};
                        const int nf = W >> 4;             // whole chunks
                        auto mfma4 = [&](const uint32_t *j, const BpVec<NB> (&bv)[4], bool in0, bool in1, bool in2,
                                         bool in3) {
                            const bool in[4] = {in0, in1, in2, in3};
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const float av = bp_a<DT>(j, k);
#pragma unroll
                                for (int b = 0; b < NB; ++b) {
                                    float xv = bv[k].v[b];
                                    if constexpr (DISC) xv = xv >= 0.f ? 1.f : -1.f;
                                    xv = in[k] ? xv : 0.f;
                                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, xv, acc[b], 0, 0, 0);
                                }
                            }
                        };
                        if (i == ih && i > 0) read4(first, i, 0);
                        const float *xop = bp_x + (orow + 4 * g4) * RT + l16 * NB;
                        BpVec<NB> xo[4], last[4];          // the unit's own x; x rows of the last chunk
#pragma unroll
                        for (int k = 0; k < 4; ++k) xo[k] = bp_lds<NB>(xop + k * RT);
                        if constexpr (!kWhole) read4(last, i, nf);
                        BpVec<NB> bv[2][4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) bv[0][k] = first[k];
                        // whole chunks: one-sided branches only (with an else for the chunk that ends the
                        // block the accumulators were copied at every chunk, each copy waiting for the
                        // matrix pipeline to drain)
#pragma unroll
                        for (int c = 0; c < MAXC; ++c) {
                            if (c < nf) {
                                if (c + 1 < MAXC) read4(bv[(c + 1) & 1], i, c + 1);
                                mfma4(&jr[i][c * CR], bv[c & 1], true, true, true, true);
                            }
                        }
                        if (MAXC < nf) {                   // those past the register-held ones
                            const int blk = (orow + xlo) / kBandRows;
                            const uint64_t tiles = kWhole ? ((const QH_CONST uint64_t *)T.tiles)[blk] : 0;
                            const bp_rsrc_t rsrc = kWhole ? bp_strip(T.bb_val, ((const QH_CONST int64_t *)T.bb_off)[blk],
                                                                     tiles, kTileElems * 4, kTileElems)
                                                          : bp_block<DT>(T.bb_val, T.bb_off, blk, W);
#pragma unroll 1
                            for (int c = MAXC; c < nf; ++c) {
                                uint32_t jt[CR];
                                BpVec<NB> bt[4];
                                bp_load_chunk<DT>(jt, rsrc, c, lane, tiles);
                                read4(bt, i, c);
                                mfma4(jt, bt, true, true, true, true);
                            }
                        }
                        // the last chunk: columns past W multiply their couplings, 0, by 0 and not by
                        // whatever those rows of x hold; quads past W are left out (one in twelve to one
                        // in four for blocks of 44 to 48 columns; 250,000 SNPs 27.7 -> 25.9 us)
                        if constexpr (!kWhole) {
                            const int Wl = W - 16 * nf - g4;   // columns of this lane's quad slots below W
                            const int Wu = W - 16 * nf;
                            auto mfma1 = [&](int k) {
                                const float av = bp_a<DT>(&jr[i][MAXC * CR], k);
#pragma unroll
                                for (int b = 0; b < NB; ++b) {
                                    float xv = last[k].v[b];
                                    if constexpr (DISC) xv = xv >= 0.f ? 1.f : -1.f;
                                    xv = 4 * k < Wl ? xv : 0.f;
                                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, xv, acc[b], 0, 0, 0);
                                }
                            };
                            if (0 < Wu) mfma1(0);
                            if (4 < Wu) mfma1(1);
                            if (8 < Wu) mfma1(2);
                            if (12 < Wu) mfma1(3);
                        }
                        if (i + 1 < UM) read4(first, i + 1, 0);
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int k = 0; k < 4; ++k) acc[b][k] *= bscale;   // exact: a power of two
                        if (field) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const int u = orow + xlo + 4 * g4 + k;
                                const float h = u < n ? ((const QH_GLOBAL float *)field)[u] : 0.f;
#pragma unroll
                                for (int b = 0; b < NB; ++b) acc[b][k] += h;
                            }
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int b = 0; b < NB; ++b)
                                ys[i][k].v[b] = ys[i][k].v[b] + (-coef * xo[k].v[b] + c0 * acc[b][k]) * a.dt;
                    }
                }
            }
            bp_barrier();                          // every wave is past its reads of x
#pragma unroll
            for (int i = 0; i < UM; ++i) __asm__ volatile("" : "+s"(uw[i]), "+s"(uo[i]));
            // x and the walls, two units at a time (all of their x rows read first); a wave's units
            // without rows (uw = 0) sit past its last one
#pragma unroll
            for (int i = 0; i < UM; i += 2) {
                if (uw[i] != 0) {
                    constexpr int P = UM > 1 ? 2 : 1;
                    BpVec<NB> xv[P][4];
                    float *xp[P];
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        xp[p] = bp_x + ((uo[i + p] >> 16) + 4 * g4) * RT + l16 * NB;
#pragma unroll
                        for (int k = 0; k < 4; ++k) xv[p][k] = bp_lds<NB>(xp[p] + k * RT);
                    }
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        if (p == 0 || uw[i + p] != 0) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
#pragma unroll
                                for (int b = 0; b < NB; ++b) {
                                    const float yn = ys[i + p][k].v[b];
                                    const float xn = xv[p][k].v[b] + a.a0 * yn * a.dt;
                                    ys[i + p][k].v[b] = fabsf(xn) > 1.0f ? 0.0f : yn;
                                    xv[p][k].v[b] = __builtin_amdgcn_fmed3f(xn, -1.0f, 1.0f);
                                }
                                bp_lds_store<NB>(xp[p] + k * RT, xv[p][k]);
                            }
                        }
                    }
                }
            }
            pump = ((const QH_CONST float *)a.pump)[min(a.kb + s + 1, a.ke - 1)];
            if (has_nbr && upub) {
                // rows that neighbours read (this wave's own LDS rows, just written)
                float *dst = xch + (t & 1) * half + (int64_t)(xlo + 4 * g4) * RT + l16 * NB;
#pragma unroll
                for (int i = 0; i < UM; ++i) {
                    if (upub >> i & 1) {
                        const int orow = uo[i] >> 16;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            bp_store<NB>(dst + (orow + k) * RT,
                                         bp_lds<NB>(bp_x + (orow + 4 * g4 + k) * RT + l16 * NB));
                    }
                }
            }
            bp_barrier();
            if (has_nbr) {
                __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (lane == 0)
                    __hip_atomic_store((QH_GLOBAL int *)(flags + J.w * kBpWaves + wave), t + 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        // final state -> memory (NaN when a wait gave up)
        const bool bad = has_nbr && bp_flag(a.err) != 0;
#pragma unroll
        for (int i = 0; i < UM; ++i) {
            if (uw[i] != 0) {
                const int orow = uo[i] >> 16;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int u = orow + xlo + 4 * g4 + k;
                    if (u < n) {
                        BpVec<NB> xv = bp_lds<NB>(bp_x + (u - xlo) * RT + l16 * NB);
#pragma unroll
                        for (int b = 0; b < NB; ++b) xv.v[b] = bad ? __builtin_nanf("") : xv.v[b];
                        bp_global_store<NB>(T.x + (int64_t)u * R + r0 + l16 * NB, xv);
                        bp_global_store<NB>(T.y + (int64_t)u * R + r0 + l16 * NB, ys[i][k]);
                    }
                }
            }
        }
    }
}

template <int DT, int NB, int UM, bool DISC>
static void launch_band_t(const BandLaunch &bl, const BandPersistArgs &args, hipStream_t st) {
    auto fn = k_band_persistent<DT, NB, UM, DISC>;
    if (hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bl.lds_bytes) !=
        hipSuccess)
        (void)hipGetLastError();
    BandPersistArgs a = args;
    void *kargs[] = {&a};
    QH_HIP(hipLaunchCooperativeKernel((const void *)fn, dim3((unsigned)bl.grid), dim3(kBpThreads), kargs,
                                      (unsigned)bl.lds_bytes, st));
}

template <bool DISC>
static void launch_band_disc(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st) {
#define QH_BP_U(DTV, NBV)                                              \
    do {                                                               \
        if (bl.um == 1) launch_band_t<DTV, NBV, 1, DISC>(bl, a, st);      \
        else if (bl.um == 2) launch_band_t<DTV, NBV, 2, DISC>(bl, a, st); \
        else if (bl.um == 4) launch_band_t<DTV, NBV, 4, DISC>(bl, a, st); \
        else launch_band_t<DTV, NBV, 8, DISC>(bl, a, st);                 \
    } while (0)
#define QH_BP(DTV)                        \
    do {                                  \
        if (bl.rt == 16) QH_BP_U(DTV, 1); \
        else QH_BP_U(DTV, 2);             \
    } while (0)
    switch (bl.dtype) {
        case QH_F32: QH_BP(QH_F32); break;
        case QH_F16: QH_BP(QH_F16); break;
        case QH_BF16: QH_BP(QH_BF16); break;
        case kBpTiles: QH_BP(kBpTiles); break;
        default: fail(QH_EUNSUPPORTED, "dtype not offered on skyline storage");
    }
#undef QH_BP
#undef QH_BP_U
}

}  // namespace qh
