// The persistent strip kernel (dense read graphs in 16- and 8-bit storage): all steps of a solve
// inside one launch, state and couplings on chip.
//
// The tables, the exchange and the step are those of the band kernel (band_persistent_kernel.h)
// with the 16-row strips of the row tiles in place of band blocks: a strip's parts of its stored
// tiles (MFMA A fragments) and its x and y sit in VGPRs for the whole solve, the 16-bit copy of
// x that the product multiplies in LDS, own rows and the neighbours' rows that the strips reach.
// The MFMAs of a strip run in the order of the per-step kernel (tile, column half), so the
// results are its results bit for bit.  A tile that is not stored inside a strip's range
// multiplies by couplings of 0, which adds exactly 0 to a sum that starts at +0 as long as x is
// finite; the solver takes the per-step kernels where it might not be (a state or field of the
// caller's).  Testing for it here instead cost 10-15 % (a branch per tile).
//
// What bounds it: the exchange and the barriers of a step (about 2.5 us), LDS reads of the copy
// behind them (2 KB per tile, strip and 16 replicas).  The tile-staging persistent kernel
// (persistent_kernel.h) moves every neighbour's column tile whole and re-reads J from LDS each
// step.
#pragma once

#include "band_persistent_kernel.h"

namespace qh {

typedef _Float16 sp_half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 sp_bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kSpRegs = 128;        // registers of couplings per lane

// registers per stored tile of a strip (two fragments)
__host__ __device__ constexpr int sp_tile_regs(int dt) { return dt == QH_FP8_ROWSCALE ? 4 : 8; }

// fragment kb of tile c, widened to the MFMA type
template <int DT>
__device__ inline sp_half8_t sp_frag(const uint32_t *j, int kb) {
    if constexpr (DT == QH_FP8_ROWSCALE) {
        return e4m3x8_to_f16_scaled(make_uint2(j[2 * kb], j[2 * kb + 1]));
    } else {
        sp_half8_t r;
        __builtin_memcpy(&r, j + 4 * kb, 16);
        return r;
    }
}
template <int DT>
__device__ inline void sp_load_tile(uint32_t *j, bp_rsrc_t strip, int c, int lane, uint64_t tiles) {
    constexpr int EB = DT == QH_FP8_ROWSCALE ? 1 : 2;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int o = bp_tile_off(tiles, c, kTileElems * EB) + kb * 512 * EB + lane * 8 * EB;
        if constexpr (EB == 1) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(strip, o, 0, 0);
            j[2 * kb] = v[0];
            j[2 * kb + 1] = v[1];
        } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(strip, o, 0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) j[4 * kb + k] = v[k];
        }
    }
}
template <int DT, bool DISC>
__device__ inline uint16_t sp_copy(float x) {
    const float v = DISC ? (x >= 0.f ? 1.f : -1.f) : x;
    return DT == QH_BF16 ? f32_to_bf16_rne(v) : f32_to_f16_rne(v);
}

// RT = 16 NB replicas per group; lane l holds rows 4 (l / 16) .. + 3 of a strip and replicas
// 16 b + l % 16 of the group.  The copy of x is laid out [row / 8][RT][8], the B operand order.
// UM strips per wave; tiles past what the registers hold are read from memory each step.
template <int DT, int NB, int UM, bool DISC>
__global__ __launch_bounds__(kBpThreads, 2) void k_strip_persistent(BandPersistArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint16_t sp_x[];
    constexpr int RT = 16 * NB;
    constexpr int EB = DT == QH_FP8_ROWSCALE ? 1 : 2;
    constexpr int CR = sp_tile_regs(DT);
    constexpr int MAXT = kSpRegs / UM / CR;        // stored tiles held per strip
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
        const int n = T.n, r0 = J.r0, xlo = J.xlo, nblk = J.nblk;
        const int n_in = J.in_b - J.in_a;
        const bool has_nbr = J.nbr1 > J.nbr0;
        // units [0, ih) of every wave need own rows only
        const int ih = has_nbr ? n_in / kBpWaves : UM;
        // the copy of x -> LDS (rows past n and the read-ahead rows hold 0)
        bp_barrier();                              // the previous job's last LDS reads are done
        for (int e = tid; e < (J.xhi - xlo + kSpPadRows) / 8 * RT; e += kBpThreads) {
            const int row = xlo + e / RT * 8;
            uint16_t h[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                h[k] = 0;
                if (row + k < n && row + k < J.xhi)
                    h[k] = sp_copy<DT, DISC>(((const QH_GLOBAL float *)T.x)[(int64_t)(row + k) * R + r0 + e % RT]);
            }
            __builtin_memcpy(__builtin_assume_aligned(sp_x + e * 8, 16), h, 16);
        }
        // units of this wave: position i * kBpWaves + wave, strips with own rows only first
        uint32_t uo[UM];                           // LDS rows of the unit's first column (low half) and own first row
        int ut[UM];                                // tiles of the unit's range, -1: no unit
        int upub = 0;                              // bit i: neighbours read unit i's rows
        uint32_t jr[UM][kSpRegs / UM];
        float xs[UM][NB][4], ys[UM][NB][4], sc[UM][4];
#pragma unroll
        for (int i = 0; i < UM; ++i) {
            const int p = i * kBpWaves + wave;
            const int q = p - n_in;
            const int rel = p < n_in ? J.in_a + p : (q < J.in_a ? q : J.in_b + (q - J.in_a));
            const bool live = p < nblk;
            const int blk = J.blk0 + (live ? rel : 0);
            const int L = ((const QH_CONST int32_t *)T.bb_lo)[blk];
            const uint64_t tiles = live ? ((const QH_CONST uint64_t *)T.tiles)[blk] : 0;
            ut[i] = live ? ((const QH_CONST int32_t *)T.bb_w)[blk] / kTile : -1;
            uo[i] = (uint32_t)(L - xlo) | (uint32_t)(blk * kBandRows - xlo) << 16;
            if (live && (rel < J.pub_a || rel >= J.pub_b)) upub |= 1 << i;
            const bp_rsrc_t rsrc = bp_strip(T.bb_val, ((const QH_CONST int64_t *)T.bb_off)[blk], tiles,
                                            kTileElems * EB, kTileElems / 4 * EB);
#pragma unroll
            for (int c = 0; c < MAXT; ++c) {
                sp_load_tile<DT>(&jr[i][c * CR], rsrc, c, lane, tiles);
                if (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (bounds the loads in flight, and their registers)
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int u = blk * kBandRows + 4 * g4 + k;
                const bool in = live && u < n;
                sc[i][k] = 1.0f;
                if constexpr (DT == QH_FP8_ROWSCALE) {
                    if (in) sc[i][k] = ((const QH_GLOBAL float *)T.scale)[u];
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int64_t idx = (int64_t)u * R + r0 + b * 16 + l16;
                    xs[i][b][k] = in ? ((const QH_GLOBAL float *)T.x)[idx] : 0.f;
                    ys[i][b][k] = in ? ((const QH_GLOBAL float *)T.y)[idx] : 0.f;
                }
            }
        }
        uint16_t *xch = (uint16_t *)(a.xch + J.xch_off);
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
                        const int own = (J.blk0 * kBandRows - xlo) * RT * 2;
                        bp_fetch(sp_x, xch + ((t - 1) & 1) * half + (int64_t)xlo * RT, own, own + nblk * kBandRows * RT * 2,
                                 (J.xhi - xlo) * RT * 2, wave, lane);
                    }
                    bp_barrier();
                }
                // (as in the band kernel: keeps invariants of the step loop from being built ahead
                // of it and spilled)
#pragma unroll
                for (int i = 0; i < UM; ++i) {
                    __asm__ volatile("" : "+s"(ut[i]), "+s"(uo[i]));
#pragma unroll
                    for (int c = 0; c < MAXT * CR; ++c) __asm__ volatile("" : "+v"(jr[i][c]));
                }
                // B fragments of tile c of unit i
                auto read_b = [&](sp_half8_t (&bv)[2][NB], int i, int c) {
                    const uint16_t *xb = sp_x + ((uo[i] & 0xffff) + c * kTile) * RT + g4 * RT * 8 + l16 * 8;
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int b = 0; b < NB; ++b) bv[kb][b] = *(const sp_half8_t *)(xb + kb * 32 * RT + b * 128);
                };
                sp_half8_t first[2][NB];
                read_b(first, 0, 0);
#pragma unroll
                for (int i = 0; i < UM; ++i) {
                    const int nt = ut[i];
                    if (nt >= 0 && (i < ih) == (ph == 0)) {
                        const int orow = uo[i] >> 16;      // LDS row of the unit's first own row
                        bp_float4_t acc[NB];
#pragma unroll
                        for (int b = 0; b < NB; ++b) acc[b] = bp_float4_t{0.f, 0.f, 0.f, 0.f};
                        auto mfma_tile = [&](const uint32_t *j, const sp_half8_t (&bv)[2][NB]) {
#pragma unroll
                            for (int kb = 0; kb < 2; ++kb) {
                                const sp_half8_t av = sp_frag<DT>(j, kb);
#pragma unroll
                                for (int b = 0; b < NB; ++b) {
                                    if constexpr (DT == QH_BF16) {
                                        sp_bf16x8_t aw, bw;
                                        __builtin_memcpy(&aw, &av, 16);
                                        __builtin_memcpy(&bw, &bv[kb][b], 16);
                                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, bw, acc[b], 0, 0, 0);
                                    } else {
                                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv[kb][b], acc[b], 0, 0, 0);
                                    }
                                }
                            }
                        };
                        if (i == ih && i > 0) read_b(first, i, 0);
                        sp_half8_t bv[2][2][NB];
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int b = 0; b < NB; ++b) bv[0][kb][b] = first[kb][b];
#pragma unroll
                        for (int c = 0; c < MAXT; ++c) {
                            if (c < nt) {
                                if (c + 1 < MAXT) read_b(bv[(c + 1) & 1], i, c + 1);
                                mfma_tile(&jr[i][c * CR], bv[c & 1]);
                            }
                        }
                        if (MAXT < nt) {                   // those past the register-held ones
                            const int blk = (orow + xlo) / kBandRows;
                            const uint64_t tiles = ((const QH_CONST uint64_t *)T.tiles)[blk];
                            const bp_rsrc_t rsrc = bp_strip(T.bb_val, ((const QH_CONST int64_t *)T.bb_off)[blk], tiles,
                                                            kTileElems * EB, kTileElems / 4 * EB);
#pragma unroll 1
                            for (int c = MAXT; c < nt; ++c) {
                                uint32_t jt[CR];
                                sp_half8_t bt[2][NB];
                                sp_load_tile<DT>(jt, rsrc, c, lane, tiles);
                                read_b(bt, i, c);
                                mfma_tile(jt, bt);
                            }
                        }
                        if (i + 1 < UM) read_b(first, i + 1, 0);
                        if constexpr (DT == QH_FP8_ROWSCALE) {
#pragma unroll
                            for (int b = 0; b < NB; ++b)
#pragma unroll
                                for (int k = 0; k < 4; ++k) acc[b][k] *= sc[i][k];
                        }
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
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const float yn = ys[i][b][k] + (-coef * xs[i][b][k] + c0 * acc[b][k]) * a.dt;
                                const float xn = xs[i][b][k] + a.a0 * yn * a.dt;
                                ys[i][b][k] = fabsf(xn) > 1.0f ? 0.0f : yn;
                                xs[i][b][k] = __builtin_amdgcn_fmed3f(xn, -1.0f, 1.0f);
                            }
                    }
                }
            }
            bp_barrier();                          // every wave is past its reads of the copy
#pragma unroll
            for (int i = 0; i < UM; ++i) {
                __asm__ volatile("" : "+s"(ut[i]), "+s"(uo[i]));
                if (ut[i] >= 0) {
                    // the strip's new copy: rows 4 g4 .. + 3 are half of a group of eight
                    const int lr = (uo[i] >> 16) + 4 * g4;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        uint64_t pk = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            // rows past n keep a copy of 0 (also in the discrete variant)
                            const uint16_t h = xlo + lr + k < n ? sp_copy<DT, DISC>(xs[i][b][k]) : (uint16_t)0;
                            pk |= (uint64_t)h << (16 * k);
                        }
                        const int o = ((lr >> 3) * RT + b * 16 + l16) * 8 + (lr & 7);
                        *(uint64_t *)(sp_x + o) = pk;
                        if (upub >> i & 1)
                            __hip_atomic_store((QH_GLOBAL uint64_t *)(xch + (t & 1) * half + (int64_t)xlo * RT + o), pk,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
            pump = ((const QH_CONST float *)a.pump)[min(a.kb + s + 1, a.ke - 1)];
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
            if (ut[i] >= 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int u = (uo[i] >> 16) + xlo + 4 * g4 + k;
                    if (u < n) {
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            const int64_t idx = (int64_t)u * R + r0 + b * 16 + l16;
                            ((QH_GLOBAL float *)T.x)[idx] = bad ? __builtin_nanf("") : xs[i][b][k];
                            ((QH_GLOBAL float *)T.y)[idx] = ys[i][b][k];
                        }
                    }
                }
            }
        }
    }
}

template <int DT, int NB, int UM, bool DISC>
static void launch_strip_t(const BandLaunch &bl, const BandPersistArgs &args, hipStream_t st) {
    auto fn = k_strip_persistent<DT, NB, UM, DISC>;
    if (hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bl.lds_bytes) !=
        hipSuccess)
        (void)hipGetLastError();
    BandPersistArgs a = args;
    void *kargs[] = {&a};
    QH_HIP(hipLaunchCooperativeKernel((const void *)fn, dim3((unsigned)bl.grid), dim3(kBpThreads), kargs,
                                      (unsigned)bl.lds_bytes, st));
}

template <bool DISC>
static void launch_strip_disc(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st) {
#define QH_SP_U(DTV, NBV)                                               \
    do {                                                                \
        if (bl.um == 1) launch_strip_t<DTV, NBV, 1, DISC>(bl, a, st);      \
        else if (bl.um == 2) launch_strip_t<DTV, NBV, 2, DISC>(bl, a, st); \
        else launch_strip_t<DTV, NBV, 4, DISC>(bl, a, st);                 \
    } while (0)
#define QH_SP(DTV)                        \
    do {                                  \
        if (bl.rt == 16) QH_SP_U(DTV, 1); \
        else QH_SP_U(DTV, 2);             \
    } while (0)
    switch (bl.dtype) {
        case QH_F16: QH_SP(QH_F16); break;
        case QH_BF16: QH_SP(QH_BF16); break;
        case QH_FP8_ROWSCALE: QH_SP(QH_FP8_ROWSCALE); break;
        default: fail(QH_EUNSUPPORTED, "the strip plan needs a 16- or 8-bit dense graph");
    }
#undef QH_SP
#undef QH_SP_U
}

}  // namespace qh
