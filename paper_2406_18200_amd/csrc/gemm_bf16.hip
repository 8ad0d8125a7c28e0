// Projections of the verify step:  Y[M][Nout] = X[M][K] . W[Nout][K]^T  for the M token rows (N branches x gamma
// drafts) of a step, bf16 / one-byte / four-bit weights, fp32 accumulation on the MFMA units, with the row-wise work
// that follows each projection fused into its epilogue.
//
//   * W is repacked once at init into MFMA A-fragment order: tile (nt, kt) = 16 output features x 32
//     inputs = 1 KiB contiguous, lane l holding W[nt*16 + l%16][kt*32 + 8*(l/16) .. +8]; all k-tiles of an
//     n-tile are contiguous.  Weights go straight to registers with coalesced 1 KiB non-temporal loads.
//   * X (activations: tiny, L2-resident) is kept in the matching B-fragment order by its producer, as a
//     hi/lo pair of bf16 values per element (two MFMAs per weight fragment): the weights stay bf16 but the
//     activations keep ~16 significant bits, so their rounding does not pile up over 32-40 layers.
//   * v_mfma_f32_16x16x32_bf16 computes Y^T tiles: D[i = feature][j = token row].
//   * Epilogues: STORE (optional per-row scale = the RMSNorm factor of the input rows), RESID (residual add,
//     next RMSNorm's gain folded into the packed hi/lo activation, per-tile sums of squares of the new
//     residual rows), SWIGLU (gate and up tiles are interleaved in the packed weight so one wavefront holds
//     both; emits the packed activation of the down projection).  The RMSNorm factor 1/rms of the input rows
//     is applied AFTER the contraction: each consuming workgroup sums the producer's per-tile sums of squares
//     in a fixed order.
// Two kernel forms share the weight layout and the epilogues: gemm_stream_kernel (gemm_stream.h: few rows, narrow
// outputs, narrow weights) and gemm_wide_kernel here (the wide outputs from 49 rows on, everything past 128 rows).
// gemm_plan chooses form, workgroup shape and split.
#include <map>
#include <mutex>
#include <type_traits>
#include "gemm_device.h"

namespace seedv {
namespace {

// Workgroup shapes: WN wavefronts side by side on different n-tile groups x WK wavefronts splitting every k-chunk of
// the same n-tiles (their partial tiles are summed through LDS at the end, in a fixed order).
template <int TM, int TN, int WN, int WK>
struct Shape {
    // tiles summed per round of the cross-wavefront reduction (<= 64 KiB of LDS per round)
    static constexpr int kRedTiles = (64 / (WK * WN)) >= 1 ? (64 / (WK * WN)) : 1;
};

// 1/rms of the input rows from the producer's per-tile sums of squares, summed in a fixed order: wavefront w
// takes rows w, w + kWaves, ...; a row of up to 512 sums is two 16-byte loads per lane, and the loads of eight
// rows are in flight together (row after row would pay a memory latency each: twelve of them at 96 rows).
template <int kWaves>
__device__ __forceinline__ void rows_rinv(const GemmArgs &a, float *s_rinv, int w, int lane, int r_lo, int r_hi) {
    // rows r_lo .. r_hi - 1 (this workgroup's share); s_rinv is indexed from r_lo
    constexpr int kRowsAtOnce = 8;
    const int nt_in = a.NT_in;
    if (nt_in <= 512 && (nt_in & 3) == 0) {
        for (int row0 = r_lo + w; row0 < r_hi; row0 += kRowsAtOnce * kWaves) {
            f32x4 v[kRowsAtOnce][2];
#pragma unroll
            for (int r = 0; r < kRowsAtOnce; ++r)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int row = min(row0 + r * kWaves, r_hi - 1), t = 4 * lane + 256 * i;
                    // (the load itself is unconditional, its value masked: a select on the value lets the compiler
                    // put the load under a branch, and a branch around a load drains the load queue at the join)
                    const u32x4 x = *reinterpret_cast<const u32x4 *>(a.ssq_in + (size_t)row * nt_in + (t < nt_in ? t : 0));
                    const uint32_t keep = t < nt_in ? 0xffffffffu : 0u;
                    v[r][i] = __builtin_bit_cast(f32x4, x & keep);
                }
#pragma unroll
            for (int r = 0; r < kRowsAtOnce; ++r) {
                const f32x4 q = v[r][0] + v[r][1];
                const float ssum = wave_reduce_sum_dpp((q[0] + q[1]) + (q[2] + q[3]));
                // (no branch: every lane writes the one value; a row past the end repeats the last row's)
                s_rinv[min(row0 + r * kWaves, r_hi - 1) - r_lo] = 1.0f / sqrtf(ssum / (float)(nt_in * 16) + a.eps);
            }
        }
    } else {
        for (int row = r_lo + w; row < r_hi; row += kWaves) {
            float ssum = 0.f;
            for (int t = lane; t < nt_in; t += 64) ssum += a.ssq_in[(size_t)row * nt_in + t];
            ssum = wave_reduce_sum(ssum);
            if (lane == 0) s_rinv[row - r_lo] = 1.0f / sqrtf(ssum / (float)(nt_in * 16) + a.eps);
        }
    }
}

// Everything after the k loop: the cross-wavefront reduction of a workgroup's WK partial tiles and the epilogue.
// `smem` is the k loop's staging memory, reused for the reduction; s_rinv holds 1/rms of the workgroup's rows.
template <int TM, int TN, int WN, int WK, int EPI>
__device__ __forceinline__ void finish_tiles(const GemmArgs &a, f32x4 (&acc)[TN][TM], char *smem, const float *s_rinv,
                                             int nt0, bool active, int mh) {
    using S = Shape<TM, TN, WN, WK>;
    constexpr int RT = S::kRedTiles < TN * TM ? S::kRedTiles : TN * TM;   // tiles per reduction round
    f32x4(*red)[WN][RT][64] = reinterpret_cast<f32x4(*)[WN][RT][64]>(smem);                 // [WK][WN][RT][64]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int wn = w % WN, wk = w / WN;
    const int g = lane >> 4, rlow = lane & 15;
    const int nt_last = a.NT - 1;
    __syncthreads();                                      // s_rinv visible; the stages are no longer read

    if (WK > 1) {
        // sum the WK partial tiles of each n-tile group through LDS (fixed order), RT tiles per round;
        // wavefronts with wk == 0 end up holding the finished tiles
#pragma unroll
        for (int t0 = 0; t0 < TN * TM; t0 += RT) {
            __syncthreads();                              // the stages / the previous round are no longer read
#pragma unroll
            for (int t = 0; t < RT; ++t)
                if (t0 + t < TN * TM) red[wk][wn][t][lane] = acc[(t0 + t) / TM][(t0 + t) % TM];
            __syncthreads();
            if (wk == 0) {
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    if (t0 + t < TN * TM) {
                        f32x4 s = red[0][wn][t][lane];
#pragma unroll
                        for (int i = 1; i < WK; ++i) s += red[i][wn][t][lane];
                        acc[(t0 + t) / TM][(t0 + t) % TM] = s;
                    }
            }
        }
    }
    if (!active || wk != 0) return;                       // the others hold no finished tiles
    const int rbase = mh * TM * 16;                       // first row of this workgroup's share

    // D[i][j]: lane holds features 4*(lane/16)+0..3 (columns) of token row lane%16
    const int ld_part = a.NT * 16;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int row = rbase + tm * 16 + rlow;
        const bool valid = row < a.M;
        if (EPI == EPI_STORE) {
            const float sc = (valid && a.ssq_in != nullptr) ? s_rinv[row - rbase] : 1.f;
            if (valid) {
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    if (nt0 + tn <= nt_last)
                        *reinterpret_cast<f32x4 *>(a.out + (size_t)row * a.ld_out + (nt0 + tn) * 16 + 4 * g) = acc[tn][tm] * sc;
            }
        } else if (EPI == EPI_RESID) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int col = (nt0 + tn) * 16 + 4 * g;
                float ss = 0.f;
                const bool tile_ok = nt0 + tn <= nt_last;
                if (valid && tile_ok) {
                    float *xp2 = a.x + (size_t)row * ld_part + col;
                    f32x4 xv = *reinterpret_cast<f32x4 *>(xp2) + acc[tn][tm];
                    *reinterpret_cast<f32x4 *>(xp2) = xv;
                    const uint2 gw = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(a.gain) + col);
                    const float gv[4] = {bf2f((uint16_t)(gw.x & 0xffff)), bf2f((uint16_t)(gw.x >> 16)),
                                         bf2f((uint16_t)(gw.y & 0xffff)), bf2f((uint16_t)(gw.y >> 16))};
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        ss += xv[i] * xv[i];
                        v[i] = xv[i] * gv[i];
                    }
                    store_act4(a.act_out, row, col, a.KT_out, v);
                }
                ss += __shfl_xor(ss, 16);
                ss += __shfl_xor(ss, 32);
                if (valid && tile_ok && g == 0) a.ssq[(size_t)row * a.NT + nt0 + tn] = ss;
            }
        } else {   // EPI_SWIGLU: tiles (nt0 + 2p, nt0 + 2p + 1) = (gate, up) of feature block nt0 / 2 + p
            if (valid) {
                const float sc = s_rinv[row - rbase];
#pragma unroll
                for (int p = 0; p < TN / 2; ++p) {
                    if (nt0 + 2 * p + 1 > nt_last) continue;          // ragged last group: no such feature block
                    float h[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float gt = acc[2 * p][tm][i] * sc, up = acc[(2 * p + 1) % TN][tm][i] * sc;
                        h[i] = gt / (1.0f + expf(-gt)) * up;
                    }
                    store_act4(a.act_out, row, ((nt0 >> 1) + p) * 16 + 4 * g, a.KT_out, h);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// Form for three to eight row tiles per workgroup.  With that many rows a k-tile of activations is 6-16 KiB
// and every wavefront reads all of it for each of its n-tiles: what limits the kernel is no longer HBM alone
// but how many activation fragments a wavefront can have on their way from LDS while its MFMAs run, and how
// many registers are left for weights in flight.  Differences from the streaming form:
//   * the activation stages are filled by global -> LDS loads that bypass the registers (each lane's 16 bytes
//     land at the stage base + 16 * lane, which is the fragment order the MFMAs read); NS stages of one weight
//     group each, filled NS - 1 groups ahead, ONE workgroup barrier per group;
//   * one, two or four n-tiles per wavefront and workgroups of eight or twelve wavefronts (3 x 4: three per
//     SIMD, at most 168 registers), chosen so that a launch is one round of workgroups over most of the CUs;
//   * weights are addressed as a wavefront-uniform base in scalar registers plus one 32-bit lane offset per
//     n-tile: with 64-bit per-lane addresses the kernel spilled at six row tiles;
//   * the LDS reads are issued as one batch per k-tile and waited for fragment by fragment (inline assembly:
//     the compiler, which cannot see that a read does not touch the stage being filled, would otherwise wait
//     for the youngest global -> LDS load, and with it for every weight load issued before, ahead of each read).
// Counting rule the waits rely on: per group every wavefront issues exactly P stage loads, then U * TN weight
// loads, all unconditional with clamped addresses (the last round of groups issues no weight loads and counts
// accordingly); loads complete in issue order.  tests/test_isa_inflight.py replays the compiled ISA against
// these counts.
struct WideParams {
    int U, GK, stage_bytes, NS, F, P, D, wait_stage, wait_weights;
    bool valid;
};
constexpr WideParams wide_params(int TM, int TN, int WN, int WK) {
    WideParams p{};
    const int waves = WN * WK, budget = 144 * 1024;
    // k-tiles per wavefront and group: two where a k-tile is only a few MFMAs, if three stages still fit
    p.U = (TM * TN < 24 && 3 * (WK * 2 * TM * 2048) <= budget) ? 2 : 1;
    p.GK = WK * p.U;                                      // k-tiles per group = per LDS stage
    p.stage_bytes = p.GK * TM * 2048;
    const int fit = budget / p.stage_bytes;
    p.NS = fit > 4 ? 4 : fit;                             // stages
    p.F = p.GK * TM * 2;                                  // 1 KiB fragments per stage
    p.P = p.F / waves;                                    // stage loads per wavefront and group
    // weight groups in flight per wavefront: about 16 KiB, and no more than the stages are filled ahead (a
    // stage load completes only after the weight loads issued before it, so deeper rings gain nothing)
    const int want = 16 / (p.U * TN) < 2 ? 2 : 16 / (p.U * TN);
    p.D = want > p.NS - 1 ? p.NS - 1 : want;
    // loads a wavefront may still have in flight at the end of group g with the stage of group g + 1 complete
    p.wait_stage = (p.NS - 1) * p.U * TN + (p.NS - 2) * p.P;
    // ... and when group g starts its MFMAs, with the weights requested D groups ago complete: the stage loads
    // and weight loads of the D - 1 groups between, and this group's stage loads
    p.wait_weights = (p.D - 1) * (p.P + p.U * TN) + p.P;
    p.valid = p.NS >= 3 && p.F % waves == 0 && p.wait_stage < 64 && p.wait_weights < 64;   // (6-bit vmcnt)
    return p;
}
template <int TM, int TN, int WN, int WK>
struct WideShape {
    static constexpr WideParams p = wide_params(TM, TN, WN, WK);
    static constexpr int kWaves = WN * WK;
    static constexpr int U = p.U, GK = p.GK, kStageBytes = p.stage_bytes, NS = p.NS, F = p.F, P = p.P, D = p.D;
    static constexpr int kWaitStage = p.wait_stage, kWaitWeights = p.wait_weights;
    static constexpr bool kValid = p.valid;
};

// The loads of the k loop are issued and waited for by hand (inline assembly): with a global -> LDS load
// among the pending ones the compiler's own counting falls back to "wait for everything" ahead of every use.
// A register filled by such a load must not be touched before the matching wait; the waits take the
// registers as in/out operands, so that nothing that uses them can be scheduled ahead of the wait.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
template <int N, int TN>
__device__ __forceinline__ void wait_weights(bf16x8 (&wf)[TN]) {
    static_assert(N >= 0 && N < 64 && (TN == 1 || TN == 2 || TN == 4), "vmcnt is a 6-bit field");
    if constexpr (TN == 1) asm volatile("s_waitcnt vmcnt(%1)" : "+v"(wf[0]) : "n"(N));
    else if constexpr (TN == 2) asm volatile("s_waitcnt vmcnt(%2)" : "+v"(wf[0]), "+v"(wf[1]) : "n"(N));
    else asm volatile("s_waitcnt vmcnt(%4)" : "+v"(wf[0]), "+v"(wf[1]), "+v"(wf[2]), "+v"(wf[3]) : "n"(N));
}
// (wavefront-uniform 64-bit base in scalar registers + a 32-bit byte offset per lane: one address register
// per load instead of two)
__device__ __forceinline__ void load_weight_nt(bf16x8 &dst, const void *base, unsigned offset) {
    asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "=v"(dst) : "v"(offset), "s"(base));
}

// All 2 * TM fragments of one k-tile (hi and lo of every row tile; 1 KiB apart) in one batch.
template <int TM>
__device__ __forceinline__ void lds_read_ktile(bf16x8 (&f)[2 * TM], unsigned addr) {
#pragma unroll
    for (int i = 0; i < 2 * TM; ++i)
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f[i]) : "v"(addr), "n"(i * 1024));
}
// Wait until at most N of the batch's reads are outstanding; the fragments named become usable.
template <int N>
__device__ __forceinline__ void lds_wait(bf16x8 &a, bf16x8 &b) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}

// The MFMAs of one k-tile, row tile by row tile: fragments 2 tm (hi) and 2 tm + 1 (lo) are waited for while the
// 2 TM - 2 tm - 2 reads issued after them may still be on their way.
template <int TM, int TN, int tm = 0>
struct KtileMfma {
    static __device__ __forceinline__ void run(bf16x8 (&f)[2 * TM], const bf16x8 (&wf)[TN], f32x4 (&acc)[TN][TM]) {
        lds_wait<2 * TM - 2 * tm - 2>(f[2 * tm], f[2 * tm + 1]);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            acc[tn][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[tn], f[2 * tm + 1], acc[tn][tm], 0, 0, 0);
            acc[tn][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[tn], f[2 * tm], acc[tn][tm], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);                // keep wait -> MFMAs -> next wait in this order
        if constexpr (tm + 1 < TM) KtileMfma<TM, TN, tm + 1>::run(f, wf, acc);
    }
};

template <int TM, int TN, int WN, int WK, int EPI>
__global__ __launch_bounds__(WN * WK * 64) void gemm_wide_kernel(GemmArgs a) {
    using S = WideShape<TM, TN, WN, WK>;
    using S0 = Shape<TM, TN, WN, WK>;
    constexpr int U = S::U, GK = S::GK, NS = S::NS, D = S::D, P = S::P, kWaves = S::kWaves;
    constexpr int kStage = S::kStageBytes;
    constexpr int RT = S0::kRedTiles < TN * TM ? S0::kRedTiles : TN * TM;
    constexpr int RED_BYTES = (WK > 1) ? WK * WN * RT * 1024 : 16;
    constexpr int XS_BYTES = NS * kStage;
    static_assert(2 * TM * 1024 <= 65536, "ds_read offsets are 16-bit");
    __shared__ __attribute__((aligned(1024))) char smem[XS_BYTES > RED_BYTES ? XS_BYTES : RED_BYTES];
    __shared__ float s_rinv[128];
    pin_args(a);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (scalar: addresses below stay in SGPRs)
    const int wn = w % WN, wk = w / WN;
    int cg, mh;
    if (!wg_coords(a, WN * TN, cg, mh)) return;          // (uniform: a padding workgroup of a row-split launch)
    const int mt0 = mh * TM, mt_last = (a.M + 15) / 16 - 1;   // first row tile of this workgroup; last one there is
    const int nt0 = (cg * WN + wn) * TN;
    const bool active = nt0 < a.NT;
    const int KT = a.KT;
    constexpr int k0 = 0;                                // (this form is never split along K across workgroups)
    const int k1 = KT;
    const int n_groups = (k1 - k0 + GK - 1) / GK;
    // Every column group walks the k range from its own starting group: the workgroups of a launch start together
    // and run in step (a barrier per group), so without this all of them read the same k position at the same
    // time -- and the weights of different n-tiles at one k position lie KT KiB apart, i.e. on few memory
    // channels.  Measured at 96 rows on the 7B shapes: QKV 34.4 -> 32.5 us, gate/up 52.6 -> 50.8, LM head 71 -> 66
    // (any odd multiplier does the same).  The sums come out in another order per column group, still a fixed
    // one.  Only where the range is whole groups (no ragged tail to meet in mid-walk).
    const bool rot_ok = a.rot != 0 && (k1 - k0) % GK == 0 && n_groups > 1;
    const int rot = rot_ok ? (cg * a.rot) % n_groups : 0;
    auto kgroup = [&](int g) { return g < n_groups ? (g + rot >= n_groups ? g + rot - n_groups : g + rot) : g; };

    f32x4 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int nt_last = a.NT - 1;
    unsigned woff[TN];                                   // byte offset of this lane's piece of k-tile 0 of each n-tile
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) woff[tn] = ((unsigned)min(nt0 + tn, nt_last) * (unsigned)KT * 64u + lane) * 16u;
    const bf16x8 *xp = reinterpret_cast<const bf16x8 *>(a.Xp) + lane;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char *)smem;   // LDS byte address

    // stage load of group g: fragment f = w + i * kWaves of the stage, f = (kk * TM + tm) * 2 + hl; k-tiles past
    // the end of the matrix are clamped (their MFMAs are skipped)
    auto stage_load = [&](int g) {
        const unsigned base = (unsigned)((g % NS) * kStage);
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int f = w + i * kWaves;
            const int kk = f / (2 * TM), r = f - kk * (2 * TM);
            const int kt = min(k0 + kgroup(g) * GK + kk, KT - 1);
            const bf16x8 *src = xp + (((size_t)min(mt0 + (r >> 1), mt_last) * KT + kt) * 2 + (r & 1)) * 64;
            __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)(smem + base + f * 1024), 16,
                                             0, 0);
        }
    };
    bf16x8 ring[D][U][TN];
    auto load_a = [&](bf16x8 (&dst)[U][TN], int g) {     // this wavefront's k-tiles of group g (clamped)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const char *base = reinterpret_cast<const char *>(a.Wp) + (size_t)min(k0 + kgroup(g) * GK + wk * U + u, k1 - 1) * 1024;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) load_weight_nt(dst[u][tn], base, woff[tn]);
        }
    };
    // prologue: the first NS - 1 stages and D weight groups, everything waited for once
#pragma unroll
    for (int g = 0; g < NS - 1; ++g) stage_load(g);
#pragma unroll
    for (int dd = 0; dd < D; ++dd) load_a(ring[dd], dd);
    // the input rows' 1/rms while the first weights are on their way (its loads come back after them, so the
    // wait inside is the prologue's wait)
    if (EPI != EPI_RESID && a.ssq_in != nullptr) rows_rinv<kWaves>(a, s_rinv, w, lane, mt0 * 16, min(a.M, (mt0 + TM) * 16));
#pragma unroll
    for (int dd = 0; dd < D; ++dd)
#pragma unroll
        for (int u = 0; u < U; ++u) wait_weights<0, TN>(ring[dd][u]);
    wait_vmcnt<0>();
    lds_barrier();

    // One group.  DD = its ring slot.  TAIL = it belongs to the last round, which requests no further weights
    // (a register that a load is still going to write must stay reserved until a wait covers that load: the
    // result of a load nobody uses would be handed to other values at once) and where the k range may end
    // inside the group; its waits count the loads that the groups before it really issued.
    auto group = [&](int g, auto dd_tag, auto tail_tag) {
        constexpr int DD = decltype(dd_tag)::value;
        constexpr bool TAIL = decltype(tail_tag)::value;
        // loads issued after the weights of this group, which were requested at the end of group g - D
        constexpr int kWaitW = TAIL ? (D - 1 - DD) * (P + U * TN) + (DD + 1) * P : S::kWaitWeights;
        // loads issued after the stage loads of group g + 1 (start of group g + 2 - NS): the weight loads of
        // those of the groups g + 2 - NS .. g that are not in the last round, the stage loads of the later ones
        constexpr int kTailWeightGroups = NS - 2 - DD > 0 ? NS - 2 - DD : 0;
        constexpr int kWaitS = TAIL ? kTailWeightGroups * U * TN + (NS - 2) * P : S::kWaitStage;
        stage_load(g + NS - 1);                           // into the stage group g - 1 was read from
        __builtin_amdgcn_sched_barrier(0);
        const unsigned sbase = lds0 + (unsigned)((g % NS) * kStage) + lane * 16;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kk = wk * U + u;
            wait_weights<kWaitW, TN>(ring[DD][u]);        // (also in a skipped k-tile: the registers stay reserved)
            if (TAIL && k0 + g * GK + kk >= k1) continue; // (uniform)
            bf16x8 f[2 * TM];
            lds_read_ktile<TM>(f, sbase + (unsigned)(kk * TM * 2048));
            KtileMfma<TM, TN>::run(f, ring[DD][u], acc);
        }
        if constexpr (!TAIL) load_a(ring[DD], g + D);     // refill this slot D groups ahead
        wait_vmcnt<kWaitS>();                             // the stage of group g + 1 is complete (this wavefront's part)
        lds_barrier();                                    // ... everybody's part; stage g % NS is free again
    };
    // groups in rounds of D (ring slots are compile-time indices); the last round is peeled
    const int n_rounds = (n_groups + D - 1) / D;
    auto round = [&](int r, auto tail_tag) {
        const int g0 = r * D;
        constexpr bool TAIL = decltype(tail_tag)::value;  // only the last round can be incomplete
        group(g0, std::integral_constant<int, 0>{}, tail_tag);
        if constexpr (D > 1) {
            if (!TAIL || g0 + 1 < n_groups) {
                group(g0 + 1, std::integral_constant<int, 1>{}, tail_tag);
                if constexpr (D > 2) {
                    if (!TAIL || g0 + 2 < n_groups) {
                        group(g0 + 2, std::integral_constant<int, 2>{}, tail_tag);
                        if constexpr (D > 3) {
                            if (!TAIL || g0 + 3 < n_groups) group(g0 + 3, std::integral_constant<int, 3>{}, tail_tag);
                        }
                    }
                }
            }
        }
        static_assert(D <= 4, "rounds are written out for up to four ring slots");
    };
    for (int r = 0; r < n_rounds - 1; ++r) round(r, std::false_type{});
    if (n_rounds > 0) round(n_rounds - 1, std::true_type{});
    // Everything still in flight lands before the registers and the staging memory get other uses: weights
    // requested for groups past the end of the k range (the ring is named, so it stays reserved up to here)
    // and stage loads past the last group.
#pragma unroll
    for (int dd = 0; dd < D; ++dd)
#pragma unroll
        for (int u = 0; u < U; ++u) wait_weights<0, TN>(ring[dd][u]);
    wait_vmcnt<0>();
    finish_tiles<TM, TN, WN, WK, EPI>(a, acc, smem, s_rinv, nt0, active, mh);
}

// Repack row-major W[n_rows][K] (bf16) into fragment tiles.  Destination tile index of source n-tile
// t is dst_tile0 + t * dst_tile_step (step 2 interleaves the gate and up projections tile by tile).
__global__ void pack_weight_kernel(const uint16_t *__restrict__ W, u32x4 *__restrict__ dst, int n_tiles,
                                   int K, int KT, int dst_tile0, int dst_tile_step) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte fragment each
    const size_t total = (size_t)n_tiles * KT * 64;
    if (idx >= total) return;
    const int lane = idx & 63;
    const size_t tile = idx >> 6;
    const int kt = tile % KT;
    const int nt = tile / KT;
    const uint16_t *src = W + (size_t)(nt * 16 + (lane & 15)) * K + kt * 32 + 8 * (lane >> 4);
    const u32x4 v = *reinterpret_cast<const u32x4 *>(src);
    dst[(((size_t)(dst_tile0 + nt * dst_tile_step)) * KT + kt) * 64 + lane] = v;
}

// The same repacking for one-byte weights: row-major codes [n_rows][K] into pairs of k-tiles of 1 KiB (lane l holds
// its eight codes of k-tile 2 kp, then those of 2 kp + 1: one 16-byte load), and the per-row scales into the order of
// the packed tiles.  The second half of an odd last pair is zero.
__global__ void pack_weight8_kernel(const uint8_t *__restrict__ W, uint2 *__restrict__ dst, int n_tiles, int K, int KT,
                                    int dst_tile0, int dst_tile_step) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 8-byte fragment each
    const int KP = (KT + 1) / 2;
    if (idx >= (size_t)n_tiles * KP * 128) return;
    const int lane = idx & 63;
    const size_t tile = idx >> 6;
    const int kt = tile % (2 * KP);
    const int nt = tile / (2 * KP);
    uint2 v = {0u, 0u};
    if (kt < KT) v = *reinterpret_cast<const uint2 *>(W + (size_t)(nt * 16 + (lane & 15)) * K + kt * 32 + 8 * (lane >> 4));
    dst[(((size_t)(dst_tile0 + nt * dst_tile_step)) * KP + (kt >> 1)) * 128 + lane * 2 + (kt & 1)] = v;
}
__global__ void pack_scale_kernel(const float *__restrict__ src, float *__restrict__ dst, int n_rows, int dst_tile0,
                                  int dst_tile_step) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n_rows) dst[(size_t)(dst_tile0 + (r >> 4) * dst_tile_step) * 16 + (r & 15)] = src[r];
}

// ... and for four-bit weights: row-major codes [n_rows][K/2] into pairs of k-tiles of 512 bytes (eight bytes per
// lane), the E8M0 block scales [n_rows][K/32] into [n-tile][pair][16 rows][2].
__global__ void pack_weight4_kernel(const uint8_t *__restrict__ W, uint32_t *__restrict__ dst, int n_tiles, int K, int KT,
                                    int dst_tile0, int dst_tile_step) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 4-byte fragment each
    const int KP = (KT + 1) / 2;
    if (idx >= (size_t)n_tiles * KP * 128) return;
    const int lane = idx & 63;
    const size_t tile = idx >> 6;
    const int kt = tile % (2 * KP);
    const int nt = tile / (2 * KP);
    uint32_t v = 0u;
    if (kt < KT) v = *reinterpret_cast<const uint32_t *>(W + ((size_t)(nt * 16 + (lane & 15)) * K + kt * 32 + 8 * (lane >> 4)) / 2);
    dst[(((size_t)(dst_tile0 + nt * dst_tile_step)) * KP + (kt >> 1)) * 128 + lane * 2 + (kt & 1)] = v;
}
__global__ void pack_mx_scale_kernel(const uint8_t *__restrict__ src, uint8_t *__restrict__ dst, int n_rows, int KT,
                                     int dst_tile0, int dst_tile_step) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one (row, k-tile) each
    const int KP = (KT + 1) / 2;
    if (idx >= (size_t)n_rows * KP * 2) return;
    const int r = idx / (2 * KP), kt = idx % (2 * KP);
    dst[((size_t)(dst_tile0 + (r >> 4) * dst_tile_step) * KP + (kt >> 1)) * 32 + (r & 15) * 2 + (kt & 1)] = kt < KT ? src[(size_t)r * KT + kt] : 0;
}

// The wide form counts its own loads; a kernel that the compiler gave spill code (scratch loads and stores
// are loads in that count too) must not run.  Checked once per kernel.
int wide_kernel_usable(const void *kernel) {
    static std::mutex mu;
    static std::map<const void *, int> seen;
    std::lock_guard<std::mutex> lock(mu);
    auto it = seen.find(kernel);
    if (it == seen.end()) {
        hipFuncAttributes fa{};
        const int rc = hip_fail(hipFuncGetAttributes(&fa, kernel), "hipFuncGetAttributes");
        if (rc) return rc;
        it = seen.emplace(kernel, (int)fa.localSizeBytes).first;
    }
    if (it->second != 0) {
        set_error("gemm: this wide kernel was compiled with %d bytes of scratch per lane and is not used", it->second);
        return SEED_E_UNSUPPORTED_DTYPE;
    }
    return SEED_OK;
}

template <int TM, int TN, int WN, int WK>
int launch_wide_shape(const GemmArgs &a, int epi, hipStream_t st) {
    using S = WideShape<TM, TN, WN, WK>;
    if constexpr (!S::kValid) {
        set_error("gemm: the wide form has no %dx%d workgroup with %d n-tiles for %d row tiles", WN, WK, TN, TM);
        return SEED_E_CAPACITY;
    } else {
        GemmArgs b = a;
        if (a.w_scale != nullptr || a.w_mx != nullptr) { set_error("gemm: the wide form streams bf16 weights only"); return SEED_E_UNSUPPORTED_DTYPE; }
        if ((size_t)a.NT * a.KT * 1024 >= ((size_t)1 << 32)) {
            set_error("gemm: the wide form addresses weights with 32-bit offsets (matrix of %d x %d tiles)", a.NT, a.KT);
            return SEED_E_CAPACITY;
        }
        const int groups = (a.NT + WN * TN - 1) / (WN * TN);
        if (b.MS < 1) b.MS = 1;
        dim3 grid(b.MS > 1 ? (groups + 7) / 8 * 8 * b.MS : groups), block(WN * WK * 64);
        int rc;
        if (epi == EPI_SWIGLU) {
            if constexpr (TN >= 2) {
                if ((rc = wide_kernel_usable((const void *)gemm_wide_kernel<TM, TN, WN, WK, EPI_SWIGLU>))) return rc;
                hipLaunchKernelGGL((gemm_wide_kernel<TM, TN, WN, WK, EPI_SWIGLU>), grid, block, 0, st, b);
            } else {
                set_error("gemm: the SwiGLU epilogue needs paired tiles");
                return SEED_E_INVALID_ARG;
            }
        } else if (epi == EPI_RESID) {
            if ((rc = wide_kernel_usable((const void *)gemm_wide_kernel<TM, TN, WN, WK, EPI_RESID>))) return rc;
            hipLaunchKernelGGL((gemm_wide_kernel<TM, TN, WN, WK, EPI_RESID>), grid, block, 0, st, b);
        } else {
            if ((rc = wide_kernel_usable((const void *)gemm_wide_kernel<TM, TN, WN, WK, EPI_STORE>))) return rc;
            hipLaunchKernelGGL((gemm_wide_kernel<TM, TN, WN, WK, EPI_STORE>), grid, block, 0, st, b);
        }
        return hip_fail(hipGetLastError(), "gemm launch");
    }
}

// Three to eight row tiles in the wide form: two or four n-tiles per wavefront.
template <int TM>
int launch_wide(const GemmArgs &a, int epi, int wn, int wk, int tn, hipStream_t st) {
#define SEEDV_SHAPE(WNv, WKv)                                                             \
    if (wn == WNv && wk == WKv)                                                           \
        return tn == 4 ? launch_wide_shape<TM, 4, WNv, WKv>(a, epi, st) : launch_wide_shape<TM, 2, WNv, WKv>(a, epi, st);
    if (tn == 2 || tn == 4) {
        SEEDV_SHAPE(4, 2) SEEDV_SHAPE(2, 4) SEEDV_SHAPE(1, 8)
    }
#undef SEEDV_SHAPE
    // twelve wavefronts, six n-tiles per workgroup: 1376 n-tiles (7B gate/up) become 230 workgroups instead of 172
    if (tn == 2 && wn == 3 && wk == 4) return launch_wide_shape<TM, 2, 3, 4>(a, epi, st);
    // ... twelve n-tiles per workgroup: the shape of the row-split launches (half the rows, twice the columns)
    if constexpr (TM <= 4) {
        if (tn == 4 && wn == 3 && wk == 4) return launch_wide_shape<TM, 4, 3, 4>(a, epi, st);
    }
    // ... and three n-tiles per workgroup, one per wavefront: 768 n-tiles (7B QKV) become 256 workgroups
    if (tn == 1 && wn == 3 && wk == 4 && epi != EPI_SWIGLU) return launch_wide_shape<TM, 1, 3, 4>(a, epi, st);
    set_error("gemm: unsupported wide workgroup shape %dx%d with %d n-tiles", wn, wk, tn);
    return SEED_E_INVALID_ARG;
}

// Multiplier of the per-column-group rotation of the k walk: in k-tiles (pairs of k-tiles for narrow weights) in the
// streaming form, in weight groups in the wide form.
constexpr int kRotation = 24, kRotationGroups = 3;

// Form, shape and split of a projection launch.
struct GemmPlan {
    bool wide;                // gemm_wide_kernel (wn x wk wavefronts), else gemm_stream_kernel
    int wn, wk;
    int tm, tn;               // row tiles of a workgroup; n-tiles of a wavefront (wide) or of a workgroup (streaming)
    int sk, ms;               // workgroups along K per column group; row shares
};

GemmPlan gemm_plan(int NT, int KT, int epi, int M, int wb, size_t part_floats) {
    const int m_tiles = (M + 15) / 16;
    GemmPlan p{};
    if (m_tiles > 8 && NT % 4 == 0 && KT >= 64 && wb == 16) {
        // Past 128 rows the launch is bound by MFMA issue and LDS reads, not by memory, so the big register tiles of
        // the wide form: up to eight row tiles x four n-tiles per wavefront (a weight fragment feeds up to 16 MFMAs,
        // an activation fragment read from LDS four), 4 x 2 wavefronts (sixteen n-tiles per workgroup) or 2 x 4
        // (eight, K split four ways inside the workgroup).  One such workgroup fills a CU, so the launch runs in whole
        // rounds of 256: shape and row tiles per workgroup are chosen for the least rounds x (tiles + 2) x k-tiles per
        // wavefront (the 2: what a workgroup costs besides its MFMAs, in tiles); 2 x 4, whose activation fragments feed
        // half as many wavefronts, costs about 1.2 times as much per MFMA (4096 x 4096 at 1999 rows: 191 us as 672
        // workgroups in three rounds, 126 us as 256 in one; at 768 rows 2 x 4 fills the chip, 4 x 2 three eighths).
        int best_tm = 0, best_wn = 4, best_cost = 1 << 30;
        for (int swn : {4, 2}) {
            const int groups = ((NT + 4 * swn - 1) / (4 * swn) + 7) / 8 * 8;
            for (int t : {8, 6, 5, 4, 3}) {
                const int shares = (m_tiles + t - 1) / t, tm = (m_tiles + shares - 1) / shares;   // tm <= t
                if (tm < 3 || !wide_params(tm, 4, swn, 8 / swn).valid) continue;
                const int cost = ((groups * shares + 255) / 256) * (tm + 2) * (swn == 4 ? 20 : 12);
                if (cost < best_cost) { best_cost = cost; best_tm = tm; best_wn = swn; }
            }
        }
        if (best_tm > 0) {
            p.wide = true; p.wn = best_wn; p.wk = 8 / best_wn; p.tm = best_tm; p.tn = 4; p.sk = 1; p.ms = (m_tiles + best_tm - 1) / best_tm;
            return p;
        }
    }
    if (m_tiles >= 4 && m_tiles <= 8 && NT >= 600 && wb == 16) {
        // The wide outputs of 49 .. 128 rows.  From five row tiles on two workgroups per column group, three or four
        // row tiles each (see wg_coords): twelve wavefronts (3 x 4); as few n-tiles per wavefront as keep the launch
        // within one round of workgroups (7B QKV: 2 -> 128 column groups x 2; 7B gate/up: 4 -> 115 x 2).
        const int half = (m_tiles + 1) / 2;
        if (m_tiles >= 5)
            for (int t : {2, 4}) {
                const int groups = ((NT + 3 * t - 1) / (3 * t) + 7) / 8 * 8;
                if (groups * 2 <= 256 && wide_params(half, t, 3, 4).valid && NT % t == 0) {
                    p.wide = true; p.wn = 3; p.wk = 4; p.tn = t; p.tm = half; p.sk = 1; p.ms = 2;
                    return p;
                }
            }
        p.tm = m_tiles; p.sk = p.ms = 1;
        // one workgroup per column group: six n-tiles per workgroup where that still is one round of workgroups and
        // eight would leave a quarter of the CUs idle (7B gate/up, 1376 n-tiles, 230 workgroups instead of 172);
        // three (one per wavefront) for the mid-width outputs (7B QKV, 768 n-tiles, 256 workgroups instead of 192)
        if (NT >= 1300 && (NT + 5) / 6 <= 256 && (NT + 7) / 8 < 200 && wide_params(m_tiles, 2, 3, 4).valid) { p.wide = true; p.wn = 3; p.wk = 4; p.tn = 2; return p; }
        if (NT < 1300 && epi != EPI_SWIGLU && (NT + 2) / 3 <= 256 && (NT + 3) / 4 < 200 && wide_params(m_tiles, 1, 3, 4).valid) { p.wide = true; p.wn = 3; p.wk = 4; p.tn = 1; return p; }
        p.wn = NT >= 1300 ? 4 : 2;
        if (m_tiles >= 5 && !wide_params(m_tiles, 2, p.wn, 8 / p.wn).valid) p.wn = 4;      // (seven, eight row tiles)
        p.wk = 8 / p.wn;
        if (m_tiles >= 5 && wide_params(m_tiles, 2, p.wn, p.wk).valid) { p.wide = true; p.tn = 2; return p; }
    }
    // Streaming form.  A workgroup's k-tile brings tn weight tiles (wb / 16 KiB each) and 2 tm activation fragments
    // of 1 KiB through the CU's 64 bytes per clock and issues 2 tm tn MFMAs of 16 cycles on four SIMDs (one half
    // KiB's time each); a CU holds one workgroup, so a launch runs in rounds of 256.
    // Split-K partials cost a round trip through memory.  All in units of 1/16 KiB through one CU.
    static const int kStore[] = {1, 2, 3, 4, 6, 8, 0}, kResid[] = {1, 2, 4, 5, 8, 0}, kSwiglu[] = {2, 4, 6, 8, 0};
    long best = -1;
    const int ms0 = (m_tiles + 5) / 6, ms1 = (m_tiles + 1) / 2 < ms0 + 3 ? (m_tiles + 1) / 2 : ms0 + 3;
    for (int ms = ms0; ms <= ms1; ++ms) {
        const int tm = (m_tiles + ms - 1) / ms;
        if ((m_tiles + tm - 1) / tm != ms) continue;      // (a share would be empty)
        for (const int *t = epi == EPI_STORE ? kStore : epi == EPI_RESID ? kResid : kSwiglu; *t; ++t) {
            const int groups = (NT + *t - 1) / *t;
            const int wgs = (ms > 1 ? (groups + 7) / 8 * 8 : groups) * ms;
            for (int sk = 1; sk <= 4; ++sk) {
                const int kt = (KT + sk - 1) / sk;
                if (sk > 1 && (kt < 16 || (size_t)sk * M * NT * 16 > part_floats || groups * ms > kMaxGemmCounters)) continue;
                const int in = *t * wb + 32 * tm, mfma = 8 * *t * tm;
                const long rounds = ((long)wgs * sk + 255) / 256;
                const long cost = rounds * ((long)kt * (in > mfma ? in : mfma) + 16 * 200) + (sk > 1 ? 16 * (300 + 4 * sk * tm * *t) : 0);
                if (best < 0 || cost < best) { best = cost; p.tm = tm; p.ms = ms; p.tn = *t; p.sk = sk; }
            }
        }
    }
    return p;
}

}  // namespace

int launch_gemm_bf16(GemmArgs a, int epi, hipStream_t st) {
    const int wb = a.w_mx != nullptr ? 4 : a.w_scale != nullptr ? 8 : 16;
    if (epi == EPI_SWIGLU && a.NT % 2 != 0) {
        set_error("gemm: the SwiGLU epilogue needs paired tiles (NT=%d)", a.NT);
        return SEED_E_INVALID_ARG;
    }
    const GemmPlan p = gemm_plan(a.NT, a.KT, epi, a.M, wb, a.part_floats);
    a.MS = p.ms;
    a.SK = p.sk;
    // (the rotated walk only while the whole activation matrix -- hi and lo halves of every row -- stays in an XCD's 4
    // MiB L2 next to the weight stream: workgroups at different k positions read different parts of it; at 384 rows
    // and more the rotation cost the narrow outputs 25-45 %)
    const bool rotate = (size_t)((a.M + 15) / 16) * 16 * a.KT * 32 * 4 <= ((size_t)2 << 20);
    if (p.wide) {
        a.rot = rotate ? kRotationGroups : 0;
        switch (p.tm) {
            case 3: return launch_wide<3>(a, epi, p.wn, p.wk, p.tn, st);
            case 4: return launch_wide<4>(a, epi, p.wn, p.wk, p.tn, st);
            case 5: return launch_wide<5>(a, epi, p.wn, p.wk, p.tn, st);
            case 6: return launch_wide<6>(a, epi, p.wn, p.wk, p.tn, st);
            case 7: return launch_wide<7>(a, epi, p.wn, p.wk, p.tn, st);
            case 8: return launch_wide<8>(a, epi, p.wn, p.wk, p.tn, st);
            default:
                set_error("gemm: the wide form runs three to eight row tiles, not %d", p.tm);
                return SEED_E_INVALID_ARG;
        }
    }
    a.rot = rotate ? kRotation : 0;
    const int units = wb == 16 ? a.KT : (a.KT + 1) / 2;
    a.kt_per_split = (units + p.sk - 1) / p.sk;
    a.SK = (units + a.kt_per_split - 1) / a.kt_per_split;
    const int groups = (a.NT + p.tn - 1) / p.tn;
    const dim3 grid(p.ms > 1 ? (groups + 7) / 8 * 8 * p.ms : groups, a.SK);
    if ((size_t)(units + 1) * 1024 * p.tn >= ((size_t)1 << 31)) {
        set_error("gemm: %d k-tiles exceed the 31-bit offsets of the weight loads", a.KT);
        return SEED_E_CAPACITY;
    }
    return wb == 4 ? launch_gemm_stream_w4(a, epi, p.tm, p.tn, grid, st)
         : wb == 8 ? launch_gemm_stream_w8(a, epi, p.tm, p.tn, grid, st) : launch_gemm_stream_w16(a, epi, p.tm, p.tn, grid, st);
}

int launch_pack_weight8(const void *codes, const float *scale, void *dst, float *scale_dst, int n_rows, int K,
                        int dst_tile0, int dst_tile_step, hipStream_t st) {
    const int n_tiles = n_rows / 16, KT = K / 32;
    const size_t total = (size_t)n_tiles * ((KT + 1) / 2) * 128;
    hipLaunchKernelGGL(pack_weight8_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const uint8_t *)codes, (uint2 *)dst, n_tiles, K, KT, dst_tile0, dst_tile_step);
    hipLaunchKernelGGL(pack_scale_kernel, dim3((n_rows + 255) / 256), dim3(256), 0, st, scale, scale_dst, n_rows,
                       dst_tile0, dst_tile_step);
    return hip_fail(hipGetLastError(), "pack launch");
}

int launch_pack_weight4(const void *codes, const void *mx_scale, void *dst, void *scale_dst, int n_rows, int K,
                        int dst_tile0, int dst_tile_step, hipStream_t st) {
    const int n_tiles = n_rows / 16, KT = K / 32;
    const size_t total = (size_t)n_tiles * ((KT + 1) / 2) * 128;
    hipLaunchKernelGGL(pack_weight4_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const uint8_t *)codes, (uint32_t *)dst, n_tiles, K, KT, dst_tile0, dst_tile_step);
    hipLaunchKernelGGL(pack_mx_scale_kernel, dim3((unsigned)(((size_t)n_rows * ((KT + 1) / 2) * 2 + 255) / 256)), dim3(256), 0, st,
                       (const uint8_t *)mx_scale, (uint8_t *)scale_dst, n_rows, KT, dst_tile0, dst_tile_step);
    return hip_fail(hipGetLastError(), "pack launch");
}

int launch_pack_weight(const void *W, void *dst, int n_rows, int K, int dst_tile0, int dst_tile_step,
                       hipStream_t st) {
    const int n_tiles = n_rows / 16, KT = K / 32;
    const size_t total = (size_t)n_tiles * KT * 64;
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const uint16_t *)W, (u32x4 *)dst, n_tiles, K, KT, dst_tile0, dst_tile_step);
    return hip_fail(hipGetLastError(), "pack launch");
}

}  // namespace seedv
