// Weight-streaming projection kernel for steps of few rows:  Y[M][Nout] = X[M][K] . W[Nout][K]^T, M <= 96 rows per
// workgroup (more rows run as row shares), bf16 / one-byte / four-bit weights, fp32 accumulation on the MFMA units,
// with the row-wise work that follows each projection fused into its epilogue.
//
// What bounds it: every weight is used by M rows only, so the floor of a launch is its weight bytes at the rate a long
// streaming read reaches (6.1 - 6.3 TB/s).  The design keeps everything else below that:
//   * All NW wavefronts of a workgroup work on the SAME TN n-tiles (16 output features each) and split K between them,
//     k-tile by k-tile.  Every activation fragment is then used by exactly one wavefront of the workgroup, so it goes
//     straight from L2 to that wavefront's registers: no LDS staging and no barrier in the k loop -- the wavefronts
//     are independent streams until their partial tiles are summed through LDS at the end.
//   * A CU's path from L2 (64 bytes per clock) carries TN weight tiles and 2 TM activation fragments (hi and lo halves
//     of TM row tiles) per k-tile, so TN is as large as leaves one round of workgroups over the 256 CUs
//     (stream_pick); narrow outputs, which have too few n-tiles for that, are split along K across SK workgroups.
//   * Each wavefront keeps a ring of D k-tiles (weights and activations) in registers on their way: 48 .. 128 KiB of
//     weights in flight per CU.  Five row tiles and more run with four wavefronts (one per SIMD) that own 512 registers each, so
//     that a deep ring still fits beside the accumulators.
//   * Loads are raw buffer loads: a k-tile past the end of the range gets an offset past the buffer's end, which
//     returns zeros without a memory access, so ragged ranges need neither branches nor clean-up code, and a
//     wavefront needs one address register per k-tile instead of two per load.
// Weight layout: fragment tiles (nt, kt) of 16 features x 32 inputs, lane l holding W[nt*16 + l%16][kt*32 + 8*(l/16)
// .. +8], all k-tiles of an n-tile contiguous; narrow weights in pairs of k-tiles (see pack_weight8 / pack_weight4).
// v_mfma_f32_16x16x32_bf16 computes Y^T tiles: D[i = feature][j = token row]; activations are hi/lo pairs of bf16
// values (two MFMAs per weight fragment), so that their rounding does not pile up over 32 - 40 layers.
#pragma once
#include "gemm_device.h"

namespace seedv {
namespace {

// Raw buffer resource over [base, base + bytes): out-of-range offsets read as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}
constexpr unsigned kPastEnd = 0x80000000u;     // an offset past the end of every buffer (all are below 2 GiB)
constexpr int kNonTemporal = 2;                // cache policy bit of the buffer loads

template <int TM, int TN, int NW, int WB>
struct StreamShape {
    static constexpr int U = WB == 16 ? 1 : 2;                        // k-tiles per unit (one weight load per n-tile)
    static constexpr int kUnitBytes = U * 64 * WB;                    // of an n-tile: 1024 / 1024 / 512
    static constexpr int kAcc = 4 * TN * TM;
    static constexpr int kWRegs = WB == 4 ? 3 : 4;                    // per n-tile and unit (four-bit: codes + scales)
    static constexpr int kPer = TN * kWRegs + U * TM * 8;             // registers of a unit in flight
    static constexpr int kLoads = TN * (WB == 4 ? 2 : 1) + U * TM * 2;
    static constexpr int kRegs = NW == 8 ? 256 : 512;
    static constexpr int kFit = (kRegs - kAcc - 32) / kPer;
    static constexpr int kCount = 60 / kLoads;                        // (vmcnt is a 6-bit counter)
    static constexpr int kMin = kFit < kCount ? kFit : kCount;
    static constexpr int D = kMin < 1 ? 1 : (kMin > 16 ? 16 : (kMin > 8 && kMin < 16 ? 8 : kMin));
};

template <int TM, int TN, int NW, int EPI, int WB>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void gemm_stream_kernel(GemmArgs a) {
    using S = StreamShape<TM, TN, NW, WB>;
    constexpr int U = S::U, D = S::D;
    constexpr int UZ = EPI == EPI_SWIGLU ? 2 : 1;                     // tiles of an epilogue unit (gate and up together)
    constexpr int PN = TN / UZ;                                       // ... units per row tile
    constexpr int UNITS = TM * PN;
    constexpr int UPW = (UNITS + NW - 1) / NW;                        // units a wavefront finishes
    constexpr int kPerRound = 128 / (NW * UZ * NW) > 0 ? 128 / (NW * UZ * NW) : 1;   // units per wavefront and LDS round
    constexpr int RU = kPerRound * NW < UNITS ? kPerRound * NW : UNITS;   // units per round: at most 128 KiB of partials
    __shared__ __attribute__((aligned(16))) f32x4 red[NW][RU * UZ][64];
    __shared__ int s_last;
    __shared__ float s_rinv[TM * 16];
    pin_args(a);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int cg, mh;
    if (!wg_coords(a, TN, cg, mh)) return;               // (uniform: a padding workgroup of a launch with row shares)
    const int KT = a.KT, KU = (KT + U - 1) / U;          // k-tiles, units of the whole matrix
    const int u0 = blockIdx.y * a.kt_per_split, n = min(KU, u0 + a.kt_per_split) - u0;   // this workgroup's units
    const int n_iter = (n + NW - 1) / NW;
    const int nt0 = cg * TN, nt_here = min(TN, a.NT - nt0);
    const int mt0 = mh * TM, mt_here = min(TM, (a.M + 15) / 16 - mt0);
    const int g = lane >> 4, rlow = lane & 15;

    const unsigned ntile_bytes = (unsigned)KU * S::kUnitBytes, mtile_bytes = (unsigned)KT * 2048u;
    const auto wr = make_rsrc((const char *)a.Wp + (size_t)nt0 * ntile_bytes, (unsigned)nt_here * ntile_bytes);
    const auto xr = make_rsrc((const char *)a.Xp + (size_t)mt0 * mtile_bytes, (unsigned)mt_here * mtile_bytes);
    const unsigned nscale_bytes = (unsigned)KU * 32u;
    const auto sr = make_rsrc(WB == 4 ? (const char *)a.w_mx + (size_t)nt0 * nscale_bytes : (const char *)a.Wp, WB == 4 ? (unsigned)nt_here * nscale_bytes : 0u);
    unsigned wso[TN], sso[TN], xso[TM];                  // (a ragged last group repeats its last tile: never stored)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        wso[tn] = (unsigned)min(tn, nt_here - 1) * ntile_bytes;
        sso[tn] = (unsigned)min(tn, nt_here - 1) * nscale_bytes;
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) xso[tm] = (unsigned)min(tm, mt_here - 1) * mtile_bytes;

    // Column groups start their walk at different places of the k range (wrapping around): workgroups that start
    // together would otherwise all read the same k position, whose weight tiles lie on few memory channels.
    const int rot = n > 0 ? (cg * a.rot) % n : 0;
    struct Slot {
        u32x4 w[TN];
        uint32_t e[WB == 4 ? TN : 1];
        bf16x8 x[U][TM][2];
    };
    Slot ring[D];
    // unit of virtual position v (i-th of this wavefront: v = i * NW + w), or "past the end"
    auto unit_of = [&](int i, int &u) {
        const int v = i * NW + w, vv = v + rot;
        u = u0 + (vv >= n ? vv - n : vv);
        return v < n;
    };
    auto load_w = [&](Slot &s, int i) {
        int u;
        const bool ok = unit_of(i, u);
        const unsigned wl = (ok ? (unsigned)u * S::kUnitBytes : kPastEnd) + (unsigned)lane * (S::kUnitBytes / 64);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            if constexpr (WB == 4) {
                const u32x2 c = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(wr, wl, wso[tn], kNonTemporal));
                s.w[tn][0] = c[0];
                s.w[tn][1] = c[1];
                s.e[tn] = __builtin_amdgcn_raw_buffer_load_b16(sr, (ok ? (unsigned)u * 32u : kPastEnd) + (unsigned)rlow * 2u, sso[tn], 0);
            } else {
                s.w[tn] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, wl, wso[tn], kNonTemporal));
            }
        }
    };
    auto load_x = [&](Slot &s, int i) {
        int u;
        const bool ok = unit_of(i, u);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int kt = u * U + q;
            const unsigned xl = (ok && (U == 1 || kt < KT) ? (unsigned)kt * 2048u : kPastEnd) + (unsigned)lane * 16u;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                s.x[q][tm][0] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(xr, xl, xso[tm], 0));
                s.x[q][tm][1] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(xr, xl + 1024u, xso[tm], 0));
            }
        }
    };
    f32x4 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const Slot &s) {
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                bf16x8 wf;
                if constexpr (WB == 16) wf = __builtin_bit_cast(bf16x8, s.w[tn]);
                else if constexpr (WB == 8) wf = widen_e4m3((u32x2){s.w[tn][2 * q], s.w[tn][2 * q + 1]});
                else wf = widen_mxfp4(s.w[tn][q], (s.e[tn] >> (8 * q)) & 0xffu);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    acc[tn][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, s.x[q][tm][1], acc[tn][tm], 0, 0, 0);
                    acc[tn][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, s.x[q][tm][0], acc[tn][tm], 0, 0, 0);
                }
            }
    };
    // The last round requests no weights.  What the epilogue needs from memory is requested ahead of its MFMAs: the
    // sums of squares of (some of) the input rows, or this wavefront's residual rows and the next norm's gains.
    constexpr bool kNorm = EPI != EPI_RESID;
    constexpr int kRowsPerWave = TM * 16 / NW;
    constexpr int kRB = kRowsPerWave < 8 ? kRowsPerWave : kRowsPerWave % 8 == 0 ? 8 : 5;   // rows per batch
    const int rbase = mh * TM * 16, r_hi = min(a.M, rbase + TM * 16);
    const bool norm = kNorm && a.ssq_in != nullptr;
    const bool norm_fast = norm && a.NT_in <= 512 && (a.NT_in & 3) == 0;
    f32x4 sv[kRB][2];
    auto ssq_request = [&](int batch) {
        // (without the fast path the loads read the start of the activation buffer and are dropped)
        const float *sp = norm_fast ? a.ssq_in : reinterpret_cast<const float *>(a.Xp);
        const int nt_in = norm_fast ? a.NT_in : 4;
#pragma unroll
        for (int r = 0; r < kRB; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int row = norm_fast ? min(rbase + w + (batch * kRB + r) * NW, r_hi - 1) : 0, t = 4 * lane + 256 * h;
                const u32x4 v = *reinterpret_cast<const u32x4 *>(sp + (size_t)row * nt_in + (t < nt_in ? t : 0));
                sv[r][h] = __builtin_bit_cast(f32x4, v & (t < nt_in ? 0xffffffffu : 0u));
            }
    };
    auto ssq_finish = [&](int batch) {
#pragma unroll
        for (int r = 0; r < kRB; ++r) {
            const f32x4 q = sv[r][0] + sv[r][1];
            const float ssum = wave_reduce_sum_dpp((q[0] + q[1]) + (q[2] + q[3]));
            s_rinv[w + (batch * kRB + r) * NW] = 1.0f / sqrtf(ssum / (float)(a.NT_in * 16) + a.eps);   // (rows past the last: unused)
        }
    };
    const int ld_part = a.NT * 16;
    f32x4 x_pre[UPW];
    uint2 gain_pre[UPW];
    auto resid_request = [&]() {
#pragma unroll
        for (int k = 0; k < UPW; ++k) {
            const int u = min(w + k * NW, UNITS - 1), tm = u / PN, tn = u - tm * PN;
            const int col = min(nt0 + tn, a.NT - 1) * 16 + 4 * g, row = min(rbase + tm * 16 + rlow, a.M - 1);
            x_pre[k] = *reinterpret_cast<const f32x4 *>(a.x + (size_t)row * ld_part + col);
            gain_pre[k] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(a.gain) + col);
        }
    };
    auto stream = [&](auto depth_tag) {
        constexpr int DD = decltype(depth_tag)::value;
        // Narrow tiles: all weights of the first round ahead of its activations, whose way is shorter (4096 x 4096 at 12
        // rows 12.1 -> 10.3 us); with many activations in flight that starves the first MFMAs instead (22016 x 4096
        // at 40 rows 38.6 -> 41.2 us).
        constexpr bool kWeightsFirst = TN <= 2 || (TN == 3 && TM <= 2);
#pragma unroll
        for (int d = 0; d < DD; ++d) {
            load_w(ring[d], d);
            if constexpr (!kWeightsFirst) load_x(ring[d], d);
        }
        if constexpr (kWeightsFirst) {
#pragma unroll
            for (int d = 0; d < DD; ++d) load_x(ring[d], d);
        }
        for (int i = 0; i + DD < n_iter; i += DD) {
#pragma unroll
            for (int d = 0; d < DD; ++d) {
                compute(ring[d]);
                load_w(ring[d], i + DD + d);
                load_x(ring[d], i + DD + d);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (kNorm) ssq_request(0);
        else resid_request();
#pragma unroll
        for (int d = 0; d < DD; ++d) compute(ring[d]);
    };
    // (a ring much deeper than a short range would mostly issue loads past its end)
    if (D > 4 && n_iter <= 4) stream(std::integral_constant<int, (D > 4 ? 4 : D)>{});
    else if (D > 8 && n_iter <= 8) stream(std::integral_constant<int, (D > 8 ? 8 : D)>{});
    else stream(std::integral_constant<int, D>{});
    if constexpr (kNorm) {
        if (norm_fast) {
            ssq_finish(0);
#pragma unroll
            for (int b = 1; b * kRB < kRowsPerWave; ++b) {
                ssq_request(b);
                ssq_finish(b);
            }
        } else if (norm) {
            for (int row = rbase + w; row < r_hi; row += NW) {
                float ssum = 0.f;
                for (int t = lane; t < a.NT_in; t += 64) ssum += a.ssq_in[(size_t)row * a.NT_in + t];
                ssum = wave_reduce_sum(ssum);
                s_rinv[row - rbase] = 1.0f / sqrtf(ssum / (float)(a.NT_in * 16) + a.eps);
            }
        }
    }

    // Sum the NW partial tiles through LDS in a fixed order; every wavefront finishes its share of the units (unit u
    // = row tile u / PN, n-tile (pair) u % PN goes to wavefront u % NW).
    f32x4 mine[UPW][UZ];
#pragma unroll
    for (int k0 = 0; k0 < UPW; k0 += kPerRound) {
        if (k0 > 0) __syncthreads();                      // the previous round has been read
#pragma unroll
        for (int ul = 0; ul < RU; ++ul) {
            const int u = k0 * NW + ul;
            if (u < UNITS) {
#pragma unroll
                for (int z = 0; z < UZ; ++z) red[w][ul * UZ + z][lane] = acc[(u % PN) * UZ + z][u / PN];
            }
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kPerRound; ++kk) {
            if (k0 + kk >= UPW) break;
            const int ul = min(w + kk * NW, RU - 1);
#pragma unroll
            for (int z = 0; z < UZ; ++z) {
                f32x4 s = red[0][ul * UZ + z][lane];
#pragma unroll
                for (int i = 1; i < NW; ++i) s += red[i][ul * UZ + z][lane];
                mine[k0 + kk][z] = s;
            }
        }
    }

    auto unit_at = [&](int k, int &tm, int &tn, int &row, int &col) {     // false: nothing to store
        const int u = w + k * NW;
        tm = min(u, UNITS - 1) / PN;
        tn = (min(u, UNITS - 1) - tm * PN) * UZ;
        row = rbase + tm * 16 + rlow;
        col = (nt0 + tn) * 16 + 4 * g;
        return u < UNITS && tn < nt_here;
    };
    if (a.SK > 1) {
        // Split along K across workgroups: publish the partial tiles; the last workgroup of this column group sums
        // all partials in a fixed order, each wavefront its own units, and runs the epilogue.
        const size_t ps = (size_t)a.M * ld_part;
#pragma unroll
        for (int k = 0; k < UPW; ++k) {
            int tm, tn, row, col;
            if (unit_at(k, tm, tn, row, col) && row < a.M)
#pragma unroll
                for (int z = 0; z < UZ; ++z)
                    store4_agent(a.part + (size_t)blockIdx.y * ps + (size_t)row * ld_part + col + 16 * z, mine[k][z]);
        }
        if (!arrive_last(&a.counters[cg * a.MS + mh], a.SK, &s_last)) return;
        constexpr int kBatch = 4;
#pragma unroll
        for (int k = 0; k < UPW; ++k) {
            int tm, tn, row, col;
            (void)unit_at(k, tm, tn, row, col);
            const float *pp = a.part + (size_t)min(row, a.M - 1) * ld_part + min(col, ld_part - 16 * UZ + 4 * g);
#pragma unroll
            for (int z = 0; z < UZ; ++z) {
                f32x4 p[kBatch];
#pragma unroll
                for (int sk = 0; sk < kBatch; ++sk) p[sk] = load4_agent(pp + 16 * z + (size_t)min(sk, a.SK - 1) * ps);
                f32x4 s = p[0];
#pragma unroll
                for (int sk = 1; sk < kBatch; ++sk)
                    if (sk < a.SK) s += p[sk];
                mine[k][z] = s;
            }
        }
    }

#pragma unroll
    for (int k = 0; k < UPW; ++k) {
        int tm, tn, row, col;
        const bool here = unit_at(k, tm, tn, row, col);   // (uniform over the wavefront)
        if (!here) continue;
        const bool valid = row < a.M;
        if constexpr (WB == 8) {
            // one scale per output feature: lane group g holds features 4g .. 4g + 3
#pragma unroll
            for (int z = 0; z < UZ; ++z) mine[k][z] *= *reinterpret_cast<const f32x4 *>(a.w_scale + col + 16 * z);
        }
        if constexpr (EPI == EPI_STORE) {
            const float sc = norm ? s_rinv[row - rbase] : 1.f;
            if (valid) *reinterpret_cast<f32x4 *>(a.out + (size_t)row * a.ld_out + col) = mine[k][0] * sc;
        } else if constexpr (EPI == EPI_RESID) {
            float ss = 0.f;
            if (valid) {
                const f32x4 xv = x_pre[k] + mine[k][0];
                *reinterpret_cast<f32x4 *>(a.x + (size_t)row * ld_part + col) = xv;
                const uint2 gw = gain_pre[k];
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
            if (valid && g == 0) a.ssq[(size_t)row * a.NT + nt0 + tn] = ss;
        } else if (valid) {   // EPI_SWIGLU: tiles (2p, 2p + 1) = (gate, up) of feature block nt0 / 2 + p
            const float sc = s_rinv[row - rbase];
            float h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float gt = mine[k][0][i] * sc, up = mine[k][UZ - 1][i] * sc;
                h[i] = gt / (1.0f + expf(-gt)) * up;
            }
            store_act4(a.act_out, row, ((nt0 + tn) >> 1) * 16 + 4 * g, a.KT_out, h);
        }
    }
}

template <int TM, int TN, int EPI, int WB>
int launch_stream_shape(const GemmArgs &a, dim3 grid, hipStream_t st) {
    constexpr int NW = TM >= 4 ? 4 : 8;
    hipLaunchKernelGGL((gemm_stream_kernel<TM, TN, NW, EPI, WB>), grid, dim3(NW * 64), 0, st, a);
    return hip_fail(hipGetLastError(), "gemm launch");
}

template <int TM, int WB>
int launch_stream_tm(const GemmArgs &a, int epi, int tn, dim3 grid, hipStream_t st) {
#define SEEDV_TN(EPIv, TNv) if (epi == EPIv && tn == TNv) return launch_stream_shape<TM, TNv, EPIv, WB>(a, grid, st);
    SEEDV_TN(EPI_STORE, 1) SEEDV_TN(EPI_STORE, 2) SEEDV_TN(EPI_STORE, 3) SEEDV_TN(EPI_STORE, 4) SEEDV_TN(EPI_STORE, 6) SEEDV_TN(EPI_STORE, 8)
    SEEDV_TN(EPI_RESID, 1) SEEDV_TN(EPI_RESID, 2) SEEDV_TN(EPI_RESID, 4) SEEDV_TN(EPI_RESID, 5) SEEDV_TN(EPI_RESID, 8)
    SEEDV_TN(EPI_SWIGLU, 2) SEEDV_TN(EPI_SWIGLU, 4) SEEDV_TN(EPI_SWIGLU, 6) SEEDV_TN(EPI_SWIGLU, 8)
#undef SEEDV_TN
    set_error("gemm: no streaming kernel with %d n-tiles for epilogue %d", tn, epi);
    return SEED_E_INVALID_ARG;
}

template <int WB>
int launch_stream_wb(const GemmArgs &a, int epi, int tm, int tn, dim3 grid, hipStream_t st) {
    switch (tm) {
        case 1: return launch_stream_tm<1, WB>(a, epi, tn, grid, st);
        case 2: return launch_stream_tm<2, WB>(a, epi, tn, grid, st);
        case 3: return launch_stream_tm<3, WB>(a, epi, tn, grid, st);
        case 4: return launch_stream_tm<4, WB>(a, epi, tn, grid, st);
        case 5: return launch_stream_tm<5, WB>(a, epi, tn, grid, st);
        case 6: return launch_stream_tm<6, WB>(a, epi, tn, grid, st);
        default:
            set_error("gemm: the streaming kernel runs one to six row tiles, not %d", tm);
            return SEED_E_CAPACITY;
    }
}

}  // namespace
}  // namespace seedv
