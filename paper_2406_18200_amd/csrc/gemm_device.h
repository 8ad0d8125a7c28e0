// Device helpers shared by the projection kernels (gemm_stream.h, gemm_bf16.hip).
#pragma once
#include "seed_internal.h"
#include "device_utils.h"

namespace seedv {
namespace {

__device__ __forceinline__ void pin_args(const GemmArgs &a) {
    asm volatile("" ::"s"(a.Wp), "s"(a.Xp), "s"(a.NT), "s"(a.KT), "s"(a.kt_per_split), "s"(a.SK), "s"(a.M),
                 "s"(a.part), "s"(a.counters), "s"(a.out), "s"(a.ld_out), "s"(a.ssq_in), "s"(a.NT_in), "s"(a.x),
                 "s"(a.gain), "s"(a.act_out), "s"(a.KT_out), "s"(a.ssq), "s"(a.eps), "s"(a.MS), "s"(a.w_scale));
}

// 8-bit weights (context dtype SEED_DTYPE_BF16_W8): the same tiles with one byte per weight, an OCP e4m3 code
// (sign, 4 exponent bits of bias 7, 3 mantissa bits; no infinities), and one float scale per output feature:
// two consecutive k-tiles of an n-tile are 1 KiB, lane l holding the 8 codes of W[nt*16 + l%16][kt*32 + 8*(l/16) .. +8]
// of the first, then of the second.  Half the bytes cross HBM; on the way into the MFMA every code is widened to the bf16 of the same value (exact: three
// mantissa bits) with the hardware's packed fp8 -> float32 conversion, and the scale multiplies the finished fp32 sums
// once, in the epilogue.
__device__ __forceinline__ bf16x8 widen_e4m3(u32x2 c) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t src = (i < 2) ? c[0] : c[1];
        const auto f = (i & 1) ? __builtin_amdgcn_cvt_pk_f32_fp8(src, true) : __builtin_amdgcn_cvt_pk_f32_fp8(src, false);
        // the bf16 of a float32 that has at most four significant bits is its upper half
        r[i] = (__float_as_uint(f[0]) >> 16) | (__float_as_uint(f[1]) & 0xffff0000u);
    }
    return __builtin_bit_cast(bf16x8, r);
}

// 4-bit weights (context dtype SEED_DTYPE_BF16_W4): the OCP microscaling format MXFP4 -- elements are E2M1 codes
// (sign, two exponent bits, one mantissa bit: 0, 0.5, 1, 1.5, 2, 3, 4, 6), every 32 consecutive inputs of an output
// feature share a power-of-two scale stored as an E8M0 byte (2^(e - 127)).  A k-tile is exactly one such block per
// row: two consecutive k-tiles of an n-tile are 512 bytes of codes, lane l holding the 8 codes of
// W[nt*16 + l%16][kt*32 + 8*(l/16) .. +8] of the first, then of the second (input k in the low nibble of byte k/2 for
// even k), plus 32 scale bytes in a separate array [nt][pair][16 rows][2].
// On the way into the MFMA a code pair becomes a bf16 pair with the hardware's scaled conversion (exact: one
// mantissa bit times a power of two), so the kernel computes with exactly the values the codes stand for.
__device__ __forceinline__ bf16x8 widen_mxfp4(uint32_t c, uint32_t e8m0) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const float scale = __uint_as_float(e8m0 << 23);
    u32x4 r;
    const bf16x2_t p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, scale, 0);
    const bf16x2_t p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, scale, 1);
    const bf16x2_t p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, scale, 2);
    const bf16x2_t p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, scale, 3);
    r[0] = __builtin_bit_cast(uint32_t, p0);
    r[1] = __builtin_bit_cast(uint32_t, p1);
    r[2] = __builtin_bit_cast(uint32_t, p2);
    r[3] = __builtin_bit_cast(uint32_t, p3);
    return __builtin_bit_cast(bf16x8, r);
}

// Which column group and which share of the rows this workgroup works on.  With MS > 1 the rows of a step are
// split over MS workgroups per column group (TM row tiles each): every workgroup then reads only its own rows'
// activations and takes MS times the columns instead.  The MS workgroups of a column group read the same weights; they are laid out so that they run on the
// SAME XCD at the same time (workgroups go to the eight XCDs round robin in launch order, so ids L and L + 8 are
// neighbours in time on one XCD): the second request finds the line in that XCD's L2 and HBM is still read once.
// The grid is rounded up to whole rounds of eight column groups; padding workgroups return at once.
__device__ __forceinline__ bool wg_coords(const GemmArgs &a, int tiles_per_wg, int &cg, int &mh) {
    cg = blockIdx.x;
    mh = 0;
    if (a.MS > 1) {
        const int L = blockIdx.x;
        mh = (L >> 3) % a.MS;
        cg = (L / (8 * a.MS)) * 8 + (L & 7);
    }
    return cg * tiles_per_wg < a.NT;
}

__device__ __forceinline__ void store_act4(uint16_t *act, int row, int col0, int KT, const float *v) {
    uint16_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_bf16(v[i], hi[i], lo[i]);
    uint16_t *dst = act + packed_offset(row, col0, KT);
    uint2 wh = {(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
    uint2 wl = {(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
    *reinterpret_cast<uint2 *>(dst) = wh;
    *reinterpret_cast<uint2 *>(dst + kActLoOffset) = wl;
}

}  // namespace
}  // namespace seedv
