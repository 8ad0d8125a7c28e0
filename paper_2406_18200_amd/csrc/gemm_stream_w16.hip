// The streaming projection kernel for weights of 16 bits.
#include "gemm_stream.h"

namespace seedv {

int launch_gemm_stream_w16(const GemmArgs &a, int epi, int tm, int tn, dim3 grid, hipStream_t st) {
    return launch_stream_wb<16>(a, epi, tm, tn, grid, st);
}

}  // namespace seedv
