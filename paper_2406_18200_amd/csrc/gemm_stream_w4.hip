// The streaming projection kernel for weights of 4 bits.
#include "gemm_stream.h"

namespace seedv {

int launch_gemm_stream_w4(const GemmArgs &a, int epi, int tm, int tn, dim3 grid, hipStream_t st) {
    return launch_stream_wb<4>(a, epi, tm, tn, grid, st);
}

}  // namespace seedv
