// The streaming projection kernel for weights of 8 bits.
#include "gemm_stream.h"

namespace seedv {

int launch_gemm_stream_w8(const GemmArgs &a, int epi, int tm, int tn, dim3 grid, hipStream_t st) {
    return launch_stream_wb<8>(a, epi, tm, tn, grid, st);
}

}  // namespace seedv
