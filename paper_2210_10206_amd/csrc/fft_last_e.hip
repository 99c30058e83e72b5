// Fused last pass + contraction: instantiations for lengths 512 and 1024, both register-resident
// with an LDS region per live bin (512 = 16 x 8 x 4 stages, 32 threads per pencil; 1024 = 16 x 16 x 4
// stages, 64 threads per pencil; up to 16 bins, split-BF16 at 1024 up to 12).
#include "fft_last.h"

namespace sb {

template <> hipError_t launch_last_for<512>(const LastArgs &a, hipStream_t s) {
    return fftlast::launch_last_rs<512, 16, 8, 4>(a, s);
}
template <> int last_rows<512>(int) { return 1; }

template <> hipError_t launch_last_for<1024>(const LastArgs &a, hipStream_t s) {
    return fftlast::launch_last_rs<1024, 16, 16, 4>(a, s);
}
template <> int last_rows<1024>(int) { return 1; }

}  // namespace sb
