// Sized pencil kernels, FP64.
#include "fft_pencil.hpp"

namespace pw {

PW_INST_PENCIL(double)

}  // namespace pw
