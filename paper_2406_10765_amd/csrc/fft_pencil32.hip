// Sized pencil kernels, FP32.
#include "fft_pencil.hpp"

namespace pw {

bool pencil_n_supported(int n) {
  switch (n) {
#define PW_CASE(NN, AA, BB) case NN:
    PW_PENCIL_SIZES(PW_CASE)
#undef PW_CASE
    return true;
  }
  return false;
}

PW_INST_PENCIL(float)

}  // namespace pw
