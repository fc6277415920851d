// FP32 passes of the lengths without instantiated kernels (fft_any.h).
#include "fft_any.h"

namespace csipm {
namespace fftk {

CSIPM_ANY(float)

}  // namespace fftk
}  // namespace csipm
