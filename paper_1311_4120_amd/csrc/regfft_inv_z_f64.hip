// The last inverse pass (contiguous axis) in float64, every length of regfft.h.
#include "regfft.h"

namespace jgb {
namespace fft {

JGB_REG_INSTANTIATE(double, RP_INV_Z, JGB_REG_LENGTHS_F64)

}  // namespace fft
}  // namespace jgb
