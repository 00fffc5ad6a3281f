// The strided inverse passes in float32, every length of regfft.h.
#include "regfft.h"

namespace jgb {
namespace fft {

JGB_REG_INSTANTIATE(float, RP_INV, JGB_REG_LENGTHS_F32)

}  // namespace fft
}  // namespace jgb
