// The fused paired pass in float64, every length of regpair.h.
#include "regpair.h"

namespace jgb {
namespace fft {

JGB_PAIR_INSTANTIATE(double, PAIR_FUSED)

}  // namespace fft
}  // namespace jgb
