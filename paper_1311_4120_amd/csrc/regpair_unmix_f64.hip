// The unmix paired pass in float64, every length of regpair.h.
#include "regpair.h"

namespace jgb {
namespace fft {

JGB_PAIR_INSTANTIATE(double, PAIR_UNMIX)

}  // namespace fft
}  // namespace jgb
