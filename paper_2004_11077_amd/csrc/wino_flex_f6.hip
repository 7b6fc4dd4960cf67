// Flex kernels for F(6x6, 3x3).
#include "wino_flex_calibrate.hpp"

namespace wino {
template struct PerMFlex<6>;
}  // namespace wino
