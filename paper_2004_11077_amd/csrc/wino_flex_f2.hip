// Flex kernels for F(2x2, 3x3).
#include "wino_flex_calibrate.hpp"

namespace wino {
template struct PerMFlex<2>;
}  // namespace wino
