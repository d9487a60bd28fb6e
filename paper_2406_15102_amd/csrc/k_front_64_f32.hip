#include "front_impl.hpp"

namespace hlq {

template struct FrontLaunch<float, 64>;

}  // namespace hlq
