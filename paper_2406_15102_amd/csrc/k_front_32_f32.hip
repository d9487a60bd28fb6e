#include "front_impl.hpp"

namespace hlq {

template struct FrontLaunch<float, 32>;

}  // namespace hlq
