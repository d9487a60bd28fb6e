#include "front_impl.hpp"

namespace hlq {

template struct FrontLaunch<float, 16>;

}  // namespace hlq
