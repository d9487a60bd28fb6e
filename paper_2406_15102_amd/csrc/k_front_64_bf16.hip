#include "front_impl.hpp"

namespace hlq {

template struct FrontLaunch<bf16_t, 64>;

}  // namespace hlq
