#include "front_impl.hpp"

namespace hlq {

template struct FrontLaunch<bf16_t, 32>;

}  // namespace hlq
