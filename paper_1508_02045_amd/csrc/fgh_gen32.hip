// fgh_gen32.hip -- the run-time-length passes in single precision.
#include "fgh_gen_launch.hpp"

namespace fgh {

FGH_GEN_INSTANTIATE(float)

}  // namespace fgh
