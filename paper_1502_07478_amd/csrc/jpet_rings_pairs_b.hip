// The passes on ring blocks, two events per wavefront (a part of its shapes; one source file each, so that they compile side by side).
#include "jpet_rings_loglik.h"

namespace jpet {
template struct Rings<218>;
template struct Rings<222>;
template struct Rings<228>;
}  // namespace jpet
