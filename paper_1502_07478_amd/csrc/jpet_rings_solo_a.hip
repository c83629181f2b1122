// The passes on ring blocks, one event per wavefront (a part of its shapes; one source file each, so that they compile side by side).
#include "jpet_rings_loglik.h"

namespace jpet {
template struct Rings<1132>;
template struct Rings<1148>;
template struct Rings<1164>;
template struct Rings<1216>;
}  // namespace jpet
