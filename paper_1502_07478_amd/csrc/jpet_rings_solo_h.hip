// The passes on ring blocks, one event per wavefront (a part of its shapes; one source file each, so that they compile side by side).
#include "jpet_rings_loglik.h"

namespace jpet {
template struct Rings<1454>;
}  // namespace jpet
