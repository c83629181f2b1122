// The passes on ring blocks, one event per wavefront (a part of its shapes; one source file each, so that they compile side by side).
#include "jpet_rings_loglik.h"

namespace jpet {
template struct Rings<1222>;
template struct Rings<1228>;
template struct Rings<1236>;
}  // namespace jpet
