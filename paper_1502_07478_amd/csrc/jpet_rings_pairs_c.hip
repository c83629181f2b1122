// The passes on ring blocks, two events per wavefront (a part of its shapes; one source file each, so that they compile side by side).
#include "jpet_rings_loglik.h"

namespace jpet {
template struct Rings<314>;
template struct Rings<318>;
}  // namespace jpet
