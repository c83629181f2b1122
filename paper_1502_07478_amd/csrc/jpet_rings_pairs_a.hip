// The passes on ring blocks, two events per wavefront (a part of its shapes; one source file each, so that they compile side by side).
#include "jpet_rings_loglik.h"

namespace jpet {
template struct Rings<108>;
template struct Rings<112>;
template struct Rings<116>;
template struct Rings<124>;
template struct Rings<210>;
template struct Rings<214>;
}  // namespace jpet
