// The binned passes with a register cache of 16 pixels per row.
#include "jpet_binned.h"

namespace jpet {
template struct Binned<16>;
}  // namespace jpet
