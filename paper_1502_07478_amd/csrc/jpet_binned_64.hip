// The binned passes with a register cache of 64 pixels per row.
#include "jpet_binned.h"

namespace jpet {
template struct Binned<64>;
}  // namespace jpet
