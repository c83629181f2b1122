// The binned passes with a register cache of 32 pixels per row.
#include "jpet_binned.h"

namespace jpet {
template struct Binned<32>;
}  // namespace jpet
