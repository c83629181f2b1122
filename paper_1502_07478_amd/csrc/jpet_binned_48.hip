// The binned passes with a register cache of 48 pixels per row.
#include "jpet_binned.h"

namespace jpet {
template struct Binned<48>;
}  // namespace jpet
