// Shared block and suffix in one launch at head dimension 128, and the launcher for both head dimensions; the source is
// combined_impl.h.
#define HG_WIDE_D 128
#include "combined_impl.h"
