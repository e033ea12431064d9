// Shared block and suffix in one launch, several query rows per KV head, head dimension 64; the source is combined_impl.h.
#define HG_WIDE_D 64
#define HG_COMBINED_TILES
#include "combined_impl.h"
