// Shared block and suffix in one launch, several query rows per KV head, head dimension 128; the source is combined_impl.h.
#define HG_WIDE_D 128
#define HG_COMBINED_TILES
#include "combined_impl.h"
