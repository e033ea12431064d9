// Shared block and suffix in one launch, one query row per KV head, head dimension 64; the source is combined_impl.h.
#define HG_WIDE_D 64
#include "combined_impl.h"
