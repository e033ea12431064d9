// Shared block and suffix in one launch, one query row per KV head, head dimension 128; the source is combined_impl.h.
#define HG_WIDE_D 128
#include "combined_impl.h"
