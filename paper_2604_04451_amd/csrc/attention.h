// The default choice of chorus_attention, for callers that prepare its queries.
#pragma once

namespace chorus {

// Whether chorus_attention runs this call in 128-key tiles by default (its variants 5 and 6). The block then hands it
// pre-scaled queries (variant 6).
bool attention_wide_tiles(long Lq, long Lk, long LkPad, int H, int dh, bool factor);

}  // namespace chorus
