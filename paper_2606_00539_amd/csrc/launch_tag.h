// The tags that tell one launch's words from those of another (k123_step.hip).
// `launches` is a word on the device, 0 at first: a launch's workgroups read it,
// and its workgroup 0 replaces it at the end.
#pragma once

#include <stdint.h>

namespace gnmr {

// The tag of a launch that finds `launches`; never the tag of the launch before,
// which is the one in the words.
constexpr uint32_t tag_of(uint32_t launches) { return launches + 1; }

// A launch that did not wait for all of its words leaves this.  Its other
// workgroups may then still be to start, and read `launches` after it was
// replaced: whatever tag they took from it, a later launch would take for its own.
// So from there on no word is written or accepted.
constexpr uint32_t kWordsLost = uint32_t(1) << 31;

constexpr bool words_lost(uint32_t tag) { return (tag & kWordsLost) != 0; }

// What a launch of that tag leaves in `launches`.
constexpr uint32_t launches_after(uint32_t tag, bool all_arrived) {
  return !all_arrived ? kWordsLost : words_lost(tag + 1) ? 0 : tag;
}

}  // namespace gnmr
