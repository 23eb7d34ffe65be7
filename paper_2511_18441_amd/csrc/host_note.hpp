// Counts of a render on their way to the host.
#pragma once

#include <stdint.h>

namespace recogs {

// Where the count scan also leaves the header's first eight words for the host: pinned
// host memory, one 64-bit word each with the call's sequence number in its upper half, so
// every word says by itself that it has arrived and no fence (a write-back of the XCD's L2)
// is needed. words null: not wanted.
struct HostNote {
    uint64_t *words;
    uint32_t seq;
};

}  // namespace recogs
