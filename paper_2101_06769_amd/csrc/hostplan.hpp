// Decisions of the host code that need no device: plain C++, so that they can be
// compiled and tested without one.
#pragma once

#include <cstddef>
#include <cstdint>

namespace mplb {

// What the runtime says of one address of host memory: whether it is
// page-locked, where the device sees it, and the allocation or registration
// around it in device addresses.
struct HostRange {
    bool page_locked = false;
    uintptr_t device = 0, start = 0;
    size_t bytes = 0;
};

// The device address of `bytes` of host memory at `host`, or 0 where a kernel
// must not write there itself: pageable or managed memory, memory that is
// not 8-byte aligned, or a buffer that one page-locked range does not hold to
// its end.  Both ends alone say nothing: the device commonly sees page-locked
// memory at its host address, so two ranges with pageable memory between them
// look like one.  query: HostRange of an address, false where the runtime
// cannot tell.
// pending: an earlier error that the caller of the library has yet to see; nothing is
// asked then, since the answer could take that error's place.
template <class Query>
uintptr_t direct_address(uintptr_t host, size_t bytes, bool pending, Query &&query)
{
    HostRange r;
    if (pending || host % 8 != 0 || !query(host, r) || !r.page_locked || r.device == 0) return 0;
    if (r.device < r.start) return 0;
    const size_t before = r.device - r.start;
    return before <= r.bytes && bytes <= r.bytes - before ? r.device : 0;
}

}  // namespace mplb
