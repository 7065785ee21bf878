// Pinned host memory that kernels read and write directly, kept by the library from its first use on: its host
// and its device address, both or neither.  A first use that fails leaves nothing behind, so the next one starts
// over and no kernel is launched on an address that was never obtained.
#pragma once
#include <stddef.h>

namespace mmee {

struct Pinned { unsigned char *host = nullptr, *map = nullptr; };

// Api: `success`, alloc(&host, bytes), address(&map, host), release(host), each returning a code of one type.
template <class Api>
auto ensure_pinned(const Api &api, Pinned &out, size_t bytes) -> decltype(api.success)
{
    if (out.map) return api.success;
    Pinned got;
    auto rc = api.alloc(&got.host, bytes);
    if (rc != api.success) return rc;
    rc = api.address(&got.map, got.host);
    if (rc != api.success) {
        (void)api.release(got.host);
        return rc;
    }
    out = got;
    return rc;
}

}  // namespace mmee
