// Growth of a scratch buffer that a kernel can do with less of, or without.
#pragma once

#include <stddef.h>

namespace lsms {

// Grows b (members p, bytes) to `want` bytes.  Where there is no memory for that, a buffer that holds
// `least` bytes is kept, or else one of `least` bytes allocated, or else b stays as it is.  alloc(bytes,
// &p) and release(p) return 0, nomem (alloc only), or another error, which ends the call and is returned;
// being short of memory is no error.  A buffer is released only after its successor is there.
template <typename Buf, typename Alloc, typename Release>
int grow_scratch(Buf& b, size_t want, size_t least, int nomem, Alloc alloc, Release release) {
  const size_t sizes[2] = {want, least};
  for (size_t bytes : sizes) {
    if (b.bytes >= bytes) return 0;
    void* p = nullptr;
    const int rc = alloc(bytes, &p);
    if (rc == nomem) continue;
    if (rc != 0) return rc;
    void* const old = b.p;
    b.p = p;
    b.bytes = bytes;
    return old ? release(old) : 0;
  }
  return 0;
}

}  // namespace lsms
