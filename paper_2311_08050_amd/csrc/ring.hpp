// Places in the descriptor upload ring (host bookkeeping only; the device array and
// its pinned image belong to Ctx).
//
// Uploads take consecutive places.  A place holds its bytes until the ring comes round
// to it again: at its end the ring waits for every reader enqueued so far and starts
// over.  A pointer is kept across later uploads (a pass uploads its thetas, then every
// factorisation's descriptors), so each place has a lifetime in uploaded bytes: at
// least 3 / 4 of the ring, whether the upload was copied or found among the latest.
// Reuse without that limit would hand out places the ring is about to overwrite.
#pragma once
#include <cstddef>
#include <cstring>
#include <vector>

namespace inla {

struct UploadRing {
  size_t size = 0, off = 0;
  struct Recent {
    size_t off, bytes;
    const void *stream;
  };
  std::vector<Recent> recent;   // the latest uploads since the ring last started over

  // The same bytes uploaded on the same stream while no more than a quarter of the ring
  // (uploads of any kind) ago: their offset.  `host` is the ring's image.
  bool find(const char *host, const void *src, size_t bytes, const void *stream, size_t &at) const {
    for (const Recent &r : recent)
      if (r.bytes == bytes && r.stream == stream && off - r.off <= size / 4 &&
          std::memcmp(host + r.off, src, bytes) == 0) {
        at = r.off;
        return true;
      }
    return false;
  }
  bool fits(size_t padded) const { return off + padded <= size; }
  void start_over() {
    off = 0;
    recent.clear();
  }
  // The next place, for bytes that may be found again (`keep`) or not.
  size_t take(size_t padded, size_t bytes, const void *stream, bool keep) {
    const size_t at = off;
    if (keep) {
      if (recent.size() >= 8) recent.erase(recent.begin());
      recent.push_back({at, bytes, stream});
    }
    off += padded;
    return at;
  }
};

}  // namespace inla
