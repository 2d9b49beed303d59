// luna_chunk_key.hip -- the key pass of the chunked attention kernel.
#include "luna_chunk_kernel.hpp"

namespace luna {

hipError_t launch_chunk_key(Dt dt, int d, const ChunkArgs& a, hipStream_t s) {
  return chunk_launch_p<kPassKey>(dt, d, a, s);
}

}  // namespace luna
