// The walking form of the rotation on 16-bit terms (design and launcher in rotate_terms.hip): a translation unit of its own,
// for the time it takes to compile.
#include "rotate_terms_device.h"

hipError_t bwla_launch_rotate_terms_many(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    return launch_terms<true>(b, blocks, threads, lds, st);
}
