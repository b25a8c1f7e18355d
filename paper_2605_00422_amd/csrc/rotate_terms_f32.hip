// The rotation of fp32 tokens by strips (design and launcher in rotate_terms.hip): a translation unit of its own, for the time
// it takes to compile.
#include "rotate_terms_device.h"

hipError_t bwla_launch_rotate_terms_f32(const RtArgs& b, bool many, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    return many ? launch_terms_f32<true>(b, blocks, threads, lds, st) : launch_terms_f32<false>(b, blocks, threads, lds, st);
}
