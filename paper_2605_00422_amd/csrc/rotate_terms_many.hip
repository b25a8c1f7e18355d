// The walking form of the rotation of bf16 tokens by strips (design and launcher in rotate_terms.hip): a translation unit of its
// own, for the time it takes to compile.
#include "rotate_terms_device.h"

hipError_t bwla_launch_rotate_terms_many(const RtArgs& b, RtKind kind, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    if (kind == RT_H16) return launch_v<8, 2, false, true, RT_H16, 768>(b, blocks, threads, lds, st);
    return launch_terms<true>(b, blocks, threads, lds, st);
}
