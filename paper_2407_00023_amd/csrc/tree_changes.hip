// The changes of the host's radix tree, written into its device mirror (pa_tree_upload).
//
// A round of a serving loop admits and evicts some tens of requests and so changes some tens of places of the mirror: token and
// slot runs, entries of the two indexes, a few kilobytes in all.  As copies of their own, one after the other on the stream, they
// held up the match behind them by several microseconds each; here one launch reads them from the pinned transfer buffer, a
// workgroup per piece, its words and where they belong asked for together - one round trip over the bus for all of them.
#include "common.h"

namespace pa {

__global__ __launch_bounds__(kChangeWords) void apply_changes_kernel(const ChangePiece* __restrict__ piece, const uint32_t* __restrict__ words,
                                                                     uint32_t* __restrict__ mirror) {
    const uint32_t w = words[static_cast<size_t>(blockIdx.x) * kChangeWords + threadIdx.x];
    const ChangePiece p = piece[blockIdx.x];
    if (threadIdx.x < p.words) mirror[p.to + threadIdx.x] = w;
}

int launch_apply_changes(const ChangePiece* piece, const uint32_t* words, int n, void* mirror, hipStream_t stream) {
    hipLaunchKernelGGL(apply_changes_kernel, dim3(static_cast<unsigned>(n)), dim3(kChangeWords), 0, stream, piece, words, static_cast<uint32_t*>(mirror));
    PA_HIP(hipGetLastError());
    return PA_OK;
}

}  // namespace pa
