// CSR construction by parts. Internal; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "triad_internal.h"

namespace triad {

// The CSR of narcs > 0 arcs over n ids below 2^rb, as triad_csr_from_arcs
// states it, unless the sizes ask for the general sort (*done false, nothing
// done). Waits for the stream.
int csr_by_parts(int64_t n, int64_t narcs, int rb, const int32_t* src, const int32_t* dst, hipStream_t s, int64_t* off,
                 int32_t* nbr, uint8_t* flg, int64_t* nnz_out, bool* done);

}  // namespace triad
