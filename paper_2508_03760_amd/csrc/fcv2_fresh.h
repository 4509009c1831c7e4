// fcv2_fresh.h -- the calls of include/fcv2.h for output memory that has never been written, used by the binding when it
// allocates the result itself.  Same arguments and results, and in addition every byte of the output is defined: the padding
// between a record's sections (and rows of the send buffer that no routed copy takes) is zero, row_src entries past the
// routed copies are -1.  The kernels write these few bytes along with the rest: filling the whole output beforehand costs a
// launch (2 to 3 us) and a second pass over it.
#pragma once
#include "../../include/fcv2.h"

#ifdef __cplusplus
extern "C" {
#endif
// record_stride must be the record's total_bytes
int fcv2_quantize_pack_slices_fresh(const void* x, uint64_t n, uint32_t n_slices, const fcv2_fmt_t* fmt, void* packed, void* stream);
int fcv2_reduce_requant_fresh(const void* const* peers, int n_peers, uint64_t n, const fcv2_fmt_t* fmt_in, const fcv2_fmt_t* fmt_out,
                              void* packed_out, float* sum_out, void* stream);
int fcv2_dispatch_quant_fresh(const void* x, const int32_t* ids, uint32_t T, uint32_t H, uint32_t K, uint32_t E, const fcv2_fmt_t* fmt,
                              void* send, int32_t* expert_offsets, int32_t* row_src, void* ws, size_t ws_bytes, void* stream);
#ifdef __cplusplus
}
#endif
