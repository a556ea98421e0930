// Host-side checks shared by the entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "vd.h"

namespace vd {
namespace host {

inline int64_t elem_bytes(int32_t dtype) { return dtype == VD_DTYPE_BF16 ? 2 : 4; }
inline int64_t align16(int64_t x) { return (x + 15) & ~int64_t(15); }
inline bool aligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

inline vd_status check_desc(const vd_cache_desc *d) {
    if (!d || !d->v) return VD_ERR_INVALID_ARG;
    if (d->dtype != VD_DTYPE_BF16 && d->dtype != VD_DTYPE_F32) return VD_ERR_INVALID_ARG;
    if (d->num_seqs < 1 || d->num_layers < 1 || d->num_kv_heads < 1 || d->num_q_heads < 1)
        return VD_ERR_INVALID_ARG;
    if (d->num_q_heads % d->num_kv_heads != 0) return VD_ERR_INVALID_ARG;
    if (d->head_dim < 1 || d->capacity < 1) return VD_ERR_INVALID_ARG;
    if (d->head_dim != 64 && d->head_dim != 128 && d->head_dim != 256) return VD_ERR_UNSUPPORTED;
    if (d->capacity > VD_MAX_CAPACITY) return VD_ERR_UNSUPPORTED;
    if (d->stride_seq < 0 || d->stride_layer < 0 || d->stride_head < 0 || d->stride_slot < 0)
        return VD_ERR_INVALID_ARG;
    if (d->stride_slot < d->head_dim) return VD_ERR_INVALID_ARG;  // rows would overlap
    if (d->num_layers > 65535) return VD_ERR_UNSUPPORTED;  // one grid row per layer
    const int64_t units = int64_t(d->num_seqs) * d->num_layers * d->num_kv_heads;
    if (units > INT32_MAX || units * int64_t(d->capacity) > (int64_t(1) << 47))
        return VD_ERR_UNSUPPORTED;
    const int64_t es = elem_bytes(d->dtype);
    // a unit's slab is addressed with 32-bit byte offsets
    if (d->stride_slot > int64_t(UINT32_MAX) / es / d->capacity) return VD_ERR_UNSUPPORTED;
    const int64_t strides[4] = {d->stride_seq, d->stride_layer, d->stride_head, d->stride_slot};
    for (int64_t s : strides)
        if (s % (16 / es) != 0) return VD_ERR_INVALID_ARG;  // every row 16-byte aligned
    if (!aligned(d->v, 16) || (d->k && !aligned(d->k, 16))) return VD_ERR_INVALID_ARG;
    if (d->k && d->k == d->v) return VD_ERR_INVALID_ARG;
    return VD_OK;
}

inline vd_status launched(hipError_t e) { return e == hipSuccess ? VD_OK : VD_ERR_HIP; }

}  // namespace host
}  // namespace vd
