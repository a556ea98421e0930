// Host side of vd_append (include/vd.h): validation, then one launch.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "vd.h"
#include "vd_check.h"
#include "vd_launch.h"

using namespace vd::host;

extern "C" vd_status vd_append(const vd_cache_desc *desc, int32_t seq, int32_t n_old, int32_t rows,
                    const void *k_rows, const int64_t *k_strides, const void *v_rows,
                    const int64_t *v_strides, int32_t *pos, int32_t pos0, vd_stream stream) {
    const vd_status st = check_desc(desc);
    if (st != VD_OK) return st;
    if (!desc->k || !k_rows || !v_rows || !k_strides || !v_strides) return VD_ERR_INVALID_ARG;
    if (seq < 0 || seq >= desc->num_seqs || n_old < 0 || rows < 1 || rows > desc->capacity - n_old)
        return VD_ERR_INVALID_ARG;
    if (pos0 < 0 || pos0 > INT32_MAX - rows) return VD_ERR_INVALID_ARG;
    if (!aligned(k_rows, 16) || !aligned(v_rows, 16) || (pos && !aligned(pos, 4)))
        return VD_ERR_INVALID_ARG;
    const int64_t es = elem_bytes(desc->dtype);
    const int64_t L = desc->num_layers, H = desc->num_kv_heads;
    const int64_t units = L * H;
    // units that share memory would be written at once
    if ((L > 1 && desc->stride_layer == 0) || (H > 1 && desc->stride_head == 0)) return VD_ERR_INVALID_ARG;
    if (units > INT32_MAX / 2) return VD_ERR_UNSUPPORTED;
    // byte offsets and the extents compared below stay far from 64 bits
    if (desc->stride_seq > (int64_t(1) << 46) / desc->num_seqs || desc->stride_layer > (int64_t(1) << 46) / L ||
        desc->stride_head > (int64_t(1) << 46) / H)
        return VD_ERR_UNSUPPORTED;
    vd::AppendParams p;
    std::memset(&p, 0, sizeof p);
    const int64_t seq_off = int64_t(seq) * desc->stride_seq * es;
    p.k = static_cast<char *>(desc->k) + seq_off;
    p.v = static_cast<char *>(desc->v) + seq_off;
    p.s_layer = desc->stride_layer * es;
    p.s_head = desc->stride_head * es;
    p.s_slot = uint32_t(desc->stride_slot * es);
    const int64_t row_bytes = desc->head_dim * es;
    // the cache's whole extent, of every sequence
    const uint64_t extent = uint64_t((desc->num_seqs - 1) * desc->stride_seq * es + (L - 1) * p.s_layer +
                                     (H - 1) * p.s_head + int64_t(desc->capacity - 1) * p.s_slot + row_bytes);
    const uintptr_t cache[2] = {reinterpret_cast<uintptr_t>(desc->k), reinterpret_cast<uintptr_t>(desc->v)};
    const void *src[2] = {k_rows, v_rows};
    const int64_t *strides[2] = {k_strides, v_strides};
    for (int i = 0; i < 2; ++i) {
        uint64_t span = uint64_t(row_bytes);
        const int64_t count[3] = {L, H, rows};
        for (int j = 0; j < 3; ++j) {
            const int64_t s = strides[i][j];
            if (s < 0 || s > (int64_t(1) << 46) / count[j] || (s * es) % 16 != 0) return VD_ERR_INVALID_ARG;
            span += uint64_t(s * es) * uint64_t(count[j] - 1);
        }
        const uintptr_t at = reinterpret_cast<uintptr_t>(src[i]);
        for (uintptr_t base : cache)
            if (at < base + extent && base < at + span) return VD_ERR_INVALID_ARG;
    }
    p.src_k = static_cast<const char *>(k_rows);
    p.src_v = static_cast<const char *>(v_rows);
    p.k_layer = k_strides[0] * es;
    p.k_head = k_strides[1] * es;
    p.k_row = k_strides[2] * es;
    p.v_layer = v_strides[0] * es;
    p.v_head = v_strides[1] * es;
    p.v_row = v_strides[2] * es;
    p.num_kv_heads = desc->num_kv_heads;
    p.units = int32_t(units);
    p.capacity = desc->capacity;
    p.slot0 = n_old;
    p.rows = rows;
    p.pos = pos ? pos + int64_t(seq) * units * desc->capacity : nullptr;
    p.pos0 = pos0;
    return launched(vd::launch_append(p, int(row_bytes), reinterpret_cast<hipStream_t>(stream)));
}
