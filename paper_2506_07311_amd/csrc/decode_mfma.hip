// Paged decode on the matrix cores: support check, dispatch over head_dim, and the head_dim 128 kernels.
#include "decode_mfma_impl.h"

namespace pa {

template void launch_decode_mfma_dim<128>(const AttnArgs&, hipStream_t);
extern template void launch_decode_mfma_dim<64>(const AttnArgs&, hipStream_t);
extern template void launch_decode_mfma_dim<256>(const AttnArgs&, hipStream_t);
template void launch_decode_short_dim<128>(const AttnArgs&, hipStream_t);
extern template void launch_decode_short_dim<64>(const AttnArgs&, hipStream_t);
extern template void launch_decode_short_dim<256>(const AttnArgs&, hipStream_t);

int32_t decode_mfma_heads_per_wg(int32_t num_kv_heads, int32_t head_dim)
{
    // head_dim 256 holds two tiles in about 250 registers: four waves per workgroup keep that inside the budget
    // of a 256-thread launch
    if (head_dim <= 128 && num_kv_heads % 8 == 0) return 8;
    return num_kv_heads % 4 == 0 ? 4 : num_kv_heads % 2 == 0 ? 2 : 1;
}

bool decode_mfma_supported(const AttnArgs& a)
{
    if (a.dtype != PA_DTYPE_BF16 && a.dtype != PA_DTYPE_F16) return false;
    const int32_t d = a.cache.head_dim;
    if (d != 64 && d != 128 && d != 256) return false;
    const int32_t G = a.num_q_heads / a.cache.num_kv_heads;
    if (G > 16 * 64) return false;                     // one grid slice per 16 heads of a group
    if (a.cache.num_kv_heads > 65535 * 8) return false;
    // per-lane byte offsets inside a 16-key block are kept in 32 bits
    if (a.cache.token_stride * 2 * 16 + a.cache.head_stride * 2 > 0x7fffffffLL) return false;
    // tile counts are kept in 32 bits (tiles hold 16 keys at head_dim 256, 32 otherwise)
    if ((int64_t)a.batch * ((a.max_seq_len + 15) / 16) > 0x7fffffffLL) return false;
    return true;
}

bool decode_short_supported(const AttnArgs& a)
{
    // one workgroup per (sequence, KV head, slice of 16 heads): the grid's y and z extents are 16-bit
    const int32_t G = a.num_q_heads / a.cache.num_kv_heads;
    return decode_mfma_supported(a) && !a.cu_q_lens && a.cache.num_kv_heads <= 65535 && (G + 15) / 16 <= 65535;
}

pa_status launch_decode_short(const AttnArgs& a, hipStream_t stream)
{
    if (a.short_nsplit > 1 && (a.short_nsplit > kShortMaxSplit || !a.short_part || !a.short_arrive)) return PA_ERR_INVALID_ARG;
    ProfileScope prof("paged_decode_short_kernel", stream);
    switch (a.cache.head_dim) {
        case 64: launch_decode_short_dim<64>(a, stream); break;
        case 128: launch_decode_short_dim<128>(a, stream); break;
        case 256: launch_decode_short_dim<256>(a, stream); break;
        default: return PA_ERR_UNSUPPORTED;
    }
    return launch_status();
}

pa_status launch_decode_mfma(const AttnArgs& a, hipStream_t stream)
{
    ProfileScope prof("paged_decode_mfma_kernel", stream);
    switch (a.cache.head_dim) {
        case 64: launch_decode_mfma_dim<64>(a, stream); break;
        case 128: launch_decode_mfma_dim<128>(a, stream); break;
        case 256: launch_decode_mfma_dim<256>(a, stream); break;
        default: return PA_ERR_UNSUPPORTED;
    }
    return launch_status();
}

}  // namespace pa
