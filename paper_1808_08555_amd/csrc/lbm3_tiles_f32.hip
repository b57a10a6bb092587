// Instantiations of the fused step (lbm3_step_impl.h) for storage float, compute float.
#include "lbm3_step_impl.h"

namespace tcg {

hipError_t tiles_f32(Fmt in, Fmt out, bool obs, bool pt, const void* fin, void* fout, const Instance* inst,
                    const Tile* tiles, int ntiles, int threads, uint32_t salt, const int64_t* step_dev,
                    int filter, double* partials, double* rho_out, hipStream_t stream)
{
    return tiles_any<float, float>(in, out, obs, pt, fin, fout, inst, tiles, ntiles, threads, salt, step_dev,
                                filter, partials, rho_out, stream);
}

int tiles_f32_occupancy(int threads) { return tiles_occupancy<float, float>(threads); }

hipError_t tiles_f32_pair(const void* fin, void* fout, const Instance* inst, const Tile* tiles,
                          int ntiles, int threads, bool pt, hipStream_t stream)
{
    return tiles_pair_any<float, float>(fin, fout, inst, tiles, ntiles, threads, 0u, 0u, nullptr, pt, stream);
}

int tiles_f32_pair_occupancy(int threads) { return pair_occupancy<float, float>(threads); }

hipError_t tiles_f32_block(const void* fin, void* fout, const BlockGrid& bg, uint32_t salt, bool pt,
                           hipStream_t stream)
{
    return tiles_block_any<float, float>(fin, fout, bg, salt, pt, stream);
}

hipError_t tiles_f32_block2(const void* fin, void* fout, const BlockGrid& bg, uint32_t salt_a, uint32_t salt_b, bool pt,
                            hipStream_t stream)
{
    return tiles_block2_any<float, float>(fin, fout, bg, salt_a, salt_b, pt, stream);
}

hipError_t tiles_f32_block_list(const void* fin, void* fout, const BlockList& bl, uint32_t salt, bool pt,
                                hipStream_t stream)
{
    return tiles_block_list_any<float, float>(fin, fout, bl, salt, pt, stream);
}

hipError_t tiles_f32_block_obs(const void* fin, const BlockGrid& bg, bool pt, double* partials, double* rho_out,
                               hipStream_t stream)
{
    return tiles_block_obs_any<float, float>(fin, bg, pt, partials, rho_out, stream);
}

}  // namespace tcg
