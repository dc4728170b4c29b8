// Stream-collide launches of the BF16 storage.
#include "collide_inst.hpp"

namespace lbmbp {

template void launch_stream_collide<Cfg<CodecBF16, D3Q19>, false>(const CollideArgs &);
template void launch_stream_collide<Cfg<CodecBF16, D3Q19>, true>(const CollideArgs &);
template void launch_stream_collide<Cfg<CodecBF16, D3Q15>, false>(const CollideArgs &);
template void launch_stream_collide<Cfg<CodecBF16, D3Q15>, true>(const CollideArgs &);

}  // namespace lbmbp
