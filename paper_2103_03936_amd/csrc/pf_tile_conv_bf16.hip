#include "pf_tile_conv.h"

namespace pf {
template int launch_conv_t<bf16_t>(hipStream_t, const char *, TileShape, TileShape, const TileArgs &);
}
