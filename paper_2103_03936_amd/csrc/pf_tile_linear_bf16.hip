#include "pf_tile_linear.h"

namespace pf {
template int launch_linear_t<bf16_t>(hipStream_t, const char *, TileShape, const TileArgs &);
}
