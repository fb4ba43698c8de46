#include "pf_tile_linear.h"

namespace pf {
template int launch_linear_t<float>(hipStream_t, const char *, TileShape, const TileArgs &);
}
