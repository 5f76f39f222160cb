// The decode kernel for five to eight query heads per workgroup at head_dim 128 (see decode_tiles_impl.h).
#include "decode_tiles_impl.h"

namespace cocktail {
template hipError_t launch_decode_tiles<128>(const DecodeParams&, int, bool, bool, int, hipStream_t);
}
