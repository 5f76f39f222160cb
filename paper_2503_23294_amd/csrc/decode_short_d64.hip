// The decode kernels for short contexts at head_dim 64 (see decode_short_impl.h).
#include "decode_short_impl.h"

namespace cocktail {
template hipError_t launch_decode_short<64>(const DecodeParams&, const ShortRec*, const ShortGroup*, int, bool, int, bool, bool, int, hipStream_t);
}
