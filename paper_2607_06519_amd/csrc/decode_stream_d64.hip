// The streaming split-K decode at head dimension 64 (decode_stream.h).
#define FDKV_STREAM_INSTANCES
#include "decode_stream.h"

namespace fdkv {
template hipError_t launch_stream<64>(const DecodeParams&, hipStream_t);
}  // namespace fdkv
