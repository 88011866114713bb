// The streaming split-K decode at head dimension 128 (decode_stream.h).
#define FDKV_STREAM_INSTANCES
#include "decode_stream.h"

namespace fdkv {
template hipError_t launch_stream<128>(const DecodeParams&, hipStream_t);
}  // namespace fdkv
