// Persistent producer / consumer kernels: bf16 with B stored N x K, A stored K x M (weight gradients),
// and the convolution gather for bf16 and KRSC weights.
#include "alcop_instantiate_stream.hip.h"
namespace alcop {
void register_stream_more(std::vector<KernelEntry>& t)
{
  ALCOP_STREAM_KEY(t, 1, 128, 128, 64, 64, 1, 0, 0)
  ALCOP_STREAM_KEY(t, 1, 128, 64, 64, 32, 1, 0, 0)
  ALCOP_STREAM_KEY(t, 1, 64, 64, 32, 32, 1, 0, 0)
  ALCOP_STREAM_KEY(t, 1, 128, 64, 64, 32, 0, 0, 0)
  // A stored K x M, B stored K x N
  ALCOP_STREAM_KEY(t, 0, 128, 128, 64, 64, 0, 0, 1)
  ALCOP_STREAM_KEY(t, 0, 64, 64, 32, 32, 0, 0, 1)
  ALCOP_STREAM_KEY(t, 1, 128, 128, 64, 64, 0, 0, 1)
  ALCOP_STREAM_KEY(t, 1, 64, 64, 32, 32, 0, 0, 1)
}
}  // namespace alcop
