// Sweep kernels of FP32 storage.
#include "sweep_kernels.hpp"

namespace slmpp {
template struct SweepLaunch<float>;
}  // namespace slmpp
