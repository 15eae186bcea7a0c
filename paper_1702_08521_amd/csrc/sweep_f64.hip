// Sweep kernels of FP64 storage.
#include "sweep_kernels.hpp"

namespace slmpp {
template struct SweepLaunch<double>;
}  // namespace slmpp
