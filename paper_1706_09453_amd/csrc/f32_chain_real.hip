// Ascending-k fp32 sums with real weights.
#include "f32_chain_launch.hpp"

namespace bnn {
void launch_chain_real(const ChainArgs& a, int act) { launch_chain<true>(a, act); }
}  // namespace bnn
