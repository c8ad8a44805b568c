// Ascending-k fp32 sums with weight bits.
#include "f32_chain_launch.hpp"

namespace bnn {
void launch_chain_bits(const ChainArgs& a, int act) { launch_chain<false>(a, act); }
}  // namespace bnn
