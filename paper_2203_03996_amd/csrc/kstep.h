// Which K-step's packed weights a kernel asks for.  Plain C++: the tests compile it for the host.
#pragma once

namespace dcnn {

// K-steps of a tap are asked for in groups of four, whose last ones may be padding (step >= steps).  Those meet zero pixels and their lanes
// ask from outside the descriptor; the wave-uniform part of the offset stays at the last K-step there is, because the range check of a raw
// buffer is `lane offset >= num_records - uniform offset`, which a uniform offset past the end would carry below zero.
constexpr int weight_step(int tap, int steps, int step) { return tap * steps + (step < steps ? step : steps - 1); }

}  // namespace dcnn
