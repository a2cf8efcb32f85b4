// When the ragged-shape kernel's 32 x 32 tiles refill their scale buffers (plain constants, free of HIP types).
//
// Batch b (b >= 0) holds the scale bytes of stages b * per .. b * per + per - 1 and lies in half b % 2 of the buffer: it takes the place
// of batch b - 2.  The waves that multiply read stage t's scale bytes right behind barrier t and wait for them between barriers t + 1 and
// t + 2, where the matrix instructions take them: until then the reads may still be on their way, since the barriers wait for no LDS
// reads.  The wave that writes waits for its LDS writes in front of its next barrier.
#pragma once

namespace mxfp4 {

// the barrier behind which batch b >= 1 is written (batch 0 is there before barrier 0)
constexpr int scale_batch_barrier(int b, int per) { return (b - 1) * per + 1; }

// no earlier than two barriers behind the last stage of batch b - 2 ...
constexpr bool scale_batch_drained(int b, int per) { return b < 2 || (b - 1) * per - 1 + 2 <= scale_batch_barrier(b, per); }
// ... and a barrier before the first stage of batch b is read
constexpr bool scale_batch_in_time(int b, int per) { return scale_batch_barrier(b, per) + 1 <= b * per; }

}  // namespace mxfp4
