// How far the host runs ahead of a CG solve on the device.
#pragma once

namespace nnqp {

// Iterations that pay: the one that covers the host's way to a launch and one
// behind it.  A launch after the end returns at once, but costs 2 us (250 k rows
// float64: 2, 3, 4, 6 ahead 12.1, 12.4, 12.7, 13.1 ms; 90 k rows with float32
// values, whose iterations take 8 us, 26.7 +- 0.3 ms at any of them).  With a
// synchronisation each 16 iterations instead the two took 18.6 and 38.5 ms.
constexpr int kAhead = 2;
constexpr int kCgChunkDefault = 16;   // nn_opts.cg_chunk of nn_default_opts

// nn_opts.cg_chunk: 0 and the default leave it to the library, any other number
// is the caller's (a loaded host may need more).
constexpr int cg_ahead(int cg_chunk)
{
    return cg_chunk > 0 && cg_chunk != kCgChunkDefault ? cg_chunk : kAhead;
}

}  // namespace nnqp
