// wm_shares.hpp -- how the work of a call is cut into shares: rules on sizes
// alone, apart from the kernels so that a host program can run them.
#pragma once
#include <cstdint>

namespace wm {

// Shapes per wave of the tile selection: equal runs for `waves` waves, times
// grid_mult as many; no fewer than fill a round of 64 candidates with lists of
// the average length (at most 8).  A grid_mult cuts runs no shorter than three
// rounds: every run pays its setup and the end's float64 pass (2^15 shapes with
// 1.7e6 candidates 19.3 us at 1 and 22.4 at 2, three shapes a run; 25 to 29 with
// two, 37 to 42 with one, where dealing batches of eight took 26 at any multiple).
inline int64_t tile_run(int64_t n, int64_t n_cand, int64_t waves, int grid_mult)
{
    const int64_t fill = n_cand > 8 * n ? 64 * n / n_cand : 8;
    const int64_t equal = (n + waves - 1) / waves;
    const int64_t rounds3 = n_cand > 0 ? 192 * n / n_cand : equal;
    const int64_t many = waves * (grid_mult < 1 ? 1 : grid_mult);
    int64_t per = (n + many - 1) / many;
    per = per < rounds3 ? (rounds3 < equal ? rounds3 : equal) : per;
    return per < fill ? fill : per;
}

// The application sweep in one block of `block` threads clears the row flags by
// itself, while a thread has at most 64 of their words: at 256 threads 4.6 us for
// the kernel with 1024 words, 6.4 with 16384 and 11.5 with 65536, where the launch
// that clears them with the whole chip takes 2 to 3.
inline bool sweep_clears_flags(int blocks, int64_t words, int block) { return blocks == 1 && words <= 64 * (int64_t)block; }

}  // namespace wm
