// group_wavek.hip -- the per-group layout's instantiation of wavek.h (a file
// of its own for its compiler flags: the vector ALU converts every result of
// the matrix cores).
#include "wavek.h"

namespace fgq {

fgq_status launch_wavek_group(const WavekArgs& a, int bits, hipStream_t st) { return launch_wavek_mode<2>(a, bits, st); }

}  // namespace fgq
