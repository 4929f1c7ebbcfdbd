// The kernel of xfp_decode_few.inc.h at 2 bits.
#include "xfp_decode_few.inc.h"

namespace xfp {

hipError_t launch_few2(int mode, const FewArgs &fa, dim3 grid, int lds, hipStream_t s)
{
    return launch_few_bits<2>(mode, fa, grid, lds, s);
}

}  // namespace xfp
