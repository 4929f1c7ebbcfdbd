// The kernel of xfp_decode_few.inc.h at 5 and 6 bits.
#include "xfp_decode_few.inc.h"

namespace xfp {

hipError_t launch_few56(int bits, const FewArgs &fa, dim3 grid, int lds, hipStream_t s)
{
    return bits == 5 ? launch_few_bits<5>(0, fa, grid, lds, s) : launch_few_bits<6>(0, fa, grid, lds, s);
}

}  // namespace xfp
