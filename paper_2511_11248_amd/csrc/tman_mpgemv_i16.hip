// Decoding mpGEMV from INTEGER tables (Sec. 6.1 "A_INT16": activations as 16-bit integers; Sec. 4.3 two-level tiling: low
// precision -- here exact integers -- inside a quantization block, floating point only across blocks).  The tables come
// from tman_build_lut_i16; the kernels take the 14-bit activations out of them and multiply them with the codes: one token as
// digits on the dot product unit (tman_mpgemv_x.hip), several on the matrix cores (tman_codes_kernel.h), where an activation
// is two exact fp16 numbers, a multiple of 8 and a rest of -4 .. 3.  A block's sums are exact there too: those of the first are multiples
// of 8 below 2^27 (128 x 79 x 8192 with 4 bits and the codes' offset), those of the rests are below 2^16.
#include "tman_mpgemv_x_kernel.h"

namespace tman {

int launch_mpgemv_i16(const Layout& L, const void* packed, const void* lut, int N, void* y, void* workspace,
                      hipStream_t st) {
    return launch_x_single<TokenSource::kTablesI16>(L, N, packed, lut, y, workspace, st);
}
int launch_mpgemv_i16_batch(const DecodeBatch& b, hipStream_t st) { return launch_x_batch<TokenSource::kTablesI16>(b, st); }

}  // namespace tman
