// Decoding mpGEMV from INTEGER tables (Sec. 6.1 "A_INT16": activations as 16-bit integers; Sec. 4.3 two-level tiling: low
// precision -- here exact integers -- inside a quantization block, floating point only across blocks).  The tables come
// from tman_build_lut_i16; the kernel takes the 14-bit activations out of them and multiplies their digits with the codes
// (tman_mpgemv_x.hip): the block sums are the integers the lookups would add up to.
#include "tman_mpgemv_x_kernel.h"

namespace tman {

int launch_mpgemv_i16(const Layout& L, const void* packed, const void* lut, int N, void* y, void* workspace,
                      hipStream_t st) {
    return launch_x_single<TokenSource::kTablesI16>(L, N, packed, lut, y, workspace, st);
}
int launch_mpgemv_i16_batch(const DecodeBatch& b, hipStream_t st) { return launch_x_batch<TokenSource::kTablesI16>(b, st); }

}  // namespace tman
