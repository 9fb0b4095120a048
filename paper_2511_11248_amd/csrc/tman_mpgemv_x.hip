// Decoding mpGEMV of one token on the 4-bit dot product unit, or for 1 and 2 bits on the matrix cores (tman_fp4_device.h):
// tman_mpgemv_x (activations in), tman_mpgemv and tman_mpgemv_i16 (tables in).
//
// y[m] = sum_G scale[m][G] * (sum_{k in G} q[m][k] x[k] - zero[m][G] * S[G]) (Sec. 2.2).  The lookups of Sec. 4.3 turn
// the inner sum into one table read per 4 weights and bit-plane; on this chip that costs 2.6 vector instructions and
// an LDS read each, and the kernel built that way was bound by vector issue (7B layer sets: uint2 g64 14.7 us, uint4
// g128 24.2 us per launch).  Here the sum is taken in integers: the activations of a quantization block become 16-bit
// fixed-point numbers, split into four signed 4-bit digits, and v_dot8c_i32_i4 multiplies eight codes with one digit
// (see tman_digits_device.h for the instruction counts and the precision).
//
// A workgroup of four waves owns one row block (64 rows, one per lane) and one K segment of at most 32 tiles.  It
// makes the digits of its segment itself (8 KB of activations -> 8 KB of digit words in LDS) while its first weight
// tiles are on their way, so a decode step needs no launch for a precompute.  Given tables, it takes the activations
// out of them: the entries of patterns 1, 2, 4 and 8 are the four activations themselves.  The sums of the four waves
// meet in LDS, segments of a long K through the workspace (tickets, fixed order of addition).
//
// What bounds it: the weight stream.  63.2 MB (7B uint2 g64) in 13.0 us = 4.9 TB/s (11.7 with neither digits nor products), 107.5 MB
// (uint4 g128) in 19.2 us = 5.6 TB/s (20.0 without: the waves then have their requests out sooner, which costs the memory system more
// than the computing does); reading alone reaches 6.0-6.15 TB/s, and about 1 us at the start (descriptor, first activations)
// and 1.5 us at the end (exchange between segments) are not covered.  What helped beside the digits, measured in
// turn on the uint2 / uint4 launch: the waves of a workgroup take its tiles in turn instead of a quarter each, so that
// a workgroup reads one contiguous stream (uint4 20.6 -> 20.1 us); ONE tile in flight per wave instead of two or three
// (uint2 14.2 -> 13.6 us with two against one, 15.2 with three: more streams in flight cost more in the memory
// system than they hide; 1 bit: two, see the kernel); no issue priorities (uint2 14.3 -> 13.9 us: they balanced vector work, which no longer
// bounds); K up to 4096 as one segment also for 4-bit weights (uint4 20.7 -> 19.6 us).
#include <algorithm>
#include <vector>

#include "tman_mpgemv_x_kernel.h"

namespace tman {

// Segments (measured on the 7B and 3.8B layer sets): a K that one workgroup can take whole - up to 32 tiles and 160 KB
// of packed weights per row block - is one segment, which spares the exchange of partial sums; a longer K is cut into
// equal segments of at most 17 tiles.
GemvPlan plan_gemv_x(const Layout& L) {
    const tman_tiling_t t = current_tiling();
    int whole = t.decode_x_whole_bytes / L.tile_bytes;
    if (whole > t.decode_x_seg_tiles) whole = t.decode_x_seg_tiles;
    if (whole < 1) whole = 1;
    return plan_segments(L, 1, L.n_ktiles <= whole ? whole : t.decode_x_long_seg_tiles);
}

// A good part of the vector instructions of a 1-bit workgroup make digits, and a large launch (all layers of a model at once) is
// bound by vector issue: its workgroups take two row blocks each, as long as that leaves at least eight per compute unit.
// 160 GEMVs of a 32-layer 3.8B model in one launch, sign form with blocks of 64: 113 us with two, 120 with one, 119 by
// lookups (launches back to back; right after an idle GPU, whose clocks are still low: 144 - 148, 150, 140); with zeros 120, 127, 129;
// width 4096, 64-blocks: 194, 210, 249.  Four: 113, with zeros 123, width 4096 230: fewer, longer workgroups end unevenly.
int batch_row_blocks(int bits, int N, long long n_workgroups, int n_units) {
    return bits == 1 && N == 1 && n_units > 0 && n_workgroups >= 16LL * n_units ? 2 : 1;
}

// The numbered launch of a batch (see order_workgroups_of): at most 8 workgroups per compute unit, as many as the LDS holds, and no
// more than 5 of 32 tiles - numbering a
// launch pays while a unit has few of them (1152 workgroups of a layer set with MLP width 14336, uint4 g128: 25.5 us on
// the plain grid, 23.3 us numbered; equal workgroups need none).
static int resident_per_unit(int count, const Layout* L, const GemvPlan* plans, int N) {
    const int np = padded_tokens(N);
    if (np > 1 && !lookups_stay(L[0].bits, np, true)) return kCodesResident;
    int max_seg_tiles = 1;
    for (int g = 0; g < count; ++g) max_seg_tiles = std::max(max_seg_tiles, plans[g].seg_tiles);
    const unsigned lds = np == 1 ? x_lds_bytes(max_seg_tiles, L[0].groups_per_tile, on_matrix_cores(L[0].bits, TokenSource::kActivations))
                                 : (unsigned)(kWaves * (kTableBytesPerKTile * np + 256 + np * kRows * 4));
    return std::max(1, std::min((int)(160u * 1024u / lds), std::min(8, 160 / max_seg_tiles)));
}
int ordered_workgroups(int count, const Layout* L, const GemvPlan* plans, int N, int n_units) {
    return count > 8 ? 0 : ordered_workgroups_of(count, L, plans, n_units, resident_per_unit(count, L, plans, N));
}
bool order_workgroups(int count, const Layout* L, const GemvPlan* plans, int N, int n_units, std::vector<uint16_t>* order) {
    return count <= 8 && order_workgroups_of(count, L, plans, n_units, resident_per_unit(count, L, plans, N), order);
}

int launch_mpgemv_x(const Layout& L, const void* packed, const void* x, void* y, void* workspace, hipStream_t st) {
    return launch_x_single<TokenSource::kActivations>(L, 1, packed, x, y, workspace, st);
}
int launch_mpgemv_x_batch(const DecodeBatch& b, hipStream_t st) { return launch_x_batch<TokenSource::kActivations>(b, st); }

}  // namespace tman
