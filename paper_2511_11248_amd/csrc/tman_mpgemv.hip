// Decoding mpGEMV through bit-serial table lookup (Sec. 2.2 "Bit-serial table lookup", Sec. 4.3
// "Mapping of LUT-based Decoding").
//
//   y[n][m] = sum_G scale[m][G] * ( sum_i 2^i sum_{j in G} T[n][j][idx_i[m][j]] - zero[m][G] * S[n][G] )
//
// Mapping onto a CDNA4 compute unit.  As in the paper's vector-core mapping the lookups are
// vectorised along the output rows: the 64 lanes of a wave hold 64 different rows and index the SAME
// 16-entry table, so the table (32 bytes = 8 LDS banks) is read by broadcast without bank conflicts,
// every lane keeps a private fp32 accumulator for its row, and nothing crosses lanes in the loop.
// The paper's two-level tiling appears as: inner tile = one quantization block (table entries summed
// in fp32, then one scale/zero application), outer tile = a 128-column tile whose 32 tables sit in LDS.
//
// Scheduling.  A decode GEMV streams each weight byte once and a whole layer lasts microseconds, so
// the kernel is organised around keeping HBM requests in flight and around short dependency chains:
//   - a workgroup of four waves owns one row block (64 rows) and one K segment of at most 32 tiles;
//     each wave takes a quarter of the segment and walks it with one or two tile blocks in flight
//     (coalesced 16-byte loads of the bit-plane chunks, the group parameters and the 1 KB table
//     slice of the tile); the table slice goes to the wave's private LDS slot, so waves do not
//     synchronise while streaming;
//   - the four partial sums of a row meet in LDS (one barrier, fixed order);
//   - only when K is longer than one segment do segments meet through memory: each publishes its
//     fp32 partial and takes a ticket, the last one adds the partials in segment order (so the result
//     does not depend on timing).  Partials and tickets use device-scope memory operations, which are
//     coherent across the chip without cache write-back or invalidation.
// All GEMVs of a decode step can share one launch (descriptor table), so the machine is filled even
// though one layer alone is too small.
//
// mpgemv_kernel serves 2 to 4 tokens of few bit-planes (lookups_stay) and reads the tables tman_build_lut made (Sec. 5: the
// precompute as a kernel of its own, shared by the layers fed from one activation).  One token goes to tman_mpgemv_x.hip, the
// rest to the matrix cores (tman_codes_kernel.h).
#include <algorithm>
#include <functional>
#include <mutex>
#include <queue>
#include <vector>

#include "tman_mpgemv_x_kernel.h"

namespace tman {

// ---------------------------------------------------------------------------------------------
// host-side planning

GemvPlan plan_segments(const Layout& L, int np, int max_seg) {
    GemvPlan p;
    p.np = np;
    p.n_seg = (L.n_ktiles + max_seg - 1) / max_seg;
    p.seg_tiles = (L.n_ktiles + p.n_seg - 1) / p.n_seg;
    p.n_seg = (L.n_ktiles + p.seg_tiles - 1) / p.seg_tiles;
    p.n_workgroups = L.n_row_blocks * p.n_seg;
    p.ticket_bytes = ((size_t)L.n_row_blocks * sizeof(int32_t) + 255) / 256 * 256;
    p.partial_bytes = p.n_seg > 1 ? (size_t)L.n_row_blocks * p.n_seg * p.np * kRows * sizeof(float) : 0;
    return p;
}

int device_units() {
    static std::once_flag once;
    static int n_units = 0;
    std::call_once(once, [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            n_units = n;
    });
    return n_units;
}

GemvPlan plan_tables(const Layout& L, int N) {
    const int np = padded_tokens(N);
    // with four or eight tokens a looked-up tile takes about twice as long: shorter segments, more workgroups (measured)
    const tman_tiling_t t = current_tiling();
    return plan_segments(L, np, np >= 4 ? t.decode_seg_tiles_many : t.decode_seg_tiles);
}

// Several tokens on the matrix cores: the kernel of small batches.  Its segments are longer (small_seg_tiles) where the launch fills the chip
// without short ones: 7B uint4 g128, N = 4, us per layer set with the table launch, segments of 24 / 32 / 43 tiles 37.5 / 33.6 /
// 29.7; a K of 44 to 50 tiles, which 43 cuts in two, is better off so on the whole (one segment,
// layer sets 2048 / 5632 and 2048 / 6400: +14 to 45 %; 3072 / 6144: -14 to +30 %).  A launch that
// leaves compute units idle (`fills` false: a single GEMV with few rows) keeps the lookups' short segments: 4096 x 11008, N = 4,
// 22 / 43 tiles 11.8 / 14.7 us, 4096 x 4096 16 / 32 tiles 8.9 / 10.0; 11008 x 4096, which fills it, 11.9 / 10.5.  A caller's own
// decode_seg_tiles (_many) decides alone.  A table batch is prepared for both kinds of tables; where only one of them is looked up (2
// bits, two tokens) the plan is this one too (7B uint2 g64 fp16, 32 / 43 tiles: 18.3 / 18.4, integers 23.7 / 20.0).
GemvPlan plan_decode(const Layout& L, int N, bool fills) {
    if (N == 1) return plan_gemv_x(L);
    const int np = padded_tokens(N);
    const tman_tiling_t t = current_tiling();
    tman_tiling_t built_in;
    (void)tman_default_tiling(&built_in);
    const int own = np >= 4 ? t.decode_seg_tiles_many : t.decode_seg_tiles;
    if (!fills || lookups_stay(L.bits, np, true) || own != (np >= 4 ? built_in.decode_seg_tiles_many : built_in.decode_seg_tiles))
        return plan_tables(L, N);
    return plan_segments(L, np, std::max(t.small_seg_tiles, own));
}
bool fills_device(long long table_workgroups) { return table_workgroups > device_units(); }

// (plan_decode never has more segments than plan_tables, which it has in a small launch.)
size_t decode_workspace_bytes(const Layout& L, int N) {
    const GemvPlan p = N == 1 ? plan_gemv_x(L) : plan_tables(L, N);
    return p.ticket_bytes + p.partial_bytes;
}

void fill_desc_plan(GemvDesc& d, const Layout& L, const GemvPlan& p, const void* packed, const void* lut, int N,
                           void* y, void* workspace) {
    d.tiles = static_cast<const uint8_t*>(packed) + kHeaderBytes;
    d.lut_t = static_cast<const uint8_t*>(lut);
    d.lut_s = d.lut_t + (size_t)L.n_ktiles * kTableBytesPerKTile * p.np;
    d.y = y;
    d.tickets = static_cast<int32_t*>(workspace);
    d.partial = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + p.ticket_bytes);
    d.M = L.M;
    d.N = N;
    d.n_row_blocks = L.n_row_blocks;
    d.n_ktiles = L.n_ktiles;
    d.seg_recip = 0xFFFFFFFFu / (uint32_t)p.n_seg;
    d.n_seg = p.n_seg;
    d.seg_tiles = p.seg_tiles;
    d.K = L.K;
}

// ---------------------------------------------------------------------------------------------
// launch

int launch_mpgemv(const Layout& L, const void* packed, const void* lut, int N, void* y, void* workspace, hipStream_t st) {
    return launch_x_single<TokenSource::kTables>(L, N, packed, lut, y, workspace, st);
}
int launch_mpgemv_batch(const DecodeBatch& b, hipStream_t st) { return launch_x_batch<TokenSource::kTables>(b, st); }

// Copies up to 16 descriptors per launch from the kernel arguments into the device table.  A GEMV whose blob
// carries a header for another shape or layout gets an empty descriptor (no workgroup of the lookup launch
// then touches it) and the mismatch is recorded in the library's status word.
struct DescChunk {
    GemvDesc d[16];
};
__global__ void write_descs_kernel(DescChunk c, int count, int bits, int group, int has_zero, GemvDesc* __restrict__ out,
                                   int* status) {
    if ((int)threadIdx.x >= count) return;
    GemvDesc d = c.d[threadIdx.x];
    if (!header_matches(d.tiles, d.M, d.K, bits, group, has_zero)) {
        d.n_row_blocks = 0;
        report_header_mismatch(status);
    }
    out[threadIdx.x] = d;
}

int launch_write_descs(const GemvDesc* host, int count, int bits, int group, int has_zero, GemvDesc* dev, hipStream_t st) {
    int* status = device_status_word();
    if (!status) return TMAN_ERR_LAUNCH;
    for (int i = 0; i < count; i += 16) {
        DescChunk c;
        int n = count - i < 16 ? count - i : 16;
        for (int j = 0; j < 16; ++j) c.d[j] = host[i + (j < n ? j : 0)];
        hipLaunchKernelGGL(write_descs_kernel, dim3(1), dim3(64), 0, st, c, n, bits, group, has_zero, dev + i, status);
    }
    return launch_status();
}

// ---------------------------------------------------------------------------------------------
// Numbering the workgroups of a batch for equal work per compute unit.
//
// With workgroup i on compute unit i mod n_units (what the dispatcher does with a launch that is resident at
// once), the numbering decides which workgroups share a unit.  The workgroups, largest first, go one by one to the
// unit with the least work so far that still has a free place (unit j has a place for ids j, j + n_units, ...);
// then the fullest unit exchanges a workgroup with another unit as long as that lowers the larger of the two
// loads; inside a unit the largest gets the lowest id.  Work of a workgroup = tile blocks of its K segment + 2
// (start and end of a workgroup cost about that).  A batch qualifies with at most 8 GEMVs (three bits of an
// entry) and no more workgroups than are resident at once: `per_unit` per compute unit.
int ordered_workgroups_of(int count, const Layout* L, const GemvPlan* plans, int n_units, int per_unit) {
    (void)L;
    if (count > 8 || n_units < 1 || per_unit < 1 || !current_tiling().decode_balance) return 0;
    int n = 0;
    for (int g = 0; g < count; ++g) {
        if (plans[g].n_workgroups > 0x1fff) return 0;
        n += plans[g].n_workgroups;
    }
    return n <= per_unit * n_units && n <= kOrderedMaxWorkgroups ? n : 0;
}

bool order_workgroups_of(int count, const Layout* L, const GemvPlan* plans, int n_units, int per_unit,
                         std::vector<uint16_t>* order) {
    const int n = ordered_workgroups_of(count, L, plans, n_units, per_unit);
    if (!n) return false;
    const int slots = (n + n_units - 1) / n_units;  // places of a unit; units from n % n_units on have one less if that is not 0
    auto places = [&](int j) { return n / n_units + (j < n % n_units ? 1 : 0); };
    struct Item {
        int cost;
        uint16_t id;
    };
    std::vector<Item> items;
    items.reserve(n);
    for (int g = 0; g < count; ++g) {
        const GemvPlan& p = plans[g];
        for (int w = 0; w < p.n_workgroups; ++w) {
            const int seg = w % p.n_seg;
            const int tiles = std::min(p.seg_tiles, L[g].n_ktiles - seg * p.seg_tiles);
            items.push_back(Item{tiles + 2, (uint16_t)((g << 13) | w)});
        }
    }
    auto larger = [](const Item& a, const Item& b) { return a.cost > b.cost; };
    std::stable_sort(items.begin(), items.end(), larger);
    // the unit with the least work and a free place, of several the first
    typedef std::pair<int, int> Unit;  // (work so far, unit)
    std::priority_queue<Unit, std::vector<Unit>, std::greater<Unit>> open;
    for (int j = 0; j < n_units; ++j)
        if (places(j) > 0) open.push(Unit(0, j));
    std::vector<int> load(n_units, 0), count_of(n_units, 0);
    std::vector<Item> mine((size_t)n_units * slots);  // by unit
    for (const Item& it : items) {
        const int j = open.top().second;
        open.pop();
        load[j] += it.cost;
        mine[(size_t)j * slots + count_of[j]++] = it;
        if (count_of[j] < places(j)) open.push(Unit(load[j], j));
    }
    for (int round = 0; round < 8 * n; ++round) {
        int hi = 0;
        for (int j = 1; j < n_units; ++j)
            if (load[j] > load[hi]) hi = j;
        const Item* const h = &mine[(size_t)hi * slots];
        int best_j = -1, best_a = -1, best_b = -1, best_max = load[hi];
        for (int j = 0; j < n_units; ++j) {
            if (j == hi || load[hi] + load[j] >= 2 * best_max) continue;  // (the larger is at least the mean)
            const Item* const q = &mine[(size_t)j * slots];
            for (int a = 0; a < count_of[hi]; ++a) {
                if (a > 0 && h[a].cost == h[a - 1].cost) continue;  // (of equal exchanges the first counts)
                for (int b = 0; b < count_of[j]; ++b) {
                    const int d = h[a].cost - q[b].cost;
                    if (d <= 0 || (b > 0 && q[b].cost == q[b - 1].cost)) continue;
                    const int m = std::max(load[hi] - d, load[j] + d);
                    if (m < best_max) best_max = m, best_j = j, best_a = a, best_b = b;
                }
            }
        }
        if (best_j < 0) break;
        Item &from = mine[(size_t)hi * slots + best_a], &to = mine[(size_t)best_j * slots + best_b];
        const int d = from.cost - to.cost;
        std::swap(from, to);
        load[hi] -= d;
        load[best_j] += d;
    }
    order->assign(n, 0);
    for (int j = 0; j < n_units; ++j) {
        Item* const q = &mine[(size_t)j * slots];
        std::stable_sort(q, q + count_of[j], larger);
        for (int r = 0; r < count_of[j]; ++r) (*order)[(size_t)r * n_units + j] = q[r].id;
    }
    return true;
}

// The numbering goes to device memory through kernel arguments, like the descriptors.
struct OrderChunk {
    uint16_t e[1024];
};
__global__ void write_order_kernel(OrderChunk c, int count, uint16_t* __restrict__ out) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) out[i] = c.e[i];
}
int launch_write_order(const std::vector<uint16_t>& order, uint16_t* dev, hipStream_t st) {
    for (size_t i = 0; i < order.size(); i += 1024) {
        OrderChunk c;
        const int n = (int)std::min<size_t>(1024, order.size() - i);
        for (int j = 0; j < 1024; ++j) c.e[j] = j < n ? order[i + j] : 0;
        hipLaunchKernelGGL(write_order_kernel, dim3(1), dim3(256), 0, st, c, n, dev + i);
    }
    return launch_status();
}

}  // namespace tman
