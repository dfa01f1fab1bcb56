// Host side of the C ABI declared in include/nfd_attn.h: argument checks, tile schedule,
// kernel selection and launches.  Only nfd_attn_create / nfd_attn_destroy allocate or free;
// no other call allocates, synchronises with the host or issues a memset, so all of them can
// be captured into a HIP graph.
#include "../../include/nfd_attn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "kernels_general.hpp"
#include "kernels_mfma.hpp"
#include "kernels_mfma16.hpp"
#include "kernels_mfma_bwd.hpp"
#include "kernels_rows.hpp"
#include "kernels_stream.hpp"

struct nfd_attn {
    nfd_dtype_t dtype;
    int device;
    int num_cus;
    void* workspace;
    size_t workspace_bytes;
    size_t plan_limit;  // workspace size the schedule is planned against (== workspace_bytes for created handles)
    char err[256];      // fixed buffer: recording an error never allocates
};

namespace {

constexpr size_t kDefaultWorkspace = (size_t)128 << 20;
// one row of one key split in the workspace: 64 bf16 partial outputs + (max, sum) in fp32
constexpr size_t kPartialRowBytes = nfd::mfma::kD * 2 + 2 * sizeof(float);

// Record an error text in the handle's fixed buffer (printf-style; no allocation) and return the code.
__attribute__((format(printf, 3, 4))) int fail(nfd_attn_t* h, int code, const char* fmt, ...) {
    if (h) {
        va_list ap;
        va_start(ap, fmt);
        std::vsnprintf(h->err, sizeof(h->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

// Launches go to the device that is current on the calling thread; pointers and workspace belong to the
// handle's device.  A mismatch would launch on the wrong device, so it is refused.
int check_device(nfd_attn_t* h) {
    int cur = -1;
    const hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return fail(h, NFD_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (cur != h->device) return fail(h, NFD_ERR_UNSUPPORTED, "the current device is not the handle's device");
    return NFD_OK;
}

int check_hip(nfd_attn_t* h, hipError_t e, const char* what) {
    if (e == hipSuccess) return NFD_OK;
    return fail(h, NFD_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

size_t elem_size(nfd_dtype_t dt) { return dt == NFD_BF16 ? 2 : 4; }

// Largest key bound of a block of query rows [r0, r0 + bm) (Sec. 3.1: a row sees all
// frames up to and including its own).
int64_t kmax_rows(int64_t r_last, int T, int P) { return ((int64_t)P + r_last / T + 1) * T; }

// How the matrix-core backward is launched.  A workgroup's time is a chain of 64-row steps (key tiles for dq, query tiles
// for dk/dv; a frame boundary's triangle makes their lengths differ), and per step the two kinds cost about the same:
//   kSeparate     dq kernel, then dk/dv kernel: each launch ends on its own tail of few running workgroups
//   kMerged       one launch holds both kinds (the per-row values come from a small launch before it): one tail
//   kMergedSmall  the same with 128 query rows / 64 keys per workgroup: links of 0.97 us instead of 1.57, three workgroups
//                 per CU instead of two, but more steps and more LDS traffic per product (1.93 / 3 against 2.7 / 2 us of
//                 CU time per step when the chip is full)
// Total steps over the workgroup slots, plus half of the longest chain, orders the last two; once the launch is more than
// three chains deep the tails no longer matter and the separate kernels win, whose workgroups share their tiles in L2.
// Measured, backward of 16 frames of 336 tokens (us; separate / merged / merged small): 12 heads 280 / 175 / 188, 24 heads
// 340 / 302 / 341, 48 heads 590 / 574 / 705, 64 heads 763 / 777 / 943; 12 heads, 11 frames of 247: 156 / 85 / 66;
// 192 heads, 20 frames of 40: 116 / 100 / 94; 32 heads, 64 frames of 576: 16 180 / 17 040 / 22 900.
enum class BwdForm { kSeparate = NFD_BWD_SEPARATE, kMerged = NFD_BWD_MERGED, kMergedSmall = NFD_BWD_MERGED_SMALL };
BwdForm bwd_form(int64_t BH, int64_t Sq, int64_t Sk, int T, int P, int num_cus) {
    int64_t longest = 0;
    auto steps = [&](int rows, int keys, int fixed) {  // of all heads, `fixed` more per workgroup
        int64_t n = 0;
        for (int64_t r = 0; r < Sq; r += rows) {
            const int64_t t = (kmax_rows(std::min(r + rows, Sq) - 1, T, P) + 63) / 64;
            longest = std::max(longest, t);
            n += t + fixed;
        }
        for (int64_t k = 0; k < Sk; k += keys) {
            const int64_t t = (Sq + 63) / 64 - std::max<int64_t>(0, (k / T - P) * T) / 64;
            longest = std::max(longest, t);
            n += t + fixed;
        }
        return (double)(n * BH);
    };
    const double all = steps(256, 192, 0);  // sets `longest`
    if (all / (2.0 * num_cus) > 3.0 * longest) return BwdForm::kSeparate;
    // a workgroup's first loads and final write cost about three steps
    const double w = steps(256, 192, 3) / (2.0 * num_cus);
    const double ws = steps(128, 64, 3) / (3.0 * num_cus);
    const double merged = std::max(2.7 * w + 0.5 * 1.57 * longest, 1.57 * longest);
    return std::max(1.93 * ws + 0.5 * 0.97 * longest, 0.97 * longest) < merged ? BwdForm::kMergedSmall : BwdForm::kMerged;
}

// How the matrix-core forward is cut into workgroups: rows per workgroup (the 32-row blocks of a head dealt evenly to `count` of
// them) and key splits.  A workgroup's time is its chain of 64-key tiles.  128-row workgroups have the shorter links, 256-row
// ones (192 rows: tiles of six blocks) less work per row; launches that do not fill the chip for long are as long as their longest
// chain and take short links.  Each choice is priced: links alone on a CU or sharing it, all work over two workgroups per CU plus
// part of the longest chain where there is more than one round, write and merge of the partials.  Fitted to the times of
// both shapes at 1 to 24 splits, 160 sizes over a bf16 cache and 70 over the 8-bit one (1 to 144 heads, 20 to 576 tokens a frame, 2
// to 64 frames, 1 to 48 of them queries), within 8 %; the rule is then 1 % behind the better of the two on average, 18 % ahead of 256-row
// tiles alone.  128-row workgroups take at most the splits that the older
// model of equal chains (tile_splits) gives 256-row ones, usually fewer: a partial output is rounded once more.  Forward, 256-row
// tiles unless they would fill less than a quarter of the CUs / this (us): 80 heads, 8 of 13 frames of 52 tokens 25.1 / 14.4; 24
// heads, 16 frames of 121 38.7 / 27.1; 12 heads, 11 frames of 247 40 / 33; 64 heads, 16 frames of 336 the same kernel.
struct FwdPrice {
    double alone128, shared128, tail128;   // us a tile
    double alone256, shared256, tail256;
    double six;                            // tiles of six blocks (48 rows per wavefront) against the others of the 256-row kernel
    double far;                            // without splits, K/V of all heads past the last-level cache: query tiles drift apart
    double fixed, combine, combine_row;    // us; per row and split
};
constexpr FwdPrice kPrice16{0.653, 0.893, 0.501, 1.054, 1.412, 0.360, 0.896, 1.029, 5.8, 2.63, 0.930e-4};
constexpr FwdPrice kPrice8{0.912, 1.098, 0.150, 1.173, 1.661, 0.373, 1.140, 1.0, 5.0, 2.97, 0.895e-4};
constexpr double kLastLevelBytes = 192e6;  // of 256 MB: room for Q, O and partials

struct RowRanges {
    int count;             // per head
    int64_t tiles, longest;  // key tiles: of a head's ranges together, of the longest
};
RowRanges row_ranges(int64_t Sq, int T, int P, int rows) {
    const int blocks = (int)((Sq + 31) / 32);
    RowRanges r{(blocks + rows / 32 - 1) / (rows / 32), 0, 0};
    const int lo = blocks / r.count, hi = blocks % r.count;
    for (int i = 0; i < r.count; ++i) {
        int b0, nb;
        nfd::mfma::q_tile_blocks(i, lo, hi, &b0, &nb);
        const int r_last = (int)std::min<int64_t>(32 * (int64_t)(b0 + nb), Sq) - 1;
        const int64_t t = (((int64_t)P + r_last / T + 1) * T + nfd::mfma::kBN - 1) / nfd::mfma::kBN;
        r.tiles += t;
        r.longest = std::max(r.longest, t);
    }
    return r;
}
double fwd_price(const FwdPrice& c, const RowRanges& r, int rows_per_wg, bool six, int64_t BH, int64_t Sq, double kv_bytes, int num_cus, int s) {
    const double cus = num_cus, wgs = (double)BH * r.count * s, k = six ? c.six : 1.0;
    const bool small = rows_per_wg == nfd::mfma::kBM / 2;
    const double alone = small ? c.alone128 : c.alone256 * k, shared = small ? c.shared128 : c.shared256 * k;
    const double longest = (double)((r.longest + s - 1) / s);
    const double work = (double)BH * ((double)r.tiles + 0.5 * r.count * (s - 1));  // the last split of a range is shorter
    // past one workgroup per CU: chains of one length end with those that share; of mixed lengths, the long ones start first and
    // the short ones share with them
    const double pairs = std::min(1.0, std::max(0.0, wgs / cus - 1.0));
    const double even = std::max(0.0, 2.0 * (double)r.tiles / ((double)r.count * (double)r.longest) - 1.0);
    double t = longest * (wgs > cus ? alone + (shared - alone) * (pairs + (1.0 - pairs) * even) : alone);
    if (wgs > 2 * cus) t = std::max(t, work * shared / (2 * cus) + (small ? c.tail128 : c.tail256) * longest * shared);
    if (s == 1 && r.count > 1 && kv_bytes > kLastLevelBytes) t *= c.far;
    return t + c.fixed + (s > 1 ? c.combine + c.combine_row * (double)(BH * Sq) * s : 0.0);
}
// Key splits of a launch of 256-row tiles (128-row ones, `few`), only when the tiles alone cannot fill the chip (cached forms).  The
// count minimises a small cost model in units of the time one workgroup needs for one key tile when
// two workgroups share a CU: workgroups run in rounds of 2 (3) per CU; a workgroup that has its CU
// to itself is about 1.2x faster (measured); every workgroup pays a fixed prologue/epilogue of
// about three tiles; the combine pass costs a launch plus the write and read of the partials,
// which grows with rows x splits (about one unit per 30000 row-partials of 136 bytes at HBM speed).
int tile_splits(const RowRanges& r, bool few, int64_t BH, int64_t Sq, int num_cus, size_t workspace_limit) {
    const int64_t slots = (int64_t)num_cus * (few ? 3 : 2), base = BH * r.count;
    if (base >= slots) return 1;
    const size_t per_split = (size_t)(BH * Sq) * kPartialRowBytes;
    double best = 1e30;
    int splits = 1;
    for (int s = 1; s <= 64 && s <= std::max<int64_t>(1, r.longest / 2); ++s) {
        if (s > 1 && per_split * s > workspace_limit) break;
        const int64_t wgs = base * s;
        const int64_t rounds = (wgs + slots - 1) / slots;
        const double len = (double)((r.longest + s - 1) / s) + 3.0;
        const double pace = wgs * 2 <= slots ? 0.83 : 1.0;
        const double combine = s > 1 ? 1.0 + (double)s * (double)(BH * Sq) / 30000.0 : 0.0;
        const double cost = rounds * len * pace + combine;
        if (cost < best) { best = cost; splits = s; }
    }
    return splits;
}

// Whether the kernels that give every row a wavefront of its own beat the tile kernels on the general path.  Both are priced as
// the time of one wavefront (one workgroup of four) times how often the chip is filled; the constants are fitted (least
// regret) to both sides measured at 1705 sizes a direction: 1 to 4096 keys and 1 to 85 rows a head, 2 to 4096 heads, ten
// widths, both types.  Taking the cheaper, forward / backward are more than a tenth slower than the row kernels at 46 / 93 of
// them (1.9 times at most), where the tile kernels alone were at over 400 / 600 (38 / 53 times).  4096 heads, fp32, D = 64, rows x
// keys (rows / tiles, us): forward 1 x 1 7.4 / 31, 4 x 16 22 / 31, 16 x 16 71 / 34; backward 1 x 1 14 / 83, 8 x 8 103 / 105,
// 16 x 16 250 / 122.
struct GeneralPrice {
    double row, row_dot, row_sum;                        // a row: fixed, per 64 keys and feature, per key and 64 features
    double tile, tile_block, tile_load, one_by_one, one_by_one_16;  // a tile: fixed, per 64 keys, and per padded feature of it
    double rows_per_cu, tiles_per_cu;                    // resident (tiles: times the workgroups per CU that the width leaves)
};
constexpr GeneralPrice kFwdPrice{2.9, 0.031, 0.058, 2.4, 0.9, 0.0012, 0.041, 0.021, 42.5, 0.82};
constexpr GeneralPrice kBwdPrice{0.14, 0.0013, 0.096, 0.81, 0.23, 0.0016, 0.045, 0.026, 61.0, 2.97};
double rows_minus_tiles(const GeneralPrice& c, nfd_dtype_t dtype, int64_t BH, int64_t rows, int64_t keys, int D, int num_cus) {
    const int DP = nfd::general::padded_width(D);
    const double k64 = (double)((keys + 63) / 64);
    const double load = c.tile_load + (D % 4 == 0 ? 0.0 : c.one_by_one + (dtype == NFD_BF16 ? c.one_by_one_16 : 0.0));
    const double row = (c.row + k64 * c.row_dot * D + (double)keys * c.row_sum * ((D + 63) / 64)) *
                       std::max(1.0, (double)(BH * rows) / (c.rows_per_cu * num_cus));
    const double tile = (c.tile + k64 * (c.tile_block + load * DP)) *
                        std::max(1.0, (double)(BH * ((rows + 15) / 16)) / (c.tiles_per_cu * std::min(8, 256 / DP) * num_cus));
    return row - tile;
}
bool rows_pay_fwd(nfd_dtype_t dtype, int64_t BH, int64_t Sq, int64_t Sk, int D, int num_cus) {
    return rows_minus_tiles(kFwdPrice, dtype, BH, Sq, Sk, D, num_cus) < 0;
}
bool rows_pay_bwd(nfd_dtype_t dtype, int64_t BH, int64_t Sq, int64_t Sk, int D, int num_cus) {
    return rows_minus_tiles(kBwdPrice, dtype, BH, Sq, Sk, D, num_cus) + rows_minus_tiles(kBwdPrice, dtype, BH, Sk, Sq, D, num_cus) < 0;
}

// Call f with the instance of the general kernels for these arguments: (element type, padded width, how features are loaded,
// 16-column blocks per workgroup).  `aligned`: all tensors 16-byte aligned.
template <typename Launch>
void general_dispatch(nfd_dtype_t dtype, int D, bool aligned, int cols, Launch f) {
    using namespace nfd::general;
    auto width = [&](auto e, auto dp) {
        constexpr int DP = decltype(dp)::value;
        auto load = [&](auto l) {
            if constexpr (DP <= 64)
                if (cols == 2) return f(e, dp, l, std::integral_constant<int, 2>{});
            f(e, dp, l, std::integral_constant<int, 1>{});
        };
        if constexpr (sizeof(e) == 4 || DP != 64)  // bf16 with D = 64 takes the other path
            if (aligned && D == DP) return load(std::integral_constant<int, kWhole>{});
        if (aligned && D % 4 == 0) return load(std::integral_constant<int, kGroups>{});
        load(std::integral_constant<int, kSingle>{});
    };
    auto type = [&](auto e) {
        switch (padded_width(D)) {
            case 32: return width(e, std::integral_constant<int, 32>{});
            case 64: return width(e, std::integral_constant<int, 64>{});
            case 128: return width(e, std::integral_constant<int, 128>{});
            default: return width(e, std::integral_constant<int, 256>{});
        }
    };
    if (dtype == NFD_FP32) type(0.f);
    else type((__bf16)0.f);
}

int64_t shift_blocks(const nfd::ShiftRun& r) { return (r.rows * r.d + 255) / 256; }
// Launch `blocks` blocks in pieces: a launch holds fewer than 2^32 threads.  (Blocks that walked several runs each did away with
// the pieces, but took 114 registers for 80 and a tenth to a third longer.)
template <typename Launch>
void in_pieces(int64_t blocks, Launch go) {
    constexpr int64_t kPiece = 1 << 23;
    for (int64_t first = 0; first < blocks; first += kPiece) go(first, dim3((unsigned)std::min(blocks - first, kPiece)));
}

// Kept units that land where only dropped ones were can be copied.  That is the better way where few are kept: the chains' grid
// covers the dropped ones (8 sequences of 16 heads, 64 frames of 576, 60 dropped: 23 us copied, 151 as chains; 33 of 64
// frames of 336: 133 and 120), and without vectors also where about as many are (8-bit, 33 of 64 frames, caches off a 16-byte
// boundary: 200 and 336).
bool shift_copied(const nfd::ShiftRun& r, bool vec) { return r.len <= (vec ? r.d / 2 : r.d); }

// A chain of the one-pass move is walked by one thread.  Past this many links (very many frames kept for each one dropped)
// the walk takes longer than copying the kept frames out to the workspace and back: 16 heads, 16 tokens a frame, one
// frame dropped: 7.1 against 9.6 us at 63 links, 11.5 against 9.5 at 127, 37 against 22 at 511.
constexpr int64_t kMaxShiftChain = 96;
bool shift_staged(const nfd_attn_t* h, const nfd::ShiftRun& r, size_t unit_bytes, int tensors) {
    return r.len > kMaxShiftChain * r.d && (size_t)(r.rows * r.len) * unit_bytes * tensors <= h->workspace_bytes;
}

}  // namespace

extern "C" {

int64_t nfd_attn_visible_pairs(int T, int kv_frames, int q_frames) {
    if (T < 1 || q_frames < 1 || kv_frames < q_frames) return -1;
    const int64_t P = (int64_t)kv_frames - q_frames, n = q_frames;
    return (int64_t)T * T * (n * P + n * (n + 1) / 2);
}

int nfd_attn_check_args(nfd_dtype_t dtype, int B, int H, int F, int T, int D, int kv_frames, int q_frames) {
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1 || q_frames < 1 || kv_frames < 1) return NFD_ERR_SHAPE;
    if (q_frames > kv_frames) return NFD_ERR_SHAPE;
    if (kv_frames > F) return NFD_ERR_CAPACITY;
    if (dtype != NFD_BF16 && dtype != NFD_FP32) return NFD_ERR_UNSUPPORTED;
    if (D > nfd::general::kMaxD) return NFD_ERR_UNSUPPORTED;
    // 32-bit row indexing inside the kernels
    if ((int64_t)F * T > (int64_t)1 << 30 || (int64_t)B * H > (int64_t)1 << 24) return NFD_ERR_UNSUPPORTED;
    return NFD_OK;
}

// The schedule, and how the launch deals it out: the row ranges per head (the plan's query tiles, or more and smaller ones) and
// whether the kernel for short key splits runs them.
enum class FwdKind { kPlain, kLse, kFp8 };
struct FwdDeal {
    int ranges;
    bool short_splits;
};
static int plan_impl(nfd_dtype_t dtype, int B, int H, int F, int T, int D, int kv_frames, int q_frames, int num_cus,
                     size_t workspace_limit, FwdKind kind, nfd_attn_plan_t* plan, FwdDeal* deal) {
    const bool kv8 = kind == FwdKind::kFp8;
    const int rc = nfd_attn_check_args(dtype, B, H, F, T, D, kv_frames, q_frames);
    if (rc != NFD_OK) return rc;
    if (num_cus <= 0) num_cus = 256;
    if (workspace_limit == 0) workspace_limit = kDefaultWorkspace;
    const int64_t BH = (int64_t)B * H, Sq = (int64_t)q_frames * T;
    const int P = kv_frames - q_frames;
    nfd_attn_plan_t pl{};
    if (dtype == NFD_BF16 && D == nfd::mfma::kD) {
        pl.kernel = 1;
        pl.block_n = nfd::mfma::kBN;
        const FwdPrice& c = kv8 ? kPrice8 : kPrice16;
        const double kv_bytes = (double)BH * kv_frames * T * nfd::mfma::kD * (kv8 ? 2.0 : 4.0);
        const int64_t blocks = (Sq + 31) / 32, tiles256 = (blocks + 7) / 8;
        const bool few = BH * tiles256 * 4 < (int64_t)num_cus;  // query tiles of 128 rows in the plan, too
        pl.block_m = few ? nfd::mfma::kBM / 2 : nfd::mfma::kBM;
        const RowRanges r = row_ranges(Sq, T, P, pl.block_m);
        pl.n_q_tiles = r.count;
        const int most = tile_splits(r, few, BH, Sq, num_cus, workspace_limit);
        int splits = most;
        *deal = {r.count, false};
        // Few 128-row tiles, key splits: the small kernel on the 32x32x16 instruction, three workgroups per CU, unless the chains
        // are long and nearly all wavefronts have rows.  Both at their best split count (us, small / pipelined): 24 heads, one
        // frame of 40 tokens over 49 11.1 / 11.9; 16 heads, two of 105 over 4 10.2 / 10.7; 48 heads, 152 over 39 (five row blocks
        // of eight) 25.3 / 27.1; 16 heads, two of 336 over 32 (21 of 24) 46.4 / 46.8, one (eleven of twelve) 29.7 / 28.7.  Over
        // the 8-bit cache the small kernel: 16 heads, one of 336 over 32 32.6 / 33.9.
        const bool full = blocks * 10 >= (int64_t)r.count * 4 * 9 && r.longest >= 8 * (int64_t)most;
        if (few && most > 1 && kind != FwdKind::kLse && (kv8 || !full)) {
            deal->short_splits = true;
        } else if (few || BH * tiles256 < 4 * (int64_t)num_cus) {  // past two rounds the 256-row links are the cheaper ones
            const bool six = (blocks + r.count - 1) / r.count == nfd::mfma::kBM48 / 32;
            const RowRanges r128 = few ? r : row_ranges(Sq, T, P, nfd::mfma::kBM / 2);
            // not for a tie; and splits for splits only where the price is clearly lower (the prices are within 8 %)
            double best = few ? 1e300 : 0.98 * fwd_price(c, r, pl.block_m, six, BH, Sq, kv_bytes, num_cus, most);
            for (int s = 1; s <= (kv8 ? 1 : most); ++s) {
                const double t = fwd_price(c, r128, nfd::mfma::kBM / 2, false, BH, Sq, kv_bytes, num_cus, s) * (s > 1 && !few ? 1.08 : 1.0);
                if (t < best) { best = t; splits = s; deal->ranges = r128.count; }
            }
        }
        if (kv8 && splits > 1 && (blocks + deal->ranges - 1) / deal->ranges <= 4) deal->short_splits = true;
        const int64_t visited = r.tiles;
        pl.n_splits = splits;
        if (BH * deal->ranges * splits > (int64_t)0x7fffffff) return NFD_ERR_UNSUPPORTED;  // grid size
        pl.n_workgroups = (int)(BH * pl.n_q_tiles * splits);
        pl.key_tiles_visited = visited * BH;
        pl.key_tiles_dense = (int64_t)pl.n_q_tiles * (((int64_t)kv_frames * T + pl.block_n - 1) / pl.block_n) * BH;
        pl.workspace_bytes = splits > 1 ? (size_t)(BH * Sq) * splits * kPartialRowBytes : 0;
    } else {
        pl.kernel = 0;
        *deal = {0, false};
        const bool rows = rows_pay_fwd(dtype, BH, Sq, (int64_t)kv_frames * T, D, num_cus);
        pl.block_m = rows ? nfd::rows::kRowsPerWorkgroup : 16 * nfd::general::cols_per_workgroup(Sq, BH, D, num_cus, true);
        pl.block_n = rows ? 64 : 16;
        pl.n_q_tiles = (int)((Sq + pl.block_m - 1) / pl.block_m);
        pl.n_splits = 1;
        const int64_t workgroups = rows ? (BH * Sq + pl.block_m - 1) / pl.block_m : BH * pl.n_q_tiles;
        if (workgroups > (int64_t)0x7fffffff) return NFD_ERR_UNSUPPORTED;
        pl.n_workgroups = (int)workgroups;
        const int64_t step = rows ? 1 : pl.block_m;  // rows that walk the same keys
        int64_t visited = 0;
        for (int64_t r = 0; r < Sq; r += step)
            visited += (kmax_rows(std::min<int64_t>(r + step, Sq) - 1, T, P) + pl.block_n - 1) / pl.block_n;
        pl.key_tiles_visited = visited * BH;
        pl.key_tiles_dense = (Sq + step - 1) / step * (((int64_t)kv_frames * T + pl.block_n - 1) / pl.block_n) * BH;
        pl.workspace_bytes = 0;
    }
    *plan = pl;
    return NFD_OK;
}

int nfd_attn_plan(nfd_dtype_t dtype, int B, int H, int F, int T, int D, int kv_frames, int q_frames,
                  int num_cus, size_t workspace_limit, nfd_attn_plan_t* plan) {
    if (!plan) return NFD_ERR_NULL;
    FwdDeal deal;
    return plan_impl(dtype, B, H, F, T, D, kv_frames, q_frames, num_cus, workspace_limit, FwdKind::kPlain, plan, &deal);
}

int nfd_attn_fwd_ranges(nfd_dtype_t dtype, int B, int H, int F, int T, int D, int kv_frames, int q_frames, int num_cus, int fp8kv,
                        int* ranges, int* n_splits) {
    if (!ranges || !n_splits) return NFD_ERR_NULL;
    nfd_attn_plan_t pl;
    FwdDeal deal;
    const int rc = plan_impl(dtype, B, H, F, T, D, kv_frames, q_frames, num_cus, 0, fp8kv ? FwdKind::kFp8 : FwdKind::kPlain, &pl, &deal);
    if (rc != NFD_OK) return rc;
    *ranges = deal.ranges;
    *n_splits = pl.n_splits;
    return rc;
}

int nfd_attn_bwd_form(nfd_dtype_t dtype, int B, int H, int F, int T, int D, int kv_frames, int q_frames, int num_cus, int* form) {
    if (!form) return NFD_ERR_NULL;
    const int rc = nfd_attn_check_args(dtype, B, H, F, T, D, kv_frames, q_frames);
    if (rc != NFD_OK) return rc;
    if (num_cus <= 0) num_cus = 256;
    const int64_t BH = (int64_t)B * H, Sq = (int64_t)q_frames * T, Sk = (int64_t)kv_frames * T;
    if (dtype == NFD_BF16 && D == nfd::mfma::kD) *form = (int)bwd_form(BH, Sq, Sk, T, kv_frames - q_frames, num_cus);
    else *form = rows_pay_bwd(dtype, BH, Sq, Sk, D, num_cus) ? NFD_BWD_ROWS : NFD_BWD_TILES;
    return NFD_OK;
}

int nfd_attn_q_tile_rows(int rows, int n_q_tiles, int q_tile, int* first_row, int* n_rows) {
    if (!first_row || !n_rows) return NFD_ERR_NULL;
    if (rows < 1 || n_q_tiles < 1 || q_tile < 0 || q_tile >= n_q_tiles) return NFD_ERR_SHAPE;
    if (rows > 1 << 30) return NFD_ERR_UNSUPPORTED;  // the row limit of the attention calls (32-bit indexing)
    const int n_blocks = (rows + 31) / 32;
    int b0, nb;
    nfd::mfma::q_tile_blocks(q_tile, n_blocks / n_q_tiles, n_blocks % n_q_tiles, &b0, &nb);
    *first_row = std::min(32 * b0, rows);  // more tiles than blocks (never planned): the surplus tiles are empty
    *n_rows = std::min(32 * (b0 + nb), rows) - *first_row;
    return NFD_OK;
}

int nfd_attn_work_item(int BH, int n_q_tiles, int n_splits, int group_q_tiles, unsigned block, int* bh, int* q_tile,
                       int* split) {
    if (!bh || !q_tile || !split) return NFD_ERR_NULL;
    if (BH < 1 || n_q_tiles < 1 || n_splits < 1) return NFD_ERR_SHAPE;
    const nfd::mfma::WorkItem w = nfd::mfma::work_item_of(block, BH, n_q_tiles, n_splits, group_q_tiles);
    if (!w.valid) return NFD_ERR_SHAPE;
    *bh = w.bh; *q_tile = w.q_tile; *split = w.split;
    return NFD_OK;
}

int nfd_attn_create(nfd_attn_t** out, nfd_dtype_t dtype, int device, size_t workspace_bytes) {
    if (!out) return NFD_ERR_NULL;
    *out = nullptr;
    if (dtype != NFD_BF16 && dtype != NFD_FP32) return NFD_ERR_UNSUPPORTED;
    nfd_attn_t* h = new (std::nothrow) nfd_attn();
    if (!h) return NFD_ERR_ALLOC;
    h->dtype = dtype;
    h->device = device;
    h->workspace = nullptr;
    h->workspace_bytes = workspace_bytes ? workspace_bytes : kDefaultWorkspace;
    h->plan_limit = h->workspace_bytes;
    h->err[0] = 0;
    int prev = 0;
    hipError_t e = hipGetDevice(&prev);
    if (e == hipSuccess) e = hipSetDevice(device);
    hipDeviceProp_t prop;
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, device);
    if (e != hipSuccess) {
        delete h;
        return NFD_ERR_HIP;
    }
    h->num_cus = prop.multiProcessorCount;
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
        (void)hipSetDevice(prev);
        delete h;
        return NFD_ERR_UNSUPPORTED;  // the kernels are written for CDNA4 only
    }
    e = hipMalloc(&h->workspace, h->workspace_bytes);
    (void)hipSetDevice(prev);
    if (e != hipSuccess) {
        delete h;
        return NFD_ERR_ALLOC;
    }
    *out = h;
    return NFD_OK;
}

int nfd_attn_destroy(nfd_attn_t* h) {
    if (!h) return NFD_OK;
    hipError_t e = hipSuccess;
    if (h->workspace) e = hipFree(h->workspace);
    delete h;
    return e == hipSuccess ? NFD_OK : NFD_ERR_HIP;
}

const char* nfd_last_error(const nfd_attn_t* h) { return h ? h->err : "null handle"; }

static void launch_frame_copy(nfd_attn_t* h, size_t es, void* kd, void* vd, const void* ks, const void* vs, int64_t BH,
                              int64_t head_dst, int64_t head_src, int64_t off_dst, int64_t off_src, int64_t len,
                              hipStream_t st);

// k_scale / v_scale non-null: k and v are the 8-bit caches (see nfd_kvcache_append_fp8).
// k_new / v_new non-null: the query frames' own K/V, to be appended to the caches k, v by this call (they are written).
static int fwd_impl(nfd_attn_t* h, const void* q, const void* k, const void* v, void* out, float* lse, int B,
                    int H, int F, int T, int D, int kv_frames, int q_frames, float scale, void* stream,
                    const float* k_scale = nullptr, const float* v_scale = nullptr, const void* k_new = nullptr,
                    const void* v_new = nullptr) {
    if (!h) return NFD_ERR_NULL;
    if (!q || !k || !v || !out) return fail(h, NFD_ERR_NULL, "q, k, v and out must be non-null");
    const bool kv8 = k_scale != nullptr;
    const bool append = k_new != nullptr;
    nfd_attn_plan_t pl;
    FwdDeal deal;
    const int rc = plan_impl(h->dtype, B, H, F, T, D, kv_frames, q_frames, h->num_cus, h->plan_limit,
                             kv8 ? FwdKind::kFp8 : lse ? FwdKind::kLse : FwdKind::kPlain, &pl, &deal);
    if (rc != NFD_OK) return fail(h, rc, "invalid shape arguments");
    // A schedule that would write partials past the workspace must never reach the device.
    if (pl.workspace_bytes > h->workspace_bytes)
        return fail(h, NFD_ERR_ALLOC, "key-split partials (%zu bytes) exceed the scratch memory (%zu bytes)", pl.workspace_bytes,
                    h->workspace_bytes);
    if (const int dc = check_device(h)) return dc;
    // The matrix-core kernels move 16-byte vectors; a view that starts in the middle of a vector would fault.
    if (pl.kernel == 1 && (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) % 16 != 0 || (uintptr_t)lse % 4 != 0))
        return fail(h, NFD_ERR_UNSUPPORTED, "q, k, v, out must be 16-byte aligned (lse 4-byte)");
    if (kv8 && pl.kernel != 1) return fail(h, NFD_ERR_UNSUPPORTED, "the 8-bit cache is built for bf16 queries and head width 64");
    if (append && pl.kernel == 1 && (((uintptr_t)k_new | (uintptr_t)v_new) % 16 != 0))
        return fail(h, NFD_ERR_UNSUPPORTED, "k_new and v_new must be 16-byte aligned");
    if (!(scale > 0.f)) scale = 1.0f / std::sqrt((float)D);

    nfd::FwdParams p{};
    p.k_scale = k_scale; p.v_scale = v_scale;
    p.Spad = (int)(((int64_t)F * T + 63) / 64 * 64);
    p.q = q; p.k = k; p.v = v; p.out = out;
    p.lse = lse;
    p.BH = B * H;
    p.Sq = q_frames * T;
    p.Sk = kv_frames * T;
    p.Scap = F * T;
    p.T = T;
    p.P = kv_frames - q_frames;
    p.D = D;
    p.n_q_tiles = pl.n_q_tiles;
    unsigned workgroups = (unsigned)pl.n_workgroups;
    if (pl.kernel == 1) {
        const int n_blocks = (p.Sq + 31) / 32;
        p.n_q_tiles = deal.ranges;
        p.blocks_lo = n_blocks / deal.ranges;
        p.n_hi = n_blocks % deal.ranges;
        workgroups = (unsigned)((int64_t)p.BH * deal.ranges * pl.n_splits);
    }
    p.n_splits = pl.n_splits;
    // K and V of all heads against the last-level cache
    p.group_q_tiles = pl.n_splits > 1 ? (double)p.BH * p.Sk * nfd::mfma::kD * 2.0 * (kv8 ? 1.0 : 2.0) > kLastLevelBytes
                                      : nfd::mfma::head_group(p.BH);
    p.scale_log2e = scale * nfd::kLog2e;
    p.Snew0 = 0x7fffffff;
    if (append) {
        // In the matrix-core kernel the workgroups read the new rows where they are and copy them into the cache on
        // the side (at most four 16-byte vectors of each tensor per thread); otherwise a copy launch goes first.
        const int64_t n_vec = (int64_t)p.BH * p.Sq * (nfd::mfma::kD / 8);
        if (pl.kernel == 1 && !kv8 && n_vec <= (int64_t)4 * workgroups * nfd::mfma::kWaves * 64) {
            p.k_new = k_new; p.v_new = v_new;
            p.Snew0 = p.P * T;
        } else {
            const int64_t frame_elems = (int64_t)T * D;
            launch_frame_copy(h, elem_size(h->dtype), const_cast<void*>(k), const_cast<void*>(v), k_new, v_new, (int64_t)B * H,
                              (int64_t)F * frame_elems, (int64_t)q_frames * frame_elems, (int64_t)p.P * frame_elems, 0,
                              (int64_t)q_frames * frame_elems, (hipStream_t)stream);
        }
    }
    if (pl.n_splits > 1) {
        p.part_o = (__bf16*)h->workspace;
        p.part_ml = (float*)(p.part_o + (size_t)p.BH * pl.n_splits * p.Sq * nfd::mfma::kD);
    }
    hipStream_t st = (hipStream_t)stream;

    if (pl.kernel == 1) {
        const dim3 grid(workgroups), block(nfd::mfma::kWaves * 64);
        auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, p); };
        using namespace nfd::mfma;
        // Which kernel runs a range depends on the 32-row blocks the largest one holds.  Measured: 8 sequences of 16
        // heads, one frame over 40 cached ones (forward / with log-sum-exp / 8-bit cache, us).
        //   1..4  one block per wavefront (which of the two such kernels: see the plan)
        //   six   48 rows per wavefront, all wavefronts with the same work: 59.9 / 62.3 / 59.3, against 65.4 / 69.0 / 70.5 with
        //         two wavefronts of 64 rows and two of 32 (which lack the pipelined loop) at the same barriers; one frame of 576
        //         tokens over 64: 750 -> 685.  At five blocks 48 rows take 49.6 against 48.5, and splitting 42 blocks into
        //         seven tiles of six instead of six of seven 75.6 against 76.5 (90.1 against 85.9 over the 8-bit cache).
        //   five  over the 8-bit cache also 48 rows: 8 sequences of 16 heads, one frame of 150 over 63: 71.8, with 64 rows 76.0 (76.3 of the
        //         kernel before); 12 such sizes take 0.93 to 1.02 of what 64 rows take.
        const int tile_blocks = p.blocks_lo + (p.n_hi > 0);
        if (tile_blocks <= 4) {
            if (deal.short_splits && kv8) go(attn_fwd_bf16_d64<true>);
            else if (deal.short_splits) go(attn_fwd_bf16_d64<false>);
            else if (kv8) go(attn_fwd_bf16_d64_m16<false, true, 2>);
            else if (lse) go(attn_fwd_bf16_d64_m16<true, false, 2>);  // training pair: scores from the queries as given
            else go(attn_fwd_bf16_d64_m16<false, false, 2>);
        } else if (!(tile_blocks == kBM48 / 32 || (kv8 && tile_blocks == 5))) {
            if (kv8) go(attn_fwd_bf16_d64_m16<false, true, 4>);
            else if (lse) go(attn_fwd_bf16_d64_m16<true, false, 4>);
            else go(attn_fwd_bf16_d64_m16<false, false, 4>);
        } else {
            if (kv8) go(attn_fwd_bf16_d64_m16<false, true, 3>);
            else if (lse) go(attn_fwd_bf16_d64_m16<true, false, 3>);
            else go(attn_fwd_bf16_d64_m16<false, false, 3>);
        }
        if (pl.n_splits > 1) {
            const int64_t total = (int64_t)p.BH * p.Sq * (nfd::mfma::kD / 4);
            hipLaunchKernelGGL(nfd::mfma::attn_combine_d64, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, p);
        }
    } else if (pl.block_m == nfd::rows::kRowsPerWorkgroup) {
        const dim3 grid(pl.n_workgroups), block(nfd::rows::kRowsPerWorkgroup * 64);
        if (h->dtype == NFD_FP32) hipLaunchKernelGGL(nfd::rows::attn_fwd_rows<float>, grid, block, 0, st, p);
        else hipLaunchKernelGGL(nfd::rows::attn_fwd_rows<__bf16>, grid, block, 0, st, p);
    } else {
        const bool aligned = ((uintptr_t)q | (uintptr_t)k | (uintptr_t)v) % 16 == 0;
        general_dispatch(h->dtype, D, aligned, pl.block_m / 16, [&](auto e, auto dp, auto load, auto cols) {
            hipLaunchKernelGGL((nfd::general::attn_fwd_general<decltype(e), decltype(dp)::value, decltype(load)::value, decltype(cols)::value>),
                               dim3(pl.n_workgroups), dim3(nfd::general::kWaves * 64), 0, st, p);
        });
    }
    return check_hip(h, hipGetLastError(), "attention launch");
}

int nfd_block_causal_attn_fwd(nfd_attn_t* h, const void* q, const void* k, const void* v, void* out, int B,
                              int H, int F, int T, int D, int kv_frames, int q_frames, float scale,
                              void* stream) {
    return fwd_impl(h, q, k, v, out, nullptr, B, H, F, T, D, kv_frames, q_frames, scale, stream);
}

// ---- forward for callers that cannot allocate ---------------------------------------------------------
// The key-split partials go to a fixed array in the code object instead of a handle's workspace.  `scratch`
// is only a host-side stand-in for the symbol: the address the kernels get is the one hipGetSymbolAddress
// returns with the device current, looked up once per device and kept in that device's pseudo-handle.
namespace {
constexpr size_t kStaticScratchBytes = NFD_NOALLOC_SCRATCH_BYTES;
constexpr int kStaticMaxDevices = 64;
struct StaticDevice {
    bool ready;
    void* scratch_ptr;  // device address of `scratch` on this device
    int num_cus;
};
StaticDevice g_static_dev[kStaticMaxDevices];
std::mutex g_static_mu;
}  // namespace
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

int nfd_block_causal_attn_fwd_noalloc(nfd_dtype_t dtype, const void* q, const void* k, const void* v, void* out, int B,
                                      int H, int F, int T, int D, int kv_frames, int q_frames, float scale, void* stream,
                                      char* err, size_t err_len) {
    nfd_attn local{};  // pseudo-handle on the stack: nothing is allocated, the error text lands in its buffer
    auto done = [&](int rc) {
        if (err && err_len) {
            std::strncpy(err, rc == NFD_OK ? "" : local.err, err_len - 1);
            err[err_len - 1] = 0;
        }
        return rc;
    };
    if (dtype != NFD_BF16 && dtype != NFD_FP32) return done(fail(&local, NFD_ERR_UNSUPPORTED, "unknown dtype"));
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return done(check_hip(&local, e, "hipGetDevice"));
    if (dev < 0 || dev >= kStaticMaxDevices) return done(fail(&local, NFD_ERR_UNSUPPORTED, "device index beyond the table of this entry point"));
    {
        std::lock_guard<std::mutex> lock(g_static_mu);
        StaticDevice& sd = g_static_dev[dev];
        if (!sd.ready) {  // first call on this device, with it current: where this device keeps its copy of the array
            void* ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) return done(check_hip(&local, e == hipSuccess ? hipErrorInvalidSymbol : e, "hipGetSymbolAddress(scratch)"));
            hipDeviceProp_t prop;
            e = hipGetDeviceProperties(&prop, dev);
            if (e != hipSuccess) return done(check_hip(&local, e, "hipGetDeviceProperties"));
            if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
                return done(fail(&local, NFD_ERR_UNSUPPORTED, "the kernels are written for gfx950 only"));
            sd.scratch_ptr = ptr;
            sd.num_cus = prop.multiProcessorCount;
            sd.ready = true;
        }
        local.workspace = sd.scratch_ptr;  // never the array's name: that is not a device address
        local.num_cus = sd.num_cus;
    }
    local.dtype = dtype;
    local.device = dev;
    local.workspace_bytes = kStaticScratchBytes;
    // The schedule is the one a handle with the default workspace would get, so the result is bit-identical to
    // nfd_block_causal_attn_fwd's; a call whose partials do not fit the array is refused (NFD_ERR_ALLOC), not re-planned.
    local.plan_limit = kDefaultWorkspace;
    return done(fwd_impl(&local, q, k, v, out, nullptr, B, H, F, T, D, kv_frames, q_frames, scale, stream));
}

int nfd_kvcache_append_attn_fwd(nfd_attn_t* h, const void* q, void* k_cache, void* v_cache, const void* k_new,
                                const void* v_new, void* out, int B, int H, int F, int T, int D, int kv_frames,
                                int q_frames, float scale, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k_new || !v_new) return fail(h, NFD_ERR_NULL, "k_new and v_new must be non-null");
    return fwd_impl(h, q, k_cache, v_cache, out, nullptr, B, H, F, T, D, kv_frames, q_frames, scale, stream, nullptr, nullptr,
                    k_new, v_new);
}

int nfd_block_causal_attn_fwd_lse(nfd_attn_t* h, const void* q, const void* k, const void* v, void* out,
                                  float* lse, int B, int H, int F, int T, int D, int kv_frames, int q_frames,
                                  float scale, void* stream) {
    if (h && !lse) return fail(h, NFD_ERR_NULL, "lse must be non-null");
    return fwd_impl(h, q, k, v, out, lse, B, H, F, T, D, kv_frames, q_frames, scale, stream);
}

int nfd_fp8_cache_bytes(int B, int H, int F, int T, int D, size_t* bytes) {
    if (!bytes) return NFD_ERR_NULL;
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1) return NFD_ERR_SHAPE;
    if (D != nfd::mfma::kD) return NFD_ERR_UNSUPPORTED;
    if ((int64_t)F * T > (int64_t)1 << 30 || (int64_t)B * H > (int64_t)1 << 24) return NFD_ERR_UNSUPPORTED;
    const int64_t Spad = ((int64_t)F * T + 63) / 64 * 64;
    *bytes = (size_t)B * H * Spad * D;
    return NFD_OK;
}

int nfd_block_causal_attn_fwd_fp8kv(nfd_attn_t* h, const void* q, const void* k8, const void* v8t,
                                    const float* k_scale, const float* v_scale, void* out, int B, int H, int F,
                                    int T, int D, int kv_frames, int q_frames, float scale, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k_scale || !v_scale) return fail(h, NFD_ERR_NULL, "k_scale and v_scale must be non-null");
    if ((uintptr_t)k_scale % 4 != 0 || (uintptr_t)v_scale % 4 != 0)
        return fail(h, NFD_ERR_UNSUPPORTED, "scales must be 4-byte aligned");
    return fwd_impl(h, q, k8, v8t, out, nullptr, B, H, F, T, D, kv_frames, q_frames, scale, stream, k_scale, v_scale);
}

int nfd_kvcache_append_fp8(nfd_attn_t* h, void* k8, void* v8t, const float* k_scale, const float* v_scale,
                           const void* k_new, const void* v_new, int B, int H, int F, int T, int D, int frame_pos,
                           int n_frames, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k8 || !v8t || !k_scale || !v_scale || !k_new || !v_new)
        return fail(h, NFD_ERR_NULL, "caches, scales and new tensors must be non-null");
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1 || n_frames < 0 || frame_pos < 0)
        return fail(h, NFD_ERR_SHAPE, "invalid shape arguments");
    if ((int64_t)frame_pos + n_frames > F) return fail(h, NFD_ERR_CAPACITY, "frame_pos + n_frames exceeds the cache capacity F");
    if (h->dtype != NFD_BF16 || D != nfd::mfma::kD)
        return fail(h, NFD_ERR_UNSUPPORTED, "the 8-bit cache is built for bf16 inputs and head width 64");
    if ((int64_t)F * T > (int64_t)1 << 30 || (int64_t)B * H > (int64_t)1 << 24)
        return fail(h, NFD_ERR_UNSUPPORTED, "shape beyond the 32-bit row indexing of the kernels");
    if (((uintptr_t)k8 | (uintptr_t)v8t | (uintptr_t)k_new | (uintptr_t)v_new) % 16 != 0 ||
        ((uintptr_t)k_scale | (uintptr_t)v_scale) % 4 != 0)
        return fail(h, NFD_ERR_UNSUPPORTED, "caches and new tensors must be 16-byte aligned (scales 4-byte)");
    if (n_frames == 0) return NFD_OK;
    if (const int dc = check_device(h)) return dc;
    const int n_rows = n_frames * T, j0 = frame_pos * T, BH = B * H;
    const int64_t Spad = ((int64_t)F * T + 63) / 64 * 64;
    hipStream_t st = (hipStream_t)stream;
    const unsigned gy = (unsigned)std::min(BH, 65535);
    const unsigned k_blocks = (unsigned)(((int64_t)n_rows * 8 + 255) / 256), v_blocks = (unsigned)((n_rows + 63) / 64);
    hipLaunchKernelGGL(nfd::kvcache_append_fp8, dim3(k_blocks + v_blocks, gy), dim3(256), 0, st, (const __bf16*)k_new,
                       (const __bf16*)v_new, (unsigned char*)k8, (unsigned char*)v8t, k_scale, v_scale, n_rows, Spad, j0,
                       BH, k_blocks);
    return check_hip(h, hipGetLastError(), "8-bit kvcache append launch");
}

int nfd_block_causal_attn_bwd(nfd_attn_t* h, const void* q, const void* k, const void* v, const void* out,
                              const void* dout, const float* lse, void* dq, void* dk, void* dv, int B, int H,
                              int F, int T, int D, int kv_frames, int q_frames, float scale, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!q || !k || !v || !out || !dout || !lse || !dq || !dk || !dv)
        return fail(h, NFD_ERR_NULL, "all tensors of the backward call must be non-null");
    const int rc = nfd_attn_check_args(h->dtype, B, H, F, T, D, kv_frames, q_frames);
    if (rc != NFD_OK) return fail(h, rc, "invalid shape arguments");
    const int64_t BH = (int64_t)B * H, Sq = (int64_t)q_frames * T, Sk = (int64_t)kv_frames * T;
    if (h->dtype != NFD_BF16 || D != nfd::mfma::kD) {
        if (const int dc = check_device(h)) return dc;
        // general path: fp32 arithmetic
        if ((size_t)(BH * Sq) * sizeof(float) > h->workspace_bytes)
            return fail(h, NFD_ERR_ALLOC, "the per-row workspace of the backward exceeds the handle's workspace");
        nfd::general::BwdParams g{};
        const int cq = nfd::general::cols_per_workgroup(Sq, BH, D, h->num_cus, false), ck = nfd::general::cols_per_workgroup(Sk, BH, D, h->num_cus, false);
        g.n_q_tiles = (int)((Sq + 16 * cq - 1) / (16 * cq));
        g.n_k_tiles = (int)((Sk + 16 * ck - 1) / (16 * ck));
        if (BH * g.n_q_tiles > (int64_t)0x7fffffff || BH * g.n_k_tiles > (int64_t)0x7fffffff)
            return fail(h, NFD_ERR_UNSUPPORTED, "too many rows for one launch of the general backward");
        if (!(scale > 0.f)) scale = 1.0f / std::sqrt((float)D);
        g.q = q; g.k = k; g.v = v; g.out = out; g.dout = dout; g.lse = lse;
        g.delta = (float*)h->workspace;
        g.dq = dq; g.dk = dk; g.dv = dv;
        g.BH = (int)BH; g.Sq = (int)Sq; g.Sk = (int)Sk; g.Scap = F * T; g.T = T; g.P = kv_frames - q_frames; g.D = D;
        g.scale = scale;
        g.scale_log2e = scale * nfd::kLog2e;
        hipStream_t gs = (hipStream_t)stream;
        const dim3 blk(nfd::general::kWaves * 64);
        if (rows_pay_bwd(h->dtype, BH, Sq, Sk, D, h->num_cus)) {
            constexpr int kR = nfd::rows::kRowsPerWorkgroup;
            const int64_t nq = (BH * Sq + kR - 1) / kR, nk = (BH * Sk + kR - 1) / kR;
            if (nq > (int64_t)0x7fffffff || nk > (int64_t)0x7fffffff)
                return fail(h, NFD_ERR_UNSUPPORTED, "too many rows for one launch of the general backward");
            const dim3 gq((unsigned)nq), gk((unsigned)nk), b4(kR * 64);
            if (h->dtype == NFD_BF16) {
                hipLaunchKernelGGL(nfd::rows::attn_bwd_dq_rows<__bf16>, gq, b4, 0, gs, g);
                hipLaunchKernelGGL(nfd::rows::attn_bwd_dkdv_rows<__bf16>, gk, b4, 0, gs, g);
            } else {
                hipLaunchKernelGGL(nfd::rows::attn_bwd_dq_rows<float>, gq, b4, 0, gs, g);
                hipLaunchKernelGGL(nfd::rows::attn_bwd_dkdv_rows<float>, gk, b4, 0, gs, g);
            }
            return check_hip(h, hipGetLastError(), "general backward launch");
        }
        const bool aligned = ((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out | (uintptr_t)dout) % 16 == 0;
        general_dispatch(h->dtype, D, aligned, cq, [&](auto e, auto dp, auto load, auto cols) {
            hipLaunchKernelGGL((nfd::general::attn_bwd_dq_general<decltype(e), decltype(dp)::value, decltype(load)::value, decltype(cols)::value>),
                               dim3((unsigned)(BH * g.n_q_tiles)), blk, 0, gs, g);
        });
        general_dispatch(h->dtype, D, aligned, ck, [&](auto e, auto dp, auto load, auto cols) {
            hipLaunchKernelGGL((nfd::general::attn_bwd_dkdv_general<decltype(e), decltype(dp)::value, decltype(load)::value, decltype(cols)::value>),
                               dim3((unsigned)(BH * g.n_k_tiles)), blk, 0, gs, g);
        });
        return check_hip(h, hipGetLastError(), "general backward launch");
    }
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out | (uintptr_t)dout | (uintptr_t)dq | (uintptr_t)dk |
         (uintptr_t)dv) % 16 != 0 || (uintptr_t)lse % 4 != 0)
        return fail(h, NFD_ERR_UNSUPPORTED, "tensors must be 16-byte aligned (lse 4-byte)");
    if ((size_t)(BH * Sq) * 2 * sizeof(float) > h->workspace_bytes)
        return fail(h, NFD_ERR_ALLOC, "the per-row workspace of the backward exceeds the handle's workspace");
    if (!(scale > 0.f)) scale = 1.0f / std::sqrt((float)D);

    nfd::mfma::BwdParams p{};
    p.q = q; p.k = k; p.v = v; p.dout = dout; p.out = out; p.lse = lse;
    p.neg_delta = (float*)h->workspace;
    p.lse2 = p.neg_delta + BH * Sq;
    p.dq = dq; p.dk = dk; p.dv = dv;
    p.BH = (int)BH; p.Sq = (int)Sq; p.Sk = (int)Sk; p.Scap = F * T; p.T = T; p.P = kv_frames - q_frames;
    const BwdForm pick = bwd_form(BH, Sq, Sk, T, kv_frames - q_frames, h->num_cus);
    const int rows = pick == BwdForm::kMergedSmall ? 128 : 256, keys = pick == BwdForm::kMergedSmall ? 64 : 192;
    p.n_q_tiles = (int)((Sq + rows - 1) / rows);
    p.n_k_blocks = (int)((Sk + keys - 1) / keys);
    p.scale = scale;
    p.scale_log2e = scale * nfd::kLog2e;
    if (BH * ((int64_t)p.n_q_tiles + p.n_k_blocks) > (int64_t)0x7fffffff)
        return fail(h, NFD_ERR_UNSUPPORTED, "too many workgroups for one launch of the backward");
    if (const int dc = check_device(h)) return dc;
    hipStream_t st = (hipStream_t)stream;
    if (pick == BwdForm::kSeparate) {
        // the dq kernel first: it writes the two per-row vectors that the dk/dv kernel reads
        hipLaunchKernelGGL(nfd::mfma::attn_bwd_dq_bf16_d64, dim3((unsigned)(BH * p.n_q_tiles)), dim3(256), 0, st, p);
        hipLaunchKernelGGL(nfd::mfma::attn_bwd_dkdv_bf16_d64, dim3((unsigned)(BH * p.n_k_blocks)), dim3(256), 0, st, p);
    } else {
        hipLaunchKernelGGL(nfd::mfma::attn_bwd_delta, dim3((unsigned)((BH * Sq * 8 + 255) / 256)), dim3(256), 0, st, p);
        const dim3 grid((unsigned)(BH * (p.n_q_tiles + p.n_k_blocks)));
        if (pick == BwdForm::kMerged) hipLaunchKernelGGL((nfd::mfma::attn_bwd_merged<4, 3, 4, 2>), grid, dim3(256), 0, st, p);
        else hipLaunchKernelGGL((nfd::mfma::attn_bwd_merged<2, 1, 3, 3>), grid, dim3(256), 0, st, p);
    }
    return check_hip(h, hipGetLastError(), "backward launch");
}

// Launch one frame-run copy (see kvcache_copy) of two tensors of equal geometry, or of one (vd == nullptr);
// all counts in elements of es bytes.
static void launch_frame_copy(nfd_attn_t* h, size_t es, void* kd, void* vd, const void* ks, const void* vs, int64_t BH,
                              int64_t head_dst, int64_t head_src, int64_t off_dst, int64_t off_src, int64_t len,
                              hipStream_t st) {
    const bool pair = vd != nullptr;
    const bool vec = (head_dst * es) % 16 == 0 && (head_src * es) % 16 == 0 && (off_dst * es) % 16 == 0 &&
                     (off_src * es) % 16 == 0 && (len * es) % 16 == 0 && ((uintptr_t)kd % 16 == 0) &&
                     ((uintptr_t)vd % 16 == 0) && ((uintptr_t)ks % 16 == 0) && ((uintptr_t)vs % 16 == 0);
    const dim3 block(256);
    auto grid_for = [&](int64_t units) {
        const int64_t gy = std::min<int64_t>(BH, 65535);
        const int64_t want_x = std::max<int64_t>(1, ((int64_t)h->num_cus * 32 + gy - 1) / gy);  // enough blocks to fill the chip
        return dim3((unsigned)std::min<int64_t>((units + 255) / 256, want_x), (unsigned)gy);
    };
    auto go = [&](auto tag, int64_t f) {  // f = elements per unit of the copy type
        typedef decltype(tag) E;
        if (pair)
            hipLaunchKernelGGL((nfd::kvcache_copy<E, true>), grid_for(len / f), block, 0, st, (E*)kd, (E*)vd, (const E*)ks,
                               (const E*)vs, head_dst / f, head_src / f, off_dst / f, off_src / f, len / f, BH);
        else
            hipLaunchKernelGGL((nfd::kvcache_copy<E, false>), grid_for(len / f), block, 0, st, (E*)kd, (E*)nullptr,
                               (const E*)ks, (const E*)nullptr, head_dst / f, head_src / f, off_dst / f, off_src / f,
                               len / f, BH);
    };
    if (vec) go(nfd::u32x4{}, (int64_t)(16 / es));
    else if (es == 1) go((unsigned char)0, 1);
    else if (es == 2) go((uint16_t)0, 1);
    else go((uint32_t)0, 1);
}

int nfd_kvcache_append(nfd_attn_t* h, void* k_cache, void* v_cache, const void* k_new, const void* v_new, int B,
                       int H, int F, int T, int D, int frame_pos, int n_frames, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k_cache || !v_cache || !k_new || !v_new) return fail(h, NFD_ERR_NULL, "cache and new tensors must be non-null");
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1 || n_frames < 0 || frame_pos < 0)
        return fail(h, NFD_ERR_SHAPE, "invalid shape arguments");
    if ((int64_t)frame_pos + n_frames > F) return fail(h, NFD_ERR_CAPACITY, "frame_pos + n_frames exceeds the cache capacity F");
    if (n_frames == 0) return NFD_OK;
    if (const int dc = check_device(h)) return dc;
    const int64_t frame_elems = (int64_t)T * D;
    launch_frame_copy(h, elem_size(h->dtype), k_cache, v_cache, k_new, v_new, (int64_t)B * H, (int64_t)F * frame_elems,
                      (int64_t)n_frames * frame_elems, (int64_t)frame_pos * frame_elems, 0,
                      (int64_t)n_frames * frame_elems, (hipStream_t)stream);
    return check_hip(h, hipGetLastError(), "kvcache append launch");
}

int nfd_kvcache_shift(nfd_attn_t* h, void* k_cache, void* v_cache, int B, int H, int F, int T, int D,
                      int kv_frames, int n_drop, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k_cache || !v_cache) return fail(h, NFD_ERR_NULL, "caches must be non-null");
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1 || kv_frames < 0 || n_drop < 0 || n_drop > kv_frames)
        return fail(h, NFD_ERR_SHAPE, "invalid shape arguments");
    if (kv_frames > F) return fail(h, NFD_ERR_CAPACITY, "kv_frames exceeds the cache capacity F");
    if (n_drop == 0 || kv_frames == n_drop) return NFD_OK;
    if (const int dc = check_device(h)) return dc;
    const size_t es = elem_size(h->dtype);
    const int64_t frame = (int64_t)T * D, BH = (int64_t)B * H;
    const bool vec = ((size_t)frame * es) % 16 == 0 && ((uintptr_t)k_cache | (uintptr_t)v_cache) % 16 == 0;
    const int64_t f = vec ? (int64_t)(16 / es) : 1;  // elements per unit
    const int64_t stride = (int64_t)F * frame / f, d = n_drop * frame / f, len = (kv_frames - n_drop) * frame / f;
    const nfd::ShiftRun rk{k_cache, stride, BH, d, len}, rv{v_cache, stride, BH, d, len};
    hipStream_t st = (hipStream_t)stream;
    if (shift_copied(rk, vec)) {
        launch_frame_copy(h, es, k_cache, v_cache, k_cache, v_cache, BH, stride * f, stride * f, 0, d * f, len * f, st);
        return check_hip(h, hipGetLastError(), "kvcache shift launch");
    }
    if (shift_staged(h, rk, f * es, 2)) {
        void* ks = h->workspace;
        void* vs = (char*)h->workspace + (size_t)(BH * len * f) * es;
        launch_frame_copy(h, es, ks, vs, k_cache, v_cache, BH, len * f, stride * f, 0, d * f, len * f, st);
        launch_frame_copy(h, es, k_cache, v_cache, ks, vs, BH, stride * f, len * f, 0, 0, len * f, st);
        return check_hip(h, hipGetLastError(), "kvcache shift launch");
    }
    const int64_t nb = shift_blocks(rk);
    in_pieces(2 * nb, [&](int64_t first, dim3 grid) {
        const dim3 block(256);
        if (vec) hipLaunchKernelGGL(nfd::kvcache_shift_inplace<nfd::u32x4>, grid, block, 0, st, rk, rv, nb, first);
        else if (es == 2) hipLaunchKernelGGL(nfd::kvcache_shift_inplace<uint16_t>, grid, block, 0, st, rk, rv, nb, first);
        else hipLaunchKernelGGL(nfd::kvcache_shift_inplace<uint32_t>, grid, block, 0, st, rk, rv, nb, first);
    });
    return check_hip(h, hipGetLastError(), "kvcache shift launch");
}

int nfd_kvcache_shift_fp8(nfd_attn_t* h, void* k8, void* v8t, int B, int H, int F, int T, int D, int kv_frames,
                          int n_drop, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k8 || !v8t) return fail(h, NFD_ERR_NULL, "caches must be non-null");
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1 || kv_frames < 0 || n_drop < 0 || n_drop > kv_frames)
        return fail(h, NFD_ERR_SHAPE, "invalid shape arguments");
    if (kv_frames > F) return fail(h, NFD_ERR_CAPACITY, "kv_frames exceeds the cache capacity F");
    if (D != nfd::mfma::kD) return fail(h, NFD_ERR_UNSUPPORTED, "the 8-bit cache is built for head width 64");
    if ((int64_t)F * T > (int64_t)1 << 30 || (int64_t)B * H > (int64_t)1 << 24)
        return fail(h, NFD_ERR_UNSUPPORTED, "shape beyond the 32-bit row indexing of the kernels");
    if (n_drop == 0 || kv_frames == n_drop) return NFD_OK;
    const int64_t Spad = ((int64_t)F * T + 63) / 64 * 64, BH = (int64_t)B * H;
    const int64_t keep_keys = (int64_t)(kv_frames - n_drop) * T;
    // part of the call's contract; nothing is staged there any more
    if (T % 16 != 0 && h->workspace_bytes < (size_t)keep_keys)
        return fail(h, NFD_ERR_ALLOC, "for T that is no multiple of 16 the workspace must hold a feature row of the kept keys");
    if (const int dc = check_device(h)) return dc;
    hipStream_t st = (hipStream_t)stream;
    // K codes: BH heads of Spad rows x 64 bytes, a frame = T rows; V codes: BH * 64 feature rows of Spad bytes, a frame =
    // T bytes of each.  When T is a multiple of 16 whole 16-key groups of V move (the order inside them is untouched).
    const bool vec = ((uintptr_t)k8 | (uintptr_t)v8t) % 16 == 0;
    const int64_t f = vec ? 16 : 1;  // bytes per unit
    const nfd::ShiftRun rk{k8, Spad * D / f, BH, (int64_t)n_drop * T * D / f, keep_keys * D / f};
    const bool copied = shift_copied(rk, vec), staged = !copied && vec && shift_staged(h, rk, 16, 1);
    if (copied) {
        launch_frame_copy(h, 1, k8, nullptr, k8, nullptr, BH, Spad * D, Spad * D, 0, (int64_t)n_drop * T * D, keep_keys * D, st);
        if (T % 16 == 0) {
            launch_frame_copy(h, 1, v8t, nullptr, v8t, nullptr, BH * D, Spad, Spad, 0, (int64_t)n_drop * T, keep_keys, st);
            return check_hip(h, hipGetLastError(), "8-bit kvcache shift launch");
        }
    } else if (staged) {
        launch_frame_copy(h, 16, h->workspace, nullptr, k8, nullptr, BH, rk.len, rk.stride, 0, rk.d, rk.len, st);
        launch_frame_copy(h, 16, k8, nullptr, h->workspace, nullptr, BH, rk.stride, rk.len, 0, 0, rk.len, st);
    }
    const int64_t nb = copied || staged ? 0 : shift_blocks(rk);
    const dim3 block(256);
    if (vec && T % 16 == 0) {
        const nfd::ShiftRun rv{v8t, Spad / 16, BH * D, (int64_t)n_drop * T / 16, keep_keys / 16};
        in_pieces(nb + rv.rows, [&](int64_t first, dim3 grid) {
            hipLaunchKernelGGL((nfd::kvcache_shift_fp8_inplace<nfd::u32x4, nfd::u32x4, false>), grid, block, 0, st, rk, rv, nb, first);
        });
    } else {
        const nfd::ShiftRun rv{v8t, Spad, BH * D, (int64_t)n_drop * T, keep_keys};
        in_pieces(nb + rv.rows, [&](int64_t first, dim3 grid) {
            if (vec) hipLaunchKernelGGL((nfd::kvcache_shift_fp8_inplace<nfd::u32x4, unsigned char, true>), grid, block, 0, st, rk, rv, nb, first);
            else hipLaunchKernelGGL((nfd::kvcache_shift_fp8_inplace<unsigned char, unsigned char, true>), grid, block, 0, st, rk, rv, nb, first);
        });
    }
    return check_hip(h, hipGetLastError(), "8-bit kvcache shift launch");
}

// ---- speculative sampling bookkeeping (host only) ---------------------------------------------
int nfd_spec_init(nfd_spec_t* s, int capacity, int window, int n_spec, int n_prompt, int total) {
    if (!s) return NFD_ERR_NULL;
    if (capacity < 1 || window < 1 || n_spec < 1 || n_prompt < 1 || total < n_prompt) return NFD_ERR_SHAPE;
    if ((int64_t)window + n_spec > capacity || n_prompt > capacity) return NFD_ERR_CAPACITY;
    s->capacity = capacity; s->window = window; s->n_spec = n_spec; s->total = total;
    s->done = n_prompt; s->cached = n_prompt; s->t_offset = 0;
    return NFD_OK;
}

int nfd_spec_next(nfd_spec_t* s, nfd_spec_step_t* step) {
    if (!s || !step) return NFD_ERR_NULL;
    if (s->done >= s->total) return 0;
    step->n_drop = std::max(0, s->cached - s->window);  // keep at most `window` frames of context
    s->cached -= step->n_drop;
    s->t_offset += step->n_drop;
    step->n_frames = std::min(s->n_spec, s->total - s->done);
    step->frame_pos = s->cached;
    step->kv_frames = s->cached + step->n_frames;
    step->q_frames = step->n_frames;
    step->t_offset = s->t_offset;
    return 1;
}

int nfd_spec_accept(nfd_spec_t* s, const nfd_spec_step_t* step, const int32_t* actions, int action_dim,
                    int* accepted) {
    if (!s || !step || !actions || !accepted) return NFD_ERR_NULL;
    if (action_dim < 1 || step->n_frames < 1 || s->done + step->n_frames > s->total) return NFD_ERR_SHAPE;
    // frames were generated under the action of frame `done` repeated: keep the leading run that matches
    const int32_t* a0 = actions + (int64_t)s->done * action_dim;
    int n = 1;
    for (; n < step->n_frames; ++n) {
        const int32_t* an = actions + (int64_t)(s->done + n) * action_dim;
        bool same = true;
        for (int d = 0; d < action_dim; ++d) same = same && an[d] == a0[d];
        if (!same) break;
    }
    *accepted = n;
    s->done += n;
    s->cached = step->frame_pos + n;  // the rejected frames' K/V are simply overwritten by the next append
    return NFD_OK;
}

int nfd_rope_check_args(nfd_dtype_t dtype, int B, int H, int F, int T, int D, int frame_pos, int n_frames,
                        int grid_h, int grid_w, int n_t, int n_h, int n_w) {
    if (B < 1 || H < 1 || F < 1 || T < 1 || D < 1 || n_frames < 0 || frame_pos < 0) return NFD_ERR_SHAPE;
    if (grid_h < 1 || grid_w < 1 || (int64_t)grid_h * grid_w != T) return NFD_ERR_SHAPE;
    if (n_t < 0 || n_h < 0 || n_w < 0 || ((n_t | n_h | n_w) & 1) || (int64_t)n_t + n_h + n_w != D) return NFD_ERR_SHAPE;
    if ((int64_t)frame_pos + n_frames > F) return NFD_ERR_CAPACITY;
    if (dtype != NFD_BF16 && dtype != NFD_FP32) return NFD_ERR_UNSUPPORTED;
    if (D > 2 * nfd::kRopeMaxPairs) return NFD_ERR_UNSUPPORTED;
    if ((int64_t)F * T > (int64_t)1 << 30 || (int64_t)B * H > (int64_t)1 << 24) return NFD_ERR_UNSUPPORTED;
    return NFD_OK;
}

// k_scale / v_scale non-null: k_cache and v_cache are the 8-bit caches.
static int rope_impl(nfd_attn_t* h, const void* q, void* q_out, void* k_cache, void* v_cache, const void* k_new,
                     const void* v_new, int B, int H, int F, int T, int D, int frame_pos, int n_frames, int t_offset,
                     int grid_h, int grid_w, int n_t, int n_h, int n_w, float theta, void* stream,
                     const float* k_scale, const float* v_scale) {
    if (!h) return NFD_ERR_NULL;
    if (!q || !q_out || !k_cache || !v_cache || !k_new || !v_new) return fail(h, NFD_ERR_NULL, "tensors must be non-null");
    const int rc = nfd_rope_check_args(h->dtype, B, H, F, T, D, frame_pos, n_frames, grid_h, grid_w, n_t, n_h, n_w);
    if (rc != NFD_OK) return fail(h, rc, "invalid rotary-embedding arguments");
    const bool kv8 = k_scale != nullptr;
    if (kv8) {
        if (h->dtype != NFD_BF16 || D != nfd::mfma::kD)
            return fail(h, NFD_ERR_UNSUPPORTED, "the 8-bit cache is built for bf16 inputs and head width 64");
        const uintptr_t any = (uintptr_t)q | (uintptr_t)q_out | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)k_new | (uintptr_t)v_new;
        if (any % 16 != 0 || ((uintptr_t)k_scale | (uintptr_t)v_scale) % 4 != 0)
            return fail(h, NFD_ERR_UNSUPPORTED, "tensors must be 16-byte aligned (scales 4-byte)");
    }
    if (n_frames == 0) return NFD_OK;
    if (const int dc = check_device(h)) return dc;
    const double th = theta > 0.f ? (double)theta : 10000.0;
    nfd::RopeTable tab{};
    {
        const int width[3] = {n_t, n_h, n_w};
        int p = 0;
        for (int ax = 0; ax < 3; ++ax)
            for (int i = 0; i < width[ax] / 2; ++i, ++p) {
                tab.inv_freq[p] = std::pow(th, -2.0 * (double)i / (double)width[ax]);
                tab.axis[p] = (unsigned char)ax;
            }
    }
    nfd::RopeParams rp{};
    rp.BH = B * H; rp.F = F; rp.T = T; rp.D = D;
    rp.frame_pos = frame_pos; rp.n_frames = n_frames;
    rp.t_pos0 = t_offset + frame_pos;
    rp.grid_w = grid_w;
    const size_t es = elem_size(h->dtype);
    {   // a feature pair is the smallest unit a thread loads
        const uintptr_t any = (uintptr_t)q | (uintptr_t)q_out | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)k_new | (uintptr_t)v_new;
        if (any % (2 * es) != 0) return fail(h, NFD_ERR_UNSUPPORTED, "tensors must be aligned to one feature pair");
    }
    const bool aligned = ((uintptr_t)q % 16 == 0) && ((uintptr_t)q_out % 16 == 0) && ((uintptr_t)k_cache % 16 == 0) &&
                         ((uintptr_t)v_cache % 16 == 0) && ((uintptr_t)k_new % 16 == 0) && ((uintptr_t)v_new % 16 == 0);
    const int wide = (int)(16 / es);  // features per 16-byte chunk
    const int vec = (aligned && D % wide == 0) ? wide : 2;
    const int64_t items = (int64_t)n_frames * T * (D / vec);
    const int64_t gx = (items + 255) / 256;
    // enough workgroups to fill the chip, otherwise as many heads per thread as possible (the
    // cosines and sines are shared by all heads)
    const int64_t want_y = std::min<int64_t>(rp.BH, std::max<int64_t>(1, ((int64_t)h->num_cus * 8 + gx - 1) / gx));
    rp.heads_per_thread = (int)((rp.BH + want_y - 1) / want_y);
    const unsigned gy = (unsigned)((rp.BH + rp.heads_per_thread - 1) / rp.heads_per_thread);
    const dim3 grid((unsigned)gx, gy), block(256);
    hipStream_t st = (hipStream_t)stream;
    const nfd::RopeFp8 f8{k_scale, v_scale, ((int64_t)F * T + 63) / 64 * 64};
    if (kv8) {  // vec == 8 here: bf16, D = 64, all tensors 16-byte aligned
        hipLaunchKernelGGL((nfd::rope_kvcache_append<__bf16, 8, true>), grid, block, 0, st, (const __bf16*)q, (__bf16*)q_out,
                           (__bf16*)k_cache, (__bf16*)v_cache, (const __bf16*)k_new, (const __bf16*)v_new, rp, tab, f8);
    } else if (h->dtype == NFD_BF16) {
        if (vec == 8)
            hipLaunchKernelGGL((nfd::rope_kvcache_append<__bf16, 8, false>), grid, block, 0, st, (const __bf16*)q, (__bf16*)q_out,
                               (__bf16*)k_cache, (__bf16*)v_cache, (const __bf16*)k_new, (const __bf16*)v_new, rp, tab, f8);
        else
            hipLaunchKernelGGL((nfd::rope_kvcache_append<__bf16, 2, false>), grid, block, 0, st, (const __bf16*)q, (__bf16*)q_out,
                               (__bf16*)k_cache, (__bf16*)v_cache, (const __bf16*)k_new, (const __bf16*)v_new, rp, tab, f8);
    } else {
        if (vec == 4)
            hipLaunchKernelGGL((nfd::rope_kvcache_append<float, 4, false>), grid, block, 0, st, (const float*)q, (float*)q_out,
                               (float*)k_cache, (float*)v_cache, (const float*)k_new, (const float*)v_new, rp, tab, f8);
        else
            hipLaunchKernelGGL((nfd::rope_kvcache_append<float, 2, false>), grid, block, 0, st, (const float*)q, (float*)q_out,
                               (float*)k_cache, (float*)v_cache, (const float*)k_new, (const float*)v_new, rp, tab, f8);
    }
    return check_hip(h, hipGetLastError(), "rotary embedding launch");
}

int nfd_rope_kvcache_append(nfd_attn_t* h, const void* q, void* q_out, void* k_cache, void* v_cache,
                            const void* k_new, const void* v_new, int B, int H, int F, int T, int D,
                            int frame_pos, int n_frames, int t_offset, int grid_h, int grid_w, int n_t,
                            int n_h, int n_w, float theta, void* stream) {
    return rope_impl(h, q, q_out, k_cache, v_cache, k_new, v_new, B, H, F, T, D, frame_pos, n_frames, t_offset, grid_h,
                     grid_w, n_t, n_h, n_w, theta, stream, nullptr, nullptr);
}

int nfd_rope_kvcache_append_fp8(nfd_attn_t* h, const void* q, void* q_out, void* k8, void* v8t, const float* k_scale,
                                const float* v_scale, const void* k_new, const void* v_new, int B, int H, int F,
                                int T, int D, int frame_pos, int n_frames, int t_offset, int grid_h, int grid_w,
                                int n_t, int n_h, int n_w, float theta, void* stream) {
    if (!h) return NFD_ERR_NULL;
    if (!k_scale || !v_scale) return fail(h, NFD_ERR_NULL, "k_scale and v_scale must be non-null");
    return rope_impl(h, q, q_out, k8, v8t, k_new, v_new, B, H, F, T, D, frame_pos, n_frames, t_offset, grid_h, grid_w,
                     n_t, n_h, n_w, theta, stream, k_scale, v_scale);
}

}  // extern "C"
