// Records shared by the host planner and the gfx950 kernels, and the launch entry points the host
// side calls.  Not part of the public boundary (that is include/lora.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lora {

// One group of tokens that share an adapter (host-side planning record).
struct SegRec {
    uint64_t a_off;     // element offset of A^T [r8][in] in the arena
    uint64_t b_off;     // element offset of B^T [out][r8] in the arena
    int64_t v_off;      // float offset of the group's first v row
    int32_t rank;
    int32_t r8;         // rank rounded up to a multiple of 8 (row length of v and of B^T)
    float scale;
    int32_t tok_start;  // first sorted position of the group in perm
    int32_t ntok;
    int32_t pad[5];
};
static_assert(sizeof(SegRec) == 64, "SegRec is 64 bytes");

// One work group's share, self-contained so that a work group needs a single round trip to memory
// before it can issue its weight loads.  128 bytes: the first 64 are read with scalar loads, the
// token list with one vector load.
struct Unit {
    uint64_t w_off;   // element offset of the unit's first weight row (A^T row p0 / B^T row p0)
    int64_t v_off;    // float offset of the unit's first v element (shrink: row tok0, column p0;
                      // expand: row tok0, column 0)
    int32_t r8;       // padded rank = row length of v and of B^T
    int32_t ntok;     // tokens in this unit: 1..16 (decode units), up to 64 (expand, prefill shrink above rank 64) or 32 (prefill shrink)
    int32_t p0;       // shrink: first rank row; expand: first output column
    int32_t pn;       // shrink: valid rank rows (1..16, multiple of 8 except the tail); expand: columns
    int32_t ks;       // shrink: k-slice index
    float scale;
    int32_t seg;
    int32_t tok0;     // first token, relative to the group
    int32_t sync_idx; // counter of this unit's (group, token tile) in a fused launch
    int32_t sync_n;   // shrink units that feed that counter per launch
    int32_t perm_off; // position of the unit's first token in the device copy of perm
    int32_t turn;     // token-heavy shrink units: the adapter, by which they begin their walk along k with another pass
    int32_t tok[16];  // batch row index of each token; entries >= ntok repeat tok[0] (units of <= 16
                      // tokens; larger units read perm[perm_off + i])
};
static_assert(sizeof(Unit) == 128, "Unit is 128 bytes");

// One run of at most 16 places of the adapted layer's row order (lora_linear: groups that fill blocks of 16 rows,
// then the tokens without adapter, then the small groups) that share an adapter and lie in one block of 16
// places.  A block of a large group holds one piece, a block of small groups one per adapter met there, or (where the plan
// gives every group blocks of its own) one beside empty places: the delta of a piece is added with the rows of the other
// pieces of its block at zero.
struct LinPiece {
    uint64_t b_off;  // element offset of the group's B^T in the arena
    int64_t v_off;   // element offset of the v row of the piece's first token
    int32_t r8;      // padded rank
    int32_t ntok;    // tokens in the piece, 1..16
    int32_t place;   // place of the first token; its row within the block is place mod 16
    int32_t pad;
};
static_assert(sizeof(LinPiece) == 32, "LinPiece is 32 bytes");
// The blocks of 16 places as a launch needs them: pieces[start[i]] .. pieces[start[i + 1] - 1] (device memory) are
// the adapters of places 16 i .. 16 i + 15; the first big_tiles * kLinTileM places take large tiles.
struct LinBlock {
    const int32_t *start;
    const LinPiece *pieces;
    int big_tiles;
};
constexpr int kComputeUnits = 256;  // of the chip
constexpr int kLinTileM = 256;  // rows of a work group's output tile (the row order is padded to a multiple)
constexpr int kLinTileN = 256;  // columns of it: two 128-column strips of B^T (the last tile of a row may hold one)

#define LORA_MAX_RANK_PADDED 256
constexpr int kTokTile = 16;   // tokens per MFMA tile (the N of a 16x16x32 MFMA)
constexpr int kRowTile = 16;   // rank rows / output columns per MFMA tile (the M)
constexpr int kThreads = 256;  // 4 wavefronts per work group

// Consecutive 64-token expand units of the same number of columns, but for those at the end of a row of y.
struct BigSection {
    int n_units, cols;
};
constexpr int kMaxBigSections = 8;  // one per projection at most

struct LaunchCtx {
    const Unit *units;
    const int32_t *perm;
    const uint16_t *arena;
    int n_units;
    int n_work;    // of n_units, those that hold tokens (lists of token-heavy shrink units are filled up with others)
    int top_rank;  // lists of token-heavy shrink units: the largest padded rank
    int n_high;    // lists of 64-token expand units: how many are above rank 128
    // lists of 64-token expand units: in which runs of equally wide ones (host memory)
    const BigSection *sections;
    int n_sections;
    int in_features;
    int out_features;
    // shrink launches that leave v as bf16 hi + lo: store s_a v (rounded to fp32 once, then split) instead of v,
    // for a consumer that adds v B_a straight into accumulators of its own (lora_linear)
    int scale_v;
};

// Hand-over of v through the segment table's counters (see the kernels): arrivals and ready counters
// per (group, token tile), the complete v as bf16 hi + lo, the launch epoch and the poll limit.
struct SyncArgs {
    unsigned *counters;
    unsigned *ready;
    unsigned *timeout_flag;
    uint16_t *v_hi;
    uint16_t *v_lo;
    unsigned epoch;
    unsigned spin_limit;
    // the k-slices' partial sums of v, which expand units of up to 16 tokens then add up themselves; NULL: the shrink launch
    // completes v_hi and v_lo
    const float *parts = nullptr;
    int n_slices = 0;
    int64_t slice_stride = 0;
};

// v_out[ks * slice_stride + ...] receives k-slice ks's partial sums (slice_stride = 0 when there is
// a single slice).  With `sync` and no sync->parts, the unit that completes a token tile also writes the tile's
// summed v as bf16 hi + lo.
hipError_t launch_shrink(const LaunchCtx &c, const uint16_t *x, int64_t ldx, int k_slice_len, float *v_out,
                         int n_slices, int64_t slice_stride, const SyncArgs *sync, hipStream_t stream);

// Whole-k shrink units: work groups of 16 wavefronts, four per k-slice of k_slice_len (n_slices <= 4
// slices cover in_features); v written complete, either as fp32 into v_f32 or (v_hi != NULL) as bf16
// hi + lo, bitwise what the k-slice units of launch_shrink give.  more_than_one_round: the launch has more
// units than the chip has compute units; it then runs as work groups of 8 wavefronts, two per compute unit
// (same bits).
hipError_t launch_shrink_wide(const LaunchCtx &c, bool more_than_one_round, const uint16_t *x, int64_t ldx,
                              int k_slice_len, int n_slices, float *v_f32, uint16_t *v_hi, uint16_t *v_lo,
                              hipStream_t stream);

// Without `sync`: v_in is v itself, fp32 and complete.  With `sync`: v comes from sync->v_hi / v_lo, or (units of up to
// 16 tokens, sync->parts) from the k-slices there, written by a shrink launch of the same epoch, v_in is not read.
// `big`: the list holds units of up to 64 tokens (token indices through perm).
hipError_t launch_expand(const LaunchCtx &c, bool big, const float *v_in, uint16_t *y, int64_t ldy, const SyncArgs *sync,
                         hipStream_t stream);

// Which launches of token-heavy shrink units alone take two work groups a unit, half of the rank rows each (see RankRows in the
// kernels; units up to rank 32 are not halved).  Counted without the places that only fill lists up: few prompts of unlike ranks have
// many.  Shrink launch in us, whole / halves: 93 units of ranks up to 219 in 176 places, 1344 features, 12.4 / 9.6, 89 of ranks 8 and
// 256 in 232, 512 features, 8.9 / 6.0, 104 of ranks 8 to 128 in 152, 896 features, 10.1 / 8.4; one prompt of 2000 tokens,
// 4096 features, rank 128 (128 units, cut along k) 15.4 / 13.1; beyond, 134 units of ranks 8 and 256, 1536 features, 13.1 / 14.2, 132 of rank
// 256 cut along k, 3392 features, 19.8 / 21.1, 174 of ranks 8 to 128 12.9 / 14.6, though 154 of ranks 8 to 128, 960 features, 11.5 / 9.2.
// Nothing above rank 32, in the halves' kernel all the same: 58 units of rank 8, 1536 features, 4.6 / 5.4, 123 of rank 32, 512 features,
// 4.2 / 4.8, 102 at 2560 features 6.2 / 6.8: it runs two work groups per compute unit where their own runs four.
constexpr int kHeavyHalvesMaxUnits = kComputeUnits / 2;
inline bool shrink_in_halves(const LaunchCtx &c) { return c.n_work <= kHeavyHalvesMaxUnits && c.top_rank > 32; }

// Shrink of token-heavy groups: one unit = (group, up to 32 tokens, all rank rows, the whole of k).
// n_hi = how many of the units are above rank 64: with none, the launch takes the kernel that fits four
// work groups on a compute unit, otherwise the one for any rank (two per compute unit).
// Writes complete v: as bf16 hi + lo into v_hi / v_lo, or (v_f32 != NULL) as fp32 into v_f32.  Units cut by
// k (sync_n = slices of the unit's tokens, ks = which) put their sums into slices of `parts` and complete v
// through `sync`'s counters (apply), or into n_slices slices of v_f32 for the caller to add up, those beyond the
// unit's own set to zero (stand-alone shrink, sync = NULL).
hipError_t launch_shrink_prefill(const LaunchCtx &c, int n_hi, const uint16_t *x, int64_t ldx, uint16_t *v_hi,
                                 uint16_t *v_lo, float *v_f32, int n_slices, int64_t slice_stride, float *parts,
                                 const SyncArgs *sync, hipStream_t stream);

// The work groups of a launch of 64-token expand units: rows of 8 units, each unit in pieces of kBigCols columns.
constexpr int kBigCols = 256;
inline int64_t big_places(const LaunchCtx &c)
{
    int64_t places = 0;
    for (int i = 0; i < c.n_sections; ++i)
        places += (int64_t)(c.sections[i].n_units + 7) / 8 * 8 * ((c.sections[i].cols + kBigCols - 1) / kBigCols);
    return places;
}
// Whether such a launch, of its own, asks for so much LDS that three work groups run on a compute unit and not four: up to rank 128, where
// less of y is under way at a time (see the kernel), but not where four hold all of it and a fourth of it would wait for the others to end.
// us a call, 512 features, three / four a compute unit, 769 to 1024 work groups: 4096 columns, 4096 tokens, rank 16 19.0 / 18.4, rank 128 26.1 /
// 24.7; 8192, two prompts of 900, rank 16 18.3 / 17.4, rank 128 25.7 / 24.2; 14336, 1024 tokens, rank 16 17.9 / 17.7, two of 512, rank 128 25.2 /
// 24.3, but rank 64 19.6 / 20.2; 1800 tokens, 8192, rank 64 18.7 / 19.0; over 160 such batches 2 % faster.
inline bool big_spread(const LaunchCtx &c) { return c.top_rank <= 128 && big_places(c) > 4 * kComputeUnits; }
// lora_expand's launches of these units, v as the caller has it (fp32 in rows): whether work groups walk up to `walk_strips` strips of their unit
// and load v once (k_expand_walk, two on a compute unit) or take 256 columns as elsewhere.  The latter load v twice a strip above rank 128, the
// former fill the chip only with enough units; where most units are above rank 128 an estimate decides (in us at rank 256; other ranks differ by
// a factor common to both).  lora_expand alone, us, 256 columns a work group / walks: 4096 columns, rank 256, 31 tiles of 64 tokens 16.0 / 16.3, 48 23.7 /
// 25.3, 63 30.1 / 26.1, 125 53.6 / 43.7, 300 119 / 114; 1024 columns, 63 tiles 10.0 / 12.4, 300 36.6 / 43.1; 2048 columns, 31 tiles 9.2 / 11.9; 8064
// columns, rank 192, 17 tiles 19.2 / 20.7, 125 87 / 67; 4736 columns, 130 tiles, 8 of 520 walks in a second round, 88 / 110; 14336 columns, rank
// 160, 125 tiles 139 / 105.  Half of the units at rank 8 and half at 256 level; one group of eight above rank 128 the walks 38 % slower; up to
// rank 128 (one chunk, v once a strip) level or slower (8064 columns, 63 tiles, rank 96 29.3 / 29.9; but 4096 columns, 125 tiles, rank 128 31.2 / 29.4).
inline int walk_strips(const LaunchCtx &c)
{
    const int most = c.sections[0].cols / 128, parts = most < 2 * kComputeUnits / c.n_units ? most : 2 * kComputeUnits / c.n_units;
    return parts > 1 ? (most + parts - 1) / parts : most;
}
inline bool expand_walks(const LaunchCtx &c)
{
    if (c.n_sections != 1 || 2 * c.n_high <= c.n_units) return false;
    const int most = c.sections[0].cols / 128, strips = walk_strips(c);
    const int64_t walks = (int64_t)c.n_units * ((most + strips - 1) / strips), round = 2 * kComputeUnits;
    const double rounds = walks <= round ? 1.0 : 0.75 * (double)((walks + round - 1) / round) + 0.25 * (double)walks / round;
    const double high = (double)c.n_high / c.n_units;  // (the others take half as long by 256 columns, and as long in walks)
    const double by_256 =
        1.5 + (0.45 + 0.55 * high) * (most == 1 ? 3.7 : 6.9) * (double)((big_places(c) + kComputeUnits - 1) / kComputeUnits);
    return rounds * (6.5 + 4.7 * strips) < 1.06 * by_256;
}

// A mixed batch's shrink in one launch: the token-heavy units of `heavy` (n_hi of them above rank 64),
// then the k-slice units of `c`, which leave partial sums in `parts` and complete v through `sync` where
// launch_shrink does.  Likewise the expand: the 64-token units of `big`, which read v from sync->v_hi / v_lo, then the
// units of `c`, which add sync->parts up or, without them, read v_hi / v_lo too.
hipError_t launch_shrink_mixed(const LaunchCtx &heavy, int n_hi, const LaunchCtx &c, const uint16_t *x, int64_t ldx,
                               int k_slice_len, float *parts, int n_slices, int64_t slice_stride,
                               const SyncArgs *sync, hipStream_t stream);
hipError_t launch_expand_mixed(const LaunchCtx &big, const LaunchCtx &c, uint16_t *y, int64_t ldy, const SyncArgs *sync,
                               hipStream_t stream);

// Both halves in one launch (shrink units first); the expand units poll `ready` of their token tile,
// at most spin_limit times each, and add the k-slices of `parts` up.
hipError_t launch_apply_fused(const LaunchCtx &shrink, const LaunchCtx &expand, const uint16_t *x, int64_t ldx,
                              int k_slice_len, float *parts, int n_slices, int64_t slice_stride, uint16_t *y,
                              int64_t ldy, const SyncArgs *sync, hipStream_t stream);

// A decode-sized batch on the whole-k plan in one launch of `grid` work groups of 16 wavefronts (at most
// one per compute unit): work group b runs shrink.units[b], then its four groups of four wavefronts run
// expand.units[4b .. 4b+3]; places with ntok == 0 are empty.  All units of one (group, token tile) sit
// at places of one residue mod 8, i.e. on one XCD, through whose L2 v (sync->v_hi / v_lo) and the
// tile's `ready` counter are handed over; the counter grows by an expand unit's sync_n per launch and
// sync->epoch is the number of such launches since the table was uploaded, this one included.
// xcc_map: 4 bits per XCD number (0..7), its position in the order in which a launch's work groups are
// dealt to the XCDs, as a probe launch found it (probe_xcc).  sync->timeout_flag is followed by 3 words
// of detail and 2 x 256 words the launches' own check of that order uses (see the kernel).  Expand units must be a single
// column pass (pn <= 512 / 256 / 128 columns up to rank 32 / 64 / beyond).
hipError_t launch_decode_fused(const LaunchCtx &shrink, const LaunchCtx &expand, int grid, const uint16_t *x,
                               int64_t ldx, int k_slice_len, int n_slices, uint16_t *y, int64_t ldy,
                               unsigned xcc_map, const SyncArgs *sync, hipStream_t stream);

// host_out[b] = XCD number (0..15) that work group b of an n-work-group launch ran on (n <= 1024).
// Synchronises the stream.
hipError_t probe_xcc(unsigned *host_out, int n_work_groups, hipStream_t stream);

// The tiles of lora_linear's batches that take no large ones, 16 rb rows x 16 cb columns: the largest that still make a work group per
// compute unit.  4096 -> 4096, us per layer of tokens without adapter (eight weights in rotation), tiles of 64 x 64 / 32 x 64 / 32 x 32
// / 16 x 32: 16 tokens 14.8 / 12.0 / 9.4 / 8.5, 64 tokens 17.7 / 13.1 / 10.8 / 13.0, 128 tokens 18.7 / 14.2 / 18.2 / 23.8, 256 tokens 19.4
// / 23.1, 512 tokens 36.2 / 48.0 (256 x 256 tiles: 65 to 69 for each of them).
struct LinSmallTiles {
    int rb, cb;
    int64_t n;  // of them
    int grid() const { return (int)(8 * ((n + 7) / 8)); }  // an eighth of them per XCD
    bool pairs() const { return grid() > kComputeUnits; }  // k_linear_rounds, two work groups per compute unit
};
inline LinSmallTiles linear_small_tiles(int n_places, int out)
{
    auto tiles = [&](int rb, int cb) { return LinSmallTiles{rb, cb, (int64_t)((n_places + 16 * rb - 1) / (16 * rb)) * (out / (16 * cb))}; };
    auto fits = [&](int rb, int cb) { return (n_places + 15) / 16 >= rb && tiles(rb, cb).n >= kComputeUnits; };
    return fits(4, 4) ? tiles(4, 4) : fits(2, 4) ? tiles(2, 4) : fits(2, 2) ? tiles(2, 2) : tiles(1, 2);
}

// The adapted layer in one pass over y: y[row] = bf16(x[row] W + s_a v[row] B_a), W in operand order
// (launch_pack_weight), s_a v as bf16 hi + lo from a shrink launch with scale_v.  n_places places in use;
// rows[m] = batch row of place m, -1 for none and from n_places to the next multiple of kLinTileM.
hipError_t launch_linear_lora(const int32_t *rows, const LinBlock *blocks, int n_places, const uint16_t *arena,
                              const uint16_t *w_packed, const uint16_t *x, int64_t ldx, int in, int out,
                              const uint16_t *v_hi, const uint16_t *v_lo, uint16_t *y, int64_t ldy,
                              hipStream_t stream);

// W^T [out][in] row-major bf16 (the layout of a linear layer's weight) -> operand order: for every
// 128-column strip and every 32-wide k step, eight 1 KB pieces (sub-block b = columns 8n + b), piece
// (kq, n) holding k = 32 step + 8 kq .. +7 of column 128 strip + 8 n + b.
hipError_t launch_pack_weight(const uint16_t *wt, int in, int out, uint16_t *dst, hipStream_t stream);

// Copies pinned host memory that the device can read, a_bytes from `a` and behind them b_bytes from `b` (multiples of 16, less than 2 GiB),
// to dev by a kernel, which reads and writes that many bytes whatever the memory holds: the caller has made sure that it holds them.
// Weak, like the two questions below: the planner also links without the kernels.
hipError_t launch_copy_in(const void *a, size_t a_bytes, const void *b, size_t b_bytes, void *dev, hipStream_t stream) __attribute__((weak));
// Whether `bytes` from p on lie in one allocation that HIP knows (a copy asks this too, and refuses what exceeds one) ...
bool allocation_holds(const void *p, size_t bytes) __attribute__((weak));
// ... of pinned host memory that a kernel on the current device reads at the same address.
bool pinned_holds(const void *host, size_t bytes) __attribute__((weak));

// v[i] = sum over slices, in slice order.
hipError_t launch_reduce_slices(const float *parts, int n_slices, int64_t slice_stride, float *v,
                                int64_t n, hipStream_t stream);

// Writes adapter (A [in][r], B [r][out], row-major bf16, device memory) in the pool's packed,
// MFMA-operand-major form: dst_a gets r8*in elements, dst_b out*r8.
hipError_t launch_pack_adapter(const uint16_t *A, const uint16_t *B, int in, int out, int r, int r8,
                               uint16_t *dst_a, uint16_t *dst_b, hipStream_t stream);

// The library's own workspace for callers that cannot allocate: a file-scope device array of
// kStaticScratchBytes in the kernels' source file.  Gives that array's address on the current device
// (looked up once per device, then kept); the host must use this address, never the array's name.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
constexpr int kMaxDevices = 64;
hipError_t static_scratch(void **ptr);

}  // namespace lora
