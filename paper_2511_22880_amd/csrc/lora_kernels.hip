// gfx950 kernels of the co-batched LoRA delta (shrink: v = x A_a, expand: y += s_a v B_a).
//
// Both adapter matrices are stored the way a 16x16x32 bf16 MFMA reads its weight operand: lane l
// supplies row (l & 15) of a 16-row weight tile and the 8 consecutive k values 8*(l >> 4) .. +7 of a
// 32-wide k step, so the pool keeps, for every 16-row tile and every k step, the 64 lanes' 16-byte
// pieces back to back.  One wavefront load of an operand is then 1 KB of consecutive bytes (a
// row-major matrix would make it 16 pieces of 64 bytes, which costs the address path of a CU about
// 3.7 times as many cycles):
//   A^T: 16-row block jb (the last block has 8 rows when the padded rank is 8 mod 16), k step s,
//        piece (kq, row n): element offset  16*jb*in + s*(32*h) + (kq*h + n)*8,  h = rows in the block
//   B^T: 128-column strip, sub-block b (the 16 columns 8*n + b), rank piece kp (8 values), column
//        slot n: element offset  128*strip*r8 + ((b*(r8/8) + kp)*16 + n)*8
// The token operand uses the same lane->k mapping, so the order of k inside a step is irrelevant to
// the result.  The 16x16 fp32 result tile has D[4*(l >> 4) + i][l & 15] in register i of lane l.
//
// Work is cut on the host into units of roughly equal adapter bytes; one work group (4 wavefronts)
// takes one unit.  No unit ever depends on another adapter's rank.
#include "lora_internal.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace lora {

// Per-work-group device clocks, in builds with -DLORA_WG_CLOCKS only (the measurement build of the
// library; see lora_debug_clock_buffer): wavefront 0 of a work group writes the 100 MHz wall clock at a
// few points of its unit into slot (work group, point) of a caller's buffer.  Ordinary builds compile
// the macro to nothing.
#ifdef LORA_WG_CLOCKS
__device__ unsigned long long *g_clock_buf = nullptr;
__device__ unsigned g_clock_slots = 0;
#define LORA_CLOCK_SLOT(slot, point)                                                                   \
    do {                                                                                               \
        if (g_clock_buf && threadIdx.x == 0 && (slot) < g_clock_slots)                                 \
            g_clock_buf[(size_t)(slot) * 8 + (point)] = wall_clock64();                                \
    } while (0)
#else
#define LORA_CLOCK_SLOT(slot, point) do { } while (0)
#endif
#define LORA_CLOCK_AT(base, point) LORA_CLOCK_SLOT((base) + blockIdx.x, point)
#define LORA_CLOCK(point) LORA_CLOCK_AT(0, point)
// expand launches keep their clocks behind those of the shrink launch of the same apply
[[maybe_unused]] constexpr unsigned kClockExpandBase = 32768;
#define LORA_CLOCK_E(point) LORA_CLOCK_AT(kClockExpandBase, point)
// by unit where a unit has several work groups: those of its first one
#define LORA_CLOCK_E_UNIT(unit, point) LORA_CLOCK_SLOT(kClockExpandBase + (unsigned)(unit), point)

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

static __device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

static __device__ __forceinline__ uint4 ld16(const uint16_t *p) { return *reinterpret_cast<const uint4 *>(p); }

// 16-byte load of data that is read exactly once per launch (a decode batch's adapter weights, the
// x rows of a token-heavy shrink): marked non-temporal, so it is not kept in the caches on its way.
// A plain read of 2 GB runs at 6.2 TB/s on this chip with ordinary loads and at 7.0 TB/s with these.
static __device__ __forceinline__ uint4 ld16_stream(const uint16_t *p)
{
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return uint4{v.x, v.y, v.z, v.w};
}

// 16-byte store of data this launch will not read again (y).
static __device__ __forceinline__ void st16_stream(uint16_t *p, uint4 v)
{
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
}

static __device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// ------------------------------------------------------------------------------------------------
// Hand-over of v between the two halves of a fused launch.  The L2 caches of the chip's eight XCDs
// are not coherent with each other, and a device-scope fence (write back / invalidate a whole L2)
// costs far more than the data is worth.  So partial sums of v that work groups of the same launch read never
// live in a cache: they are stored and loaded with device-scope relaxed atomics (64 bits at a time), which go
// through to memory.  In the single-launch form a shrink work group waits until its stores have completed, then
// bumps the ready counter of its (group, token tile), and the expand work groups add the k-slices up
// themselves, each for its own tokens, behind a wait for all of the tile's bumps.  (With the shrink unit that
// arrived last adding them up, v took three trips through memory, a counter behind each.  Calls one after the other, us: one
// token of rank 16, 4096 -> 4096, 6.7 -> 5.8; three tokens of ranks 8 to 32, 8192 -> 8192, 9.7 -> 8.4; 60 tokens of four adapters
// of rank 16, 4096 -> 4096, 9.2 -> 8.1.)
// In launches of their own the expand units of up to 16 tokens (k_expand_parts, k_expand_mixed<kSlicesByExpand>) add the slices up as well where
// that is the shorter way (expand_adds_slices in lora_host.cpp), and the
// shrink units of k-slices leave plain stores and end: to wait for its stores, its counter and, in the last unit of a tile, for the
// other slices hold a work group's place for longer than its products take.  Calls one after the other, us, completed in the
// shrink launch / added up in the expand launch: 16 tokens of 10 adapters, 4096 -> 4096, 10.0 / 8.0; 80 tokens of four of rank 128,
// 16384 -> 16384, 21.2 / 18.2; 500 tokens of 100 adapters of rank 256, 4096 -> 4096 (6400 and 3200 units), 77.3 / 76.5.
// Else, and for lora_linear, the shrink launch completes them as bf16 hi + lo, which every column reads: a unit
// bumps the arrival counter of its tile, the one whose bump completes the tile's count adds the slices up and sets the counter back
// to zero (a launch leaves the table as it found it, so a launch replayed from a captured graph finds what the first one found).
// Token-heavy units that are cut along k do the same (complete_tile).
// The ready counters only grow (the target is epoch, the number of such launches the table has seen, times
// the tile's units), so nothing is cleared between launches.  The wait is bounded: at the limit
// the work group records it in *timeout_flag and goes on, so every wavefront reaches its end.
// Shrink units come first in the grid and never wait, and work groups are dispatched in grid order,
// so a waiting expand unit never keeps a shrink unit from running.
// ------------------------------------------------------------------------------------------------
struct Sync {
    unsigned *counters;       // arrivals, one per (group, token tile); NULL = no hand-over through counters
    unsigned *ready;          // one per tile: bumped by every shrink unit of a single-launch apply
    unsigned *timeout_flag;
    uint16_t *v_hi;           // complete v as two bf16 terms, same indexing as the fp32 partial sums
    uint16_t *v_lo;
    unsigned epoch;
    unsigned spin_limit;
    int wait;                 // expand units poll `ready` (single launch) or not (expand launched after shrink)
    int scale_v;              // shrink: v_hi / v_lo receive s_a v, not v
    // the k-slices' partial sums of v, which the expand units add up (NULL: v_hi and v_lo are complete)
    const float *parts;
    int n_slices;
    int64_t slice_stride;
};

static __device__ __forceinline__ void st_through_f32x4(float *p, f32x4 v)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    uint64_t *q = reinterpret_cast<uint64_t *>(p);
    const f32x2 lo = {v[0], v[1]}, hi = {v[2], v[3]};
    __hip_atomic_store(q, __builtin_bit_cast(uint64_t, lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, __builtin_bit_cast(uint64_t, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

static __device__ __forceinline__ f32x4 ld_through_f32x4(const float *p)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    const uint64_t *q = reinterpret_cast<const uint64_t *>(p);
    const f32x2 lo = __builtin_bit_cast(f32x2, __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const f32x2 hi = __builtin_bit_cast(f32x2, __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return f32x4{lo[0], lo[1], hi[0], hi[1]};
}

// The s_waitcnt immediate of the gfx9 family (gfx950 included): vmcnt in bits 3:0 and 15:14, expcnt in
// bits 6:4, lgkmcnt in bits 11:8; a field at its maximum waits for nothing.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "the hand-built s_waitcnt immediate below is the gfx9 encoding: this file is for gfx950"
#endif
constexpr unsigned kWaitcntVmcnt0 = (0u << 0) | (7u << 4) | (15u << 8) | (0u << 14);  // vmcnt(0), nothing else
static_assert(kWaitcntVmcnt0 == 0x0F70, "vmcnt(0) expcnt(7) lgkmcnt(15)");

// This wavefront's vector memory operations (its stores among them) have completed.  The two signal
// fences keep the compiler from moving memory operations across the wait in either direction.
static __device__ __forceinline__ void stores_done()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(kWaitcntVmcnt0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// at most N of this wavefront's vector memory operations are still under way
template <int N>
static __device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

static __device__ __forceinline__ void st_through_u16x8(uint16_t *p, uint4 v)
{
    uint64_t *q = reinterpret_cast<uint64_t *>(p);
    __hip_atomic_store(q, (uint64_t)v.x | ((uint64_t)v.y << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, (uint64_t)v.z | ((uint64_t)v.w << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

static __device__ __forceinline__ uint4 ld_through_u16x8(const uint16_t *p)
{
    const uint64_t *q = reinterpret_cast<const uint64_t *>(p);
    const uint64_t a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
}

// until the tile's n shrink units of this launch have stored their part of v
static __device__ __forceinline__ void wait_for(const Sync &sy, int idx, int n)
{
    if (threadIdx.x == 0) {
        const unsigned target = sy.epoch * (unsigned)n;
        unsigned spins = 0;
        while ((int)(__hip_atomic_load(sy.ready + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
            if (++spins > sy.spin_limit) {
                atomicOr(sy.timeout_flag, 1u);
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
    }
    __syncthreads();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

static __device__ __forceinline__ uint32_t pack_bf16_rne(float a, float b)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const f32x2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// 8 floats -> bf16 hi (nearest) and bf16 lo (nearest of the remainder): hi + lo keeps ~16 mantissa bits
static __device__ __forceinline__ void split_bf16(f32x4 f0, f32x4 f1, uint4 &ph, uint4 &pl)
{
    ph.x = pack_bf16_rne(f0[0], f0[1]);
    ph.y = pack_bf16_rne(f0[2], f0[3]);
    ph.z = pack_bf16_rne(f1[0], f1[1]);
    ph.w = pack_bf16_rne(f1[2], f1[3]);
    pl.x = pack_bf16_rne(f0[0] - bf16_bits_to_f32(ph.x & 0xFFFFu), f0[1] - __uint_as_float(ph.x & 0xFFFF0000u));
    pl.y = pack_bf16_rne(f0[2] - bf16_bits_to_f32(ph.y & 0xFFFFu), f0[3] - __uint_as_float(ph.y & 0xFFFF0000u));
    pl.z = pack_bf16_rne(f1[0] - bf16_bits_to_f32(ph.z & 0xFFFFu), f1[1] - __uint_as_float(ph.z & 0xFFFF0000u));
    pl.w = pack_bf16_rne(f1[2] - bf16_bits_to_f32(ph.w & 0xFFFFu), f1[3] - __uint_as_float(ph.w & 0xFFFF0000u));
}

constexpr int kMaxSlices = 4;  // upper bound of the shrink's k-slices

// Who adds the k-slices of v up.  A template argument of the bodies: with all three ways compiled into one, chosen by what the
// launch was given, the expand units that read complete v paid for the others' registers and code (mixed launches, 1344 -> 4224, rank
// 64, expand launch 17.5 us with, 16.7 without; 1984 -> 9856 28.5 / 27.9).
enum Slices {
    kSlicesByShrink,  // the shrink unit that completes a token tile: v_hi and v_lo are complete
    kSlicesByExpand,  // the expand units of the next launch, each those of its own tokens
    kSlicesByWaiting  // the same in one launch, behind the wait for the tile's shrink units
};

// the k-slices' partial sums of 8 consecutive v elements.  EARLIER: of an earlier launch, else read through to memory.
template <bool EARLIER>
static __device__ __forceinline__ void load_slices(const float *__restrict__ src, int n_slices, int64_t slice_stride,
                                                   f32x4 (&p0)[kMaxSlices], f32x4 (&p1)[kMaxSlices])
{
#pragma unroll
    for (int sl = 0; sl < kMaxSlices; ++sl) {
        const int64_t off = (int64_t)(sl < n_slices ? sl : 0) * slice_stride;
        p0[sl] = EARLIER ? *reinterpret_cast<const f32x4 *>(src + off) : ld_through_f32x4(src + off);
        p1[sl] = EARLIER ? *reinterpret_cast<const f32x4 *>(src + off + 4) : ld_through_f32x4(src + off + 4);
    }
}

// their sum, in slice order
static __device__ __forceinline__ void add_slices(const f32x4 (&p0)[kMaxSlices], const f32x4 (&p1)[kMaxSlices], int n_slices,
                                                  f32x4 &f0, f32x4 &f1)
{
    f0 = p0[0];
    f1 = p1[0];
#pragma unroll
    for (int sl = 1; sl < kMaxSlices; ++sl)
        if (sl < n_slices) {
            f0 += p0[sl];
            f1 += p1[sl];
        }
}

// ------------------------------------------------------------------------------------------------
// shrink: one unit = (group, <=16 tokens, 16 rank rows, one k-slice).  The four wavefronts split the
// k-slice.  Each issues its 16-byte weight loads up front (rows of A^T straight into the MFMA's
// row operand); meanwhile the work group stages the tokens' x slab for this k-slice in LDS with
// coalesced loads, from which every wavefront reads its token operand.  Each wavefront accumulates
// a 16x16 tile (rank row x token); the four tiles are summed through LDS in wavefront order.
// ------------------------------------------------------------------------------------------------
constexpr int kShrinkSteps = 8;                   // 32-wide k steps per wavefront per pass
constexpr int kSlabK = 4 * 32 * kShrinkSteps;     // k range staged per pass (all four wavefronts)
constexpr int kSlabRow = kSlabK + 8;              // LDS row length in bf16, padded by 16 bytes
constexpr int kShrinkLds = kTokTile * kSlabRow * 2 + 4 * 64 * 16;

static __device__ __forceinline__ void shrink_body(const Unit &u, const uint16_t *__restrict__ arena,
                                                   const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                   int k_slice_len, float *__restrict__ v_out, int n_slices,
                                                   int64_t slice_stride, char *lds, const Sync &sy)
{
    uint16_t(*slab)[kSlabRow] = reinterpret_cast<uint16_t(*)[kSlabRow]>(lds);
    f32x4(*red)[64] = reinterpret_cast<f32x4(*)[64]>(lds + kTokTile * kSlabRow * 2);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int i = lane & 15;
    const int kq = lane >> 4;

    const int ntok = u.ntok, pn = u.pn, ks = u.ks;
    const bool w_ok = i < pn;
    const bool x_ok = i < ntok;
    // this lane's 16-byte piece of a k step of the unit's row block (pn = rows in the block: 16 or 8)
    const uint16_t *wrow = arena + u.w_off + (kq * pn + (w_ok ? i : 0)) * 8;
    // slab staging: thread tid copies 16-byte chunk (tid & 127) of tokens (tid >> 7), +2, +4, ...
    const int s_chunk = tid & 127;
    const int s_tok0 = __builtin_amdgcn_readfirstlane(tid >> 7);  // wavefront-uniform

    const int kslice_beg = ks * k_slice_len;
    int kslice_end = kslice_beg + k_slice_len;
    if (kslice_end > in) kslice_end = in;

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const uint4 zero = {0u, 0u, 0u, 0u};
    for (int kp = kslice_beg; kp < kslice_end; kp += kSlabK) {
        // this wavefront's k range inside the pass
        const int kbeg = kp + wave * (32 * kShrinkSteps);
        uint4 a[kShrinkSteps];
#pragma unroll
        for (int q = 0; q < kShrinkSteps; ++q) {
            const int k = kbeg + 32 * q;
            a[q] = (k < kslice_end) ? ld16_stream(wrow + (int64_t)k * pn) : zero;
        }
        if (kp != kslice_beg) __syncthreads();  // previous pass's slab is no longer being read
        {
            const int k = kp + 8 * s_chunk;
            if (k < kslice_end) {
                uint4 xs[kTokTile / 2];
#pragma unroll
                for (int t = 0; t < kTokTile / 2; ++t) {
                    const int tok = s_tok0 + 2 * t;
                    xs[t] = (tok < ntok) ? ld16(x + (int64_t)u.tok[tok] * ldx + k) : zero;
                }
#pragma unroll
                for (int t = 0; t < kTokTile / 2; ++t) {
                    const int tok = s_tok0 + 2 * t;
                    if (tok < ntok) *reinterpret_cast<uint4 *>(&slab[tok][8 * s_chunk]) = xs[t];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kShrinkSteps; ++q) {
            const int k = kbeg + 32 * q;
            if (k < kslice_end) {
                const uint4 aa = w_ok ? a[q] : zero;
                // rows of tokens beyond ntok hold whatever LDS held: they only reach accumulator columns
                // that are never stored, and an unconditional 16-byte read stays one instruction
                const uint4 bb = *reinterpret_cast<const uint4 *>(&slab[i][k - kp + 8 * kq]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aa), as_bf16x8(bb), acc, 0, 0, 0);
            }
        }
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {
        const bool meets = sy.counters && (sy.wait || !sy.parts);  // other units of this launch wait for this one
        f32x4 t = red[0][lane];
        t += red[1][lane];
        t += red[2][lane];
        t += red[3][lane];
        if (x_ok && 4 * kq < pn) {
            float *dst = v_out + (int64_t)ks * slice_stride + u.v_off + (int64_t)i * u.r8 + 4 * kq;
            if (meets)
                st_through_f32x4(dst, t);
            else
                *reinterpret_cast<f32x4 *>(dst) = t;
        }
        if (meets) {
            // count this unit in; where no expand unit adds the slices up, the unit that completes its token tile does and
            // leaves the tile's v as bf16 hi + lo
            stores_done();
            if (sy.wait) {
                if (lane == 0) atomicAdd(sy.ready + u.sync_idx, 1u);
                return;
            }
            unsigned old = 0;
            if (lane == 0) old = atomicAdd(sy.counters + u.sync_idx, 1u);
            old = __builtin_amdgcn_readfirstlane(old);
            // nothing below (the loads of the other units' partial sums) moves up in front of the arrival
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            if (old + 1u == (unsigned)u.sync_n) {
                // the last of this launch's arrivals at the tile: the counter goes back to zero for the
                // next launch (nothing else touches it before this launch ends)
                if (lane == 0) atomicExch(sy.counters + u.sync_idx, 0u);
                const int64_t tile_off = u.v_off - u.p0;
                const int tasks = ntok * (u.r8 >> 3);
                const float vs = sy.scale_v ? u.scale : 1.f;
                for (int task = lane; task < tasks; task += 64) {
                    f32x4 p0[kMaxSlices], p1[kMaxSlices], f0, f1;
                    load_slices<false>(v_out + tile_off + 8 * task, n_slices, slice_stride, p0, p1);
                    add_slices(p0, p1, n_slices, f0, f1);
                    uint4 ph, pl;
                    split_bf16(vs * f0, vs * f1, ph, pl);
                    st_through_u16x8(sy.v_hi + tile_off + 8 * task, ph);
                    st_through_u16x8(sy.v_lo + tile_off + 8 * task, pl);
                }
            }
        }
    }
}

// A unit record read with one 128-byte request per wavefront: word w of the record in lane w (and w + 32).
// Its fields are then taken from that register (unit_word), so that a unit's operand loads are one trip to
// memory behind the start of its work group, not two (the token list after the token count).  Used by the
// one-launch decode kernel for its shrink units, every one of which is on the launch's critical path (15.4 ->
// 15.0 us on a 256-token batch; for its expand units' records, which are read while the shrink units run,
// 15.0 -> 15.2 us); in the launches of several rounds (k_shrink_wide, k_expand) it changed nothing or
// cost a little (28.9 -> 29.3 us for 2,560 expand units), so they read the record field by field.
static_assert(offsetof(Unit, w_off) == 0 && offsetof(Unit, v_off) == 8 && offsetof(Unit, r8) == 16 &&
                  offsetof(Unit, ntok) == 20 && offsetof(Unit, p0) == 24 && offsetof(Unit, pn) == 28 &&
                  offsetof(Unit, sync_idx) == 48 && offsetof(Unit, tok) == 64,
              "the words of a unit record as unit_word's callers number them");
static __device__ __forceinline__ uint32_t load_unit_words(const Unit *u)
{
    return reinterpret_cast<const uint32_t *>(u)[threadIdx.x & 31];
}
static __device__ __forceinline__ uint32_t unit_word(uint32_t rec, int w)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)rec, w);
}

// ------------------------------------------------------------------------------------------------
// shrink, whole-k units: one unit = (group, <=16 tokens, 16 rank rows or one half of them, all of k), one work group of
// 16 wavefronts.  Used when the batch's units fit the chip in one round: each compute unit then
// streams one row block of one adapter with 128 KB of loads in flight, and v leaves complete (no
// partial sums in memory, no counters).  The work group is four k-slice units in one: wavefronts
// 4j .. 4j+3 do exactly the arithmetic of the four wavefronts of a k-slice unit for slice j, and the
// tiles are added in the same order (inside a slice by wavefront, then the slices), so the result
// is bitwise the one the k-slice path gives.  Every wavefront requests its 8 weight operands and its
// own piece of the tokens' x rows (coalesced, two tokens per load), turns the x piece into MFMA
// operand order through a private LDS region (no work-group barrier), and runs its 8 MFMAs.
// ------------------------------------------------------------------------------------------------
constexpr int kWideWaves = 4 * kMaxSlices;
constexpr int kWideThreads = 64 * kWideWaves;
constexpr int kWideK = 32 * kShrinkSteps;  // k range of one wavefront per pass
constexpr int kWideRow = kWideK + 8;       // LDS row length in bf16, padded by 16 bytes
constexpr int kWideSlab = kTokTile * kWideRow * 2;
constexpr int kWideLds = kWideWaves * kWideSlab + kWideWaves * 64 * 16;
constexpr int kWideHalfWaves = kWideWaves / 2;  // the same unit by 8 wavefronts, two of the 16 roles each

// WAVES = 16: one work group per compute unit.  WAVES = 8: every wavefront takes two of the sixteen roles
// in turn (role = wavefront, then wavefront + 8: the same place in another k-slice), and two work groups
// share a compute unit: for launches of more units than the chip has compute units, where one unit's
// record fetch, ramp and reduction then run beside the other's loads instead of between two units'
// (544 units of 8192 input features: 32.7 -> 29.9 us; four wavefronts in four roles, four work groups per
// compute unit: 32.4 us).
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES, kWideWaves / WAVES) void k_shrink_wide(const Unit *__restrict__ units,
                                                              const uint16_t *__restrict__ arena,
                                                              const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                              int k_slice_len, int n_slices,
                                                              float *__restrict__ v_f32,
                                                              uint16_t *__restrict__ v_hi,
                                                              uint16_t *__restrict__ v_lo, int scale_v)
{
    constexpr int ROLES = kWideWaves / WAVES;
    // the sixteen partial tiles: behind the x regions, or (8 wavefronts, so that two work groups fit the
    // compute unit's LDS) at the start of the x region of the wavefront that computed them
    constexpr bool kRedInSlab = WAVES < kWideWaves;
    __shared__ __attribute__((aligned(16))) char lds[kRedInSlab ? WAVES * kWideSlab : kWideLds];
    static_assert(ROLES * 64 * 16 <= kWideSlab, "a wavefront's partial tiles fit its x region");
    LORA_CLOCK(0);
    const Unit &u = units[blockIdx.x];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = wave & 3;      // its place among a slice's four wavefronts
    const int i = lane & 15;
    const int kq = lane >> 4;
    uint16_t(*slab)[kWideRow] = reinterpret_cast<uint16_t(*)[kWideRow]>(lds + wave * kWideSlab);
    auto red = [&](int role) __attribute__((always_inline)) -> f32x4 * {
        char *at = kRedInSlab ? lds + (role % WAVES) * kWideSlab + (role / WAVES) * (64 * 16)
                              : lds + kWideWaves * kWideSlab + role * (64 * 16);
        return reinterpret_cast<f32x4 *>(at);
    };

    const int ntok = u.ntok, pn = u.pn;
    const bool w_ok = i < pn;
    const bool x_ok = i < ntok;
    // the unit's rows are rows row0 .. row0 + pn - 1 of a block of blk_rows rows of A^T (all of the
    // block, or one half of a 16-row block), which starts at w_off
    const int blk_rows = min(kRowTile, u.r8 - (u.p0 & ~(kRowTile - 1)));
    const int row0 = u.p0 & (kRowTile - 1);
    const uint16_t *wrow = arena + u.w_off + (kq * blk_rows + row0 + (w_ok ? i : 0)) * 8;
    // x staging: lane -> token 2t + half, 16-byte chunk s_chunk of the wavefront's 256 k.  The unit's
    // token list repeats its first token beyond ntok, so every listed row is a valid row of x.
    const int half = lane >> 5;
    const int s_chunk = lane & 31;
    const uint16_t *xrow[kTokTile / 2];
#pragma unroll
    for (int t = 0; t < kTokTile / 2; ++t) xrow[t] = x + (int64_t)(half ? u.tok[2 * t + 1] : u.tok[2 * t]) * ldx;

    f32x4 accs[ROLES];
    const uint4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int ro = 0; ro < ROLES; ++ro) {
    const int slice = (wave + WAVES * ro) >> 2;  // the k-slice this role works on
    const int kslice_beg = slice * k_slice_len;
    int kslice_end = kslice_beg + k_slice_len;
    if (kslice_end > in) kslice_end = in;
    if (slice >= n_slices) kslice_end = kslice_beg;

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int kp = kslice_beg; kp < kslice_end; kp += 4 * kWideK) {
        const int kbeg = kp + wq * kWideK;  // wavefront-uniform
        if (kbeg >= kslice_end) break;
        uint4 a[kShrinkSteps];
#pragma unroll
        for (int q = 0; q < kShrinkSteps; ++q) {
            const int k = kbeg + 32 * q;
            a[q] = (k < kslice_end) ? ld16_stream(wrow + (int64_t)k * blk_rows) : zero;
        }
        // in is a multiple of 64, so a 16-byte chunk is either inside the row or wholly beyond it;
        // chunks beyond it are fetched from the row's last chunk instead and never enter an MFMA
        int kx = kbeg + 8 * s_chunk;
        if (kx > in - 8) kx = in - 8;
        uint4 xs[kTokTile / 2];
#pragma unroll
        for (int t = 0; t < kTokTile / 2; ++t)
            if (2 * t < ntok) xs[t] = ld16(xrow[t] + kx);
#pragma unroll
        for (int t = 0; t < kTokTile / 2; ++t)
            if (2 * t < ntok) *reinterpret_cast<uint4 *>(&slab[2 * t + half][8 * s_chunk]) = xs[t];
        // the region is private to this wavefront and LDS operations of a wavefront complete in order
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
        for (int q = 0; q < kShrinkSteps; ++q) {
            const int k = kbeg + 32 * q;
            if (k < kslice_end) {
                const uint4 aa = w_ok ? a[q] : zero;
                // rows of tokens beyond ntok hold whatever LDS held: they only reach accumulator columns
                // that are never stored, and an unconditional 16-byte read stays one instruction
                const uint4 bb = *reinterpret_cast<const uint4 *>(&slab[i][32 * q + 8 * kq]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aa), as_bf16x8(bb), acc, 0, 0, 0);
            }
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
    }
    accs[ro] = acc;
    }
    // (the x region is this wavefront's own, and its LDS operations complete in order)
#pragma unroll
    for (int ro = 0; ro < ROLES; ++ro) red(wave + WAVES * ro)[lane] = accs[ro];
    __syncthreads();
    // the first wavefront of every slice adds the slice's four tiles (in wavefront order), then
    // wavefront 0 adds the slices (in slice order): the order of the k-slice plan, two short steps
    // instead of sixteen reads by one wavefront
#pragma unroll
    for (int ro = 0; ro < ROLES; ++ro) {
        const int role = wave + WAVES * ro;
        if (wq == 0 && (role >> 2) < n_slices) {
            f32x4 ts = red(role)[lane];
            ts += red(role + 1)[lane];
            ts += red(role + 2)[lane];
            ts += red(role + 3)[lane];
            red(role)[lane] = ts;
        }
    }
    __syncthreads();
    if (wave == 0) {
        f32x4 t = red(0)[lane];
#pragma unroll
        for (int sl = 1; sl < kMaxSlices; ++sl)
            if (sl < n_slices) t += red(4 * sl)[lane];
        // register r of lane (i, kq) is rank row 4*kq + r of the block for token i
        if (x_ok && 4 * kq < pn) {
            const int64_t off = u.v_off + (int64_t)i * u.r8 + 4 * kq;
            if (v_hi) {
                if (scale_v) t = u.scale * t;
                uint2 h, l;
                h.x = pack_bf16_rne(t[0], t[1]);
                h.y = pack_bf16_rne(t[2], t[3]);
                l.x = pack_bf16_rne(t[0] - bf16_bits_to_f32(h.x & 0xFFFFu), t[1] - __uint_as_float(h.x & 0xFFFF0000u));
                l.y = pack_bf16_rne(t[2] - bf16_bits_to_f32(h.y & 0xFFFFu), t[3] - __uint_as_float(h.y & 0xFFFF0000u));
                *reinterpret_cast<uint2 *>(v_hi + off) = h;
                *reinterpret_cast<uint2 *>(v_lo + off) = l;
            } else {
                *reinterpret_cast<f32x4 *>(v_f32 + off) = t;
            }
        }
        LORA_CLOCK(4);
    }
}

// ------------------------------------------------------------------------------------------------
// shrink of token-heavy groups (prefill) up to rank 64: one unit = (group, 32 tokens, all rank
// rows, all of k).  The four wavefronts split k into quarters; each streams its quarter of the
// tokens' x rows exactly once.  x comes from HBM with coalesced loads (a wavefront load covers 256
// bytes of each of 4 tokens), XD passes of 128 k ahead, and is turned into MFMA operand order through
// an LDS region private to the wavefront, so no work-group barrier sits in the k loop.  (Loading the
// token operand straight from memory, 16 rows x 64 bytes per load, costs the address path 3.7 times
// as much per byte.)  The rows of A^T come from L2 (every token tile of the group re-reads them),
// requested WD k steps ahead because a step of a low rank is far shorter than a round trip to L2,
// and are shared by the TB token blocks in registers.  The four partial tiles are summed through
// LDS (re-using the x regions) in a fixed order (3+1, 2+0, then 1+0) and v leaves complete: as bf16
// hi + lo for the expand, or as fp32.  JB = 16-row blocks of A^T (1, 2, 4).
// ------------------------------------------------------------------------------------------------
constexpr int kPfTokens = 32;
constexpr int kPfPassK = 128;                 // k per pass of a wavefront
constexpr int kPfRow = kPfPassK + 8;          // LDS row length in bf16, padded by 16 bytes
constexpr int kPfSlab = kPfTokens * kPfRow * 2;
constexpr int kPrefillLds = 4 * kPfSlab;

// A piece of memory that other XCDs' units write or read in this launch, in 16-byte accesses that go through to
// memory (the cache bits of an agent-scope atomic, which stops at 8 bytes).  base is wavefront-uniform.
struct Through {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Through(float *base, int floats)
        : r(__builtin_amdgcn_make_buffer_rsrc(base, 0, floats * 4, 0x00020000)) {}
    static constexpr int kAgent = 16;  // sc1
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    __device__ __forceinline__ void st(int quad, f32x4 f) const
    {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f), r, 16 * quad, 0, kAgent);
    }
    __device__ __forceinline__ f32x4 ld(int quad) const
    {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, 16 * quad, 0, kAgent));
    }
};

// An adapter's rows of A^T in 16-byte loads whose address is a lane's element offset, a register's, and a wavefront's, a scalar: the
// loads of a k loop then need no 64-bit addition per lane and no registers for its results.  22,532 tokens, us a call with an address
// per load / this way: rank 64 4096 -> 4096 113.0 / 111.1, 14336 -> 1024 177.3 / 172.7, rank 256 250.4 / 247.3 and 418.9 / 407.9; ranks up to
// 32 level; k_shrink_prefill no longer spills its one register.  base is wavefront-uniform.
struct Rows {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Rows(const uint16_t *base, int elements)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, (int)(2u * (unsigned)elements), 0x00020000)) {}
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    __device__ __forceinline__ uint4 ld(int lane, int wave) const
    {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(2u * (unsigned)lane), (int)(2u * (unsigned)wave), 0);
        return uint4{v.x, v.y, v.z, v.w};
    }
};

// four elements of v, at element index `at`, as bf16 hi + lo
static __device__ __forceinline__ void store_v4(f32x4 f, int64_t at, uint16_t *__restrict__ v_hi, uint16_t *__restrict__ v_lo)
{
    uint2 h, l;
    h.x = pack_bf16_rne(f[0], f[1]);
    h.y = pack_bf16_rne(f[2], f[3]);
    l.x = pack_bf16_rne(f[0] - bf16_bits_to_f32(h.x & 0xFFFFu), f[1] - __uint_as_float(h.x & 0xFFFF0000u));
    l.y = pack_bf16_rne(f[2] - bf16_bits_to_f32(h.y & 0xFFFFu), f[3] - __uint_as_float(h.y & 0xFFFF0000u));
    *reinterpret_cast<uint2 *>(v_hi + at) = h;
    *reinterpret_cast<uint2 *>(v_lo + at) = l;
}

// threadIdx.x for the stores behind a unit's k loop, where the compiler cannot see it: it computes what depends on the
// thread index before the loop otherwise, and carries it through on spilled registers (k_shrink_prefill 9 spilled, one
// this way; rank 64, 16 prompts of 1000 tokens, uncut, 4096 features, shrink launch 34.5 -> 30.4 us).
static __device__ __forceinline__ int late_thread()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The rank rows of a token-heavy shrink unit that a work group takes: all of them, or (launches of few units, shrink_in_halves) one of
// two halves.  A compute unit passes about 50 GB/s of x and A^T together, so a launch of few units lasts as long as
// one of them however many compute units stand idle; halves read x twice (the second time from the L2: both run on one XCD) and every
// row of A^T once, and nothing is added up between them.  Shrink launch in us, whole / halves: one prompt of 2000 tokens, 4096 features,
// rank 128 (128 units, cut along k) 15.4 / 13.1, rank 192 18.3 / 16.4, 1024 tokens at 14336 features 29.5 / 23.2; uncut, 1984 features,
// 2000 tokens (32 units) 17.2 / 14.1, 7900 tokens of rank 192 (124) 21.8 / 18.7.
struct RankRows {
    int first, n;  // rank rows first .. first + n - 1 (first a multiple of 16, n of 8)
    int part, of;  // which of how many work groups
};

// How token-heavy units leave v, whole or as slices of its sums.  In rows as everyone's v lies (for lora_shrink's caller and
// lora_linear), or, for the 64-token expand units (`tiled`), in the order in which an MFMA takes it: 16 tokens at a time, element (token
// n, rank row j) of h tokens at (j / 8 * h + n) * 8 + j % 8.  A wavefront's load of an operand is then 1 KB of consecutive bytes instead
// of 64 bytes of each of 16 rows, which cost a compute unit's address path 3.7 times as long, and so are the stores straight from
// the registers that the MFMAs left.
static __device__ __forceinline__ int tiled_quad(int r8, int ntok, int tok, int j4)
{
    const int b = tok >> 4, h = min(16, ntok - 16 * b);
    return 4 * b * r8 + ((j4 >> 1) * h + (tok & 15)) * 2 + (j4 & 1);
}

// where element quad i of those rows lies in the unit's v, in quads from its first element; i counts n / 4 quads per token
static __device__ __forceinline__ int quad_place(const Unit &u, const RankRows &rr, int i, bool tiled)
{
    if (rr.of == 1) return i;
    const int quads = rr.n >> 2;
    if (tiled) {
        const int b = i / (16 * quads), h = min(16, u.ntok - 16 * b);
        return i + 4 * b * (u.r8 - rr.n) + (rr.first >> 2) * h;
    }
    const int tok = i / quads;
    return tok * (u.r8 >> 2) + (rr.first >> 2) + (i - tok * quads);
}

// The end of a token-heavy shrink unit, by all threads of its work group: rows row0 .. row0 + rows - 1 of the unit's
// v are one run of memory (or, of half the rank rows, a run per token or 16), which goes out in 16-byte pieces, neighbouring threads side by
// side; quad(i) = the sums of its elements 4 i .. 4 i + 3.  (Straight from the MFMA registers a wavefront's stores to rows were 8 bytes of
// each of 64 pieces of lines; written through to memory those were most of a cut unit's time: 2000 tokens of rank 128 at
// 4096 features, 128 units, shrink launch 20.4 -> 15.2 us.)
// Whole units write v.  Units cut along k leave their sums in slice u.ks of the fp32 partial sums: plainly for the
// stand-alone shrink (v_f32: the caller adds the slices up, and slice 0's unit clears those this group does not
// use), else through to memory for the unit that completes the tile (complete_tile).
template <class Quad>
static __device__ __forceinline__ void store_heavy_rows(const Unit &u, const RankRows &rr, int n_ks, int row0, int rows, Quad quad,
                                                        uint16_t *__restrict__ v_hi, uint16_t *__restrict__ v_lo,
                                                        float *__restrict__ v_f32, int n_slices, int64_t slice_stride,
                                                        float *__restrict__ parts, float vs, bool tiled)
{
    const int n = rows * (rr.n >> 2);
    const int64_t at = u.v_off + (int64_t)row0 * u.r8;
    if (n_ks > 1 && !v_f32) {
        const Through slice(parts + (int64_t)u.ks * slice_stride + at, rows * u.r8);
        for (int i = late_thread(); i < n; i += kThreads) slice.st(quad_place(u, rr, i, tiled), quad(i));
    } else if (v_f32) {
        float *dst = v_f32 + (int64_t)u.ks * slice_stride + at;
        for (int i = late_thread(); i < n; i += kThreads) reinterpret_cast<f32x4 *>(dst)[quad_place(u, rr, i, false)] = quad(i);
        if (n_ks > 1 && u.ks == 0)
            for (int sl = n_ks; sl < n_slices; ++sl)
                for (int i = late_thread(); i < n; i += kThreads)
                    reinterpret_cast<f32x4 *>(dst + (int64_t)sl * slice_stride)[quad_place(u, rr, i, false)] = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
        for (int i = late_thread(); i < n; i += kThreads) store_v4(vs * quad(i), at + 4 * quad_place(u, rr, i, tiled), v_hi, v_lo);
    }
}

// A cut unit whose sums are on their way to memory: the one of the tile's n_ks that arrives last at the tile's counter
// adds the slices in slice order and leaves v as bf16 hi + lo.  Halves of the rank rows have a counter each where the tile has two
// (it has one per 16 tokens), else the last of all completes all rows.  `word`: an LDS word that nothing else uses any more.
static __device__ __forceinline__ void complete_tile(const Unit &u, const RankRows &rr, int n_ks, int64_t slice_stride,
                                                     float *__restrict__ parts, uint16_t *__restrict__ v_hi,
                                                     uint16_t *__restrict__ v_lo, float vs, bool tiled, const Sync &sy, unsigned *word)
{
    stores_done();
    __syncthreads();  // every wavefront's partial sums are out
    const bool own = rr.of == 1 || u.ntok > kTokTile;
    unsigned *const counter = sy.counters + u.sync_idx + (own ? rr.part : 0);
    if (threadIdx.x == 0) *word = atomicAdd(counter, 1u);
    __syncthreads();
    if (*word + 1u != (unsigned)(own ? n_ks : n_ks * rr.of)) return;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);  // the loads of the slices stay behind the arrival
    if (threadIdx.x == 0) atomicExch(counter, 0u);  // back to zero for the next launch
    const RankRows all = own ? rr : RankRows{0, u.r8, 0, 1};
    const int n = u.ntok * (all.n >> 2), len = u.ntok * u.r8;
    const Through s0(parts + u.v_off, len), s1(parts + u.v_off + slice_stride, len);
    if (n_ks <= 2) {
#pragma unroll 4
        for (int i = late_thread(); i < n; i += kThreads) {
            const int q = quad_place(u, all, i, tiled);
            store_v4(vs * (s0.ld(q) + s1.ld(q)), u.v_off + 4 * q, v_hi, v_lo);
        }
    } else {
        const Through s2(parts + u.v_off + 2 * slice_stride, len);
        const Through s3(parts + u.v_off + (n_ks > 3 ? 3 : 2) * slice_stride, len);
#pragma unroll 4
        for (int i = late_thread(); i < n; i += kThreads) {
            const int q = quad_place(u, all, i, tiled);
            f32x4 f = s0.ld(q) + s1.ld(q);
            f += s2.ld(q);
            const f32x4 f3 = s3.ld(q);
            if (n_ks > 3) f += f3;
            store_v4(vs * f, u.v_off + 4 * q, v_hi, v_lo);
        }
    }
}

// which of n passes along k adapter i's units begin with, where they begin in turn: i modulo the largest power of two up to n
static __device__ __forceinline__ int first_pass(int i, int n) { return n > 0 ? i & ((1 << (31 - __builtin_clz(n))) - 1) : 0; }

template <int JB, int TB, int WD, int XD = 1>
static __device__ __forceinline__ void shrink_prefill_ksplit(const Unit &u, const RankRows &rr, const int32_t *__restrict__ perm,
                                                             const uint16_t *__restrict__ arena,
                                                             const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                             uint16_t *__restrict__ v_hi,
                                                             uint16_t *__restrict__ v_lo, float *__restrict__ v_f32,
                                                             int n_slices, int64_t slice_stride, char *lds,
                                                             float *__restrict__ parts, const Sync &sy)
{
    constexpr int NT = JB * TB;
    constexpr int NL = 4 * TB;  // x loads of a wavefront per pass: 4 tokens each
    static_assert(TB <= 2 && 16 * TB <= kPfTokens, "tokens of a unit");
    static_assert(4 * NT * 64 * 16 + 4 <= kPrefillLds, "the wavefronts' partial tiles and a word fit the LDS");
    static_assert(WD == 1 || WD == 2 || WD == 4, "the weight ring must divide the 4 steps of a pass");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t(*slab)[kPfRow] = reinterpret_cast<uint16_t(*)[kPfRow]>(lds + wave * kPfSlab);
    f32x4(*red)[NT][64] = reinterpret_cast<f32x4(*)[NT][64]>(lds);  // re-uses the x regions after the k loop
    const int n = lane & 15;
    const int kq = lane >> 4;
    const int r8 = rr.n;  // of this work group
    const int ntok = u.ntok;

    // staging: load t of a pass takes tokens 4t .. 4t+3, this lane token 4t + kq, 16-byte chunk n
    const uint16_t *xrow[NL];
#pragma unroll
    for (int t = 0; t < NL; ++t) {
        const int tok = min(4 * t + kq, ntok - 1);
        xrow[t] = x + (int64_t)perm[u.perm_off + tok] * ldx;
    }
    // The caller picks JB from the rank; telling the compiler so removes the branches around the row
    // blocks that always exist (with a branch per block the same loop ran 2.4 times slower).
    __builtin_assume(r8 <= 16 * JB && (JB == 1 ? r8 >= 8 : r8 > 8 * JB));
    const Rows wa(arena + u.w_off + (int64_t)rr.first * in, r8 * in);
    int woff[JB];  // element offset of this lane's 16-byte piece in k step 0 of row block jb
    int wh[JB];    // rows in block jb (16, or 8 for the last block of a padded rank that is 8 mod 16)
    // The loop below has no branch: a block beyond the padded rank (ranks 33..48 of the bucket up to 64) is
    // worked as a copy of the last block that exists, and its sums are never stored.
    static_assert(JB <= 4, "ranks above 64 take the row-split body");
    const int nblk = (r8 + 15) >> 4;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const int jbc = min(jb, nblk - 1);
        const int h = min(16, r8 - 16 * jbc);
        wh[jb] = h > 0 ? h : 16;
        // lanes n >= 8 of an 8-row block read the piece of row n - 8: they only reach accumulator rows
        // beyond the padded rank, which are never stored
        woff[jb] = 16 * jbc * in + (kq * wh[jb] + (n & (wh[jb] - 1))) * 8;
    }

    f32x4 acc[JB][TB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[jb][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // this wavefront's quarter of the unit's k range: all of k, or (in launches of few units, which
    // last as long as a unit's walk through k) k-slice u.ks of u.sync_n, multiples of 128 long
    const int n_ks = u.sync_n > 1 ? u.sync_n : 1;
    const int ks_len = n_ks > 1 ? ((in / n_ks + 127) / 128) * 128 : in;
    const int ks_beg = min(in, u.ks * ks_len);
    const int ks_end = min(in, ks_beg + ks_len);
    const int kquarter = ((ks_end - ks_beg + 3) / 4 + 31) & ~31;
    const int kbeg = ks_beg + wave * kquarter;
    const int kend = min(ks_end, kbeg + kquarter);

    {
        // Loads without conditions (rows of tokens beyond ntok are the last token's, see xrow; a chunk beyond
        // the row is fetched from the row's last chunk and a k step beyond the row from its last step; none
        // of them enters an MFMA whose sums are stored): with a branch around a load the compiler no
        // longer counts the loads in flight and waits for all of them at every wait, the x of the passes
        // ahead included, so that every pass of 128 of k took a whole trip to memory.
        const int npass = kend > kbeg ? (kend - kbeg + kPfPassK - 1) / kPfPassK : 0;
        const int nfull = kend > kbeg ? (kend - kbeg) / kPfPassK : 0;
        // The passes in order, but from another one for every adapter where the wavefronts' quarters lie whole multiples of 4 KB apart: all
        // units of a launch walk k at about the same pace, and would ask a part of the memory's channels at any one time.  By adapter
        // and not by tile, so that a row's sums come in one order wherever its token sits in the group, and the tiles of a group still
        // share its rows of A^T.  A call in us, in order / by tile / by adapter: 19,675 tokens of 32 adapters, 8192 -> 1024, rank 8 80.6 / 72.2 /
        // 71.8, rank 32 92.8 / 85.8 / 84.9, rank 64 107.7 / 107.7 / 102; 10,082 tokens, 16384 -> 1024, rank 8 76.9 / 71.2 / 68.6, rank 32 86.3 / 82.5 /
        // 81.8, rank 64 105 / 107 / 101.  Few prompts level: four of 700, 8192 -> 1024, 21.6 / 21.4 / 21.4.
        const int turn = kquarter * 2 % 4096 == 0 ? first_pass(u.turn, nfull) : 0;
        auto pass_k = [&](int i) __attribute__((always_inline)) {
            return kbeg + kPfPassK * (i < nfull ? (i + turn < nfull ? i + turn : i + turn - nfull) : i);
        };
        auto x_all = [&](int k0, uint4(&xq)[NL]) __attribute__((always_inline)) {
            const int kx = min(k0 + 8 * n, in - 8);
#pragma unroll
            for (int t = 0; t < NL; ++t) xq[t] = ld16_stream(xrow[t] + kx);
        };
        auto w_step = [&](int k, int jb) __attribute__((always_inline)) {
            return wa.ld(woff[jb], min(k, in - 32) * wh[jb]);
        };
        auto stage = [&](const uint4(&xq)[NL]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NL; ++t) *reinterpret_cast<uint4 *>(&slab[4 * t + kq][8 * n]) = xq[t];
        };
        auto k_step = [&](int d, const uint4(&wd)[JB]) __attribute__((always_inline)) {
            bf16x8 xo[TB];
#pragma unroll
            for (int tb = 0; tb < TB; ++tb)
                xo[tb] = as_bf16x8(*reinterpret_cast<const uint4 *>(&slab[16 * tb + n][32 * d + 8 * kq]));
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                const bf16x8 ww = as_bf16x8(wd[jb]);
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
                    acc[jb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ww, xo[tb], acc[jb][tb], 0, 0, 0);
            }
        };
        auto wave_sync = [&]() __attribute__((always_inline)) {
            // the region is private to this wavefront and LDS operations of a wavefront complete in order
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        };
        // XD passes of x and WD k steps of A^T are in flight per wavefront (registers)
        uint4 xq[XD][NL], w[WD][JB];
#pragma unroll
        for (int q = 0; q < XD; ++q) x_all(pass_k(min(q, max(npass - 1, 0))), xq[q]);
#pragma unroll
        for (int d = 0; d < WD; ++d)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) w[d][jb] = w_step(pass_k(0) + 32 * d, jb);
        int i0 = 0, k1 = pass_k(0), kx = pass_k(XD);
        const int kturn = kbeg + kPfPassK * nfull;  // behind the last whole pass comes the first
        for (; i0 + 2 * XD <= nfull; i0 += XD) {
#pragma unroll
            for (int q = 0; q < XD; ++q) {
                const int k0 = k1;
                k1 = k1 + kPfPassK < kturn ? k1 + kPfPassK : kbeg;
                stage(xq[q]);
                x_all(kx, xq[q]);
                kx = kx + kPfPassK < kturn ? kx + kPfPassK : kbeg;
                wave_sync();
#pragma unroll
                for (int d = 0; d < kPfPassK / 32; ++d) {
                    k_step(d, w[d % WD]);
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        w[d % WD][jb] = w_step(d + WD < 4 ? k0 + 32 * (d + WD) : k1 + 32 * (d + WD - 4), jb);
                }
                wave_sync();
            }
        }
        // the last passes (fewer than 2 XD full ones and maybe a shorter one): the same under conditions
        for (; i0 < npass; i0 += XD) {
#pragma unroll
        for (int q = 0; q < XD; ++q) {
            const int i = i0 + q;
            if (i < npass) {
                const int k0 = pass_k(i), k1 = pass_k(i + 1);
                stage(xq[q]);
                if (i + XD < npass) x_all(pass_k(i + XD), xq[q]);
                wave_sync();
#pragma unroll
                for (int d = 0; d < kPfPassK / 32; ++d) {
                    const int k = k0 + 32 * d;
                    if (k < kend) {
                        k_step(d, w[d % WD]);
                        if (d + WD < 4 || i + 1 < npass) {
#pragma unroll
                            for (int jb = 0; jb < JB; ++jb)
                                w[d % WD][jb] = w_step(d + WD < 4 ? k + 32 * WD : k1 + 32 * (d + WD - 4), jb);
                        }
                    }
                }
                wave_sync();
            }
        }
        }
    }

    // the four k-quarters' sums meet in LDS, added as (0 + 2) + (1 + 3)
    __syncthreads();  // every wavefront has finished with its x region
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) red[wave][jb * TB + tb][lane] = acc[jb][tb];
    __syncthreads();
    const float vs = sy.scale_v ? u.scale : 1.f;
    const bool tiled = !v_f32 && !sy.scale_v;
    const int quads = r8 >> 2;
    // lane (n, kq) of tile (jb, tb) holds v[token 16 tb + n][16 jb + 4 kq + e]
    auto quad = [&](int i) __attribute__((always_inline)) {
        int tok, j4;
        if (tiled) {
            const int b = TB > 1 && i >= 16 * quads ? 1 : 0, h2 = 2 * min(16, ntok - 16 * b), k = i - 16 * b * quads;
            const int kp = ntok == 16 * TB ? k >> 5 : (int)((unsigned)k / (unsigned)h2);
            tok = 16 * b + ((k - kp * h2) >> 1);
            j4 = 2 * kp + (k & 1);
        } else {
            tok = i / quads;
            j4 = i - tok * quads;
        }
        const int t = (j4 >> 2) * TB + (tok >> 4), l = (j4 & 3) * 16 + (tok & 15);
        return (red[0][t][l] + red[2][t][l]) + (red[1][t][l] + red[3][t][l]);
    };
    store_heavy_rows(u, rr, n_ks, 0, ntok, quad, v_hi, v_lo, v_f32, n_slices, slice_stride, parts, vs, tiled);
    if (n_ks == 1 || v_f32) return;
    complete_tile(u, rr, n_ks, slice_stride, parts, v_hi, v_lo, vs, tiled, sy, reinterpret_cast<unsigned *>(lds + 4 * NT * 64 * 16));
}

// Token-heavy units above rank 64: 16 * TB tokens, all rank rows, all of k or a slice of it.  Here the
// four wavefronts split the rank rows (JBW blocks of 16 each) instead of k: every 16-byte piece of
// A^T is then loaded once per work group, straight into the registers of the one wavefront that owns
// its rows, and x, which all four need, is staged once per work group in LDS (two buffers of 128 of k,
// one barrier per pass).  With k split over the wavefronts as above, a unit of 32 tokens loads all of
// A^T for 32 tokens' worth of x: at rank 128 four times the bytes of x, which made the compute units'
// vector caches, not memory, the bound (uniform rank 128 on cfg2's routing: 78 us against 35 us at
// rank 8; 62 us with this body).  No sums cross wavefronts: each stores the rows of v it owns straight
// from its registers (tiled), or puts them into LDS, from where they leave in rows.  (Up to
// rank 64 the k-split body of 32 tokens stayed as fast or faster: 50 us at uniform rank 64 either way.
// Ranks 129..192 take three row blocks per wavefront and 64 tokens, ranks 193..256 four and 32 tokens, the
// accumulators of 64 not fitting the registers: against units of 16 tokens with k split, the shrink
// launch at uniform rank 160 / 192 / 256 went from 105 / 121 / 156 us to 78 / 86 / 112.)
template <int JBW, int TB, int PD, int WP>
static __device__ __forceinline__ void shrink_prefill_rowsplit(const Unit &u, const RankRows &rr, const int32_t *__restrict__ perm,
                                                               const uint16_t *__restrict__ arena,
                                                               const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                               uint16_t *__restrict__ v_hi,
                                                               uint16_t *__restrict__ v_lo, float *__restrict__ v_f32,
                                                               int n_slices, int64_t slice_stride, char *lds,
                                                               float *__restrict__ parts, const Sync &sy)
{
    constexpr int TOK = 16 * TB;
    constexpr int SP = kPfPassK / 32;  // k steps of a pass
    static_assert(PD % 2 == 0 && PD % WP == 0, "the rings are indexed by the pass's place in a round of PD");
    static_assert(2 * TOK * kPfRow * 2 <= kPrefillLds, "two x buffers fit the LDS");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t(*buf)[kPfRow] = reinterpret_cast<uint16_t(*)[kPfRow]>(lds);  // [2 * TOK] rows
    const int n = lane & 15;
    const int kq = lane >> 4;
    const int r8 = rr.n;  // of this work group
    const int ntok = u.ntok;

    // staging: thread (xr, xc) copies 16-byte chunk xc of tokens xr, xr + 16, ...
    const int xr = threadIdx.x >> 4, xc = threadIdx.x & 15;
    const uint16_t *xrow[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) xrow[i] = x + (int64_t)perm[u.perm_off + min(xr + 16 * i, ntok - 1)] * ldx;

    // A wavefront whose row blocks lie beyond the padded rank (ranks that are not multiples of 64) works on
    // the last block that exists instead: its sums are never stored, and the loop needs no branch for it.
    const Rows wa(arena + u.w_off + (int64_t)rr.first * in, r8 * in);
    const int nblk = (r8 + 15) >> 4;
    int woff[JBW], wh[JBW];
#pragma unroll
    for (int j = 0; j < JBW; ++j) {
        const int jb = min(wave * JBW + j, nblk - 1);
        const int h = min(16, r8 - 16 * jb);
        wh[j] = h;
        // lanes n >= 8 of an 8-row block read the piece of row n - 8: they only reach accumulator rows
        // beyond the padded rank, which are never stored
        woff[j] = 16 * jb * in + (kq * h + (n & (h - 1))) * 8;
    }

    f32x4 acc[JBW][TB];
#pragma unroll
    for (int j = 0; j < JBW; ++j)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[j][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int n_ks = u.sync_n > 1 ? u.sync_n : 1;
    const int ks_len = n_ks > 1 ? ((in / n_ks + 127) / 128) * 128 : in;
    const int kbeg = min(in, u.ks * ks_len);
    const int kend = min(in, kbeg + ks_len);
    const int npass = (kend - kbeg + kPfPassK - 1) / kPfPassK;
    const int nfull = (kend - kbeg) / kPfPassK;  // passes that hold 128 of k (in is a multiple of 64: the last may hold 64)
    // The passes in order, but one further for every adapter, as above.  A call in us, in order / by adapter: rank 256 14336 -> 1024 394 / 386,
    // 8192 -> 2048 264 / 260, 4096 -> 4096 216 / 211; rank 192 14336 -> 1024 255 / 250; rank 128 8192 -> 2048 152.9 / 150.7.  (One further for
    // every tile of a group 370, 253, 211, 241 and 151, but a row's sums then come in an order that depends on where its token sits.)
    const int turn = first_pass(u.turn, nfull);
    auto pass_k = [&](int i) __attribute__((always_inline)) {
        return kbeg + kPfPassK * (i < nfull ? (i + turn < nfull ? i + turn : i + turn - nfull) : i);
    };

    // Loads without conditions (rows of tokens beyond ntok are the last token's, see xrow; a chunk beyond
    // the row is fetched from the row's last chunk and a k step beyond kend from the last step, neither
    // enters an MFMA): with a branch around a load the compiler no longer counts the loads in flight and
    // waits for all of them, the ones requested for later passes included, at every wait.
    auto x_pass = [&](int k0, uint4(&xs)[TB]) __attribute__((always_inline)) {
        const int kx = min(k0 + 8 * xc, in - 8);
#pragma unroll
        for (int i = 0; i < TB; ++i) xs[i] = ld16_stream(xrow[i] + kx);
    };
    auto w_step = [&](int k, int j) __attribute__((always_inline)) {
        return wa.ld(woff[j], min(k, in - 32) * wh[j]);
    };
    auto stage = [&](int base, const uint4(&xs)[TB]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < TB; ++t) *reinterpret_cast<uint4 *>(&buf[base + xr + 16 * t][8 * xc]) = xs[t];
    };
    // one 32-wide k step of the pass staged at `base`: rows of tokens beyond ntok hold the last token's x
    // and only reach accumulator columns that are never stored
    auto k_step = [&](int base, int d, const uint4(&ws)[JBW]) __attribute__((always_inline)) {
        bf16x8 xo[TB];
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
            xo[tb] = as_bf16x8(*reinterpret_cast<const uint4 *>(&buf[base + 16 * tb + n][32 * d + 8 * kq]));
#pragma unroll
        for (int j = 0; j < JBW; ++j) {
            const bf16x8 ww = as_bf16x8(ws[j]);
#pragma unroll
            for (int tb = 0; tb < TB; ++tb)
                acc[j][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ww, xo[tb], acc[j][tb], 0, 0, 0);
        }
    };

    // PD passes of x and WP passes of A^T are in flight per wavefront (registers).  The steady state has
    // no branch: pass i stages its x, asks for the x of pass i + PD, and after each k step for the rows of
    // A^T of the same step of pass i + WP.  One barrier per pass: the buffer a pass writes was last read
    // two passes ago, and every wavefront has passed the previous pass's barrier since those reads.
    uint4 xs[PD][TB], w[WP][SP][JBW];
#pragma unroll
    for (int q = 0; q < PD; ++q) {
        x_pass(pass_k(min(q, max(npass - 1, 0))), xs[q]);
        if (q < WP) {
#pragma unroll
            for (int d = 0; d < SP; ++d)
#pragma unroll
                for (int j = 0; j < JBW; ++j) w[q][d][j] = w_step(pass_k(q) + 32 * d, j);
        }
    }
#ifdef LORA_WG_CLOCKS
    unsigned long long c_wait = 0;  // from the top of a pass to the barrier's exit, summed over the passes
#endif
    int i0 = 0, kw = pass_k(WP), kx = pass_k(PD);
    const int kturn = kbeg + kPfPassK * nfull;  // behind the last whole pass comes the first
    for (; i0 + 2 * PD <= nfull; i0 += PD) {
#pragma unroll
        for (int q = 0; q < PD; ++q) {
            const int base = (q & 1) * TOK;
#ifdef LORA_WG_CLOCKS
            const unsigned long long c_top = wall_clock64();
#endif
            stage(base, xs[q]);
            x_pass(kx, xs[q]);
            kx = kx + kPfPassK < kturn ? kx + kPfPassK : kbeg;
            __syncthreads();
#ifdef LORA_WG_CLOCKS
            c_wait += wall_clock64() - c_top;
#endif
#pragma unroll
            for (int d = 0; d < SP; ++d) {
                k_step(base, d, w[q % WP][d]);
#pragma unroll
                for (int j = 0; j < JBW; ++j) w[q % WP][d][j] = w_step(kw + 32 * d, j);
            }
            kw = kw + kPfPassK < kturn ? kw + kPfPassK : kbeg;
        }
    }
    // the last passes (fewer than 2 PD, the last maybe 64 of k): the same, with every request and every k
    // step under its condition
#pragma unroll
    for (int q = 0; q < 2 * PD; ++q) {
        const int i = i0 + q;
        if (i < npass) {
            const int k0 = pass_k(i), kw = pass_k(i + WP);
            const int base = (q & 1) * TOK;
            stage(base, xs[q % PD]);
            if (i + PD < npass) x_pass(pass_k(i + PD), xs[q % PD]);
            __syncthreads();
#pragma unroll
            for (int d = 0; d < SP; ++d) {
                if (k0 + 32 * d < kend) k_step(base, d, w[q % WP][d]);
                if (i + WP < npass) {
#pragma unroll
                    for (int j = 0; j < JBW; ++j) w[q % WP][d][j] = w_step(kw + 32 * d, j);
                }
            }
        }
    }
#ifdef LORA_WG_CLOCKS
    if (g_clock_buf && threadIdx.x == 0 && blockIdx.x < g_clock_slots) g_clock_buf[(size_t)blockIdx.x * 8 + 1] = c_wait;
    LORA_CLOCK(2);
#endif
    const float vs = sy.scale_v ? u.scale : 1.f;
    const bool tiled = !v_f32 && !sy.scale_v;
    // lane (n, kq) holds, for token block tb and its row block j, v[token 16 tb + n][16 jb + 4 kq + e]
    if (tiled) {
        const Through slice(parts + (int64_t)(n_ks > 1 ? u.ks : 0) * slice_stride + u.v_off, ntok * u.r8);
        const int late = late_thread(), ln = late & 15, lk = (late >> 4) & 3;
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int j = 0; j < JBW; ++j) {
                const int j4 = 4 * (wave * JBW + j) + lk;
                if (j4 < (r8 >> 2) && 16 * tb + ln < ntok) {
                    const int q = tiled_quad(u.r8, ntok, 16 * tb + ln, (rr.first >> 2) + j4);
                    if (n_ks > 1)
                        slice.st(q, acc[j][tb]);
                    else
                        store_v4(acc[j][tb], u.v_off + 4 * q, v_hi, v_lo);
                }
            }
        if (n_ks > 1) complete_tile(u, rr, n_ks, slice_stride, parts, v_hi, v_lo, vs, true, sy, reinterpret_cast<unsigned *>(lds + kPrefillLds - 16));
        return;
    }
    // rows: they meet in LDS as they lie in v, all of the unit's tokens at once where they fit, else half of them
    constexpr int GO = 16 * TB * 64 * JBW * 4 + 16 <= kPrefillLds ? TB : TB / 2;
    static_assert(16 * GO * 64 * JBW * 4 + 16 <= kPrefillLds, "the rows in LDS");
    f32x4 *rows = reinterpret_cast<f32x4 *>(lds);
    const int quads = r8 >> 2;
#pragma unroll
    for (int g = 0; g < TB; g += GO) {
        __syncthreads();  // the x buffers, then the rows of the first half, have been read
#pragma unroll
        for (int tb = 0; tb < GO; ++tb)
#pragma unroll
            for (int j = 0; j < JBW; ++j) {
                const int j4 = 4 * (wave * JBW + j) + kq;
                if (j4 < quads) rows[(16 * tb + n) * quads + j4] = acc[j][g + tb];
            }
        __syncthreads();
        if (16 * g < ntok)
            store_heavy_rows(u, rr, n_ks, 16 * g, min(16 * GO, ntok - 16 * g), [&](int i) { return rows[i]; }, v_hi, v_lo, v_f32,
                             n_slices, slice_stride, parts, vs, false);
    }
    if (n_ks == 1 || v_f32) return;
    complete_tile(u, rr, n_ks, slice_stride, parts, v_hi, v_lo, vs, false, sy, reinterpret_cast<unsigned *>(lds + kPrefillLds - 16));
}

// One wavefront copies 1 KB from memory into LDS without passing through registers: lane l's 16 bytes
// at gptr (per lane) land at lds_piece + 16*l (lds_piece wave-uniform).  Written as an instruction the
// compiler does not look into: for its own form of this load it waits until the copy has landed
// before the wavefront may issue anything else that touches LDS or the registers involved, which
// leaves nothing of the overlap the copy exists for.  The caller waits and synchronises the work group before anyone
// reads the destination: for all of the wavefront's memory operations (vmcnt(0)), or for all but the last N, if at least N that the compiler
// knows of are issued behind the copies on every way to the wait: a branch or a scheduling barrier between keeps them there.
static __device__ __forceinline__ void dma16_to_lds(const uint4 *gptr, const uint4 *lds_piece)
{
    const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds_piece);
    // M0 carries the LDS address of the piece; its old value is put back, so the register the
    // compiler reserves for itself is unchanged after the statement
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\t"
                 "s_mov_b32 m0, %0"
                 : "=&s"(saved_m0)
                 : "v"(gptr), "s"(lds_addr)
                 : "memory");
}

// Two and four such copies, to consecutive KB from LDS address `to`, for a loop in which every instruction beside its matrix
// instructions counts.  An instruction's offset is added to the address in memory and to the one in LDS, so M0 is set once:
// copy q's source is given less q KB.
static __device__ __forceinline__ void dma16x2_to_lds(const void *g0, const void *g1, uint32_t to)
{
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\t"
                 "global_load_lds_dwordx4 %2, off offset:1024\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0)
                 : "v"(g0), "v"(g1), "s"(to)
                 : "memory");
}
static __device__ __forceinline__ void dma16x4_to_lds(const void *g0, const void *g1, const void *g2, const void *g3, uint32_t to)
{
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\t"
                 "global_load_lds_dwordx4 %2, off offset:1024\n\tglobal_load_lds_dwordx4 %3, off offset:2048\n\t"
                 "global_load_lds_dwordx4 %4, off offset:3072\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0)
                 : "v"(g0), "v"(g1), "v"(g2), "v"(g3), "s"(to)
                 : "memory");
}

// Picks the body by the unit's rank rows.  ANY = false: the launch holds no unit above rank 64 and the
// bodies fit 128 registers (four work groups per compute unit).  ANY = true: any rank (two work groups
// per compute unit); ranks above 64 take the row-split body, with 64 tokens up to rank 192 and 32 above.
template <bool ANY>
static __device__ __forceinline__ void prefill_dispatch(const Unit &u, const int32_t *__restrict__ perm,
                                                        const uint16_t *__restrict__ arena,
                                                        const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                        uint16_t *__restrict__ v_hi, uint16_t *__restrict__ v_lo,
                                                        float *__restrict__ v_f32, int n_slices,
                                                        int64_t slice_stride, char *lds,
                                                        float *__restrict__ parts, const Sync &sy)
{
    const int r8 = u.r8;
    const RankRows rr = {0, r8, 0, 1};
    // (three in flight for ranks up to 32: cfg2 4096 -> 4096 shrink 48.3 against 43.9 us)
    constexpr int XD = ANY ? 2 : 1;  // passes of x in flight per wavefront: two where two work groups share a compute unit
    if (r8 <= 16)
        shrink_prefill_ksplit<1, 2, 4, XD>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    else if (r8 <= 32)
        shrink_prefill_ksplit<2, 2, 4, XD>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    else if (!ANY)  // the launcher takes this form only for batches whose token-heavy units are all up to rank 64
        shrink_prefill_ksplit<4, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    else if (r8 <= 64)
        shrink_prefill_ksplit<4, 2, 4, XD>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    else if constexpr (ANY) {
        if (r8 <= 128)
            shrink_prefill_rowsplit<2, 4, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
        else if (r8 <= 192)
            shrink_prefill_rowsplit<3, 4, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
        else  // 32 tokens: the 16 accumulator tiles of 64 tokens x 64 rank rows per wavefront do not fit the registers
            shrink_prefill_rowsplit<4, 2, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    }
}

__global__ __launch_bounds__(kThreads, 4) void k_shrink_prefill(const Unit *__restrict__ units,
                                                                const int32_t *__restrict__ perm,
                                                                const uint16_t *__restrict__ arena,
                                                                const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                                uint16_t *__restrict__ v_hi,
                                                                uint16_t *__restrict__ v_lo,
                                                                float *__restrict__ v_f32, int n_slices,
                                                                int64_t slice_stride, float *__restrict__ parts, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kPrefillLds];
    if (units[blockIdx.x].ntok <= 0) return;  // a place the planner filled so that every XCD's list has the same length
    LORA_CLOCK(0);
    prefill_dispatch<false>(units[blockIdx.x], perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride,
                            lds, parts, sy);
    LORA_CLOCK(4);
}

// A launch of few token-heavy units of any rank, two work groups a unit (RankRows).  They run on one XCD (b mod 8), a row of 8 behind
// the other.  Units up to rank 32 are the first one's alone.
__global__ __launch_bounds__(kThreads, 2) void k_shrink_halves(const Unit *__restrict__ units,
                                                               const int32_t *__restrict__ perm,
                                                               const uint16_t *__restrict__ arena,
                                                               const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                               uint16_t *__restrict__ v_hi, uint16_t *__restrict__ v_lo,
                                                               float *__restrict__ v_f32, int n_slices, int64_t slice_stride,
                                                               float *__restrict__ parts, int n_units, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kPrefillLds];
    const int at = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7), part = (blockIdx.x >> 3) & 1;
    if (at >= n_units || units[at].ntok <= 0) return;  // behind the list, or a place that only pads an XCD's share of it
    const Unit &u = units[at];
    const int r8 = u.r8, half = r8 <= 32 ? r8 : (r8 / 2 + 15) & ~15;
    if (part && half == r8) return;
    LORA_CLOCK(0);
    const RankRows rr = {part * half, part ? r8 - half : half, part, half == r8 ? 1 : 2};
    if (r8 <= 64) {
        if (rr.n <= 16)
            shrink_prefill_ksplit<1, 2, 4, 2>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
        else
            shrink_prefill_ksplit<2, 2, 4, 2>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    } else if (r8 <= 128)
        shrink_prefill_rowsplit<1, 4, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    else if (r8 <= 192)
        shrink_prefill_rowsplit<2, 4, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    else
        shrink_prefill_rowsplit<2, 2, 2, 1>(u, rr, perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride, lds, parts, sy);
    LORA_CLOCK(4);
}

// A batch that has units above rank 64 runs all its token-heavy units here, in one launch: two
// launches one after the other (high ranks here, the rest above) measured slower, the first one
// leaving most of the chip idle.
__global__ __launch_bounds__(kThreads, 2) void k_shrink_prefill_any(const Unit *__restrict__ units,
                                                                    const int32_t *__restrict__ perm,
                                                                    const uint16_t *__restrict__ arena,
                                                                    const uint16_t *__restrict__ x, int64_t ldx,
                                                                    int in, uint16_t *__restrict__ v_hi,
                                                                    uint16_t *__restrict__ v_lo,
                                                                    float *__restrict__ v_f32, int n_slices,
                                                                    int64_t slice_stride, float *__restrict__ parts, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kPrefillLds];
    if (units[blockIdx.x].ntok <= 0) return;  // a place the planner filled so that every XCD's list has the same length
    LORA_CLOCK(0);
    prefill_dispatch<true>(units[blockIdx.x], perm, arena, x, ldx, in, v_hi, v_lo, v_f32, n_slices, slice_stride,
                           lds, parts, sy);
    LORA_CLOCK(4);
}

// ------------------------------------------------------------------------------------------------
// expand: one unit = (group, <=16 tokens, a run of output columns made of 128-column strips).
// MFMA orientation: tokens down (operand from v), output columns across (operand straight from
// 16-byte loads of B^T rows).  Inside a strip, MFMA b (0..7) takes column 8*n + b for its column
// slot n, so that after the eight MFMAs lane n holds 8 consecutive columns of up to 4 tokens: y is
// then read and written 16 bytes per lane.  The four wavefronts of a work group split the unit by
// strip and by k step (rank >= 128: one strip, one 32-wide slice of the rank each); partial tiles
// meet in LDS and are added in wavefront order by the y update, which all 256 threads share.
// v enters as two bf16 terms (hi + lo), so it keeps about 16 mantissa bits.
// ------------------------------------------------------------------------------------------------
constexpr int kStrip = 128;           // output columns per strip
constexpr int kPartRow = kStrip + 4;  // LDS row length of a partial tile in floats (padded)
constexpr int kExpandLds = 4 * kTokTile * kPartRow * 4;

// v operand of one 32-wide k step from the caller's fp32 v (complete, as lora_expand takes it): token n, 8 values,
// split into bf16 hi + lo.  Two plain 16-byte loads, so that those of all k steps go out together.  (Read
// through the loop that adds k-slices up, every k step was a trip to memory of its own with four times the
// loads: expand launch of 19,675 tokens of ranks 8..128, 4096 columns, 86 -> 69 us.)
static __device__ __forceinline__ void load_v_operand(const float *__restrict__ src, bool ok, bf16x8 &vhi, bf16x8 &vlo)
{
    f32x4 f0 = *reinterpret_cast<const f32x4 *>(src), f1 = *reinterpret_cast<const f32x4 *>(src + 4);
    if (!ok) {
        f0 = f32x4{0.f, 0.f, 0.f, 0.f};
        f1 = f0;
    }
    uint4 ph, pl;
    split_bf16(f0, f1, ph, pl);
    vhi = as_bf16x8(ph);
    vlo = as_bf16x8(pl);
}

// KSTEPS: 32-wide steps that cover the padded rank (1, 2, 4 or 8).
// BY: where v comes from, unless it is the caller's (VF32).
template <int KSTEPS, bool VF32, Slices BY>
static __device__ __forceinline__ void expand_body(const Unit &u, const uint16_t *__restrict__ arena,
                                                   const float *__restrict__ v_in, uint16_t *__restrict__ y, int64_t ldy, char *lds, const Sync &sy)
{
    constexpr int P = KSTEPS < 4 ? KSTEPS : 4;  // wavefronts that share one strip (each a part of the rank)
    constexpr int S = 4 / P;                    // strips per pass of the work group
    constexpr int ITEMS = KSTEPS / P;           // k steps per wavefront (1, or 2 for rank > 128)
    float(*part)[kTokTile][kPartRow] = reinterpret_cast<float(*)[kTokTile][kPartRow]>(lds);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int n = lane & 15;
    const int kq = lane >> 4;
    const int r8 = u.r8;
    const int ntok = u.ntok;
    const int ncols = u.pn;
    const uint4 zero = {0u, 0u, 0u, 0u};
    const int my_strip = wave / P;
    const int my_part = wave % P;

    // epilogue role of this thread: token e_tok, 8 columns starting at 8*e_cg of every strip
    const int e_tok = tid >> 4;
    const int e_cg = tid & 15;
    const bool e_ok = e_tok < ntok;
    const float scale = u.scale;
    // The row of y this thread updates, fetched before anything else: a wavefront's loads return in request order, so
    // requested behind the weights it would come back with the last of them, and the loads of y (which need it) would
    // only start then, a second trip to memory on the unit's critical path.
    const int64_t row = u.tok[e_ok ? e_tok : 0];
    __builtin_amdgcn_sched_barrier(0);

    int jc[ITEMS];
    bool j_ok[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int j = 32 * (my_part + P * it) + 8 * kq;
        j_ok[it] = j < r8;
        jc[it] = j_ok[it] ? j : 0;
    }
    // where this lane's piece of v begins (its token's row, k step it of the wavefront)
    auto v_at = [&](int it) __attribute__((always_inline)) {
        return u.v_off + (int64_t)(n < ntok && j_ok[it] ? n : 0) * r8 + jc[it];
    };

#pragma unroll 1  // else its first pass is taken out of the loop: half as much code again
    for (int c0 = 0; c0 < ncols; c0 += S * kStrip) {
        const int cs = c0 + my_strip * kStrip;  // this wavefront's strip
        const bool strip_ok = cs < ncols;
        // this lane's piece of sub-block 0, rank piece 0 of the wavefront's strip; sub-block b is
        // 16*r8 elements further, rank piece kp 128 elements further
        const uint16_t *brow = arena + u.w_off + (int64_t)(strip_ok ? cs : 0) * r8 + n * 8;
        // weights: row (column of y) cs + 8*n + b, 16 bytes at jc, of the wavefront's first k step.  Ranks above 128, two k
        // steps: the second's are requested as the first's registers come free.  (With both requested behind the wait for v a launch
        // of 10 units lasted 6.6 us, now 5.7; 6076 units of 576 -> 11136, ranks 1 to 256, 52.5 -> 49.6.)
        uint4 w[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) w[b] = ld16_stream(brow + b * 16 * r8 + jc[0] * 16);
        // nothing that needs the row index (a wait for its load) moves up in front of these requests
        __builtin_amdgcn_sched_barrier(0);

        uint16_t *e_y = y + row * ldy + u.p0 + 8 * e_cg;
        uint4 yv[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            // no per-lane condition around the 16-byte load (it would be split into four masked
            // 4-byte loads): threads without a token read the unit's first token's row
            yv[s] = zero;
            if (c0 + s * kStrip < ncols) yv[s] = ld16_stream(e_y + c0 + s * kStrip);
        }
        // (single launch) y and the weights of the first k step are on their way while v is waited for
        if (BY == kSlicesByWaiting && c0 == 0) wait_for(sy, u.sync_idx, u.sync_n);
        uint4 vh[ITEMS], vl[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const bool ok = (n < ntok) && j_ok[it];
            uint4 ph, pl;
            if (VF32) {
                bf16x8 h, l;
                load_v_operand(v_in + v_at(it), ok, h, l);
                ph = __builtin_bit_cast(uint4, h);
                pl = __builtin_bit_cast(uint4, l);
            } else if (BY == kSlicesByShrink) {
                ph = ld16(sy.v_hi + v_at(it));
                pl = ld16(sy.v_lo + v_at(it));
            } else {
                f32x4 p0[kMaxSlices], p1[kMaxSlices], f0, f1;
                load_slices<BY == kSlicesByExpand>(sy.parts + v_at(it), sy.n_slices, sy.slice_stride, p0, p1);
                add_slices(p0, p1, sy.n_slices, f0, f1);
                split_bf16(f0, f1, ph, pl);
            }
            vh[it] = ok ? ph : zero;
            vl[it] = ok ? pl : zero;
        }

        if (c0 > 0) __syncthreads();  // the previous pass's partial tiles have been consumed
        f32x4 acc[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bf16x8 ww = as_bf16x8(j_ok[it] ? w[b] : zero);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vh[it]), ww, acc[b], 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vl[it]), ww, acc[b], 0, 0, 0);
                if (it + 1 < ITEMS) w[b] = ld16_stream(brow + b * 16 * r8 + jc[it + 1] * 16);
            }
        }
        if (strip_ok) {
            // lane (n, kq) holds tokens 4*kq + e, columns 8*n + b
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int tok = 4 * kq + e;
                if (tok < ntok) {
                    const f32x4 lo = {acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
                    const f32x4 hi = {acc[4][e], acc[5][e], acc[6][e], acc[7][e]};
                    *reinterpret_cast<f32x4 *>(&part[wave][tok][8 * n]) = lo;
                    *reinterpret_cast<f32x4 *>(&part[wave][tok][8 * n + 4]) = hi;
                }
            }
        }
        __syncthreads();
        if (e_ok) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if (c0 + s * kStrip < ncols) {
                    f32x4 d0 = *reinterpret_cast<const f32x4 *>(&part[s * P][e_tok][8 * e_cg]);
                    f32x4 d1 = *reinterpret_cast<const f32x4 *>(&part[s * P][e_tok][8 * e_cg + 4]);
#pragma unroll
                    for (int p = 1; p < P; ++p) {
                        d0 += *reinterpret_cast<const f32x4 *>(&part[s * P + p][e_tok][8 * e_cg]);
                        d1 += *reinterpret_cast<const f32x4 *>(&part[s * P + p][e_tok][8 * e_cg + 4]);
                    }
                    const uint4 yy = yv[s];
                    uint4 o;
                    o.x = pack_bf16_rne(bf16_bits_to_f32(yy.x & 0xFFFFu) + scale * d0[0],
                                        __uint_as_float(yy.x & 0xFFFF0000u) + scale * d0[1]);
                    o.y = pack_bf16_rne(bf16_bits_to_f32(yy.y & 0xFFFFu) + scale * d0[2],
                                        __uint_as_float(yy.y & 0xFFFF0000u) + scale * d0[3]);
                    o.z = pack_bf16_rne(bf16_bits_to_f32(yy.z & 0xFFFFu) + scale * d1[0],
                                        __uint_as_float(yy.z & 0xFFFF0000u) + scale * d1[1]);
                    o.w = pack_bf16_rne(bf16_bits_to_f32(yy.w & 0xFFFFu) + scale * d1[2],
                                        __uint_as_float(yy.w & 0xFFFF0000u) + scale * d1[3]);
                    st16_stream(e_y + c0 + s * kStrip, o);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// expand of token-heavy groups: one unit = (group, up to 64 tokens, a run of 128-column strips), a work group takes two of the
// strips.  Each wavefront owns 16 of the tokens and all of the rank, so nothing is summed across wavefronts; a strip's B^T tile
// (128 columns x rank, one contiguous piece of the pool) is copied into LDS once per work group and read from there by the four
// wavefronts; the MFMA result (token x column, lane n holding 8 consecutive columns of 4 tokens) goes straight to the y update,
// 16 bytes per lane, four 256-byte row pieces per store.
// y, read and written once, is nearly all the bytes, and what the memory gives for it depends on how much of it is asked for at a
// time and where: a kernel that only adds to 161 MB in place takes 51 us (6.4 TB/s) in the order of the addresses, 51 to 54 with 64
// rows x 512 bytes per work group, neighbours along the row, 56 with 64 x 256, 60 to 63 with a work group that walks 2 KB of its
// rows in steps of 256 bytes, 67 with 8 KB.  So a work group takes 64 tokens x 256 columns and ends, and the work groups of a row of
// units are neighbours in the launch.  19,675 tokens, 4096 / 8192 / 14336 columns, expand launch in us, a run of 8 to 28 strips walked by
// each work group / as here: rank 16 63.7 / 54.4, 136 / 106, 233 / 191; rank 64 68.4 / 58.9, 141 / 114, 242 / 203; rank 128 81.6 / 69.9,
// 165 / 132, 280 / 235; rank 256 130 / 105, 288 / 208, 521 / 390.  (The tiles in another order, or rows known to be consecutive without
// a look at perm: level.)
// That asks for v and B^T oftener, which therefore come in whole KB of operand order (tiled_quad; B^T as the pool holds it), and for
// 128 registers and 32 KB of LDS, four work groups on a compute unit: the low ranks' tiles of both strips, or one strip's up to rank
// 128, or half of one's.  Up to rank 128 launches of their own and of more than those four (big_spread) ask for 16 KB of LDS more, so that
// three run there: less of y is under way at a time (rank 16 56.6 / 54.4, rank 64 61.8 / 58.9, rank 128 70.9 / 69.9; two per compute unit 61.5,
// 64.0, 80.9), while above the fourth hides more of the copies (rank 256 106 / 109).  Beside units of up to 16 tokens (k_expand_mixed) four
// are as fast as three or up to 3 % faster.
// ------------------------------------------------------------------------------------------------
constexpr int kBigStrips = 2;                 // strips of a work group
constexpr int kBigTile = 32 * 1024;           // bytes of B^T in LDS at a time
constexpr int kBigSpread = 16 * 1024;         // LDS that a launch asks for beside it where big_spread says so
static_assert(kBigStrips * kStrip == kBigCols, "columns of a work group");

typedef __attribute__((ext_vector_type(16), aligned(4))) int i32x16;

// mine[e] = v[4 * (lane / 16) + e], of scalars: a quarter of the wavefront at a time, all lanes of which run here.  (The compiler makes branches
// of it, or takes registers that spill.)
static __device__ __forceinline__ void rows_by_quarter(const i32x16 &v, int (&mine)[4])
{
    unsigned long long all;
    asm volatile("s_mov_b64 %4, exec\n\ts_mov_b32 exec_lo, 0xffff\n\ts_mov_b32 exec_hi, 0\n\t"
        "v_mov_b32 %0, %5\n\tv_mov_b32 %1, %6\n\tv_mov_b32 %2, %7\n\tv_mov_b32 %3, %8\n\t"
        "s_mov_b32 exec_lo, 0xffff0000\n\t"
        "v_mov_b32 %0, %9\n\tv_mov_b32 %1, %10\n\tv_mov_b32 %2, %11\n\tv_mov_b32 %3, %12\n\t"
        "s_mov_b32 exec_lo, 0\n\ts_mov_b32 exec_hi, 0xffff\n\t"
        "v_mov_b32 %0, %13\n\tv_mov_b32 %1, %14\n\tv_mov_b32 %2, %15\n\tv_mov_b32 %3, %16\n\t"
        "s_mov_b32 exec_hi, 0xffff0000\n\t"
        "v_mov_b32 %0, %17\n\tv_mov_b32 %1, %18\n\tv_mov_b32 %2, %19\n\tv_mov_b32 %3, %20\n\t"
        "s_mov_b64 exec, %4"
        : "=&v"(mine[0]), "=&v"(mine[1]), "=&v"(mine[2]), "=&v"(mine[3]), "=&s"(all)
        : "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]), "s"(v[8]), "s"(v[9]), "s"(v[10]),
          "s"(v[11]), "s"(v[12]), "s"(v[13]), "s"(v[14]), "s"(v[15]));
}

// eight columns of y, plus scale times element e of the sums of each
static __device__ __forceinline__ uint4 add_scaled(uint4 yy, float scale, const f32x4 (&acc)[8], int e)
{
    uint4 o;
    o.x = pack_bf16_rne(bf16_bits_to_f32(yy.x & 0xFFFFu) + scale * acc[0][e], __uint_as_float(yy.x & 0xFFFF0000u) + scale * acc[1][e]);
    o.y = pack_bf16_rne(bf16_bits_to_f32(yy.y & 0xFFFFu) + scale * acc[2][e], __uint_as_float(yy.y & 0xFFFF0000u) + scale * acc[3][e]);
    o.z = pack_bf16_rne(bf16_bits_to_f32(yy.z & 0xFFFFu) + scale * acc[4][e], __uint_as_float(yy.z & 0xFFFF0000u) + scale * acc[5][e]);
    o.w = pack_bf16_rne(bf16_bits_to_f32(yy.w & 0xFFFFu) + scale * acc[6][e], __uint_as_float(yy.w & 0xFFFF0000u) + scale * acc[7][e]);
    return o;
}

// KSTEPS: 32-wide steps of a chunk of the rank (1, 2 or 4); CHUNKS of 128 of it.
template <int KSTEPS, int CHUNKS, bool VF32>
static __device__ __forceinline__ void expand_big_body(const Unit &u, int c0, const int32_t *__restrict__ perm,
                                                       const uint16_t *__restrict__ arena,
                                                       const float *__restrict__ v_in, uint16_t *__restrict__ y, int64_t ldy, char *lds, const Sync &sy)
{
    static_assert(CHUNKS == 1 || KSTEPS == 4, "a chunk is 128 of the rank");
    constexpr int HELD = KSTEPS <= 2 ? kBigStrips : 1;  // strips whose tiles the LDS holds at a time
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15;
    const int kq = lane >> 4;
    const int r8 = u.r8;
    const int ntok_all = u.ntok;
    const int nstrips = min(kBigStrips, (u.pn - c0) / kStrip);
    const uint4 zero = {0u, 0u, 0u, 0u};
    const float scale = u.scale;
    const int tile_pieces = 16 * r8;  // 16-byte pieces in one strip's tile (128 * r8 * 2 / 16)
    const int nt = min(kTokTile, ntok_all - kTokTile * wave);  // may be <= 0: the wavefront only helps copying
    uint4 *ltile = reinterpret_cast<uint4 *>(lds);
    const uint4 *gtile = reinterpret_cast<const uint4 *>(arena + u.w_off + (int64_t)c0 * r8);

    // Batch rows of the wavefront's tokens, through the scalar cache in one load.  Behind the group's last token it brings other groups', or
    // what lies behind perm in the table, where the unit list alone is longer than 60 bytes; none of those is used.  (One load a
    // token, each at an address of its own, and a choice by branches stood in front of the requests: launches of one round of work groups of
    // ranks up to 32 lasted longer than those of the units that walked their strips.  us a call, such units / a load a token / this way, 4096
    // columns: 17 tiles, rank 16 10.9 / 11.6 / 10.7, 32 tiles 12.3 / 12.5 / 11.7; 4096 features, 24 tiles, rank 8 14.1 / 14.4 / 13.8.  Ranks up to 32
    // of many tokens, where the memory is busy anyhow, lose by it: 19,600 tokens, rank 16, 4096 columns 75.3 / 73.5 / 74.3, 8192 145 / 136.4 / 136.9.)
    const i32x16 row = *reinterpret_cast<const i32x16 *>(perm + u.perm_off + (nt > 0 ? kTokTile * wave : 0));

    // Chunk c of the tile of strip s into LDS (HELD > 1: of all strips), 1 KB per wavefront and step, nothing through registers: sub-block
    // b and k step st take 64 pieces in operand order whatever the rank, so that the reads' addresses differ by constants.  Rank
    // pieces beyond the padded rank are copies of the first one.
    auto copy_tile = [&](int s, int c) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < HELD; ++h) {
            if (h > 0 && h >= nstrips) break;
#pragma unroll
            for (int st = 0; st < KSTEPS; ++st) {
                if (128 * c + 32 * st < r8) {
                    int kp = 16 * c + 4 * st + kq;
                    kp = 8 * kp < r8 ? kp : 0;
#pragma unroll
                    for (int bb = 0; bb < 2; ++bb) {
                        // Ranks of 65 to 128, where half of the tile is asked for at a time and in front of the products: the tiles of tokens
                        // begin with different sub-blocks, not all of an XCD's work groups with the same lines of its L2.  us a call, 512 features,
                        // rank 128, in order / in turn: 4096 columns, 32 tiles 18.0 / 17.6, 19,600 tokens 87.7 / 85.9; 14336 columns 258.5 / 255.0; above
                        // rank 128 level, up to rank 64 1 % slower.
                        const int b = (2 * wave + bb + (KSTEPS == 4 && CHUNKS == 1 ? u.tok0 >> 6 : 0)) & 7;
                        dma16_to_lds(gtile + (int64_t)(s + h) * tile_pieces + (b * (r8 >> 3) + kp) * 16 + n,
                                     ltile + ((h * 8 + b) * KSTEPS + st) * 64);
                    }
                }
            }
        }
    };
    uint4 vh[KSTEPS], vl[KSTEPS];
    auto load_v = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int st = 0; st < KSTEPS; ++st) {
            const int j = 128 * c + 32 * st + 8 * kq;
            const bool ok = n < nt && j < r8;
            uint4 ph, pl;
            if (!VF32) {
                const int64_t off = u.v_off + 16 * wave * r8 + (j < r8 ? j : 0) * nt + 8 * min(n, nt - 1);
                ph = ld16(sy.v_hi + off);
                pl = ld16(sy.v_lo + off);
            } else {
                bf16x8 h, l;
                load_v_operand(v_in + u.v_off + (int64_t)(ok ? kTokTile * wave + n : 0) * r8 + (j < r8 ? j : 0), ok, h, l);
                ph = __builtin_bit_cast(uint4, h);
                pl = __builtin_bit_cast(uint4, l);
            }
            vh[st] = ok ? ph : zero;
            vl[st] = ok ? pl : zero;
        }
    };
    f32x4 acc[8];
    auto compute = [&](int held, int c) __attribute__((always_inline)) {
        const uint4 *t = ltile + lane;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            if (c == 0) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < KSTEPS; ++st) {
                if (128 * c + 32 * st < r8) {  // uniform
                    const uint4 wv = t[((held * 8 + b) * KSTEPS + st) * 64];
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vh[st]), as_bf16x8(wv), acc[b], 0, 0, 0);
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vl[st]), as_bf16x8(wv), acc[b], 0, 0, 0);
                }
            }
        }
    };
    // the MFMA leaves tokens 4*kq + e (e = 0..3), columns 8*n .. 8*n+7 of the strip in this lane
    uint16_t *yrow[4];
    uint4 yv[kBigStrips][4];
    auto update = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (4 * kq + e < nt) st16_stream(yrow[e] + s * kStrip, add_scaled(yv[s][e], scale, acc, e));
        }
    };

    // unconditional (rows of absent tokens are the wavefront's first token's: a per-lane condition around a 16-byte load makes the compiler split it
    // into four masked 4-byte loads)
    auto fetch_y = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) yv[s][e] = ld16_stream(yrow[e] + s * kStrip);
    };
    copy_tile(0, 0);
    __builtin_amdgcn_sched_barrier(0);  // the rows of y behind the copies: the wait below counts them
    if (nt > 0) {
        load_v(0);
        __builtin_amdgcn_sched_barrier(0);
        int mine[4];
        rows_by_quarter(row, mine);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 4 * kq + e < nt ? mine[e] : row[0];
            yrow[e] = y + (int64_t)r * ldy + u.p0 + c0 + 8 * n;
        }
        fetch_y(0);
        if (HELD > 1 && nstrips > 1) {
            fetch_y(1);
            wait_vm<8>();  // all but the rows of y: the copies have landed
        } else {
            wait_vm<4>();
        }
    } else {
        wait_vm<0>();
    }
    __syncthreads();
    if (HELD > 1) {
        if (nt <= 0) return;
#pragma unroll
        for (int s = 0; s < kBigStrips; ++s)
            if (s < nstrips) {
                compute(s, 0);
                update(s);
            }
    } else {
        static_assert(kBigStrips == 2, "two strips, one after the other");
        auto multiply = [&](int s) __attribute__((always_inline)) {
            if (nt > 0) compute(0, 0);
            if (CHUNKS > 1) {
                __syncthreads();  // everyone has read the chunk
                copy_tile(s, 1);
                if (nt > 0) load_v(1);
                wait_vm<0>();
                __syncthreads();
                if (nt > 0) compute(0, 1);
            }
        };
        multiply(0);
        if (nstrips > 1) {
            __syncthreads();
            copy_tile(1, 0);
            // (the rows of y stand in a block of their own behind the copies; a scheduling barrier here made ranks up to 64, which do not
            // come this way, 2 to 4 % slower by other registers)
            if (nt > 0) {
                if (CHUNKS > 1) load_v(0);
                fetch_y(1);
                update(0);
            }
            // behind the copies: four rows of y, and a full wavefront's four stores
            if (nt == kTokTile)
                wait_vm<8>();
            else if (nt > 0)
                wait_vm<4>();
            else
                wait_vm<0>();
            __syncthreads();
            multiply(1);
            if (nt > 0) update(1);
        } else if (nt > 0) {
            update(0);
        }
    }
}

// All of a unit that its work groups use, in one trip to the scalar cache and not field by field where each is first needed.
static __device__ __forceinline__ void load_big_unit(const Unit &u)
{
    asm volatile("" ::"s"(u.w_off), "s"(u.v_off), "s"(u.r8), "s"(u.ntok), "s"(u.p0), "s"(u.pn), "s"(u.scale), "s"(u.perm_off), "s"(u.tok0));
}

template <bool VF32>
static __device__ __forceinline__ void expand_big_dispatch(const Unit &u, int c0, const int32_t *__restrict__ perm,
                                                           const uint16_t *__restrict__ arena,
                                                           const float *__restrict__ v_in, uint16_t *__restrict__ y, int64_t ldy, char *lds, const Sync &sy)
{
    const int r8 = u.r8;
    if (r8 <= 32)
        expand_big_body<1, 1, VF32>(u, c0, perm, arena, v_in, y, ldy, lds, sy);
    else if (r8 <= 64)
        expand_big_body<2, 1, VF32>(u, c0, perm, arena, v_in, y, ldy, lds, sy);
    else if (r8 <= 128)
        expand_big_body<4, 1, VF32>(u, c0, perm, arena, v_in, y, ldy, lds, sy);
    else
        expand_big_body<4, 2, VF32>(u, c0, perm, arena, v_in, y, ldy, lds, sy);
}

// ------------------------------------------------------------------------------------------------
// The same units with v as the caller of lora_expand has it, fp32 in rows, in launches mostly of ranks above 128 (expand_walks): a work group walks
// strips of its unit and each wavefront loads its tokens' v once, as bf16 hi + lo of every k step in registers.  There v is more bytes than
// a strip's rows of y, 32 of each of 16 rows at a time, and work groups of two strips and two chunks of the rank load it four times.
// A launch of few units takes several work groups a unit, as many as stay within two per compute unit.
// The tile of a strip is 128 * r8 * 2 bytes: two buffers of 32 KB up to rank 128, above one of 64 KB, filled between two strips; while a
// strip computes, the next one's rows of y (and tile) are on their way.
// ------------------------------------------------------------------------------------------------
constexpr int kWalkTile = 64 * 1024;

template <int KSTEPS>
static __device__ __forceinline__ void expand_walk_body(const Unit &u, int c0, int nstrips, const int32_t *__restrict__ perm,
                                                        const uint16_t *__restrict__ arena, const float *__restrict__ v_in,
                                                        uint16_t *__restrict__ y, int64_t ldy, char *lds)
{
    static_assert(KSTEPS <= 8, "ranks up to 256");
    constexpr bool TWO = KSTEPS <= 4;  // buffers
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6, wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int n = lane & 15;
    const int kq = lane >> 4;
    const int r8 = u.r8;
    const uint4 zero = {0u, 0u, 0u, 0u};
    const int32_t *toks = perm + u.perm_off;
    const float scale = u.scale;
    const int tile_pieces = 16 * r8;  // 16-byte pieces in one strip's tile
    const int nt = min(kTokTile, u.ntok - kTokTile * wave);  // may be <= 0: the wavefront only helps copying
    uint4 vh[KSTEPS], vl[KSTEPS];
    bool j_ok[KSTEPS];
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st) {
        const int j = 32 * st + 8 * kq;
        j_ok[st] = j < r8;
        const bool ok = n < nt && j_ok[st];
        bf16x8 h, l;
        load_v_operand(v_in + u.v_off + (int64_t)(ok ? kTokTile * wave + n : 0) * r8 + (j_ok[st] ? j : 0), ok, h, l);
        vh[st] = ok ? __builtin_bit_cast(uint4, h) : zero;
        vl[st] = ok ? __builtin_bit_cast(uint4, l) : zero;
    }
    // the MFMA leaves tokens 4*kq + e (e = 0..3), columns 8*n .. 8*n+7 of the strip in this lane
    uint16_t *yrow[4];
    bool y_ok[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        y_ok[e] = 4 * kq + e < nt;
        yrow[e] = y + (int64_t)toks[y_ok[e] ? kTokTile * wave + 4 * kq + e : 0] * ldy + u.p0 + c0 + 8 * n;
    }
    const uint4 *gtile = reinterpret_cast<const uint4 *>(arena + u.w_off + (int64_t)c0 * r8);  // strip s starts tile_pieces * s further
    uint4 *ltile = reinterpret_cast<uint4 *>(lds);
    // From the first strip on, or (walks and rows of whole multiples of 4 KB) every tile of tokens of a group from another one: all units walk at
    // about the same pace and would ask a part of the memory's channels for y at any one time.  (19,675 tokens, rank 128, 8192 columns 184 / 167 us.)
    const int turn = nstrips * kStrip * 2 % 4096 == 0 && (ldy * 2) % 4096 == 0 ? (u.tok0 >> 6) * 5 % nstrips : 0;
    auto strip_at = [&](int i) __attribute__((always_inline)) { return i + turn < nstrips ? i + turn : i + turn - nstrips; };
    // 1 KB per wavefront and step, nothing through registers; the tile is a multiple of 64 pieces, so a wavefront's is whole or absent
    auto copy_tile = [&](int buf, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2 * KSTEPS; ++q) {
            const int piece0 = 64 * wave_u + kThreads * q;
            if (piece0 < tile_pieces) dma16_to_lds(gtile + (int64_t)s * tile_pieces + piece0 + lane, ltile + buf * 2048 + piece0);
        }
    };
    uint4 ya[4], yb[4];
    auto fetch_y = [&](int s, uint4(&yv)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) yv[e] = ld16_stream(yrow[e] + s * kStrip);  // unconditional, as above
    };
    auto compute = [&](int s, int buf, const uint4(&yv)[4]) __attribute__((always_inline)) {
        if (nt <= 0) return;
        const uint4 *t = ltile + buf * 2048;
        f32x4 acc[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < KSTEPS; ++st) {
                if (32 * st < r8) {  // uniform
                    // (sub-block b, rank piece 4*st + kq, column slot n; lanes beyond the padded rank read piece 0, their v is zero)
                    const uint4 wv = t[(b * (r8 >> 3) + (j_ok[st] ? 4 * st + kq : 0)) * 16 + n];
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vh[st]), as_bf16x8(wv), acc[b], 0, 0, 0);
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vl[st]), as_bf16x8(wv), acc[b], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (y_ok[e]) st16_stream(yrow[e] + s * kStrip, add_scaled(yv[e], scale, acc, e));
    };

    // (stores_done waits by the builtin, so the compiler knows that y is there; behind wait_vm<0> it waits once more, for what has been asked
    // for since: rank 192, 14336 columns, 63 tiles 58.8 / 62.2 us)
    copy_tile(0, strip_at(0));
    fetch_y(strip_at(0), ya);
    stores_done();
    __syncthreads();
    for (int s = 0; s < nstrips; s += 2) {
        // even strips from buffer 0, odd strips from buffer 1 (above rank 128 all from the one buffer, when everyone has read the strip before)
        if (s + 1 < nstrips) {
            if (TWO) copy_tile(1, strip_at(s + 1));
            fetch_y(strip_at(s + 1), yb);
        }
        compute(strip_at(s), 0, ya);
        if (s + 1 >= nstrips) break;
        if (!TWO) {
            __syncthreads();
            copy_tile(0, strip_at(s + 1));
        }
        stores_done();
        __syncthreads();
        if (s + 2 < nstrips) {
            if (TWO) copy_tile(0, strip_at(s + 2));
            fetch_y(strip_at(s + 2), ya);
        }
        compute(strip_at(s + 1), TWO ? 1 : 0, yb);
        if (s + 2 >= nstrips) break;
        if (!TWO) {
            __syncthreads();
            copy_tile(0, strip_at(s + 2));
        }
        stores_done();
        __syncthreads();
    }
}

// Which unit and which of its strips work group b of a launch of 64-token units takes: a row of 8 units takes 8 * subs work groups,
// each unit's on places of one residue mod 8, i.e. on one XCD.  subs = how many work groups a unit of the list has; lists of several
// projections of unlike width have sections behind the first one.  (With the widest projection's subs for all of them, work groups
// without columns returning at once, q|k|v of 9,100 tokens took 55.5 us, 52.5 without those.)
struct BigMore {
    int n;                                                                       // sections behind the first
    int first_place[kMaxBigSections], first_unit[kMaxBigSections], subs[kMaxBigSections];  // the end in [n], n < kMaxBigSections
};
struct BigPlace {
    int unit, c0;  // unit < 0: none
    __device__ __forceinline__ BigPlace(int b, int n_first, int subs, const BigMore &more)
    {
        int from = 0, to = n_first;
        const int rows = (n_first + 7) >> 3;
        if (b >= 8 * rows * subs) {
            int s = 0;
            while (s + 1 < more.n && b >= more.first_place[s + 1]) ++s;
            b -= more.first_place[s];
            from = more.first_unit[s];
            to = more.first_unit[s + 1];
            subs = more.subs[s];
        }
        const int t = b >> 3;
        const int q = (subs & (subs - 1)) ? (int)((unsigned)t / (unsigned)subs) : t >> __builtin_ctz(subs);
        unit = from + 8 * q + (b & 7);
        if (unit >= to) unit = -1;
        c0 = (t - q * subs) * (kBigStrips * kStrip);
    }
};

template <bool VF32, Slices BY = kSlicesByShrink>
static __device__ __forceinline__ void expand_dispatch(const Unit &u, const uint16_t *__restrict__ arena,
                                                       const float *__restrict__ v_in, uint16_t *__restrict__ y, int64_t ldy, char *lds, const Sync &sy)
{
    const int r8 = u.r8;
    if (r8 <= 32)
        expand_body<1, VF32, BY>(u, arena, v_in, y, ldy, lds, sy);
    else if (r8 <= 64)
        expand_body<2, VF32, BY>(u, arena, v_in, y, ldy, lds, sy);
    else if (r8 <= 128)
        expand_body<4, VF32, BY>(u, arena, v_in, y, ldy, lds, sy);
    else
        expand_body<8, VF32, BY>(u, arena, v_in, y, ldy, lds, sy);
}


// ------------------------------------------------------------------------------------------------
// Decode apply in one launch.  A decode co-batch is a few tens of megabytes of adapter weights read
// once: at that size a launch lasts about as long as its first and its last byte take to arrive, and
// two launches pay that twice.  Here one grid of at most one work group (16 wavefronts) per compute
// unit does both halves:
//   * work group b runs shrink unit b exactly as k_shrink_wide does (same tiles, same order of
//     additions, so v and y are bitwise those of the two launches), then each of its four groups of
//     four wavefronts runs expand unit 4b + q as k_expand does.  Empty places in either list (ntok
//     == 0) are skipped.  The expand units' B^T operands and rows of y are requested as soon as the
//     work group's part of v has been stored, so the chip's loads of B^T follow those of A^T without
//     the tail, the pause and the ramp of a launch boundary;
//   * v is handed over inside an XCD.  Each of the chip's XCDs has an L2 of its own, and a store that
//     must reach memory queues behind everything the chip has requested (several microseconds once
//     the loads of B^T are out).  The work groups of a launch go to the XCDs in turn (work group b to
//     the XCD of b mod 8), and the host puts every shrink unit and every expand unit of one (group,
//     token tile) at places of one residue mod 8: v is then written with plain stores into that XCD's
//     L2, the tile's ready counter is bumped by an atomic that the L2 executes, the expand units poll it
//     with a returning atomic (executed by the L2 as well; a plain load could be served by the compute
//     unit's L1) and read v with agent-scope loads, which pass the compute unit's L1 and are served
//     by the L2.  (Not plain loads behind an L1 invalidate: at work-group scope the invalidate does
//     nothing here, and a 128-byte line of v can hold rows of two tiles, so that a unit of the same work
//     group may have fetched the line before this tile's rows were stored; the agent-scope
//     invalidate, which does drop the lines, made the launch 2.6 times as long.)
//     The counters only grow: the target is epoch * sync_n, epoch = such launches the table has seen.
//     Every work group checks that the work groups on its XCD all have its residue (see the start of
//     the kernel); if not it sets bit 1 of the time-out flag: the launch's result is then not valid
//     and lora_segments_check says so.
//   * every work group stores its part of v before its first wait, and the grid fits the chip, so
//     every wait ends; it is bounded all the same (spin_limit polls, then bit 0 of the flag).
// ------------------------------------------------------------------------------------------------
constexpr int kDecodeMaxGrid = 256;  // work groups of the launch at most (one per compute unit)
static_assert(4 * kExpandLds <= kWideWaves * kWideSlab, "the four expand units' partial tiles fit where the x regions were");

// returning atomic OR with 0: the counter's value as the L2 holds it
static __device__ __forceinline__ unsigned l2_counter_value(unsigned *p)
{
    unsigned v;
    const unsigned zero = 0u;
    asm volatile("global_atomic_or %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p), "v"(zero) : "memory");
    return v;
}

// atomic add executed by the L2, nothing returned
static __device__ __forceinline__ void l2_counter_add(unsigned *p, unsigned n)
{
    asm volatile("global_atomic_add %0, %1, off" : : "v"(p), "v"(n) : "memory");
}

__global__ __launch_bounds__(kWideThreads) void k_decode_fused(
    const Unit *__restrict__ s_units, int n_s, const Unit *__restrict__ e_units, int n_e,
    const uint16_t *__restrict__ arena, const uint16_t *__restrict__ x, int64_t ldx, int in, int k_slice_len,
    int n_slices, uint16_t *__restrict__ y, int64_t ldy, unsigned xcc_map, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kWideLds + 64];  // + one flag per group of four wavefronts, 8 words of the XCD check
    const int bid = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = wave >> 2;  // shrink: the k-slice this wavefront works on; expand: its group of four
    const int wq = wave & 3;      // its place among the four
    const int i = lane & 15;
    const int kq = lane >> 4;
    const uint4 zero = {0u, 0u, 0u, 0u};
    uint16_t(*slab)[kWideRow] = reinterpret_cast<uint16_t(*)[kWideRow]>(lds + wave * kWideSlab);
    f32x4(*red)[64] = reinterpret_cast<f32x4(*)[64]>(lds + kWideWaves * kWideSlab);
    volatile unsigned *qflag = reinterpret_cast<volatile unsigned *>(lds + kWideLds) + slice;
    if (tid < 4) reinterpret_cast<volatile unsigned *>(lds + kWideLds)[tid] = 0u;
    // the shrink unit's record, one request (load_unit_words)
    const uint32_t s_rec = load_unit_words(s_units + (bid < n_s ? bid : 0));
    // Which XCD do the work groups of each residue run on?  The hardware deals the work groups of a
    // launch to the XCDs in turn, but not every launch starts at the same XCD: all that the hand-over
    // needs is that work groups of one residue mod 8 share an XCD, i.e. that every work group on an XCD
    // finds the same difference d between its place and the XCD's position in the dealing order
    // (xcc_map: 4 bits per XCD number, its position as a probe launch found it).  Each work group
    // leaves (epoch, XCD, d) in a word of its own (a plain store: nothing waits for it); the words
    // alternate between two sets from launch to launch, and the last work group of the following launch
    // (the one with the lightest shrink unit, where a trip to memory in front of the operand loads
    // costs the launch nothing) reads what the finished launch left: two values of d on one XCD mean
    // that its result cannot be trusted (bit 1 of the time-out flag).  The host reads the last launch's
    // set itself.
    // hardware register XCC_ID, bits 3:0
    const unsigned xcc = __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u;
    const unsigned my_d = ((unsigned)bid - ((xcc < 8u ? xcc_map >> (4 * xcc) : 0u) & 15u)) & 7u;
    unsigned *const xcd_words = sy.timeout_flag + 4;  // [2][kDecodeMaxGrid]
    if (bid == (int)gridDim.x - 1 && sy.epoch > 1u) {
        volatile unsigned *seen = reinterpret_cast<volatile unsigned *>(lds + kWideLds) + 4;  // 8 words
        if (tid < 8) seen[tid] = 0u;
        __syncthreads();
        if (tid < (int)gridDim.x) {
            const unsigned left = xcd_words[kDecodeMaxGrid * ((sy.epoch + 1u) & 1u) + tid];
            if ((left >> 8) == ((sy.epoch - 1u) & 0xFFFFFFu)) {
                if ((left & 0x80u) == 0u)
                    atomicOr(const_cast<unsigned *>(seen) + ((left >> 4) & 7u), 1u << (left & 7u));
                else
                    atomicOr(sy.timeout_flag, 2u);  // an XCD number beyond 7
            }
        }
        __syncthreads();
        if (tid < 8) {
            const unsigned d_seen = seen[tid];
            if (d_seen & (d_seen - 1u)) {
                atomicOr(sy.timeout_flag, 2u);
                sy.timeout_flag[2] = (tid << 8) | d_seen;  // the XCD and the differences seen there
            }
        }
    }
    if (tid == 0) xcd_words[kDecodeMaxGrid * (sy.epoch & 1u) + bid] = (sy.epoch << 8) | (xcc << 4) | my_d;
    LORA_CLOCK(0);
#ifdef LORA_WG_CLOCKS
    if (g_clock_buf && tid == 0 && blockIdx.x < g_clock_slots)
        g_clock_buf[(size_t)blockIdx.x * 8 + 5] = 1000 + (__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u);
#endif

    // ---- the shrink unit ----
    auto s_word = [&](int w) __attribute__((always_inline)) { return unit_word(s_rec, w); };
    const int ntok = (int)s_word(5), pn = (int)s_word(7);
    const bool s_has = bid < n_s && ntok > 0;
    if (s_has) {
        const uint64_t u_w_off = s_word(0) | ((uint64_t)s_word(1) << 32);
        const int64_t u_v_off = (int64_t)(s_word(2) | ((uint64_t)s_word(3) << 32));
        const int u_r8 = (int)s_word(4), u_p0 = (int)s_word(6), u_sync_idx = (int)s_word(12);
        const bool w_ok = i < pn;
        const int blk_rows = min(kRowTile, u_r8 - (u_p0 & ~(kRowTile - 1)));
        const int row0 = u_p0 & (kRowTile - 1);
        const uint16_t *wrow = arena + u_w_off + (kq * blk_rows + row0 + (w_ok ? i : 0)) * 8;
        const int half = lane >> 5;
        const int s_chunk = lane & 31;
        const uint16_t *xrow[kTokTile / 2];
#pragma unroll
        for (int t = 0; t < kTokTile / 2; ++t) {
            const int tok_even = (int)s_word(16 + 2 * t), tok_odd = (int)s_word(17 + 2 * t);
            xrow[t] = x + (int64_t)(half ? tok_odd : tok_even) * ldx;
        }
        const int kslice_beg = slice * k_slice_len;
        int kslice_end = kslice_beg + k_slice_len;
        if (kslice_end > in) kslice_end = in;
        if (slice >= n_slices) kslice_end = kslice_beg;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int kp = kslice_beg; kp < kslice_end; kp += 4 * kWideK) {
            const int kbeg = kp + wq * kWideK;  // wavefront-uniform
            if (kbeg >= kslice_end) break;
            uint4 a[kShrinkSteps];
#pragma unroll
            for (int q = 0; q < kShrinkSteps; ++q) {
                const int k = kbeg + 32 * q;
                a[q] = (k < kslice_end) ? ld16_stream(wrow + (int64_t)k * blk_rows) : zero;
            }
            int kx = kbeg + 8 * s_chunk;
            if (kx > in - 8) kx = in - 8;
            uint4 xs[kTokTile / 2];
#pragma unroll
            for (int t = 0; t < kTokTile / 2; ++t)
                if (2 * t < ntok) xs[t] = ld16(xrow[t] + kx);
#pragma unroll
            for (int t = 0; t < kTokTile / 2; ++t)
                if (2 * t < ntok) *reinterpret_cast<uint4 *>(&slab[2 * t + half][8 * s_chunk]) = xs[t];
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
            for (int q = 0; q < kShrinkSteps; ++q) {
                const int k = kbeg + 32 * q;
                if (k < kslice_end) {
                    const uint4 aa = w_ok ? a[q] : zero;
                    const uint4 bb = *reinterpret_cast<const uint4 *>(&slab[i][32 * q + 8 * kq]);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aa), as_bf16x8(bb), acc, 0, 0, 0);
                }
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        }
        LORA_CLOCK(1);
        // the sixteen tiles added in the order of the k-slice plan (inside a slice by wavefront, then the
        // slices), by wavefront 0 alone: one barrier instead of two
        red[wave][lane] = acc;
        __syncthreads();
        if (wave == 0) {
            f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sl = 0; sl < kMaxSlices; ++sl) {
                if (sl < n_slices) {
                    f32x4 ts = red[4 * sl][lane];
                    ts += red[4 * sl + 1][lane];
                    ts += red[4 * sl + 2][lane];
                    ts += red[4 * sl + 3][lane];
                    t = sl ? t + ts : ts;
                }
            }
            if (i < ntok && 4 * kq < pn) {
                const int64_t off = u_v_off + (int64_t)i * u_r8 + 4 * kq;
                uint2 h, l;
                h.x = pack_bf16_rne(t[0], t[1]);
                h.y = pack_bf16_rne(t[2], t[3]);
                l.x = pack_bf16_rne(t[0] - bf16_bits_to_f32(h.x & 0xFFFFu), t[1] - __uint_as_float(h.x & 0xFFFF0000u));
                l.y = pack_bf16_rne(t[2] - bf16_bits_to_f32(h.y & 0xFFFFu), t[3] - __uint_as_float(h.y & 0xFFFF0000u));
                *reinterpret_cast<uint2 *>(sy.v_hi + off) = h;
                *reinterpret_cast<uint2 *>(sy.v_lo + off) = l;
            }
        }
        // Nobody requests expand operands before the stores of v have been issued: a compute unit passes
        // its memory operations on in the order they were issued, and behind 120 KB of requests for B^T
        // the stores would reach the L2 microseconds later.
        __syncthreads();
        LORA_CLOCK(7);
        if (wave == 0) {
            stores_done();  // the stores have reached the L2
            if (lane == 0) l2_counter_add(sy.ready + u_sync_idx, 1u);
            LORA_CLOCK(2);
        }
    } else {
        __syncthreads();  // the flags in LDS are set
    }

    // ---- the expand unit of this group of four wavefronts ----
    const int e_idx = 4 * bid + slice;
    const Unit *eu = e_units + (e_idx < n_e ? e_idx : 0);
    const int e_ntok = e_idx < n_e ? eu->ntok : 0;
    const bool e_has = e_ntok > 0;
    const int qtid = tid & 255;
    const int e_tok = qtid >> 4;  // epilogue role: token e_tok of the unit, 8 columns from 8*e_cg of every strip
    const int e_cg = qtid & 15;
    float(*part)[kTokTile][kPartRow] = reinterpret_cast<float(*)[kTokTile][kPartRow]>(lds + slice * kExpandLds);
    const int e_r8 = eu->r8, e_ncols = eu->pn;
    const int P = e_r8 <= 32 ? 1 : (e_r8 <= 64 ? 2 : 4);  // wavefronts that share a strip, each a part of the rank
    const int S = 4 / P;                                   // strips per pass
    const int my_strip = wq / P, my_part = wq % P;
    const int j0 = 32 * my_part + 8 * kq, j1 = 32 * (my_part + 4) + 8 * kq;
    const bool j_ok0 = j0 < e_r8, j_ok1 = j1 < e_r8;
    const int jc0 = j_ok0 ? j0 : 0, jc1 = j_ok1 ? j1 : 0;
    const bool strip_ok = my_strip * kStrip < e_ncols;
    uint4 w[8], yv[4];
    uint16_t *e_y = y;
    const uint16_t *brow = arena;
    if (e_has) {
        // requests that do not need v: the B^T operands of the first k step and the rows of y
        const int64_t row = eu->tok[e_tok < e_ntok ? e_tok : 0];
        brow = arena + eu->w_off + (int64_t)(strip_ok ? my_strip * kStrip : 0) * e_r8 + i * 8;
#pragma unroll
        for (int b = 0; b < 8; ++b) w[b] = ld16_stream(brow + b * 16 * e_r8 + jc0 * 16);
        e_y = y + row * ldy + eu->p0 + 8 * e_cg;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            yv[s] = zero;
            if (s < S && s * kStrip < e_ncols) yv[s] = ld16_stream(e_y + s * kStrip);
        }
        // Wait for the tile's v.  The first wavefront of the four polls the tile's counter in the L2 and
        // tells the other three through LDS.
        if (wq == 0) {
            const unsigned target = sy.epoch * (unsigned)eu->sync_n;
            unsigned spins = 0;
            // one lane polls (an atomic is executed once per lane, even on one address)
            for (;;) {
                unsigned seen = 0u;
                if (lane == 0) seen = l2_counter_value(sy.ready + eu->sync_idx);
                seen = __builtin_amdgcn_readfirstlane(seen);
                if ((int)(seen - target) >= 0) break;
                if (++spins > sy.spin_limit) {
                    if (lane == 0) atomicOr(sy.timeout_flag, 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(4);
            }
            if (lane == 0) *qflag = 1u;
        } else {
            unsigned spins = 0;
            while (*qflag == 0u) {
                if (++spins > sy.spin_limit) break;  // the polling wavefront reports the time-out
                __builtin_amdgcn_s_sleep(2);
            }
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        LORA_CLOCK(3);
        const bool ok0 = (i < e_ntok) && j_ok0;
        const int64_t off0 = eu->v_off + (int64_t)(ok0 ? i : 0) * e_r8 + jc0;
        // Agent-scope loads, which do not stop at this compute unit's vector cache: a 128-byte line of v
        // can hold rows of two token tiles, and another unit of this work group may have fetched the line
        // for its own tile before this tile's rows were stored (seen as rows without their delta, on a
        // first, cold launch at 14,336 input features, where the shrink units end far apart).
        uint4 vh0 = ld_through_u16x8(sy.v_hi + off0), vl0 = ld_through_u16x8(sy.v_lo + off0);
        uint4 vh1 = zero, vl1 = zero;
        const bool ok1 = (i < e_ntok) && j_ok1;
        if (e_r8 > 128) {
            const int64_t off1 = eu->v_off + (int64_t)(ok1 ? i : 0) * e_r8 + jc1;
            vh1 = ld_through_u16x8(sy.v_hi + off1);
            vl1 = ld_through_u16x8(sy.v_lo + off1);
        }
        if (!ok0) vh0 = vl0 = zero;
        if (!ok1) vh1 = vl1 = zero;
        f32x4 acc[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bf16x8 ww = as_bf16x8(j_ok0 ? w[b] : zero);
            acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vh0), ww, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vl0), ww, acc[b], 0, 0, 0);
        }
        if (e_r8 > 128) {
            // the second k step of ranks above 128 re-uses the operand registers
#pragma unroll
            for (int b = 0; b < 8; ++b) w[b] = ld16_stream(brow + b * 16 * e_r8 + jc1 * 16);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bf16x8 ww = as_bf16x8(j_ok1 ? w[b] : zero);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vh1), ww, acc[b], 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vl1), ww, acc[b], 0, 0, 0);
            }
        }
        if (strip_ok) {
            // lane (n, kq) holds tokens 4*kq + e, columns 8*n + b
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int tok = 4 * kq + e;
                if (tok < e_ntok) {
                    const f32x4 lo = {acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
                    const f32x4 hi = {acc[4][e], acc[5][e], acc[6][e], acc[7][e]};
                    *reinterpret_cast<f32x4 *>(&part[wq][tok][8 * i]) = lo;
                    *reinterpret_cast<f32x4 *>(&part[wq][tok][8 * i + 4]) = hi;
                }
            }
        }
    }
    __syncthreads();
    if (e_has && e_tok < e_ntok) {
        const float scale = eu->scale;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s < S && s * kStrip < e_ncols) {
                f32x4 d0 = *reinterpret_cast<const f32x4 *>(&part[s * P][e_tok][8 * e_cg]);
                f32x4 d1 = *reinterpret_cast<const f32x4 *>(&part[s * P][e_tok][8 * e_cg + 4]);
                for (int p = 1; p < P; ++p) {
                    d0 += *reinterpret_cast<const f32x4 *>(&part[s * P + p][e_tok][8 * e_cg]);
                    d1 += *reinterpret_cast<const f32x4 *>(&part[s * P + p][e_tok][8 * e_cg + 4]);
                }
                const uint4 yy = yv[s];
                uint4 o;
                o.x = pack_bf16_rne(bf16_bits_to_f32(yy.x & 0xFFFFu) + scale * d0[0],
                                    __uint_as_float(yy.x & 0xFFFF0000u) + scale * d0[1]);
                o.y = pack_bf16_rne(bf16_bits_to_f32(yy.y & 0xFFFFu) + scale * d0[2],
                                    __uint_as_float(yy.y & 0xFFFF0000u) + scale * d0[3]);
                o.z = pack_bf16_rne(bf16_bits_to_f32(yy.z & 0xFFFFu) + scale * d1[0],
                                    __uint_as_float(yy.z & 0xFFFF0000u) + scale * d1[1]);
                o.w = pack_bf16_rne(bf16_bits_to_f32(yy.w & 0xFFFFu) + scale * d1[2],
                                    __uint_as_float(yy.w & 0xFFFF0000u) + scale * d1[3]);
                st16_stream(e_y + s * kStrip, o);
            }
        }
    }
    LORA_CLOCK(4);
}

// One work group per place of a launch writes the XCD it runs on (hardware register XCC_ID, bits 3:0).
__global__ void k_probe_xcc(unsigned *out)
{
    if (threadIdx.x == 0) out[blockIdx.x] = __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u;
}

constexpr int kFusedLds = kShrinkLds > kExpandLds ? kShrinkLds : kExpandLds;

__global__ __launch_bounds__(kThreads) void k_shrink(const Unit *__restrict__ units,
                                                     const uint16_t *__restrict__ arena,
                                                     const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                     int k_slice_len, float *__restrict__ v_out, int n_slices,
                                                     int64_t slice_stride, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kShrinkLds];
    LORA_CLOCK(0);
    shrink_body(units[blockIdx.x], arena, x, ldx, in, k_slice_len, v_out, n_slices, slice_stride, lds, sy);
    LORA_CLOCK(4);
}

// Units of up to 16 tokens (BIG is false: those of 64 run in k_expand_big), whose token indices are their own.  VF32: v is fp32 from
// the caller (stand-alone expand).
template <bool BIG, bool VF32>
__global__ __launch_bounds__(kThreads, 4) void k_expand(const Unit *__restrict__ units, const int32_t *__restrict__ /* perm */,
                                                        const uint16_t *__restrict__ arena, const float *__restrict__ v_in,
                                                        uint16_t *__restrict__ y, int64_t ldy, Sync sy)
{
    static_assert(!BIG, "units of up to 16 tokens");
    __shared__ __attribute__((aligned(16))) char lds[kExpandLds];
    LORA_CLOCK_E(0);
    expand_dispatch<VF32>(units[blockIdx.x], arena, v_in, y, ldy, lds, sy);
    LORA_CLOCK_E(4);
}

// Units of up to 64 tokens (token-heavy groups), token indices from perm, `subs` work groups a unit.
template <bool VF32>
__global__ __launch_bounds__(kThreads, 4) void k_expand_big(const Unit *__restrict__ units, int n_first, int subs,
                                                            const int32_t *__restrict__ perm,
                                                            const uint16_t *__restrict__ arena,
                                                            const float *__restrict__ v_in, uint16_t *__restrict__ y,
                                                            int64_t ldy, Sync sy, BigMore more)
{
    __shared__ __attribute__((aligned(16))) char lds[kBigTile];
    const BigPlace p(blockIdx.x, n_first, subs, more);
    if (p.unit < 0) return;
    const Unit &u = units[p.unit];
    load_big_unit(u);
    if (p.c0 >= u.pn) return;
    if (p.c0 == 0) LORA_CLOCK_E_UNIT(p.unit, 0);
    expand_big_dispatch<VF32>(u, p.c0, perm, arena, v_in, y, ldy, lds, sy);
    if (p.c0 == 0) LORA_CLOCK_E_UNIT(p.unit, 4);
}

// ... and with v from the caller in launches mostly of ranks above 128: a work group walks `strips` of its unit's.
__global__ __launch_bounds__(kThreads, 2) void k_expand_walk(const Unit *__restrict__ units, int n_units, int strips,
                                                             const int32_t *__restrict__ perm, const uint16_t *__restrict__ arena,
                                                             const float *__restrict__ v_in, uint16_t *__restrict__ y, int64_t ldy)
{
    __shared__ __attribute__((aligned(16))) char lds[kWalkTile];
    const int part = (int)(blockIdx.x / (unsigned)n_units), unit = (int)blockIdx.x - part * n_units;
    const Unit &u = units[unit];
    const int r8 = u.r8, c0 = part * strips * kStrip;
    if (c0 >= u.pn) return;
    const int n = min(strips, (u.pn - c0) / kStrip);
    if (c0 == 0) LORA_CLOCK_E_UNIT(unit, 0);
    if (r8 <= 32)
        expand_walk_body<1>(u, c0, n, perm, arena, v_in, y, ldy, lds);
    else if (r8 <= 64)
        expand_walk_body<2>(u, c0, n, perm, arena, v_in, y, ldy, lds);
    else if (r8 <= 128)
        expand_walk_body<4>(u, c0, n, perm, arena, v_in, y, ldy, lds);
    else
        expand_walk_body<8>(u, c0, n, perm, arena, v_in, y, ldy, lds);
    if (c0 == 0) LORA_CLOCK_E_UNIT(unit, 4);
}

// Units of up to 16 tokens whose v the launch before left as k-slices' partial sums.
__global__ __launch_bounds__(kThreads, 4) void k_expand_parts(const Unit *__restrict__ units, const uint16_t *__restrict__ arena,
                                                              uint16_t *__restrict__ y, int64_t ldy, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kExpandLds];
    LORA_CLOCK_E(0);
    expand_dispatch<false, kSlicesByExpand>(units[blockIdx.x], arena, nullptr, y, ldy, lds, sy);
    LORA_CLOCK_E(4);
}

// Both halves in one launch: blocks [0, n_shrink) are shrink units, the rest expand units that wait
// for their tokens' v through the counters.
__global__ __launch_bounds__(kThreads, 4) void k_apply_fused(const Unit *__restrict__ shrink_units, int n_shrink,
                                                          const Unit *__restrict__ expand_units,
                                                          const uint16_t *__restrict__ arena,
                                                          const uint16_t *__restrict__ x, int64_t ldx, int in,
                                                          int k_slice_len, float *__restrict__ parts, int n_slices,
                                                          int64_t slice_stride, uint16_t *__restrict__ y,
                                                          int64_t ldy, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kFusedLds];
    const int b = blockIdx.x;
    if (b < n_shrink)
        shrink_body(shrink_units[b], arena, x, ldx, in, k_slice_len, parts, n_slices, slice_stride, lds, sy);
    else
        expand_dispatch<false, kSlicesByWaiting>(expand_units[b - n_shrink], arena, nullptr, y, ldy, lds, sy);
}

// A mixed batch in two launches on one queue: the token-heavy groups' units first in the grid (they
// last longest), the decode-sized groups' k-slice units behind them, which fill the places the long
// units leave.  Every unit does what it does in a launch of its own kind: the token-heavy shrink
// units write v complete as bf16 hi + lo, the k-slice units leave partial sums and the one that
// completes a token tile writes its hi + lo; both kinds of expand unit read v from there.
constexpr int kMixedShrinkLds = kPrefillLds > kShrinkLds ? kPrefillLds : kShrinkLds;
constexpr int kMixedExpandLds = kBigTile > kExpandLds ? kBigTile : kExpandLds;

template <bool ANY>
__global__ __launch_bounds__(kThreads, ANY ? 2 : 4) void k_shrink_mixed(
    const Unit *__restrict__ heavy_units, int n_heavy, const Unit *__restrict__ units,
    const int32_t *__restrict__ perm, const uint16_t *__restrict__ arena, const uint16_t *__restrict__ x, int64_t ldx,
    int in, int k_slice_len, float *__restrict__ parts, int n_slices, int64_t slice_stride, Sync sy)
{
    __shared__ __attribute__((aligned(16))) char lds[kMixedShrinkLds];
    const int b = blockIdx.x;
    if (b < n_heavy && heavy_units[b].ntok <= 0) return;  // a place that only pads an XCD's list of token-heavy units
    LORA_CLOCK(0);
    if (b < n_heavy)
        prefill_dispatch<ANY>(heavy_units[b], perm, arena, x, ldx, in, sy.v_hi, sy.v_lo, nullptr, n_slices,
                              slice_stride, lds, parts, sy);
    else
        shrink_body(units[b - n_heavy], arena, x, ldx, in, k_slice_len, parts, n_slices, slice_stride, lds, sy);
    LORA_CLOCK(4);
}

template <Slices BY>
__global__ __launch_bounds__(kThreads, 4) void k_expand_mixed(const Unit *__restrict__ big_units, int n_first, int subs, int big_grid,
                                                              const Unit *__restrict__ units,
                                                              const uint16_t *__restrict__ arena, const int32_t *__restrict__ perm,
                                                              uint16_t *__restrict__ y, int64_t ldy, Sync sy, BigMore more)
{
    __shared__ __attribute__((aligned(16))) char lds[kMixedExpandLds];
    const int b = blockIdx.x;
    if (b < big_grid) {
        const BigPlace p(b, n_first, subs, more);
        if (p.unit < 0) return;
        const Unit &u = big_units[p.unit];
        load_big_unit(u);
        if (p.c0 >= u.pn) return;
        if (p.c0 == 0) LORA_CLOCK_E_UNIT(p.unit, 0);
        expand_big_dispatch<false>(u, p.c0, perm, arena, nullptr, y, ldy, lds, sy);
        if (p.c0 == 0) LORA_CLOCK_E_UNIT(p.unit, 4);
    } else {
        [[maybe_unused]] const int n_big = more.n ? more.first_unit[more.n] : n_first;
        LORA_CLOCK_E_UNIT(n_big + b - big_grid, 0);
        expand_dispatch<false, BY>(units[b - big_grid], arena, nullptr, y, ldy, lds, sy);
        LORA_CLOCK_E_UNIT(n_big + b - big_grid, 4);
    }
}

__global__ __launch_bounds__(256) void k_reduce_slices(const float *__restrict__ parts, int n_slices,
                                                       int64_t slice_stride, float *__restrict__ v, int64_t n)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n) return;
    float acc = parts[idx];
    for (int sl = 1; sl < n_slices; ++sl) acc += parts[idx + (int64_t)sl * slice_stride];
    v[idx] = acc;
}

// ------------------------------------------------------------------------------------------------
// The adapted layer as one GEMM whose epilogue adds the delta: y = bf16(x W + s_a (x A_a) B_a), y written
// once and never read (the delta on its own reads y and writes it back: two thirds of its traffic on
// token-heavy batches).  Rows are taken in the order "tokens grouped by adapter", without padding between
// the groups; x is gathered and y scattered through that order, so no copy of either is made.  A 16-row
// MFMA block may hold several adapters: its delta is added piece by piece (LinPiece), each piece's MFMAs
// with the other rows' v at zero.
//   * One work group (8 wavefronts) computes a 256 x 256 tile, wavefront w the rows 64 (w mod 4) .. + 63
//     of it and the 128-column strip w / 4: 4 x 8 MFMA tiles of 16 x 16, 128 accumulator registers.  With
//     the columns of sub-block b being 8 n + b, lane n ends up with 8 consecutive columns of 4 tokens per
//     row block, and y leaves in 16-byte pieces.  (A compute unit takes about 50 GB/s from the L2s
//     whatever it runs; a 256 x 128 tile draws 48 KB per 64 of k and sat exactly at that rate, 720 us for
//     cfg2's 22.5 k x 4096 x 4096; two strips per tile share the 32 KB of x.)
//   * Everything is copied by loads that write LDS directly, through two rings that take all of a compute unit's LDS: x in
//     three slots of 64 of k, W in four of 32.  No request passes through registers the compiler tracks, so the waits are
//     exact.  W comes packed in operand order (1 KB per wavefront operand, see launch_pack_weight), so a 32-wide k step of a
//     strip is 8 KB of consecutive bytes.  x is gathered in operand order by the copy itself, in full cache lines: a copy
//     takes 128 bytes (64 of k) of 8 rows (64 bytes of 16 rows took twice as long to arrive).  Inside a 1 KB block of x, piece p
//     of row r sits in slot 8 r + (p XOR r), so that the 8 lanes that read one piece of 8 rows meet 8 bank groups.
//   * Per k step a compute unit's LDS hands out 96 KB and its matrix units work 1024 cycles: either alone takes about as long
//     as the other, so they have to run beside each other.  The two wavefronts of a SIMD (one of each strip) therefore take
//     turns: a k step is a phase that reads the step's 12 operands from LDS and requests copies, and a phase of its 32 MFMAs,
//     with a barrier behind every phase and the second strip's wavefronts one phase behind, so that in every phase one
//     wavefront of each SIMD multiplies while the other reads.  With all eight reading and then multiplying behind one barrier per
//     pair of k steps the matrix units were busy half of the time, now 73 %; us for x W alone (19,675 tokens,
//     before / now / the library's product): 4096 -> 4096 561 / 470 / 603, 1024 -> 4096 158 / 140 / 161, 8192 -> 8192 2227 /
//     1860 / 1902; the adapted layer at 4096 -> 4096 623 / 543.  The reading phase is the longer one: every instruction in
//     it counts (four copies behind one setting of M0 instead of four 2 %), and it holds four copies, not six and two (1.5 %),
//     in front of the reads (1.5 %).  Phases of 16 MFMAs 4 - 6 % slower; copies requested between the MFMAs 4 %; raised wave
//     priority for the MFMAs nothing.  Lines touched 4 to 16 pairs ahead, so that copies hit the L2: 1 to 5 % slower, the
//     copies do not wait for memory.
//   * Before the k loop, while its first copies are on their way, every wavefront starts its accumulators with
//     (s v_hi + s v_lo) B_a of its rows' adapters: ceil(r8 / 32) more k steps (v rows, and B^T in the pool's
//     operand order, the very pieces the expand kernels read; v was scaled before its split), B^T taken once
//     for all row blocks of one adapter.
// ------------------------------------------------------------------------------------------------
constexpr int kLinThreads = 512;
constexpr int kLinXRing = 3, kLinWRing = 4;
constexpr int kLinXBuf = kLinTileM * 128;               // bytes of x per slot: 64 of k
constexpr int kLinWBuf = 8 * 1024 * (kLinTileN / 128);  // bytes of W per slot: one k step of 2 strips, 8 KB each
constexpr int kLinLds = kLinXRing * kLinXBuf + kLinWRing * kLinWBuf;  // 160 KB, all of a compute unit's LDS: one work group per compute unit
static_assert(kLinTileM == 256 && kLinTileN == 256, "the wavefront roles below are written for 256 x 256");

// v B_a of one piece for NB sub-blocks from b0 of the strip at column c0: rows outside the piece get zero.  NK
// 32-wide steps of the rank from j0, all their operands requested before the first is used.
template <int NB, int NK>
static __device__ __forceinline__ void lin_delta_steps(const LinPiece &pc, int j0, const uint16_t *__restrict__ bt, int b0,
                                                       bool row_ok, int64_t v_row, int kq,
                                                       const uint16_t *__restrict__ v_hi,
                                                       const uint16_t *__restrict__ v_lo, f32x4 (&dl)[NB])
{
    const uint4 zero = {0u, 0u, 0u, 0u};
    const int r8 = pc.r8;
    uint4 vh[NK], vl[NK], w[NK][NB];
#pragma unroll
    for (int st = 0; st < NK; ++st) {
        const int j = j0 + 32 * st + 8 * kq, jc = j < r8 ? j : 0;  // lanes beyond the rank: any address, v at zero
        vh[st] = ld16(v_hi + v_row + jc);
        vl[st] = ld16(v_lo + v_row + jc);
        // piece (sub-block b0 + b, rank piece jc / 8, column slot n) of the strip's B^T tile
#pragma unroll
        for (int b = 0; b < NB; ++b) w[st][b] = ld16(bt + ((b0 + b) * (r8 >> 3) + (jc >> 3)) * 128);
    }
#pragma unroll
    for (int st = 0; st < NK; ++st) {
        const bool ok = row_ok && j0 + 32 * st + 8 * kq < r8;
        const bf16x8 h = as_bf16x8(ok ? vh[st] : zero), l = as_bf16x8(ok ? vl[st] : zero);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            dl[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, as_bf16x8(w[st][b]), dl[b], 0, 0, 0);
            dl[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, as_bf16x8(w[st][b]), dl[b], 0, 0, 0);
        }
    }
}

template <int NB, int NK>
static __device__ __forceinline__ void lin_delta(const LinPiece &pc, const uint16_t *__restrict__ arena, size_t c0, int b0,
                                                 int n, int kq, const uint16_t *__restrict__ v_hi,
                                                 const uint16_t *__restrict__ v_lo, f32x4 (&dl)[NB])
{
    const int r8 = pc.r8, row = n - (pc.place & 15);
    const bool row_ok = row >= 0 && row < pc.ntok;
    const uint16_t *bt = arena + pc.b_off + c0 * r8 + n * 8;
    const int64_t v_row = pc.v_off + (int64_t)(row_ok ? row : 0) * r8;
#pragma unroll
    for (int b = 0; b < NB; ++b) dl[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (r8 <= 32)
        lin_delta_steps<NB, 1>(pc, 0, bt, b0, row_ok, v_row, kq, v_hi, v_lo, dl);
    else if (r8 <= 64)
        lin_delta_steps<NB, 2>(pc, 0, bt, b0, row_ok, v_row, kq, v_hi, v_lo, dl);
    else
        for (int j = 0; j < r8; j += 32 * NK) lin_delta_steps<NB, NK>(pc, j, bt, b0, row_ok, v_row, kq, v_hi, v_lo, dl);
}

// adds it to the piece's own rows: the zeros above times another adapter's weights are zero only if those are
// finite, and what an adapter holds must not reach the tokens of its neighbours
template <int NB>
static __device__ __forceinline__ void lin_add(const LinPiece &pc, int kq, const f32x4 (&dl)[NB], f32x4 (&acc)[NB])
{
    const int row0 = pc.place & 15;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool mine = 4 * kq + e >= row0 && 4 * kq + e < row0 + pc.ntok;
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b][e] = mine ? acc[b][e] + dl[b][e] : acc[b][e];
    }
}

static __device__ __forceinline__ void linear_big_body(
    int mt, int nt, const int32_t *__restrict__ rows, const int32_t *__restrict__ start,
    const LinPiece *__restrict__ pieces, const uint16_t *__restrict__ arena, const uint16_t *__restrict__ wp,
    const uint16_t *__restrict__ x, int64_t ldx, int in, int out, const uint16_t *__restrict__ v_hi,
    const uint16_t *__restrict__ v_lo, uint16_t *__restrict__ y, int64_t ldy, char *lds)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave & 3;                     // rows 64 rw .. 64 rw + 63 of the tile
    const int strip = 2 * nt + (wave >> 2);      // this wavefront's 128-column strip
    // out is a multiple of 128: the last tile may hold one strip.  The four wavefronts without one take part in everything
    // up to the epilogue, so that copies and barriers count alike, and multiply strip 0's W for nothing; with all eight behind one
    // barrier per pair of k steps they left that out, and the tile was slower still: 19,664 tokens at 4096 -> 384 169 -> 148 us,
    // 8,000 at 4096 -> 640 123 -> 101, at 256 -> 384 27.6 -> 25.9.
    const bool has_strip = strip * 128 < out;
    const int n = lane & 15, kq = lane >> 4;
    const int m0 = mt * kLinTileM;
    // Copies of x.  A copy takes 8 rows x 128 bytes (64 of k): full cache lines; with 64 bytes of 16 rows per
    // copy the same bytes took twice as long to arrive (0.57 against 0.33 us per 32 of k and compute unit
    // in a kernel that only copies).  A slot holds the tile's 256 rows as 32 blocks of 1 KB; this wavefront fills blocks
    // 4 wave .. + 3, its lane l the slot l of a block with piece (l mod 8) XOR (l / 8) of row l / 8, so that the 8 lanes
    // that read one piece of 8 rows meet 8 different bank groups.
    char *const xring = lds, *const wring = lds + kLinXRing * kLinXBuf;
    const uint16_t *xsrc[4];
    {
        const int r = lane >> 3, piece = (lane & 7) ^ r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = rows[m0 + 8 * (4 * wave + j) + r];
            xsrc[j] = x + (int64_t)(row < 0 ? 0 : row) * ldx + 8 * piece - 512 * j;  // as dma16x4_to_lds takes it
        }
    }
    // copies of W: k step h of a strip is 8 KB at wp + (strip * (in / 32) + h) * 4096 elements; the four
    // wavefronts of a strip copy two of its eight 1 KB pieces each.  (The wavefronts of a strip the matrix
    // does not have copy strip 0's pieces into their unused half: every wavefront then has the same
    // number of copies in flight, which the waits below count.)
    const uint4 *wsrc = reinterpret_cast<const uint4 *>(wp + (size_t)(has_strip ? strip : 0) * (in / 32) * 4096) + 2 * rw * 64 + lane;
    const int w_half = (wave >> 2) * (kLinWBuf / 2);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds);
    const uint32_t x_end = lds0 + kLinXRing * kLinXBuf, w_end = lds0 + kLinLds;
    uint32_t x_to = lds0 + 4 * wave * 1024, w_to = x_end + w_half + 2 * rw * 1024;  // where the next pair, the next k step goes
    auto issue_x = [&]() __attribute__((always_inline)) {
        dma16x4_to_lds(xsrc[0], xsrc[1], xsrc[2], xsrc[3], x_to);
#pragma unroll
        for (int q = 0; q < 4; ++q) xsrc[q] += 64;
        x_to = x_to + kLinXBuf >= x_end ? x_to - (kLinXRing - 1) * kLinXBuf : x_to + kLinXBuf;
    };
    auto issue_w = [&]() __attribute__((always_inline)) {
        dma16x2_to_lds(wsrc, wsrc, w_to);  // the second KB lies behind the first in both places
        wsrc += 512;
        w_to = w_to + kLinWBuf >= w_end ? w_to - (kLinWRing - 1) * kLinWBuf : w_to + kLinWBuf;
    };

    f32x4 acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int np = in / 64;  // pairs of k steps
    issue_x();
    issue_w();
    if (np > 1) issue_x();
    issue_w();
    if (np > 1) issue_w();
    // ---- the delta, while the first copies are on their way: the accumulators start with it ----
    const int c0 = strip * 128;
    if (has_strip) {
        const int32_t *st = start + (m0 >> 4) + 4 * rw;
        unsigned todo = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) todo |= (st[i] < st[i + 1] ? 1u : 0u) << i;
        // The first piece of every block: one pass over the rank for all blocks that share its adapter, B^T once
        // for all of them.
        while (todo) {
            const LinPiece &p0 = pieces[st[__builtin_ctz(todo)]];
            const int r8 = p0.r8;
            const uint16_t *bt = arena + p0.b_off + (size_t)c0 * r8 + n * 8;
            unsigned run = 0;
            bool row_ok[4];
            int64_t v_row[4];
            int lo[4], hi[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const LinPiece &pc = pieces[(todo >> i) & 1u ? st[i] : st[__builtin_ctz(todo)]];
                const bool in_run = ((todo >> i) & 1u) && pc.b_off == p0.b_off;
                run |= (in_run ? 1u : 0u) << i;
                lo[i] = pc.place & 15;
                hi[i] = lo[i] + pc.ntok;
                row_ok[i] = in_run && n >= lo[i] && n < hi[i];
                v_row[i] = pc.v_off + (int64_t)(row_ok[i] ? n - lo[i] : 0) * r8;
            }
            todo &= ~run;
            auto steps = [&](auto nk, int j0) __attribute__((always_inline)) {
                constexpr int NK = decltype(nk)::value;
                uint4 w[NK][8], vh[NK][4], vl[NK][4];
#pragma unroll
                for (int s = 0; s < NK; ++s) {
                    const int j = j0 + 32 * s + 8 * kq, jc = j < r8 ? j : 0;  // lanes beyond the rank: v at zero
#pragma unroll
                    for (int b = 0; b < 8; ++b) w[s][b] = ld16(bt + (size_t)(b * (r8 >> 3) + (jc >> 3)) * 128);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        vh[s][i] = ld16(v_hi + v_row[i] + jc);
                        vl[s][i] = ld16(v_lo + v_row[i] + jc);
                    }
                }
#pragma unroll
                for (int s = 0; s < NK; ++s)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if ((run >> i) & 1u) {
                            const bool ok = row_ok[i] && j0 + 32 * s + 8 * kq < r8;
                            const bf16x8 h = as_bf16x8(ok ? vh[s][i] : uint4{0u, 0u, 0u, 0u});
                            const bf16x8 l = as_bf16x8(ok ? vl[s][i] : uint4{0u, 0u, 0u, 0u});
#pragma unroll
                            for (int b = 0; b < 8; ++b) {
                                acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, as_bf16x8(w[s][b]), acc[i][b], 0, 0, 0);
                                acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, as_bf16x8(w[s][b]), acc[i][b], 0, 0, 0);
                            }
                        }
            };
            for (int j = 0; j < r8; j += 32) steps(std::integral_constant<int, 1>{}, j);
            // the zeros above times the adapter's weights are zero only if those are finite, and what an adapter
            // holds must not reach the tokens of its neighbours
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (((run >> i) & 1u) && hi[i] - lo[i] < 16)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool mine = 4 * kq + e >= lo[i] && 4 * kq + e < hi[i];
#pragma unroll
                        for (int b = 0; b < 8; ++b) acc[i][b][e] = mine ? acc[i][b][e] : 0.f;
                    }
        }
        // blocks where adapters meet: the pieces behind the first
#pragma unroll
        for (int i = 0; i < 4; ++i)
            for (int q = st[i] + 1; q < st[i + 1]; ++q) {
                f32x4 dl[8];
                lin_delta<8, 1>(pieces[q], arena, (size_t)c0, 0, n, kq, v_hi, v_lo, dl);
                lin_add(pieces[q], kq, dl, acc[i]);
            }
    }
    // Nothing the compiler knows of is in flight now: without this it would take loads of the delta (some are under
    // conditions) to be outstanding still, and wait for them, and so for the copies, in every pass of the loop.
    stores_done();

    // the end of a phase: every wavefront has come this far
    auto phase_end = [&]() __attribute__((always_inline)) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
    };
    // .. of a phase that read from LDS: what it read is in registers, and the slots may be written
    auto operands_here = [&]() __attribute__((always_inline)) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        phase_end();
    };
    phase_end();
    if (wave >= 4) phase_end();  // the second strip's wavefronts run one phase behind the first's
    int xget = 0, wget = 0;      // ring places of the pair and the k step being computed, in bytes
    const int xlane = (8 * rw + (n >> 3)) * 1024 + (n & 7) * 128;
    bf16x8 xo[4], wo[8];
    auto read = [&](int ks) __attribute__((always_inline)) {
        // row 16 i + n of this wavefront's rows: block 8 rw + 2 i + n / 8, row n mod 8 of it, piece 4 ks + kq
        const int p = ((4 * ks + kq) ^ (n & 7)) * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i) xo[i] = as_bf16x8(*reinterpret_cast<const uint4 *>(xring + xget + xlane + p + 2048 * i));
#pragma unroll
        for (int b = 0; b < 8; ++b) wo[b] = as_bf16x8(*reinterpret_cast<const uint4 *>(wring + wget + w_half + (b * 64 + lane) * 16));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto compute = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int b = 0; b < 8; ++b)
                acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xo[i], wo[b], acc[i][b], 0, 0, 0);
        phase_end();
    };
    for (int j = 0; j < np; ++j) {
        if (j + 2 < np) issue_x();
        read(0);
        // W of step 2 j + 1 has landed: behind it were requested W of step 2 j + 2 and x of pair j + 2
        if (j + 2 < np)
            wait_vm<6>();
        else if (j + 1 < np)
            wait_vm<2>();
        else
            wait_vm<0>();
        operands_here();
        compute();
        wget = wget == (kLinWRing - 1) * kLinWBuf ? 0 : wget + kLinWBuf;
        if (j + 1 < np) issue_w();
        if (j + 2 < np) issue_w();
        read(1);
        // x of pair j + 1 and W of step 2 j + 2 have landed: behind them x of pair j + 2, W of steps 2 j + 3 and 2 j + 4
        if (j + 2 < np)
            wait_vm<8>();
        else if (j + 1 < np)
            wait_vm<2>();
        operands_here();
        compute();
        wget = wget == (kLinWRing - 1) * kLinWBuf ? 0 : wget + kLinWBuf;
        xget = xget == (kLinXRing - 1) * kLinXBuf ? 0 : xget + kLinXBuf;
    }
    if (wave < 4) phase_end();
    if (!has_strip) return;

#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // lane (n, kq) holds tokens 4 kq + e of the block, columns c0 + 8 n .. + 7
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = rows[m0 + 64 * rw + 16 * i + 4 * kq + e];
            if (row >= 0) {
                uint4 o;
                o.x = pack_bf16_rne(acc[i][0][e], acc[i][1][e]);
                o.y = pack_bf16_rne(acc[i][2][e], acc[i][3][e]);
                o.z = pack_bf16_rne(acc[i][4][e], acc[i][5][e]);
                o.w = pack_bf16_rne(acc[i][6][e], acc[i][7][e]);
                st16_stream(y + (int64_t)row * ldy + c0 + 8 * n, o);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same layer for batches of few tokens, where 256 x 256 tiles would leave most of the chip idle (256 tokens
// x 4096 columns: 16 tiles) and the time is that of bringing W in once.  Tiles of 16 RB tokens x 16 CB columns
// (CB sub-blocks of a 128-column strip), one work group each, whose 8 (or 4) wavefronts split k: wavefront w takes
// the 64-wide pieces w, w + 8 (w + 4), ... of k, so that what a work group has in flight lies side by side in memory.
// No operand is shared between wavefronts, so there is no barrier in the loop and no LDS copy of W: a
// wavefront's W operands come straight from memory in operand order (1 KB per load), its x as full cache lines
// (128 bytes of 8 rows per load) that pass through a private LDS region to become operands; D pieces of both
// are in flight per wavefront (registers).  The delta of the tile's adapters is dealt to the wavefronts piece
// by piece and added to their partial sums; these meet in LDS and are added in wavefront order.
// 256 tokens of 62 adapters at 4096 -> 4096: 84 us per layer with 256 x 256 tiles and every group in blocks of its own (138
// without), 31 us here (the shrink launch, 8 us, included; 19 us for x W alone).  What bounds it is what a compute unit draws: 0.5 MB of W and 0.5 MB of x per
// 64 x 64 tile at 60 - 70 GB/s.
// ------------------------------------------------------------------------------------------------
constexpr int kLinSmallWaves = kLinThreads / 64;
// Where there are more tiles than compute units, a tile takes a work group of half as many wavefronts and two work groups share a
// compute unit: what a tile waits for (its rows, the first operands, v and B^T, the sums) then passes beside another's products, and
// up to 512 tiles are one round.  k_linear_small -> k_linear_rounds, us per layer: 576 -> 8192, 208 tokens (512 tiles) 24.9 -> 19.2; 832 -> 4864, 544
// tokens (688) 32.3 -> 27.9; 1728 -> 5120, 630 tokens (800) 49.0 -> 43.3; 8192 -> 2432, 1068 tokens (648) 109 -> 101; 32 x 64 tiles, 7168 -> 640,
// 1428 tokens (456) 57.4 -> 55.2; 16 x 32, 1536 -> 2688, 81 tokens (504) 15.7 -> 14.6, 8192 -> 4224, 28 tokens (264) 34.9 -> 33.8.
constexpr int kLinRoundsWaves = kLinSmallWaves / 2;

template <int RB, int CB, int WAVES>
constexpr int kLinSmallLds = WAVES * 1024 * (2 * RB > RB * CB ? 2 * RB : RB * CB);  // x regions, then partial sums

// Tile `blk` of those of the rows from place m_first on (a multiple of 256), m_tiles row tiles.
template <int RB, int CB, int D, int WAVES>
static __device__ __forceinline__ void linear_small_body(
    int blk, int m_first, int m_tiles, const int32_t *__restrict__ rows, const int32_t *__restrict__ start,
    const LinPiece *__restrict__ pieces, const uint16_t *__restrict__ arena, const uint16_t *__restrict__ wp,
    const uint16_t *__restrict__ x, int64_t ldx, int in, int out, const uint16_t *__restrict__ v_hi,
    const uint16_t *__restrict__ v_lo, uint16_t *__restrict__ y, int64_t ldy, char *lds)
{
    constexpr int NX = 2 * RB;               // x loads of a wavefront per piece of k: 8 rows each
    constexpr int kSlab = 16 * RB * 128;     // bytes of a wavefront's x region: 16 RB rows of 64 k
    constexpr int kTiles = RB * CB;
    static_assert(8 % CB == 0, "a tile lies in one strip");
    // Work group b runs on XCD b mod 8: every XCD an eighth of the tiles, a run of them in the order column tile,
    // row tile, so that W and the adapters' B^T of a column tile enter one or two L2s and the partial lines of a
    // strip's y meet there.  (Whole strips dealt to the XCDs left some of them with nothing or twice the others'
    // share: 1428 tokens at 7168 -> 640, 5 strips, 52.5 -> 48.6 us per
    // layer; 2796 tokens at 1664 -> 640 63.0 -> 47.0; 81 tokens at 1536 -> 2688 19.5 -> 16.6; multiples of 8 level.)
    constexpr int SUB = 8 / CB;
    const int total = m_tiles * (out / (16 * CB)), per_xcd = (total + 7) >> 3;
    const int idx = (blk & 7) * per_xcd + (blk >> 3);
    if ((blk >> 3) >= per_xcd || idx >= total) return;
    const int ct = idx / m_tiles, mt = idx - ct * m_tiles;
    const int strip = ct / SUB, b0 = ct % SUB * CB;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kq = lane >> 4;
    const int m0 = m_first + mt * 16 * RB;

    f32x4 acc[RB][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int np = in >> 6;  // 64-wide pieces of k
    const int mine = wave < np ? (np - 1 - wave) / WAVES + 1 : 0;
    if (mine > 0) {
        // x: lane -> row lane / 8 of the load's 8, 16-byte chunk lane mod 8; in the region chunk c of row r sits in
        // slot c XOR (r mod 8), so that neither the writes nor the operand reads meet in a bank
        char *slab = lds + wave * kSlab;
        const int lr = lane >> 3, lc = lane & 7;
        const uint16_t *xrow[NX];
#pragma unroll
        for (int t = 0; t < NX; ++t) {
            const int row = rows[m0 + 8 * t + lr];
            xrow[t] = x + (int64_t)(row < 0 ? 0 : row) * ldx + 64 * wave + 8 * lc;
        }
        // (wavefront-uniform addresses plus a 32-bit lane offset: no address registers per load)
        const uint16_t *wbase = wp + ((size_t)strip * (in / 32) + 2 * wave) * 4096 + b0 * 512;
        const unsigned lane8 = lane * 8;
        uint4 xq[D][NX], wq[D][2][CB];
        // Loads without branches (around one the compiler would wait for everything in flight): past the last
        // piece all lanes ask for one and the same line, and what comes is not used.
        auto load_x = [&](int i, uint4(&xs)[NX]) __attribute__((always_inline)) {
            const bool ok = i < mine;
#pragma unroll
            for (int t = 0; t < NX; ++t) xs[t] = ld16(ok ? xrow[t] + (size_t)i * (64 * WAVES) : x);
        };
        auto load_w = [&](int i, uint4(&ws)[2][CB]) __attribute__((always_inline)) {
            const bool ok = i < mine;
            const uint16_t *at = ok ? wbase + (size_t)i * (2 * WAVES) * 4096 : wbase;
            const unsigned off = ok ? lane8 : 0u;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int b = 0; b < CB; ++b) ws[ks][b] = ld16(at + ks * 4096 + b * 512 + off);
        };
        auto wave_sync = [&]() __attribute__((always_inline)) {
            // the region is private to this wavefront and LDS operations of a wavefront complete in order
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        };
        auto stage = [&](const uint4(&xs)[NX]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NX; ++t)
                *reinterpret_cast<uint4 *>(slab + (8 * t + lr) * 128 + ((lc ^ lr) << 4)) = xs[t];
        };
        auto compute = [&](const uint4(&ws)[2][CB]) __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                bf16x8 xo[RB];
#pragma unroll
                for (int i = 0; i < RB; ++i)
                    xo[i] = as_bf16x8(*reinterpret_cast<const uint4 *>(slab + (16 * i + n) * 128 +
                                                                       (((4 * ks + kq) ^ (n & 7)) << 4)));
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xo[i], as_bf16x8(ws[ks][b]), acc[i][b], 0, 0, 0);
            }
        };
#pragma unroll
        for (int q = 0; q < D; ++q) {
            // requested in the order of the loop below, which the compiler's count of what is in flight relies on
            load_x(q, xq[q]);
            __builtin_amdgcn_sched_barrier(0);
            load_w(q, wq[q]);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int i0 = 0; i0 < mine; i0 += D) {
#pragma unroll
            for (int q = 0; q < D; ++q) {
                stage(xq[q]);
                load_x(i0 + q + D, xq[q]);
                wave_sync();
                if (i0 + q < mine) compute(wq[q]);
                load_w(i0 + q + D, wq[q]);
                wave_sync();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // ---- the delta: the tile's pieces in turn to the wavefronts ----
    {
        const int q_end = start[(m0 >> 4) + RB];
        for (int q = start[m0 >> 4] + wave; q < q_end; q += WAVES) {
            f32x4 dl[CB];
            lin_delta<CB, 4>(pieces[q], arena, (size_t)strip * 128, b0, n, kq, v_hi, v_lo, dl);
            const int at = (pieces[q].place - m0) >> 4;
#pragma unroll
            for (int i = 0; i < RB; ++i)
                if (i == at) lin_add(pieces[q], kq, dl, acc[i]);
        }
    }

    // ---- the wavefronts' sums, in wavefront order, and the store of y ----
    __syncthreads();  // everyone has left the x regions
    f32x4(*red)[kTiles][64] = reinterpret_cast<f32x4(*)[kTiles][64]>(lds);
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int b = 0; b < CB; ++b) red[wave][i * CB + b][lane] = acc[i][b];
    __syncthreads();
    for (int o = tid; o < RB * 256; o += 64 * WAVES) {
        // row 16 i + 4 kq + e of the tile, columns 8 n + b0 .. + CB - 1 of the strip
        const int i = o >> 8, l = (o >> 2) & 63, e = o & 3;
        const int row = rows[m0 + 16 * i + 4 * (l >> 4) + e];
        if (row < 0) continue;
        float f[CB];
#pragma unroll
        for (int b = 0; b < CB; ++b) f[b] = reinterpret_cast<const float *>(&red[0][i * CB + b][l])[e];
#pragma unroll
        for (int w = 1; w < WAVES; ++w)
#pragma unroll
            for (int b = 0; b < CB; ++b) f[b] += reinterpret_cast<const float *>(&red[w][i * CB + b][l])[e];
        uint32_t *dst = reinterpret_cast<uint32_t *>(y + (int64_t)row * ldy + strip * 128 + 8 * (l & 15) + b0);
#pragma unroll
        for (int b = 0; b < CB; b += 2) dst[b >> 1] = pack_bf16_rne(f[b], f[b + 1]);
    }
}

template <int RB, int CB, int D>
__global__ __launch_bounds__(kLinThreads, 1) void k_linear_small(
    const int32_t *__restrict__ rows, const int32_t *__restrict__ start, const LinPiece *__restrict__ pieces, int m_tiles,
    const uint16_t *__restrict__ arena, const uint16_t *__restrict__ wp, const uint16_t *__restrict__ x, int64_t ldx,
    int in, int out, const uint16_t *__restrict__ v_hi, const uint16_t *__restrict__ v_lo, uint16_t *__restrict__ y,
    int64_t ldy)
{
    __shared__ __attribute__((aligned(16))) char lds[kLinSmallLds<RB, CB, kLinSmallWaves>];
    linear_small_body<RB, CB, D, kLinSmallWaves>(blockIdx.x, 0, m_tiles, rows, start, pieces, arena, wp, x, ldx, in, out, v_hi,
                                                 v_lo, y, ldy, lds);
}

template <int RB, int CB, int D>
__global__ __launch_bounds__(64 * kLinRoundsWaves, 2) void k_linear_rounds(
    const int32_t *__restrict__ rows, const int32_t *__restrict__ start, const LinPiece *__restrict__ pieces, int m_tiles,
    const uint16_t *__restrict__ arena, const uint16_t *__restrict__ wp, const uint16_t *__restrict__ x, int64_t ldx,
    int in, int out, const uint16_t *__restrict__ v_hi, const uint16_t *__restrict__ v_lo, uint16_t *__restrict__ y,
    int64_t ldy)
{
    __shared__ __attribute__((aligned(16))) char lds[kLinSmallLds<RB, CB, kLinRoundsWaves>];
    linear_small_body<RB, CB, D, kLinRoundsWaves>(blockIdx.x, 0, m_tiles, rows, start, pieces, arena, wp, x, ldx, in, out, v_hi,
                                                  v_lo, y, ldy, lds);
}

// The first n_big work groups take 256 x 256 tiles of the first m_big row tiles, the others 64 x 64 tiles of the
// rows behind them, which fill the compute units that the last round of large tiles leaves idle.
__global__ __launch_bounds__(kLinThreads, 1) void k_linear_lora(
    const int32_t *__restrict__ rows, const int32_t *__restrict__ start, const LinPiece *__restrict__ pieces, int n_big,
    int m_big, int n_tiles, int m_small, const uint16_t *__restrict__ arena, const uint16_t *__restrict__ wp,
    const uint16_t *__restrict__ x, int64_t ldx, int in, int out, const uint16_t *__restrict__ v_hi,
    const uint16_t *__restrict__ v_lo, uint16_t *__restrict__ y, int64_t ldy)
{
    __shared__ __attribute__((aligned(16))) char lds[kLinLds];
    static_assert(kLinSmallLds<4, 4, kLinSmallWaves> <= kLinLds, "a small tile fits the LDS of a large one");
    if ((int)blockIdx.x >= n_big) {
        linear_small_body<4, 4, 2, kLinSmallWaves>((int)blockIdx.x - n_big, m_big * kLinTileM, m_small, rows, start, pieces, arena,
                                                   wp, x, ldx, in, out, v_hi, v_lo, y, ldy, lds);
        return;
    }
    // Work group b runs on XCD b mod 8.  Each XCD takes a run of row tiles, and the 32 work groups it runs
    // at a time (one per compute unit) are 8 row tiles x 4 column tiles that walk k together: every
    // chunk of x and of W that one of them brings into the XCD's L2 serves four or eight of them.
    const int xcd = blockIdx.x & 7, jloc = blockIdx.x >> 3;
    const int ngroups_n = (n_tiles + 3) >> 2;
    const int grp = jloc >> 5, within = jloc & 31;
    const int mt_loc = (grp / ngroups_n) * 8 + (within >> 2);
    const int nt = (grp % ngroups_n) * 4 + (within & 3);
    const int share = m_big >> 3, extra = m_big & 7;  // the first `extra` XCDs take one row tile more
    if (mt_loc >= share + (xcd < extra ? 1 : 0) || nt >= n_tiles) return;
    linear_big_body(xcd * share + min(xcd, extra) + mt_loc, nt, rows, start, pieces, arena, wp, x, ldx, in, out, v_hi, v_lo,
                    y, ldy, lds);
}

template <int RB, int CB, int D>
static void launch_linear_small(const LinSmallTiles &t, const int32_t *rows, const int32_t *start, const LinPiece *pieces, int n_places,
                                const uint16_t *arena, const uint16_t *w_packed, const uint16_t *x, int64_t ldx, int in,
                                int out, const uint16_t *v_hi, const uint16_t *v_lo, uint16_t *y, int64_t ldy,
                                hipStream_t stream)
{
    const int m_tiles = (n_places + 16 * RB - 1) / (16 * RB);
    const int grid = t.grid();
    if (t.pairs())
        hipLaunchKernelGGL((k_linear_rounds<RB, CB, D>), dim3((unsigned)grid), dim3(64 * kLinRoundsWaves), 0, stream, rows, start,
                           pieces, m_tiles, arena, w_packed, x, ldx, in, out, v_hi, v_lo, y, ldy);
    else
        hipLaunchKernelGGL((k_linear_small<RB, CB, D>), dim3((unsigned)grid), dim3(kLinThreads), 0, stream, rows, start,
                           pieces, m_tiles, arena, w_packed, x, ldx, in, out, v_hi, v_lo, y, ldy);
}

// W^T [out][in] row-major -> operand order (see launch_pack_weight).  One thread per destination element.
__global__ __launch_bounds__(256) void k_pack_w(const uint16_t *__restrict__ wt, int in, int out,
                                                uint16_t *__restrict__ dst)
{
    const int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (d >= (int64_t)in * out) return;
    const int ksteps = in / 32;
    const int e = (int)(d & 7);
    const int slot = (int)((d >> 3) & 63);
    const int b = (int)((d >> 9) & 7);
    const int64_t rest = d >> 12;  // strip * ksteps + kstep
    const int kstep = (int)(rest % ksteps);
    const int strip = (int)(rest / ksteps);
    const int col = 128 * strip + 8 * (slot & 15) + b;
    const int k = 32 * kstep + 8 * (slot >> 4) + e;
    dst[d] = wt[(int64_t)col * in + k];
}

// ------------------------------------------------------------------------------------------------
// Writes an adapter's packed form (see the top of this file), both matrices in one launch: the first n_a
// work groups (of one wavefront) take A, the others B.  An adapter is at most a few megabytes and a launch
// lasts as long as its shortest chain of trips to memory, so what counts is that there is one launch and not
// two, and that every load is requested at once.  A thread reads an 8 x 8 block with eight 16-byte loads of
// consecutive columns, turns it in registers and writes eight 16-byte pieces: for A (8 k of 8 rank rows)
// they are 128 consecutive bytes of a row block, for B (8 rank rows of 8 columns) one piece of each of the
// strip's eight sub-blocks, 16 threads side by side.  Where a 16-byte load is not possible (A's rows start
// at multiples of 2 r bytes: r not a multiple of 8; or a source that is not 16-byte aligned) a thread
// gathers one 16-byte piece with eight 2-byte loads.  16 adapters of ranks 8 .. 128 at 4096 -> 4096, one call
// each: 109 us with a launch per matrix and a thread per element, 68 us this way.
// ------------------------------------------------------------------------------------------------
constexpr int kPackThreads = 64;

// words of row i of the transpose of the 8 x 8 block of 16-bit values whose rows are `in`
static __device__ __forceinline__ uint4 block_column(const uint4 (&in)[8], int i)
{
    auto word = [&](const uint4 &v) __attribute__((always_inline)) {
        return (i >> 1) == 0 ? v.x : (i >> 1) == 1 ? v.y : (i >> 1) == 2 ? v.z : v.w;
    };
    auto pair = [&](const uint4 &lo, const uint4 &hi) __attribute__((always_inline)) {
        return (i & 1) ? (word(lo) >> 16) | (word(hi) & 0xFFFF0000u) : (word(lo) & 0xFFFFu) | (word(hi) << 16);
    };
    return uint4{pair(in[0], in[1]), pair(in[2], in[3]), pair(in[4], in[5]), pair(in[6], in[7])};
}

__global__ __launch_bounds__(kPackThreads) void k_pack_adapter(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B,
                                                               int in, int out, int r, int r8, int vec_a, int vec_b,
                                                               unsigned n_a, uint16_t *__restrict__ dst_a,
                                                               uint16_t *__restrict__ dst_b)
{
    const uint4 zero = {0u, 0u, 0u, 0u};
    const int octets = r8 >> 3;
    if (blockIdx.x < n_a) {
        const unsigned t = blockIdx.x * kPackThreads + threadIdx.x;
        if (vec_a) {
            // octet jo of the rank rows (r = r8 here), octet ko of k
            const int jo = (int)(t % (unsigned)octets), ko = (int)(t / (unsigned)octets);
            if (ko >= in >> 3) return;
            uint4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = ld16_stream(A + (int64_t)(8 * ko + i) * r + 8 * jo);
            const int jb = jo >> 1, h = min(16, r8 - 16 * jb);
            uint16_t *d = dst_a + (int64_t)16 * jb * in + (int64_t)(ko >> 2) * 32 * h + ((ko & 3) * h + 8 * (jo & 1)) * 8;
#pragma unroll
            for (int i = 0; i < 8; ++i) *reinterpret_cast<uint4 *>(d + 8 * i) = block_column(v, i);
        } else {
            // one 16-byte piece: 8 k of rank row j
            const int j = (int)(t % (unsigned)r8), ko = (int)(t / (unsigned)r8);
            if (ko >= in >> 3) return;
            uint32_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = A[(int64_t)(8 * ko + i) * r + min(j, r - 1)];
            const int jb = j >> 4, h = min(16, r8 - 16 * jb);
            const uint4 p = {e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
            *reinterpret_cast<uint4 *>(dst_a + (int64_t)16 * jb * in + (int64_t)(ko >> 2) * 32 * h +
                                       ((ko & 3) * h + (j & 15)) * 8) = j < r ? p : zero;
        }
        return;
    }
    const unsigned t = (blockIdx.x - n_a) * kPackThreads + threadIdx.x;
    if (vec_b) {
        // columns 8 co .. + 7 of rank rows 8 kp .. + 7
        const int co = (int)(t % (unsigned)(out >> 3)), kp = (int)(t / (unsigned)(out >> 3));
        if (kp >= octets) return;
        uint4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = ld16_stream(B + (int64_t)min(8 * kp + i, r - 1) * out + 8 * co);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (8 * kp + i >= r) v[i] = zero;
        uint16_t *d = dst_b + (int64_t)128 * (co >> 4) * r8 + (kp * 16 + (co & 15)) * 8;
#pragma unroll
        for (int b = 0; b < 8; ++b) *reinterpret_cast<uint4 *>(d + (int64_t)b * octets * 128) = block_column(v, b);
    } else {
        // one 16-byte piece: 8 rank rows of column c
        const int c = (int)(t % (unsigned)out), kp = (int)(t / (unsigned)out);
        if (kp >= octets) return;
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = B[(int64_t)min(8 * kp + i, r - 1) * out + c];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (8 * kp + i >= r) e[i] = 0u;
        *reinterpret_cast<uint4 *>(dst_b + (int64_t)128 * (c >> 7) * r8 + (((c & 7) * octets + kp) * 16 + ((c & 127) >> 3)) * 8) =
            uint4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
}

// ------------------------------------------------------------------------------------------------
// Pinned host memory to the device: n_a pieces of 16 bytes from `a`, then those of `b`, one a thread.  A kernel between kernels of one
// queue instead of the copy engine, which the queue waits for and which waits for the queue, about 10 us each way round: a batch
// planned anew in front of every launch of it, us per step: 256 tokens through 32 layers 494 -> 480, through eight layers of seven
// projections, four objects, 1086 -> 1053, 31 tokens of 92 adapters through one projection, 4928 -> 2048, 33 -> 24 (the rest is
// the host's).  Where the host plans for longer than the device works, a launch costs it about 0.7 us more than a copy, and of five arguments
// 0.5 us more than of one struct: four objects of 500 tokens, copies / five arguments / a struct 228.6 / 232.0 / 230.0, of 256 tokens
// 152.5 / 157.9 / 155.7, one of 500 tokens 34.9 / 35.7 / 35.4.
// The loads have system scope: the host's memory serves them, whatever a cache holds of what was read there before.
// They are 16 bytes wide: with 8 (atomic) loads the link gives half of its 47 GB/s.
// ------------------------------------------------------------------------------------------------
struct CopyIn {
    const uint4 *a, *b;
    uint4 *dst;
    unsigned n_a, n;  // pieces of a, and in all
};
__global__ __launch_bounds__(256) void k_copy_in(CopyIn c)
{
    const unsigned at = blockIdx.x * 256 + threadIdx.x;
    if (at >= c.n) return;
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    constexpr int kSystem = 17;  // sc0 sc1
    u32x4 v;
    if (at < c.n_a)
        v = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(c.a), 0, (int)(16u * c.n_a), 0x00020000),
                                                  (int)(16u * at), 0, kSystem);
    else
        v = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(c.b), 0, (int)(16u * (c.n - c.n_a)), 0x00020000),
                                                  (int)(16u * (at - c.n_a)), 0, kSystem);
    c.dst[at] = uint4{v.x, v.y, v.z, v.w};
}

// ------------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------------
static Sync make_sync(const SyncArgs *a, int wait, int scale_v = 0)
{
    Sync sy;
    if (!a) {
        sy = Sync{nullptr, nullptr, nullptr, nullptr, nullptr, 0u, 0u, 0, scale_v, nullptr, 0, 0};
    } else {
        sy = Sync{a->counters, a->ready, a->timeout_flag, a->v_hi, a->v_lo, a->epoch, a->spin_limit, wait, scale_v,
                  a->parts, a->n_slices, a->slice_stride};
    }
    return sy;
}

hipError_t launch_copy_in(const void *a, size_t a_bytes, const void *b, size_t b_bytes, void *dev, hipStream_t stream)
{
    const size_t bytes = a_bytes + b_bytes;
    if (!bytes) return hipSuccess;
    if (a_bytes % 16 || b_bytes % 16 || bytes >= (size_t)1 << 31 || ((uintptr_t)a | (uintptr_t)b | (uintptr_t)dev) % 16)
        return hipErrorInvalidValue;
    const unsigned n = (unsigned)(bytes / 16);
    const CopyIn c = {(const uint4 *)a, (const uint4 *)b, (uint4 *)dev, (unsigned)(a_bytes / 16), n};
    hipLaunchKernelGGL(k_copy_in, dim3((n + 255) / 256), dim3(256), 0, stream, c);
    return hipGetLastError();
}

hipError_t launch_shrink(const LaunchCtx &c, const uint16_t *x, int64_t ldx, int k_slice_len, float *v_out,
                         int n_slices, int64_t slice_stride, const SyncArgs *sync, hipStream_t stream)
{
    if (c.n_units <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_shrink, dim3(c.n_units), dim3(kThreads), 0, stream, c.units, c.arena, x, ldx,
                       c.in_features, k_slice_len, v_out, n_slices, slice_stride, make_sync(sync, 0, c.scale_v));
    return hipGetLastError();
}

hipError_t launch_shrink_wide(const LaunchCtx &c, bool more_than_one_round, const uint16_t *x, int64_t ldx,
                              int k_slice_len, int n_slices, float *v_f32, uint16_t *v_hi, uint16_t *v_lo,
                              hipStream_t stream)
{
    if (c.n_units <= 0) return hipSuccess;
    if (n_slices < 1 || n_slices > kMaxSlices) return hipErrorInvalidValue;
    if (more_than_one_round)
        hipLaunchKernelGGL(k_shrink_wide<kWideHalfWaves>, dim3(c.n_units), dim3(64 * kWideHalfWaves), 0, stream,
                           c.units, c.arena, x, ldx, c.in_features, k_slice_len, n_slices, v_f32, v_hi, v_lo, c.scale_v);
    else
        hipLaunchKernelGGL(k_shrink_wide<kWideWaves>, dim3(c.n_units), dim3(kWideThreads), 0, stream, c.units,
                           c.arena, x, ldx, c.in_features, k_slice_len, n_slices, v_f32, v_hi, v_lo, c.scale_v);
    return hipGetLastError();
}

// The places of a launch of 64-token expand units, section by section.
struct BigGrid {
    int n_first = 0, subs = 1;
    int64_t places = 0;
    BigMore more = {};
    explicit BigGrid(const LaunchCtx &c)
    {
        int unit = 0;
        for (int i = 0; i < c.n_sections; ++i) {
            const int per_unit = (c.sections[i].cols + kBigCols - 1) / kBigCols;
            if (i == 0) {
                n_first = c.sections[0].n_units;
                subs = per_unit;
            } else {
                more.first_place[more.n] = (int)std::min<int64_t>(places, 0x7FFFFFFF);
                more.first_unit[more.n] = unit;
                more.subs[more.n] = per_unit;
                more.first_unit[++more.n] = unit + c.sections[i].n_units;
            }
            unit += c.sections[i].n_units;
            places += (int64_t)(c.sections[i].n_units + 7) / 8 * 8 * per_unit;
        }
    }
};

hipError_t launch_expand(const LaunchCtx &c, bool big, const float *v_in, uint16_t *y, int64_t ldy, const SyncArgs *sync,
                         hipStream_t stream)
{
    if (c.n_units <= 0) return hipSuccess;
    if (!sync && !v_in) return hipErrorInvalidValue;
    const Sync sy = make_sync(sync, 0);
    const dim3 g(c.n_units), b(kThreads);
    if (big && !sync && expand_walks(c)) {
        const int most = c.sections[0].cols / kStrip, strips = walk_strips(c);
        const int64_t grid = (int64_t)c.n_units * ((most + strips - 1) / strips);
        if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_expand_walk, dim3((unsigned)grid), b, 0, stream, c.units, c.n_units, strips, c.perm, c.arena, v_in, y, ldy);
    } else if (big) {
        if (c.n_sections > kMaxBigSections) return hipErrorInvalidValue;
        const BigGrid bg(c);
        if (bg.places > 0x7FFFFFFF) return hipErrorInvalidValue;
        const dim3 gb((unsigned)bg.places);
        const unsigned more_lds = big_spread(c) ? kBigSpread : 0;
        if (sync)
            hipLaunchKernelGGL(k_expand_big<false>, gb, b, more_lds, stream, c.units, bg.n_first, bg.subs, c.perm, c.arena, v_in, y, ldy,
                               sy, bg.more);
        else
            hipLaunchKernelGGL(k_expand_big<true>, gb, b, more_lds, stream, c.units, bg.n_first, bg.subs, c.perm, c.arena, v_in, y, ldy,
                               sy, bg.more);
    } else if (sync && sync->parts)
        hipLaunchKernelGGL(k_expand_parts, g, b, 0, stream, c.units, c.arena, y, ldy, sy);
    else if (sync)
        hipLaunchKernelGGL((k_expand<false, false>), g, b, 0, stream, c.units, c.perm, c.arena, v_in, y, ldy, sy);
    else
        hipLaunchKernelGGL((k_expand<false, true>), g, b, 0, stream, c.units, c.perm, c.arena, v_in, y, ldy, sy);
    return hipGetLastError();
}

hipError_t launch_apply_fused(const LaunchCtx &cs, const LaunchCtx &ce, const uint16_t *x, int64_t ldx,
                              int k_slice_len, float *parts, int n_slices, int64_t slice_stride, uint16_t *y,
                              int64_t ldy, const SyncArgs *sync, hipStream_t stream)
{
    const int total = cs.n_units + ce.n_units;
    if (total <= 0) return hipSuccess;
    if (!sync || !sync->parts) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_apply_fused, dim3(total), dim3(kThreads), 0, stream, cs.units, cs.n_units, ce.units,
                       cs.arena, x, ldx, cs.in_features, k_slice_len, parts, n_slices, slice_stride, y, ldy,
                       make_sync(sync, 1));
    return hipGetLastError();
}

hipError_t launch_decode_fused(const LaunchCtx &cs, const LaunchCtx &ce, int grid, const uint16_t *x, int64_t ldx,
                               int k_slice_len, int n_slices, uint16_t *y, int64_t ldy, unsigned xcc_map,
                               const SyncArgs *sync, hipStream_t stream)
{
    if (cs.n_units <= 0 && ce.n_units <= 0) return hipSuccess;
    if (!sync || grid < 1 || grid > kDecodeMaxGrid || n_slices < 1 || n_slices > kMaxSlices || cs.n_units > grid || ce.n_units > 4 * grid ||
        cs.n_units < 1 || ce.n_units < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_decode_fused, dim3(grid), dim3(kWideThreads), 0, stream, cs.units, cs.n_units, ce.units,
                       ce.n_units, cs.arena, x, ldx, cs.in_features, k_slice_len, n_slices, y, ldy, xcc_map,
                       make_sync(sync, 1));
    return hipGetLastError();
}

// Where the work groups of a launch run: host_out[b] = XCD of work group b of an n-work-group launch (n <=
// kProbeSlots).  Synchronous; its buffer is a device array of this file's own.
constexpr int kProbeSlots = 1024;
static __device__ unsigned xcc_probe_buf[kProbeSlots];

hipError_t probe_xcc(unsigned *host_out, int n_work_groups, hipStream_t stream)
{
    if (n_work_groups < 1 || n_work_groups > kProbeSlots) return hipErrorInvalidValue;
    void *buf = nullptr;
    hipError_t e = hipGetSymbolAddress(&buf, HIP_SYMBOL(xcc_probe_buf));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_probe_xcc, dim3(n_work_groups), dim3(64), 0, stream, (unsigned *)buf);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(stream)) != hipSuccess) return e;
    return hipMemcpy(host_out, buf, sizeof(unsigned) * (size_t)n_work_groups, hipMemcpyDeviceToHost);
}

hipError_t launch_shrink_prefill(const LaunchCtx &c, int n_hi, const uint16_t *x, int64_t ldx, uint16_t *v_hi,
                                 uint16_t *v_lo, float *v_f32, int n_slices, int64_t slice_stride, float *parts,
                                 const SyncArgs *sync, hipStream_t stream)
{
    if (c.n_units <= 0) return hipSuccess;
    if (n_hi < 0 || n_hi > c.n_units) return hipErrorInvalidValue;
    const Sync sy = make_sync(sync, 0, c.scale_v);
    if (shrink_in_halves(c))
        hipLaunchKernelGGL(k_shrink_halves, dim3((c.n_units + 7) / 8 * 16), dim3(kThreads), 0, stream, c.units, c.perm, c.arena, x, ldx,
                           c.in_features, v_hi, v_lo, v_f32, n_slices, slice_stride, parts, c.n_units, sy);
    else if (n_hi > 0)
        hipLaunchKernelGGL(k_shrink_prefill_any, dim3(c.n_units), dim3(kThreads), 0, stream, c.units, c.perm, c.arena,
                           x, ldx, c.in_features, v_hi, v_lo, v_f32, n_slices, slice_stride, parts, sy);
    else
        hipLaunchKernelGGL(k_shrink_prefill, dim3(c.n_units), dim3(kThreads), 0, stream, c.units, c.perm, c.arena, x,
                           ldx, c.in_features, v_hi, v_lo, v_f32, n_slices, slice_stride, parts, sy);
    return hipGetLastError();
}

hipError_t launch_shrink_mixed(const LaunchCtx &heavy, int n_hi, const LaunchCtx &c, const uint16_t *x, int64_t ldx,
                               int k_slice_len, float *parts, int n_slices, int64_t slice_stride,
                               const SyncArgs *sync, hipStream_t stream)
{
    const int total = heavy.n_units + c.n_units;
    if (total <= 0) return hipSuccess;
    if (!sync || n_hi < 0 || n_hi > heavy.n_units) return hipErrorInvalidValue;
    const Sync sy = make_sync(sync, 0, c.scale_v);
    if (n_hi > 0)
        hipLaunchKernelGGL(k_shrink_mixed<true>, dim3(total), dim3(kThreads), 0, stream, heavy.units, heavy.n_units,
                           c.units, c.perm, c.arena, x, ldx, c.in_features, k_slice_len, parts, n_slices,
                           slice_stride, sy);
    else
        hipLaunchKernelGGL(k_shrink_mixed<false>, dim3(total), dim3(kThreads), 0, stream, heavy.units, heavy.n_units,
                           c.units, c.perm, c.arena, x, ldx, c.in_features, k_slice_len, parts, n_slices,
                           slice_stride, sy);
    return hipGetLastError();
}

hipError_t launch_expand_mixed(const LaunchCtx &big, const LaunchCtx &c, uint16_t *y, int64_t ldy, const SyncArgs *sync,
                               hipStream_t stream)
{
    if (big.n_sections > kMaxBigSections) return hipErrorInvalidValue;
    const BigGrid bg(big);
    const int64_t total = bg.places + c.n_units;
    if (total <= 0) return hipSuccess;
    if (!sync || total > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (sync->parts)
        hipLaunchKernelGGL(k_expand_mixed<kSlicesByExpand>, dim3((unsigned)total), dim3(kThreads), 0, stream, big.units, bg.n_first,
                           bg.subs, (int)bg.places, c.units, c.arena, c.perm, y, ldy, make_sync(sync, 0), bg.more);
    else
        hipLaunchKernelGGL(k_expand_mixed<kSlicesByShrink>, dim3((unsigned)total), dim3(kThreads), 0, stream, big.units, bg.n_first,
                           bg.subs, (int)bg.places, c.units, c.arena, c.perm, y, ldy, make_sync(sync, 0), bg.more);
    return hipGetLastError();
}

hipError_t launch_linear_lora(const int32_t *rows, const LinBlock *blocks, int n_places, const uint16_t *arena,
                              const uint16_t *w_packed, const uint16_t *x, int64_t ldx, int in, int out,
                              const uint16_t *v_hi, const uint16_t *v_lo, uint16_t *y, int64_t ldy,
                              hipStream_t stream)
{
    if (n_places <= 0) return hipSuccess;
    if (in % 64 || out % 128 || out <= 0 || in < 64) return hipErrorInvalidValue;
    const int n_tiles = (out + kLinTileN - 1) / kLinTileN;
    const int32_t *start = blocks->start;
    const LinPiece *pieces = blocks->pieces;
    const int m_big = std::min(blocks->big_tiles, (n_places + kLinTileM - 1) / kLinTileM);
    if (m_big < 0) return hipErrorInvalidValue;
    if (m_big == 0) {
        const LinSmallTiles t = linear_small_tiles(n_places, out);
        auto go = [&](auto rb, auto cb, auto d) {
            launch_linear_small<decltype(rb)::value, decltype(cb)::value, decltype(d)::value>(
                t, rows, start, pieces, n_places, arena, w_packed, x, ldx, in, out, v_hi, v_lo, y, ldy, stream);
        };
        using std::integral_constant;
        if (t.rb == 4)
            go(integral_constant<int, 4>{}, integral_constant<int, 4>{}, integral_constant<int, 2>{});
        else if (t.cb == 4)
            go(integral_constant<int, 2>{}, integral_constant<int, 4>{}, integral_constant<int, 2>{});
        else if (t.rb == 2)
            go(integral_constant<int, 2>{}, integral_constant<int, 2>{}, integral_constant<int, 3>{});
        else
            go(integral_constant<int, 1>{}, integral_constant<int, 2>{}, integral_constant<int, 4>{});
        return hipGetLastError();
    }
    const int m_small = n_places > m_big * kLinTileM ? (n_places - m_big * kLinTileM + 63) / 64 : 0;
    // per XCD: groups of 32 work groups = 8 row tiles x 4 column tiles (see the kernel)
    const int64_t n_big = (int64_t)8 * 32 * (((m_big + 7) / 8 + 7) / 8) * ((n_tiles + 3) / 4);
    const int64_t grid = n_big + (int64_t)8 * (((int64_t)m_small * (out / 64) + 7) / 8);
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_linear_lora, dim3((unsigned)grid), dim3(kLinThreads), 0, stream, rows, start, pieces, (int)n_big, m_big,
                       n_tiles, m_small, arena, w_packed, x, ldx, in, out, v_hi, v_lo, y, ldy);
    return hipGetLastError();
}

hipError_t launch_pack_weight(const uint16_t *wt, int in, int out, uint16_t *dst, hipStream_t stream)
{
    const int64_t n = (int64_t)in * out;
    if (n <= 0 || in % 32 || out % 128) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pack_w, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, wt, in, out, dst);
    return hipGetLastError();
}

hipError_t launch_reduce_slices(const float *parts, int n_slices, int64_t slice_stride, float *v, int64_t n,
                                hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_reduce_slices, dim3((unsigned)blocks), dim3(256), 0, stream, parts, n_slices,
                       slice_stride, v, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Workspace of the entry point that allocates nothing (lora_apply_static): each GPU the library runs
// on holds one copy of this array, at its own address, until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; every use of its memory goes through the
// address looked up here, once per device, with that device current.
// ------------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void **ptr)
{
    static std::atomic<void *> addr[kMaxDevices];
    *ptr = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *p = addr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev].store(p, std::memory_order_release);  // two threads racing here store the same address
    }
    *ptr = p;
    return hipSuccess;
}

hipError_t launch_pack_adapter(const uint16_t *A, const uint16_t *B, int in, int out, int r, int r8,
                               uint16_t *dst_a, uint16_t *dst_b, hipStream_t stream)
{
    // threads: one per 8 x 8 block, or (no 16-byte loads) one per 16-byte piece
    const int vec_a = r % 8 == 0 && (uintptr_t)A % 16 == 0, vec_b = (uintptr_t)B % 16 == 0;
    const int64_t ta = (int64_t)(in / 8) * (vec_a ? r8 / 8 : r8), tb = (int64_t)(r8 / 8) * (vec_b ? out / 8 : out);
    const int64_t ga = (ta + kPackThreads - 1) / kPackThreads, gb = (tb + kPackThreads - 1) / kPackThreads;
    if (ga + gb > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pack_adapter, dim3((unsigned)(ga + gb)), dim3(kPackThreads), 0, stream, A, B, in, out, r, r8, vec_a,
                       vec_b, (unsigned)ga, dst_a, dst_b);
    return hipGetLastError();
}

}  // namespace lora

#ifdef LORA_WG_CLOCKS
// Measurement build only: device buffer of 8 clock values per work group for the next launches (NULL = off).
extern "C" int lora_debug_clock_buffer(unsigned long long *dev_buf, unsigned n_work_groups)
{
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(lora::g_clock_buf), &dev_buf, sizeof dev_buf);
    if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(lora::g_clock_slots), &n_work_groups, sizeof n_work_groups);
    return (int)e;
}
#endif
