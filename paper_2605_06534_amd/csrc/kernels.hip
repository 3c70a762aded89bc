// HIP kernels for gfx950 (wave64): diff + mask + count + scan + shard-aware bucket write
// (Sec. 4.2 "Sparsity-aware Weight Transfer", App. F D2S), scatter-apply (App. F S2D), the dense
// shard copy (Sec. 4.2 "Shard-aware Weight Transfer"), transport objects (Sec. 4.2 "Asynchronous
// Weight Transfer") and bandwidth probes.
//
// Everything here is bound by HBM traffic; there is no contraction, so no MFMA.  The encode
// kernel reads each weight once with 128-bit loads and writes only the changed entries.
#include <hip/hip_runtime.h>

#include <mutex>

#include "rose_internal.h"

namespace rose {

// ---------------------------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------------------------

typedef unsigned long long u64;

__device__ __forceinline__ uint32_t rne_bf16(uint32_t u) {
    // fp32 pattern -> bf16 pattern, nearest, ties to even: add half an ulp of the kept part
    // minus one, plus the lowest kept bit, then truncate.  NaN keeps its top bits, quieted.
    uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? ((u >> 16) | 0x0040u) : r;
}

// Two at a time with the conversion instruction: the same patterns as rne_bf16 for every one of the 2^32 inputs in
// either half, NaNs and subnormals included.  (In integer steps this was 190 of the 780 vector instructions that the fp32
// ticket kernel spends on a tile and wave: two 32B-style layers, 1.6 %: 2.69 ms, 2.64 this way; with arithmetic payloads
// 2.98 and 2.79; 2 M weights 8.2 and 7.4 us.)
__device__ __forceinline__ uint32_t pack_rne(uint32_t lo, uint32_t hi) {
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(__uint_as_float(lo)), "v"(__uint_as_float(hi)));
    return r;
}

// 8-bit mask of the 16-bit lanes of x that are non-zero (bit e = element e, little endian).
// A packed 16-bit min with 1 turns the two halves of a dword into 0 / 1 (bits 0 and 16) in one
// instruction; the four dwords are merged first (even elements in bits 0,2,4,6, odd ones in
// 16,18,20,22) and the odd ones folded down at the end.
__device__ __forceinline__ uint32_t nz16_pair(uint32_t x) {
    uint32_t b;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(b) : "v"(x), "v"(0x00010001u));
    return b;
}
__device__ __forceinline__ uint32_t nz16_mask(uint4 x) {
    const uint32_t t = nz16_pair(x.x) | (nz16_pair(x.y) << 2) | (nz16_pair(x.z) << 4) | (nz16_pair(x.w) << 6);
    return (t | (t >> 15)) & 0xFFu;
}

// element e (0..7) of a vector of eight 16-bit patterns
__device__ __forceinline__ uint32_t pick16(uint4 v, uint32_t e) {
    uint32_t a = (e & 4u) ? ((e & 2u) ? v.w : v.z) : ((e & 2u) ? v.y : v.x);
    return (e & 1u) ? (a >> 16) : (a & 0xFFFFu);
}

// ---------------------------------------------------------------------------------------------
// Arithmetic payload (Sec. 4.2 writes the update as W_t = W_{t-1} + dW_t).  An entry carries
// d = bf16(new - old) if d is a number and bf16(old + d) is exactly the new pattern; otherwise it
// carries the new pattern and bit 31 of its index says so (escape).  Sums and differences of two
// bf16 values are formed in fp32 and rounded to nearest even: the fp32 result is exact unless the
// operands lie more than 16 binades apart, and then it sits so close to the larger operand that
// the second rounding cannot cross a tie, so the result is the correctly rounded bf16 one.
// Subnormals are kept (the kernels are built with IEEE denormal handling for fp32).
// ---------------------------------------------------------------------------------------------
#ifndef ROSE_ARITH_HWCVT
#define ROSE_ARITH_HWCVT 1     // 1: round with the packed fp32 -> bf16 conversion instruction (checked against
                               // the integer rounding below and the CPU reference on all 2^32 pattern pairs; where
                               // payloads are formed of every element, 6.7 G at 5 %, 5.60 ms instead of 6.14 ms)
#endif
// the two fp32 values rounded to bf16 (nearest even), packed: lo in bits 0..15, hi in 16..31.
// A NaN stays a NaN (its low 16 bits are zero here, so the rounding add cannot carry out of them).
__device__ __forceinline__ uint32_t pack_bf16_pair(float lo, float hi) {
#if ROSE_ARITH_HWCVT
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
    return r;
#else
    const uint32_t a = __float_as_uint(lo), b = __float_as_uint(hi);
    const uint32_t ra = a + 0x7FFFu + ((a >> 16) & 1u), rb = b + 0x7FFFu + ((b >> 16) & 1u);
    return (ra >> 16) | (rb & 0xFFFF0000u);
#endif
}
// payloads of the two elements of a dword; *b01 gets 1 in bit 0 / bit 16 for an escaped element
__device__ __forceinline__ uint32_t arith_pair(uint32_t o, uint32_t n, uint32_t *b01) {
    const float ol = __uint_as_float(o << 16), oh = __uint_as_float(o & 0xFFFF0000u);
    const float nl = __uint_as_float(n << 16), nh = __uint_as_float(n & 0xFFFF0000u);
    const uint32_t d = pack_bf16_pair(nl - ol, nh - oh);
    const uint32_t back = pack_bf16_pair(ol + __uint_as_float(d << 16), oh + __uint_as_float(d & 0xFFFF0000u));
    // a half of (mx ^ 0x7F80...) is non-zero where d is a NaN: magnitude above the pattern of infinity
    uint32_t mx;
    asm("v_pk_max_u16 %0, %1, %2" : "=v"(mx) : "v"(d & 0x7FFF7FFFu), "v"(0x7F807F80u));
    const uint32_t bad = (back ^ n) | (mx ^ 0x7F807F80u);
    const uint32_t b = nz16_pair(bad);
    *b01 = b;
    const uint32_t take_new = b * 0xFFFFu;              // 0xFFFF in the halves that escape
    return (n & take_new) | (d & ~take_new);
}
// the same for one element (patterns in the low halves)
__device__ __forceinline__ uint32_t arith_one(uint32_t o, uint32_t n, bool *escapes) {
    const float was = __uint_as_float(o << 16);
    const uint32_t d = pack_bf16_pair(__uint_as_float(n << 16) - was, 0.0f);
    const uint32_t back = pack_bf16_pair(was + __uint_as_float(d << 16), 0.0f);
    *escapes = back != n || (d & 0x7FFFu) > 0x7F80u;
    return *escapes ? n : d;
}
// the same for a vector of eight; esc8 bit e = element e escapes
__device__ __forceinline__ uint4 arith_vec(uint4 o, uint4 n, uint32_t *esc8) {
    uint32_t b0, b1, b2, b3;
    uint4 p;
    p.x = arith_pair(o.x, n.x, &b0);
    p.y = arith_pair(o.y, n.y, &b1);
    p.z = arith_pair(o.z, n.z, &b2);
    p.w = arith_pair(o.w, n.w, &b3);
    const uint32_t t = b0 | (b1 << 2) | (b2 << 4) | (b3 << 6);
    *esc8 = (t | (t >> 15)) & 0xFFu;
    return p;
}

// inclusive prefix sum over the 64 lanes of a wave with DPP moves (no LDS traffic): shifts by
// 1, 2, 4, 8 inside each row of 16 lanes, then the row totals are broadcast into the following
// rows (lane 15 of a row into the next row, lane 31 into the upper half).  A lane without a
// source keeps the 0 passed as the old value.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15 -> rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31 -> rows 2, 3
    return x;
}

// the OR of x over each group of four lanes
__device__ __forceinline__ uint32_t or_of_four(uint32_t x) {
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, true);     // quad_perm 1,0,3,2
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, true);     // quad_perm 2,3,0,1
    return x;
}

// Cache policy of the encode kernel's streams (measured on the 7B workload: both hints together
// take 0.27 ms off 5.65 ms; either alone gains nothing): the two tensors are read once and the
// bucket entries are written once, so both are marked non-temporal.
#ifndef ROSE_NT_LOADS
#define ROSE_NT_LOADS 1
#endif
constexpr int kRefreshWide = 200;      // entries per tile up to which a refresh writes 128-byte lines, see encode_body
// 128-bit load / store through the global address space (pointers fetched from a table would
// otherwise be treated as generic and use the slower flat instructions).  The address needs no more
// than the alignment of a 16-bit element: the compiler emits the same instruction, and the memory
// pipeline cuts what crosses a line.  Two streams read in 16 KB tiles: 6.6 TB/s at aligned addresses,
// 6.5 with one stream 2 or 4 bytes off, 5.6 - 6.2 with both off (see tile_ctx).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef __attribute__((address_space(1))) u32x4_any global_u32x4;
__device__ __forceinline__ uint4 gload16(const void *p) {
    u32x4 v = *reinterpret_cast<const global_u32x4 *>(reinterpret_cast<uintptr_t>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
// the same for data that is read once: tells the caches not to keep it
__device__ __forceinline__ uint4 gload16_stream(const void *p) {
#if ROSE_NT_LOADS
    u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const global_u32x4 *>(reinterpret_cast<uintptr_t>(p)));
#else
    u32x4 v = *reinterpret_cast<const global_u32x4 *>(reinterpret_cast<uintptr_t>(p));
#endif
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void gstore16_stream(void *p, uint4 v) {
    u32x4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<global_u32x4 *>(reinterpret_cast<uintptr_t>(p)));
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
typedef __attribute__((address_space(1))) u32x2_any global_u32x2;
__device__ __forceinline__ void gstore8_stream(void *p, uint32_t x, uint32_t y) {
    u32x2 w = {x, y};
    __builtin_nontemporal_store(w, reinterpret_cast<global_u32x2 *>(reinterpret_cast<uintptr_t>(p)));
}

// Single elements the same way.  (Flat accesses may come back out of turn: where one can be on its way, the compiler
// waits for everything instead of for the load it needs.)
typedef __attribute__((address_space(1))) uint16_t global_u16;
typedef __attribute__((address_space(1))) uint32_t global_u32;
__device__ __forceinline__ uint32_t gload_u16(const void *p) { return *reinterpret_cast<const global_u16 *>(reinterpret_cast<uintptr_t>(p)); }
__device__ __forceinline__ uint32_t gload_u32(const void *p) { return *reinterpret_cast<const global_u32 *>(reinterpret_cast<uintptr_t>(p)); }
__device__ __forceinline__ void gstore_u16(void *p, uint32_t v) { *reinterpret_cast<global_u16 *>(reinterpret_cast<uintptr_t>(p)) = (uint16_t)v; }

// Uniform (per-workgroup) table reads through the constant address space, so that they become
// scalar loads served by the scalar cache instead of vector loads.  Only used for what the launch itself does not
// write: the plan's piece / tile tables, the caller's pointer tables, and in apply a bucket's indices and
// segment table, which an earlier launch has written (the scalar cache is clean when a kernel starts).
typedef __attribute__((address_space(4))) const uint32_t const_u32;
typedef __attribute__((address_space(4))) const uint64_t const_u64;
__device__ __forceinline__ uint32_t cload32(const void *p) {
    return *reinterpret_cast<const_u32 *>(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ uint64_t cload64(const void *p) {
    return *reinterpret_cast<const_u64 *>(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ Piece load_piece(const Piece *p) {
    static_assert(sizeof(Piece) == 7 * 8, "piece is read as seven 64-bit words");
    static_assert(kTile <= (1 << 13), "a ring entry keeps the offset inside a tile in 13 bits");
    uint64_t w[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) w[i] = cload64(reinterpret_cast<const uint64_t *>(p) + i);
    Piece pc;
    __builtin_memcpy(&pc, w, sizeof pc);
    return pc;
}

// source element of piece-relative local index k
__device__ __forceinline__ int64_t src_index(const Piece &pc, uint32_t k, bool use_magic) {
    if (pc.flags & kPieceStrided) {
        uint32_t q = use_magic ? (__umulhi(k, pc.magic) >> pc.shift) : (k / (uint32_t)pc.run);
        return pc.src_off + (int64_t)q * pc.stride + (k - q * (uint32_t)pc.run);
    }
    return pc.src_off + k;
}

// shard-local index of element k of the piece
__device__ __forceinline__ uint32_t dst_index(const Piece &pc, uint32_t k, bool use_magic) {
    if (pc.flags & kPieceDstStrided) {
        uint32_t q = use_magic ? (__umulhi(k, pc.magic) >> pc.shift) : (k / (uint32_t)pc.run);
        return (uint32_t)pc.local_base + q * (uint32_t)pc.lstride + (k - q * (uint32_t)pc.run);
    }
    return (uint32_t)pc.local_base + k;
}

// Tile loaders.  A lane's vector j holds the eight 16-bit patterns at piece-relative local indices
// k .. k+7 with k = k_wave + (j * 64 + lane) * 8.
//
// Loading (raw registers) is split from conversion (fp32 -> bf16) so that a tile's loads can be issued long
// before its data is needed.
template <int SRC_F32> struct RawTile;
template <> struct RawTile<0> { uint4 v[kIters]; };
template <> struct RawTile<1> { uint4 lo[kIters], hi[kIters]; };

__device__ __forceinline__ uint4 raw_to_bf16(const RawTile<0> &r, int j) { return r.v[j]; }
__device__ __forceinline__ uint4 raw_to_bf16(const RawTile<1> &r, int j) {
    return make_uint4(pack_rne(r.lo[j].x, r.lo[j].y), pack_rne(r.lo[j].z, r.lo[j].w),
                      pack_rne(r.hi[j].x, r.hi[j].y), pack_rne(r.hi[j].z, r.hi[j].w));
}

// General path (last vector of a piece, very short runs, odd addresses): one vector, element by element;
// patterns past the end of the piece read as zero.
template <int SRC_F32>
__device__ __forceinline__ uint4 load_vec_general(const void *base, const Piece &pc, uint32_t k) {
    // deliberately one element at a time in a rolled loop: this path is rare and must stay small
    uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
#pragma unroll 1
    for (uint32_t i = 0; i < (uint32_t)kVec; ++i) {
        uint32_t v = 0;
        if (k + i < (uint32_t)pc.len) {
            int64_t s = src_index(pc, k + i, false);
            v = SRC_F32 ? rne_bf16(static_cast<const uint32_t *>(base)[s])
                        : (uint32_t) static_cast<const uint16_t *>(base)[s];
        }
        v <<= (i & 1u) * 16u;
        const uint32_t q = i >> 1;
        w0 |= (q == 0) ? v : 0u;
        w1 |= (q == 1) ? v : 0u;
        w2 |= (q == 2) ? v : 0u;
        w3 |= (q == 3) ? v : 0u;
    }
    return make_uint4(w0, w1, w2, w3);
}

// Vectors that straddle the end of a run (kPieceSplit: runs of at least 8 elements that are no multiple
// of 8).  Element i < left of the vector at k lies left from the end of its run, the others at the start
// of the next run.  A 128-bit load at src_index(k) holds the former in place, and one at
// split_tail_at(k) the latter in place; both stay between the vector's first and last element.
__device__ __forceinline__ uint32_t split_left(const Piece &pc, uint32_t k, uint32_t *q) {
    *q = __umulhi(k, pc.magic) >> pc.shift;
    return (*q + 1) * (uint32_t)pc.run - k;              // elements of k's run from k on: below 8 if it straddles
}
__device__ __forceinline__ int64_t split_tail_at(const Piece &pc, uint32_t q, uint32_t left) {
    return pc.src_off + (int64_t)(q + 1) * pc.stride - left;
}
// elements 0 .. left-1 of a, the others of b
__device__ __forceinline__ uint4 split_merge(uint4 a, uint4 b, uint32_t left) {
    auto part = [&](uint32_t x, uint32_t y, int32_t d) {  // d: how many of the dword's two elements x gives
        const uint32_t m = d >= 2 ? 0xFFFFFFFFu : d == 1 ? 0xFFFFu : 0u;
        return (x & m) | (y & ~m);
    };
    const int32_t l = (int32_t)left;
    return make_uint4(part(a.x, b.x, l), part(a.y, b.y, l - 2), part(a.z, b.z, l - 4), part(a.w, b.w, l - 6));
}

__device__ __forceinline__ uint4 xor4(uint4 a, uint4 b) { return make_uint4(a.x ^ b.x, a.y ^ b.y, a.z ^ b.z, a.w ^ b.w); }

// ---------------------------------------------------------------------------------------------
// Prefix sums across workgroups.
//
// Every tile needs the number of entries that earlier tiles of its chain (= destination shard)
// produce.  Tiles are grouped in blocks of kBlock consecutive tiles of a chain.  A worker publishes
// each tile's count ("aggregate") in the tile's descriptor word and moves on.  A few workgroups of
// the grid do not walk tiles: each of their waves SERVES blocks (block s, s + n_servers, ...): it
// reads the block's 64 aggregates with one load per poll, scans them, publishes the block total,
// looks back over earlier BLOCK words (64 blocks = 4096 tiles per load) for the block's offset and
// writes every tile of the block its exclusive prefix into the tile's word.  Workers read only
// their own tiles' words, so no worker ever walks a chain or waits for a slower worker's tile
// other than through the answer it needs.
//
// A descriptor is one 64-bit word, status in the top two bits, value below, written and read with
// relaxed device-scope atomics: the word carries all a reader needs, nothing else is ordered by it.
//
// Progress: the whole grid (workers and servers) is resident at once: the launcher sizes it from
// the occupancy query.  A worker publishes a tile's count before it ever waits for that tile's
// prefix, and the rules at struct Walk keep it from waiting for a block that still needs a count
// from the waiter itself; a server waits for counts of its current block and for earlier blocks.
// So every wait is for something a running wave produces without waiting on the waiter.  Waits
// are bounded anyway:
// after ROSE_SPIN_LIMIT failed polls, or once the abort flag is set, a wave stops waiting, sets
// the flag, and the launch is reported as failed; every wave always reaches the end of the kernel.
// ---------------------------------------------------------------------------------------------
constexpr u64 kStatusShift = 62;
constexpr u64 kStatusAggregate = 1;   // tile word: the tile's count;  block word: the block's count
constexpr u64 kStatusPrefix = 2;      // tile word: the tile's exclusive prefix;  block word: count of
                                      // this block and all earlier blocks of the chain
constexpr u64 kValueMask = (1ull << kStatusShift) - 1;

#ifndef ROSE_WRITE_PERIOD_LOG2
#define ROSE_WRITE_PERIOD_LOG2 12     // ticks of the 100 MHz clock between windows (2^12: 41 us; encode_walk doubles it)
#endif
// Ticks a window is open, for the tile order and density a launch runs with (rule: encode_walk).
#ifndef ROSE_WRITE_OPEN_TIMED
#define ROSE_WRITE_OPEN_TIMED 1024    // 10 us
#endif
#ifndef ROSE_WRITE_OPEN_NEAR
#define ROSE_WRITE_OPEN_NEAR 1536     // 15 us
#endif
#ifndef ROSE_WRITE_OPEN_WIDE
#define ROSE_WRITE_OPEN_WIDE 2048     // 20 us
#endif
constexpr uint32_t kPollLead = 800;   // ticks before a window from which on prefixes are asked for
#ifndef ROSE_COUNT_AHEAD
#define ROSE_COUNT_AHEAD 1    // count the rest of a ticket's tiles before waiting for room (dense inputs)
#endif
#ifndef ROSE_SPIN_LIMIT
#define ROSE_SPIN_LIMIT (1u << 22)   // failed polls after which a wave gives up and flags the launch
#endif

__device__ __forceinline__ void desc_store(u64 *p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 desc_load(u64 *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workspace is one array of 64-bit words: header (abort flag, ticket counters), tile words,
// block words.  All of it starts at zero, but for the words that say how the update goes.
__global__ void reset_kernel(u64 *workspace, int64_t n_words, uint32_t form, uint32_t walk) {
    static_assert(kWsFormWord % 2 == 1 && kWsWalkWord == kWsFormWord + 1, "an upper half and the lower half behind it");
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n_words; i += (int64_t)gridDim.x * blockDim.x) workspace[i] = i == kWsFormWord / 2 ? (u64)form << 32 : i == kWsWalkWord / 2 ? (u64)walk : 0;
}

// After encode: if any wave gave up waiting, mark every bucket as invalid (total = -1) so that
// rose_bucket_check reports it and apply does nothing.
__global__ void finalize_kernel(EncodeArgs a) {
    if (threadIdx.x < (unsigned)a.tp && *a.abort_flag) a.bucket[threadIdx.x].seg_off[a.n_tensors] = -1;
}

// Asking for a ticket without waiting for it.  The counter's answer is in flight from one
// iteration of the worker loop to the next; a value in flight must not live in a register the
// compiler knows about (it may copy such a register at any time, before the answer has arrived).
// So each encode kernel keeps one VGPR out of the compiler's hands (amdgpu_num_vgpr stops the
// allocator below it) and the two routines here name it directly.
//   ticket_request: lane 0 of the calling wave adds 1 to *counter; the old value will arrive in
//                   lane 0 of the reserved register.  Nothing waits.
//   ticket_take:    waits for every outstanding vector memory operation of the wave, then reads
//                   the reserved register.
// A kernel with 4 waves per SIMD has 128 registers per lane (CLASS = 0), one with 3 has 168 (1),
// one with 2 has 256 (2).
#define ROSE_TICKET_VGPR_0 "v127"
#define ROSE_TICKET_VGPR_1 "v167"
#define ROSE_TICKET_VGPR_2 "v255"
constexpr int kNumVgpr0 = 126, kNumVgpr1 = 166, kNumVgpr2 = 254;     // what the compiler may use
#define ROSE_TICKET_REQUEST(REG)                                                                              \
    asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, 1\n\tglobal_atomic_add " REG                         \
                 ", %1, %2, %3 sc0\n\ts_mov_b64 exec, %0"                                                     \
                 : "=&s"(saved) : "v"(zero), "v"(one), "s"(counter) : "memory", REG)
#define ROSE_TICKET_TAKE(REG) asm volatile("s_waitcnt vmcnt(0)\n\tv_mov_b32 %0, " REG : "=v"(t) : : "memory")
template <int CLASS>
__device__ __forceinline__ void ticket_request(unsigned int *counter) {
    unsigned long long saved;
    const unsigned int zero = 0, one = 1;
    if constexpr (CLASS == 2) ROSE_TICKET_REQUEST(ROSE_TICKET_VGPR_2);
    else if constexpr (CLASS == 1) ROSE_TICKET_REQUEST(ROSE_TICKET_VGPR_1);
    else ROSE_TICKET_REQUEST(ROSE_TICKET_VGPR_0);
}
template <int CLASS>
__device__ __forceinline__ unsigned int ticket_take() {
    unsigned int t;
    if constexpr (CLASS == 2) ROSE_TICKET_TAKE(ROSE_TICKET_VGPR_2);
    else if constexpr (CLASS == 1) ROSE_TICKET_TAKE(ROSE_TICKET_VGPR_1);
    else ROSE_TICKET_TAKE(ROSE_TICKET_VGPR_0);
    return t;
}
#undef ROSE_TICKET_REQUEST
#undef ROSE_TICKET_TAKE

__device__ __forceinline__ bool has_prefix(u64 word) { return (word >> kStatusShift) == kStatusPrefix; }

// bounded wait bookkeeping; returns false when the wave must stop waiting
__device__ __forceinline__ bool keep_waiting(unsigned int *abort_flag, unsigned int &spins, int lane) {
    if (++spins > ROSE_SPIN_LIMIT ||
        ((spins & 63u) == 0 && __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
        if (lane == 0) __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    __builtin_amdgcn_s_sleep(2);
    return true;
}

// sum of a 64-bit value over the wave
__device__ __forceinline__ u64 wave_sum64(u64 v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, 64);
    return v;
}

// Offset of block `blk` (index into block_desc) inside its chain whose first block is
// `blk_first`: the published total of all earlier blocks.  One wave; each step reads 64 earlier
// block words (nearest first), needs every word nearer than the first prefix to hold at least an
// aggregate, and sums them.
__device__ __forceinline__ bool block_look_back(u64 *block_desc, unsigned int *abort_flag, int32_t blk,
                                                int32_t blk_first, int lane, u64 *out) {
    u64 excl = 0;
    int32_t look = blk - 1;
    unsigned int spins = 0;
    for (;;) {
        int32_t at = look - lane;
        u64 v = (at >= blk_first) ? desc_load(block_desc + at) : (kStatusPrefix << kStatusShift);
        u64 st = v >> kStatusShift;
        u64 pref = __ballot(st == kStatusPrefix);
        u64 empty = __ballot(st == 0);
        int first_pref = pref ? __ffsll((long long)pref) - 1 : 64;
        u64 need = (first_pref >= 63) ? ~0ull : ((1ull << (first_pref + 1)) - 1);
        if (empty & need) {
            if (!keep_waiting(abort_flag, spins, lane)) return false;
            continue;
        }
        excl += wave_sum64((lane <= first_pref) ? (v & kValueMask) : 0);
        if (pref) break;
        look -= 64;
    }
    *out = excl;
    return true;
}

// A serving wave: blocks server, server + n_servers, ... of those that are walked, in their order.
template <int TURNS>
__device__ __forceinline__ void serve_blocks(const EncodeArgs &a, int32_t server, int lane) {
    int32_t shard = 0;
    for (int32_t at = server; at < a.n_blocks; at += a.n_servers) {
        const WalkedBlock walked = nth_block<TURNS>(a, at, shard);
        const int32_t blk = walked.blk;
        shard = walked.shard;
        const int32_t blk_first = a.block_first[shard];
        const int32_t first_tile = a.chain_first[shard] + (blk - blk_first) * kBlock;
        const int32_t n = min(kBlock, a.chain_first[shard + 1] - first_tile);   // tiles in this block
        unsigned int spins = 0;
        bool ok = true;
        u64 agg = 0;
        for (;;) {   // lane i takes the count of the block's tile i
            u64 v = (lane < n) ? desc_load(a.tile_desc + first_tile + lane) : (kStatusAggregate << kStatusShift);
            if (__ballot((v >> kStatusShift) == 0) == 0) {
                agg = v & kValueMask;
                break;
            }
            if (!keep_waiting(a.abort_flag, spins, lane)) {
                ok = false;
                break;
            }
        }
        const uint32_t incl = wave_incl_scan((uint32_t)agg);    // <= 64 tiles * kTile entries
        const uint32_t block_total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        u64 block_excl = 0;
        if (ok && blk > blk_first) {
            if (lane == 0) desc_store(a.block_desc + blk, (kStatusAggregate << kStatusShift) | block_total);
            ok = block_look_back(a.block_desc, a.abort_flag, blk, blk_first, lane, &block_excl);
        }
        // published even after giving up, so that nobody keeps waiting on this block
        if (lane == 0) desc_store(a.block_desc + blk, (kStatusPrefix << kStatusShift) | (block_excl + block_total));
        if (lane < n)
            desc_store(a.tile_desc + first_tile + lane,
                       (kStatusPrefix << kStatusShift) | (block_excl + (incl - (uint32_t)agg)));
    }
}

// ---------------------------------------------------------------------------------------------
// encode: persistent workgroups.  The first n_server_wgs workgroups serve prefixes (above), the
// others are workers that walk the tiles their tickets name (see ticket_tile and struct Walk).
//
// Worker, per tile: (1) the tile's 128-bit loads were issued one tile earlier; XOR old and new
// into an 8-bit change mask per vector, (2) see which parked tiles' prefixes have arrived,
// poll for the others, ask for a ticket, (3) issue the NEXT tile's loads, (4) wave prefix sums of
// the popcounts, wave totals through LDS, (5) publish the tile's count, copy out parked tiles, (6) park the tile's
// entries, compacted, in an LDS ring and go on (the order of the memory operations matters: see
// the comment in encode_body).  The wait for a tile's prefix is deferred: parked tiles are polled
// one lane per tile, in iterations near a window, without waiting; only when the ring (kRing entries) or the
// queue of parked tiles (kQueue) is full, and at the end, does a workgroup wait.  This keeps
// loads in flight while counts travel between workgroups.  The ring holds any tile, all of whose elements may have changed.
// Inside a tile wave w covers a contiguous part and walks it in kIters steps of 512 elements,
// so the order (wave, step, lane, element) is ascending local index.
// ---------------------------------------------------------------------------------------------
#ifndef ROSE_RING
#define ROSE_RING 8192
#endif
#ifndef ROSE_QUEUE
#define ROSE_QUEUE 64         // (16 to 64 measure the same in the spread order; the timed order holds tiles back for a
                              // whole period between windows)
#endif
constexpr int kRing = ROSE_RING;        // entries parked per workgroup (power of two)
constexpr int kQueue = ROSE_QUEUE;      // tiles parked per workgroup (<= 64)
static_assert(kRing >= kTile, "a tile's entries fit the ring, however many they are");
static_assert((kRing & (kRing - 1)) == 0 && (kQueue & (kQueue - 1)) == 0 && kQueue <= 64,
              "ring and queue sizes must be powers of two, the queue at most a wave");

enum : int { kLoadVec = 0, kLoadGeneral = 1 };
enum : int { kDrainOldest = 0, kDrainAll = 1, kDrainReady = 2 };


struct TileCtx {
    Piece pc;
    const uint16_t *old_base;
    const void *new_base;
    uint32_t k_tile;    // the tile's elements are k_tile .. k_tile + kTile - 1, as far as the piece has them (the first
                        // tile of a piece that is shifted begins up to kShiftElems - 1 below 0)
    uint32_t shift;     // elements by which the piece's tiles are shifted
    uint32_t limit;     // the piece's length for a tile that reaches past either end, 0xFFFFFFFF for a full tile
    uint32_t vec;       // bit 0: 128-bit loads are legal for this tile; bit 2: its vectors may straddle runs
    int32_t piece;      // index of pc in the piece table
};

__device__ __forceinline__ TileCtx tile_ctx(const EncodeArgs &a, int32_t tile) {
    TileCtx c;
    c.piece = cload32(a.tile_piece + tile);
    c.pc = load_piece(a.pieces + c.piece);
    c.old_base = reinterpret_cast<const uint16_t *>(cload64(a.old_ptrs + c.pc.tensor));
    c.new_base = reinterpret_cast<const void *>(cload64(a.new_ptrs + c.pc.tensor));
    // uniform choice: 128-bit loads at whatever element they start, as long as runs hold a whole vector (a
    // decoder whose tensors start at odd elements and whose rows are 765 elements a shard, 131 M weights:
    // 526 us with one element per load for such tiles, 151 us this way)
    c.vec = ((c.pc.flags & kPieceLoad16) && ((((uintptr_t)c.old_base) | ((uintptr_t)c.new_base)) & 1u) == 0 &&
             c.pc.len >= kVec) ? ((c.pc.flags & kPieceSplit) ? 5u : 1u) : 0u;
    // Tensors that lie one right behind the other begin anywhere.  128-bit loads at any alignment are legal, but a wave's
    // load then touches a 128-byte line more than it fills, and a refresh writes parts of lines.  So the tiles of a piece
    // of several tiles are moved down to the old tensor's lines (the new one's too, where both are laid out alike), if
    // all its rows begin equally far from a line (kPieceShift); rows in runs then have vectors that straddle two.  Packed,
    // eight 7B-style layers, 2 %: 1695 -> 1310 us (at lines 1275), with refresh 2653 -> 2025, fp32 masters 2101 -> 2030; all 32
    // layers at 5 % 6392 -> 5158; 131 M weights in rows of 765 elements a shard 121 -> 100; 64 MiB 19.9 -> 15.7.
    c.shift = (c.vec && (c.pc.flags & kPieceShift))
                  ? (uint32_t)((reinterpret_cast<uintptr_t>(c.old_base) >> 1) + (uintptr_t)c.pc.src_off) & (uint32_t)(kShiftElems - 1) : 0u;
    if ((c.pc.flags & kPieceStrided) && (c.shift & (uint32_t)(kVec - 1))) c.vec |= 4u;
    c.k_tile = (uint32_t)(tile - c.pc.first_tile) * (uint32_t)kTile - c.shift;
    c.limit = ((int32_t)c.k_tile >= 0 && c.k_tile + (uint32_t)kTile <= (uint32_t)c.pc.len) ? 0xFFFFFFFFu : (uint32_t)c.pc.len;
    return c;
}

// What a worker keeps of a tile while it handles it (uniform, a few scalars: the full context is
// only needed to issue the loads and in rare paths, which build it again).
struct TileMeta {
    uint32_t out_base;  // local index of the tile's first element (piece with contiguous local indices),
                        // else the tile's first element number k inside its piece
    int32_t piece;      // -1, or the piece whose table entry maps element numbers to local indices
    int32_t shard;
    int32_t seg;        // tensor whose segment starts with this tile, else -1
    uint32_t limit;     // see TileCtx
    uint32_t vec;       // bit 0: 128-bit loads are legal; bit 1: piece of a replicated tensor; bit 2: see TileCtx
    uint32_t k_tile;
};
__device__ __forceinline__ TileMeta tile_meta(const TileCtx &c, int32_t tile) {
    TileMeta m;
    const bool dst_strided = (c.pc.flags & kPieceDstStrided) != 0;
    m.out_base = dst_strided ? c.k_tile : (uint32_t)c.pc.local_base + c.k_tile;
    m.piece = dst_strided ? c.piece : -1;
    m.shard = c.pc.shard;
    m.seg = ((c.pc.flags & kPieceFirst) && tile == c.pc.first_tile) ? c.pc.tensor : -1;
    m.limit = c.limit;
    m.vec = c.vec | ((c.pc.flags & kPieceReplicated) ? 2u : 0u);
    m.k_tile = c.k_tile;
    return m;
}

// A lane's vector j is to hold the eight elements from k on.  One that reaches past an end of the piece is loaded
// from its first or last eight elements instead, `moved` elements away, and put in place afterwards: no vector is loaded
// element by element, none from outside the piece.
__device__ __forceinline__ int32_t vector_moved(uint32_t limit, uint32_t k) {
    const int32_t at = (int32_t)k, top = (int32_t)limit - kVec;
    return (at < 0 ? 0 : at > top ? top : at) - at;
}
__device__ __forceinline__ uint4 in_place(uint4 v, int32_t moved) {
    u64 lo = (u64)v.y << 32 | v.x, hi = (u64)v.w << 32 | v.z;
    const int32_t s = (moved < 0 ? -moved : moved) * 16, r = s & 63;
    if (moved >= 0) {
        if (s >= 64) { hi = lo; lo = 0; }
        if (r) hi = hi << r | lo >> (64 - r);
        lo <<= r;
    } else {
        if (s >= 64) { lo = hi; hi = 0; }
        if (r) lo = lo >> r | hi << (64 - r);
        hi >>= r;
    }
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}
// the same for the mask of its elements that differ; those that are not its own go
__device__ __forceinline__ uint32_t in_place(uint32_t mask, int32_t moved) {
    const int32_t s = moved < 0 ? -moved : moved;
    return s >= kVec ? 0u : moved >= 0 ? (mask << s) & 0xFFu : mask >> s;
}

// Issue a tile's 128-bit loads of the old and the new tensor: both use the same element offsets,
// which are worked out once.  t_off = wave * kWaveSpan + lane * kVec.
template <int NEW_F32>
__device__ __forceinline__ void raw_zero(int j, RawTile<0> &ro, RawTile<NEW_F32> &rn) {
    ro.v[j] = make_uint4(0, 0, 0, 0);
    if constexpr (NEW_F32) rn.lo[j] = rn.hi[j] = make_uint4(0, 0, 0, 0);
    else rn.v[j] = make_uint4(0, 0, 0, 0);
}
// one vector of the old and of the new tensor at element `off` from uniform bases
template <int NEW_F32, typename OFF>
__device__ __forceinline__ void load_raw_at(const uint16_t *o, const void *n, OFF off, int j, RawTile<0> &ro,
                                            RawTile<NEW_F32> &rn) {
    ro.v[j] = gload16_stream(o + off);
    if constexpr (NEW_F32) {
        rn.lo[j] = gload16_stream(static_cast<const uint32_t *>(n) + off);
        rn.hi[j] = gload16_stream(static_cast<const uint32_t *>(n) + off + 4);
    } else {
        rn.v[j] = gload16_stream(static_cast<const uint16_t *>(n) + off);
    }
}
// All of a tile's loads are issued unconditionally (no zeroing, no predication: nothing but the
// loads themselves ever writes the load registers); see vector_moved for the ends of the piece.
template <int NEW_F32>
__device__ __forceinline__ void load_raw_pair(const TileCtx &c, uint32_t t_off, RawTile<0> &ro, RawTile<NEW_F32> &rn) {
    // One instruction sequence for both kinds of piece: a contiguous piece is walked as a strided
    // one whose row number is always 0 (magic 0).
    const bool strided = (c.pc.flags & kPieceStrided) != 0;
    const uint32_t magic = strided ? c.pc.magic : 0u, shift = strided ? c.pc.shift : 0u;
    const uint32_t run = strided ? (uint32_t)c.pc.run : 0u;
    const int64_t stride = strided ? c.pc.stride : 0;
#pragma unroll
    for (int j = 0; j < kIters; ++j) {
        uint32_t k = c.k_tile + t_off + (uint32_t)j * 64 * kVec;
        k += (uint32_t)vector_moved((uint32_t)c.pc.len, k);
        const uint32_t q = __umulhi(k, magic) >> shift;
        const int64_t e = c.pc.src_off + (int64_t)q * stride + (k - q * run);
        load_raw_at<NEW_F32>(c.old_base, c.new_base, e, j, ro, rn);
    }
}

// eight new patterns from element e on, any alignment
template <int NEW_F32>
__device__ __forceinline__ uint4 load_new_vec(const void *base, int64_t e) {
    if constexpr (NEW_F32) {
        const uint32_t *p32 = static_cast<const uint32_t *>(base) + e;
        const uint4 lo = gload16(p32), hi = gload16(p32 + 4);
        return make_uint4(pack_rne(lo.x, lo.y), pack_rne(lo.z, lo.w), pack_rne(hi.x, hi.y), pack_rne(hi.z, hi.w));
    } else {
        return gload16(static_cast<const uint16_t *>(base) + e);
    }
}

// A tile's patterns, old and new, whatever its shape and alignment: the 128-bit loads of load_raw_pair, then the tails of
// vectors that straddle two runs, or everything element by element.  For kernels that do not keep a tile's loads in flight
// across other work (the ticket kernel has its own form of this).
template <int NEW_F32>
__device__ __forceinline__ void load_tile_pair(const TileCtx &c, uint32_t t_off, uint4 (&o)[kIters], uint4 (&n)[kIters]) {
    RawTile<0> ro;
    RawTile<NEW_F32> rn;
    if (c.vec & 1u) {
        load_raw_pair<NEW_F32>(c, t_off, ro, rn);
#pragma unroll
        for (int j = 0; j < kIters; ++j) {
            o[j] = ro.v[j];
            n[j] = raw_to_bf16(rn, j);
        }
        if (!(c.vec & 4u)) return;
    }
#pragma unroll
    for (int j = 0; j < kIters; ++j) {
        const uint32_t k = c.k_tile + t_off + (uint32_t)(j * 64) * kVec;
        if (!(c.vec & 1u)) {
            if (k >= (uint32_t)c.pc.len) {              // (at once: a tile of a small tensor holds hardly anything else)
                o[j] = n[j] = make_uint4(0, 0, 0, 0);
            } else {
                o[j] = load_vec_general<0>(c.old_base, c.pc, k);
                n[j] = load_vec_general<NEW_F32>(c.new_base, c.pc, k);
            }
        } else if (!vector_moved((uint32_t)c.pc.len, k)) {
            uint32_t q;
            const uint32_t left = split_left(c.pc, k, &q);
            if (left < (uint32_t)kVec) {
                const int64_t e = split_tail_at(c.pc, q, left);
                o[j] = split_merge(o[j], gload16(c.old_base + e), left);
                n[j] = split_merge(n[j], load_new_vec<NEW_F32>(c.new_base, e), left);
            }
        }
    }
}
// The masks of the elements of such a tile that differ; vectors at an end of the piece are put in place.
__device__ __forceinline__ void tile_masks(const TileCtx &c, uint32_t t_off, uint4 (&o)[kIters], uint4 (&n)[kIters],
                                           uint32_t (&mask)[kIters]) {
#pragma unroll
    for (int j = 0; j < kIters; ++j) mask[j] = nz16_mask(xor4(o[j], n[j]));
    if ((c.vec & 1u) && c.limit != 0xFFFFFFFFu) {
#pragma unroll
        for (int j = 0; j < kIters; ++j) {
            const int32_t moved = vector_moved(c.limit, c.k_tile + t_off + (uint32_t)(j * 64) * kVec);
            mask[j] = in_place(mask[j], moved);
            if (moved && mask[j]) {
                o[j] = in_place(o[j], moved);
                n[j] = in_place(n[j], moved);
            }
        }
    }
}

// (uniform anyway: said here, the table look-ups stay scalar)
template <int TURNS>
__device__ __forceinline__ int32_t ticket_tile(const EncodeArgs &a, int32_t ticket, int32_t j) {
    return tile_of_ticket<TURNS>(a, __builtin_amdgcn_readfirstlane(ticket), __builtin_amdgcn_readfirstlane(j));
}
template <int TURNS>
__device__ __forceinline__ int walk_step(const EncodeArgs &a, Walk &w, int32_t *tile) {
    return walk_step(a.batch, w, tile, [&](int32_t ticket, int32_t j) { return ticket_tile<TURNS>(a, ticket, j); });
}
// A value that is no ticket marks the launch as failed: the register it arrives in is only reserved by asking the compiler, see
// ticket_request.
__device__ __forceinline__ void walk_accept(const EncodeArgs &a, Walk &w, uint32_t n) {
    if (!walk_accept(a.n_tickets, w, n)) __hip_atomic_store(a.abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive rank of each of this lane's vectors inside the wave's span; returns the wave's total.  The
// per-vector counts (<= 8, wave totals <= 512) are scanned two at a time in 16-bit fields.
__device__ __forceinline__ uint32_t vector_ranks(const uint32_t (&mask)[kIters], uint32_t (&rank)[kIters]) {
    uint32_t wave_total = 0;
#pragma unroll
    for (int j = 0; j < kIters; j += 2) {
        const uint32_t c0 = __popc(mask[j]);
        const uint32_t c1 = (j + 1 < kIters) ? __popc(mask[j + 1]) : 0u;
        const uint32_t inc = wave_incl_scan(c0 | (c1 << 16));
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        rank[j] = wave_total + (inc & 0xFFFFu) - c0;
        wave_total += tot & 0xFFFFu;
        if (j + 1 < kIters) {
            rank[j + 1] = wave_total + (inc >> 16) - c1;
            wave_total += tot >> 16;
        }
    }
    return wave_total;
}

// Entry k as it is written: an arithmetic payload is formed here, of the compacted entries only.
template <int ARITH>
__device__ __forceinline__ uint32_t parked(uint32_t k, const uint32_t *s_entry, const uint16_t *s_was) {
    const uint32_t entry = s_entry[k];
    if constexpr (!ARITH) return entry;
    bool escapes;
    const uint32_t payload = arith_one(s_was[k], entry & 0xFFFFu, &escapes);
    return (entry & 0x7FFF0000u) | payload | (escapes ? 0x80000000u : 0u);
}

// Local index of a parked entry of a run whose elements are numbered from `base` on: an entry keeps the low 15 bits of its
// element's number (bit 31 is the escape's), and a run spans less than 2^15 elements.
constexpr int kRunTiles = 4;
static_assert(kRunTiles <= kWaves, "a wave takes a tile of a run");
static_assert(kRunTiles * kTile <= 1 << 15, "15 bits tell the elements of a run apart");
__device__ __forceinline__ uint32_t run_local(uint32_t entry, uint32_t base) {
    return base + (((entry - (base << 16)) >> 16) & 0x7FFFu);
}

// The cnt entries that lie in the ring from `off` on go to positions excl .. of a bucket.  All threads of the workgroup.
// A wave's stores begin at multiples of 32 entries of the BUCKET, not of the run, so that every store but the first and last
// of a run fills whole 64-byte lines (otherwise each wave's store starts and ends inside a line and the line's 32-byte halves
// are written twice: 1.20 x the bytes at the memory).
// A thread takes four entries, whose places are found together and which leave as one 128-bit and one 64-bit store.  All
// workgroups copy out in the same windows of time, the memory then waits for them, and a load is away for less time than an
// entry after the other takes (without its stores, an entry a lane, copying out cost 8.6 GB read 0.18 ms of 1.53 at 5 %).
template <int ARITH, bool ESCAPES>
__device__ __forceinline__ void write_run(const EncodeArgs &a, int32_t shard, int32_t piece, uint32_t base, uint32_t off, u64 excl,
                                          uint32_t cnt, const uint32_t *s_ring, const uint16_t *s_was) {
    const BucketDev b = a.bucket[shard];
    if (!ARITH && piece < 0 && excl + cnt <= (u64)b.capacity) {
        int32_t *const idx = b.idx + excl;
        uint16_t *const val = b.val + excl;
        const int32_t n = (int32_t)cnt, first = (int32_t)(threadIdx.x * 4) - (int32_t)((uint32_t)excl & 31u);
        // places of the ring are read whether they are the run's or not: no lane waits for LDS twice
        auto four = [&](int32_t k, uint32_t (&e)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = s_ring[(off + (uint32_t)(k + i)) & (uint32_t)(kRing - 1)];
        };
        auto put = [&](int32_t k, const uint32_t (&e)[4]) {
            uint32_t local[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) local[i] = run_local(e[i], base) | (ESCAPES ? e[i] & 0x80000000u : 0u);
            if (k >= 0 && k + 4 <= n) {
                gstore16_stream(idx + k, make_uint4(local[0], local[1], local[2], local[3]));
                gstore8_stream(val + k, __builtin_amdgcn_perm(e[1], e[0], 0x05040100u), __builtin_amdgcn_perm(e[3], e[2], 0x05040100u));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (k + i >= 0 && k + i < n) {
                        __builtin_nontemporal_store((int32_t)local[i], idx + k + i);
                        __builtin_nontemporal_store((uint16_t)e[i], val + k + i);
                    }
            }
        };
        for (int32_t k = first; k < n; k += kThreads * 4) {
            uint32_t e[4];
            four(k, e);
            put(k, e);
        }
        return;
    }
    // a run that ends behind the bucket's end, or whose local indices come in strided runs
    uint32_t l_base = 0, l_run = 0, l_magic = 0, l_shift = 0, l_stride = 0;
    if (piece >= 0) {
        const Piece pc = load_piece(a.pieces + piece);
        l_base = (uint32_t)pc.local_base;
        l_run = (uint32_t)pc.run;
        l_magic = pc.magic;
        l_shift = pc.shift;
        l_stride = (uint32_t)pc.lstride;
    }
    const uint32_t phase = (uint32_t)excl & 31u;
    for (uint32_t kk = threadIdx.x; kk < cnt + phase; kk += kThreads) {
        const uint32_t k = kk - phase;                 // (wraps below phase: caught by the first test)
        const u64 pos = excl + k;
        if (kk >= phase && pos < (u64)b.capacity) {
            const uint32_t entry = parked<ARITH>((off + k) & (kRing - 1), s_ring, s_was);
            uint32_t local = run_local(entry, base);
            if (piece >= 0) {                          // it is the element's number inside the piece here
                // (runs of one element have no magic divisor: the quotient is the number itself)
                const uint32_t q = l_run == 1u ? local : (__umulhi(local, l_magic) >> l_shift);
                local = l_base + q * l_stride + (local - q * l_run);
            }
            if constexpr (ESCAPES) local |= entry & 0x80000000u;
            __builtin_nontemporal_store((int32_t)local, b.idx + pos);
            __builtin_nontemporal_store((uint16_t)entry, b.val + pos);
        }
    }
}

// The same for a run of tiles of several pieces (tensors of a tile or two): its tiles are numbered each by itself, and a wave
// takes one of them.  (Each as a run of its own / this way, us at 1 %: tensors of half a tile a shard 653 / 588, fp32 masters 796 / 733;
// of one tile 744 / 697; of two 868 / 845.  An entry's tile found by compares in write_run instead, real models are 1 % slower.)
template <int ARITH, bool ESCAPES>
__device__ __forceinline__ void write_tile(const BucketDev &b, uint32_t base, uint32_t off, u64 excl, uint32_t cnt, int lane,
                                           const uint32_t *s_ring, const uint16_t *s_was) {
    const uint32_t phase = (uint32_t)excl & 31u;
#pragma unroll 1
    for (uint32_t kk = (uint32_t)lane; kk < cnt + phase; kk += 64) {
        const uint32_t k = kk - phase;                 // (wraps below phase: caught by the first test)
        const u64 pos = excl + k;
        if (kk >= phase && pos < (u64)b.capacity) {
            const uint32_t entry = parked<ARITH>((off + k) & (kRing - 1), s_ring, s_was);
            uint32_t local = run_local(entry, base);
            if constexpr (ESCAPES) local |= entry & 0x80000000u;
            __builtin_nontemporal_store((int32_t)local, b.idx + pos);
            __builtin_nontemporal_store((uint16_t)entry, b.val + pos);
        }
    }
}

// PAYLOAD = 1: arithmetic payloads formed of the compacted entries; 2: of every element, before they are compacted.
template <int NEW_F32, int REFRESH, int PAYLOAD>
__device__ __forceinline__ void encode_body(const EncodeArgs &a) {
    constexpr int ARITH = PAYLOAD == 1;                // entries carry the old pattern beside them
    constexpr int FORMED = PAYLOAD == 2;               // entries are payloads from the start
    static_assert(!(FORMED && REFRESH), "a refresh needs the new patterns");
    // Blocks in turns: a refresh writes lines of what it reads all the time, and the memory takes that better where they lie in
    // several places (eight 7B-style layers with embedding and head, TP4, at 1 / 5 / 15 %: chain by chain 1813 / 2190 / 2428 us, in
    // turns 1750 / 2109 / 2397; arithmetic payloads at 2 % 1978 and 1899, fp32 masters 2695 and 2653; but arithmetic payloads of
    // fp32 masters, with half the waves, 2624 and 2652: not those).  Others write to the buckets only, which then are several at a
    // time too: at 5 / 10 % 1334 / 1546 us, in turns 1349 / 1599.
    constexpr int TURNS = REFRESH && !(NEW_F32 && ARITH);
    // Runs of tiles of one piece only, see write_tile: with that beside it this kernel's ordinary runs take 1.2 % longer (eight
    // 7B-style layers at 5 %: 1379 and 1399 us), which is more than small tensors gain where there are few (all of half a tile: 757 and
    // 724 us, of one 752 and 720, of two 991 and 998).
    constexpr bool STRAIGHT = !NEW_F32 && !REFRESH && ARITH;
    // register class, see ticket_request
    constexpr int WIDE = (NEW_F32 && REFRESH && ARITH) ? 2 : (NEW_F32 || ARITH) ? 1 : 0;
    __shared__ uint32_t s_ring[kRing];      // an entry: low 15 bits of its element's number (TileMeta::out_base) << 16 | new pattern
    __shared__ uint16_t s_was[ARITH ? kRing : 1];    // arithmetic payload: the old patterns, from which it is formed
    __shared__ uint32_t s_wave_total[2][kWaves];
    __shared__ u64 s_excl[2][kQueue];       // prefixes of the tiles an iteration copies out, oldest first
    __shared__ u64 s_excl_sync[kQueue];     // the same for a blocking drain
    __shared__ int32_t s_nready[2];
    __shared__ uint32_t s_q_count[kQueue];
    __shared__ uint32_t s_q_off[kQueue];
    __shared__ uint32_t s_q_base[kQueue];   // see TileMeta::out_base
    __shared__ int32_t s_q_piece[kQueue];   // see TileMeta::piece
    __shared__ int32_t s_q_shard[kQueue];
    __shared__ int32_t s_q_seg[kQueue];     // tensor whose segment starts with this tile, else -1
    __shared__ int32_t s_q_last[kQueue];    // 1 if the tile is the last of its chain
    __shared__ int32_t s_ok, s_ready;
    __shared__ int32_t s_ticket[2], s_ticket_sync;
    __shared__ uint32_t s_count_only[kWaves];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int32_t)blockIdx.x < a.n_server_wgs) {
        serve_blocks<TURNS>(a, (int32_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(wave), lane);
        return;
    }

    // Uniform bookkeeping, kept identical in every thread.  The queue is a circular FIFO whose i-th
    // oldest tile sits in slot (q_head + i) mod kQueue; the ring holds their entries in that order.
    //
    // Order of the memory operations of one iteration.  The hardware counts outstanding vector
    // memory operations in issue order, and the compiler can only wait for "all but the newest
    // n" with an n it can count at compile time; behind loops and branches it has to wait for
    // everything.  So results are taken in only at the top of an iteration, where everything in
    // flight is wanted anyway, and the long-latency loads of the next tile are issued after all that
    // is asked for (the poll, the ticket request) and before the bucket stores, which nothing waits for by themselves:
    //   top   the tile's data has landed; so have last iteration's poll answers and ticket
    //   (a)   change masks of this tile (frees the load registers)
    //   (b)   wave 0 takes in the poll answers and announces (through LDS, valid after this
    //         iteration's barrier) which parked tiles can be copied out
    //   (c)   wave 0 polls the parked tiles without a prefix; thread 0 asks for a ticket
    //   (d)   the NEXT tile's loads are issued
    //   (e)   scan, barrier, publish this tile's count, copy out the announced tiles, park this tile's entries
    // (Copied out in (b), in front of the loads, 8.6 GB read take 1.419 ms at 1 %, this way 1.411.)
    int q_head = 0, q_len = 0;
    uint32_t ring_used = 0, ring_head = 0;
    int parity = 0;
    int n_gone = 0;             // tiles copied out since wave 0's lanes were last moved down
    // wave 0 only: lane i tracks the i-th oldest parked tile
    int32_t wq_tile = 0;
    u64 wq_w = 0;               // the newest copy of its descriptor word: the prefix once the status says so
    u64 polled = 0;             // written only by the poll's load (in flight across the iteration boundary)
    int n_polled = 0;           // lanes of wave 0 whose tiles the poll in flight covers
    bool ticket_out = false;    // a ticket has been asked for and not yet taken in

    // copy the n oldest parked tiles to the buckets (prefixes in excl[0..n)); returns ring entries freed.
    // Tiles that follow each other in the bucket (up to four: same shard, each starting where the one
    // before ends; their entries follow each other in the ring as well) are written as one run.
    auto copy_out = [&](int n, const u64 *excl_by_age, bool ok) -> uint32_t {
        // lane i looks at the i-th oldest tile, so that the waves wait for LDS once and not tile by tile
        const bool mine = lane < n;
        const int slot = (q_head + lane) & (kQueue - 1);
        const uint32_t count = mine ? s_q_count[slot] : 0u, off = s_q_off[slot], base = s_q_base[slot];
        const int32_t piece = s_q_piece[slot], shard = s_q_shard[slot];
        const u64 excl = mine ? excl_by_age[lane] : 0;
        const uint32_t excl_lo = (uint32_t)excl, excl_hi = (uint32_t)(excl >> 32);
        const uint32_t freed = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(count), 63);
        if (!ok) return freed;
        auto of = [](uint32_t x, int t) { return (uint32_t)__builtin_amdgcn_readlane((int)x, t); };
        if (wave == 0) {                               // segment ends (few tiles have one)
            const int32_t seg = s_q_seg[slot], last = s_q_last[slot];
            for (u64 ends = __ballot(mine & ((seg >= 0) | (last != 0))); ends; ends &= ends - 1) {
                const int i = __ffsll((long long)ends) - 1;
                int64_t *const seg_off = a.bucket[of((uint32_t)shard, i)].seg_off;
                const u64 at = (u64)of(excl_hi, i) << 32 | of(excl_lo, i);
                if (lane == 0) {
                    if ((int32_t)of((uint32_t)seg, i) >= 0) seg_off[of((uint32_t)seg, i)] = (int64_t)at;
                    if (of((uint32_t)last, i)) seg_off[a.n_tensors] = (int64_t)(at + of(count, i));
                }
            }
        }
        // (positions that continue each other agree in their low halves; all lanes take part in the moves)
        auto below = [](uint32_t x) {                  // the lane below's
            return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xf, 0xf, false);     // wave_shr:1
        };
        const uint32_t shard_b = below((uint32_t)shard), piece_b = below((uint32_t)piece), base_b = below(base), end_b = below(excl_lo + count);
        const bool next = (lane > 0) & ((uint32_t)shard == shard_b) & ((int32_t)((uint32_t)piece & piece_b) < 0) & (excl_lo == end_b) &
                          (!STRAIGHT | (base == base_b + (uint32_t)kTile));
        const u64 starts = __ballot(mine & !next), apart = __ballot(base != base_b + (uint32_t)kTile);   // (of another piece)
        for (int i = 0; i < n;) {
            // everything about the run is uniform: scalar registers, the bucket's pointers come through scalar loads
            const u64 behind = starts >> i >> 1;
            int g = behind ? __ffsll((long long)behind) : n - i;
            g = g < kRunTiles ? g : kRunTiles;
            if (!STRAIGHT && __builtin_expect((apart >> i >> 1 & ((1u << (g - 1)) - 1u)) != 0, 0)) {
                const int t = i + __builtin_amdgcn_readfirstlane(wave);
                if (t < i + g)
                    write_tile<ARITH, PAYLOAD != 0>(a.bucket[of((uint32_t)shard, t)], of(base, t), of(off, t), (u64)of(excl_hi, t) << 32 | of(excl_lo, t),
                                                    of(count, t), lane, s_ring, s_was);
            } else {
                const u64 first = (u64)of(excl_hi, i) << 32 | of(excl_lo, i);
                const uint32_t cnt = of(excl_lo, i + g - 1) + of(count, i + g - 1) - (uint32_t)first;
                write_run<ARITH, PAYLOAD != 0>(a, (int32_t)of((uint32_t)shard, i), (int32_t)of((uint32_t)piece, i), of(base, i), of(off, i),
                                               first, cnt, s_ring, s_was);
            }
            i += g;
        }
        return freed;
    };
    auto pop = [&](int n, uint32_t freed) {      // forget the n oldest tiles
        q_head = (q_head + n) & (kQueue - 1);
        q_len -= n;
        ring_used -= freed;
        n_gone += n;
    };
    auto move_lanes = [&]() {    // wave 0 moves its lanes down by the tiles that are gone (the poll has been taken in or is forgotten)
        if (wave == 0 && n_gone > 0) {
            wq_tile = __shfl(wq_tile, lane + n_gone, 64);
            wq_w = __shfl(wq_w, lane + n_gone, 64);
        }
        n_gone = 0;
    };

    // Blocking drain, for when there is no room to park (or at the end): waits until the oldest
    // parked tile (all = false) or every parked tile (all = true) has its prefix, and copies out
    // every leading tile whose prefix is known; these include the announced ones.
    // mode kDrainOldest / kDrainAll as described; kDrainReady waits for nothing: it looks once and
    // copies out what has its prefix by now.
    auto drain = [&](int mode) {
        const bool all = mode == kDrainAll;
        move_lanes();                                  // (a poll in flight is forgotten: its tiles are polled again)
        n_polled = 0;
        __syncthreads();                               // parked entries visible; earlier copies done
        if (wave == 0) {
            bool ok = true;
            int n_ready = q_len;
            unsigned int spins = 0;
            for (;;) {
                if (lane < q_len && !has_prefix(wq_w)) wq_w = desc_load(a.tile_desc + wq_tile);
                const u64 unknown = __ballot(lane < q_len && !has_prefix(wq_w));
                n_ready = unknown ? __ffsll((long long)unknown) - 1 : q_len;
                if (mode == kDrainReady || (all ? (n_ready == q_len) : (n_ready >= 1 || q_len == 0))) break;
                if (!keep_waiting(a.abort_flag, spins, lane)) {
                    ok = false;         // give up: drop everything that is parked
                    n_ready = q_len;
                    break;
                }
            }
            if (lane < n_ready) s_excl_sync[lane] = wq_w & kValueMask;
            if (lane == 0) {
                s_ok = ok ? 1 : 0;
                s_ready = n_ready;
            }
        }
        __syncthreads();
        const int n_ready = __builtin_amdgcn_readfirstlane(s_ready);
        const uint32_t freed = copy_out(n_ready, s_excl_sync, s_ok != 0);
        __syncthreads();                               // ring and queue slots may be reused
        pop(n_ready, freed);
        move_lanes();
    };

    // Tiles come from tickets (dynamic, so that faster workgroups take more): thread 0 asks for a
    // ticket well before it is needed; the answer is handed to the others through LDS at the
    // barrier of the following iteration.
    Walk walk;
    walk.ticket = -1;
    walk.j = a.batch;
    walk.next_ticket = 0;
    walk.redo_through = 0;
    walk.have_next = false;
    walk.exhausted = false;
    walk.careful = false;
    walk.redo = false;
    // all threads; two barriers; no waiting for other workgroups.  Takes in the ticket that is on
    // its way, if any, else asks for one.
    auto settle_ticket = [&]() {
        if (threadIdx.x == 0) {
            if (!ticket_out) ticket_request<WIDE>(a.ticket);
            s_ticket_sync = (int32_t)ticket_take<WIDE>();
        }
        ticket_out = false;
        __syncthreads();
        walk_accept(a, walk, (uint32_t)__builtin_amdgcn_readfirstlane(s_ticket_sync));
        __syncthreads();
    };
    // Count-only pass over one tile (all threads, rolled loads: this is rare): publishes its count.
    auto publish_count = [&](int32_t t) {
        const TileCtx c = tile_ctx(a, __builtin_amdgcn_readfirstlane(t));
        uint32_t cnt = 0;
        if ((c.vec & 1u) && c.limit == 0xFFFFFFFFu) {
            // a whole tile with 128-bit loads (cached: the tile is read again soon); kept rolled, one
            // pair of vectors at a time, because the next tile's loads occupy the load registers
#pragma unroll 1
            for (int j = 0; j < kIters; ++j) {
                const uint32_t k = c.k_tile + (uint32_t)wave * kWaveSpan + (uint32_t)(j * 64 + lane) * kVec;
                const int64_t e = src_index(c.pc, k, true);
                const uint4 o = gload16(c.old_base + e);
                uint4 n;
                n = load_new_vec<NEW_F32>(c.new_base, e);
                uint32_t m = nz16_mask(xor4(o, n));
                if (c.vec & 4u) {                      // the part of the vector that lies in the next run
                    uint32_t q;
                    const uint32_t left = split_left(c.pc, k, &q);
                    if (left < (uint32_t)kVec) {
                        const int64_t e2 = split_tail_at(c.pc, q, left);
                        const uint32_t keep = (1u << left) - 1u;
                        m = (m & keep) |
                            (nz16_mask(xor4(gload16(c.old_base + e2), load_new_vec<NEW_F32>(c.new_base, e2))) & ~keep);
                    }
                }
                cnt += __popc(m);
            }
        } else {
#pragma unroll 1
            for (int j = 0; j < kIters; ++j) {
                const uint32_t k = c.k_tile + (uint32_t)wave * kWaveSpan + (uint32_t)(j * 64 + lane) * kVec;
                const uint4 o = load_vec_general<0>(c.old_base, c.pc, k);
                const uint4 n = load_vec_general<NEW_F32>(c.new_base, c.pc, k);
                cnt += __popc(nz16_mask(xor4(o, n)));
            }
        }
        const uint32_t wave_cnt = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(cnt), 63);
        __syncthreads();                               // earlier readers of s_count_only are done
        if (lane == 0) s_count_only[wave] = wave_cnt;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t total = 0;
            for (int w = 0; w < kWaves; ++w) total += s_count_only[w];
            desc_store(a.tile_desc + t, (kStatusAggregate << kStatusShift) | total);
        }
    };
    int32_t tile = -1;
    for (;;) {
        const int st = walk_step<TURNS>(a, walk, &tile);
        if (st == kWalkTile) break;
        if (st == kWalkDone) return;
        settle_ticket();
    }
    walk.careful = false;                              // nothing is parked yet, nothing has waited
    bool cur_redo = false;
    const uint32_t t_off = (uint32_t)wave * kWaveSpan + (uint32_t)lane * kVec;
    RawTile<0> raw_old;
    RawTile<NEW_F32> raw_new;
#pragma unroll
    for (int j = 0; j < kIters; ++j) raw_zero(j, raw_old, raw_new);
    // the tile's context, its loads (if 128-bit loads are legal for it), and what is kept of it
    auto start_tile = [&](int32_t t) -> TileMeta {
        const TileCtx c = tile_ctx(a, __builtin_amdgcn_readfirstlane(t));
        if (c.vec) load_raw_pair<NEW_F32>(c, t_off, raw_old, raw_new);
        return tile_meta(c, t);
    };
    TileMeta cur, nxt;
    bool loaded = false;                               // the tile's loads have been issued

    for (;;) {
        // All of the following are the same in every lane; saying so keeps them, and everything
        // derived from them, in scalar registers.
        tile = __builtin_amdgcn_readfirstlane(tile);
        q_head = __builtin_amdgcn_readfirstlane(q_head);
        q_len = __builtin_amdgcn_readfirstlane(q_len);
        ring_used = (uint32_t)__builtin_amdgcn_readfirstlane((int)ring_used);
        ring_head = (uint32_t)__builtin_amdgcn_readfirstlane((int)ring_head);
        parity = __builtin_amdgcn_readfirstlane(parity);
        n_gone = __builtin_amdgcn_readfirstlane(n_gone);
        n_polled = __builtin_amdgcn_readfirstlane(n_polled);
        walk.ticket = __builtin_amdgcn_readfirstlane(walk.ticket);
        walk.j = __builtin_amdgcn_readfirstlane(walk.j);
        walk.next_ticket = __builtin_amdgcn_readfirstlane(walk.next_ticket);
        walk.redo_through = __builtin_amdgcn_readfirstlane(walk.redo_through);
        {
            const int flags = __builtin_amdgcn_readfirstlane((int)loaded | (int)cur_redo << 1 | (int)ticket_out << 2 |
                                                             (int)walk.have_next << 3 | (int)walk.exhausted << 4 |
                                                             (int)walk.careful << 5 | (int)walk.redo << 6);
            loaded = flags & 1;
            cur_redo = flags & 2;
            ticket_out = flags & 4;
            walk.have_next = flags & 8;
            walk.exhausted = flags & 16;
            walk.careful = flags & 32;
            walk.redo = flags & 64;
        }
        cur = loaded ? nxt : start_tile(tile);         // not loaded: the first tile, or one named late
        // From here until the next tile's loads are issued this workgroup has no tile on its way (only now and then a vector's tail,
        // a poll and a ticket), so its waves go first.
        // (Among equals the oldest wave of a SIMD goes first, always: of four workgroups on a CU one then walked 160 tiles
        // where another walked 360, all others' entries waited in their rings for its counts, and at 5 % two of five tiles
        // left outside the windows because a ring was full.  This way they walk 200 to 320.)
        __builtin_amdgcn_s_setprio(3);
        // ---- (a) change masks ----
        const uint32_t k_wave = cur.k_tile + (uint32_t)wave * kWaveSpan;
        uint4 nv[kIters];                              // the new patterns (FORMED: the payloads)
        uint4 ov[ARITH ? kIters : 1];                  // the old ones
        uint32_t mask[kIters];
        uint32_t escaped = 0;                          // FORMED: bit 8 j + e: element e of vector j escapes
        // Always taken from the load registers, also for a tile that has no 128-bit loads (its
        // result is replaced below): this way every path consumes what was loaded, and the
        // compiler never has to wait for memory before the registers are loaded again.
#pragma unroll
        for (int j = 0; j < kIters; ++j) {
            nv[j] = raw_to_bf16(raw_new, j);
            mask[j] = nz16_mask(xor4(raw_old.v[j], nv[j]));
            if constexpr (ARITH) ov[j] = raw_old.v[j];
            if constexpr (FORMED) {
                uint32_t esc8;
                nv[j] = arith_vec(raw_old.v[j], nv[j], &esc8);
                escaped |= esc8 << (8 * j);
            }
        }
        // pin the above here: the load registers are dead from this point on, whatever the
        // scheduler would prefer
#pragma unroll
        for (int j = 0; j < kIters; ++j)
            asm volatile("" : "+v"(mask[j]), "+v"(nv[j].x), "+v"(nv[j].y), "+v"(nv[j].z), "+v"(nv[j].w));
        if constexpr (ARITH) {
#pragma unroll
            for (int j = 0; j < kIters; ++j) asm volatile("" : "+v"(ov[j].x), "+v"(ov[j].y), "+v"(ov[j].z), "+v"(ov[j].w));
        }
        if constexpr (FORMED) asm volatile("" : "+v"(escaped));
        // (the rare cases are marked as such: laid out in line they cost the fp32 kernels 2 % of an update of 67 M
        // elements)
        if (__builtin_expect((cur.vec & 1u) != 0, 1)) {
            if (__builtin_expect(cur.limit != 0xFFFFFFFFu, 0)) {
#pragma unroll
                for (int j = 0; j < kIters; ++j) {
                    const int32_t moved = vector_moved(cur.limit, k_wave + (uint32_t)(j * 64 + lane) * kVec);
                    mask[j] = in_place(mask[j], moved);
                    if (moved && mask[j]) {
                        nv[j] = in_place(nv[j], moved);
                        if constexpr (ARITH) ov[j] = in_place(ov[j], moved);
                    }
                    if constexpr (FORMED)
                        escaped = (escaped & ~(0xFFu << (8 * j))) | (in_place((escaped >> (8 * j)) & 0xFFu, moved) << (8 * j));
                }
            }
            // Runs that are no multiple of 8 elements: the vectors that straddle the end of a run hold
            // their first elements only; the rest is loaded now.  A lane takes its first such vector,
            // whichever of its four that is, then its second: with runs of 512 elements or more hardly
            // any lane has two, and the tile waits for one round of loads.
            if (__builtin_expect((cur.vec & 4u) != 0, 0)) {
                const TileCtx c = tile_ctx(a, __builtin_amdgcn_readfirstlane(tile));
                uint32_t todo = 0, masks = 0;          // (the four masks in one register: this loop needs many)
#pragma unroll
                for (int j = 0; j < kIters; ++j) {
                    const uint32_t k = k_wave + (uint32_t)(j * 64 + lane) * kVec;
                    uint32_t q;
                    if (!vector_moved((uint32_t)c.pc.len, k) && split_left(c.pc, k, &q) < (uint32_t)kVec) todo |= 1u << j;
                    masks |= mask[j] << (8 * j);
                }
#pragma unroll 1
                while (todo) {
                    const uint32_t js = __ffs(todo) - 1;
                    todo &= todo - 1;
                    uint32_t q;
                    const uint32_t left = split_left(c.pc, k_wave + (js * 64 + (uint32_t)lane) * kVec, &q);
                    const int64_t e = split_tail_at(c.pc, q, left);
                    const uint4 o = gload16(c.old_base + e);
                    uint4 n = load_new_vec<NEW_F32>(c.new_base, e);
                    const uint32_t tail = 0xFFu & ~((1u << left) - 1u);
                    masks = (masks & ~(tail << (8 * js))) | ((nz16_mask(xor4(o, n)) & tail) << (8 * js));
                    if constexpr (FORMED) {
                        uint32_t esc8;
                        n = arith_vec(o, n, &esc8);
                        escaped = (escaped & ~(tail << (8 * js))) | ((esc8 & tail) << (8 * js));
                    }
#pragma unroll
                    for (int jj = 0; jj < kIters; ++jj) {
                        // (a vector that is not meant keeps all its elements: no branch, hence no second set of registers)
                        const uint32_t l = (uint32_t)jj == js ? left : (uint32_t)kVec;
                        nv[jj] = split_merge(nv[jj], n, l);
                        if constexpr (ARITH) ov[jj] = split_merge(ov[jj], o, l);
                    }
                }
#pragma unroll
                for (int j = 0; j < kIters; ++j) mask[j] = (masks >> (8 * j)) & 0xFFu;
            }
        } else {
            // runs of fewer than 8 elements, pieces of fewer than 8, odd addresses.  Kept as a rolled loop (one
            // vector in flight) so that this rare path does not set the kernel's register budget;
            // the selects put the result into static slots
            const TileCtx c = tile_ctx(a, __builtin_amdgcn_readfirstlane(tile));
#pragma unroll 1
            for (int j = 0; j < kIters; ++j) {
                uint32_t k = k_wave + (uint32_t)(j * 64 + lane) * kVec;
                uint4 o = load_vec_general<0>(c.old_base, c.pc, k);
                uint4 n = load_vec_general<NEW_F32>(c.new_base, c.pc, k);
                uint32_t m = nz16_mask(xor4(o, n));
                if constexpr (FORMED) {
                    uint32_t esc8;
                    n = arith_vec(o, n, &esc8);
                    escaped = (escaped & ~(0xFFu << (8 * j))) | (esc8 << (8 * j));
                }
#pragma unroll
                for (int jj = 0; jj < kIters; ++jj) {
                    if (jj == j) {
                        nv[jj] = n;
                        mask[jj] = m;
                        if constexpr (ARITH) ov[jj] = o;
                    }
                }
            }
        }

        // ---- (b) poll answers and ticket of the previous iteration ----
        const bool accept_now = ticket_out;
        if (accept_now && threadIdx.x == 0) {
            s_ticket[parity] = (int32_t)ticket_take<WIDE>();   // nothing else is in flight here
        }
        ticket_out = false;
        if (wave == 0 && lane < n_polled && !has_prefix(wq_w)) wq_w = polled;
        move_lanes();
        bool poll = true;
        if (wave == 0) {
            const u64 unknown = __ballot(lane < q_len && !has_prefix(wq_w));
            int n_ready = unknown ? __ffsll((long long)unknown) - 1 : q_len;
            // Bucket stores go out in windows of time that all workgroups share (a
            // constant-rate clock every wave can read): a steady trickle of writes among the reads
            // costs the memory far more than the same bytes written in bursts (a plain streaming
            // kernel that reads two streams at 7.1 TB/s loses 22 % when it writes 1.5 % of what it
            // reads tile by tile, and 6 % when it writes the same bytes in such windows).  Outside a
            // window parked tiles simply stay parked, unless the queue is more than three quarters
            // full.  The ring may fill up: a workgroup that finds no room copies out what is ready at
            // once (drain).  Announcing early, from three quarters of the ring on, writes more of the
            // entries outside the windows (7B-style workload at 4 %: 5.04 ms; 4.74 ms this way).
            if (a.window_open) {
                const uint32_t now = (uint32_t)__builtin_amdgcn_s_memrealtime();
                const bool open = (now & a.window_mask) < a.window_open;
                if (!open && q_len <= kQueue * 3 / 4) n_ready = 0;
                // Prefixes are asked for from 8 us before a window on: what has none by then has had time to get one, and asked
                // for in every iteration they cost the reads (two 32B-style layers of fp32 masters, 1.6 %: 2547 us, this way 2527;
                // 1.9 G weights hardly changed, bf16 1191 and 1187, fp32 masters 1841 and 1829; asked for from 16 us before,
                // the same and at 5 % 0.5 % more).
                poll = open || ((now + kPollLead) & a.window_mask) < a.window_open || q_len > kQueue / 2;
            }
            if (lane < n_ready) s_excl[parity][lane] = wq_w & kValueMask;
            if (lane == 0) s_nready[parity] = n_ready;
            // ---- (c) poll: one lane per parked tile that has no prefix yet ----
            if (poll && lane < q_len && !has_prefix(wq_w)) polled = desc_load(a.tile_desc + wq_tile);
        }
        n_polled = poll ? q_len : 0;                   // (counts in wave 0 only)
        // ask for the next ticket as soon as the one fetched ahead has been taken into use
        if (!walk.have_next && !accept_now && !walk.exhausted && !walk.redo) {
            if (threadIdx.x == 0) ticket_request<WIDE>(a.ticket);
            ticket_out = true;
        }

        // ---- (d) the next tile's loads go out now and stay in flight during everything below ----
        int32_t next = -1;
        const int32_t ticket_before = walk.ticket;
        int next_state = walk_step<TURNS>(a, walk, &next);     // kWalkNeedTicket: decided after the barrier
        next_state = __builtin_amdgcn_readfirstlane(next_state);   // uniform anyway: scalar branches below
        next = __builtin_amdgcn_readfirstlane(next);
        bool nxt_redo = walk.redo;
        loaded = next_state == kWalkTile;
        if (loaded) nxt = start_tile(next);

        __builtin_amdgcn_s_setprio(0);
        // ---- (e) ranks of the entries ----
        uint32_t rank[kIters];
        const uint32_t wave_total = vector_ranks(mask, rank);
        if (lane == 0) s_wave_total[parity][wave] = wave_total;
        __syncthreads();
        if (accept_now) walk_accept(a, walk, (uint32_t)__builtin_amdgcn_readfirstlane(s_ticket[parity]));
        const int n_announced = __builtin_amdgcn_readfirstlane(s_nready[parity]);
        uint32_t wave_excl = 0, tile_total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            uint32_t c = s_wave_total[parity][w];
            if (w < wave) wave_excl += c;
            tile_total += c;
        }
        tile_total = (uint32_t)__builtin_amdgcn_readfirstlane((int)tile_total);   // uniform: scalar bookkeeping below
        parity ^= 1;

        // publish the count: a serving wave turns it into this tile's prefix
        if (threadIdx.x == 0 && !cur_redo)
            desc_store(a.tile_desc + tile, (kStatusAggregate << kStatusShift) | tile_total);

        // copy out what was announced, while the next tile's loads are on their way; not before tiles are counted ahead, since
        // others wait for those counts
        const bool no_slot = q_len == kQueue, no_place = ring_used + tile_total > (uint32_t)kRing, crowded = no_slot || no_place;
        const bool ahead = ROSE_COUNT_AHEAD && !a.adjacent && no_place && q_len < a.batch;      // see below
        if (n_announced > 0 && !ahead) {
            const uint32_t freed = copy_out(n_announced, s_excl[parity ^ 1], true);
            pop(n_announced, freed);
            if (crowded) __syncthreads();              // what is parked next may take the places of what is being copied
            if (no_slot) {                             // and there is no lane for it (the poll in flight is forgotten)
                move_lanes();
                n_polled = 0;
            }
        }

        // Room to park?  Making room may wait, and nothing may wait, or be walked again, while a ticket is on its way.
        if (ticket_first(walk, ticket_out, q_len == kQueue || ring_used + tile_total > (uint32_t)kRing, ahead)) settle_ticket();
        // A same-group ticket has just been accepted: nothing may wait now.  This tile is not
        // parked; it is walked again after the count-only pass at the end of the iteration.
        // Tiles so dense that the ring does not hold a ticket's worth (fewer tiles are parked than a
        // ticket has, and there is no room for this one), with tiles of the current ticket still
        // uncounted: waiting now would make every worker of a later group wait for those counts
        // while this one waits for the prefix of the same ticket's first tile, and the groups of
        // workers would take turns instead of running side by side.  So the rest of the ticket is
        // counted first and the ticket's tiles, this one included, are walked again without
        // publishing, exactly as for a same-group pair (below).
        bool dense = false;
#if ROSE_COUNT_AHEAD
        // the next tile is of the same ticket: not all of the ticket is counted
        const bool mid_ticket = !walk.careful && !cur_redo && !walk.redo && next_state == kWalkTile &&
                                walk.ticket == ticket_before;
        if (a.adjacent) {
            // A ticket's tiles are neighbours, so its uncounted tiles may lie in the very block whose
            // prefixes a wait would be for: in the middle of a ticket nothing may wait at all.  First
            // look, without waiting, whether prefixes have arrived since the last poll.
            if (__builtin_expect(mid_ticket && (q_len == kQueue || ring_used + tile_total > (uint32_t)kRing), 0)) {
                if (q_len > 0) drain(kDrainReady);
                dense = q_len == kQueue || ring_used + tile_total > (uint32_t)kRing;
            }
        } else if (__builtin_expect(ahead, 0)) {
            // (also where the announced tiles would make room: their neighbours will not have left in time for this
            // ticket's next tiles, whose wait would then hold up all others.  And they stay where they are: their stores would
            // hold up the counts.  Eight 7B-style layers with embedding and head, TP4, 40 / 50 %, ms: by the room they leave 4.60 /
            // 6.06, by the room there was and copied out first 3.54 / 4.25, this way 3.38 / 3.86; 60 / 80 % 3.82 / 4.17 either way)
            dense = mid_ticket;
        }
#endif
        const bool skip = walk.careful || dense;
        if (!skip) {
            while (q_len == kQueue || ring_used + tile_total > (uint32_t)kRing) drain(kDrainOldest);
        }

        const int32_t chain_last = a.chain_first[cur.shard + 1] - 1;
        const int32_t seg = cur.seg;
        if (!skip) {
            // park the entries: ring slot = ring_head + rank inside the tile
            const uint32_t base = ring_head + wave_excl;
#pragma unroll
            for (int j = 0; j < kIters; ++j) {
                uint32_t m = mask[j];
                uint32_t slot = base + rank[j];
                const uint32_t number0 = cur.out_base + t_off + (uint32_t)(j * 64) * kVec;
                while (m) {
                    const uint32_t e = __ffs(m) - 1;
                    m &= m - 1;
                    uint32_t number = (number0 + e) << 16;         // (bit 31 counts only where it is an escape)
                    if constexpr (FORMED) number = (number & 0x7FFF0000u) | (escaped >> (8 * j + e)) << 31;
                    s_ring[slot & (kRing - 1)] = number | (pick16(nv[j], e) & 0xFFFFu);
                    if constexpr (ARITH) s_was[slot & (kRing - 1)] = (uint16_t)pick16(ov[j], e);
                    ++slot;
                }
            }
            if (threadIdx.x == 0) {
                const int slot = (q_head + q_len) & (kQueue - 1);
                s_q_count[slot] = tile_total;
                s_q_off[slot] = ring_head;
                s_q_base[slot] = cur.out_base;
                s_q_piece[slot] = cur.piece;
                s_q_shard[slot] = cur.shard;
                s_q_seg[slot] = seg;
                s_q_last[slot] = tile == chain_last;
            }
            if (wave == 0 && lane == q_len + n_gone) {
                wq_tile = tile;
                wq_w = 0;
            }
            ++q_len;
            ring_used += tile_total;
            ring_head = (ring_head + tile_total) & (kRing - 1);
        }

        // Sender refresh (W_{t-1} <- W_t for what this tile covers): only now that the tile is known
        // not to be walked again, and never for replicated tensors, which other destinations' tiles
        // still have to read (a small kernel after this one copies those).
        if constexpr (REFRESH) {
            if (!skip && !(cur.vec & 2u)) {
                const TileCtx c = tile_ctx(a, __builtin_amdgcn_readfirstlane(tile));
                uint16_t *ob = const_cast<uint16_t *>(c.old_base);
                // Whole 64-byte lines (four lanes' vectors), or 128-byte ones where changes are few, go back if
                // anything in them has changed: the memory takes whole lines far better than parts of
                // them, and better than the whole tile at any density (twelve 8B-style layers, single
                // vectors up to 160 entries a tile and whole tiles above / 64-byte / 128-byte lines: 3.91 / 3.44 / 3.35
                // ms at 1 %, 4.21 / 3.75 / 3.70 at 2 %, 4.15 / 4.07 / 4.10 at 5 %, 4.47 / 4.47 / 4.47 at 12 %).
                const bool wide = tile_total <= (uint32_t)kRefreshWide;
#pragma unroll
                for (int j = 0; j < kIters; ++j) {
                    uint32_t line = or_of_four(mask[j]);
                    const uint32_t pair = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)line, 0x141, 0xf, 0xf, true);  // row_half_mirror
                    if (wide) line |= pair;
                    if (line) {
                        const uint32_t k = c.k_tile + t_off + (uint32_t)(j * 64) * kVec;
                        bool one = (cur.vec & 1u) && (c.limit == 0xFFFFFFFFu || !vector_moved(c.limit, k));
                        if (cur.vec & 4u) {
                            uint32_t q;
                            one = one && split_left(c.pc, k, &q) >= (uint32_t)kVec;
                        }
                        if (one) {
                            u32x4 w = {nv[j].x, nv[j].y, nv[j].z, nv[j].w};     // unchanged elements keep their bits
                            __builtin_nontemporal_store(w, reinterpret_cast<global_u32x4 *>(reinterpret_cast<uintptr_t>(ob + src_index(c.pc, k, true))));
                        } else {
                            uint32_t m = mask[j];
                            while (m) {
                                const uint32_t e = __ffs(m) - 1;
                                m &= m - 1;
                                ob[src_index(c.pc, k + e, false)] = (uint16_t)pick16(nv[j], e);
                            }
                        }
                    }
                }
            }
        }

        // The rare cases that the next tile could not be named before the barrier above, or that a
        // same-group ticket has arrived: settle them now; the next tile's loads are then issued at
        // the top of the next iteration.
        bool late = false;
        bool redo_cur = skip;                          // this iteration's tile was not parked
        for (;;) {
            if (walk.careful || dense) {
                // the ticket in use (tA) and the one just accepted (tB) are of one group: publish
                // the counts of everything not yet published, then walk those tiles again.  The
                // dense case (above) is the same with no second ticket: the rest of tA is counted
                // and tA is walked again from this iteration's tile on.
                const bool pair = walk.careful;
                const int32_t tA = walk.ticket, tB = walk.next_ticket;
                const int32_t j_end = pair ? 2 * a.batch : a.batch;
                int32_t j_from = a.batch;               // first slot of tA to walk again
                if (redo_cur)
                    for (int32_t j = 0; j < a.batch; ++j)
                        if (ticket_tile<TURNS>(a, tA, j) == tile) j_from = j;
                redo_cur = false;
                // slot j_from itself is published (it is this iteration's tile); when tA is used up
                // (j_from = kBatch) every slot of tB is still to be counted
#pragma unroll 1
                for (int32_t j = j_from < a.batch ? j_from + 1 : a.batch; j < j_end; ++j) {
                    const int32_t t = j < a.batch ? ticket_tile<TURNS>(a, tA, j) : ticket_tile<TURNS>(a, tB, j - a.batch);
                    if (t >= 0) publish_count(t);
                }
                __syncthreads();
                if (threadIdx.x == 0)                  // diagnostic words: how often each happened
                    __hip_atomic_fetch_add(a.abort_flag + (pair ? kWsCarefulWord : kWsAheadWord), 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                walk.careful = false;
                dense = false;
                walk.redo = true;
                walk.redo_through = pair ? tB : tA;
                walk.j = j_from - 1;
                next_state = walk_step<TURNS>(a, walk, &next);
                late = true;
            }
            if (next_state != kWalkNeedTicket) break;
            if (!walk.have_next && !walk.exhausted) {
                settle_ticket();
                if (walk.careful) continue;
            }
            next_state = walk_step<TURNS>(a, walk, &next);
            late = true;
        }
        if (late) {
            nxt_redo = walk.redo;
            loaded = false;
        }
        if (next_state == kWalkDone) break;
        cur_redo = nxt_redo;
        tile = next;
    }
    while (q_len > 0) drain(kDrainAll);
}

// The instantiations get their own register budgets: 4 waves per SIMD (128 VGPRs) fit the bf16
// kernels without spills; the fp32-master kernels hold twice the raw data, and those that form arithmetic
// payloads keep old and new patterns side by side (and half as much LDS again): those get 3
// (the one that does all three at once: 2).  Arithmetic payloads are formed of the compacted entries: formed of every
// element, with 4 waves, they are 400 instructions a wave and tile for some 30 that are needed (eight
// 7B-style layers, TP4, 1 / 5 / 10 %: 1428 / 1603 / 1822 us, this way 1311 / 1516 / 1733; with refresh 2 % 2050 and
// 1996; two 32B-style layers of fp32 masters, 1.6 / 5 %: 2772 / 3059 and 2645 / 2972, with refresh 3939 and 3688).
// Where much changes that turns for bf16 weights without refresh, whose payloads are then formed of every element
// (encode_elements_kernel, see kElementsPpm).
// REFRESH = 1 also writes the new bf16 values over the old ones; ARITH = 1 emits arithmetic payloads.
template <int NEW_F32, int REFRESH, int ARITH> __global__ void encode_kernel(EncodeArgs a);
#define ROSE_ENCODE_KERNEL(F32, REFRESH, ARITH, WAVES, VGPRS)                                                         \
    template <>                                                                                                       \
    __global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES), amdgpu_num_vgpr(VGPRS))) \
    void encode_kernel<F32, REFRESH, ARITH>(EncodeArgs a) {                                                           \
        encode_body<F32, REFRESH, ARITH>(a);                                                                          \
    }
ROSE_ENCODE_KERNEL(0, 0, 0, 4, kNumVgpr0)
ROSE_ENCODE_KERNEL(0, 1, 0, 4, kNumVgpr0)
ROSE_ENCODE_KERNEL(0, 0, 1, 3, kNumVgpr1)
ROSE_ENCODE_KERNEL(0, 1, 1, 3, kNumVgpr1)
ROSE_ENCODE_KERNEL(1, 0, 0, 3, kNumVgpr1)
ROSE_ENCODE_KERNEL(1, 1, 0, 3, kNumVgpr1)
ROSE_ENCODE_KERNEL(1, 0, 1, 3, kNumVgpr1)
ROSE_ENCODE_KERNEL(1, 1, 1, 2, kNumVgpr2)
#undef ROSE_ENCODE_KERNEL
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 4), amdgpu_num_vgpr(kNumVgpr0)))
void encode_elements_kernel(EncodeArgs a) {
    encode_body<0, 0, 2>(a);
}

// ---------------------------------------------------------------------------------------------
// encode in two launches, without tickets (launch_encode says when).  Nothing waits for another workgroup, so there
// is nothing to reset, no ticket, no serving wave and no drain at the end.  The first launch reads every tile, one
// workgroup a tile, and counts its changes; the second adds up the counts in front of its tiles and writes the
// entries.  Two forms:
//   staged    the first launch parks a tile's compacted entries in the tile's slot of the workspace, the second copies
//             them to the bucket.  A tile that holds more than its slot does parks nothing and is read again.
//   read again   no slots: the second launch reads every tile a second time.
// ---------------------------------------------------------------------------------------------
enum : int { kTickets = 0, kStaged = 1, kReadAgain = 2, kTicketsElements = 3 };
// The header is this call's, whatever the workspace held: no wait gave up, no tile was counted ahead of one, no tickets.
__device__ __forceinline__ void write_header(const EncodeArgs &a, uint32_t form) {
    if (threadIdx.x <= kWsAheadWord) a.abort_flag[threadIdx.x] = 0;
    if (threadIdx.x == kWsTilesWord) a.abort_flag[kWsTilesWord] = (uint32_t)a.n_tiles;
    if (threadIdx.x == kWsFormWord) a.abort_flag[kWsFormWord] = form;
    if (threadIdx.x == kWsFormWord + 1) *a.ticket = 0;
}

constexpr int kGroupMost = 16;           // tiles a workgroup of the second launch copies out at most

// Refresh: the lines of the tile in which anything changed, from registers.  Whole 64-byte lines, or 128-byte ones where
// changes are few (see encode_body), non-temporal (16 M
// weights at 5 %, inputs from memory: 48.9 us with ordinary stores, 35.4 this way; with the inputs in the caches the same).
__device__ __forceinline__ void refresh_tile(const TileCtx &c, uint32_t t_off, bool wide, const uint32_t (&mask)[kIters],
                                             const uint4 (&n)[kIters]) {
    uint16_t *ob = const_cast<uint16_t *>(c.old_base);
#pragma unroll
    for (int j = 0; j < kIters; ++j) {
        const uint32_t k = c.k_tile + t_off + (uint32_t)(j * 64) * kVec;
        uint32_t q, m = mask[j], line = or_of_four(m);
        const uint32_t pair = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)line, 0x141, 0xf, 0xf, true);      // row_half_mirror
        if (wide) line |= pair;
        if (!line) continue;
        if ((c.vec & 1u) && !vector_moved((uint32_t)c.pc.len, k) && !((c.vec & 4u) && split_left(c.pc, k, &q) < (uint32_t)kVec)) {
            gstore16_stream(ob + src_index(c.pc, k, true), n[j]);
        } else {
            while (m) {
                const uint32_t e = __ffs(m) - 1;
                m &= m - 1;
                ob[src_index(c.pc, k + e, false)] = (uint16_t)pick16(n[j], e);
            }
        }
    }
}

// The changed elements of a vector go to consecutive places in LDS: offset in the tile << 16 | new pattern, and for
// arithmetic payloads the old pattern beside it.
template <int ARITH>
__device__ __forceinline__ void park_vector(uint32_t in_tile, uint32_t m, uint4 o, uint4 n, uint32_t at, uint32_t *s_entry,
                                            uint16_t *s_was) {
    while (m) {
        const uint32_t e = __ffs(m) - 1;
        m &= m - 1;
        s_entry[at] = ((in_tile + e) << 16) | pick16(n, e);
        if constexpr (ARITH) s_was[at] = (uint16_t)pick16(o, e);
        ++at;
    }
}
template <int NEW_F32, int REFRESH, int ARITH>
__global__ __launch_bounds__(kThreads) void stage_tiles_kernel(EncodeArgs a, uint16_t *counts, uint32_t *slots, int32_t slot_size,
                                                               int32_t stream) {
    __shared__ uint32_t s_entry[kStageSlot];
    __shared__ uint16_t s_was[ARITH ? kStageSlot : 1];
    __shared__ uint32_t s_cnt[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t tile = (int32_t)blockIdx.x;
    const TileCtx c = tile_ctx(a, tile);
    const uint32_t t_off = (uint32_t)wave * kWaveSpan + (uint32_t)lane * kVec;
    uint4 o[kIters], n[kIters];
    uint32_t mask[kIters], rank[kIters];
    load_tile_pair<NEW_F32>(c, t_off, o, n);
    tile_masks(c, t_off, o, n, mask);
    const uint32_t wave_total = vector_ranks(mask, rank);
    if (lane == 0) s_cnt[wave] = wave_total;
    __syncthreads();
    uint32_t wave_excl = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) wave_excl += s_cnt[w];
        total += s_cnt[w];
    }
    if (threadIdx.x == 0) counts[tile] = (uint16_t)total;
    if (tile == 0) write_header(a, kStaged);
    total = (uint32_t)__builtin_amdgcn_readfirstlane((int)total);
    if (total == 0 || total > (uint32_t)slot_size) return;
#pragma unroll
    for (int j = 0; j < kIters; ++j)                           // (offsets from where an unshifted tile would begin)
        park_vector<ARITH>(t_off + (uint32_t)(j * 64) * kVec - c.shift, mask[j], o[j], n[j],
                           wave_excl + rank[j], s_entry, s_was);
    if constexpr (REFRESH) {
        if (!(c.pc.flags & kPieceReplicated)) refresh_tile(c, t_off, total <= (uint32_t)kRefreshWide, mask, n);
    }
    __syncthreads();
    uint32_t *slot = slots + (size_t)tile * (uint32_t)slot_size;
    for (uint32_t k = threadIdx.x; k < total; k += kThreads) {
        const uint32_t entry = parked<ARITH>(k, s_entry, s_was);
        if (stream) __builtin_nontemporal_store(entry, slot + k);
        else slot[k] = entry;
    }
}

// First launch, nothing parked.
template <int NEW_F32>
__global__ __launch_bounds__(kThreads) void count_tiles_kernel(EncodeArgs a, uint16_t *counts) {
    __shared__ uint32_t s_cnt[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const TileCtx c = tile_ctx(a, (int32_t)blockIdx.x);
    const uint32_t t_off = (uint32_t)wave * kWaveSpan + (uint32_t)lane * kVec;
    uint4 o[kIters], n[kIters];
    uint32_t mask[kIters];
    load_tile_pair<NEW_F32>(c, t_off, o, n);
    tile_masks(c, t_off, o, n, mask);
    uint32_t cnt = 0;
#pragma unroll
    for (int j = 0; j < kIters; ++j) cnt += __popc(mask[j]);
    const uint32_t wave_cnt = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(cnt), 63);
    if (lane == 0) s_cnt[wave] = wave_cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int w = 0; w < kWaves; ++w) total += s_cnt[w];
        counts[blockIdx.x] = (uint16_t)total;
    }
    if (blockIdx.x == 0) write_header(a, kReadAgain);
}

// What the second launch needs of a tile besides its count.
struct EmitTile {
    uint32_t start;     // entries of the workgroup's earlier tiles
    uint32_t base;      // local index of the tile's first element; with a piece, the element's number inside it
    int32_t piece;      // -1, or the piece whose table entry maps element numbers to local indices
};

// local index of the element at number `k` of a piece whose local indices come in strided runs (runs of one element
// have no magic divisor: the quotient is the number itself)
__device__ __forceinline__ uint32_t strided_local(const Piece &p, uint32_t k) {
    const uint32_t run = (uint32_t)p.run;
    const uint32_t q = run == 1u ? k : (__umulhi(k, p.magic) >> p.shift);
    return (uint32_t)p.local_base + q * (uint32_t)p.lstride + (k - q * run);
}

// A tile read (again), compacted in LDS a PART-th of its waves at a time, written.  `before` is called while the loads
// are on their way and returns the wave's share of the entries in front of the tile, besides the `excl` that are known;
// with SEGMENTS the tile's segment ends are written too.
template <int NEW_F32, int REFRESH, int ARITH, int PARTS, bool SEGMENTS, typename BEFORE>
__device__ __forceinline__ void emit_read(const EncodeArgs &a, int32_t tile, u64 excl, BEFORE before, uint32_t *s_entry,
                                          uint16_t *s_was, uint32_t *s_before, uint32_t *s_cnt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const TileCtx c = tile_ctx(a, tile);
    const uint32_t t_off = (uint32_t)wave * kWaveSpan + (uint32_t)lane * kVec;
    uint4 o[kIters], n[kIters];
    load_tile_pair<NEW_F32>(c, t_off, o, n);
    const uint32_t share = before(c);
    uint32_t mask[kIters], rank[kIters];
    tile_masks(c, t_off, o, n, mask);
    const uint32_t wave_total = vector_ranks(mask, rank);
    if (lane == 0) {
        s_before[wave] = share;
        s_cnt[wave] = wave_total;
    }
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        excl += s_before[w];
        total += s_cnt[w];
    }
    const BucketDev b = a.bucket[c.pc.shard];
    if (SEGMENTS && threadIdx.x == 0) {
        if ((c.pc.flags & kPieceFirst) && tile == c.pc.first_tile) b.seg_off[c.pc.tensor] = (int64_t)excl;
        if (tile == a.chain_first[c.pc.shard + 1] - 1) b.seg_off[a.n_tensors] = (int64_t)(excl + total);
    }
    const bool dst_strided = (c.pc.flags & kPieceDstStrided) != 0;
#pragma unroll 1
    for (int part = 0; part < kWaves; part += kWaves / PARTS) {
        if (part) __syncthreads();                             // the part before has been written
        uint32_t at0 = 0, here = 0;
#pragma unroll
        for (int w = 0; w < kWaves / PARTS; ++w) {
            if (part + w < wave) at0 += s_cnt[part + w];
            here += s_cnt[part + w];
        }
        if (PARTS == 1 || (wave >= part && wave < part + kWaves / PARTS)) {
#pragma unroll
            for (int j = 0; j < kIters; ++j) {
                const uint32_t in_tile = t_off + (uint32_t)(j * 64) * kVec;
                if constexpr (ARITH && PARTS == 1) {           // payloads of all elements: fewer steps one behind the other
                    uint32_t esc8, m = mask[j], at = at0 + rank[j];
                    const uint4 pay = arith_vec(o[j], n[j], &esc8);
                    while (m) {
                        const uint32_t e = __ffs(m) - 1;
                        m &= m - 1;
                        s_entry[at++] = ((in_tile + e) << 16) | pick16(pay, e) | ((esc8 >> e) << 31);
                    }
                } else {
                    park_vector<ARITH>(in_tile, mask[j], o[j], n[j], at0 + rank[j], s_entry, s_was);
                }
            }
        }
        if constexpr (REFRESH) {
            if ((PARTS == 1 || part == 0) && !(c.pc.flags & kPieceReplicated)) refresh_tile(c, t_off, false, mask, n);
        }
        __syncthreads();
        const uint32_t phase = (uint32_t)excl & 31u;           // lined up with the bucket's lines, see copy_out
        for (uint32_t kk = threadIdx.x; kk < here + phase; kk += kThreads) {
            const uint32_t k = kk - phase;
            const u64 pos = excl + k;
            if (kk >= phase && pos < (u64)b.capacity) {
                const uint32_t entry = parked<(ARITH && PARTS > 1)>(k, s_entry, s_was);
                uint32_t local = c.k_tile + ((entry >> 16) & (uint32_t)(kTile - 1));
                uint32_t q = 0;                                // (a piece with contiguous local indices: run 0 of a strided one)
                if (dst_strided) q = c.pc.run == 1 ? local : (__umulhi(local, c.pc.magic) >> c.pc.shift);
                local = (uint32_t)c.pc.local_base + q * (uint32_t)c.pc.lstride + (local - q * (uint32_t)c.pc.run);
                b.idx[pos] = (int32_t)(local | (ARITH ? entry & 0x80000000u : 0u));
                b.val[pos] = (uint16_t)entry;
            }
        }
        excl += here;
    }
}

// This thread's share of the counts of tiles begin .. end - 1, added up over the wave.
__device__ __forceinline__ uint32_t wave_share_of_counts(const uint16_t *counts, int32_t begin, int32_t end) {
    const uint16_t *p = counts + begin;
    const uint32_t m = (uint32_t)(end - begin), whole = m / 8;
    uint32_t sum = 0;
    for (uint32_t i = threadIdx.x; i < whole; i += kThreads) {
        const uint4 v = gload16(p + i * 8);
        sum += (v.x & 0xFFFFu) + (v.x >> 16) + (v.y & 0xFFFFu) + (v.y >> 16) + (v.z & 0xFFFFu) + (v.z >> 16) + (v.w & 0xFFFFu) +
               (v.w >> 16);
    }
    if (threadIdx.x < m % 8) sum += gload_u16(p + whole * 8 + threadIdx.x);
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(sum), 63);
}

// Second launch, every tile read again: one workgroup a tile.
template <int NEW_F32, int REFRESH, int ARITH>
__global__ __launch_bounds__(kThreads) void emit_tiles_kernel(EncodeArgs a, const uint16_t *counts) {
    __shared__ uint32_t s_entry[kTile];
    __shared__ uint32_t s_before[kWaves], s_cnt[kWaves];
    const int32_t tile = (int32_t)blockIdx.x;
    emit_read<NEW_F32, REFRESH, ARITH, 1, true>(
        a, tile, 0, [&](const TileCtx &c) { return wave_share_of_counts(counts, a.chain_first[c.pc.shard], tile); }, s_entry,
        nullptr, s_before, s_cnt);
}

// A workgroup copies out 2^group_log2 neighbouring tiles of one chain, as far as they are in their slots.  Returns whether
// the group is a single tile that is not; *tile and *excl are then its number and the entries in front of it.
template <int ARITH>
__device__ __forceinline__ bool copy_group(const EncodeArgs &a, const uint16_t *counts, const uint32_t *slots, int32_t slot_size,
                                           int32_t group_log2, uint32_t *s_before, int32_t *tile, u64 *excl_out) {
    __shared__ EmitTile s_tile[kGroupMost + 1];
    __shared__ uint32_t s_over;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t group = 1 << group_log2;
    const int32_t first = (int32_t)blockIdx.x << group_log2, blk = first / kBlock;
    int32_t shard = 0;
    while (blk >= a.block_first[shard + 1]) ++shard;
    const int32_t chain_begin = a.chain_first[shard], chain_end = a.chain_first[shard + 1];
    const int32_t t0 = chain_begin + first - a.block_first[shard] * kBlock;
    if (t0 >= chain_end) return false;
    const int32_t n = chain_end - t0 < group ? chain_end - t0 : group;
    const BucketDev b = a.bucket[shard];

    // lane i of wave 0: tile t0 + i
    const bool mine = wave == 0 && lane < n;
    int32_t my_piece = 0;
    uint32_t count = 0, start = 0, early = 0;
    if (mine) {
        my_piece = a.tile_piece[t0 + lane];
        count = gload_u16(counts + t0 + lane);
    }
    // a single tile's first entries need not wait for their count
    const uint32_t *from = slots + (size_t)t0 * (uint32_t)slot_size;
    if (group == 1 && (uint32_t)slot_size >= (uint32_t)kThreads) early = gload_u32(from + threadIdx.x);
    // entries of the chain's earlier tiles (as many as all tiles have elements at most: they fit 32 bits, see kStageMostTiles)
    const uint32_t before = wave_share_of_counts(counts, chain_begin, t0);
    if (lane == 0) s_before[wave] = before;
    int32_t seg = -1;                                          // tensor whose segment starts with the tile
    if (wave == 0) {
        EmitTile t = {0, 0, -1};
        if (mine) {
            const Piece *pc = a.pieces + my_piece;
            const uint32_t k_tile = (uint32_t)(t0 + lane - pc->first_tile) * (uint32_t)kTile;
            t.piece = (pc->flags & kPieceDstStrided) ? my_piece : -1;
            t.base = k_tile + (t.piece < 0 ? (uint32_t)pc->local_base : 0u);
            if ((pc->flags & kPieceFirst) && t0 + lane == pc->first_tile) seg = pc->tensor;
        }
        const uint32_t incl = wave_incl_scan(count);
        start = incl - count;
        t.start = start;
        if (lane <= group) s_tile[lane] = t;
        const u64 over = __ballot(count > (uint32_t)slot_size);
        if (lane == 0) s_over = over != 0;
    }
    __syncthreads();
    u64 excl = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) excl += s_before[w];
    if (mine) {
        if (seg >= 0) b.seg_off[seg] = (int64_t)(excl + start);
        if (t0 + lane == chain_end - 1) b.seg_off[a.n_tensors] = (int64_t)(excl + start + count);
    }

    auto write = [&](u64 pos, uint32_t entry, uint32_t base, int32_t piece) {
        if (pos >= (u64)b.capacity) return;
        uint32_t local = base + (uint32_t)((int32_t)(entry << 1) >> 17);       // (negative in the first tile of a shifted piece)
        if (piece >= 0) local = strided_local(a.pieces[piece], local);
        __builtin_nontemporal_store((int32_t)(local | (ARITH ? entry & 0x80000000u : 0u)), b.idx + pos);
        __builtin_nontemporal_store((uint16_t)entry, b.val + pos);
    };
    // entries begin .. end - 1 of the workgroup's, from their slots; lined up with the bucket's lines, see copy_out
    constexpr int U = 4;                                       // loads a thread has in flight
    auto copy = [&](uint32_t begin, uint32_t end) {
        const uint32_t phase = (uint32_t)(excl + begin) & 31u;
        for (uint32_t kk = threadIdx.x; kk < end - begin + phase; kk += kThreads * U) {
            uint32_t x[U], base[U];
            int32_t piece[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t r = kk + (uint32_t)(u * kThreads) - phase;      // (wraps below phase)
                const uint32_t k = r < end - begin ? begin + r : begin;
                uint32_t s = 0;
                for (int32_t h = group >> 1; h >= 1; h >>= 1) s += s_tile[s + (uint32_t)h].start <= k ? (uint32_t)h : 0u;
                const EmitTile t = s_tile[s];
                base[u] = t.base;
                piece[u] = t.piece;
                x[u] = gload_u32(from + (size_t)s * (uint32_t)slot_size + (k - t.start));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t r = kk + (uint32_t)(u * kThreads) - phase;
                if (r < end - begin) write(excl + begin + r, x[u], base[u], piece[u]);
            }
        }
    };
    if (!s_over) {
        uint32_t all = s_tile[group].start, done = 0;
        if (group == 1 && (uint32_t)slot_size >= (uint32_t)kThreads) {
            done = all < (uint32_t)kThreads ? all : (uint32_t)kThreads;
            if (threadIdx.x < done) write(excl + threadIdx.x, early, s_tile[0].base, s_tile[0].piece);
        }
        if (all > done) copy(done, all);
        return false;
    }
    *tile = t0;
    *excl_out = excl;
    if (group == 1) return true;
    for (int32_t i = 0; i < n; ++i) {
        const uint32_t begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tile[i].start);
        const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tile[i + 1].start);
        if (end > begin && end - begin <= (uint32_t)slot_size) copy(begin, end);
    }
    return false;
}

// Second launch, staged: the first group_wgs workgroups copy out groups of tiles.  A tile past its slot is read again: by
// its workgroup, if that has no other; else by one of those behind, to which such tiles are dealt so that neighbours go to
// different ones.  Changes that lie close together had one workgroup read 2 to 16 tiles one behind the other: 2 % of
// 192 MiB, all in neighbouring tiles, 117 us that way and 42 this way; of 480 MiB 238 and 88; of 1200 MiB 349 and 206;
// all of 192 MiB at 30 % 109 and 84.  With 2048 workgroups for it, what the device holds at once, 384 MiB at 30 % take 176 us,
// with kOverWgs 160.  Where no tile is past its slot they look at their counts and end (850 MiB 154 us with and without).
constexpr int kOverWgs = 8192;
static_assert((kStageMostTiles + kOverWgs - 1) / kOverWgs <= 64, "a wave looks at a workgroup's tiles");
template <int NEW_F32, int REFRESH, int ARITH>
__global__ __launch_bounds__(kThreads) void emit_staged_kernel(EncodeArgs a, const uint16_t *counts, const uint32_t *slots,
                                                              int32_t slot_size, int32_t group_log2, int32_t group_wgs) {
    __shared__ uint32_t s_entry[kTile / 2];
    __shared__ uint16_t s_was[ARITH ? kTile / 2 : 1];
    __shared__ uint32_t s_before[kWaves], s_cnt[kWaves];
    const bool grouped = (int32_t)blockIdx.x < group_wgs;
    int32_t mine = 0;                                          // a tile for each bit of `over`
    u64 over = 1, excl = 0;
    if (grouped) {
        if (!copy_group<ARITH>(a, counts, slots, slot_size, group_log2, s_before, &mine, &excl)) return;
    } else {
        const int32_t wgs = (int32_t)gridDim.x - group_wgs;
        mine = (int32_t)blockIdx.x - group_wgs + (int32_t)(threadIdx.x & 63) * wgs;
        over = __ballot(mine < a.n_tiles && gload_u16(counts + (mine < a.n_tiles ? mine : 0)) > (uint32_t)slot_size);
    }
    for (; over; over &= over - 1) {
        const int32_t tile = __builtin_amdgcn_readlane(mine, __ffsll((unsigned long long)over) - 1);
        __syncthreads();                                       // s_before and the tile before's s_entry have been read
        emit_read<NEW_F32, REFRESH, ARITH, 2, false>(
            a, tile, excl,
            [&](const TileCtx &c) { return grouped ? 0u : wave_share_of_counts(counts, a.chain_first[c.pc.shard], tile); },
            s_entry, s_was, s_before, s_cnt);
    }
}

// Replicated tensors after an encode with refresh: old <- bf16(new), whole tensors (they are small).
__global__ __launch_bounds__(256) void refresh_replicated_kernel(const int32_t *list, const int64_t *numel, int32_t n,
                                                                 void *const *old_ptrs, const void *const *new_ptrs,
                                                                 int new_is_f32) {
    for (int32_t i = blockIdx.y; i < n; i += gridDim.y) {
        const int32_t t = list[i];
        uint16_t *o = static_cast<uint16_t *>(old_ptrs[t]);
        const int64_t cnt = numel[i];
        for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < cnt; k += (int64_t)gridDim.x * blockDim.x)
            o[k] = new_is_f32 ? (uint16_t)rne_bf16(static_cast<const uint32_t *>(new_ptrs[t])[k])
                              : static_cast<const uint16_t *>(new_ptrs[t])[k];
    }
}

// ---------------------------------------------------------------------------------------------
// apply (App. F S2D): every entry's value goes to its local index of the receiver's copy.
//
// Scattered 2-byte stores reach memory as byte-masked partial writes of the lines they touch,
// which the memory side turns into read-modify-writes of its own.  Between about 1 and 8 % of
// the elements the kernel does better to do the read-modify-write itself, one 64-byte line at a time,
// with 128-bit accesses marked non-temporal (a line is touched once per launch; 7B-style workload at 5 %,
// one shard: 1.22 ms, with direct stores 1.37): a wave takes 64 consecutive entries (ascending local index inside a segment,
// so the entries of a line are neighbours), finds the distinct lines they touch, loads those lines
// into LDS, patches the entries in, and stores the lines back whole.
//
// A line's entries may straddle two waves' chunks (a line holds at most 32 entries, a chunk 64):
// the line belongs to the wave that holds its FIRST entry; that wave also applies the entries of
// its last line that lie in the next chunk, and the next wave skips them.  This division holds whether
// a chunk's entries then go by whole lines or by direct stores.  Lines are lines of the ADDRESS, whatever
// element a tensor starts at.  Entries whose own 16-byte part of the line is not entirely inside the tensor
// (the first and last few elements of a tensor that starts or ends between multiples of 16 bytes; the part
// may hold elements of its neighbour in a packed buffer) are stored directly; the line path never touches
// those bytes.
//
// What bounds it between 1 and 8 %: the memory's rate for this pattern (reads come in 128-byte units, writes
// in 64: 5.9 TB/s of them at 5 %), and below it the time a chunk's rounds of loads take, so registers and
// waits matter: the line loads stand under no condition, which would make the compiler wait for one before
// the next (1.50 against 1.38 ms at 8 %), and the kernel keeps to 64 registers (a version that spilled a few
// took 1.45 ms at 5 % instead of 1.17).
// ---------------------------------------------------------------------------------------------
// How a launch is laid out is chosen by what the bucket can hold, by itself and against the elements of the shard;
// how its chunks are written, by what they hold.
//   Workgroups of 8 waves, and of 4 up to 8192 chunks, which do not fill the device: 328 workgroups of 8 leave some
//   CUs with twice the work of the others (4096 x 4096, one shard, 1 %: 8.1 us with 8, 6.9 with 4; 0.5 %: 5.5 and 4.6).
//   below 1/24   apply_kernel<1>, 4 waves per SIMD: where the touched lines lie apart the memory does better with
//                fewer of them in flight (7B-style workload, one shard, against 8 waves: 0.79 and 0.84 ms at 2 %,
//                0.67 and 0.71 at 1.5 %, 0.55 and 0.56 at 1 %; buckets of a 67 M shard with room for 3.75 %: 36.3 and
//                38.2 us; with room for 4.4 % it loses 5 %).  Not up to 8192 chunks: fewer waves are in flight anyway,
//                and lone entries do better by lines (67 M elements, 0.1 %: 4.2 us, 5.3 with it).
//   below 1/20   apply_kernel<0>, 5 waves per SIMD in workgroups of 4 (against 8 in workgroups of 8, with room for
//                4.75 %: 1.045 and 1.078 ms, 67 M elements 38.5 and 40.5 us; with room for 5.6 % 134 - 268 M elements
//                lose 8 %)
//   up to 1/3    apply_kernel<0>, 8 waves per SIMD, and twice kApplyBlocks workgroups: a wave that takes a second
//                chunk waits for the stores of its first, but a wave that finds none costs too (one shard with 1x /
//                2x / 4x: 1.21 / 1.16 / 1.16 ms at 5 %, 1.62 / 1.53 / 1.40 at 12 %; at 0.2 % with room for 10 %:
//                178 / 203 / 259 us)
//   above        kApplyBlocks workgroups (of 8 waves)
// A bucket that turns out to hold 1/7 of the shard goes by direct stores throughout (apply_direct).
constexpr int kApplyWaves = 8, kApplySmallWaves = 4, kApplySmallChunks = 8192;
constexpr int kApplyBlocks = 256 * 256, kApplySparseDiv = 24, kApplyMiddleDiv = 20, kApplyDenseDiv = 7, kApplyRoomyDiv = 3;
#ifndef ROSE_APPLY_LINE
#define ROSE_APPLY_LINE 64                      // bytes moved around an entry: 64 or 32 (32 halves the bytes at low
                                                // density and is slower all the same: 7B workload 3.61 instead of
                                                // 2.43 ms at 1 %, 7.91 instead of 5.20 ms at 5 %: the memory moves
                                                // 64-byte units)
#endif
constexpr int kLineElems = ROSE_APPLY_LINE / 2; // line of 16-bit elements
constexpr int kLineShift = ROSE_APPLY_LINE == 128 ? 6 : ROSE_APPLY_LINE == 64 ? 5 : 4;
constexpr int kLineParts = kLineElems / 8;      // 16-byte parts of a line
constexpr int kLinesPerRound = 64 / kLineParts; // lines a wave moves with one load per lane
constexpr int kLineRounds = 64 / kLinesPerRound;     // rounds of one load per lane that move up to 64 lines
constexpr int kDirectPerLine = 3, kLoneDen = 10;     // direct stores, see apply_chunk
static_assert(ROSE_APPLY_LINE == 128 || ROSE_APPLY_LINE == 64 || ROSE_APPLY_LINE == 32, "line size");


__device__ __forceinline__ void lds_wave_fence() {
    // LDS operations of one wave are carried out in order; this keeps the compiler from moving
    // them across and waits for the ones issued so far.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Segment of entry e (wave-uniform, e < seg_off[n]): the largest t in [0, n) with seg_off[t] <= e.  Up to 512
// segments all ends are read at once and counted; more of them take a 64-ary search, one parallel probe per
// round (two rounds up to 4096).
__device__ __forceinline__ int32_t wave_find_segment(const int64_t *seg_off, int32_t n, int64_t e, int lane) {
    if (n <= 512) {
        int64_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = j * 64 + lane < n ? seg_off[j * 64 + lane] : INT64_MAX;
        int32_t cnt = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) cnt += __popcll(__ballot(v[j] <= e));
        return cnt > 0 ? cnt - 1 : 0;
    }
    int32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const int32_t step = (hi - lo + 63) >> 6;
        const int32_t probe = lo + lane * step;
        const bool le = probe < hi && seg_off[probe] <= e;   // true on a prefix of the lanes, lane 0 included
        const int k = __popcll(__ballot(le)) - 1;
        lo += k * step;
        hi = hi < lo + step ? hi : lo + step;
    }
    return lo;
}

// value an entry leaves at its element: the payload itself, or (arithmetic payload, no escape)
// bf16(current + payload), see arith_pair
__device__ __forceinline__ uint16_t apply_value(uint32_t cur, uint32_t val, bool add) {
    if (!add) return (uint16_t)val;
    return (uint16_t)pack_bf16_pair(__uint_as_float(cur << 16) + __uint_as_float(val << 16), 0.0f);
}

// A segment of the bucket and the tensor it belongs to: all uniform, fetched with scalar loads.
struct Segment {
    int32_t t, numel;
    int64_t start, end;
    uint16_t *dst;
};
__device__ __forceinline__ Segment load_segment(const BucketDev &b, const int32_t *local_numel, void *const *dst_ptrs,
                                                int32_t t) {
    Segment s;
    s.t = t;
    s.start = (int64_t)cload64(b.seg_off + t);
    s.end = (int64_t)cload64(b.seg_off + t + 1);
    s.dst = reinterpret_cast<uint16_t *>(cload64(dst_ptrs + t));
    s.numel = (int32_t)cload32(local_numel + t);
    return s;
}
// the segment that holds entry e, from s or one before it on (ends: e < total <= seg_off[n_tensors])
__device__ __forceinline__ void next_segment(const BucketDev &b, const int32_t *local_numel, void *const *dst_ptrs,
                                             int64_t e, Segment &s) {
    while (e >= s.end) s = load_segment(b, local_numel, dst_ptrs, s.t + 1);
}

// Dense buckets: every entry is one 2-byte store, nothing else.  Where most lines take many entries the
// memory merges the stores, and the work per entry is what binds the line path (7B-style workload, one
// shard: 3.27 against 1.90 ms at 30 %, 4.95 against 2.25 at 50 %, 1.85 against 1.63 at 15 %).  Two chunks per
// wave: one does better where the grid has a wave for each, four never.
constexpr int kDirectChunks = 2;
__device__ __forceinline__ void apply_direct(const BucketDev &b, int32_t n_tensors, const int32_t *local_numel,
                                             void *const *dst_ptrs, int arith, int64_t total, int64_t wbase, int lane) {
    const int32_t idx_mask = arith ? 0x7FFFFFFF : -1;
    int32_t idx[kDirectChunks];
    uint32_t val[kDirectChunks];
#pragma unroll
    for (int u = 0; u < kDirectChunks; ++u) {
        const int64_t e = wbase + u * 64 + lane;
        idx[u] = 0;
        val[u] = 0;
        if (e < total) {
            idx[u] = b.idx[e];
            val[u] = b.val[e];
        }
    }
    Segment s = load_segment(b, local_numel, dst_ptrs,
                             __builtin_amdgcn_readfirstlane(wave_find_segment(b.seg_off, n_tensors, wbase, lane)));
    const int64_t wend = wbase + kDirectChunks * 64 < total ? wbase + kDirectChunks * 64 : total;
    for (int64_t pos = wbase; pos < wend; pos = s.end) {
        next_segment(b, local_numel, dst_ptrs, pos, s);
#pragma unroll
        for (int u = 0; u < kDirectChunks; ++u) {
            const int64_t e = wbase + u * 64 + lane;
            const uint32_t i = (uint32_t)(idx[u] & idx_mask);
            if (e >= pos && e < s.end && e < wend && i < (uint32_t)s.numel) {   // an index outside the tensor is dropped
                const bool add = arith && idx[u] >= 0;
                const uint16_t v = apply_value(add ? s.dst[i] : 0u, val[u], add);
                __builtin_nontemporal_store(v, s.dst + i);
            }
        }
    }
}

// Line of an entry that may go through the line path (depends on the entry alone): its 16-byte part lies inside
// the tensor.  Lines are lines of the address: the tensor starts `mis` elements behind the start of one.  (An
// address that is not a multiple of 2 has no elements in lines: no entry has one.)
constexpr uint32_t kNoLine = 0xFFFFFFFFu;
struct Lines {
    uint32_t mis, numel, lim;                           // lim: elements from the first line's start to the tensor's end
    __device__ __forceinline__ Lines(const uint16_t *dst, int32_t tensor_numel) {
        const uint64_t base = reinterpret_cast<uint64_t>(dst);
        mis = (uint32_t)(base >> 1) & (uint32_t)(kLineElems - 1);
        numel = (base & 1u) ? 0u : (uint32_t)tensor_numel;
        lim = numel + mis;                              // below 2^31 + 32
    }
    __device__ __forceinline__ uint32_t of(uint32_t i) const {
        const uint32_t p = i + mis;
        return (i < numel && (p & ~7u) >= mis && (p | 7u) < lim) ? p >> kLineShift : kNoLine;
    }
};

// What a chunk holds in a lane: its entry, and (lanes below kLineElems) the entry 64 further on, the next chunk's.
struct ChunkEntry {
    uint32_t idx, val, idx2, val2, prev_idx;            // prev_idx: index of the entry before the chunk
    bool add, add2, look;                               // look: the entry of the next chunk exists
};

// A chunk that holds entries of several segments (s: the first one's): every lane finds its own segment, and the
// entries the chunk owns go by direct stores.  The ends of the next 64 segments are read by one lane each and
// searched by moves between lanes; only behind those a lane searches the table.  (Segment after segment, with a
// round of dependent loads for each, an apply into 2000 tensors of 40 elements at 5 % took 32.5 us; this way 3.9.)
__device__ __forceinline__ void apply_mixed(const BucketDev &b, int32_t n_tensors, const int32_t *local_numel,
                                            void *const *dst_ptrs, const Segment &s, const ChunkEntry &c, int64_t wbase,
                                            int n, int lane) {
    const int32_t at = s.t + 1 + lane;
    const int64_t away = (at < n_tensors ? b.seg_off[at] : INT64_MAX) - wbase;
    const int32_t end = away < 64 ? (int32_t)away : 64;
    int32_t k = 0;                                      // ends at or before this lane's entry
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1)
        if (__shfl(end, k + step - 1, 64) <= lane) k += step;
    int32_t t = s.t + k;
    if (k == 63 && t + 1 < n_tensors && b.seg_off[t + 1] <= wbase + lane) {      // (rare: 64 segments or more)
        int32_t hi = n_tensors;
        while (hi - t > 1) {
            const int32_t mid = (t + hi) >> 1;
            if (b.seg_off[mid] <= wbase + lane) t = mid; else hi = mid;
        }
    }
    uint16_t *const dst = static_cast<uint16_t *>(dst_ptrs[t]);
    const int32_t numel = local_numel[t];
    const Lines lines(dst, numel);
    const uint32_t line = lane < n ? lines.of(c.idx) : kNoLine;
    // leading lanes that continue the previous chunk's last line were applied with that chunk
    uint32_t before = (uint32_t)__shfl_up((int)line, 1, 64);
    int32_t t_before = __shfl_up(t, 1, 64);
    if (lane == 0) {
        before = wbase > s.start ? lines.of(c.prev_idx) : kNoLine;
        t_before = t;
    }
    const u64 same_m = __ballot(line != kNoLine && line == before && t == t_before);
    const u64 lead = same_m & ~(same_m + 1);
    auto store_one = [](uint16_t *d, uint32_t i, uint32_t v, bool plus) {
        __builtin_nontemporal_store(apply_value(plus ? d[i] : 0u, v, plus), d + i);
    };
    if (lane < n && !((lead >> lane) & 1u) && c.idx < (uint32_t)numel) store_one(dst, c.idx, c.val, c.add);
    // entries of the next chunk that still lie in this chunk's last line
    const uint32_t line63 = (uint32_t)__builtin_amdgcn_readlane((int)line, 63);
    if (line63 != kNoLine) {
        const Segment last = load_segment(b, local_numel, dst_ptrs, __builtin_amdgcn_readlane(t, 63));
        const Lines last_lines(last.dst, last.numel);
        if (c.look && wbase + 64 + lane < last.end && last_lines.of(c.idx2) == line63)
            store_one(last.dst, c.idx2, c.val2, c.add2);
    }
}

// One chunk of 64 entries.  What it needs comes in three rounds of loads: the entries, the entries behind
// them and the segment ends; the segment's tensor, by scalar loads; the lines.  All that concerns the segment
// is uniform; a chunk with entries of several goes another way (apply_mixed).
//   LONE    also lines that take one entry each go by direct stores
// A chunk's owned entries go by direct 2-byte stores where they are crowded, three or more to a line (from
// 8 % on the line path's work per entry binds it: 7B-style workload, one shard, 1.32 against 1.29 ms at 8 %, 2.21
// against 1.72 at 20 %), and with LONE where hardly two share a line (0.1 %: 78 against 85 us).
template <int LONE>
__device__ __forceinline__ void apply_chunk(const BucketDev &b, int32_t n_tensors, const int32_t *local_numel,
                                            void *const *dst_ptrs, int arith, int64_t total, int64_t wbase, int lane,
                                            uint4 (*s_line)[kLineParts], uint32_t *s_no) {
    const int32_t idx_mask = arith ? 0x7FFFFFFF : -1;
    const int64_t e = wbase + lane, e2 = e + 64;
    const int n = total - wbase < 64 ? (int)(total - wbase) : 64;      // entries of the chunk
    ChunkEntry c;
    c.look = lane < kLineElems && e2 < total;
    int32_t idx_raw = 0, idx2_raw = 0;
    c.val = c.val2 = 0;
    if (lane < n) {
        idx_raw = b.idx[e];
        c.val = b.val[e];
    }
    if (c.look) {
        idx2_raw = b.idx[e2];
        c.val2 = b.val[e2];
    }
    c.prev_idx = cload32(b.idx + (wbase > 0 ? wbase - 1 : 0)) & (uint32_t)idx_mask;      // (unused in the first chunk)
    const Segment s = load_segment(b, local_numel, dst_ptrs,
                                   __builtin_amdgcn_readfirstlane(wave_find_segment(b.seg_off, n_tensors, wbase, lane)));
    c.idx = (uint32_t)(idx_raw & idx_mask);
    c.idx2 = (uint32_t)(idx2_raw & idx_mask);
    c.add = arith && idx_raw >= 0;
    c.add2 = arith && idx2_raw >= 0;
    asm volatile("" :: "s"(s.dst), "s"(s.numel));       // the segment's loads go out together, in front of the branch
    if (s.end - wbase < n) {
        apply_mixed(b, n_tensors, local_numel, dst_ptrs, s, c, wbase, n, lane);
        return;
    }
    const int part = lane % kLineParts;
    uint16_t *lines16 = reinterpret_cast<uint16_t *>(s_line);
    const Lines lines(s.dst, s.numel);
    const uint64_t line0 = reinterpret_cast<uint64_t>(s.dst) & ~(uint64_t)(ROSE_APPLY_LINE - 1);
    const bool in = lane < n;
    const uint32_t line = in ? lines.of(c.idx) : kNoLine;
    // same line as the entry before?  lane 0 looks at the last entry of the previous chunk
    const uint32_t before0 = wbase > s.start ? lines.of(c.prev_idx) : kNoLine;
    const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp((int)before0, (int)line, 0x138, 0xf, 0xf, false);  // wave_shr:1
    const u64 ok_m = __ballot(line != kNoLine);
    const u64 same_m = __ballot(line == before) & ok_m;
    // leading lanes that continue the previous chunk's last line were applied with that chunk
    const u64 owned_m = ok_m & ~(same_m & ~(same_m + 1));
    const bool owned = (owned_m >> lane) & 1u;
    const bool loose = in && line == kNoLine && c.idx < (uint32_t)s.numel;   // an index outside the tensor is dropped
    // entries of the next chunk that still lie in this chunk's last line
    const uint32_t line63 = (uint32_t)__builtin_amdgcn_readlane((int)line, 63);
    const bool ext = (owned_m >> 63) && c.look && e2 < s.end && lines.of(c.idx2) == line63;
    // distinct lines of the owned entries
    const u64 heads = owned_m & ~(same_m & (owned_m << 1));
    const int n_lines = __popcll(heads);
    uint16_t *const dst = s.dst;
    auto store_one = [&](uint32_t i, uint32_t v, bool plus) {
        __builtin_nontemporal_store(apply_value(plus ? dst[i] : 0u, v, plus), dst + i);
    };
    const int n_owned = __popcll(owned_m);
    // (one comparison, both factors are negative or neither is: a second branch costs the kernel 20
    // registers and with them its occupancy)
    const int crowded = n_owned - kDirectPerLine * n_lines, not_lone = LONE ? kLoneDen * n_owned - (kLoneDen + 1) * n_lines : 1;
    if (crowded * not_lone >= 0) {
        if (owned || loose) store_one(c.idx, c.val, c.add);
        if (ext) store_one(c.idx2, c.val2, c.add2);
    } else {
        const bool head = (heads >> lane) & 1u;
        const int slot = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(heads >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)heads, 0u)) - (head ? 0 : 1);
        if (head) s_no[slot] = line;
        lds_wave_fence();
        // Load the lines: kLineParts lanes per line, kLinesPerRound lines per round, every round's load
        // before the first is put into LDS.  Nothing here is under a condition, so that the compiler
        // need not wait between the rounds: a lane without a line, or whose part lies outside the
        // tensor, loads the part of the first owned entry, into a place that nothing reads.
        const uint32_t some = ((uint32_t)__builtin_amdgcn_readlane((int)c.idx, __ffsll((long long)heads) - 1) + lines.mis) >> 3;
        uint4 lv[kLineRounds];
        uint32_t at[kLineRounds];                   // 16-byte part, counted from the first line
        bool on[kLineRounds];
#pragma unroll
        for (int r = 0; r < kLineRounds; ++r) at[r] = s_no[r * kLinesPerRound + lane / kLineParts];
#pragma unroll
        for (int r = 0; r < kLineRounds; ++r) {
            at[r] = at[r] * kLineParts + (uint32_t)part;
            on[r] = (r * kLinesPerRound + lane / kLineParts < n_lines) & (at[r] * 8u >= lines.mis) & (at[r] * 8u + 8u <= lines.lim);
            at[r] = on[r] ? at[r] : some;
            lv[r] = gload16_stream(reinterpret_cast<const void *>(line0 + (uint64_t)at[r] * 16u));
        }
#pragma unroll
        for (int r = 0; r < kLineRounds; ++r) s_line[r * kLinesPerRound + lane / kLineParts][part] = lv[r];
        lds_wave_fence();

        // patch
        if (owned) {
            uint16_t *q = lines16 + slot * kLineElems + ((c.idx + lines.mis) & (uint32_t)(kLineElems - 1));
            *q = apply_value(*q, c.val, c.add);
        }
        if (ext) {
            uint16_t *q = lines16 + (n_lines - 1) * kLineElems + ((c.idx2 + lines.mis) & (uint32_t)(kLineElems - 1));
            *q = apply_value(*q, c.val2, c.add2);
        }
        lds_wave_fence();

        // store the lines back whole
#pragma unroll
        for (int r = 0; r < kLineRounds; ++r) {
            if (on[r]) {
                const uint4 v4 = s_line[r * kLinesPerRound + lane / kLineParts][part];
                u32x4 w = {v4.x, v4.y, v4.z, v4.w};
                __builtin_nontemporal_store(w, reinterpret_cast<global_u32x4 *>(line0 + (uint64_t)at[r] * 16u));
            }
        }
        if (loose) store_one(c.idx, c.val, c.add);
        lds_wave_fence();                           // the LDS slots are reused
    }
}

template <int SPARSE, int WAVES>
__device__ __forceinline__ void apply_body(const BucketDev &b, int32_t n_tensors, const int32_t *local_numel,
                                           void *const *dst_ptrs, int arith, int64_t dense_from) {
    __shared__ uint4 s_line[WAVES][64][kLineParts];         // wave, line slot, 16-byte part
    __shared__ uint32_t s_no[WAVES][64];                    // line numbers
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t total = b.seg_off[n_tensors];
    if (total > b.capacity) total = b.capacity;
    const int64_t first = (int64_t)blockIdx.x * WAVES + wave, n_waves = (int64_t)gridDim.x * WAVES;
    if (!SPARSE && total >= dense_from) {
        for (int64_t wbase = first * kDirectChunks * 64; wbase < total; wbase += n_waves * kDirectChunks * 64)
            apply_direct(b, n_tensors, local_numel, dst_ptrs, arith, total, wbase, lane);
    } else {
        for (int64_t wbase = first * 64; wbase < total; wbase += n_waves * 64)
            apply_chunk<SPARSE>(b, n_tensors, local_numel, dst_ptrs, arith, total, wbase, lane, s_line[wave], s_no[wave]);
    }
}

// PER_SIMD: waves per SIMD that the kernel is held to
template <int SPARSE, int WAVES, int PER_SIMD>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(PER_SIMD, PER_SIMD)))
void apply_kernel(BucketDev b, int32_t n_tensors, const int32_t *local_numel, void *const *dst_ptrs, int arith,
                  int64_t dense_from) {
    apply_body<SPARSE, WAVES>(b, n_tensors, local_numel, dst_ptrs, arith, dense_from);
}

// ---------------------------------------------------------------------------------------------
// Transport objects (Sec. 4.2 "Asynchronous Weight Transfer": fixed-size buckets that describe
// themselves): a range of a destination's entries with a header and its own segment table, see
// the layout in the header file.  pack copies; apply checks the header on the device and then
// runs the ordinary apply on the arrays inside the object.
// ---------------------------------------------------------------------------------------------
__host__ __device__ inline size_t up16(size_t x) { return (x + 15) & ~(size_t)15; }
__host__ __device__ inline size_t object_idx_off(int32_t n_tensors) { return up16(64 + 8 * ((size_t)n_tensors + 1)); }
__host__ __device__ inline size_t object_size(int32_t n_tensors, int64_t n) {
    return object_idx_off(n_tensors) + up16(4 * (size_t)n) + up16(2 * (size_t)n);
}

// LOADS: 128-bit loads of indices a lane has in flight (1024 entries of a workgroup each)
template <int LOADS>
__global__ __launch_bounds__(256) void pack_kernel(BucketDev b, int32_t shard, int32_t n_tensors, int64_t first,
                                                   int64_t n, int32_t payload, char *obj) {
    int64_t total = b.seg_off[n_tensors];
    if (total > b.capacity) total = b.capacity;
    const bool ok = total >= 0 && first + n <= total;          // else: an object nobody will apply
    const size_t a_off = object_idx_off(n_tensors), b_off = a_off + up16(4 * (size_t)n);
    if (blockIdx.x == 0) {
        if (threadIdx.x < 16) {
            uint32_t w = 0;
            if (threadIdx.x == 0) w = ok ? ROSE_OBJECT_MAGIC : 0u;
            if (threadIdx.x == 1) w = 1u;
            if (threadIdx.x == 2) w = (uint32_t)shard;
            if (threadIdx.x == 3) w = (uint32_t)n_tensors;
            if (threadIdx.x == 4) w = (uint32_t)(u64)first;
            if (threadIdx.x == 5) w = (uint32_t)((u64)first >> 32);
            if (threadIdx.x == 6) w = (uint32_t)(u64)n;
            if (threadIdx.x == 7) w = (uint32_t)((u64)n >> 32);
            if (threadIdx.x == 8) w = (uint32_t)payload;
            reinterpret_cast<uint32_t *>(obj)[threadIdx.x] = w;
        }
        int64_t *seg = reinterpret_cast<int64_t *>(obj + 64);
        for (int32_t t = threadIdx.x; t <= n_tensors; t += blockDim.x) {
            int64_t v = b.seg_off[t] - first;
            seg[t] = v < 0 ? 0 : (v > n ? n : v);
        }
        // the segment table and the index and value arrays end on 16-byte boundaries: zero the slack
        if (threadIdx.x == 0 && n_tensors % 2 == 0) seg[n_tensors + 1] = 0;
        int32_t *idx = reinterpret_cast<int32_t *>(obj + a_off);
        uint16_t *val = reinterpret_cast<uint16_t *>(obj + b_off);
        if (threadIdx.x < 4 && n + threadIdx.x < (int64_t)(up16(4 * (size_t)n) / 4)) idx[n + threadIdx.x] = 0;
        if (threadIdx.x < 8 && n + threadIdx.x < (int64_t)(up16(2 * (size_t)n) / 2)) val[n + threadIdx.x] = 0;
    }
    if (!ok) return;
    int32_t *idx = reinterpret_cast<int32_t *>(obj + a_off);
    uint16_t *val = reinterpret_cast<uint16_t *>(obj + b_off);
    // 128-bit accesses, read and written once: the object's arrays are aligned, the bucket's range starts at any
    // entry.  A workgroup's loads are all in flight together.  (84 M entries in eight objects: 234 us with an entry
    // per lane, 192 us this way.)
    constexpr int kTileEntries = LOADS * 1024, kValLoads = LOADS > 1 ? LOADS / 2 : 1, kValLanes = LOADS > 1 ? 256 : 128;
    const int32_t *from_idx = b.idx + first;
    const uint16_t *from_val = b.val + first;
    // Large objects: each array's tiles begin at a 128-byte line of the object, the entries in front of it go singly (the
    // same eight objects: 189.0 us with stores across lines, 186.3 this way; 400 M entries in one bucket 885 and 864).
    int64_t n_idx = n, n_val = n;
    if constexpr (LOADS > 1) {
        const int64_t h_idx = ((0u - (uint32_t)reinterpret_cast<uintptr_t>(idx)) & 127u) / 4;
        const int64_t h_val = ((0u - (uint32_t)reinterpret_cast<uintptr_t>(val)) & 127u) / 2;
        n_idx = n > h_idx ? n - h_idx : 0;
        n_val = n > h_val ? n - h_val : 0;
        if (blockIdx.x == 0) {
            if ((int64_t)threadIdx.x < n - n_idx) idx[threadIdx.x] = from_idx[threadIdx.x];
            if ((int64_t)threadIdx.x < n - n_val) val[threadIdx.x] = from_val[threadIdx.x];
        }
        idx += n - n_idx;
        from_idx += n - n_idx;
        val += n - n_val;
        from_val += n - n_val;
    }
    const int64_t n_least = n_idx < n_val ? n_idx : n_val, n_most = n_idx < n_val ? n_val : n_idx;
    for (int64_t e0 = (int64_t)blockIdx.x * kTileEntries; e0 < n_most; e0 += (int64_t)gridDim.x * kTileEntries) {
        uint4 vi[LOADS], vv[kValLoads];
        if (e0 + kTileEntries <= n_least) {
#pragma unroll
            for (int j = 0; j < LOADS; ++j) vi[j] = gload16_stream(from_idx + e0 + (j * 256 + threadIdx.x) * 4);
            if (threadIdx.x < kValLanes) {
#pragma unroll
                for (int j = 0; j < kValLoads; ++j) vv[j] = gload16_stream(from_val + e0 + (j * 256 + threadIdx.x) * 8);
            }
#pragma unroll
            for (int j = 0; j < LOADS; ++j) gstore16_stream(idx + e0 + (j * 256 + threadIdx.x) * 4, vi[j]);
            if (threadIdx.x < kValLanes) {
#pragma unroll
                for (int j = 0; j < kValLoads; ++j) gstore16_stream(val + e0 + (j * 256 + threadIdx.x) * 8, vv[j]);
            }
        } else {                                        // the last tile: whole vectors, then the few entries behind them
            const int64_t left_i = min(max(n_idx - e0, (int64_t)0), (int64_t)kTileEntries), i_end = left_i & ~(int64_t)3;
            const int64_t left_v = min(max(n_val - e0, (int64_t)0), (int64_t)kTileEntries), v_end = left_v & ~(int64_t)7;
#pragma unroll
            for (int j = 0; j < LOADS; ++j) {
                const int64_t e = (j * 256 + threadIdx.x) * 4;
                if (e < i_end) vi[j] = gload16_stream(from_idx + e0 + e);
            }
#pragma unroll
            for (int j = 0; j < kValLoads; ++j) {
                const int64_t e = (j * 256 + threadIdx.x) * 8;
                if (e < v_end) vv[j] = gload16_stream(from_val + e0 + e);
            }
#pragma unroll
            for (int j = 0; j < LOADS; ++j) {
                const int64_t e = (j * 256 + threadIdx.x) * 4;
                if (e < i_end) gstore16_stream(idx + e0 + e, vi[j]);
            }
#pragma unroll
            for (int j = 0; j < kValLoads; ++j) {
                const int64_t e = (j * 256 + threadIdx.x) * 8;
                if (e < v_end) gstore16_stream(val + e0 + e, vv[j]);
            }
            if (threadIdx.x < left_i - i_end) idx[e0 + i_end + threadIdx.x] = from_idx[e0 + i_end + threadIdx.x];
            if (threadIdx.x < left_v - v_end) val[e0 + v_end + threadIdx.x] = from_val[e0 + v_end + threadIdx.x];
        }
    }
}

// true if the 64-byte header describes an object of this plan that fits object_bytes
__host__ __device__ inline bool object_header_ok(const uint32_t *h, int32_t n_tensors, size_t object_bytes, int64_t *n_out) {
    const int64_t first = (int64_t)((u64)h[4] | ((u64)h[5] << 32));
    const int64_t n = (int64_t)((u64)h[6] | ((u64)h[7] << 32));
    *n_out = n;
    if (h[0] != ROSE_OBJECT_MAGIC || h[1] != 1u || (int32_t)h[3] != n_tensors || first < 0 || n < 0) return false;
    if (h[8] > 1u) return false;                                        // payload kind: 0 new pattern, 1 arithmetic
    if (n > (int64_t)(object_bytes / 6)) return false;
    return object_size(n_tensors, n) <= object_bytes;
}

// the arrays inside an object whose header has passed object_header_ok
__device__ __forceinline__ BucketDev object_arrays(const char *obj, int32_t n_tensors, int64_t n) {
    const size_t a_off = object_idx_off(n_tensors), b_off = a_off + up16(4 * (size_t)n);
    BucketDev b;
    b.idx = reinterpret_cast<int32_t *>(const_cast<char *>(obj + a_off));
    b.val = reinterpret_cast<uint16_t *>(const_cast<char *>(obj + b_off));
    b.capacity = n;
    b.seg_off = reinterpret_cast<int64_t *>(const_cast<char *>(obj + 64));
    return b;
}

// Object apply runs as three launches on the stream: the verdict word is cleared, a pass over the
// segment table and all indices writes `ticket` into it if the object is not in order, and the apply
// pass leaves at once if it finds the ticket there.
__global__ void object_clear_kernel(u64 *verdict) { *verdict = 0; }

// Segment table: starts at 0, never decreases, ends at n.  Indices (escape bit masked off for
// arithmetic payloads): strictly ascending inside a segment, which is what lets the apply pass
// give every 64-byte piece of a tensor to exactly one wave.  An index may only fail to exceed its
// predecessor where a segment starts.  A wave whose entries hold such places marks the starts among its 256
// entries in a bit map: one look-up of the segments there, then 64 starts per load.  (With a search through the table
// for each such entry an object of 4000 entries in 2000 tensors took 19.2 us to check and apply, this way 8.8.)
template <int LOADS>
__global__ __launch_bounds__(256) void object_validate_kernel(const char *obj, size_t object_bytes, int32_t n_tensors,
                                                              int32_t n_buckets, u64 *verdict, u64 ticket) {
    __shared__ uint32_t s_starts[4][8];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t h[9];
    for (int i = 0; i < 9; ++i) h[i] = reinterpret_cast<const uint32_t *>(obj)[i];
    int64_t n;
    if (!object_header_ok(h, n_tensors, object_bytes, &n) || h[2] >= (uint32_t)n_buckets) return;   // apply rejects it too
    const BucketDev b = object_arrays(obj, n_tensors, n);
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t t = gid; t < n_tensors; t += stride) {
        const int64_t lo = b.seg_off[t], hi = b.seg_off[t + 1];
        bad |= lo < 0 || hi < lo || hi > n;
    }
    const int32_t m = h[8] ? 0x7FFFFFFF : -1;
    // Four neighbours per 128-bit load (the array is padded to whole ones), the one before them from the lane
    // below; LOADS of them in flight per lane.  (Eight objects of 84 M entries checked and applied: 1376 us with two
    // 4-byte loads an entry, 1318 us this way.)
    for (int64_t e0 = (int64_t)blockIdx.x * (LOADS * 1024); e0 < n; e0 += (int64_t)gridDim.x * (LOADS * 1024)) {
        uint4 v[LOADS];
        int32_t first[LOADS];
        uint32_t falls = 0;                             // bit 4 j + i: entry i of load j does not exceed the one before
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int64_t e = e0 + (j * 256 + threadIdx.x) * 4;
            v[j] = make_uint4(0, 0, 0, 0);
            first[j] = -1;
            if (e < n) {
                v[j] = gload16(b.idx + e);
                if (lane == 0 && e > 0) first[j] = b.idx[e - 1] & m;
            }
        }
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int64_t e = e0 + (j * 256 + threadIdx.x) * 4;
            const int32_t x[4] = {(int32_t)v[j].x & m, (int32_t)v[j].y & m, (int32_t)v[j].z & m, (int32_t)v[j].w & m};
            int32_t before = __builtin_amdgcn_update_dpp(first[j], x[3], 0x138, 0xf, 0xf, false);    // wave_shr:1
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (e + i > 0 && e + i < n && x[i] <= before) falls |= 1u << (4 * j + i);
                before = x[i];
            }
        }
        // allowed only where some segment starts
#pragma unroll 1
        for (int j = 0; j < LOADS; ++j) {
            const uint32_t mine = (falls >> (4 * j)) & 15u;
            if (!__ballot(mine != 0)) continue;
            const int64_t base = e0 + (j * 256 + wave * 64) * 4;       // the wave's 256 entries begin here
            if (lane < 8) s_starts[wave][lane] = 0;
            lds_wave_fence();
            for (int32_t t = __builtin_amdgcn_readfirstlane(wave_find_segment(b.seg_off, n_tensors, base, lane));
                 t < n_tensors; t += 64) {
                const int64_t at = (t + lane < n_tensors ? b.seg_off[t + lane] : INT64_MAX) - base;
                if (at >= 0 && at < 256) atomicOr(&s_starts[wave][at >> 5], 1u << (at & 31));
                if (__ballot(at >= 256)) break;
            }
            lds_wave_fence();
            bad |= (mine & ~(s_starts[wave][lane >> 3] >> (4 * (lane & 7)))) != 0;
            lds_wave_fence();                           // the map is used again
        }
    }
    if (bad) *verdict = ticket;
}

template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void apply_object_kernel(const char *obj, size_t object_bytes, int32_t n_tensors,
                                                                  int32_t n_buckets, int32_t tp,
                                                                  const int32_t *local_numel, void *const *dst_ptrs,
                                                                  const u64 *verdict, u64 ticket) {
    uint32_t h[9];
    for (int i = 0; i < 9; ++i) h[i] = reinterpret_cast<const uint32_t *>(obj)[i];
    int64_t n;
    if (!object_header_ok(h, n_tensors, object_bytes, &n)) return;     // uniform: every thread leaves
    if (h[2] >= (uint32_t)n_buckets) return;
    if (*verdict == ticket) return;                                    // the validation pass found it out of order
    const BucketDev b = object_arrays(obj, n_tensors, n);
    if (b.seg_off[0] != 0 || b.seg_off[n_tensors] != n) return;
    apply_body<0, WAVES>(b, n_tensors, local_numel + (size_t)(h[2] / (uint32_t)tp) * n_tensors, dst_ptrs, (int)h[8], INT64_MAX);
}

// ---------------------------------------------------------------------------------------------
// dense copy of one shard: the same tiles as encode, moved instead of compared.  One tile per workgroup, all
// of its loads in flight together, loads and stores non-temporal: what a plain copy does best with (2 GiB:
// 5.0 - 5.4 TB/s from a grid of 2048 or 8192 workgroups, 5.9 from one workgroup per tile, 6.1 with both hints).
// Loads take any alignment at little cost, stores do not (5.7 TB/s), so a tile's vectors are lined up with
// the DESTINATION: they begin `head` elements into the piece, which the first tile copies one by one.  Pieces of several
// tiles are lined up with 128-byte lines, not with vectors only (packed, eight 7B-style layers, TP4: 1445 -> 1313 us, fp32
// masters 2117 -> 1932).
// (Eight 7B-style layers, TP4, four shards: 1416 -> 1287 us; packed at odd elements: 4130 -> 1421 us at TP2; rows of
// 765 elements a shard, 131 M weights: 248 -> 89 us; figures before that.)
// ---------------------------------------------------------------------------------------------
constexpr int kCopyAtOnce = 2048;       // workgroups (of 256 threads, 8 waves per SIMD)
template <int NEW_F32>
__global__ __launch_bounds__(kThreads) void dense_copy_kernel(CopyArgs a) {
    const int32_t tile = a.tile_begin + (int32_t)blockIdx.x;
    const int32_t piece = cload32(a.tile_piece + tile);
    const Piece pc = load_piece(a.pieces + piece);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const void *new_base = reinterpret_cast<const void *>(cload64(a.new_ptrs + pc.tensor));
    uint16_t *dst = reinterpret_cast<uint16_t *>(cload64(a.dst_ptrs + pc.tensor));
    const uint32_t len = (uint32_t)pc.len;
    const uint32_t k_tile = (uint32_t)(tile - cload32(a.first_tile + piece)) * (uint32_t)kTile;
    if (k_tile >= len) return;                          // a tile for being moved (kPieceShift), or an empty piece
    const bool dst_strided = (pc.flags & kPieceDstStrided) != 0;
    const uint32_t line = len > (uint32_t)kTile ? (uint32_t)kShiftElems : (uint32_t)kVec;     // (a short piece: little to copy singly)
    const uint32_t head = dst_strided ? 0u : (0u - ((uint32_t)((uintptr_t)dst >> 1) + (uint32_t)pc.local_base)) & (line - 1u);
    const uint32_t k0 = k_tile + head, k_lane = k0 + (uint32_t)wave * kWaveSpan + (uint32_t)lane * kVec;
    auto copy_one = [&](uint32_t k) {
        const int64_t s = src_index(pc, k, false);
        gstore_u16(dst + dst_index(pc, k, false), NEW_F32 ? rne_bf16(gload_u32(static_cast<const uint32_t *>(new_base) + s))
                                                          : gload_u16(static_cast<const uint16_t *>(new_base) + s));
    };
    if (k_tile == 0 && threadIdx.x < head && threadIdx.x < len) copy_one(threadIdx.x);
    const bool vec = (pc.flags & kPieceLoad16) && ((((uintptr_t)new_base) | ((uintptr_t)dst)) & 1u) == 0 &&
                     k0 + (uint32_t)kVec <= len && (!dst_strided || pc.run >= kVec);
    if (!vec) {
#pragma unroll 1
        for (int j = 0; j < kIters; ++j)
            for (uint32_t i = 0; i < (uint32_t)kVec; ++i) {
                const uint32_t k = k_lane + (uint32_t)(j * 64) * kVec + i;
                if (k < len) copy_one(k);
            }
        return;
    }
    // may a vector straddle the end of a run, on either side?
    const bool src_split = (pc.flags & kPieceStrided) && (((uint32_t)pc.run | head) & 7u);
    const bool dst_split = dst_strided && ((uint32_t)pc.run & 7u);
    RawTile<NEW_F32> r;
#pragma unroll
    for (int j = 0; j < kIters; ++j) {                  // unconditional, see load_raw_pair
        uint32_t k = k_lane + (uint32_t)(j * 64) * kVec;
        if (k + kVec > len) k = k0;
        const int64_t e = src_index(pc, k, true);
        if constexpr (NEW_F32) {
            r.lo[j] = gload16_stream(static_cast<const uint32_t *>(new_base) + e);
            r.hi[j] = gload16_stream(static_cast<const uint32_t *>(new_base) + e + 4);
        } else {
            r.v[j] = gload16_stream(static_cast<const uint16_t *>(new_base) + e);
        }
    }
    // The ordinary tile by itself: among the rare cases its stores lie lines of code apart, and a launch that does
    // not last long pays for each (one matrix of 1 M elements: 3.4 us, 3.7 that way; fp32 masters 3.8 and 4.3).
    if (!src_split && !dst_split && k0 + (uint32_t)kTile <= len) {
        // A bf16 launch whose workgroups are all resident reads first and writes then (four shards of 8192 x 4096:
        // 24.0 us, 27.9 with each store as soon as its load is there; with the input in memory 28.6 and 33.8); longer
        // ones do better without (1 GiB in four shards: 330 us, 337 with the wait), fp32 masters too.
        if (!NEW_F32 && gridDim.x <= (unsigned)kCopyAtOnce) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < kIters; ++j)
            gstore16_stream(dst + dst_index(pc, k_lane + (uint32_t)(j * 64) * kVec, true), raw_to_bf16(r, j));
        return;
    }
#pragma unroll
    for (int j = 0; j < kIters; ++j) {
        const uint32_t k = k_lane + (uint32_t)(j * 64) * kVec;
        uint32_t left = kVec, q = 0;
        if (src_split || dst_split) left = split_left(pc, k, &q);
        if (k + kVec > len || (dst_split && left < (uint32_t)kVec)) {
            for (uint32_t i = 0; i < (uint32_t)kVec; ++i)
                if (k + i < len) copy_one(k + i);
            continue;
        }
        uint4 v = raw_to_bf16(r, j);
        if (src_split && left < (uint32_t)kVec) v = split_merge(v, load_new_vec<NEW_F32>(new_base, split_tail_at(pc, q, left)), left);
        gstore16_stream(dst + dst_index(pc, k, true), v);
    }
}

// ---------------------------------------------------------------------------------------------
// bandwidth probe: grid-stride 128-bit copy, or read-only with a checksum
// ---------------------------------------------------------------------------------------------
constexpr int kBwThreads = 256;

__global__ __launch_bounds__(256) void bw_copy_kernel(const uint4 *src, uint4 *dst, size_t n16) {
    size_t i = (size_t)blockIdx.x * (kBwThreads * 4) + threadIdx.x;
    const size_t step = (size_t)gridDim.x * (kBwThreads * 4);
    for (; i < n16; i += step) {
        uint4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            size_t at = i + (size_t)j * kBwThreads;
            v[j] = at < n16 ? src[at] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            size_t at = i + (size_t)j * kBwThreads;
            if (at < n16) dst[at] = v[j];
        }
    }
}

// (non-temporal loads, eight in flight per lane: 7.1 TB/s; ordinary loads, four in flight: 6.1 - 6.2)
__global__ __launch_bounds__(256) void bw_read_kernel(const uint4 *src, size_t n16, u64 *sink) {
    size_t i = (size_t)blockIdx.x * (kBwThreads * 8) + threadIdx.x;
    const size_t step = (size_t)gridDim.x * (kBwThreads * 8);
    uint32_t acc = 0;
    for (; i < n16; i += step) {
        uint4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            size_t at = i + (size_t)j * kBwThreads;
            v[j] = at < n16 ? gload16_stream(src + at) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc += v[j].x ^ v[j].y ^ v[j].z ^ v[j].w;
    }
    // The data-dependent test keeps the loads alive; it is true for about one lane in 2^32, so
    // the probe is not slowed down by atomics on one address.
    if (acc == 0x9E3779B9u) atomicAdd(sink, 1ull);
}

// Mixed probe: the traffic of an encode launch without any of its work.  Reads two streams in
// 16 KB chunks (non-temporal, like encode) and writes w16 16-byte vectors per chunk, contiguous
// across chunks, to a third.  TIMED = 0: every chunk's output is written at once.  TIMED = 1: it is
// held back (nothing is stored anywhere: the probe only remembers which chunks are due) and written
// in the windows of time of the encode kernel's timed tile order, or when 64 chunks are due.
template <int TIMED>
__global__ __launch_bounds__(256) void bw_mix_kernel(const uint4 *a, const uint4 *b, uint4 *dst, size_t n_chunks,
                                                     uint32_t w16, u64 *sink) {
    uint4 acc = make_uint4(0, 0, 0, 0);
    size_t due_from = blockIdx.x;                      // the oldest chunk whose output has not been written
    uint32_t n_due = 0;
    auto write_chunk = [&](size_t c) {
        for (uint32_t k = threadIdx.x; k < w16; k += kBwThreads) {
            u32x4 w = {acc.x, acc.y, acc.z, acc.w};
            __builtin_nontemporal_store(w, reinterpret_cast<global_u32x4 *>(reinterpret_cast<uintptr_t>(dst + c * (size_t)w16 + k)));
        }
    };
    for (size_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        uint4 va[4], vb[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            va[j] = gload16_stream(a + c * 1024 + j * kBwThreads + threadIdx.x);
            vb[j] = gload16_stream(b + c * 1024 + j * kBwThreads + threadIdx.x);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = xor4(acc, xor4(va[j], vb[j]));
        if (!TIMED) {
            write_chunk(c);
        } else {
            ++n_due;
            const uint32_t now = (uint32_t)__builtin_amdgcn_s_memrealtime();
            const bool open = (now & ((1u << ROSE_WRITE_PERIOD_LOG2) - 1u)) < ROSE_WRITE_OPEN_TIMED;
            if (open || n_due >= 64u) {
                for (; n_due > 0; --n_due, due_from += gridDim.x) write_chunk(due_from);
            }
        }
    }
    if (TIMED)
        for (; n_due > 0; --n_due, due_from += gridDim.x) write_chunk(due_from);
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u) atomicAdd(sink, 1ull);
}

// Line probe: the memory traffic of an apply launch without its work.  A wave takes 128 consecutive
// lines of 64 bytes, 16 per round (4 lanes per line); the lines whose hash is below the threshold are
// loaded (all loads first, non-temporal like apply's), changed and stored back.
__device__ __forceinline__ uint32_t line_hash(size_t i) {
    uint32_t x = (uint32_t)i * 0x9E3779B1u ^ (uint32_t)((uint64_t)i >> 32);
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return x;
}
__global__ __launch_bounds__(256) void bw_lines_kernel(uint4 *dst, size_t n_lines, uint32_t threshold) {
    const int lane = threadIdx.x & 63;
    const size_t base = ((size_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 128;
    uint4 v[8];
    bool on[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const size_t line = base + (size_t)(r * 16 + lane / 4);
        on[r] = line < n_lines && line_hash(line) < threshold;
        v[r] = make_uint4(0, 0, 0, 0);
        if (on[r]) v[r] = gload16_stream(dst + line * 4 + (lane & 3));
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (on[r]) {
            const size_t line = base + (size_t)(r * 16 + lane / 4);
            u32x4 w = {v[r].x + 1u, v[r].y, v[r].z, v[r].w};
            __builtin_nontemporal_store(w, reinterpret_cast<global_u32x4 *>(reinterpret_cast<uintptr_t>(dst + line * 4 + (lane & 3))));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
// workgroups per CU the encode grid may use (bounded by what fits at once)
#ifndef ROSE_WGS_PER_CU
#define ROSE_WGS_PER_CU 8
#endif

// the encode kernel variant for (fp32 master input, sender refresh, arithmetic payload)
typedef void (*EncodeKernel)(EncodeArgs);
// Arithmetic payloads of bf16 weights, without refresh: formed of every element from this density on, of the compacted
// entries below.  One matrix, us, of elements / of entries, 1000 MiB: 10 % 288 / 268, 20 % 348 / 342, 25 % 411 / 405,
// 30 % 430 / 432, 35 % 520 / 541, 60 % 640 / 721, 100 % 734 / 857; 400 MiB: 20 % 159 / 152, 25 % 174 / 174, 30 % 180 / 183,
// 100 % 316 / 357.  Where more comes than the last time, entries lose more (1200 MiB, 1 % seen, 25 / 60 / 100 % come:
// 936 / 843 / 976 and 1337 / 977 / 1202), so the line is for the most that the buckets could hold.
constexpr int32_t kElementsPpm = 300000;
constexpr int kElementsVariant = 8;
static EncodeKernel encode_variant(int new_is_f32, int refresh, int arith) {
    static const EncodeKernel table[8] = {encode_kernel<0, 0, 0>, encode_kernel<1, 0, 0>, encode_kernel<0, 1, 0>,
                                          encode_kernel<1, 1, 0>, encode_kernel<0, 0, 1>, encode_kernel<1, 0, 1>,
                                          encode_kernel<0, 1, 1>, encode_kernel<1, 1, 1>};
    return table[(new_is_f32 ? 1 : 0) + (refresh ? 2 : 0) + (arith ? 4 : 0)];
}

typedef void (*CountKernel)(EncodeArgs, uint16_t *);
typedef void (*StageKernel)(EncodeArgs, uint16_t *, uint32_t *, int32_t, int32_t);
typedef void (*EmitKernel)(EncodeArgs, const uint16_t *);
typedef void (*EmitStagedKernel)(EncodeArgs, const uint16_t *, const uint32_t *, int32_t, int32_t, int32_t);
static StageKernel stage_variant(int new_is_f32, int refresh, int arith) {
    static const StageKernel table[8] = {stage_tiles_kernel<0, 0, 0>, stage_tiles_kernel<1, 0, 0>, stage_tiles_kernel<0, 1, 0>,
                                         stage_tiles_kernel<1, 1, 0>, stage_tiles_kernel<0, 0, 1>, stage_tiles_kernel<1, 0, 1>,
                                         stage_tiles_kernel<0, 1, 1>, stage_tiles_kernel<1, 1, 1>};
    return table[(new_is_f32 ? 1 : 0) + (refresh ? 2 : 0) + (arith ? 4 : 0)];
}
static EmitStagedKernel emit_staged_variant(int new_is_f32, int refresh, int arith) {
    static const EmitStagedKernel table[8] = {emit_staged_kernel<0, 0, 0>, emit_staged_kernel<1, 0, 0>, emit_staged_kernel<0, 1, 0>,
                                              emit_staged_kernel<1, 1, 0>, emit_staged_kernel<0, 0, 1>, emit_staged_kernel<1, 0, 1>,
                                              emit_staged_kernel<0, 1, 1>, emit_staged_kernel<1, 1, 1>};
    return table[(new_is_f32 ? 1 : 0) + (refresh ? 2 : 0) + (arith ? 4 : 0)];
}
static EmitKernel emit_variant(int new_is_f32, int refresh, int arith) {
    static const EmitKernel table[8] = {emit_tiles_kernel<0, 0, 0>, emit_tiles_kernel<1, 0, 0>, emit_tiles_kernel<0, 1, 0>,
                                        emit_tiles_kernel<1, 1, 0>, emit_tiles_kernel<0, 0, 1>, emit_tiles_kernel<1, 0, 1>,
                                        emit_tiles_kernel<0, 1, 1>, emit_tiles_kernel<1, 1, 1>};
    return table[(new_is_f32 ? 1 : 0) + (refresh ? 2 : 0) + (arith ? 4 : 0)];
}

// Number of workgroups of each encode kernel variant that fit on the current device at once.
int encode_resident_all(int resident[kEncodeKernels]) {
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return (int)e;
    for (int v = 0; v < kEncodeKernels; ++v) {
        int per_cu = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, v == kElementsVariant ? encode_elements_kernel : encode_variant(v & 1, v & 2, v & 4), kThreads, 0);
        if (e != hipSuccess) return (int)e;
        if (per_cu < 1 || cus < 1) return (int)hipErrorInvalidValue;
        if (per_cu > ROSE_WGS_PER_CU) per_cu = ROSE_WGS_PER_CU;
        resident[v] = cus * per_cu;
    }
    return 0;
}

// Built-in scratch for callers that cannot allocate (rose_delta_encode_static).  In host code the
// array's name only stands for the symbol: its address on a device comes from hipGetSymbolAddress
// with that device current, each device has its own copy, and only that pointer is ever handed to
// a kernel.
static __device__ __align__(256) unsigned long long scratch[ROSE_STATIC_SCRATCH_BYTES / sizeof(unsigned long long)];
constexpr int kMaxDevices = 64;
int static_scratch(void **ptr, size_t *bytes) {
    static std::mutex mu;
    static void *per_device[kMaxDevices] = {nullptr};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return (int)hipErrorInvalidValue;
        per_device[dev] = p;
    }
    *ptr = per_device[dev];
    *bytes = sizeof(scratch);
    return 0;
}

#ifndef ROSE_SERVER_WGS
#define ROSE_SERVER_WGS 16          // workgroups of the grid that serve prefixes (kWaves servers each)
#endif

// How a launch in this tile order walks its tiles: tiles per ticket, and how long of each period the bucket stores may go out
// (0: always).  ppm: changed elements per million, -1 unknown; room_ppm: as many as the buckets could hold.
//   timed       4 tiles, 10 us of each 82; from kLongBelowPpm on of each 41: the entries of a period have to fit the ring.
//   neighbours  4 tiles and 10 us of 41 as well, as long as the ring holds them and no more is expected (the buckets hold no more
//               than kNearRoomPpm; an update that overflows them may be slow), without refresh; else 3 tiles, whose prefixes are
//               ready sooner and leave the ring room, and longer windows, so that less waits: up to 5 % 15 us, above, and where
//               payloads are formed of every element, 20 us.
// Eight 7B-style layers without embedding and head, TP4, one process, same buffers, ms (bf16 / fp32 masters / arithmetic payloads):
//                 1 %                  3 %                  4 %                  5 %                  6 %                  7 %
//   4 x 10 of 82  1.057 1.594 1.064    1.102 1.641 1.115    1.159 1.711 1.184    1.223 1.837 1.236    1.269 1.954 1.291    1.342 2.015 1.356
//   4 x 10 of 41  1.075 1.658 1.080    1.115 1.700 1.138    1.131 1.716 1.173    1.158 1.747 1.210    1.214 1.821 1.266    1.311 1.936 1.320
//   3 x 15        1.156 1.702 1.158    1.190 1.744 1.209    1.204 1.765 1.231    1.226 1.779 1.256    1.241 1.801 1.280    1.291 1.853 1.318
//   3 x 20        1.160 1.742 1.157    1.190 1.797 1.212    1.206 1.813 1.238    1.223 1.824 1.261    1.237 1.841 1.285    1.284 1.866 1.330
// Where the density is the last launch's and more comes, 4 tiles lose far more than 3 (4 / 3 tiles: 12 % 1.61 / 1.38, 20 % 2.03 /
// 1.80, 30 % 4.12 / 2.31).  With refresh, in turns, 4 tiles lose from 4 % on too (room for 5.6 / 6.3 %, 4 and 3 tiles: eight such
// layers with embedding and head 2.09 / 2.06, 2.12 / 2.09; six 8B-style ones 2.67 / 2.62, 2.67 / 2.63; a sender's share of a 32B
// style 2.27 / 2.23, 2.31 / 2.27; packed 2.09 / 2.07, 2.11 / 2.09; arithmetic payloads 2.09 / 2.06, 2.04 / 2.00; fp32 masters 2.64
// / 2.61); the timed order's 4 tiles and periods of 82 us, below that, do refreshes no harm.
constexpr int32_t kLongBelowPpm = 33000, kNearBelowPpm = 50000;
constexpr int32_t kNearFourPpm = 65000, kNearFourPpmF32 = 57000, kNearRoomPpm = 80000;
static void encode_walk(int order, int32_t ppm, int32_t room_ppm, int new_is_f32, bool of_elements, bool refresh, EncodeArgs *a) {
    a->adjacent = order == ROSE_TILE_ORDER_SPREAD ? 0 : 1;
    a->batch = kBatch;
    a->window_open = 0;
    a->window_mask = (1u << ROSE_WRITE_PERIOD_LOG2) - 1u;
    const bool four = !of_elements && !refresh && ppm >= 0 && ppm < (new_is_f32 ? kNearFourPpmF32 : kNearFourPpm) && room_ppm < kNearRoomPpm;
    if (order == ROSE_TILE_ORDER_TIMED || (order == ROSE_TILE_ORDER_NEIGHBOURS && four)) {
        a->batch = kBatchTimed;
        a->window_open = ROSE_WRITE_OPEN_TIMED;
        if (order == ROSE_TILE_ORDER_TIMED && ppm >= 0 && ppm < kLongBelowPpm) a->window_mask = 2 * a->window_mask + 1;
    } else if (order == ROSE_TILE_ORDER_NEIGHBOURS) {
        const bool near = !of_elements && ppm >= 0 && ppm < kNearBelowPpm;
        a->window_open = near ? ROSE_WRITE_OPEN_NEAR : ROSE_WRITE_OPEN_WIDE;
    }
}

// Updates that go in two launches instead of by tickets, and how.  What bounds the ticket kernel on updates that are not
// large is its counter (14 ns a ticket, two requests a workgroup), the way from a count to its prefix and the launches around
// it, about 40 us; the staged form pays for writing and reading every entry once more instead.  One matrix of 4096 columns,
// us per call, inputs (and the slots) in the caches / 512 MB written elsewhere before each call:
//                  read again     staged        tickets (with nothing read twice)
//   bf16  10 MiB   6.7 / 10.6     7.0 / 10.3    33                             1 %
//         16 MiB   7.9 / 12.2     7.4 / 11.3    33                             1 %
//         64 MiB   21.9 / 28.2    14.3 / 18.9   40 / 41                        1 %
//         64 MiB   26.0 / 34.5    18.9 / 26.7   42 / 43                        10 %
//         64 MiB   33.4 / 39.1    35.2 / 41.5   48 / 48                        30 % (past the slots: read again)
//        192 MiB                  37 / 41       65 / 65                        1 %
//        450 MiB                  84 / 91       113 / 112                      1 %
//        450 MiB                  104 / 120     123 / 123                      5 %
//        600 MiB                  134 / 157     154 / 150                      5 %
//       1200 MiB                  222 / 243     246 / 242                      1 %
//   fp32  600 MiB                 131 / 140     150 / 149                      3 %
//   arithmetic, bf16 1000 MiB     229 / 259     258 / 259                      5 %
//               bf16 2000 MiB     365 / 399     430 / 432                      1 %
//   refresh,    bf16 1000 MiB     277 / 314     322 / 319                      5 %
// So: read again below 12 MiB, where the second reading comes out of the caches at once, and below 24 MiB from 10 % on (16 MiB at
// 5 / 10 / 15 %: read again 8.7 9.1 9.8, staged 8.5 9.1 10.4; 24 MiB: 10.2 10.6 11.3 and 9.6 10.5 11.7), and where the slots do
// not hold the tiles; staged up to kStagedMib of the density, half as much again for arithmetic payloads and refresh; by tickets
// above.  Slots have to hold twice what is expected of a tile, since densities differ between the rows of a model (31 MiB of
// fp32 masters, 12 % with a rate of its own for each 4096 elements: parked 20.4 us, read again 16.4), from 48 to 80 MiB, where
// parking gains more, 1.25 times (75 MiB of the same: 31.4 and 34.7).
// The density is that of the last update looked at, and another may come.  What is past its slot is read again, so that the
// staged form then takes (1 % seen, one matrix, bf16, us, in the caches; beside it reading again up to 80 MiB, tickets above):
//   comes     64 MiB         192 MiB     300 MiB     384 MiB     850 MiB     1200 MiB
//     1 %     14.7  22.2      37   64     57   84     73  101    154  183    219  244
//    10 %     22.1  26.2      55   71     78   92    106  113    348  222    510  302
//    13 %     24.4  27.6      60   74     83   94    156  119    354  224    527  303
//    20 %     29.0  29.9      69   97    123  121    160  150    368  308    581  431
//    30 %     35.2  33.4      88   98    129  133    168  158    422  333    613  448
//   100 %     49.8  46.5     121  163    200  231    254  291    569  617    820  894
// (the worst between these: 64 MiB at 25 % 35.6 and 31.5, with arithmetic payloads 42 and 33; 300 MiB at 17 % 121 and 112).
// From 48 to 300 MiB a wrong guess costs little beside what a right one gains, and the last density is taken.  Elsewhere the
// form goes by the most that the buckets could hold where that is more: above 300 MiB, as the table shows, and below 48 MiB,
// where reading again is nearly as fast (32 MiB, 1 %: 11.7 and 9.7) and a wrong guess dear (25 % come: 15.7 and 21.7).  With no
// density at all (no bucket checked yet, buckets with room for everything) updates are read again up to 80 MiB and go by
// tickets above.
// group: a workgroup of the second launch takes more tiles the more there are and the less they hold (1 % / 5 %,
// 1, 2, 4, 8, 16 tiles: 64 MiB 15.0 14.4 14.8 15.0 16.6 / 16.7 17.4 18.7 21.6 27.5; 512 MiB 114 103 98 96 96 / 130 120 112 114
// 114).  stream: slots written non-temporal from 192 MiB on (512 MiB, 1 %: 95.7 / 102.4 without, 95.8 / 100.1 with; 1 GiB
// 188.6 / 207.9 and 186.5 / 191.4; 64 MiB 14.9 / 19.4 and 15.3 / 19.8).
struct TwoLaunches {
    int form, group_log2, stream;
};
constexpr int64_t kReadAgainMib = 12, kReadAgainDenseMib = 24, kUnknownMib = 80, kStreamMib = 192, kGuessFromMib = 48, kGuessToMib = 300;
constexpr int32_t kReadAgainDensePpm = 100000;
constexpr struct {
    int32_t below_ppm;
    int64_t mib;
} kStagedMib[] = {{12000, 1200}, {22000, 850}, {32000, 700}, {55000, 480}, {85000, 400}, {125000, 300}};
static_assert((kUnknownMib << 20) / 4 < (int64_t)1 << 31 && kStageMostTiles * kTile < (int64_t)1 << 31,
              "the second launch adds up entries in 32 bits");
static TwoLaunches two_launches(const EncodeArgs &a, int new_is_f32, int refresh, int arith, int32_t ppm, int32_t room_ppm) {
    const int64_t bytes = (int64_t)a.n_tiles * kTile * (new_is_f32 ? 6 : 4), mib = (bytes + (1 << 19)) >> 20;
    const bool guess = mib >= kGuessFromMib && mib <= kGuessToMib;
    const int32_t by = ppm < 0 ? 1000000 : guess || room_ppm < ppm ? ppm : room_ppm;
    const int64_t expected = (int64_t)by * kTile / 1000000;
    TwoLaunches t = {kTickets, 0, mib >= kStreamMib};
    if (mib <= kUnknownMib) {
        const bool read_again = mib <= kReadAgainMib || (mib <= kReadAgainDenseMib && by >= kReadAgainDensePpm);
        const int64_t room = mib < kGuessFromMib ? expected * 2 + 64 : expected * 5 / 4 + 64;
        t.form = read_again || a.slot_size < kThreads || room > a.slot_size ? kReadAgain : kStaged;
    } else if (expected * 2 + 64 <= a.slot_size) {
        for (const auto &line : kStagedMib)
            if (by < line.below_ppm) {
                if (mib <= (refresh || arith ? line.mib * 3 / 2 : line.mib)) t.form = kStaged;
                break;
            }
    }
    const int g = (mib >= 32) + (mib >= 96) + (mib >= 192) + (mib >= 384) - (by > 30000) - (by > 80000);
    t.group_log2 = g > 0 ? g : 0;
    return t;
}
static void launch_refresh_replicated(const EncodeArgs &a, int new_is_f32, const RefreshArgs *refresh, hipStream_t st) {
    if (refresh && refresh->n > 0)
        hipLaunchKernelGGL(refresh_replicated_kernel, dim3(8, refresh->n > 1024 ? 1024 : refresh->n), dim3(256), 0, st,
                           refresh->list, refresh->numel, refresh->n, const_cast<void *const *>(a.old_ptrs), a.new_ptrs,
                           new_is_f32);
}

// The refresh of bf16 weights does better with three workgroups on a CU than with the four that fit, but where it writes next to
// nothing: fewer lines are on their way back among fewer reads (eight 7B-style layers with embedding and head, TP4, four and three,
// us: in turns, 0.1 % 1459 / 1518, 0.5 % 1657 / 1690, 1 % 1773 / 1743, 5 % 2160 / 2107, TP1 at 2 % 1921 / 1872; chain by chain, 10
// % 2370 / 2316, 20 % 2604 / 2564, 30 % 3134 / 2897).  Not from a third on, where tickets are counted ahead (35 % 3964 / 4111, 40 %
// 4065 / 4196, 60 % 4620 / 4789, TP1 at 40 % 3493 / 3831), nor where pieces are short and every tile begins with a walk through
// tables (500 M weights, pieces of half a tile, 1 % 806 / 963; of 2 / 4 / 6 / 8 / 12 tiles, 1 % 534 / 601, 493 / 521, 493 / 499,
// 538 / 527, 491 / 487, 2 % 557 / 616, 533 / 541, 535 / 527, 594 / 578, 535 / 521).  Packed tensors and a sender's share of a 32B
// style gain less, and lose where little changes (1 / 5 / 20 %, packed 1760 / 1789, 2140 / 2118, 2639 / 2616, a share 1941 / 1939,
// 2317 / 2263, 2771 / 2737, aligned weights beside them 1757 / 1741, 2120 / 2075, 2604 / 2571; at 20 % with other buffers packed
// 2361 / 2403, a share 2466 / 2541). Without refresh it holds for aligned weights (5 % 1352 / 1334), not for packed ones (1382 /
// 1401) nor for such a share (1385 / 1393).
constexpr int32_t kRefreshFewerPpm = 9000, kRefreshFewerToPpm = 333000, kRefreshFewerTiles = 6;

int launch_encode(const EncodeArgs &args, const EncodeArgs &fewer, int new_is_f32, const RefreshArgs *refresh, int arith, const int *resident_of,
                  int worker_cap, int order, bool order_free, int32_t ppm, int32_t room_ppm, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    EncodeArgs a = args;
    if (order_free && worker_cap == 0) {
        const int r = refresh ? 1 : 0;
        const TwoLaunches two = two_launches(a, new_is_f32, r, arith, ppm, room_ppm);
        if (two.form != kTickets) {
            uint16_t *counts = reinterpret_cast<uint16_t *>(a.tile_desc);
            if (two.form == kStaged) {
                hipLaunchKernelGGL(stage_variant(new_is_f32, r, arith), dim3(a.n_tiles), dim3(kThreads), 0, st, a, counts, a.slots,
                                   a.slot_size, two.stream);
                const int32_t group_wgs = a.n_blocks * (kBlock >> two.group_log2);
                const int32_t over_wgs = two.group_log2 == 0 ? 0 : a.n_tiles < kOverWgs ? a.n_tiles : kOverWgs;
                hipLaunchKernelGGL(emit_staged_variant(new_is_f32, r, arith), dim3(group_wgs + over_wgs), dim3(kThreads), 0, st, a,
                                   counts, a.slots, a.slot_size, two.group_log2, group_wgs);
            } else {
                const CountKernel count = new_is_f32 ? count_tiles_kernel<1> : count_tiles_kernel<0>;
                hipLaunchKernelGGL(count, dim3(a.n_tiles), dim3(kThreads), 0, st, a, counts);
                hipLaunchKernelGGL(emit_variant(new_is_f32, r, arith), dim3(a.n_tiles), dim3(kThreads), 0, st, a, counts);
            }
            launch_refresh_replicated(a, new_is_f32, refresh, st);
            return (int)hipGetLastError();
        }
    }
    const bool of_elements = arith && !new_is_f32 && !refresh && (ppm < 0 || ppm >= kElementsPpm || room_ppm >= kElementsPpm);
    int resident = resident_of[of_elements ? kElementsVariant : (new_is_f32 ? 1 : 0) + (refresh ? 2 : 0) + (arith ? 4 : 0)];
    if (ppm < 0 || ppm >= kSpreadFromPpm) a = fewer;           // see `moved` in plan.cpp
    encode_walk(order, ppm, room_ppm, new_is_f32, of_elements, refresh != nullptr, &a);
    // In turns: refreshes of little, by all workers.  (Of more, they were faster in turns as well: at 15 % 2428 and 2397 us, fp32 masters
    // at 20 % 6.6 and 4.5 ms.  They have been walked chain by chain since an encode of 40 % in turns by 70 workers gave up waiting; that
    // was no fault of the turns but a ticket on its way while tiles were counted ahead, see ticket_first.)
    a.turns = Turns{0, 0, 0, 0, 0};
    if (refresh && worker_cap == 0 && ppm >= 0 && ppm < kSpreadFromPpm && a.adjacent) a.turns = turns_of(a.block_first, a.tp);
    if (refresh && !new_is_f32 && !arith && (ppm < 0 || (ppm >= kRefreshFewerPpm && ppm < kRefreshFewerToPpm)) &&
        a.n_tiles / kRefreshFewerTiles >= a.n_pieces)
        resident -= resident / 4;
    if (resident < 1) return (int)hipErrorInvalidValue;
    // servers: one wave per block at most, ROSE_SERVER_WGS workgroups at most, and never more than
    // a quarter of what is resident.  They are the first workgroups of the grid, so they are
    // resident before any worker waits for them.
    int server_wgs = (a.n_blocks + kWaves - 1) / kWaves;
    if (server_wgs > ROSE_SERVER_WGS) server_wgs = ROSE_SERVER_WGS;
    if (server_wgs > resident / 4) server_wgs = resident / 4;
    if (server_wgs < 1) server_wgs = 1;
    int workers = resident - server_wgs;
    if (workers > a.n_tiles) workers = a.n_tiles;
    // the caller's cap: fewer workers than the device holds (never fewer than the progress
    // argument below needs)
    if (worker_cap > kBlock && worker_cap < workers) workers = worker_cap;
    // Progress with dynamic tickets: see the comment at struct Walk.  A worker that waits holds no
    // unpublished tile in the block it waits for or in an earlier one; what it waits for can still
    // need tickets of a partly handed-out group to be taken, by a worker that holds none of that
    // group's kBlock tickets.  Hence: more workers than tickets in a group.
    if (workers < 1) return (int)hipErrorInvalidValue;
    if (workers < a.n_tiles && workers <= kBlock) return (int)hipErrorInvalidValue;   // device holds too few workgroups
    a.n_server_wgs = server_wgs;
    a.n_servers = server_wgs * kWaves;
    a.n_tickets = ((a.n_blocks + a.batch - 1) / a.batch) * kBlock;
    // header, tile words and block words are one array
    const int64_t n_words = (int64_t)(kWsHeaderBytes / sizeof(u64)) + a.n_tiles + a.n_blocks;
    int reset_blocks = (int)((n_words + 1023) / 1024);
    if (reset_blocks > 2048) reset_blocks = 2048;
    hipLaunchKernelGGL(reset_kernel, dim3(reset_blocks), dim3(256), 0, st, reinterpret_cast<u64 *>(a.abort_flag), n_words,
                       (uint32_t)(of_elements ? kTicketsElements : kTickets), (uint32_t)(a.batch | a.turns.chains << 8));
    const dim3 grid(workers + server_wgs), block(kThreads);
    hipLaunchKernelGGL(of_elements ? encode_elements_kernel : encode_variant(new_is_f32, refresh ? 1 : 0, arith), grid, block, 0, st, a);
    launch_refresh_replicated(a, new_is_f32, refresh, st);
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(64), 0, st, a);
    return (int)hipGetLastError();
}

typedef void (*ApplyKernel)(BucketDev, int32_t, const int32_t *, void *const *, int, int64_t);
int launch_apply(const BucketDev &b, int32_t n_tensors, const int32_t *local_numel, void *const *dst_ptrs,
                 int arith, int64_t shard_elems, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool small = b.capacity <= (int64_t)kApplySmallChunks * 64;
    const bool sparse = !small && b.capacity < shard_elems / kApplySparseDiv;
    const bool middle = !small && !sparse && b.capacity < shard_elems / kApplyMiddleDiv;
    const ApplyKernel kernel = small ? apply_kernel<0, kApplySmallWaves, 8>
                             : sparse ? apply_kernel<1, kApplyWaves, 4>
                             : middle ? apply_kernel<0, kApplySmallWaves, 5> : apply_kernel<0, kApplyWaves, 8>;
    const int waves = small || middle ? kApplySmallWaves : kApplyWaves, per_wg = waves * 64;
    const int64_t want = (b.capacity + per_wg - 1) / per_wg;
    const int most = (sparse || b.capacity >= shard_elems / kApplyRoomyDiv ? kApplyBlocks : 2 * kApplyBlocks) * (kApplyWaves / waves);
    const int blocks = want < 1 ? 1 : (want > most ? most : (int)want);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(per_wg), 0, st, b, n_tensors, local_numel, dst_ptrs, arith,
                       shard_elems / kApplyDenseDiv);
    return (int)hipGetLastError();
}

// Entries up to which objects are packed and checked by workgroups of 1024 entries, one load a lane: 2048 of them.
// (Checked and applied, small objects: 0.9 us less than with 4096 entries a workgroup.  Packed, us, an entry per
// lane / 4096 / 1024: 168 k entries 2.9 / 4.1 / 3.0, from memory 5.0 / 9.0 / 3.8; 840 k 3.7 / 4.0 / 3.9, from memory
// 8.6 / 7.3 / 4.5.)
constexpr int64_t kFewEntries = 1 << 21;
int launch_pack(const BucketDev &b, int32_t shard, int32_t n_tensors, int64_t first, int64_t n, int32_t payload,
                void *object, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool few = n <= kFewEntries;
    const int64_t tile = few ? 1024 : 4096, want = (n + tile - 1) / tile;
    const int blocks = want < 1 ? 1 : (want > (1 << 20) ? 1 << 20 : (int)want);
    const auto pack = few ? pack_kernel<1> : pack_kernel<4>;
    hipLaunchKernelGGL(pack, dim3(blocks), dim3(256), 0, st, b, shard, n_tensors, first, n, payload, static_cast<char *>(object));
    return (int)hipGetLastError();
}

int launch_apply_object(const void *object, size_t object_bytes, int32_t n_tensors, int32_t n_buckets, int32_t tp,
                        const int32_t *local_numel, void *const *dst_ptrs, unsigned long long *verdict,
                        unsigned long long ticket, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool small = object_bytes / 6 <= (size_t)kApplySmallChunks * 64;
    const int per_wg = (small ? kApplySmallWaves : kApplyWaves) * 64;
    const int64_t want = ((int64_t)(object_bytes / 6) + per_wg - 1) / per_wg;
    const int blocks = want < 1 ? 1 : (want > kApplyBlocks ? kApplyBlocks : (int)want);
    const auto apply = small ? apply_object_kernel<kApplySmallWaves> : apply_object_kernel<kApplyWaves>;
    // one load a lane until that fills the device, then four
    const bool few = object_bytes / 6 <= (size_t)kFewEntries;
    const int64_t vtile = few ? 1024 : 4096, vwant = ((int64_t)(object_bytes / 6) + vtile - 1) / vtile;
    const int vblocks = vwant < 1 ? 1 : (vwant > 4096 ? 4096 : (int)vwant);
    const auto check = few ? object_validate_kernel<1> : object_validate_kernel<4>;
    hipLaunchKernelGGL(object_clear_kernel, dim3(1), dim3(1), 0, st, verdict);
    hipLaunchKernelGGL(check, dim3(vblocks), dim3(256), 0, st, static_cast<const char *>(object), object_bytes, n_tensors,
                       n_buckets, verdict, ticket);
    hipLaunchKernelGGL(apply, dim3(blocks), dim3(per_wg), 0, st, static_cast<const char *>(object),
                       object_bytes, n_tensors, n_buckets, tp, local_numel, dst_ptrs, verdict, ticket);
    return (int)hipGetLastError();
}

size_t object_bytes_for(int32_t n_tensors, int64_t n) { return object_size(n_tensors, n); }
bool object_header_valid(const uint32_t *h, int32_t n_tensors, size_t object_bytes, int64_t *n) {
    return object_header_ok(h, n_tensors, object_bytes, n);
}

int launch_dense_copy(const CopyArgs &a, int new_is_f32, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (a.n_tiles <= 0) return 0;
    if (new_is_f32)
        hipLaunchKernelGGL(dense_copy_kernel<1>, dim3(a.n_tiles), dim3(kThreads), 0, st, a);
    else
        hipLaunchKernelGGL(dense_copy_kernel<0>, dim3(a.n_tiles), dim3(kThreads), 0, st, a);
    return (int)hipGetLastError();
}

int launch_bw_probe(const void *src, void *dst, size_t bytes, uint64_t *sink, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    size_t n16 = bytes / 16;
    if (n16 == 0) return 0;
    size_t want = (n16 + kBwThreads * 4 - 1) / (kBwThreads * 4);
    int blocks = want > 256 * 32 ? 256 * 32 : (int)want;
    if (dst)
        hipLaunchKernelGGL(bw_copy_kernel, dim3(blocks), dim3(kBwThreads), 0, st,
                           static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), n16);
    else
        hipLaunchKernelGGL(bw_read_kernel, dim3(blocks), dim3(kBwThreads), 0, st,
                           static_cast<const uint4 *>(src), n16, reinterpret_cast<u64 *>(sink));
    return (int)hipGetLastError();
}

int launch_bw_probe_lines(void *dst, size_t n_lines, uint32_t threshold, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_lines == 0) return 0;
    const size_t blocks = (n_lines + 511) / 512;
    if (blocks > 0x7FFFFFFFull) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(bw_lines_kernel, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<uint4 *>(dst), n_lines, threshold);
    return (int)hipGetLastError();
}

int launch_bw_probe_mixed(const void *a, const void *b, void *dst, size_t n_chunks, uint32_t w16, int timed,
                          uint64_t *sink, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_chunks == 0) return 0;
    int blocks = n_chunks > 256 * 32 ? 256 * 32 : (int)n_chunks;
    if (timed)
        hipLaunchKernelGGL(bw_mix_kernel<1>, dim3(blocks), dim3(kBwThreads), 0, st, static_cast<const uint4 *>(a),
                           static_cast<const uint4 *>(b), static_cast<uint4 *>(dst), n_chunks, w16,
                           reinterpret_cast<u64 *>(sink));
    else
        hipLaunchKernelGGL(bw_mix_kernel<0>, dim3(blocks), dim3(kBwThreads), 0, st, static_cast<const uint4 *>(a),
                           static_cast<const uint4 *>(b), static_cast<uint4 *>(dst), n_chunks, w16,
                           reinterpret_cast<u64 *>(sink));
    return (int)hipGetLastError();
}

}  // namespace rose
