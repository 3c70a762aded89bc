// Internal declarations shared by the host planner, the C ABI and the kernel launchers.
#pragma once

#include <atomic>
#include <cstddef>
#include <cstdint>
#include <mutex>
#include <vector>

#include "rose_delta.h"

namespace rose {

// Tile geometry of the encode / dense-copy kernels: one workgroup of kThreads lanes walks one
// tile; a lane takes kIters vectors of kVec 16-bit elements (one 128-bit load each).
#ifndef ROSE_THREADS
#define ROSE_THREADS 256
#endif
constexpr int kThreads = ROSE_THREADS;
constexpr int kWaves = kThreads / 64;
constexpr int kVec = 8;
#ifndef ROSE_ITERS
#define ROSE_ITERS 4
#endif
constexpr int kIters = ROSE_ITERS;
constexpr int kWaveSpan = 64 * kVec * kIters;      // elements one wave covers in a tile
constexpr int kTile = kThreads * kVec * kIters;    // elements per tile
constexpr int kShiftElems = 64;                     // 16-bit elements in a 128-byte line
constexpr int kShiftFewestTiles = 4;                // tiles of a piece that is moved (kPieceShift) ...
constexpr int kShiftLeastTiles = 32;                // ... at the price of one more

enum : int32_t {
    kPieceFirst = 1,    // first piece of its (tensor, shard) segment
    kPieceStrided = 4,  // runs of `run` elements every `stride` source elements
    kPieceReplicated = 16, // piece of a replicated tensor: several destinations read the same source
    kPieceLoad16 = 32,  // a vector of kVec elements is one 128-bit load of the source, at any alignment: the source is
                        // contiguous or its runs are at least kVec long (then two, see kPieceSplit)
    kPieceSplit = 64,   // with kPieceLoad16: source runs that are no multiple of kVec, a vector may straddle two
    kPieceShift = 128,  // its tiles may be moved down to 128-byte lines of the source: several tiles, and the source is
                        // contiguous or in runs and strides of whole lines.  There are tiles enough for the piece moved
                        // as far as can be (one more where it fills its last one; that is empty if nothing is moved)
    kPieceDstStrided = 8 // runs of `run` elements every `lstride` LOCAL indices (the sender's slice
                        // covers only part of each row of the destination shard)
};

// One part of a (tensor, shard) segment: element k = 0 .. len-1 of the piece lies at
//   source element  src_off + k                              (contiguous)
//                   src_off + (k / run) * stride + k % run   (kPieceStrided: a column block of a
//                                                             row-parallel matrix)
//   local index     local_base + k                           (contiguous)
//                   local_base + (k / run) * lstride + k % run   (kPieceDstStrided)
// Both are ascending in k.
struct Piece {
    int64_t src_off;
    int64_t stride;
    int32_t tensor;
    int32_t shard;
    int32_t local_base;
    int32_t len;
    int32_t run;
    uint32_t magic;      // k / run == mulhi(k, magic) >> shift for k < 2^31 (run >= 2)
    uint32_t shift;
    int32_t first_tile;
    int32_t flags;
    int32_t lstride;
};
static_assert(sizeof(Piece) == 56, "Piece layout is shared with device code");

// Pieces, shard by shard, and the tiles they are cut into: one prefix chain of tiles per shard, in blocks of kBlock.
struct Tiles {
    std::vector<Piece> pieces;
    std::vector<int32_t> tile_piece;           // piece of each tile
    int32_t chain_first[ROSE_MAX_TP + 1] = {0};
    int32_t block_first[ROSE_MAX_TP + 1] = {0};
};

#ifdef __HIP__
#define ROSE_BOTH __host__ __device__
#else
#define ROSE_BOTH
#endif
#define ROSE_INLINE ROSE_BOTH inline __attribute__((always_inline))

// host side of the magic-number division used for strided pieces
void make_magic(uint32_t divisor, uint32_t *magic, uint32_t *shift);
ROSE_BOTH inline uint32_t magic_div(uint32_t k, uint32_t magic, uint32_t shift) {
    return (uint32_t)(((uint64_t)k * magic) >> 32) >> shift;
}

// Blocks are numbered chain by chain, and walked in that order, or (where a launch walks in turns) those of the chains
// chain .. chain + chains - 1 in turn, a block of each, `each` times; what the longer ones have besides comes behind.  The
// blocks of one chain are walked in their order in any case, which is all that the waits for prefixes rest on.
struct Turns {
    int32_t chain, chains, each;
    uint32_t magic, shift;                  // k / chains
};
Turns turns_of(const int32_t *block_first, int32_t n_chains);
struct WalkedBlock {
    int32_t shard, blk;
};
// the n-th block that is walked in turns
ROSE_BOTH inline WalkedBlock walked_block(const Turns &t, const int32_t *block_first, int32_t n) {
    WalkedBlock b;
    int32_t x = n - block_first[t.chain];
    const int32_t in_turn = t.chains * t.each;
    if (x >= 0 && x < in_turn) {
        const int32_t q = (int32_t)magic_div((uint32_t)x, t.magic, t.shift);
        b.shard = t.chain + (x - q * t.chains);
        b.blk = block_first[b.shard] + q;
        return b;
    }
    if (x >= in_turn && n < block_first[t.chain + t.chains]) {
        b.shard = t.chain;
        x -= in_turn;
        for (int32_t rest; x >= (rest = block_first[b.shard + 1] - block_first[b.shard] - t.each); ++b.shard) x -= rest;
        b.blk = block_first[b.shard] + t.each + x;
        return b;
    }
    b.shard = 0;
    b.blk = n;
    while (n >= block_first[b.shard + 1]) ++b.shard;
    return b;
}

struct BucketDev {
    int32_t *idx;
    uint16_t *val;
    int64_t capacity;
    int64_t *seg_off;
};

struct EncodeArgs {
    BucketDev bucket[ROSE_MAX_TP];
    int32_t chain_first[ROSE_MAX_TP + 1];   // first tile of each shard's chain; [tp] = n_tiles
    const Piece *pieces;
    const int32_t *tile_piece;
    const void *const *old_ptrs;
    const void *const *new_ptrs;
    int32_t block_first[ROSE_MAX_TP + 1];   // first block descriptor of each shard's chain
    unsigned long long *tile_desc;          // one descriptor per tile
    unsigned long long *block_desc;         // one descriptor per block of kBlock tiles of a chain
    unsigned int *abort_flag;               // workspace header: set when a wait gave up
    int32_t n_tiles;
    int32_t n_pieces;
    int32_t n_blocks;
    int32_t n_tensors;
    int32_t tp;
    int32_t n_server_wgs;                   // workgroups 0 .. n_server_wgs-1 serve prefixes, the rest walk tiles
    int32_t n_servers;                      // waves that serve prefixes (kWaves per serving workgroup)
    int32_t n_tickets;                      // tickets the counter hands out
    int32_t adjacent;                       // a ticket's tiles are neighbours in the bucket (see ticket_tile)
    int32_t batch;                          // tiles per ticket
    uint32_t window_open;                   // clock ticks of a period in which bucket stores go out (0: always)
    uint32_t window_mask;                   // ticks of a period (a power of two) less one
    Turns turns;                            // in which a refresh walks its blocks
    unsigned int *ticket;                   // workspace header: the ticket counter
    uint32_t *slots;                        // one slot of slot_size entries per tile (see stage_tiles_kernel)
    int32_t slot_size;                      // 0: the workspace has no room for slots
};

// Tiles of one chain are grouped in blocks of kBlock; a serving wave gathers a block's counts
// and hands every tile of the block its prefix.
constexpr int kBlock = 64;

// A ticket hands a worker a batch of tiles: the tiles at one position of as many consecutive blocks
// (a "group" of blocks has kBlock tickets).  All tickets come from one counter, in order.  The
// counter serves one ticket in about 14 ns, whoever asks: with 3 tiles (96 KB of input) per ticket it
// alone caps a launch at about 6 TB/s; the launches that can read faster than that take 4 (encode_walk).
#ifndef ROSE_BATCH
#define ROSE_BATCH 3
#endif
#ifndef ROSE_BATCH_TIMED
#define ROSE_BATCH_TIMED 4
#endif
constexpr int kBatch = ROSE_BATCH, kBatchTimed = ROSE_BATCH_TIMED;

// The n-th block in the order in which a launch walks them.
template <int TURNS>
ROSE_INLINE WalkedBlock nth_block(const EncodeArgs &a, int32_t n, int32_t shard) {
    if constexpr (TURNS) return walked_block(a.turns, a.block_first, n);
    while (n >= a.block_first[shard + 1]) ++shard;     // (blocks are numbered chain by chain; shard: that of an earlier one)
    return {shard, n};
}

// The j-th tile of a ticket, or -1 if there is none.  A ticket stands for a.batch tiles (kBatch below; the
// launcher picks it).  A group of kBatch consecutive blocks has
// kBatch * kBlock tile positions ("slots", block after block) and kBlock tickets.  Two orders:
// spread (a.adjacent = 0): ticket n of the group stands for position n of each of the group's blocks, so
// that a block's 64 tiles are walked by 64 workers at once and its prefixes are ready one tile-time
// later; neighbours (a.adjacent = 1): ticket n stands for the kBatch NEIGHBOURING slots
// n * kBatch .. n * kBatch + kBatch - 1.  Neighbouring slots are
// neighbouring tiles of one chain (except where a chain ends inside the group: a chain's short last
// block has no tile for its last positions), so the entries of a ticket's tiles follow each other in
// the bucket and are written as one run: only the two ends of a ticket's run share 64-byte lines of
// the bucket with another workgroup's.  (Measured on the 7B-style workload with every run padded to
// whole lines, which is what no shared lines at all would give: 3 % faster at 1 - 5 %, 7 % at 10 %.)
// The price: a block's prefixes are ready kBatch tile-times later, so more entries wait in the ring,
// which pays while the ring holds them (see launch_encode for who picks the order).  Uniform.
template <int TURNS>
ROSE_INLINE int32_t tile_of_ticket(const EncodeArgs &a, int32_t ticket, int32_t j) {
    int32_t blk = (ticket / kBlock) * a.batch + j, pos = ticket & (kBlock - 1);
    if (a.adjacent) {
        const int32_t slot = (ticket & (kBlock - 1)) * a.batch + j;
        blk = (ticket / kBlock) * a.batch + slot / kBlock;
        pos = slot & (kBlock - 1);
    }
    if (blk >= a.n_blocks) return -1;
    const WalkedBlock b = nth_block<TURNS>(a, blk, 0);
    const int32_t t = a.chain_first[b.shard] + (b.blk - a.block_first[b.shard]) * kBlock + pos;
    return t < a.chain_first[b.shard + 1] ? t : -1;
}

// A worker's position in the tile order it is given by its tickets (uniform state).
//
// Waiting and tickets.  A worker may wait for the prefix of a parked tile X only while every tile
// it holds a ticket for and has not published lies in a block walked later than X's (see Turns): then the earliest
// block that is not fully published never depends on a waiting worker, and all waits end.  Tickets
// are taken in order, so the tiles of a worker's tickets lie in later and later groups, except
// when two tickets in a row fall into the SAME group (few workers are taking tickets, e.g. while
// most of them wait).  Such a pair is handled with care: from the moment the second ticket is
// accepted nothing waits until the counts of all tiles of both tickets are published by a
// count-only pass; then those tiles are walked again ("redo", without publishing) in the normal
// way.  While redoing, no further ticket is asked for, nor is one on its way when a redo begins (see ticket_first): one of
// the same group, accepted in the middle of a redo, would have tiles counted that are published already, and a count stored
// over a prefix is a prefix that nobody stores again.
// The same machinery serves tiles so dense that the ring does not hold a ticket's worth of them: a
// worker that would have to wait for room with fewer tiles parked than a ticket has, and with tiles
// of the current ticket still uncounted, counts those first and walks the ticket again from the
// current tile on.  (Waiting there is allowed by the rule above, but every later group of workers
// would wait for those counts in turn, and the groups would run one after the other.)
struct Walk {
    int32_t ticket, j;          // ticket in use (-1: none yet) and its batch slot
    int32_t next_ticket;        // ticket fetched ahead of time
    int32_t redo_through;       // last ticket of a redo
    bool have_next;
    bool exhausted;             // the counter has run out
    bool careful;               // a same-group ticket was accepted; its counts are not published yet
    bool redo;                  // tiles up to the end of ticket redo_through are published already
};
enum : int { kWalkTile = 0, kWalkNeedTicket = 1, kWalkDone = 2 };

// Whether a ticket that is on its way is taken in before the tile at hand is dealt with: where the worker may come to wait
// for room (full), since the ticket could be of the current one's group, and where it will count the rest of the current ticket
// and walk it again (ahead).
ROSE_INLINE bool ticket_first(const Walk &w, bool ticket_out, bool full, bool ahead) {
    return ticket_out && !w.careful && (full || ahead);
}

// take in the counter's answer n; false if it is none
ROSE_INLINE bool walk_accept(int32_t n_tickets, Walk &w, uint32_t n) {
    if (n >= (uint32_t)n_tickets) {
        w.exhausted = true;
    } else if ((int32_t)n <= w.ticket) {
        // One counter hands the tickets out in order, so a worker's tickets increase.  A value that
        // does not is not a ticket: walk no further.
        w.exhausted = true;
        return false;
    } else {
        w.next_ticket = (int32_t)n;
        w.have_next = true;
        if (w.ticket >= 0 && (int32_t)n / kBlock == w.ticket / kBlock) w.careful = true;
    }
    return true;
}

// Advance to the next tile; tile_of(ticket, j): see tile_of_ticket.  kWalkNeedTicket: the current ticket is used up and no
// further one is at hand (ask the counter, then call again); kWalkDone: no tiles are left.
template <typename TILE_OF>
ROSE_INLINE int walk_step(int32_t batch, Walk &w, int32_t *tile, const TILE_OF &tile_of) {
    for (;;) {
        while (w.j + 1 < batch) {
            ++w.j;
            const int32_t t = tile_of(w.ticket, w.j);
            if (t >= 0) {
                *tile = t;
                return kWalkTile;
            }
        }
        w.j = batch;
        if (w.redo && w.ticket == w.redo_through) w.redo = false;
        if (!w.have_next) return w.exhausted ? kWalkDone : kWalkNeedTicket;
        w.ticket = w.next_ticket;
        w.have_next = false;
        w.j = -1;
    }
}

// workspace layout (bytes): header, tile descriptors, block descriptors
constexpr size_t kWsAbortOff = 0;
constexpr int kWsCarefulWord = 2;      // 32-bit word 2 of the header counts same-group ticket pairs (diagnostic)
constexpr int kWsAheadWord = 3;        // 32-bit word 3: how often tiles were counted ahead of a wait (diagnostic)
constexpr int kWsTilesWord = 4;        // 32-bit word 4: tiles of a launch without tickets, else 0
constexpr int kWsFormWord = 5;         // 32-bit word 5: 0 after tickets (3: payloads formed of every element), 1 entries parked, 2 all read again
constexpr int kWsWalkWord = 6;         // 32-bit word 6, after tickets: tiles a ticket, and from bit 8 on how many chains took turns
constexpr size_t kWsTicketOff = 4096;
constexpr size_t kWsHeaderBytes = 8192;
// Behind them (at a multiple of 256 bytes): room for compacted entries, a slot per tile, of the plans that may be encoded
// without tickets.  A call asks for the part in front only and uses what room there is.
constexpr int64_t kStageMostTiles = 65536;               // 2 GiB read in bf16
constexpr size_t kStageMostBytes = ROSE_STATIC_SCRATCH_BYTES;   // all of it together, so that the built-in scratch holds it
constexpr int kStageSlot = 2016;                         // entries of a slot at most: 24 % of a tile, 8 KB of LDS a workgroup

// Plans of at most so many tiles have a numbering of their own for the dense copy's (copy_tiles).
constexpr int64_t kCopyOwnTiles = 65536;

struct CopyArgs {
    const Piece *pieces;
    const int32_t *tile_piece;              // piece of each tile
    const int32_t *first_tile;              // first tile of each piece
    const void *const *new_ptrs;
    void *const *dst_ptrs;
    int32_t tile_begin;
    int32_t n_tiles;
};

constexpr int32_t kSpreadFromPpm = 75000;  // changed elements per million from which tiles are taken in the spread order

// kernel launchers (kernels.hip); all return a hipError_t as int
// replicated tensors to copy new -> old after an encode with refresh (device arrays of n entries)
struct RefreshArgs {
    const int32_t *list;
    const int64_t *numel;
    int32_t n;
};
// resident: workgroups of each kernel variant that fit on the device at once (encode_resident_all);
// worker_cap: 0, or the most workgroups that may walk tiles; order: ROSE_TILE_ORDER_SPREAD, _NEIGHBOURS or _TIMED;
// order_free: nobody asked for that order, small updates may go without tickets; ppm: changed elements per
// million as far as known or bounded, else -1; room_ppm: as many as the buckets could hold
// a, fewer: with the plan's tiles and with those where only the longer pieces are moved (everything else is alike)
int launch_encode(const EncodeArgs &a, const EncodeArgs &fewer, int new_is_f32, const RefreshArgs *refresh, int arith, const int *resident,
                  int worker_cap, int order, bool order_free, int32_t ppm, int32_t room_ppm, void *stream);
// resident workgroups of each of the encode kernel variants on the current device
// (index: fp32 input + 2 * refresh + 4 * arithmetic payload; 8: arithmetic payloads formed of every element)
constexpr int kEncodeKernels = 9;
int encode_resident_all(int resident[kEncodeKernels]);
// Address and size of the library's built-in scratch array on the current device (one array per
// device, found once per device with hipGetSymbolAddress and kept).
int static_scratch(void **ptr, size_t *bytes);
// shard_elems: elements of the destination shard's tensors together (the kernel compares the entry
// count with it to choose how it walks the entries)
int launch_apply(const BucketDev &b, int32_t n_tensors, const int32_t *local_numel, void *const *dst_ptrs,
                 int arith, int64_t shard_elems, void *stream);
int launch_dense_copy(const CopyArgs &a, int new_is_f32, void *stream);
int launch_pack(const BucketDev &b, int32_t shard, int32_t n_tensors, int64_t first, int64_t n, int32_t payload,
                void *object, void *stream);
// local_numel: [n_stages][n_tensors]; the object's shard word b selects row b / tp.  verdict: one word of
// device memory that belongs to this call until its kernels have run; ticket: a value no other call
// that shares the word uses.
int launch_apply_object(const void *object, size_t object_bytes, int32_t n_tensors, int32_t n_buckets, int32_t tp,
                        const int32_t *local_numel, void *const *dst_ptrs, unsigned long long *verdict,
                        unsigned long long ticket, void *stream);
size_t object_bytes_for(int32_t n_tensors, int64_t n);
bool object_header_valid(const uint32_t *header, int32_t n_tensors, size_t object_bytes, int64_t *n);
int launch_bw_probe(const void *src, void *dst, size_t bytes, uint64_t *sink, void *stream);
int launch_bw_probe_lines(void *dst, size_t n_lines, uint32_t threshold, void *stream);
int launch_bw_probe_mixed(const void *a, const void *b, void *dst, size_t n_chunks, uint32_t w16, int timed,
                          uint64_t *sink, void *stream);

}  // namespace rose

// words of device memory that object applies use to hand the validation pass's verdict to the apply pass
constexpr int kVerdictSlots = 4096;

struct rose_plan : rose::Tiles {               // (its tiles with all pieces moved that may be)
    int32_t tp_src = 1, src_rank = 0;          // the sender holds shard src_rank of tp_src of every tensor
    int32_t tp = 0;
    // pipeline stages (Sec. 4.2: TP and PP on both sides): the sender is stage stage_src of pp_src and holds
    // the tensors of that stage only; the receiving side has pp_dst stages of tp shards each.  Bucket (and
    // prefix chain) b = stage * tp + shard.
    int32_t n_layers = 0, pp_src = 1, stage_src = 0, pp_dst = 1;
    int32_t n_buckets = 0;                     // tp * pp_dst
    int32_t n_tensors = 0;
    std::vector<rose_tensor_desc> tensors;
    std::vector<int32_t> stage_src_of, stage_dst_of;   // [n_tensors] stage that holds each tensor on either side
    std::vector<int64_t> global_base;          // [n_tensors + 1]
    rose::Tiles fewer;                         // tiles with only the longer pieces moved (no pieces: the plan's own)
    std::vector<int32_t> copy_piece;           // piece of each of the dense copy's tiles (empty: it has the encode's)
    std::vector<int32_t> copy_first;           // first of its tiles of each piece
    int32_t copy_chain_first[ROSE_MAX_TP + 1] = {0};
    mutable std::atomic<int32_t> worker_cap{0};     // rose_plan_set_worker_cap
    mutable std::atomic<int32_t> tile_order{0};     // rose_plan_set_tile_order
    mutable std::atomic<int32_t> seen_density_ppm{-1};   // changed elements per million as estimated from the last
                                                         // bucket total that rose_bucket_check read back (-1: none yet)
    int64_t capacity_sum = 0;                            // entries of all buckets together if every element changed
    mutable std::atomic<uint64_t> verdict_ticket{0};
    // device copies of pieces / tile_piece, made on first use on a device (the only device the plan is used on)
    mutable std::mutex mu;
    mutable int device = -1;
    mutable void *d_tables = nullptr;          // the allocation that holds all of these
    mutable rose::Piece *d_pieces = nullptr;
    mutable int32_t *d_tile_piece = nullptr;
    mutable rose::Piece *d_fewer_pieces = nullptr;     // the same of `fewer`, if there are
    mutable int32_t *d_fewer_tile_piece = nullptr;
    mutable int32_t *d_copy = nullptr;         // copy_first, then copy_piece
    mutable int32_t *d_local_numel = nullptr;  // [pp_dst][n_tensors] elements of a shard's copy of each tensor
                                               // (0 where the stage does not hold the tensor)
    mutable int32_t *d_repl_list = nullptr;    // replicated tensors this sender holds (ordinals) and their sizes
    mutable int64_t *d_repl_numel = nullptr;
    mutable int32_t n_repl = 0;
    mutable unsigned long long *d_verdict = nullptr;   // [kVerdictSlots]
    mutable int resident[rose::kEncodeKernels] = {0};   // see encode_resident_all
    mutable bool uses_mail = false;            // holds a share of the pinned words of bucket checks (api.cpp)
    mutable void *static_ws = nullptr;         // the library's built-in scratch on `device`
    mutable size_t static_ws_bytes = 0;
};

namespace rose {
size_t workspace_need(const rose_plan *p);     // bytes of scratch that an encode cannot do without
}
