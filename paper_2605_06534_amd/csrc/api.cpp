// C ABI: argument checks, the plan's device tables, and hand-off to the kernel launchers.
#include <hip/hip_runtime_api.h>

#include <cstring>

#include "rose_internal.h"

namespace {

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Pinned host words that bucket checks read totals back into: a copy into ordinary memory goes through a
// staging buffer of the runtime's (8 bytes and the wait: 20.5 us; into pinned memory 12.2).  One small array
// for all plans that are resident somewhere, allocated with the first of them (180 us) and freed with the
// last.  A check holds one word while it runs; without the array, or with no word free, it uses ordinary
// memory.
class Mail {
public:
    bool share() {                                      // a plan becomes resident
        std::lock_guard<std::mutex> lock(mu_);
        if (!words_) {
            void *p = nullptr;
            if (hipHostMalloc(&p, kWords * sizeof(int64_t), hipHostMallocPortable) != hipSuccess) {
                (void)hipGetLastError();
                return false;
            }
            words_ = static_cast<int64_t *>(p);
            used_ = 0;
        }
        ++plans_;
        return true;
    }
    void give_back() {
        std::lock_guard<std::mutex> lock(mu_);
        if (--plans_ > 0 || used_) return;              // (a word that stayed taken keeps the array)
        (void)hipHostFree(words_);
        words_ = nullptr;
    }
    int64_t *take() {
        std::lock_guard<std::mutex> lock(mu_);
        if (!words_ || !~used_) return nullptr;
        const int i = __builtin_ctzll(~used_);
        used_ |= 1ull << i;
        return words_ + i;
    }
    void put(int64_t *word) {
        std::lock_guard<std::mutex> lock(mu_);
        used_ &= ~(1ull << (word - words_));
    }

private:
    static constexpr int kWords = 64;
    std::mutex mu_;
    int64_t *words_ = nullptr;
    uint64_t used_ = 0;                                 // bit i: word i is taken
    int plans_ = 0;
};
Mail mail;
constexpr size_t kOneCopyBytes = (size_t)1 << 20;       // tables gathered on the host; larger ones go there one by one

constexpr int32_t kNeighboursBelowPpm = rose::kSpreadFromPpm, kTimedBelowPpm = 40000;   // see encode_common

// Copy the piece and tile tables to the current device once; later calls on the same device
// reuse them.  A plan is bound to the first device it is used on.  `may_allocate` = false: only
// report whether the plan is resident here (nothing is allocated, ROSE_ERR_SCRATCH if it is not).
rose_status device_tables_locked(const rose_plan *p, bool may_allocate);
rose_status device_tables(const rose_plan *p, bool may_allocate = true) {
    std::lock_guard<std::mutex> lock(p->mu);
    try {
        return device_tables_locked(p, may_allocate);
    } catch (...) {                                     // host memory ran out while building the tables
        return ROSE_ERR_HIP;
    }
}

rose_status device_tables_locked(const rose_plan *p, bool may_allocate) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return ROSE_ERR_HIP;
    if (p->device == dev) return ROSE_OK;
    if (p->device != -1) return ROSE_ERR_ARG;
    if (!may_allocate) return ROSE_ERR_SCRATCH;

    // elements of a shard's copy of each tensor, per receiving stage (0: the stage does not hold it)
    std::vector<int32_t> numel((size_t)p->pp_dst * p->n_tensors, 0);
    for (int32_t i = 0; i < p->n_tensors; ++i) {
        const rose_tensor_desc &t = p->tensors[i];
        numel[(size_t)p->stage_dst_of[i] * p->n_tensors + i] =
            (int32_t)(t.rows * t.cols / (t.rule == ROSE_REPLICATED ? 1 : p->tp));
    }
    // replicated tensors the sender holds: a refresh copies them whole, sent from here or not
    std::vector<int32_t> repl;
    std::vector<int64_t> repl_numel;
    for (int32_t i = 0; i < p->n_tensors; ++i) {
        const rose_tensor_desc &t = p->tensors[i];
        if (t.rule == ROSE_REPLICATED && t.rows * t.cols > 0 && p->stage_src_of[i] == p->stage_src) {
            repl.push_back(i);
            repl_numel.push_back(t.rows * t.cols);
        }
    }
    // All tables lie in one allocation, and small ones go there in one copy: with an allocation and a copy for each a plan of
    // one matrix took 85 us (and that was before the dense copy had tables of its own), this way 64; one of 32 layers of
    // hidden 4096, TP4, 270 either way.
    struct Part {
        const void *from;                               // nullptr: zeros
        size_t bytes, at;
    };
    std::vector<Part> parts;
    size_t total = 0;
    auto add = [&](const void *from, size_t bytes) {
        parts.push_back({from, bytes, total});
        total += (bytes + 255) / 256 * 256;
        return parts.back().at;
    };
    auto add_table = [&](const auto &t) { return add(t.data(), t.size() * sizeof t[0]); };
    const size_t verdict_at = add(nullptr, kVerdictSlots * sizeof(unsigned long long));
    const size_t pieces_at = add_table(p->pieces), tile_piece_at = add_table(p->tile_piece);
    const size_t fewer_pieces_at = add_table(p->fewer.pieces), fewer_tile_piece_at = add_table(p->fewer.tile_piece);
    std::vector<int32_t> copy_table(p->copy_first);
    copy_table.insert(copy_table.end(), p->copy_piece.begin(), p->copy_piece.end());
    const size_t copy_at = add_table(copy_table), numel_at = add_table(numel);
    const size_t repl_at = add_table(repl), repl_numel_at = add_table(repl_numel);
    std::vector<char> all(total <= kOneCopyBytes ? total : 0);
    for (const Part &t : parts)
        if (!all.empty() && t.from && t.bytes) std::memcpy(all.data() + t.at, t.from, t.bytes);

    int resident[rose::kEncodeKernels];
    void *sws = nullptr;
    size_t sws_bytes = 0;
    char *base = nullptr;
    bool ok = hipMalloc(reinterpret_cast<void **>(&base), total) == hipSuccess;
    if (ok && !all.empty()) ok = hipMemcpy(base, all.data(), total, hipMemcpyHostToDevice) == hipSuccess;
    for (size_t i = 0; ok && all.empty() && i < parts.size(); ++i) {
        const Part &t = parts[i];
        if (!t.bytes) continue;
        ok = (t.from ? hipMemcpy(base + t.at, t.from, t.bytes, hipMemcpyHostToDevice) : hipMemset(base + t.at, 0, t.bytes)) == hipSuccess;
    }
    ok = ok && rose::encode_resident_all(resident) == 0 && rose::static_scratch(&sws, &sws_bytes) == 0;
    if (!ok) {
        if (base) (void)hipFree(base);
        return ROSE_ERR_HIP;
    }
    p->d_tables = base;
    p->d_verdict = reinterpret_cast<unsigned long long *>(base + verdict_at);
    p->d_pieces = reinterpret_cast<rose::Piece *>(base + pieces_at);
    p->d_tile_piece = reinterpret_cast<int32_t *>(base + tile_piece_at);
    if (!p->fewer.pieces.empty()) {
        p->d_fewer_pieces = reinterpret_cast<rose::Piece *>(base + fewer_pieces_at);
        p->d_fewer_tile_piece = reinterpret_cast<int32_t *>(base + fewer_tile_piece_at);
    }
    p->d_copy = reinterpret_cast<int32_t *>(base + copy_at);
    p->d_local_numel = reinterpret_cast<int32_t *>(base + numel_at);
    p->d_repl_list = reinterpret_cast<int32_t *>(base + repl_at);
    p->d_repl_numel = reinterpret_cast<int64_t *>(base + repl_numel_at);
    p->n_repl = (int32_t)repl.size();
    std::memcpy(p->resident, resident, sizeof resident);
    if (!p->uses_mail) p->uses_mail = mail.share();
    p->static_ws = sws;
    p->static_ws_bytes = sws_bytes;
    p->device = dev;
    return ROSE_OK;
}

rose_status check_bucket(const rose_bucket &b) {
    if (b.capacity < 0 || !b.seg_off) return ROSE_ERR_ARG;
    if (b.capacity > 0 && (!b.idx || !b.val)) return ROSE_ERR_ARG;
    if (!aligned(b.idx, 16) || !aligned(b.val, 16) || !aligned(b.seg_off, 8)) return ROSE_ERR_ALIGN;
    return ROSE_OK;
}

}  // namespace

extern "C" rose_status rose_plan_upload(const rose_plan *p) {
    if (!p) return ROSE_ERR_ARG;
    return device_tables(p);
}

extern "C" void rose_shard_plan_destroy(rose_plan *p) {
    if (!p) return;
    if (p->d_tables) (void)hipFree(p->d_tables);
    if (p->uses_mail) mail.give_back();
    delete p;
}

// Changed elements per million that these buckets could hold: no update of more of them is of use to anyone.
static int32_t room_ppm(const rose_plan *p, const rose_bucket *buckets) {
    double room = 0;
    for (int32_t d = 0; d < p->n_buckets; ++d) room += (double)(buckets[d].capacity > 0 ? buckets[d].capacity : 0);
    return p->capacity_sum > 0 && room < (double)p->capacity_sum ? (int32_t)(1e6 * room / (double)p->capacity_sum) : 1000000;
}

// Changed elements per million that a launch into these buckets is expected to find (-1: unknown): as many as the last time
// something was read back, until then as many as the buckets could hold.
static int32_t expected_ppm(const rose_plan *p, const rose_bucket *buckets) {
    const int32_t seen = p->seen_density_ppm.load(std::memory_order_relaxed);
    const int32_t room = seen < 0 ? room_ppm(p, buckets) : 0;
    return seen >= 0 ? seen : room < 1000000 ? room : -1;
}

// The tile order a launch into these buckets uses: the caller's choice, else by density.
static int pick_tile_order(const rose_plan *p, int32_t ppm) {
    int order = p->tile_order.load(std::memory_order_relaxed);
    if (order != ROSE_TILE_ORDER_AUTO_PICK) return order;
    return ppm < 0 ? ROSE_TILE_ORDER_SPREAD
                   : ppm < kTimedBelowPpm ? ROSE_TILE_ORDER_TIMED
                                          : ppm < kNeighboursBelowPpm ? ROSE_TILE_ORDER_NEIGHBOURS : ROSE_TILE_ORDER_SPREAD;
}

extern "C" rose_status rose_plan_pick_tile_order(const rose_plan *p, const rose_bucket *buckets, int32_t *order) {
    if (!p || !buckets || !order) return ROSE_ERR_ARG;
    *order = pick_tile_order(p, expected_ppm(p, buckets));
    return ROSE_OK;
}

// workspace = nullptr: the library's built-in scratch (the call must not allocate)
static rose_status encode_common(const rose_plan *p, const void *const *old_ptrs, const void *const *new_ptrs,
                                 int32_t new_dtype, const rose_bucket *buckets, void *workspace,
                                 size_t workspace_bytes, bool refresh, bool arith, void *stream) {
    const bool built_in = workspace == nullptr && workspace_bytes == (size_t)-1;
    if (!p || !old_ptrs || !new_ptrs || !buckets || (!workspace && !built_in)) return ROSE_ERR_ARG;
    if (new_dtype != ROSE_BF16 && new_dtype != ROSE_FP32_RNE) return ROSE_ERR_ARG;
    const size_t need = rose::workspace_need(p);
    if (!aligned(old_ptrs, 8) || !aligned(new_ptrs, 8)) return ROSE_ERR_ALIGN;
    rose::EncodeArgs a;
    std::memset(&a, 0, sizeof a);
    for (int32_t d = 0; d < p->n_buckets; ++d) {
        rose_status s = check_bucket(buckets[d]);
        if (s != ROSE_OK) return s;
        a.bucket[d].idx = buckets[d].idx;
        a.bucket[d].val = buckets[d].val;
        a.bucket[d].capacity = buckets[d].capacity;
        a.bucket[d].seg_off = buckets[d].seg_off;
    }
    rose_status s = device_tables(p, !built_in);
    if (s != ROSE_OK) return s;
    if (built_in) {
        if (need > p->static_ws_bytes) return ROSE_ERR_SCRATCH;
        workspace = p->static_ws;
        workspace_bytes = p->static_ws_bytes;
    }
    if (workspace_bytes < need) return ROSE_ERR_ARG;
    if (!aligned(workspace, 256)) return ROSE_ERR_ALIGN;
    a.old_ptrs = old_ptrs;
    a.new_ptrs = new_ptrs;
    char *ws = static_cast<char *>(workspace);
    a.abort_flag = reinterpret_cast<unsigned int *>(ws + rose::kWsAbortOff);
    a.ticket = reinterpret_cast<unsigned int *>(ws + rose::kWsTicketOff);
    a.tile_desc = reinterpret_cast<unsigned long long *>(ws + rose::kWsHeaderBytes);
    a.tp = p->n_buckets;
    a.n_tensors = p->n_tensors;
    rose::EncodeArgs fewer = a;
    auto set_tiles = [&](rose::EncodeArgs *e, const rose::Tiles &t, const rose::Piece *pieces, const int32_t *tile_piece) {
        std::memcpy(e->chain_first, t.chain_first, sizeof e->chain_first);
        std::memcpy(e->block_first, t.block_first, sizeof e->block_first);
        e->pieces = pieces;
        e->tile_piece = tile_piece;
        e->n_tiles = (int32_t)t.tile_piece.size();
        e->n_pieces = (int32_t)t.pieces.size();
        e->n_blocks = t.block_first[p->n_buckets];
        e->block_desc = e->tile_desc + e->n_tiles;
    };
    set_tiles(&a, *p, p->d_pieces, p->d_tile_piece);
    if (p->d_fewer_pieces) set_tiles(&fewer, p->fewer, p->d_fewer_pieces, p->d_fewer_tile_piece);
    else fewer = a;
    const size_t slots_at = (need + 255) / 256 * 256;
    if (a.n_tiles > 0 && a.n_tiles <= rose::kStageMostTiles && workspace_bytes > slots_at) {
        const size_t room = (workspace_bytes - slots_at) / sizeof(uint32_t) / (size_t)a.n_tiles / 32 * 32;   // whole lines
        a.slots = reinterpret_cast<uint32_t *>(ws + slots_at);
        a.slot_size = (int32_t)(room < (size_t)rose::kStageSlot ? room : (size_t)rose::kStageSlot);
    }
    rose::RefreshArgs r{p->d_repl_list, p->d_repl_numel, p->n_repl};
    const bool f32 = new_dtype == ROSE_FP32_RNE;
    // Tile order: the caller's choice, else picked from the density the plan's last checked launch showed
    // (7B-style workload on the same buffers, ms: timed 4.66 / 4.74 at 3.5 / 4 % where neighbours takes 4.78 /
    // 4.77, which pays from 4.5 % on; neighbours 5.29 / 5.46 / 6.19 at 7 / 8 / 10 % where spread takes
    // 5.37 / 5.47 / 5.63).
    const int32_t ppm = expected_ppm(p, buckets);
    const int order = pick_tile_order(p, ppm);
    const bool order_free = p->tile_order.load(std::memory_order_relaxed) == ROSE_TILE_ORDER_AUTO_PICK;
    return rose::launch_encode(a, fewer, f32, refresh ? &r : nullptr, arith ? 1 : 0, p->resident,
                               p->worker_cap.load(std::memory_order_relaxed), order, order_free, ppm,
                               room_ppm(p, buckets), stream) == 0
               ? ROSE_OK
               : ROSE_ERR_HIP;
}

extern "C" rose_status rose_delta_encode(const rose_plan *p, const void *const *old_ptrs,
                                         const void *const *new_ptrs, int32_t new_dtype,
                                         const rose_bucket *buckets, void *workspace,
                                         size_t workspace_bytes, void *stream) {
    return encode_common(p, old_ptrs, new_ptrs, new_dtype, buckets, workspace, workspace_bytes, false, false, stream);
}

extern "C" rose_status rose_delta_encode_refresh(const rose_plan *p, void *const *old_ptrs,
                                                 const void *const *new_ptrs, int32_t new_dtype,
                                                 const rose_bucket *buckets, void *workspace,
                                                 size_t workspace_bytes, void *stream) {
    return encode_common(p, const_cast<const void *const *>(old_ptrs), new_ptrs, new_dtype, buckets, workspace,
                         workspace_bytes, true, false, stream);
}

extern "C" rose_status rose_delta_encode_ex(const rose_plan *p, void *const *old_ptrs, const void *const *new_ptrs,
                                            int32_t new_dtype, uint32_t flags, const rose_bucket *buckets,
                                            void *workspace, size_t workspace_bytes, void *stream) {
    if (flags & ~(uint32_t)(ROSE_ENCODE_REFRESH | ROSE_ENCODE_ARITH)) return ROSE_ERR_ARG;
    return encode_common(p, const_cast<const void *const *>(old_ptrs), new_ptrs, new_dtype, buckets, workspace,
                         workspace_bytes, (flags & ROSE_ENCODE_REFRESH) != 0, (flags & ROSE_ENCODE_ARITH) != 0, stream);
}

extern "C" rose_status rose_delta_encode_static(const rose_plan *p, void *const *old_ptrs,
                                                const void *const *new_ptrs, int32_t new_dtype, uint32_t flags,
                                                const rose_bucket *buckets, void *stream) {
    if (flags & ~(uint32_t)(ROSE_ENCODE_REFRESH | ROSE_ENCODE_ARITH)) return ROSE_ERR_ARG;
    return encode_common(p, const_cast<const void *const *>(old_ptrs), new_ptrs, new_dtype, buckets, nullptr, (size_t)-1,
                         (flags & ROSE_ENCODE_REFRESH) != 0, (flags & ROSE_ENCODE_ARITH) != 0, stream);
}

static rose_status apply_common(const rose_plan *p, int32_t d, const rose_bucket *bucket, int32_t payload,
                                void *const *dst_ptrs, void *stream) {
    if (!p || !bucket || !dst_ptrs || d < 0 || d >= p->n_buckets) return ROSE_ERR_ARG;
    if (payload != ROSE_PAYLOAD_NEW && payload != ROSE_PAYLOAD_ARITH) return ROSE_ERR_ARG;
    rose_status s = check_bucket(*bucket);
    if (s != ROSE_OK) return s;
    if (!aligned(dst_ptrs, 8)) return ROSE_ERR_ALIGN;
    rose::BucketDev b{bucket->idx, bucket->val, bucket->capacity, bucket->seg_off};
    s = device_tables(p);
    if (s != ROSE_OK) return s;
    const int32_t *local_numel = p->d_local_numel + (size_t)(d / p->tp) * p->n_tensors;
    int64_t shard_elems = 0;
    for (int32_t i = 0; i < p->n_tensors; ++i)
        if (p->stage_dst_of[i] == d / p->tp) {
            const rose_tensor_desc &t = p->tensors[i];
            shard_elems += t.rows * t.cols / (t.rule == ROSE_REPLICATED ? 1 : p->tp);
        }
    return rose::launch_apply(b, p->n_tensors, local_numel, dst_ptrs, payload, shard_elems, stream) == 0 ? ROSE_OK
                                                                                                       : ROSE_ERR_HIP;
}

extern "C" rose_status rose_delta_apply(const rose_plan *p, int32_t d, const rose_bucket *bucket,
                                        void *const *dst_ptrs, void *stream) {
    return apply_common(p, d, bucket, ROSE_PAYLOAD_NEW, dst_ptrs, stream);
}

extern "C" rose_status rose_delta_apply_ex(const rose_plan *p, int32_t d, const rose_bucket *bucket, int32_t payload,
                                           void *const *dst_ptrs, void *stream) {
    return apply_common(p, d, bucket, payload, dst_ptrs, stream);
}

extern "C" rose_status rose_dense_copy(const rose_plan *p, int32_t d, const void *const *new_ptrs,
                                       int32_t new_dtype, void *const *dst_ptrs, void *stream) {
    if (!p || !new_ptrs || !dst_ptrs || d < 0 || d >= p->n_buckets) return ROSE_ERR_ARG;
    if (new_dtype != ROSE_BF16 && new_dtype != ROSE_FP32_RNE) return ROSE_ERR_ARG;
    if (!aligned(new_ptrs, 8) || !aligned(dst_ptrs, 8)) return ROSE_ERR_ALIGN;
    rose::CopyArgs a;
    std::memset(&a, 0, sizeof a);
    rose_status s = device_tables(p);
    if (s != ROSE_OK) return s;
    a.pieces = p->d_pieces;
    a.tile_piece = p->copy_piece.empty() ? p->d_tile_piece : p->d_copy + p->copy_first.size();
    a.first_tile = p->d_copy;
    a.new_ptrs = new_ptrs;
    a.dst_ptrs = dst_ptrs;
    a.tile_begin = p->copy_chain_first[d];
    a.n_tiles = p->copy_chain_first[d + 1] - p->copy_chain_first[d];
    return rose::launch_dense_copy(a, new_dtype == ROSE_FP32_RNE, stream) == 0 ? ROSE_OK : ROSE_ERR_HIP;
}

extern "C" rose_status rose_bucket_check(const rose_plan *p, const rose_bucket *bucket, void *stream,
                                         int64_t *required) {
    if (!p || !bucket || !bucket->seg_off) return ROSE_ERR_ARG;
    int64_t total = 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int64_t *word = mail.take();
    int64_t *to = word ? word : &total;
    // (a word whose copy may still be on its way after an error stays taken)
    // The runtime's copy and wait, not a kernel that writes the total for the host to look at: the stream is to be
    // synchronised, with its errors, and seg_off may lie where only the runtime can read it.  (Such a kernel and its look took
    // 14.0 us a check where this takes 19.7 as a caller in Python sees it; with the wait behind them 22.5.)
    if (hipMemcpyAsync(to, bucket->seg_off + p->n_tensors, sizeof total, hipMemcpyDeviceToHost, st) != hipSuccess)
        return ROSE_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return ROSE_ERR_HIP;
    if (word) {
        total = *static_cast<volatile int64_t *>(word);
        mail.put(word);
    }
    if (required) *required = total;
    if (total < 0) return ROSE_ERR_HIP;     // the encode launch gave up (see rose_delta_encode)
    if (p->capacity_sum > 0) {
        // what this bucket says about the update's density, taking the buckets to be about equal
        const double ppm = 1e6 * (double)total * p->n_buckets / (double)p->capacity_sum;
        p->seen_density_ppm.store(ppm > 1e6 ? 1000000 : (int32_t)ppm, std::memory_order_relaxed);
    }
    return total > bucket->capacity ? ROSE_ERR_CAPACITY : ROSE_OK;
}

extern "C" rose_status rose_bw_probe(const void *src, void *dst, size_t bytes, uint64_t *sink, void *stream) {
    if (!src || (bytes & 15u)) return ROSE_ERR_ARG;
    if (!dst && !sink) return ROSE_ERR_ARG;
    if (!aligned(src, 16) || !aligned(dst, 16) || !aligned(sink, 8)) return ROSE_ERR_ALIGN;
    return rose::launch_bw_probe(src, dst, bytes, sink, stream) == 0 ? ROSE_OK : ROSE_ERR_HIP;
}

static rose_status probe_mixed(const void *src_a, const void *src_b, void *dst, size_t read_bytes,
                               size_t write_bytes_per_chunk, int timed, uint64_t *sink, void *stream) {
    if (!src_a || !src_b || !dst || !sink) return ROSE_ERR_ARG;
    if ((read_bytes % ROSE_PROBE_CHUNK) || (write_bytes_per_chunk & 15u) || write_bytes_per_chunk > ROSE_PROBE_CHUNK)
        return ROSE_ERR_ARG;
    if (!aligned(src_a, 16) || !aligned(src_b, 16) || !aligned(dst, 16) || !aligned(sink, 8)) return ROSE_ERR_ALIGN;
    return rose::launch_bw_probe_mixed(src_a, src_b, dst, read_bytes / ROSE_PROBE_CHUNK,
                                       (uint32_t)(write_bytes_per_chunk / 16), timed, sink, stream) == 0
               ? ROSE_OK
               : ROSE_ERR_HIP;
}

extern "C" rose_status rose_bw_probe_mixed(const void *src_a, const void *src_b, void *dst, size_t read_bytes,
                                           size_t write_bytes_per_chunk, uint64_t *sink, void *stream) {
    return probe_mixed(src_a, src_b, dst, read_bytes, write_bytes_per_chunk, 0, sink, stream);
}

extern "C" rose_status rose_bw_probe_mixed_timed(const void *src_a, const void *src_b, void *dst, size_t read_bytes,
                                                 size_t write_bytes_per_chunk, uint64_t *sink, void *stream) {
    return probe_mixed(src_a, src_b, dst, read_bytes, write_bytes_per_chunk, 1, sink, stream);
}

extern "C" rose_status rose_bw_probe_lines(void *dst, size_t bytes, uint32_t touched_per_2_32, void *stream) {
    if (!dst || (bytes & 63u)) return ROSE_ERR_ARG;
    if (!aligned(dst, 64)) return ROSE_ERR_ALIGN;
    return rose::launch_bw_probe_lines(dst, bytes / 64, touched_per_2_32, stream) == 0 ? ROSE_OK : ROSE_ERR_HIP;
}

extern "C" rose_status rose_object_bytes(const rose_plan *p, int64_t n_entries, size_t *bytes) {
    if (!p || !bytes || n_entries < 0) return ROSE_ERR_ARG;
    *bytes = rose::object_bytes_for(p->n_tensors, n_entries);
    return ROSE_OK;
}

static rose_status pack_common(const rose_plan *p, int32_t d, const rose_bucket *bucket, int32_t payload,
                               int64_t first_entry, int64_t n_entries, void *object, size_t object_bytes,
                               void *stream) {
    if (!p || !bucket || !object || d < 0 || d >= p->n_buckets || first_entry < 0 || n_entries < 0) return ROSE_ERR_ARG;
    if (payload != ROSE_PAYLOAD_NEW && payload != ROSE_PAYLOAD_ARITH) return ROSE_ERR_ARG;
    rose_status s = check_bucket(*bucket);
    if (s != ROSE_OK) return s;
    if (!aligned(object, 16)) return ROSE_ERR_ALIGN;
    if (first_entry + n_entries > bucket->capacity) return ROSE_ERR_ARG;
    if (object_bytes < rose::object_bytes_for(p->n_tensors, n_entries)) return ROSE_ERR_CAPACITY;
    rose::BucketDev b{bucket->idx, bucket->val, bucket->capacity, bucket->seg_off};
    return rose::launch_pack(b, d, p->n_tensors, first_entry, n_entries, payload, object, stream) == 0 ? ROSE_OK
                                                                                                       : ROSE_ERR_HIP;
}

extern "C" rose_status rose_bucket_pack(const rose_plan *p, int32_t d, const rose_bucket *bucket, int64_t first_entry,
                                        int64_t n_entries, void *object, size_t object_bytes, void *stream) {
    return pack_common(p, d, bucket, ROSE_PAYLOAD_NEW, first_entry, n_entries, object, object_bytes, stream);
}

extern "C" rose_status rose_bucket_pack_ex(const rose_plan *p, int32_t d, const rose_bucket *bucket, int32_t payload,
                                           int64_t first_entry, int64_t n_entries, void *object, size_t object_bytes,
                                           void *stream) {
    return pack_common(p, d, bucket, payload, first_entry, n_entries, object, object_bytes, stream);
}

extern "C" rose_status rose_object_apply(const rose_plan *p, const void *object, size_t object_bytes,
                                         void *const *dst_ptrs, void *stream) {
    if (!p || !object || !dst_ptrs) return ROSE_ERR_ARG;
    if (!aligned(object, 16) || !aligned(dst_ptrs, 8)) return ROSE_ERR_ALIGN;
    if (object_bytes < rose::object_bytes_for(p->n_tensors, 0)) return ROSE_ERR_ARG;
    rose_status s = device_tables(p);
    if (s != ROSE_OK) return s;
    // the validation pass leaves its verdict in one of the plan's words; tickets tell the calls apart
    const uint64_t ticket = p->verdict_ticket.fetch_add(1, std::memory_order_relaxed) + 1;
    return rose::launch_apply_object(object, object_bytes, p->n_tensors, p->n_buckets, p->tp, p->d_local_numel, dst_ptrs,
                                     p->d_verdict + ticket % kVerdictSlots, ticket, stream) == 0
               ? ROSE_OK
               : ROSE_ERR_HIP;
}

extern "C" rose_status rose_object_check(const rose_plan *p, const void *object, size_t object_bytes, void *stream,
                                         int32_t *shard, int64_t *first_entry, int64_t *n_entries,
                                         int32_t *payload) {
    if (!p || !object || object_bytes < 64) return ROSE_ERR_ARG;
    uint32_t h[16];
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(h, object, sizeof h, hipMemcpyDeviceToHost, st) != hipSuccess) return ROSE_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return ROSE_ERR_HIP;
    int64_t n = 0;
    if (!rose::object_header_valid(h, p->n_tensors, object_bytes, &n)) return ROSE_ERR_ARG;
    if ((int32_t)h[2] < 0 || (int32_t)h[2] >= p->n_buckets) return ROSE_ERR_ARG;
    if (shard) *shard = (int32_t)h[2];
    if (first_entry) *first_entry = (int64_t)((uint64_t)h[4] | ((uint64_t)h[5] << 32));
    if (n_entries) *n_entries = n;
    if (payload) *payload = (int32_t)h[8];
    return ROSE_OK;
}
