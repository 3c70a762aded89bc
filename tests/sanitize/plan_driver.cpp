// Runs the host planner (csrc/plan.cpp, no GPU code) under AddressSanitizer and
// UndefinedBehaviorSanitizer: plans for every rule, sender-side degrees, group-interleaved fused
// tensors and rejected descriptors; every query; every element's index map against the element
// count per shard.  Built and started by tests/test_host_sanitizers.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "rose_internal.h"

static void fail(const char *what, int rc) {
    std::printf("FAILED: %s (%d)\n", what, rc);
    std::exit(1);
}

static rose_tensor_desc desc(int64_t rows, int64_t cols, int32_t rule, std::vector<int64_t> sec = {}, int32_t groups = 0) {
    rose_tensor_desc t;
    std::memset(&t, 0, sizeof t);
    t.rows = rows;
    t.cols = cols;
    t.rule = (rose_rule)rule;
    t.n_sections = (int32_t)sec.size();
    for (size_t i = 0; i < sec.size(); ++i) t.section_rows[i] = sec[i];
    t.src_groups = groups;
    return t;
}

static void copy_tiles(const rose_plan *p, int32_t tp) {
    // the dense copy's tiles: each piece as many as it fills, one if it is empty, one piece behind the other; those of
    // the encode for a plan of many
    int64_t c = 0;
    for (size_t k = 0; k < p->pieces.size(); ++k) {
        const rose::Piece &pc = p->pieces[k];
        const int32_t next = k + 1 < p->pieces.size() ? p->pieces[k + 1].first_tile : (int32_t)p->tile_piece.size();
        const int64_t nt = p->copy_piece.empty() ? next - pc.first_tile : pc.len == 0 ? 1 : (pc.len + rose::kTile - 1) / rose::kTile;
        if (p->copy_first[k] != c || c < p->copy_chain_first[pc.shard] || c + nt > p->copy_chain_first[pc.shard + 1])
            fail("first tile of a copy", (int)k);
        const std::vector<int32_t> &of = p->copy_piece.empty() ? p->tile_piece : p->copy_piece;
        for (int64_t j = 0; j < nt; ++j, ++c)
            if (c >= (int64_t)of.size() || of[c] != (int32_t)k) fail("piece of a copy's tile", (int)c);
        if (p->copy_piece.empty() && pc.first_tile != p->copy_first[k]) fail("shared tiles", (int)k);
    }
    if (c != p->copy_chain_first[tp] || (!p->copy_piece.empty() && c != (int64_t)p->copy_piece.size())) fail("tiles of a copy", (int)c);
    if (p->copy_piece.empty() != (p->tile_piece.size() > (size_t)rose::kCopyOwnTiles)) fail("whose tiles", (int)c);
}

// the tiles of one numbering: every piece's in order, as many as its elements need, chains and blocks as they follow
static void tiles(const rose::Tiles &t, int32_t n_chains, bool all) {
    int64_t n = 0;
    int32_t blocks = 0;
    for (size_t k = 0; k < t.pieces.size(); ++k) {
        const rose::Piece &pc = t.pieces[k];
        const bool shift = (pc.flags & rose::kPieceShift) != 0;
        const int64_t filled = (pc.len + rose::kTile - 1) / rose::kTile, reached = (pc.len + rose::kShiftElems - 1 + rose::kTile - 1) / rose::kTile;
        if (pc.first_tile != n || n < t.chain_first[pc.shard] || n >= t.chain_first[pc.shard + 1]) fail("first tile", (int)k);
        if (shift && (pc.len <= rose::kTile || (!all && filled < (reached == filled ? rose::kShiftFewestTiles : rose::kShiftLeastTiles)))) fail("moved", (int)k);
        const int64_t nt = pc.len == 0 ? 1 : shift ? reached : filled;
        for (int64_t j = 0; j < nt; ++j, ++n)
            if (n >= (int64_t)t.tile_piece.size() || t.tile_piece[n] != (int32_t)k) fail("piece of a tile", (int)n);
    }
    if (n != (int64_t)t.tile_piece.size() || t.chain_first[n_chains] != n) fail("tiles", (int)n);
    for (int32_t b = 0; b < n_chains; ++b) {
        if (t.block_first[b] != blocks) fail("blocks", b);
        blocks += (t.chain_first[b + 1] - t.chain_first[b] + rose::kBlock - 1) / rose::kBlock;
    }
    if (t.block_first[n_chains] != blocks) fail("blocks", n_chains);
}

static void both_tiles(const rose_plan *p, int32_t n_chains) {
    tiles(*p, n_chains, true);
    if (p->fewer.pieces.empty()) return;
    tiles(p->fewer, n_chains, false);
    if (p->fewer.pieces.size() != p->pieces.size() || p->fewer.tile_piece.size() > p->tile_piece.size()) fail("two numberings", 0);
}

static void walk(const std::vector<rose_tensor_desc> &ts, int32_t tp, int32_t tp_src, int32_t src_rank) {
    rose_plan *p = nullptr;
    rose_status s = rose_shard_plan_create_src(ts.data(), (int32_t)ts.size(), tp, tp_src, src_rank, &p);
    if (s != ROSE_OK) fail("create", s);
    int64_t v = 0;
    size_t bytes = 0;
    if (rose_plan_n_tensors(p) != (int32_t)ts.size() || rose_plan_tp(p) != tp) fail("counts", 0);
    if (rose_plan_workspace_bytes(p, &bytes) != ROSE_OK || bytes < 8192) fail("workspace", 0);
    if (rose_plan_n_tiles(p, &v) != ROSE_OK || v < 1) fail("tiles", 0);
    for (int32_t d = 0; d < tp; ++d)
        if (rose_plan_bucket_capacity(p, d, &v) != ROSE_OK || v < 0) fail("capacity", d);
    for (int32_t t = 0; t < (int32_t)ts.size(); ++t) {
        int64_t base = 0, src = 0;
        if (rose_plan_tensor_base(p, t, &base) != ROSE_OK) fail("base", t);
        if (rose_plan_src_numel(p, t, &src) != ROSE_OK) fail("src numel", t);
        std::vector<int64_t> seen(tp, 0);
        const int64_t n = src;                      // the map takes an index inside the sender's slice
        int64_t sent = 0;
        for (int64_t g = 0; g < n; ++g) {
            int32_t d0 = 0, nd = 0, loc = 0;
            if (rose_plan_map_index(p, t, g, &d0, &nd, &loc) != ROSE_OK) fail("map", (int)g);
            if (nd == 0) continue;                  // not sent by this sender
            ++sent;
            for (int32_t d = d0; d < d0 + nd; ++d) {
                int64_t ln = 0;
                if (rose_plan_local_numel(p, t, d, &ln) != ROSE_OK) fail("local numel", d);
                if (loc < 0 || loc >= ln) fail("local index out of range", (int)g);
                ++seen[d];
            }
        }
        const bool sends = ts[t].rule != ROSE_REPLICATED || t % tp_src == src_rank;
        if (sent != (sends ? n : 0)) fail("a sender sends its whole slice, or nothing of a replicated tensor", t);
    }
    copy_tiles(p, tp);
    both_tiles(p, tp);
    delete p;                                        // the plan owns no device memory before its first device call
}

int main() {
    std::vector<rose_tensor_desc> ts = {
        desc(3, 41, ROSE_REPLICATED), desc(0, 16, ROSE_SPLIT_ROWS), desc(16, 37, ROSE_SPLIT_ROWS),
        desc(5, 64, ROSE_SPLIT_COLS), desc(64, 9, ROSE_FUSED_ROWS, {32, 16, 16}), desc(2, 20000, ROSE_SPLIT_COLS),
        desc(1, 3 * 8192 + 5, ROSE_REPLICATED), desc(8, 2 * 8192 - 3, ROSE_SPLIT_ROWS), desc(1, 2 * 8192, ROSE_REPLICATED),
    };
    for (int32_t tp : {1, 2, 4, 8})
        for (int32_t tp_src : {1, 2, 4, 8})
            for (int32_t s = 0; s < tp_src; ++s) walk(ts, tp, tp_src, s);
    std::vector<rose_tensor_desc> g = {desc(128, 12, ROSE_FUSED_ROWS, {64, 32, 32}, 8)};
    for (int32_t tp : {1, 2, 4, 8})
        for (int32_t tp_src : {1, 2, 4, 8})
            for (int32_t s = 0; s < tp_src; ++s) walk(g, tp, tp_src, s);
    std::vector<rose_tensor_desc> many = {desc(8, 7, ROSE_REPLICATED), desc(8, (int64_t)8192 * 8192, ROSE_SPLIT_ROWS), desc(8, 8192 * 2, ROSE_SPLIT_ROWS)};
    rose_plan *large = nullptr;
    if (rose_shard_plan_create(many.data(), 3, 4, &large) != ROSE_OK) fail("create", 0);
    copy_tiles(large, 4);
    both_tiles(large, 4);
    if (!large->copy_piece.empty()) fail("a plan of many tiles shares them", 0);
    delete large;
    // descriptors the planner must turn down without touching anything
    rose_plan *p = nullptr;
    std::vector<rose_tensor_desc> bad = {desc(6, 4, ROSE_SPLIT_ROWS)};
    if (rose_shard_plan_create(bad.data(), 1, 4, &p) != ROSE_ERR_SHAPE || p) fail("non-divisible rows", 0);
    bad = {desc(1, (int64_t)1 << 31, ROSE_REPLICATED)};
    if (rose_shard_plan_create(bad.data(), 1, 1, &p) != ROSE_ERR_UNSUPPORTED || p) fail("too large", 0);
    bad = {desc(12, 4, ROSE_FUSED_ROWS, {8, 8})};
    if (rose_shard_plan_create(bad.data(), 1, 2, &p) != ROSE_ERR_SHAPE || p) fail("sections", 0);
    if (rose_shard_plan_create(nullptr, 1, 2, &p) != ROSE_ERR_ARG) fail("null", 0);
    if (rose_shard_plan_create(ts.data(), (int32_t)ts.size(), 32, &p) != ROSE_ERR_UNSUPPORTED) fail("tp", 0);
    std::printf("ok\n");
    return 0;
}
