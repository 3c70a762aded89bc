// The walk of the encode kernel's workers, their tickets, their rings and the waves that serve prefixes, as a simulation of
// discrete events over the kernel's own rules (rose_internal.h): chains of any length, few workers and many, late starts,
// every tile order.  Every tile is counted once, no count is stored over a prefix, all waits end, and every tile leaves once
// with its prefix.
#include <cstdio>
#include <cstdlib>
#include <deque>
#include <memory>
#include <queue>
#include <random>

#include "rose_internal.h"

using namespace rose;

constexpr int kRing = 8192, kQueue = 64;
enum : int { kEmpty = 0, kCount = 1, kPrefix = 2 };

// The rules under test, or a mistake that the simulation has to find: announced tiles leave although the rest of the ticket
// is to be counted ahead, and only the room that is left then decides whether the ticket on its way is taken in first.
struct Rules {
    bool right;
};

struct Outcome {
    int twice = 0, lost = 0;    // tiles counted again; prefixes that a count was stored over
    int ahead = 0, pairs = 0;   // how often tiles were counted ahead, and for a second ticket of the same group
    bool ended = true, right = true;
};

struct Sim {
    EncodeArgs a;
    bool turns;
    std::mt19937 rng;
    Rules rules;
    Outcome out;
    std::vector<int> count, state, block_state;
    std::vector<int64_t> prefix, block_sum, want, left_at;
    uint32_t counter = 0;

    int pick(int n) { return (int)(rng() % (unsigned)n); }
    double unit() { return (double)rng() / 4294967296.0; }
    int32_t tile_of(int32_t ticket, int32_t j) const { return turns ? tile_of_ticket<1>(a, ticket, j) : tile_of_ticket<0>(a, ticket, j); }
    void publish(int32_t t) {
        if (state[t] != kEmpty) ++out.twice;
        if (state[t] == kPrefix) ++out.lost;
        state[t] = kCount;
    }
};

struct Worker {
    Sim &s;
    Walk w;
    std::deque<int32_t> parked;
    std::deque<bool> known, polled;
    int ring = 0, n_polled = 0;
    bool ticket_out = false, cur_redo = false, skip = false, dense = false, redo_cur = false, late = false;
    uint32_t asked = 0;
    int32_t tile = -1, next = -1, j_from = 0;
    int next_state = 0;
    bool nxt_redo = false;
    std::deque<int32_t> to_count;
    enum { kStart, kIterate, kRoom, kPark, kSettle, kCounting, kDrain, kDone } at = kStart;

    explicit Worker(Sim &sim) : s(sim) {
        w = Walk{-1, s.a.batch, 0, 0, false, false, false, false};
    }
    int step_walk(int32_t *t) {
        return walk_step(s.a.batch, w, t, [&](int32_t ticket, int32_t j) { return s.tile_of(ticket, j); });
    }
    void accept(uint32_t n) {
        if (!walk_accept(s.a.n_tickets, w, n)) s.out.right = false;
    }
    void settle() {
        if (!ticket_out) asked = s.counter++;
        ticket_out = false;
        accept(asked);
    }
    bool full() const { return (int)parked.size() == kQueue || ring + s.count[tile] > kRing; }
    void leave(int n) {
        for (; n > 0; --n) {
            const int32_t t = parked.front();
            if (s.prefix[t] != s.want[t] || s.left_at[t] >= 0) s.out.right = false;
            s.left_at[t] = s.prefix[t];
            ring -= s.count[t];
            parked.pop_front();
            known.pop_front();
        }
    }
    int ready() const {
        int n = 0;
        while (n < (int)known.size() && known[n]) ++n;
        return n;
    }
    void look() {
        n_polled = 0;
        for (size_t i = 0; i < parked.size(); ++i) known[i] = known[i] || s.state[parked[i]] == kPrefix;
    }

    // one action; false: it waits
    bool act() {
        switch (at) {
        case kStart:
            for (;;) {
                const int st = step_walk(&tile);
                if (st == kWalkTile) break;
                if (st == kWalkDone) {
                    at = kDone;
                    return true;
                }
                settle();
            }
            w.careful = false;
            at = kIterate;
            return true;
        case kIterate: {
            const bool accept_now = ticket_out;
            ticket_out = false;
            for (int i = 0; i < n_polled && i < (int)known.size(); ++i) known[i] = known[i] || polled[i];
            int n_announced = ready();
            bool poll = true;
            if (s.a.window_open) {                     // windows of time: open now and then
                const bool open = s.pick(4) == 0;
                if (!open && (int)parked.size() <= kQueue * 3 / 4) n_announced = 0;
                poll = open || s.pick(4) == 0 || (int)parked.size() > kQueue / 2;
            }
            polled.clear();
            n_polled = 0;
            if (poll) {
                for (int32_t t : parked) polled.push_back(s.state[t] == kPrefix);
                n_polled = (int)parked.size();
            }
            const uint32_t answer = asked;
            if (!w.have_next && !accept_now && !w.exhausted && !w.redo) {
                asked = s.counter++;
                ticket_out = true;
            }
            const int32_t ticket_before = w.ticket;
            next_state = step_walk(&next);
            nxt_redo = w.redo;
            if (accept_now) accept(answer);
            if (!cur_redo) s.publish(tile);
            const bool no_place = ring + s.count[tile] > kRing;
            const bool ahead = !s.a.adjacent && no_place && (int)parked.size() < s.a.batch;
            if (ahead && s.rules.right) n_announced = 0;
            leave(n_announced);
            n_polled = n_polled > n_announced ? n_polled - n_announced : 0;
            for (int i = 0; i < n_announced && !polled.empty(); ++i) polled.pop_front();
            if (ticket_first(w, ticket_out, full(), ahead && s.rules.right)) settle();
            const bool mid_ticket = !w.careful && !cur_redo && !w.redo && next_state == kWalkTile && w.ticket == ticket_before;
            dense = false;
            if (s.a.adjacent) {
                if (mid_ticket && full()) {
                    look();
                    leave(ready());
                    dense = full();
                }
            } else if (ahead) {
                dense = mid_ticket;
            }
            skip = w.careful || dense;
            at = skip || !full() ? kPark : kRoom;
            if (at == kRoom && ticket_out) s.out.right = false;       // nothing waits while a ticket is on its way
            return true;
        }
        case kRoom:
            look();
            if (!ready()) return false;
            leave(ready());
            if (!full()) at = kPark;
            return true;
        case kPark:
            if (!skip) {
                parked.push_back(tile);
                known.push_back(false);
                ring += s.count[tile];
            }
            late = false;
            redo_cur = skip;
            at = kSettle;
            return true;
        case kSettle:
            if (w.careful || dense) {
                const bool pair = w.careful;
                const int32_t tA = w.ticket, tB = w.next_ticket, j_end = pair ? 2 * s.a.batch : s.a.batch;
                j_from = s.a.batch;
                if (redo_cur)
                    for (int32_t j = 0; j < s.a.batch; ++j)
                        if (s.tile_of(tA, j) == tile) j_from = j;
                redo_cur = false;
                for (int32_t j = j_from < s.a.batch ? j_from + 1 : s.a.batch; j < j_end; ++j) {
                    const int32_t t = j < s.a.batch ? s.tile_of(tA, j) : s.tile_of(tB, j - s.a.batch);
                    if (t >= 0) to_count.push_back(t);
                }
                ++(pair ? s.out.pairs : s.out.ahead);
                at = kCounting;
                return true;
            }
            if (next_state == kWalkNeedTicket) {
                if (!w.have_next && !w.exhausted) {
                    settle();
                    if (w.careful) return true;
                }
                next_state = step_walk(&next);
                late = true;
                return true;
            }
            if (late) nxt_redo = w.redo;
            if (next_state == kWalkDone) {
                at = kDrain;
                return true;
            }
            cur_redo = nxt_redo;
            tile = next;
            at = kIterate;
            return true;
        case kCounting:
            if (!to_count.empty()) {
                s.publish(to_count.front());
                to_count.pop_front();
                return true;
            }
            w.redo_through = w.careful ? w.next_ticket : w.ticket;
            w.careful = dense = false;
            w.redo = true;
            w.j = j_from - 1;
            next_state = step_walk(&next);
            late = true;
            at = kSettle;
            return true;
        case kDrain:
            look();
            if (ready() < (int)parked.size()) return false;
            leave(ready());
            at = kDone;
            return true;
        case kDone: return true;
        }
        return true;
    }
};

struct Server {
    Sim &s;
    int32_t at;
    bool counted = false;
    Server(Sim &sim, int32_t first) : s(sim), at(first) {}
    bool act() {
        const WalkedBlock b = s.turns ? nth_block<1>(s.a, at, 0) : nth_block<0>(s.a, at, 0);
        const int32_t blk_first = s.a.block_first[b.shard], first = s.a.chain_first[b.shard] + (b.blk - blk_first) * kBlock;
        const int32_t end = first + kBlock < s.a.chain_first[b.shard + 1] ? first + kBlock : s.a.chain_first[b.shard + 1];
        if (!counted) {
            int64_t sum = 0;
            for (int32_t t = first; t < end; ++t) {
                if (s.state[t] == kEmpty) return false;
                sum += s.count[t];
            }
            s.block_sum[b.blk] = sum;
            s.block_state[b.blk] = kCount;
            return counted = true;
        }
        int64_t excl = 0;
        for (int32_t k = b.blk - 1; k >= blk_first; --k) {
            if (s.block_state[k] == kEmpty) return false;
            excl += s.block_sum[k];
            if (s.block_state[k] == kPrefix) break;
        }
        s.block_state[b.blk] = kPrefix;
        s.block_sum[b.blk] += excl;
        for (int32_t t = first; t < end; ++t) {
            s.state[t] = kPrefix;
            s.prefix[t] = excl;
            excl += s.count[t];
        }
        at += s.a.n_servers;
        counted = false;
        return true;
    }
    bool done() const { return at >= s.a.n_blocks; }
};

struct Shape {
    std::vector<int> chains;    // tiles of each
    int workers, servers, batch;
    bool adjacent, windows, turns;
    double density, uneven, late;      // late: iterations over which the workers start
};

static Outcome simulate(const Shape &h, Rules rules, unsigned seed) {
    Sim s;
    s.a = EncodeArgs{};
    s.rng.seed(seed);
    s.rules = rules;
    s.turns = h.turns;
    const int n = (int)h.chains.size();
    for (int d = 0; d < ROSE_MAX_TP; ++d) {
        const int tiles = d < n ? h.chains[d] : 0;
        s.a.chain_first[d + 1] = s.a.chain_first[d] + tiles;
        s.a.block_first[d + 1] = s.a.block_first[d] + (tiles + kBlock - 1) / kBlock;
    }
    s.a.tp = n;
    s.a.n_tiles = s.a.chain_first[n];
    s.a.n_blocks = s.a.block_first[n];
    s.a.batch = h.batch;
    s.a.adjacent = h.adjacent;
    s.a.window_open = h.windows;
    s.a.n_servers = h.servers;
    s.a.n_tickets = (s.a.n_blocks + h.batch - 1) / h.batch * kBlock;
    if (h.turns) s.a.turns = turns_of(s.a.block_first, n);
    s.state.assign(s.a.n_tiles, kEmpty);
    s.block_state.assign(s.a.n_blocks, kEmpty);
    s.block_sum.assign(s.a.n_blocks, 0);
    s.prefix.assign(s.a.n_tiles, -1);
    s.left_at.assign(s.a.n_tiles, -1);
    for (int d = 0; d < n; ++d) {
        int64_t sum = 0;
        for (int t = 0; t < h.chains[d]; ++t) {
            const double x = h.density * (1 + h.uneven * (2 * s.unit() - 1)) * kTile;
            s.count.push_back(x > kTile ? kTile : x < 0 ? 0 : (int)x);
            s.want.push_back(sum);
            sum += s.count.back();
        }
    }
    std::vector<std::unique_ptr<Worker>> workers;
    std::vector<std::unique_ptr<Server>> servers;
    typedef std::pair<double, int> Event;
    std::priority_queue<Event, std::vector<Event>, std::greater<Event>> events;
    std::vector<double> pace;
    const int cap = h.workers < s.a.n_tiles ? h.workers : s.a.n_tiles;
    for (int i = 0; i < cap; ++i) {
        workers.emplace_back(new Worker(s));
        pace.push_back(0.7 + 0.6 * s.unit());
        events.push({h.late * s.unit(), i});
    }
    for (int i = 0; i < h.servers && i < s.a.n_blocks; ++i) {
        servers.emplace_back(new Server(s, i));
        events.push({0, cap + i});
    }
    double last = 0;
    while (!events.empty()) {
        const Event e = events.top();
        events.pop();
        bool moved, done;
        double after;
        if (e.second < cap) {
            Worker &w = *workers[e.second];
            const bool heavy = w.at == Worker::kIterate || w.at == Worker::kCounting;
            moved = w.act();
            done = w.at == Worker::kDone;
            after = !moved ? 0.3 : heavy ? pace[e.second] * (0.8 + 0.4 * s.unit()) : 0.05 * s.unit();
        } else {
            Server &v = *servers[e.second - cap];
            moved = v.act();
            done = v.done();
            after = 0.1 + 0.2 * s.unit();
        }
        if (moved) last = e.first;
        if (e.first > last + 100 + h.late) {           // all wait: the launch would give up
            s.out.ended = false;
            break;
        }
        if (!done) events.push({e.first + after, e.second});
    }
    if (s.out.ended)
        for (int t = 0; t < s.a.n_tiles; ++t) s.out.right = s.out.right && s.left_at[t] == s.want[t];
    return s.out;
}

static Shape draw(std::mt19937 &rng, int kind) {
    auto pick = [&](int n) { return (int)(rng() % (unsigned)n); };
    auto unit = [&]() { return (double)rng() / 4294967296.0; };
    Shape h;
    switch (pick(5)) {
    case 0: h.chains.assign(3, 158); break;
    case 1: h.chains.assign(12, 20); break;
    case 2:
        h.chains.assign(4, 1 + pick(8));
        h.chains[pick(4)] = 400 + pick(400);
        break;
    case 3: h.chains.assign(1 + pick(8), 64 * (1 + pick(6))); break;
    default:
        for (int i = 1 + pick(6); i > 0; --i) h.chains.push_back(1 + pick(300));
    }
    h.workers = pick(3) ? 65 + pick(26) : 65 + pick(400);
    h.servers = pick(2) ? 64 : 1 + pick(8);
    h.adjacent = kind != 0;
    h.batch = kind == 2 ? kBatchTimed : kBatch;
    h.windows = kind != 0;
    h.turns = pick(2) != 0;
    h.density = pick(4) ? 0.3 + 0.7 * unit() : 0.02 + 0.3 * unit();
    h.uneven = pick(2) ? 0.05 : unit();
    h.late = pick(2) ? 0 : 20 * unit();
    return h;
}

int main() {
    const Rules rule = {true}, wrong = {false};
    std::mt19937 rng(7);
    Outcome all, found;
    for (int kind = 0; kind < 3; ++kind)               // spread; neighbours by three and by four
        for (int round = 0; round < 500; ++round) {
            const Shape h = draw(rng, kind);
            const Outcome o = simulate(h, rule, (unsigned)round);
            if (o.twice || o.lost || !o.ended || !o.right) {
                std::printf("failed: kind %d round %d, %d workers, %d chains, %.2f, turns %d: %d counted twice, %d lost, ended %d, right %d\n", kind,
                            round, h.workers, (int)h.chains.size(), h.density, h.turns, o.twice, o.lost, o.ended, o.right);
                return 1;
            }
            all.ahead += o.ahead;
            all.pairs += o.pairs;
            if (kind == 0) {                           // the ticket not taken in first: the simulation has to find that
                const Outcome x = simulate(h, wrong, (unsigned)round);
                found.twice += x.twice;
                found.lost += x.lost;
                found.ended = found.ended && x.ended;
            }
        }
    std::printf("counted ahead %d times, %d pairs; the wrong rule: %d counted twice, %d prefixes lost, gave up %d\n", all.ahead, all.pairs,
                found.twice, found.lost, !found.ended);
    if (!all.ahead || !all.pairs || !found.lost || found.ended) {
        std::printf("failed: the simulation does not reach what it is for\n");
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
