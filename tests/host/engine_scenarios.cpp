// The host engine on a stand-in device (fake_device.h): one scenario a run,
// named on the command line.  Exit status 0 and "passed" = pass.
#include "fake_device.h"

#include "../../paper_1205_0106_amd/csrc/amq_engine.hip"

#include <set>

#include <sys/mman.h>

static int g_failed = 0;
#define CHECK(c)                                                                  \
    do {                                                                          \
        if (!(c)) {                                                               \
            fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c);       \
            ++g_failed;                                                           \
        }                                                                         \
    } while (0)

static am_option option(int64_t n_paths, int32_t n_dates)
{
    am_option o;
    memset(&o, 0, sizeof o);
    o.params = am_params{100.0, 100.0, 0.05, 0.2, 1.0, 0, 1};
    o.n_paths = n_paths;
    o.n_dates = n_dates;
    return o;
}

// A wait runs out in a sweep over both storage types before the options of
// one type are claimed: none of the book's options reads as priced, whichever
// type had the wait (the words of a result that was never written hold an
// earlier price).
static void mixed_timeout()
{
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    const am_server_config cfg{(size_t)256 << 20, 1e12, 64, 1, b, AM_FP32_BULK, 1};
    std::mutex gate;
    std::unique_lock<std::mutex> hold(gate);
    std::atomic<int> mixed{0};
    fake::on_sweep_batch = [&](const amq::BatchOpt *, const int32_t *, const amq::BatchGlobal &g, int, int mode) {
        if (mode != amq::kMixed) {
            std::lock_guard<std::mutex> wait(gate);   // the first batch runs until the others are queued
            return;
        }
        mixed++;
        *g.err = 1u;
    };
    am_server *sv = nullptr;
    CHECK(am_server_create(&cfg, &sv) == AM_OK);
    const am_option first = option(20000, 4), f32 = option(40000, 5), f64 = option(3000, 6);
    CHECK(am_server_submit(sv, &first, 0, -1.0) == AM_OK);
    am_result r[8];
    int32_t n = 0;
    double st[4] = {0};
    while (st[0] < 1.0) {   // (the first batch is counted once its launch returns: wait for the slot by its pool bytes)
        CHECK(am_server_stats(sv, st) == AM_OK);
        if (st[3] > 0.0) break;
    }
    CHECK(am_server_submit(sv, &f32, 1, -1.0) == AM_OK);
    CHECK(am_server_submit(sv, &f64, 2, -1.0) == AM_OK);
    CHECK(am_server_submit(sv, &f32, 3, -1.0) == AM_OK);
    hold.unlock();
    int got = 0, late = 0;
    for (int spin = 0; got < 4 && spin < 5000; ++spin) {
        CHECK(am_server_poll(sv, r, 8, &n) == AM_OK);
        for (int i = 0; i < n; ++i) {
            ++got;
            if (r[i].request_id > 0 && r[i].status == AM_ETIMEOUT) ++late;
        }
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
    }
    CHECK(am_server_destroy(sv) == AM_OK);
    CHECK(got == 4 && mixed == 1);
    CHECK(late == 3);
}

// The calls logged since the last time, in order, as "wait:A", "sweep:A",
// "record:A" or "graph:A" on stream A.
static std::vector<std::string> logged(const std::map<const void *, char> &name)
{
    std::vector<std::string> out;
    for (const std::string &l : fake::log) {
        char what[16];
        void *s = nullptr, *o = nullptr;
        if (sscanf(l.c_str(), "%15s %p %p", what, &s, &o) < 2) continue;
        const auto it = name.find(s);
        out.push_back(std::string(what) + ":" + (it == name.end() ? '?' : it->second));
    }
    fake::log.clear();
    return out;
}

// Sweeps that may fill the device run in enqueue order whatever enqueued them:
// single options, books and replays of captured books.
static void order_across_streams()
{
    using V = std::vector<std::string>;
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    const hipStream_t A = (hipStream_t)0xA0, B = (hipStream_t)0xB0;
    const std::map<const void *, char> name = {{A, 'A'}, {B, 'B'}};
    const am_option o = option(20000, 4);
    void *w1 = nullptr, *w2 = nullptr;
    CHECK(fake::alloc(&w1, am_workspace_bytes(o.n_paths, o.n_dates, b, AM_FP64)) == hipSuccess);
    const size_t nb = am_batch_workspace_bytes(&o, 1, b, AM_FP64);
    CHECK(fake::alloc(&w2, nb) == hipSuccess);
    const auto single = [&](hipStream_t s) {
        return am_price_american_ex(&o.params, o.n_paths, o.n_dates, b, AM_FP64, w1,
                                    am_workspace_bytes(o.n_paths, o.n_dates, b, AM_FP64), s, nullptr);
    };
    am_batch_graph *g = nullptr;
    CHECK(am_batch_graph_create(&o, 1, b, AM_FP64, w2, nb, &g) == AM_OK);
    fake::log.clear();
    CHECK(single(A) == AM_OK);
    CHECK(logged(name) == (V{"sweep:A", "record:A"}));
    // (a replay's second record is its own end)
    CHECK(am_batch_graph_launch(g, B) == AM_OK);
    CHECK(logged(name) == (V{"wait:B", "graph:B", "record:B", "record:B"}));
    CHECK(am_batch_graph_launch(g, B) == AM_OK);
    CHECK(logged(name) == (V{"graph:B", "record:B", "record:B"}));
    CHECK(single(A) == AM_OK);
    CHECK(logged(name) == (V{"wait:A", "sweep:A", "record:A"}));
    CHECK(am_price_batch(&o, 1, b, AM_FP64, w2, nb, B, nullptr) == AM_OK);
    CHECK(logged(name) == (V{"wait:B", "sweep:B", "record:B"}));
    CHECK(am_batch_graph_launch(g, A) == AM_OK);
    CHECK(logged(name) == (V{"wait:A", "graph:A", "record:A", "record:A"}));
    // a call into the caller's own capture leaves the order as it was
    fake::capturing = B;
    CHECK(single(B) == AM_OK);
    fake::capturing = nullptr;
    CHECK(logged(name) == (V{"sweep:B"}));
    CHECK(single(A) == AM_OK);
    CHECK(logged(name) == (V{"sweep:A", "record:A"}));
    // what a graph reads is gone after am_shutdown
    CHECK(am_shutdown() == AM_OK);
    CHECK(am_batch_graph_launch(g, A) == AM_EINVAL);
    CHECK(am_batch_graph_destroy(g) == AM_OK);
}

// Whether a batch sweep's grid finishes with only `room` groups resident at a
// time (the rest start as others leave): every group claims its queue's next
// tile and holds it until all of that option's tiles are held.
static bool finishes(const amq::BatchGlobal &g, const int32_t *tile_opt, int grid, int room)
{
    std::vector<int> next(g.q_off, g.q_off + g.queues);
    std::map<int32_t, int> tiles, held;             // per option
    for (int t = 0; t < g.total_tiles; ++t) tiles[tile_opt[t]]++;
    std::vector<std::pair<int, int32_t>> resident;  // (queue, option held)
    int started = 0, done = 0;
    for (;;) {
        bool moved = false;
        while (started < grid && (int)resident.size() < room) {
            const int q = started++ % g.queues;
            moved = true;
            if (next[q] >= g.q_off[q + 1]) continue;
            resident.push_back({q, tile_opt[next[q]++]});
            held[resident.back().second]++;
        }
        for (size_t i = 0; i < resident.size();) {
            auto &[q, o] = resident[i];
            if (held[o] < tiles[o]) { ++i; continue; }
            moved = true;
            ++done;
            if (next[q] < g.q_off[q + 1]) {
                o = tile_opt[next[q]++];
                held[o]++;
                ++i;
            } else {
                resident.erase(resident.begin() + i);
            }
        }
        if (done == g.total_tiles) return true;
        if (!moved) return false;
    }
}

// A book finishes with one group a compute unit, however many a unit may hold
// (other work on the device can leave no more), and options share the device
// through several claim queues only where every group has a unit of its own.
static void claim_queues()
{
    struct Shape { int n, step; int64_t n_paths; int32_t n_dates; };
    const Shape shapes[] = {{1, 0, 20000, 4}, {2, 9, 60000, 9}, {8, 0, 700000, 7}, {6, 37, 1 << 20, 5}, {12, 5000, 9000, 40},
                            {8, 0, 1 << 19, 6}, {5, 0, 900000, 6}, {40, 1000, 30000, 12}, {300, 77, 16000, 10},
                            {3, 0, 4000000, 3}, {64, 0, 65536, 8}, {65, 0, 65536, 8}};
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    int launches = 0, queued = 0;
    fake::on_sweep_batch = [&](const amq::BatchOpt *, const int32_t *tile_opt, const amq::BatchGlobal &g, int grid, int) {
        ++launches;
        CHECK(g.queues == 1 || g.queues == amq::kClaimQueues);
        CHECK(g.q_off[0] == 0 && g.q_off[g.queues] == g.total_tiles);
        if (g.queues > 1) {
            ++queued;
            CHECK(grid <= fake::kCus && grid % g.queues == 0);
            for (int q = 0; q < g.queues; ++q) CHECK(g.q_off[q + 1] - g.q_off[q] <= grid / g.queues);
        }
        CHECK(grid <= fake::kCus * fake::batch_groups_per_cu);
        CHECK(finishes(g, tile_opt, grid, fake::kCus));
    };
    for (const Shape &s : shapes)
        for (int dtype : {AM_FP64, AM_FP32_BULK}) {
            std::vector<am_option> o;
            for (int i = 0; i < s.n; ++i) o.push_back(option(s.n_paths + (int64_t)s.step * i, s.n_dates + i % 5));
            const size_t nb = am_batch_workspace_bytes(o.data(), s.n, b, dtype);
            void *w = nullptr;
            CHECK(nb > 0 && fake::alloc(&w, nb) == hipSuccess);
            CHECK(am_price_batch(o.data(), s.n, b, dtype, w, nb, (hipStream_t)0xA0, nullptr) == AM_OK);
            fake::release(w);
        }
    CHECK(launches > 20 && queued > 8 && queued < launches);
    // served batches share the device: one queue
    const am_server_config cfg{(size_t)256 << 20, 1e12, 64, 2, b, AM_FP64, 1};
    queued = 0;
    am_server *sv = nullptr;
    CHECK(am_server_create(&cfg, &sv) == AM_OK);
    const am_option o = option(20000, 4);
    for (int i = 0; i < 6; ++i) CHECK(am_server_submit(sv, &o, i, -1.0) == AM_OK);
    CHECK(am_server_destroy(sv) == AM_OK);
    CHECK(queued == 0);
}

// Batches served side by side: whatever is in flight, the requests' groups fit
// in what every compute unit has room for in any placement; larger ones run
// alone.
static void served_share()
{
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    const int64_t tile = 256 * 32;
    for (int sure = 1; sure <= 2; ++sure)
        for (int streams : {1, 2, 3, 8}) {
            fake::batch_sure_per_cu = sure;
            const int share = sure * fake::kCus / streams;
            const am_server_config cfg{(size_t)2 << 30, 1e12, 1, streams, b, AM_FP64, 1};
            am_server *sv = nullptr;
            std::mutex mu;
            std::map<int, bool> alone;   // by tiles
            const auto note = [&](int tiles) {
                for (Slot &sl : sv->slots)
                    if (sl.reqs.size() == 1 && !sl.busy && (sl.reqs[0].opt.n_paths + tile - 1) / tile == tiles) {
                        std::lock_guard<std::mutex> lk(mu);
                        alone[tiles] = sl.exclusive;
                    }
            };
            fake::on_sweep_batch = [&](const amq::BatchOpt *o, const int32_t *, const amq::BatchGlobal &, int grid, int) {
                CHECK(grid >= o[0].G);
                note(o[0].G);
            };
            fake::on_sweep = [&](const amq::SweepArgs &a) { note((int)((a.N + tile - 1) / tile)); };
            CHECK(am_server_create(&cfg, &sv) == AM_OK);
            const int sizes[] = {1, share - 1, share, share + 1, 2 * fake::kCus};
            int id = 0;
            for (int t : sizes)
                if (t >= 1 && t <= 2 * fake::kCus) {
                    const am_option o = option(t * tile, 2);
                    CHECK(am_server_submit(sv, &o, id++, -1.0) == AM_OK);
                }
            const am_option too_big = option((2 * fake::kCus + 1) * tile, 2);
            CHECK(am_server_submit(sv, &too_big, 99, -1.0) == AM_EDIM);
            CHECK(am_server_destroy(sv) == AM_OK);   // finishes what is queued
            for (const auto &[t, a] : alone) CHECK(a == (t > share));
            CHECK(alone.size() >= 3);
        }
}

// Every schedule's segment forms: each covers every date, a node's parents are in
// the slots that it reads, and the form that a launch of many blocks takes leaves
// room for four generation groups in a CU's LDS.
static void segments()
{
    for (int M = 1; M <= amq::kMaxDates; ++M) {
        const std::vector<amq::BridgeNode> all = make_schedule(M);
        std::vector<std::pair<int, int>> parent(M + 1, {0, 0});
        std::vector<int> slot_date(amq::kMaxSlots, 0);
        for (const auto &n : all) {
            parent[n.m] = {n.sl == amq::kAnchorSlot ? -1 : slot_date[n.sl], n.sr == amq::kAnchorSlot ? -1 : slot_date[n.sr]};
            slot_date[n.dst] = n.m;
        }
        SegSchedule S;
        CHECK(host_schedule(M, &S) == AM_OK);
        for (int v = 0; v < amq::kSegVariants && S.len[v]; ++v) {
            CHECK(S.len[v] == seg_len(M, v));
            std::set<int> dates;
            for (int s = 0; s < 1 << v; ++s) {
                std::vector<int> slot(amq::kMaxSlots, -2);
                slot[0] = 0;
                slot[amq::kAnchorSlot] = -1;
                for (int q = 0; q < S.len[v]; ++q) {
                    const amq::GenNode &n = S.nodes[S.off[v] + s * S.len[v] + q];
                    const int m = n.md & 0xFFFF, sl = (n.slots & 0xFF) / 2, sr = (n.slots >> 8 & 0xFF) / 2, d = (n.slots >> 16) / 2;
                    // (of a last node's repeats too: the same value again)
                    CHECK(slot[sl] == parent[m].first && (slot[sr] == parent[m].second || n.wr == 0.0));
                    slot[d] = m;
                    dates.insert(m);
                }
            }
            CHECK((int)dates.size() == M);
        }
        const int v = gen_variant(M, (int64_t)1 << 30);
        CHECK(S.len[v] > 0 && 4 * amq::gen_lds_bytes(S.len[v]) <= amq::kLdsCu);
    }
}

// The tile list of a book fits the table it is uploaded to, also where one part's
// holds both parts' lists; a plan whose table is too short is refused before the
// upload.
static void tile_table()
{
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    DevState *st = nullptr;
    CHECK(get_state(&st) == AM_OK);
    for (int n32 : {0, 1, 3, 40})
        for (int n64 : {0, 1, 50, 200}) {
            if (n32 + n64 == 0) continue;
            std::vector<am_option> o;
            for (int i = 0; i < n32; ++i) o.push_back(option(16384 + 40000 * (i % 2), 3));
            for (int i = 0; i < n64; ++i) o.push_back(option(10 + 80 * i, 3));
            SplitBatch B;
            split_batch(o.data(), (int32_t)o.size(), AM_FP32_BULK, B);
            int words = 0;
            fake::on_sweep_batch = [&](const amq::BatchOpt *, const int32_t *, const amq::BatchGlobal &g, int, int) {
                words = g.total_tiles;
            };
            void *w = nullptr;
            CHECK(fake::alloc(&w, B.total) == hipSuccess);
            CHECK(enqueue_split(st, B, b, AM_FP32_BULK, (char *)w, (hipStream_t)0xA0, nullptr, true, nullptr, 0, nullptr) == AM_OK);
            CHECK(B.one_sweep == (n32 > 0 && n64 > 0));
            if (B.one_sweep) {
                const size_t room[2] = {B.P[0].off_part - B.P[0].off_tiles, B.P[1].off_part - B.P[1].off_tiles};
                CHECK((size_t)words * 4 <= (room[0] > room[1] ? room[0] : room[1]));
            }
            for (int h = 0; h < 2; ++h) B.P[h].off_part = B.P[h].off_tiles;
            CHECK(enqueue_split(st, B, b, AM_FP32_BULK, (char *)w, (hipStream_t)0xA0, nullptr, true, nullptr, 0, nullptr) == AM_EDEVICE);
            fake::release(w);
        }
}

// No limit on the polls of a wait makes it endless: a wait that counts four polls
// as one exceeds the limit before its 32-bit count wraps.
static void spin_limit()
{
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    const am_option o = option(20000, 4);
    const size_t nb = am_workspace_bytes(o.n_paths, o.n_dates, b, AM_FP64);
    void *w = nullptr;
    CHECK(fake::alloc(&w, nb) == hipSuccess);
    uint32_t seen = 0;
    fake::on_sweep = [&](const amq::SweepArgs &a) { seen = a.spin_limit; };
    for (uint32_t limit : {1u, 1000u, (1u << 30) - 2, (1u << 30) - 1, 1u << 30, 0xFFFFFFFFu, 0u}) {
        am_debug_set_spin_limit(limit);
        CHECK(am_price_american_ex(&o.params, o.n_paths, o.n_dates, b, AM_FP64, w, nb, (hipStream_t)0xA0, nullptr) == AM_OK);
        CHECK(seen > 0 && seen < 0xFFFFFFFFu / 4);
        if (limit && limit <= (1u << 30) - 2) CHECK(seen == limit);
    }
}

// However many groups of a register-resident tile a compute unit holds, a single
// option takes one a unit at most, and every size has a tile.
static void one_group_a_unit()
{
    DevState *st = nullptr;
    CHECK(get_state(&st) == AM_OK);
    fake::small_groups_per_cu = 2;
    for (int fp64 : {0, 1})
        for (int laguerre : {0, 1})
            for (int degree : {0, 2, 6})
                for (int64_t n = 1000; n < 4000000; n += n / 7) {
                    Plan p{0, 0, 0};
                    CHECK(choose_plan(st, n, fp64, laguerre, degree, &p) == AM_OK);
                    if (p.wg == 512 && p.ppt <= 8) CHECK(p.G <= fake::kCus);
                }
}

// Options of more tiles than compute units leave the book's tile list and are swept
// by themselves, with a group a unit at most and on the book's error word; one
// that the device does not hold is refused.
static void wide_options()
{
    const am_basis b{AM_BASIS_MONOMIAL, 2};
    for (int dtype : {AM_FP64, AM_FP32_BULK}) {
        const int64_t tile = 256 * (dtype == AM_FP64 ? 32 : 64), top = 2 * fake::kCus * tile;
        const am_option sizes[] = {option(256 * tile, 2), option(256 * tile + 1, 2), option(30000, 3), option(top, 2), option(700, 4)};
        for (int mask = 1; mask < 32; ++mask) {
            std::vector<am_option> o;
            std::set<int64_t> expect, seen;
            int listed = 0;
            for (int i = 0; i < 5; ++i) {
                if (!(mask >> i & 1)) continue;
                o.push_back(sizes[i]);
                if (i == 1 || i == 3) expect.insert(sizes[i].n_paths);
                else ++listed;
            }
            uint32_t *err = nullptr;
            int books = 0;
            fake::on_sweep_batch = [&](const amq::BatchOpt *o32, const int32_t *tile_opt, const amq::BatchGlobal &g, int grid, int) {
                ++books;
                err = g.err;
                std::set<int32_t> in(tile_opt, tile_opt + g.total_tiles);
                listed -= (int)in.size();
                for (int32_t t : in) CHECK((t < 0 ? g.opts64[t & 0x7FFFFFFF] : o32[t]).G <= fake::kCus);
                CHECK(finishes(g, tile_opt, grid, fake::kCus));
            };
            fake::on_sweep = [&](const amq::SweepArgs &a) {
                seen.insert(a.N);
                CHECK(a.G <= fake::kCus && a.G > fake::kCus / 2);
                CHECK((int64_t)a.G * 2 * tile >= a.N);   // (a 512-thread tile has two of the batch's)
                CHECK(!books || a.err == err);
            };
            const size_t nb = am_batch_workspace_bytes(o.data(), (int32_t)o.size(), b, dtype);
            void *w = mmap(nullptr, nb, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
            CHECK(w != MAP_FAILED);
            CHECK(am_price_batch(o.data(), (int32_t)o.size(), b, dtype, w, nb, (hipStream_t)0xA0, nullptr) == AM_OK);
            munmap(w, nb);
            CHECK(seen == expect && listed == 0);
        }
        const am_option too_big = option(top + 1, 2);
        const size_t nb = am_batch_workspace_bytes(&too_big, 1, b, dtype);
        CHECK(am_price_batch(&too_big, 1, b, dtype, (void *)256, nb, (hipStream_t)0xA0, nullptr) == AM_EDIM);
    }
}

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> scenarios = {
        {"mixed_timeout", mixed_timeout},
        {"order_across_streams", order_across_streams},
        {"claim_queues", claim_queues},
        {"served_share", served_share},
        {"segments", segments},
        {"tile_table", tile_table},
        {"spin_limit", spin_limit},
        {"one_group_a_unit", one_group_a_unit},
        {"wide_options", wide_options},
    };
    const auto it = scenarios.find(argc > 1 ? argv[1] : "");
    if (it == scenarios.end()) {
        for (const auto &s : scenarios) printf("%s\n", s.first.c_str());
        return 2;
    }
    it->second();
    printf(g_failed ? "%d checks failed\n" : "passed\n", g_failed);
    return g_failed ? 1 : 0;
}
