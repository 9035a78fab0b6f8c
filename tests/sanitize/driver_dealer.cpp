// Who gets which item of a backward in one pass, and that nobody waits for good: chain_take, as the kernel runs it, over lists as plans hold them
// (csrc/flexsp_host.hip is part of this program), by workgroups that take turns in a random order between any two accesses.  Few or many of them
// resident, dies with one, with many and with none; a workgroup that ends makes room for the next, on any die.
#include <condition_variable>
#include <cstdio>
#include <map>
#include <memory>
#include <mutex>
#include <random>
#include <thread>
#include <tuple>

#include "flexsp_host.hip"

namespace flexsp {
hipError_t launch_pack(const void *, void *, int64_t, int, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_pack_many(int, const void *const *, void *const *, int64_t, const int32_t *, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge(const uint16_t *, const float *, const uint16_t *, const float *, uint16_t *, float *, int64_t, int, int, int32_t, int32_t, int32_t,
                            int32_t, int32_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge_acc(float *, float *, const uint16_t *, const float *, uint16_t *, int64_t, int, int, int32_t, int32_t, int32_t, int32_t, int32_t,
                                int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t static_scratch_init(int) { return hipErrorUnknown; }
}  // namespace flexsp

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAILED: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

struct Stuck {};  // thrown in every thread once nothing has happened for long

struct Chip {
    const flexsp_plan *p;
    std::mt19937 rng;
    std::vector<int> before;  // the item that an item waits for, or -1
    std::vector<int> drawn;   // how often
    std::vector<char> done;
    unsigned long long word[kChainDies] = {};
    unsigned taken = 0;  // bundles
    int left = 0;        // workgroups that have not started
    long idle = 0;       // turns since something happened
    bool stuck = false;

    // one thread runs at a time; it hands over where another workgroup could come in
    std::mutex m;
    std::vector<std::unique_ptr<std::condition_variable>> cv;
    std::vector<int> alive;
    int turn = -1;
    void pass_on()
    {
        if (alive.empty()) return;
        turn = alive[rng() % alive.size()];
        cv[turn]->notify_one();
    }
    void yield(std::unique_lock<std::mutex> &l, int me)
    {
        if (++idle > 400000) stuck = true;
        pass_on();
        cv[me]->wait(l, [&] { return turn == me; });
        if (stuck) throw Stuck{};
    }

    struct Die {
        Chip &c;
        std::unique_lock<std::mutex> &l;
        int me, die;
        void others() { c.yield(l, me); }
        unsigned long long draw()
        {
            others();
            c.idle = c.word[die] & kChainDone ? c.idle : 0;
            return c.word[die]++;
        }
        unsigned long long look()
        {
            others();
            return c.word[die];
        }
        void put(unsigned long long w)
        {
            others();
            c.idle = 0;
            c.word[die] = w;
        }
        uint32_t bundle()
        {
            others();
            return c.taken++;
        }
        uint32_t low(unsigned long long w) { return (uint32_t)w; }
        uint32_t high(unsigned long long w) { return (uint32_t)(w >> 32); }
        void rest() { others(); }
    };
    void workgroup(std::unique_lock<std::mutex> &l, int me, int die)
    {
        Die d{*this, l, me, die};
        const int32_t *offsets = p->chain_bundles.data();
        const int bundles = (int)p->chain_bundles.size() - 1;
        for (int item = chain_take(d, d.draw(), offsets, bundles); item >= 0;) {
            drawn[item]++;
            idle = 0;
            while (before[item] >= 0 && !done[before[item]]) d.others();
            const unsigned long long pending = d.draw();  // (in front of the item's last output)
            d.others();
            done[item] = 1;
            idle = 0;
            item = chain_take(d, pending, offsets, bundles);
        }
    }
    // `dies`: where a workgroup may be; `resident` of them at a time, `grid` in all
    void run(int dies, int resident, int grid)
    {
        left = grid;
        std::vector<std::thread> threads;
        std::unique_lock<std::mutex> start(m);
        for (int t = 0; t < resident; t++) {
            cv.emplace_back(new std::condition_variable);
            alive.push_back(t);
        }
        for (int t = 0; t < resident; t++)
            threads.emplace_back([this, t, dies] {
                std::unique_lock<std::mutex> l(m);
                cv[t]->wait(l, [&] { return turn == t; });
                try {
                    while (left > 0 && !stuck) {
                        left--;
                        workgroup(l, t, rng() % 3 ? (int)(rng() % dies) : t % dies);
                    }
                } catch (const Stuck &) {
                }
                for (size_t i = 0; i < alive.size(); i++)
                    if (alive[i] == t) alive.erase(alive.begin() + i--);
                pass_on();
            });
        pass_on();
        start.unlock();
        for (auto &t : threads) t.join();
    }
};

int main()
{
    flexsp_ctx *ctx = nullptr;
    CHECK(flexsp_ctx_create(&ctx, -1) == FLEXSP_OK);
    std::vector<std::vector<int>> batches = {std::vector<int>(64, 1024), {8192}, {}, {4097, 1, 64, 65, 127, 0, 128, 129, 191, 255, 256, 257, 640, 4224, 2048}};
    for (int i = 0; i < 12; i++)
        for (int s : {130, 257, 383, 511, 300, 256}) batches[2].push_back(s);
    batches[3].insert(batches[3].end(), 12, 896);
    std::mt19937 rng(3);
    int runs = 0;
    for (size_t n = 0; n < batches.size(); n++) {
        std::vector<int32_t> cu(1, 0);
        for (int s : batches[n]) cu.push_back(cu.back() + s);
        const int heads = n == 0 ? 1 : 8;
        flexsp_plan *p = nullptr;
        CHECK(flexsp_plan_create(ctx, cu.data(), (int)batches[n].size(), heads, heads, 128, 1, &p) == FLEXSP_OK);
        CHECK(!p->chain.empty());
        std::map<std::tuple<int, int, int>, int> at;
        for (size_t i = 0; i < p->chain.size(); i++) at[{p->chain[i].seq_start, p->chain[i].head, p->chain[i].tile}] = (int)i;
        const struct {
            int dies, resident, grid;
        } chips[] = {{8, 1, 1}, {8, 2, 2}, {1, 12, 12}, {2, 3, 30}, {8, 8, 8}, {8, 24, 24}, {16, 40, 40}, {8, 40, 256}, {3, 33, 64}};
        for (const auto &chip : chips) {
            Chip c;
            c.p = p;
            c.rng.seed(rng());
            c.drawn.assign(p->chain.size(), 0);
            c.done.assign(p->chain.size(), 0);
            for (const flexsp_item &it : p->chain) c.before.push_back(it.tile ? at.at({it.seq_start, it.head, it.tile - 1}) : -1);
            c.run(chip.dies, chip.resident, chip.grid);
            if (c.stuck) std::fprintf(stderr, "batch %zu, %d dies, %d of %d workgroups: nothing happens any more\n", n, chip.dies, chip.resident, chip.grid);
            CHECK(!c.stuck && c.left == 0);
            for (size_t i = 0; i < p->chain.size(); i++) CHECK(c.drawn[i] == 1 && c.done[i]);
            runs++;
        }
        flexsp_plan_destroy(p);
    }
    flexsp_ctx_destroy(ctx);
    std::printf("dealer: ok (%d runs)\n", runs);
    return 0;
}
