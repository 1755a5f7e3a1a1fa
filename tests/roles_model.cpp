// Two launches that hold gate/up and down workgroups, on a model device: XCDs with a few places for workgroups each, every XCD
// taking the two launches' workgroups in an order of its own.  Runs the waiting protocol that the kernels run (dfk_roles.h) and
// prints, per launch, how many down workgroups gave up, how many parked, and whether work was done once each and the words are
// zero again.
//   roles_model <may park: 0 or 1> <order: 0 same, 1 opposite, 2 down workgroups first> <seed> <poll limit>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <deque>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#include "dfk_roles.h"

struct HostMem {
    static unsigned load(const unsigned* p) { return __atomic_load_n(p, __ATOMIC_RELAXED); }
    static void store(unsigned* p, unsigned v) { __atomic_store_n(p, v, __ATOMIC_RELAXED); }
    static unsigned fetch_add(unsigned* p, unsigned v) { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
    static void settle() { std::atomic_thread_fence(std::memory_order_seq_cst); }
    static void pause() { std::this_thread::yield(); }
};

constexpr int kXcds = 2, kPlaces = 3, kSlices = 24, kSplits = 6, kBlocks = 4, kDown = kSplits * kBlocks;

struct Launch {
    std::vector<unsigned> words = std::vector<unsigned>(1024, 0u), list = std::vector<unsigned>(kDown, ~0u);
    dfk::RoleShape shape{kDown, kSplits, 8};
    std::atomic<int> published[kSlices] = {}, done[kDown] = {};
    std::atomic<int> gave_up{0}, parked{0}, early{0};
    bool may_park;
    int limit;

    void gateup(int s) {
        ++published[s];
        HostMem::settle();
        HostMem::fetch_add(&words[dfk::kRoleCount0 + s / (kSlices / kSplits) * shape.stride], 1u);
    }
    // as down_km_body: what the last one to pass has to go through is the caller's business
    bool down(int wg, bool stand_in) {
        const int js = wg / kBlocks, per = kSlices / kSplits;
        unsigned* const notes = may_park && !stand_in ? list.data() : nullptr;
        const int got = dfk::role_wait<HostMem>(words.data(), shape, js, per, limit, notes, wg);
        if (got == dfk::kRoleParked) { ++parked; return false; }
        if (got == dfk::kRoleGaveUp) ++gave_up;
        const unsigned before = stand_in ? 0u : dfk::role_pass<HostMem>(words.data());
        for (int s = js * per; s < (js + 1) * per; ++s) early += got == dfk::kRoleReady && !published[s];
        ++done[wg];
        if (stand_in || dfk::role_left(shape, before) != 1u) return false;
        if (before >> 16) return true;
        dfk::role_clear<HostMem>(words.data(), shape);
        return false;
    }
    void run(int wg) {
        if (wg < kSlices) return gateup(wg);
        const int own = wg - kSlices;
        if (!down(own, false)) return;
        const unsigned n = HostMem::load(&words[dfk::kRoleNotes]);
        for (unsigned i = 0; i < n; ++i)
            if ((int)HostMem::load(&list[i]) != own) down((int)HostMem::load(&list[i]), true);
        dfk::role_clear<HostMem>(words.data(), shape);
    }
};

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    const bool may_park = std::atoi(argv[1]);
    const int order = std::atoi(argv[2]), limit = std::atoi(argv[4]);
    std::mt19937 rng((unsigned)std::atoi(argv[3]));
    Launch launches[2];
    for (auto& l : launches) { l.may_park = may_park; l.limit = limit; }
    struct Item { Launch* l; int wg; };
    std::deque<Item> queue[kXcds];
    std::mutex mu[kXcds];
    for (int x = 0; x < kXcds; ++x)
        for (int k = 0; k < 2; ++k) {
            Launch* l = &launches[order == 1 ? k ^ x : k];
            for (int i = x; i < kSlices + kDown; i += kXcds)
                queue[x].push_back({l, order == 2 ? (i + kSlices) % (kSlices + kDown) : i});
        }
    std::vector<std::thread> places;
    for (int x = 0; x < kXcds; ++x)
        for (int p = 0; p < kPlaces; ++p)
            places.emplace_back([&, x, nap = (int)(rng() % 200)]() {
                std::this_thread::sleep_for(std::chrono::microseconds(nap));
                for (;;) {
                    Item it;
                    {
                        std::lock_guard<std::mutex> lk(mu[x]);
                        if (queue[x].empty()) return;
                        it = queue[x].front();
                        queue[x].pop_front();
                    }
                    it.l->run(it.wg);
                }
            });
    for (auto& t : places) t.join();
    for (auto& l : launches) {
        int once = 1, zero = 1;
        for (auto& d : l.done) once &= d == 1;
        for (auto& s : l.published) once &= s == 1;
        for (unsigned w : l.words) zero &= w == 0u;
        std::printf("%d %d %d %d %d\n", l.gave_up.load(), l.parked.load(), once, zero, l.early.load());
    }
    return 0;
}
