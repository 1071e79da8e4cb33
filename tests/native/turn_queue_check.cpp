// Runs the push queue's protocol (turn_queue.hpp) with threads as waves.  One
// wave reads the count late: only when another has gone on to add the next
// turn's entries, or after a while if none can.  Every wave has to empty at
// the same turns, no turn may overflow the queue and no barrier may be left
// waiting.  "late_read" runs the protocol that decides from a count read
// behind the turn's only barrier instead, which must not pass.
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#include "../../paper_2608_16308_amd/csrc/turn_queue.hpp"

using namespace std::chrono_literals;
constexpr uint32_t CAP = 64, PER_WAVE = 4;
constexpr int WAVES = 4, TURNS = 24;
constexpr uint32_t TURN = PER_WAVE * WAVES;

struct Group {
    std::mutex mu;
    std::condition_variable cv;
    int waiting = 0;
    uint64_t gen = 0;
    std::atomic<bool> stuck{false};
    std::chrono::milliseconds patience{30000};  // at a barrier
    std::atomic<uint32_t> count{0}, most{0}, taken{0};
    std::atomic<int> adding[WAVES] = {};  // the turn each wave has begun to add in
    bool barrier()
    {
        std::unique_lock<std::mutex> l(mu);
        const uint64_t g = gen;
        if (++waiting == WAVES) {
            waiting = 0;
            ++gen;
            cv.notify_all();
            return true;
        }
        if (!cv.wait_for(l, patience, [&] { return gen != g || stuck; })) {
            stuck = true;
            cv.notify_all();
        }
        return !stuck;
    }
};

struct Ops {
    Group &g;
    int wave, slow, turn = 0;
    void barrier() { g.barrier(); }
    uint32_t count()
    {
        if (wave == slow) {  // late, as a wave that the others leave behind
            const auto end = std::chrono::steady_clock::now() + 20ms;
            auto ahead = [&] {
                for (int w = 0; w < WAVES; ++w)
                    if (w != wave && g.adding[w] > turn) return true;
                return false;
            };
            while (!ahead() && std::chrono::steady_clock::now() < end) std::this_thread::yield();
            if (ahead()) std::this_thread::sleep_for(1ms);  // (the add itself)
        }
        return g.count;
    }
};

// found[turn][wave]: entries the wave queues in the turn
static bool run(bool late_read, int slow, const std::vector<std::vector<uint32_t>> &found)
{
    Group g;
    if (late_read) g.patience = 300ms;
    std::vector<std::vector<int>> emptied(WAVES);
    uint32_t total = 0;
    for (const auto &f : found)
        for (uint32_t k : f) total += k;
    auto wave = [&](int w) {
        Ops ops{g, w, slow};
        uint32_t room = CAP, n = 0;
        auto empty = [&](int turn) {
            emptied[(size_t)w].push_back(turn);
            g.barrier();
            if (w == 0) {
                g.taken += n;
                g.count = 0;
            }
            g.barrier();
        };
        for (int turn = 0; turn < TURNS && !g.stuck; ++turn) {
            ops.turn = turn - 1;  // the last turn whose entries this wave has added
            if (!late_read && dbs::queue_is_full<CAP, TURN>(room, n, ops)) empty(turn);
            g.adding[w] = turn;
            const uint32_t c = g.count.fetch_add(found[(size_t)turn][(size_t)w]) + found[(size_t)turn][(size_t)w];
            for (uint32_t m = g.most; c > m && !g.most.compare_exchange_weak(m, c);) {}
            if (late_read) {
                ops.turn = turn;
                g.barrier();
                n = ops.count();
                if (n > CAP - TURN) empty(turn);
            }
        }
        g.barrier();
        if (w == 0) g.taken += g.count;
    };
    std::vector<std::thread> pool;
    for (int w = 0; w < WAVES; ++w) pool.emplace_back(wave, w);
    for (auto &t : pool) t.join();
    bool ok = !g.stuck && g.most <= CAP && g.taken == total;
    for (int w = 1; w < WAVES; ++w) ok = ok && emptied[(size_t)w] == emptied[0];
    return ok;
}

int main(int argc, char **argv)
{
    const bool late = argc > 1 && !std::strcmp(argv[1], "late_read");
    std::mt19937 rng(7);
    int bad = 0, runs = 0;
    for (int pattern = 0; pattern < 4; ++pattern) {
        std::vector<std::vector<uint32_t>> found(TURNS, std::vector<uint32_t>(WAVES));
        for (auto &f : found)
            for (auto &k : f) k = pattern == 0 ? PER_WAVE : pattern == 1 ? 1 : rng() % (PER_WAVE + 1);
        for (int slow = 0; slow < WAVES; ++slow, ++runs) bad += run(late, slow, found) ? 0 : 1;
    }
    std::printf("%d of %d runs wrong\n", bad, runs);
    return bad ? 1 : 0;
}
