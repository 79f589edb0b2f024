// Exercises gpr::Room: fixed sequences, then threads that take and give room at random.  Prints "ok".
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "gpr_room.h"

#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

static gpr::Room::Key key(long k) { return {(const void *)k, std::thread::id()}; }

int main()
{
    {
        gpr::Room r;
        CHECK(!r.others(key(1)));
        CHECK(r.try_take(key(1), 192, 256) && !r.others(key(1)) && r.others(key(2)));
        CHECK(!r.try_take(key(2), 192, 256));              // more than is left
        CHECK(r.try_take(key(2), 64, 256));                // exactly what is left
        CHECK(!r.try_take(key(3), 8, 256));
        CHECK(r.try_take(key(1), 100, 256));               // the same stream again: its launches follow each other
        r.give(key(1));
        CHECK(!r.try_take(key(3), 8, 256));                // its first launch still has the room
        r.give(key(1));
        CHECK(r.try_take(key(3), 192, 256));
        r.give(key(2));
        r.give(key(3));
        CHECK(r.try_take(key(4), 512, 256));               // more than the device: all of it
        CHECK(!r.try_take(key(5), 8, 256));
        std::atomic<int> order{0};
        int first = 0, second = 0;
        std::thread a([&] { r.take(key(6), 256, 256); first = ++order; r.give(key(6)); });
        while (!r.others(key(4))) std::this_thread::yield();   // (it waits, so later ones queue behind it)
        CHECK(!r.try_take(key(4), 8, 256));                // nobody overtakes who waits
        std::thread b([&] { r.take(key(7), 8, 256); second = ++order; r.give(key(7)); });
        r.give(key(4));
        a.join();
        b.join();
        CHECK(first >= 1 && second >= 1 && order == 2 && !r.others(key(4)));
    }
    {
        gpr::Room r;
        std::vector<std::atomic<int>> held(8);
        for (auto &h : held) h = 0;
        std::vector<std::thread> th;
        std::atomic<int> worst{0};
        for (int t = 0; t < 8; ++t)
            th.emplace_back([&, t] {
                std::mt19937 g(t);
                for (int k = 0; k < 6000; ++k) {
                    const int u = 8 * (1 + (int)(g() % 32));
                    bool in = true;
                    if (g() % 2) r.take(key(t + 1), u, 256);
                    else in = r.try_take(key(t + 1), u, 256);
                    if (!in) continue;
                    held[t] = u;
                    int sum = 0;
                    for (auto &h : held) sum += h;
                    // (a thread's figure is set after its room is taken and cleared before it is given: the sum is never above)
                    int w = worst;
                    while (sum > w && !worst.compare_exchange_weak(w, sum)) {}
                    held[t] = 0;
                    r.give(key(t + 1));
                }
            });
        for (auto &t : th) t.join();
        CHECK(worst <= 256 && worst >= 128);
        CHECK(!r.others(key(99)) && r.try_take(key(99), 256, 256));
    }
    std::printf("ok\n");
    return 0;
}
