// Host test of the work queue's claims (rkc_queue.h): one thread per lane of a
// group, in step at every shuffle, and other groups that claim from the same
// heads between any two reads of one.  Whatever they do, all lanes of the group
// must see the same positions, and every position must be claimed exactly once.
// Prints "OK" and exits 0 on success.
#include <condition_variable>
#include <cstdio>
#include <mutex>
#include <thread>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0

static struct { unsigned x; } blockIdx;
static thread_local struct { unsigned x; } threadIdx;

struct Params {
    int *queue;
    int n_cells, groups_total;
};
static Params P;

// Lanes still in the call meet at each shuffle; one that has returned drops out.
struct Meet {
    std::mutex m;
    std::condition_variable cv;
    int active = 0, waiting = 0, value = 0, given[2] = {0, 0};
    unsigned turn = 0;
    int shuffle(int lane, int v) {
        std::unique_lock<std::mutex> l(m);
        if (lane == 0) value = v;
        const unsigned t = turn;
        ++waiting;
        cv.notify_all();
        if (waiting >= active) release();
        else cv.wait(l, [&] { return turn != t; });
        return given[t & 1];
    }
    void drop() {
        std::unique_lock<std::mutex> l(m);
        --active;
        cv.notify_all();
        if (waiting > 0 && waiting >= active) release();
    }
    // lane 0 writes after the reads that the other lanes make in the same step
    void others_arrived() {
        std::unique_lock<std::mutex> l(m);
        cv.wait(l, [&] { return waiting >= active - 1; });
    }
    void release() {
        given[turn & 1] = value;   // the next turn may overwrite value before all have woken
        waiting = 0;
        ++turn;
        cv.notify_all();
    }
};
static Meet meet;

static std::mutex mem;
static int others_every, reads;   // another group claims after every n-th read of a head
static std::vector<int> claimed;  // claims of each position

static void count(int part, int i) {
    const long pos = (long)P.groups_total + part + (long)i * 16;
    if (pos < P.n_cells) ++claimed[(size_t)pos];
}
static int atomicAdd(int *q, int v) {
    meet.others_arrived();
    std::lock_guard<std::mutex> l(mem);
    const int old = *q;
    *q += v;
    count((int)((q - P.queue) / 32), old);
    return old;
}
static int atomic_load(const int *q) {
    std::lock_guard<std::mutex> l(mem);
    const int v = *q;
    if (others_every && ++reads % others_every == 0) {
        count((int)((q - P.queue) / 32), v);
        ++const_cast<int *>(q)[0];
    }
    return v;
}
#define __hip_atomic_load(p, order, scope) atomic_load(p)
#define __shfl(v, lane, width) meet.shuffle((int)threadIdx.x % (width), v)
#define __builtin_amdgcn_readfirstlane(x) (x)

#include "rkc_queue.h"

template <int G>
static bool run(int n_cells, int groups_total, int every, unsigned block) {
    static_assert(rkcdev::QUEUE_PARTS == 16 && rkcdev::QUEUE_STRIDE == 32, "count() below");
    std::vector<int> queue(rkcdev::QUEUE_INTS, 0);
    P = Params{queue.data(), n_cells, groups_total};
    claimed.assign((size_t)n_cells, 0);
    others_every = every;
    reads = 0;
    blockIdx.x = block;
    std::vector<std::vector<int>> got(G);
    std::vector<rkcdev::Claim<G>> claim(G);
    // one call of next() at a time, as the integrator's loop has it
    for (int call = 0; call <= n_cells; ++call) {
        meet.active = G;
        std::vector<std::thread> lanes;
        for (int g = 0; g < G; ++g)
            lanes.emplace_back([&, g] {
                threadIdx.x = (unsigned)g;
                if (call == 0) claim[g].init();
                got[g].push_back(claim[g].next(P, g));
                meet.drop();
            });
        for (auto &t : lanes) t.join();
        for (int g = 1; g < G; ++g)
            if (got[g].back() != got[0].back() || claim[g].part != claim[0].part ||
                claim[g].left != claim[0].left) {
                std::printf("FAIL G %d n %d groups %d every %d: lane %d has position %d, part %d; "
                            "lane 0 %d, part %d\n", G, n_cells, groups_total, every, g,
                            got[g].back(), claim[g].part, got[0].back(), claim[0].part);
                return false;
            }
        if (got[0].back() == n_cells) break;
    }
    for (int i = groups_total; i < n_cells; ++i)
        if (claimed[(size_t)i] != 1) {
            std::printf("FAIL G %d n %d groups %d every %d: position %d claimed %d times\n", G,
                        n_cells, groups_total, every, i, claimed[(size_t)i]);
            return false;
        }
    return true;
}

int main() {
    bool ok = true;
    // fewer cells than groups, fewer than parts, parts of unequal length; the
    // others silent, or claiming after every read, or after some
    for (int n : {3, 9, 21, 57})
        for (int every : {0, 1, 3, 7})
            for (unsigned block : {0u, 5u}) {
                ok = ok && run<8>(n, 4, every, block) && run<32>(n, 4, every, block) &&
                     run<64>(n, 4, every, block);
            }
    if (ok) std::printf("OK\n");
    return ok ? 0 : 1;
}
