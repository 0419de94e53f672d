// Runs token_tree (csrc/tokens.hpp) on the host, a fiber per thread, under different orders of the
// threads between two barriers, and checks that every thread passes the same barriers, that a count
// overflow is reported, and that the trees are those of popping one cycle after the other.
#include <ucontext.h>

#include <algorithm>
#include <cstdlib>
#include <random>
#include <vector>

#include "tokens.hpp"

Dim threadIdx{0}, blockDim{0}, blockIdx{0};

namespace {

enum Order { kAscending, kDescending, kShuffled, kOrders };

struct Fiber {
    ucontext_t context;
    std::vector<char> stack;
    bool at_barrier = false, ended = false;
};

std::vector<Fiber> fibers;
ucontext_t scheduler;
int current = 0;
bool preempt = false;
std::mt19937 rng(1);
std::function<void()> body;

void fiber_main() {
    body();
    fibers[current].ended = true;
    swapcontext(&fibers[current].context, &scheduler);
}

void yield() { swapcontext(&fibers[current].context, &scheduler); }

// Runs the work-group; false: some threads ended while others wait at a barrier.
bool run(int threads, Order order, std::function<void()> f) {
    body = std::move(f);
    blockDim.x = static_cast<uint32_t>(threads);
    fibers = std::vector<Fiber>(threads);
    for (Fiber& t : fibers) {
        t.stack.resize(1 << 16);
        getcontext(&t.context);
        t.context.uc_stack.ss_sp = t.stack.data();
        t.context.uc_stack.ss_size = t.stack.size();
        t.context.uc_link = nullptr;
        makecontext(&t.context, fiber_main, 0);
    }
    std::vector<int> turn(threads);
    for (int i = 0; i < threads; ++i) turn[i] = order == kDescending ? threads - 1 - i : i;
    while (true) {
        // every thread to its next barrier or its end
        std::vector<int> left = turn;
        if (order == kShuffled) std::shuffle(left.begin(), left.end(), rng);
        while (!left.empty()) {
            const size_t at = preempt ? rng() % left.size() : 0;
            current = left[at];
            threadIdx.x = static_cast<uint32_t>(current);
            swapcontext(&scheduler, &fibers[current].context);
            if (fibers[current].at_barrier || fibers[current].ended) left.erase(left.begin() + static_cast<long>(at));
        }
        const auto ended = std::count_if(fibers.begin(), fibers.end(), [](const Fiber& t) { return t.ended; });
        if (ended == threads) return true;
        if (ended != 0) return false;
        for (Fiber& t : fibers) t.at_barrier = false;
    }
}

struct Graph {
    int n = 0, root = 0;
    std::vector<std::vector<std::pair<uint32_t, double>>> row;   // neighbour, weight up to it
    void edge(uint32_t a, uint32_t b, double w) {
        for (auto [x, y] : {std::pair{a, b}, std::pair{b, a}})
            row[x].push_back({y, (row[x].empty() ? 0.0 : row[x].back().second) + w});
    }
};
Graph graph;

}  // namespace

void __syncthreads() {
    fibers[current].at_barrier = true;
    yield();
}
void switch_point() {
    if (preempt && rng() % 4 == 0) yield();
}

namespace rwc {
namespace {
uint32_t kCntMax = 0;
uint32_t draw(uint32_t v, uint32_t k, uint32_t sample) {
    uint64_t z = (static_cast<uint64_t>(sample) << 40) ^ (static_cast<uint64_t>(v) << 24) ^ k;
    for (int i = 0; i < 2; ++i) {
        z += 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z ^= z >> 27;
    }
    const auto& row = graph.row[v];
    const double x = static_cast<double>(z >> 11) * 0x1p-53 * row.back().second;
    for (const auto& [to, upto] : row)
        if (x < upto) return to;
    return row.back().first;
}
}  // namespace
}  // namespace rwc

using namespace rwc;

namespace {

Graph grid(int a, int b, double heavy) {   // heavy: the weight of the last edge of the first and the last row
    Graph g;
    g.n = a * b;
    g.root = (a / 2) * b + b / 2;
    g.row.resize(g.n);
    for (int i = 0; i < a; ++i)
        for (int j = 0; j < b; ++j) {
            const uint32_t u = static_cast<uint32_t>(i * b + j);
            if (j + 1 < b) g.edge(u, u + 1, j + 2 == b && (i == 0 || i + 1 == a) ? heavy : 1.0);
            if (i + 1 < a) g.edge(u, u + static_cast<uint32_t>(b), 1.0);
        }
    return g;
}

// One tree; the error word, or -1 if the barriers did not pair.
template <bool kWide>
int tree(int threads, Order order, uint32_t sample, std::vector<uint32_t>* arrows, std::vector<uint32_t>* counts) {
    TokenLayout layout(graph.n);
    const GraphArgs args{graph.n, graph.root, nullptr, 1u << 30, graph.n};
    std::vector<uint32_t> lds(static_cast<size_t>(layout.words()) + 64), cnt(graph.n), node(graph.n), ready(graph.n);
    uint32_t ctl[8] = {}, err = 0;
    const bool paired = run(threads, order, [&] {
        TokenTree<kWide> w;
        if constexpr (kWide) {
            w.node = node.data();
            w.ready = ready.data();
            w.width = 32u - static_cast<uint32_t>(__builtin_clz(static_cast<uint32_t>(graph.n - 1)));
        } else {
            w.node = lds.data();
            w.ready = reinterpret_cast<uint16_t*>(lds.data() + layout.nodes);
        }
        token_tree<false, kWide>(args, sample, 0, layout, lds.data() + layout.nodes + layout.ready_words, w, cnt.data(), ctl,
                                 &err);
    });
    if (!paired) return -1;
    *counts = cnt;
    const uint32_t bits = kWide ? 32u - static_cast<uint32_t>(__builtin_clz(static_cast<uint32_t>(graph.n - 1))) : 15u;
    arrows->resize(graph.n);
    for (int v = 0; v < graph.n; ++v) (*arrows)[v] = (kWide ? node[v] : lds[v]) & ((1u << bits) - 1u);
    return static_cast<int>(err);
}

// Wilson's algorithm on the same stacks, one walk after the other.
void serial(uint32_t sample, std::vector<uint32_t>* arrows, std::vector<uint32_t>* counts) {
    std::vector<char> in_tree(graph.n, 0);
    in_tree[graph.root] = 1;
    arrows->assign(graph.n, 0);
    counts->assign(graph.n, 0);
    (*arrows)[graph.root] = static_cast<uint32_t>(graph.root);
    for (int s = 0; s < graph.n; ++s) {
        for (uint32_t u = static_cast<uint32_t>(s); !in_tree[u]; u = (*arrows)[u]) (*arrows)[u] = draw(u, (*counts)[u]++, sample);
        for (uint32_t u = static_cast<uint32_t>(s); !in_tree[u]; u = (*arrows)[u]) in_tree[u] = 1;
    }
}

template <bool kWide>
int check(const char* what, int threads, uint32_t samples, bool overflows) {
    int bad = 0;
    std::vector<uint32_t> a, c, ra, rc;
    for (uint32_t s = 0; s < samples; ++s) {
        serial(s, &ra, &rc);
        for (int o = 0; o < kOrders; ++o) {
            const int err = tree<kWide>(threads, static_cast<Order>(o), s, &a, &c);
            const bool right = overflows ? err == static_cast<int>(kErrCountOverflow) : err == 0 && a == ra && c == rc;
            if (!right && ++bad <= 3)
                std::printf("%s, %s, order %d, sample %u: %s\n", what, kWide ? "wide" : "narrow", o, s,
                            err < 0 ? "the barriers do not pair" : "wrong result");
        }
    }
    return bad;
}

template <bool kWide>
int all() {
    int bad = 0;
    for (int p = 0; p < (kWide ? 2 : 1); ++p) {
        preempt = p == 1;
        kCntMax = (1u << 24) - 1;
        graph = grid(5, 7, 1.0);
        bad += check<kWide>("5x7", 8, 20, false);
        graph = grid(3, 11, 50.0);
        bad += check<kWide>("3x11 with heavy ends", 12, 20, false);
        if (!preempt) {
            graph = grid(29, 41, 1.0);   // more nodes than the lists hold
            bad += check<kWide>("29x41", 16, 3, false);
        }
        if (!preempt) {
            graph = grid(29, 41, 1.0);
            kCntMax = 4;
            bad += check<kWide>("29x41, overflow", 16, 2, true);
        }
        graph = grid(1, 9, 5000.0);   // the end pair goes back and forth until its count overflows
        kCntMax = 60;
        bad += check<kWide>("overflow", 8, 30, true);
    }
    return bad;
}

}  // namespace

int main() {
    const int bad = all<false>() + all<true>();
    std::printf("%d wrong\n", bad);
    return bad == 0 ? 0 : 1;
}
