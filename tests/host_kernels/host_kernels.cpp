// Runs the kernels on the CPU, thread by thread, and checks what does not depend on values:
//   every access lies in the workspace, in an input or output at its size, in the launch's LDS, or in the program itself;
//   every wave of a workgroup meets the same barriers (or none: it has ended before the first one);
//   between two barriers no wave touches LDS that another one writes (what is never read may be written by all);
//   what a workgroup reads of another one of its launch was stored past the caches, and complete when the position was counted that
//   the reading wave has waited for, however late every count shows;
//   a wave that has given up a wait for another workgroup waits no more, and what it reads from then on is NaN.
// The interval between two barriers that an access falls into, and its address, depend on the wave, the lane and the
// shape alone, so the threads need not run side by side.
//
// usage: host_kernels B T I H hidden lambda_cs fwd|bwd|all  dilation [dilation ...]   (blocks of one layer)
//        host_kernels plan ... the same: what the plan chose per layer, nothing is run
//        host_kernels step B T I H hidden m1 m2 lambda_cs lengths dilation [dilation ...]: all kernels of a training step and of
//        a forecast; lengths: of every 64 series (a wave's bounds are those of its own lane here), separated by commas
//        host_kernels uncleared ... the same, with what a workspace may hold in the words of the launches of several layers
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <tuple>
#include <unordered_map>
#include <vector>

#include "esrnn_internal.h"
#include "three_term.h"

dim3 threadIdx, blockIdx, gridDim;

namespace {
struct Range { const char *begin, *end; };
std::vector<Range> g_memory;        // what the kernels may touch beside LDS, the stack and the program's own data
const char *g_stack;
size_t g_dynamic_lds;
int g_wave, g_interval;
bool g_stuck;                       // nothing that a wave waits for ever comes
int g_looks;                        // of this thread, while it waited

// ---- launches whose workgroups follow each other: they run one after the other here, in the order of their tickets ----
struct Launch {
    bool on = false;
    const char *ws = nullptr, *words = nullptr, *words_end = nullptr;
    std::vector<int> writer;                    // per float of the workspace: the workgroup that wrote it, and
    std::vector<int> count;                     // the first count of it that covers that store (kNever: none does)
    std::unordered_map<int, const char *> word; // by workgroup
    std::unordered_map<const char *, std::vector<int>> counts;     // by word: all that it has held, rising
} g_launch;
constexpr int kNever = 1 << 30;
struct Stored { int at, seq, interval; bool shared; };
struct Counted { int interval, value; };
// of the workgroup that runs
int g_group;
std::vector<Counted> g_counted;
std::unordered_map<int, int> g_complete;        // float of the workspace: interval in which its store is known to be complete
struct Need { int wave, wait, value; const char *word; };
std::vector<Need> g_needs;                      // what its waves have read: (wave, wait before it) has to have seen value in word
std::map<std::tuple<int, int, const char *>, int> g_seen;          // what they saw
// of the thread that runs
std::vector<Stored> g_stored;
int g_issued, g_waits, g_view;                  // stores so far; waits for another workgroup that have ended; counts seen of its word
const char *g_word;                             // that it looks at
bool g_fresh;                                   // the next look shows one count more
char g_what[96];
struct Use { unsigned short readers, writers; };
std::unordered_map<size_t, std::vector<Use>> g_lds;      // by address / 2, then by interval

[[noreturn]] void fail(const char *why)
{
    printf("FAIL %s: %s (block %u %u, wave %d, after barrier %d)\n", g_what, why, blockIdx.x, blockIdx.y, g_wave, g_interval);
    exit(1);
}

// zeros, where the kernels may read and write
template <class T>
T *memory(size_t n)
{
    const size_t bytes = (n * sizeof(T) + 255) / 256 * 256;
    char *p = static_cast<char *>(aligned_alloc(256, bytes));
    memset(p, 0, bytes);
    g_memory.push_back({p, p + n * sizeof(T)});
    return reinterpret_cast<T *>(p);
}

bool known(const char *p, int bytes)
{
    for (const Range &r : g_memory)
        if (p >= r.begin && p + bytes <= r.end) return true;
    return false;
}
}  // namespace

// an access to the workspace in a launch whose workgroups follow each other
static void follow(const char *p, int bytes, bool write, bool shared)
{
    Launch &l = g_launch;
    if (!l.on || p < l.ws || p >= l.ws + 4 * l.writer.size() || (p >= l.words && p < l.words_end)) return;
    for (int at = (int)((p - l.ws) / 4), end = at + std::max(bytes / 4, 1); at < end; ++at) {
        if (write) {
            g_stored.push_back({at, g_issued, kNever, shared});
        } else if (l.writer[at] >= 0 && l.writer[at] != g_group) {
            if (!shared) fail("another workgroup's data read through the caches");
            if (l.count[at] == kNever) fail("another workgroup's data read that no count covers");
            g_needs.push_back({g_wave, g_waits, l.count[at], l.word[l.writer[at]]});
        }
    }
}

__attribute__((section("lds"), aligned(256))) float host_dynamic_lds[40960];     // the most a workgroup has
extern "C" char __start_lds, __stop_lds, __executable_start, end;
static void touch(const void *at, int bytes, bool write)
{
    const char *p = static_cast<const char *>(at);
    if (p < &__start_lds || p >= &__stop_lds) {
        const bool own = (p >= &__executable_start && p < &end) || (p >= static_cast<char *>(__builtin_frame_address(0)) && p < g_stack);
        if (!own && !known(p, bytes)) fail("access outside the workspace, the inputs and the outputs");
        if (!own) follow(p, bytes, write, false);
        return;
    }
    const char *dynamic = reinterpret_cast<const char *>(host_dynamic_lds);
    if (p >= dynamic && p < dynamic + sizeof host_dynamic_lds && p + bytes > dynamic + g_dynamic_lds) fail("access past the LDS of the launch");
    for (int i = 0; i < std::max(bytes / 2, 1); ++i) {
        std::vector<Use> &u = g_lds[reinterpret_cast<size_t>(p) / 2 + i];
        if (u.size() <= (size_t)g_interval) u.resize(g_interval + 1, Use{0, 0});
        (write ? u[g_interval].writers : u[g_interval].readers) |= 1u << g_wave;
    }
}
#define X(n, T)                                                                            \
    extern "C" void __sanitizer_cov_load##n(T *at) { touch(at, n, false); }                \
    extern "C" void __sanitizer_cov_store##n(T *at) { touch(at, n, true); }
X(1, uint8_t) X(2, uint16_t) X(4, uint32_t) X(8, uint64_t) X(16, __uint128_t)
#undef X

void host_barrier() { ++g_interval; }

unsigned long long host_ballot(bool complete)
{
    if (!complete) return 0;
    if (g_launch.on) {
        g_seen[{g_wave, g_waits + 1, g_word}] = g_view ? g_launch.counts[g_word][g_view - 1] : 0;
        ++g_waits;
    }
    return ~0ull;
}
void host_sleep()
{
    if (++g_looks > HOST_MOST_LOOKS) fail(g_stuck ? "a wave waits again after it has given up a wait" : "a wave waits for what never comes");
    g_fresh = true;
}
void host_wait(int but)
{
    for (Stored &st : g_stored)
        if (st.interval == kNever && st.seq < g_issued - but) st.interval = g_interval;
}
void host_read(host_rsrc r, unsigned at, int shared, void *to, int bytes)
{
    const char *p = r.base + at;
    if (at + bytes > r.bytes) fail("read past the end of a buffer");
    if (!known(p, bytes)) fail("access outside the workspace, the inputs and the outputs");
    memcpy(to, p, bytes);
    if (g_launch.on && p >= g_launch.words && p < g_launch.words_end) {
        const std::vector<int> &counts = g_launch.counts[g_word = p];
        if (g_fresh && g_view < (int)counts.size()) ++g_view;
        g_fresh = false;
        const int count = g_view ? counts[g_view - 1] : 0;
        memcpy(to, &count, bytes);
    } else {
        follow(p, bytes, false, shared);
    }
}
void host_write(host_rsrc r, unsigned at, int shared, const void *from, int bytes)
{
    char *p = const_cast<char *>(r.base) + at;
    if (at + bytes <= r.bytes) {        // (else it is dropped)
        if (!known(p, bytes)) fail("access outside the workspace, the inputs and the outputs");
        memcpy(p, from, bytes);
        if (g_launch.on && p >= g_launch.words && p < g_launch.words_end) {
            int value;
            memcpy(&value, from, 4);
            g_launch.word[g_group] = p;
            std::vector<int> &counts = g_launch.counts[p];
            if (!shared || value < (counts.empty() ? 0 : counts.back())) fail("a count that falls, or is kept in a cache");
            if (counts.empty() || value > counts.back()) counts.push_back(value);
            g_counted.push_back({g_interval, value});
        } else {
            follow(p, bytes, true, shared);
        }
    }
    ++g_issued;
}

// a thread of the workgroup has ended
static void thread_done()
{
    for (const Stored &st : g_stored) {
        g_launch.writer[st.at] = g_group;
        int &complete = g_complete[st.at];
        complete = std::max(complete, st.shared ? st.interval : kNever);
    }
    g_stored.clear();
    g_issued = g_waits = g_view = 0;
    g_word = nullptr;
    g_fresh = false;
}
// all threads have
static void group_done()
{
    for (const auto &[at, complete] : g_complete) {
        g_launch.count[at] = kNever;
        for (const Counted &c : g_counted)      // (a barrier lies between the wait and the count)
            if (c.interval > complete) g_launch.count[at] = std::min(g_launch.count[at], c.value);
    }
    for (const Need &n : g_needs) {
        const auto seen = g_seen.find({n.wave, n.wait, n.word});
        g_wave = n.wave;
        if (seen == g_seen.end() || seen->second < n.value) fail("another workgroup's data read before they are known to be complete");
    }
    g_complete.clear();
    g_counted.clear();
    g_needs.clear();
    g_seen.clear();
    ++g_group;
}

void host_run(dim3 grid, int threads, size_t dynamic_lds, void (*thread)(void *), void *context)
{
    gridDim = grid;
    g_dynamic_lds = dynamic_lds;
    for (blockIdx.y = 0; blockIdx.y < grid.y; ++blockIdx.y)
        for (blockIdx.x = 0; blockIdx.x < grid.x; ++blockIdx.x) {
            g_lds.clear();
            int barriers = 0;
            for (int t = 0; t < threads; ++t) {
                threadIdx.x = t;
                g_wave = t / 64;
                g_interval = g_looks = 0;
                thread(context);
                if (g_launch.on) thread_done();
                if (barriers > 0 && g_interval > 0 && barriers != g_interval) fail("waves meet different numbers of barriers");
                barriers = std::max(barriers, g_interval);
            }
            for (const auto &e : g_lds) {
                unsigned readers = 0;
                for (const Use &u : e.second) readers |= u.readers;
                if (!readers) continue;
                for (size_t i = 0; i < e.second.size(); ++i) {
                    const unsigned w = e.second[i].writers, all = w | e.second[i].readers;
                    if (w && (all & (all - 1))) {
                        g_interval = (int)i;
                        g_wave = __builtin_ctz(w);
                        fail("LDS written by this wave is touched by another one with no barrier in between");
                    }
                }
            }
            if (g_launch.on) group_done();
        }
}

using namespace esrnn;

// every kernel of a training step, with and without a reverse pass to come, and of a forecast
static int step(const Plan &pl, const std::vector<int> &lens, bool uncleared)
{
    float *ws = memory<float>(pl.total_floats);
    const float *y = memory<float>((size_t)pl.T * pl.B), *es = memory<float>((size_t)pl.K * pl.B), *weights = memory<float>(pl.n_weights);
    float *loss = memory<float>(1), *in_sample = memory<float>((size_t)pl.P * pl.B * pl.H), *ahead = memory<float>((size_t)pl.B * pl.H);
    float *grad_es = memory<float>((size_t)pl.K * pl.B), *grad_weights = memory<float>(pl.n_weights);
    int32_t *lengths = memory<int32_t>(pl.B), *shorter = memory<int32_t>(pl.B);
    for (int b = 0; b < pl.B; ++b) {
        lengths[b] = lens[b / 64 % lens.size()];
        shorter[b] = lengths[b] - pl.H;
    }
    auto run = [&](const char *what, int layer, hipError_t e) {
        if (e == hipSuccess) return;
        printf("FAIL %s %d: not launched\n", what, layer);
        exit(1);
    };
#define RUN(layer, call) (snprintf(g_what, sizeof g_what, "%s, layer %d", #call, layer), run(#call, layer, call))
    // around a launch of several layers.  (`uncleared`: a reverse pass given a workspace that no forward pass has run in, whose
    // words are whatever is there)
    auto begin = [&](size_t at, int groups) {
        unsigned *const words = reinterpret_cast<unsigned *>(ws + at);
        const size_t n = (size_t)(1 + groups) * kWordStride;
        g_stuck = uncleared;
        if (uncleared) return void(std::fill_n(words, n, 0xbf80bf80u));
        for (int i = 0; i <= groups; ++i)
            if (words[i * kWordStride]) fail("words that are not cleared");
        g_launch = Launch{true, reinterpret_cast<char *>(ws), reinterpret_cast<char *>(words), reinterpret_cast<char *>(words + n),
                          std::vector<int>(pl.total_floats, -1), std::vector<int>(pl.total_floats, kNever), {}, {}};
        g_group = 0;
    };
    auto done = [&] { g_launch.on = false; };
    for (int pass = 0; pass < 3; ++pass) {
        const bool reverse = pass == 0, predict = pass == 2;
        const ForwardMode mode{reverse, predict ? reinterpret_cast<unsigned *>(ws + pl.O) : nullptr, predict};
        const int32_t *n = predict ? reinterpret_cast<const int32_t *>(ws + pl.len_ext) : lengths;
        RUN(-1, launch_es_forward(pl, y, predict ? shorter : lengths, es, weights, ws, mode, nullptr));
        RUN(-1, launch_window_forward(pl, nullptr, ws, nullptr));
        for (int l = 0; l < pl.L; ++l) RUN(l, launch_lstm_forward(pl, l, n, weights, ws, mode, nullptr));
        if (pl.together_fwd) {
            begin(pl.together_words, pl.together_groups);
            // (sums of the residual input and a state that is not formed here: the input's NaN has to show in them)
            const size_t out = pl.layer[pl.together_fwd - 1].out, size = (size_t)pl.P * pl.NB * pl.HT * 64;
            if (out) std::fill_n(ws + out, size, 0.0f);
            RUN(pl.together_fwd, launch_lstm_forward_together(pl, n, weights, ws, mode, nullptr));
            done();
            if (uncleared && out && std::none_of(ws + out, ws + out + size, [](float v) { return v != v; })) fail("no NaN after a wait was given up");
        }
        if (predict) {
            RUN(-1, launch_head_last(pl, n, ws, ahead, nullptr));
            continue;
        }
        RUN(-1, launch_head(pl, n, ws, reverse, nullptr));
        RUN(-1, launch_loss_and_forecasts(pl, n, ws, loss, in_sample, nullptr));
        if (!reverse) continue;
        for (int l = pl.L - 1; l >= 0; --l) RUN(l, launch_lstm_backward(pl, l, n, ws, nullptr));
        if (pl.together_bwd) {
            begin(pl.together_words_bwd, pl.together_groups_bwd);
            RUN(pl.together_bwd, launch_lstm_backward_together(pl, n, ws, nullptr));
            done();
        }
        RUN(-1, launch_window_backward(pl, n, ws, true, nullptr));
        RUN(-1, launch_es_backward(pl, y, n, es, ws, grad_es, grad_weights, nullptr));
    }
#undef RUN
    printf("ok\n");
    return 0;
}

int main(int argc, char **argv)
{
    g_stack = static_cast<const char *>(__builtin_frame_address(0)) + 4096;
    const bool plan_only = argc > 1 && !strcmp(argv[1], "plan");
    if (plan_only) { --argc; ++argv; }
    if (argc < 9) return 2;
    esrnn_config c{};
    static Plan pl;
    const bool uncleared = !strcmp(argv[1], "uncleared");
    if (uncleared || !strcmp(argv[1], "step")) {
        c.B = atoi(argv[2]); c.T = atoi(argv[3]); c.I = atoi(argv[4]); c.H = atoi(argv[5]); c.hidden = atoi(argv[6]);
        c.m1 = atoi(argv[7]); c.m2 = atoi(argv[8]); c.lambda_cs = (float)atof(argv[9]);
        c.n_seas = (c.m1 > 0) + (c.m2 > 0);
        c.lambda_lv = 1.0f;
        c.tau = 0.5f;
        std::vector<int> lens;
        for (char *at = argv[10]; at; at = strchr(at, ',') ? strchr(at, ',') + 1 : nullptr) lens.push_back(atoi(at));
        c.n_blocks = argc - 11;
        for (int i = 0; i < c.n_blocks; ++i) { c.layers_in_block[i] = 1; c.dilation[i][0] = atoi(argv[11 + i]); }
        if (c.B % 64 || build_plan(c, pl) != ESRNN_OK) { printf("refused\n"); return 1; }
        return step(pl, lens, uncleared);
    }
    c.B = atoi(argv[1]); c.T = atoi(argv[2]); c.I = atoi(argv[3]); c.H = atoi(argv[4]); c.hidden = atoi(argv[5]);
    c.lambda_cs = (float)atof(argv[6]);
    c.tau = 0.5f;
    const bool fwd = strcmp(argv[7], "bwd"), bwd = strcmp(argv[7], "fwd");
    c.n_blocks = argc - 8;
    for (int i = 0; i < c.n_blocks; ++i) { c.layers_in_block[i] = 1; c.dilation[i][0] = atoi(argv[8 + i]); }
    if (build_plan(c, pl) != ESRNN_OK) { printf("refused\n"); return 1; }
    if (plan_only) {
        printf("total %zu\n", pl.total_floats);
        for (int l = 0; l < pl.L; ++l)
            printf("layer %d dilation %d narrow %d %d chains %d %d\n", l, pl.layer[l].dil, pl.layer[l].narrow_fwd,
                   pl.layer[l].narrow_bwd, pl.layer[l].chains, pl.layer[l].chains_bwd);
        printf("together %d %d\n", pl.together_fwd, pl.together_bwd);
        return 0;
    }
    float *ws = memory<float>(pl.total_floats);
    // tiles of different lengths, one without any position
    for (int t = 0; t < pl.NB; ++t) reinterpret_cast<int32_t *>(ws + pl.pmax)[t] = t == 0 ? pl.P : t == 1 ? (pl.P + 1) / 2 : 0;
    int32_t *lengths = memory<int32_t>(c.B);
    std::fill(lengths, lengths + c.B, c.T);
    for (int l = 0; l < pl.L; ++l) {
        const LayerPlan &lp = pl.layer[l];
        for (int stash = 0; fwd && stash < 2; ++stash) {
            snprintf(g_what, sizeof g_what, "forward, layer %d (%d, %d unit tiles)", l, pl.HT, lp.KXT);
            if (launch_lstm_forward(pl, l, lengths, nullptr, ws, ForwardMode{stash != 0, nullptr}, nullptr) != hipSuccess) return 3;
        }
        if (bwd && bwd_three_term(pl.HT)) {
            snprintf(g_what, sizeof g_what, "reverse, layer %d (%d, %d unit tiles)", l, pl.HT, lp.KXT);
            const LstmBwdSources src{{ws + lp.gsrc[0], ws + lp.gsrc[lp.n_gsrc >= 2]}, std::min(lp.n_gsrc, 2)};
            if (launch_lstm_backward_three_term(pl, l, src, lengths, ws, nullptr) != hipSuccess) return 3;
        }
    }
    printf("ok\n");
    return 0;
}
