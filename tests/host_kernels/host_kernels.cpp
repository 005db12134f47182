// Runs the 16-series LSTM kernels on the CPU, thread by thread, and checks what does not depend on values:
//   every global access lies in the workspace;
//   every wave of a workgroup meets the same barriers;
//   between two barriers no wave touches LDS that another one writes.
// The interval between two barriers that an access falls into, and its address, depend on the wave, the lane and the
// shape alone, so the threads need not run side by side.
//
// usage: host_kernels B T I H hidden lambda_cs fwd|bwd|all  dilation [dilation ...]   (blocks of one layer)
//        host_kernels plan ... the same: what the plan chose per layer, nothing is run
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <unordered_map>
#include <vector>

#include "esrnn_internal.h"
#include "three_term.h"

dim3 threadIdx, blockIdx, gridDim;

namespace {
const char *g_ws, *g_ws_end;
int g_wave, g_interval;
char g_what[96];
struct Use { unsigned short readers, writers; };
std::unordered_map<size_t, std::vector<Use>> g_lds;      // by address / 2, then by interval

[[noreturn]] void fail(const char *why)
{
    printf("FAIL %s: %s (block %u %u, wave %d, after barrier %d)\n", g_what, why, blockIdx.x, blockIdx.y, g_wave, g_interval);
    exit(1);
}
}  // namespace

extern "C" char __start_lds, __stop_lds;
static void touch(const void *at, int bytes, bool write)
{
    const char *p = static_cast<const char *>(at);
    if (p < &__start_lds || p >= &__stop_lds) return;
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
void host_global(const void *at, int bytes)
{
    const char *p = static_cast<const char *>(at);
    if (p < g_ws || p + bytes > g_ws_end) fail("global access outside the workspace");
}

// one launch: kernel(args) for every thread of the grid
void host_launch(void (*thread)(const void *), const void *args, dim3 grid, int threads)
{
    gridDim = grid;
    for (blockIdx.y = 0; blockIdx.y < grid.y; ++blockIdx.y)
        for (blockIdx.x = 0; blockIdx.x < grid.x; ++blockIdx.x) {
            g_lds.clear();
            int barriers = -1;
            for (int t = 0; t < threads; ++t) {
                threadIdx.x = t;
                g_wave = t / 64;
                g_interval = 0;
                thread(args);
                if (barriers >= 0 && barriers != g_interval) fail("waves meet different numbers of barriers");
                barriers = g_interval;
            }
            for (const auto &e : g_lds)
                for (size_t i = 0; i < e.second.size(); ++i) {
                    const unsigned w = e.second[i].writers, all = w | e.second[i].readers;
                    if (w && (all & (all - 1))) {
                        g_interval = (int)i;
                        g_wave = __builtin_ctz(w);
                        fail("LDS written by this wave is touched by another one with no barrier in between");
                    }
                }
        }
}

namespace esrnn {
// (the 4-series kernels are not built here)
hipError_t launch_lstm_forward_narrow(const Plan &, int, const int32_t *, const float *, float *, hipStream_t) { return hipErrorInvalidValue; }
}  // namespace esrnn

int main(int argc, char **argv)
{
    using namespace esrnn;
    const bool plan_only = argc > 1 && !strcmp(argv[1], "plan");
    if (plan_only) { --argc; ++argv; }
    if (argc < 9) return 2;
    esrnn_config c{};
    c.B = atoi(argv[1]); c.T = atoi(argv[2]); c.I = atoi(argv[3]); c.H = atoi(argv[4]); c.hidden = atoi(argv[5]);
    c.lambda_cs = (float)atof(argv[6]);
    c.tau = 0.5f;
    const bool fwd = strcmp(argv[7], "bwd"), bwd = strcmp(argv[7], "fwd");
    c.n_blocks = argc - 8;
    for (int i = 0; i < c.n_blocks; ++i) { c.layers_in_block[i] = 1; c.dilation[i][0] = atoi(argv[8 + i]); }
    static Plan pl;
    if (build_plan(c, pl) != ESRNN_OK) { printf("refused\n"); return 1; }
    if (plan_only) {
        printf("total %zu\n", pl.total_floats);
        for (int l = 0; l < pl.L; ++l)
            printf("layer %d dilation %d narrow %d %d chains %d %d\n", l, pl.layer[l].dil, pl.layer[l].narrow_fwd,
                   pl.layer[l].narrow_bwd, pl.layer[l].chains, pl.layer[l].chains_bwd);
        return 0;
    }
    float *ws = static_cast<float *>(aligned_alloc(256, pl.total_floats * 4));
    memset(ws, 0, pl.total_floats * 4);
    g_ws = reinterpret_cast<const char *>(ws);
    g_ws_end = g_ws + pl.total_floats * 4;
    // tiles of different lengths, one without any position
    for (int t = 0; t < pl.NB; ++t) reinterpret_cast<int32_t *>(ws + pl.pmax)[t] = t == 0 ? pl.P : t == 1 ? (pl.P + 1) / 2 : 0;
    std::vector<int32_t> lengths(c.B, c.T);
    for (int l = 0; l < pl.L; ++l) {
        const LayerPlan &lp = pl.layer[l];
        for (int stash = 0; fwd && stash < 2; ++stash) {
            snprintf(g_what, sizeof g_what, "forward, layer %d (%d, %d unit tiles)", l, pl.HT, lp.KXT);
            if (launch_lstm_forward(pl, l, lengths.data(), nullptr, ws, ForwardMode{stash != 0, nullptr}, nullptr) != hipSuccess) return 3;
        }
        if (bwd && bwd_three_term(pl.HT)) {
            snprintf(g_what, sizeof g_what, "reverse, layer %d (%d, %d unit tiles)", l, pl.HT, lp.KXT);
            const LstmBwdSources src{{ws + lp.gsrc[0], ws + lp.gsrc[lp.n_gsrc >= 2]}, std::min(lp.n_gsrc, 2)};
            if (launch_lstm_backward_three_term(pl, l, src, lengths.data(), ws, nullptr) != hipSuccess) return 3;
        }
    }
    printf("ok\n");
    return 0;
}
