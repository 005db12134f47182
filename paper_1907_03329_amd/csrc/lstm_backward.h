// Reverse pass of a dilated LSTM layer (Section 3.2, Table 1), 16 series per workgroup, hidden sizes up to 52: the
// kernel template and its launcher, included by the units that instantiate it.  (The forward pass and the general
// structure - series tiles x residue classes of the dilation - are described in lstm_forward.h.)
//
// Per position p of a chain (descending), with [x ; h] = [x_p ; h_{p-d}]:
//   A. every lane turns (dh, dc) of its hidden unit into the four gate pre-activation gradients da;
//   B. d[x ; h] = W^T da;
//   C. dW += da (x) [x ; h], contraction over the 16 series, in accumulators for the whole launch.
// All products run on the bf16 matrix pipe with fp32 accuracy (three_term.h).
//
// Kinds of waves, one barrier per position:
//   chain waves (two or three unit tiles each) carry the recurrence: A, and B for the h rows, split over the waves along
//     the contraction, so that a wave multiplies what it has just computed in registers; the partial results meet in
//     LDS and every wave sums those of its own units.  They also leave the three parts of da in LDS.
//   factor waves (hidden sizes up to 40) read the stash and form whatever of A does not depend on the recurrent
//     gradient, two positions ahead: a chain wave takes the factors of the next position out of one half of their buffer
//     while those of the one after it go to the other half. Before the loop a barrier of its own stands between the
//     first taking and the first refilling of the same half. A chain wave then has a dozen dependent instructions between the barrier and its
//     first product.  At 13 unit tiles the sixteen waves of a workgroup are taken: there seven chain waves of two tiles
//     do it themselves, one position ahead.
//   dx waves (one 16-row tile each) do B for the x rows, which nothing in the recurrence waits for, one position
//     behind, from the parts in LDS.  If the last tile of h rows has room for the x tiles that do not fill a tile of
//     their own, the chain waves' products carry them, and a dx wave sums and stores them.
//   dW waves (two rows of tiles each) do C one position behind.  They bring [x ; h], two positions ahead; both
//     operands are needed transposed (series along the contraction) and are read with the LDS transpose load.
// No wave waits for its own stores: those that load do not store, except a dx wave that brings a tile of [x ; h] where the
// dW waves do not suffice.
//
// What bounds it. Hidden 40, 4096 series, 61 positions: 90 - 94 us a layer (fp32 kernel: 128 - 131 us), first layer 70
// - 73 us (103 us), i.e. 1.45 us a position; 370 - 414 MB of traffic at 4.1 TB/s, where a large copy reaches 5.2. Without
// the dW waves' part it is 69 us, without dx and dW 61 us; without the dW products alone 82 us: the reads of
// transposed operands from LDS (80 of 195 KB a position) weigh more than the products (matrix pipe busy 36 %). Hidden
// 50, 240 steps, 1.64 - 1.82 GB: 440 - 485 us (780 - 810 us), first layer 340 - 375 us (517 us). Tried without gain: chain
// waves that form their own factors (12 waves: 90 us, first layer 74 us; alone on the chip 1.03 us a position against
// 0.92), five chain waves of two tiles (two of them share a SIMD), raised priority of the chain waves (+2 %), all
// operands of a consumer read at once (+3 %), dW waves that own 32 columns and read them from memory with 32x32
// products (54 KB less through LDS, but 97 us, first layer 85 us: three waves are then the longest of a position).
//
// LDS home of 16 rows x 16 series in one of the three parts: the four rows of a lane group as one 8-byte chunk per
// lane, [chunk][series], so that the wave that computes them writes whole chunks; the second half is shifted by 32
// bytes, which spreads the four chunks that a transpose load reads together over different banks.
//
// The transpose load (ds_read_b64_tr_b16, checked on the device): of each 16 lanes, lane i receives as element j what
// lane 4 j + i / 4 addressed, element i % 4.
#pragma once

#include "esrnn_internal.h"
#include "three_term.h"

namespace esrnn {

namespace {

struct LstmBwdArgs {
    const u32x2 *wpack;   // [row tiles of x, then of h][unit tile][part][64]: A operands of W^T da
    const float *xsrc;    // TL(4*KXT)
    const float *gates, *c, *hid;
    const float *gsrc[2]; // TL(HP): the gradient arriving at the hidden output is the sum of these
    int n_gsrc;           // 1 or 2; gsrc[1] repeats gsrc[0] when there is one
    float *gdst;          // TL(4*KXT)
    float *dw_partial;    // [NB*chains][HT*MB][4][64]
    float *db_partial;    // [NB*chains][HT][4][4]
    int NB, d;
    const int32_t *pmax;  // [NB] positions the longest series of a tile has: the tile's chains stop there
    // cell-state penalty (Section 8.4) of a block's first layer, kernels instantiated with CP only
    const int32_t *lengths;
    const Scalars *sc;
    float two_lambda_cs;
    int B, T, I, H;
};

// The positions of a workgroup in order: residue classes r, r + step, ..., each from its last position down.  Scalar,
// without branches and without 64-bit arithmetic (what a chain wave spends on it is on the critical path).
struct ChainWalk {
    int p;                          // position
    int r, step, d, base, top_mod, classes, NB, bt;
    __device__ ChainWalk(int first, int step_, int d_, int positions, int NB_, int bt_)
        : r(first), step(step_), d(d_), top_mod((positions - 1) % d_), classes(min(d_, positions)), NB(NB_), bt(bt_)
    {
        base = positions - 1 - top_mod;
        p = first < classes ? last(first) : 0;
    }
    __device__ int last(int rr) const { return base + rr - (rr > top_mod ? d : 0); }
    __device__ unsigned tile() const { return (unsigned)p * NB + bt; }      // (P NB < 2^31: B T is at most 2^30)
    __device__ int count() const    // (of a walk at its start)
    {
        if (r >= classes) return 0;
        const int n = (classes - 1 - r) / step + 1, longer = r <= top_mod ? (top_mod - r) / step + 1 : 0;
        return n * (base / d) + longer;
    }
    __device__ void next()          // stays at the last one
    {
        const int r2 = r + step, below = p - d, over = r2 < classes ? last(r2) : p;
        r = below < 0 && r2 < classes ? r2 : r;
        p = below >= 0 ? below : over;
    }
};
// tile `tile` of an array of tiles of `floats` floats
__device__ __forceinline__ const char *tile_at(const float *array, unsigned tile, unsigned floats)
{
    return reinterpret_cast<const char *>(array) + (unsigned long long)tile * (4u * floats);
}
// f(0), f(1), f(0), ... n times (arguments are compile-time constants): which half of a double buffer a position uses.
// Straight runs without an exit in between, or registers of requests in flight are copied - and waited for - there.
template <class F>
__device__ __forceinline__ void alternate(int n, F &&f)
{
    for (int k = 0; k + 1 < n; k += 2) {
        f(std::integral_constant<int, 0>{});
        f(std::integral_constant<int, 1>{});
    }
    if (n & 1) f(std::integral_constant<int, 0>{});
}

// Waits for a loaded operand here.  (Otherwise the wait ends up in the loop, where it covers every request in flight.)
__device__ __forceinline__ void arrived(u32x4 &v) { asm volatile("" : "+v"(v)); }
// A copy in a register of its own.  (A value that outlives the next request for its register would otherwise keep
// that request out of the register, and the loop would copy what has been requested instead, waiting for it.)  An
// instruction the compiler knows, so that it keeps its distance from matrix instructions that still read the register
// (inline assembly does not).
__device__ __forceinline__ float own_register(float v) { return __builtin_canonicalizef(v); }

// Workgroups are alone on their compute unit (for their registers), so the waves of one fill it: four per SIMD.
template <int HT, int KXT, bool CP>
__global__ void __launch_bounds__(64 * bwd_waves(HT, KXT), (bwd_waves(HT, KXT) + 3) / 4) lstm_backward_kernel(LstmBwdArgs a)
{
    constexpr int KT = KXT + HT, MB = (KT + 3) / 4;        // unit tiles and 16-column tiles of [x ; h]
    constexpr int RX = bwd_x_row_tiles(HT, KXT), RH = bwd_h_row_tiles(HT), ML = bwd_merged_tiles(HT, KXT);
    constexpr int NC = bwd_chain_waves(HT), NW = bwd_dw_waves(HT), NF = bwd_factor_waves(HT), HTE = bwd_even_tiles(HT);
    constexpr int HM = HT + ML;                            // unit tiles the chain waves' products give
    constexpr bool kTail = HT % 2 != 0;                    // a last row of dW tiles, dealt to the dW waves by columns
    constexpr int XC = (MB + NW - 1) / NW;                 // columns of it per wave
    constexpr int D = HT <= 10 ? 2 : 1;                    // positions the stash is requested ahead
    constexpr bool kReadAhead = HT <= 10;                  // dW and dx waves read operands from LDS one tile ahead (registers)
    static_assert(MB <= NW + RX, "every column tile needs a wave that brings it");

    __shared__ __align__(16) char da_lds[2][HTE * 3 * kPartBytes];   // [pair of unit tiles][part][unit tile of the pair]
    __shared__ __align__(16) char xh_lds[2][MB * 3 * kPartBytes];
    __shared__ float part_lds[2][NC][HM][64];
    __shared__ f32x4 factor_lds[NF > 0 ? 2 : 1][NF > 0 ? HT : 1][2][64];
    static_assert(sizeof(da_lds) + sizeof(xh_lds) + sizeof(part_lds) + sizeof(factor_lds) <= 128 * 1024,
                  "LDS budget of the reverse kernel");

    const int lane = threadIdx.x & 63, bt = blockIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index, known to be uniform
    const int g = lane >> 4, n = lane & 15;
    const int Pt = a.pmax[bt];      // the chains of this tile stop at its longest series
    const size_t part = (size_t)bt * gridDim.y + blockIdx.y;
    constexpr unsigned xtile = KXT * 64, htile = HT * 64;
    const unsigned lane4 = 4 * lane, lane16 = 16 * lane;
    auto da_at = [](int mt, int q) { return ((mt >> 1) * 6 + 2 * q + (mt & 1)) * kPartBytes; };
    const int own = 8 * lane + 32 * (lane >> 5);           // this lane's chunk inside a part
    const ChainWalk start(blockIdx.y, gridDim.y, a.d, Pt, a.NB, bt);
    const int n_steps = start.count();

    // ---- [x ; h] of one position, column tile nb: requested two positions ahead, split, left in LDS.
    float xraw[2][4];
    auto request_xh = [&](int set, int nb, const ChainWalk &at) {
        // scalar choices of a base, no branch around a request; tiles past the end alias the last one
        const char *x = tile_at(a.xsrc, at.tile(), xtile);
        const char *h = tile_at(a.hid, at.tile() - (at.p >= a.d ? (unsigned)a.d * a.NB : 0u), htile) - KXT * 256;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = min(4 * nb + e, KT - 1);
            xraw[set][e] = buf_load(make_rsrc(q < KXT ? x : h), lane4, q * 256);
        }
    };
    auto store_xh = [&](int set, int buf, int nb, bool has_prev) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = 4 * nb + e;
            v[e] = q < KXT || (q < KT && has_prev) ? xraw[set][e] : 0.0f;
        }
        const Parts p0 = split_pair<true>(v[0], v[1]), p1 = split_pair<true>(v[2], v[3]);
        char *dst = xh_lds[buf] + nb * 3 * kPartBytes + own;
        *reinterpret_cast<u32x2 *>(dst) = u32x2{p0.hi, p1.hi};
        *reinterpret_cast<u32x2 *>(dst + kPartBytes) = u32x2{p0.mid, p1.mid};
        *reinterpret_cast<u32x2 *>(dst + 2 * kPartBytes) = u32x2{p0.lo, p1.lo};
    };
    // A wave that consumes what the chain waves leave: `work(buf, tile, aside)` after the barrier that completes a
    // position.  LOAD: it also brings column tile nb, in `aside`, which `work` calls once its first operands are on
    // their way from LDS.  Every wave of the workgroup meets the same barriers.
    auto consumer = [&](auto load, int nb, auto &&work) {
        constexpr bool LOAD = decltype(load)::value;
        if (n_steps == 0) return;
        if constexpr (NF > 0) {                            // (the first factors complete; the first of them taken)
            lds_barrier();
            lds_barrier();
        }
        ChainWalk now = start, ask = start;
        int at[3];                                         // LOAD: the next three positions, the last one ask's
        if constexpr (LOAD) {
            const bool first = start.p >= a.d;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (i == 2) store_xh(0, 0, nb, first);
                __builtin_amdgcn_sched_barrier(0);
                request_xh(i % 2, nb, ask);
                ask.next();
                at[i] = ask.p;
            }
        }
        alternate(n_steps, [&](auto u) {
            constexpr int U = decltype(u)::value;
            lds_barrier();
            work(U, now.tile(), [&]() {
                if constexpr (LOAD) {
                    __builtin_amdgcn_sched_barrier(0);
                    store_xh(U ^ 1, U ^ 1, nb, at[0] >= a.d);
                    __builtin_amdgcn_sched_barrier(0);
                    request_xh(U ^ 1, nb, ask);
                    ask.next();
                    at[0] = at[1];
                    at[1] = at[2];
                    at[2] = ask.p;
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            now.next();
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ---- what a position's step A needs of the stash, for unit tiles t0 and t0 + 1: requested D positions ahead of
    // its use.  With the gates and the arriving gradients comes the cell state of the position that follows in the walk:
    // inside a chain that is the predecessor's, which this position needs too.
    f32x4 gt[D][2];
    float cnext[D][2], ga[D][2], gb[D][2], ccur[2];
    auto request = [&](int set, int t0, auto njc, unsigned tile, unsigned next_tile) {
        constexpr int nj = decltype(njc)::value;
        const buf_rsrc r_g = make_rsrc(tile_at(a.gates, tile, 4 * htile)), r_c = make_rsrc(tile_at(a.c, next_tile, htile));
        const buf_rsrc r_a = make_rsrc(tile_at(a.gsrc[0], tile, htile)), r_b = make_rsrc(tile_at(a.gsrc[1], tile, htile));
#pragma unroll
        for (int j = 0; j < nj; ++j) {
            gt[set][j] = buf_load4(r_g, lane16, (t0 + j) * 1024);
            cnext[set][j] = buf_load(r_c, lane4, (t0 + j) * 256);
            ga[set][j] = buf_load(r_a, lane4, (t0 + j) * 256);
            gb[set][j] = buf_load(r_b, lane4, (t0 + j) * 256);
        }
    };
    auto request_first_c = [&](int t0, auto njc, unsigned tile) {
        constexpr int nj = decltype(njc)::value;
        const buf_rsrc r_c = make_rsrc(tile_at(a.c, tile, htile));
#pragma unroll
        for (int j = 0; j < nj; ++j) ccur[j] = buf_load(r_c, lane4, (t0 + j) * 256);
    };
    const float g2_scale = a.n_gsrc >= 2 ? 1.0f : 0.0f;
    int n_valid = 0;                    // positions below this take part in the loss for this lane's series (CP only)
    float pen = 0.0f;
    if constexpr (CP) {
        const int col = bt * kTileN + n;
        const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
        n_valid = len - a.I - a.H + 1;
        pen = a.two_lambda_cs * a.sc->inv_n_cs;
    }
    // factors of step A that do not depend on the recurrent gradient, as two quads:
    // dc = dcreg + (gs + dhreg) ad + pc;  da = (dc ki, dc kf, dc kg, (gs + dhreg) ko);  dcreg = dc f
    auto factors = [&](int set, int j, int p, f32x4 (&f)[2]) {
        const f32x4 v = gt[set][j];                        // input, forget, candidate, output gate
        const float tc = tanh_f(ccur[j]), cp = p >= a.d ? cnext[set][j] : 0.0f;
        f[0] = f32x4{v[0] * v[2] * (1.0f - v[0]), v[1] * cp * (1.0f - v[1]), v[0] * (1.0f - v[2] * v[2]),
                     v[3] * tc * (1.0f - v[3])};           // ki, kf, kg, ko
        f[1] = f32x4{own_register(ga[set][j]) + g2_scale * gb[set][j], v[3] * (1.0f - tc * tc), own_register(v[1]),
                     CP && p < n_valid ? pen * ccur[j] : 0.0f};   // gs, ad, f, pc
        ccur[j] = own_register(cnext[set][j]);
    };

    if (wv < NC) {
        // =========================== chain waves ===========================
        const int s = wv;
        auto chains = [&](auto njc) {
            // NJ unit tiles: 2 s and 2 s + 1, whose products take whole groups of four pairs, and 2 NC + s, a rest of two pairs
            constexpr int NJ = decltype(njc)::value, NP = NJ < 2 ? NJ : 2;
            constexpr std::integral_constant<int, NP> np;
            auto tile_of = [&](int j) { return j < 2 ? 2 * s + j : 2 * NC + s; };
            u32x4 w[RH][3], w3[RH][2];
#pragma unroll
            for (int mb = 0; mb < RH; ++mb) {
                const u32x2 *src = a.wpack + ((size_t)RX + mb) * HTE * 3 * 64 + lane;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const u32x2 w0 = src[(2 * s * 3 + q) * 64], w1 = src[((2 * s + 1) * 3 + q) * 64];
                    w[mb][q] = u32x4{w0[0], w0[1], w1[0], w1[1]};
                }
                if constexpr (NJ > 2) {
                    const u32x2 *t = src + (2 * NC + s) * 3 * 64;
                    const u32x2 hi = t[0], mid = t[64], lo = t[128];
                    w3[mb][0] = u32x4{hi[0], hi[1], mid[0], mid[1]};
                    w3[mb][1] = u32x4{hi[0], hi[1], lo[0], lo[1]};
                }
            }
#pragma unroll
            for (int mb = 0; mb < RH; ++mb) {
#pragma unroll
                for (int q = 0; q < 3; ++q) arrived(w[mb][q]);
                if constexpr (NJ > 2) { arrived(w3[mb][0]); arrived(w3[mb][1]); }
            }
            float dhreg[NJ], dcreg[NJ], db[NJ][4];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                dhreg[j] = dcreg[j] = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) db[j][r] = 0.0f;
            }
            f32x4 f[NJ][2];
            // at[i]: the position i steps from now.  Without factor waves the walk is D + 2 positions ahead, and `ask` is
            // the next tile to request; its successor is the walk's.
            constexpr int AT = NF > 0 ? 2 : D + 2;
            ChainWalk walk = start;
            int at[AT];
            unsigned ask = walk.tile();
            if constexpr (NF > 0) {
                at[0] = walk.p;
                walk.next();
                at[1] = walk.p;
                if (n_steps > 0) {
                    lds_barrier();                         // factors of the first two positions complete
#pragma unroll
                    for (int j = 0; j < NJ; ++j) { f[j][0] = factor_lds[0][tile_of(j)][0][lane]; f[j][1] = factor_lds[0][tile_of(j)][1][lane]; }
                    lds_barrier();                         // taken: the factor waves' next position goes to the same half
                }
            } else if (n_steps > 0) {
                request_first_c(2 * s, np, ask);
#pragma unroll
                for (int i = 0; i <= D; ++i) {
                    at[i] = walk.p;
                    walk.next();
                    if (i == D) {
#pragma unroll
                        for (int j = 0; j < NP; ++j) factors(0, j, at[0], f[j]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    request(i % D, 2 * s, np, ask, walk.tile());
                    ask = walk.tile();
                    __builtin_amdgcn_sched_barrier(0);
                }
                at[D + 1] = walk.p;
            }
            alternate(n_steps, [&](auto u) {
                constexpr int U = decltype(u)::value;
                // A: gate gradients, their parts to LDS and into the operand of B
                float da[NJ][4];
                unsigned parts[NJ][3][2];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const float dh = f[j][1][0] + dhreg[j];
                    float dc = dcreg[j] + dh * f[j][1][1];
                    if constexpr (CP) dc += f[j][1][3];
#pragma unroll
                    for (int r = 0; r < 3; ++r) da[j][r] = dc * f[j][0][r];
                    da[j][3] = dh * f[j][0][3];
                    dcreg[j] = dc * f[j][1][2];
                    const Parts p0 = split_pair<true>(da[j][0], da[j][1]), p1 = split_pair<true>(da[j][2], da[j][3]);
#pragma unroll
                    for (int q = 0; q < 3; ++q) { parts[j][q][0] = part_of(p0, q); parts[j][q][1] = part_of(p1, q); }
#pragma unroll
                    for (int r = 0; r < 4; ++r) db[j][r] += da[j][r];
                }
                // (The scheduler sees one position at a time.  Left alone it moves the uses of what was requested two
                // positions ago to the top of a position, and requests in between the uses of the registers they
                // fill, which then are copied at the end: both wait for requests that have just gone out.)
                __builtin_amdgcn_sched_barrier(0);
                // B: the h rows (and merged x rows), this wave's share of the contraction
                f32x4 acc[RH];
#pragma unroll
                for (int mb = 0; mb < RH; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                u32x4 b[3];
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    b[q] = u32x4{parts[0][q][0], parts[0][q][1], NP > 1 ? parts[NP - 1][q][0] : 0u, NP > 1 ? parts[NP - 1][q][1] : 0u};
                auto pairs = [&](auto from, auto to) {
                    static_for<decltype(from)::value, decltype(to)::value>([&](auto ic) {
                        constexpr TtPair t = tt_group_rising(decltype(ic)::value);
#pragma unroll
                        for (int mb = 0; mb < RH; ++mb) acc[mb] = mfma_bf16(w[mb][t.a], b[t.b], acc[mb]);
                    });
                };
                auto third = [&](int k) {                  // (hi, lo) (lo, hi);  (hi, mid) mid;  (hi, mid) hi
                    if constexpr (NJ > 2) {
                        const unsigned (&p)[3][2] = parts[NJ - 1];
                        const int q0 = 2 - k, q1 = k == 1 ? 1 : 0;
                        const u32x4 bb = u32x4{p[q0][0], p[q0][1], p[q1][0], p[q1][1]};
#pragma unroll
                        for (int mb = 0; mb < RH; ++mb) acc[mb] = mfma_bf16(w3[mb][k == 0], bb, acc[mb]);
                    }
                };
                // Largest terms first: an accumulator smaller than the sum it receives loses its low bits downwards
                // (three_term.h), and a bias of dh adds up over positions and series.
                pairs(std::integral_constant<int, 5>{}, std::integral_constant<int, 6>{});
                third(2);
                pairs(std::integral_constant<int, 0>{}, std::integral_constant<int, 5>{});
                third(1);
                third(0);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        *reinterpret_cast<u32x2 *>(da_lds[U] + da_at(tile_of(j), q) + own) = u32x2{parts[j][q][0], parts[j][q][1]};
                }
                const bool last_of_chain = at[0] < a.d;
                if constexpr (NF > 0) {
                    __builtin_amdgcn_sched_barrier(0);     // (the factors take the registers of the operands)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) { f[j][0] = factor_lds[U ^ 1][tile_of(j)][0][lane]; f[j][1] = factor_lds[U ^ 1][tile_of(j)][1][lane]; }
                    walk.next();
                    at[0] = at[1];
                    at[1] = walk.p;
                } else {
                    constexpr int set = (U + 1) % D;
#pragma unroll
                    for (int j = 0; j < NP; ++j) factors(set, j, at[1], f[j]);
                    walk.next();
#pragma unroll
                    for (int i = 0; i <= D; ++i) at[i] = at[i + 1];
                    at[D + 1] = walk.p;
                    __builtin_amdgcn_sched_barrier(0);
                    request(set, 2 * s, np, ask, walk.tile());
                    ask = walk.tile();
                }
#pragma unroll
                for (int mb = 0; mb < RH; ++mb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * mb + r < HM) part_lds[U][s][4 * mb + r][lane] = acc[mb][r];
                lds_barrier();          // da, [x ; h] and partial results of the position complete
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float t = part_lds[U][0][tile_of(j)][lane];
#pragma unroll
                    for (int i = 1; i < NC; ++i) t += part_lds[U][i][tile_of(j)][lane];
                    dhreg[j] = last_of_chain ? 0.0f : t;
                    dcreg[j] = last_of_chain ? 0.0f : dcreg[j];
                }
            });
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float tot = group16_sum(db[j][r]);
                    if (n == 0) a.db_partial[(part * HT + tile_of(j)) * 16 + g * 4 + r] = tot;
                }
        };
        if (HT > 2 * NC && s < HT - 2 * NC) chains(std::integral_constant<int, (HT > 2 * NC ? 3 : 2)>{});
        else if (kTail && s == NC - 1) chains(std::integral_constant<int, 1>{});
        else chains(std::integral_constant<int, 2>{});
    } else if (wv < NC + NW) {
        // =========================== dW waves ===========================
        const int s = wv - NC;                             // rows 2 s, 2 s + 1 of dW tiles
        f32x4 dw[2][MB], dwt[XC];
#pragma unroll
        for (int i = 0; i < MB; ++i) dw[0][i] = dw[1][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < XC; ++i) dwt[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        // Operand of one instruction: the lane groups 0 and 1 give series 0 .. 7 and 8 .. 15 of one part, the groups
        // 2 and 3 of another; a lane's eight series are two transpose loads, 32 bytes apart.
        const int tr = ((n & 3) * 16 + 8 * (g & 1) + (n >> 2)) * 8 + 32 * ((n & 3) >> 1);
        const int hl = tr + (g >= 2 ? 4 * kPartBytes : 0);                   // (hi | lo) of da
        const int hm = tr + (g >= 2 ? kPartBytes : 0);                       // (hi | mid) of [x ; h]
        const int lh = tr + (g >= 2 ? 0 : 2 * kPartBytes);                   // (lo | hi) of [x ; h]
        auto quad = [&](const char *at) {
            const u32x2 v0 = lds_read_transposed(at), v1 = lds_read_transposed(at + 32);
            return u32x4{v0[0], v0[1], v1[0], v1[1]};
        };
        auto work = [&](int buf, unsigned, auto &&aside) {
            auto read_row = [&](int row, u32x4 (&v)[3]) {  // (hi | hi), (mid | mid), (hi | lo) of da
                const char *base = da_lds[buf] + da_at(row, 0);
                v[0] = quad(base + tr);
                v[1] = quad(base + tr + 2 * kPartBytes);
                v[2] = quad(base + hl);
            };
            u32x4 ar[2][3], xb[2][2];                      // (hi | mid), (lo | hi) of [x ; h], one column tile ahead
            auto read_column = [&](int nb) {
                const char *base = xh_lds[buf] + nb * 3 * kPartBytes;
                xb[nb & 1][0] = quad(base + hm);
                xb[nb & 1][1] = quad(base + lh);
            };
            if constexpr (kReadAhead) read_column(0);
            read_row(2 * s, ar[0]);
            read_row(2 * s + 1, ar[1]);
            aside();
            static_for<0, MB>([&](auto nbc) {
                constexpr int nb = decltype(nbc)::value;
                if constexpr (!kReadAhead) read_column(nb);
                else if constexpr (nb + 1 < MB) read_column(nb + 1);
                const u32x4 (&x)[2] = xb[nb & 1];
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int j = 0; j < 2; ++j) dw[j][nb] = mfma_bf16(ar[j][k], x[k == 2], dw[j][nb]);
                if constexpr (kTail)
                    if (nb % NW == s) {
                        u32x4 at[3];
                        read_row(HT - 1, at);
#pragma unroll
                        for (int k = 0; k < 3; ++k) dwt[nb / NW] = mfma_bf16(at[k], x[k == 2], dwt[nb / NW]);
                    }
                if constexpr (kReadAhead) __builtin_amdgcn_sched_barrier(0);   // (or the reads end up right before their uses)
            });
        };
        if (s < MB) consumer(std::true_type{}, s, work);
        else consumer(std::false_type{}, 0, work);
        // Row 4 u + gate of a result is unit u, its column 4 k + e is unit k of [x ; h] tile e; the reduction wants
        // component = unit, lane = 16 gate + (4 e + k).
        const int at = g * 64 + 4 * (n & 3) + (n >> 2);
        auto put = [&](int row, int nb, const f32x4 &v) {
            float *dst = a.dw_partial + (part * (HT * MB) + row * MB + nb) * 256 + at;
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[16 * r] = v[r];
        };
#pragma unroll
        for (int nb = 0; nb < MB; ++nb) {
            put(2 * s, nb, dw[0][nb]);
            put(2 * s + 1, nb, dw[1][nb]);
            if (kTail && nb % NW == s) put(HT - 1, nb, dwt[nb / NW]);
        }
    } else if (NF > 0 && wv >= NC + NW + RX) {
        // =========================== factor waves ===========================
        // Unit tiles 2 s and 2 s + 1; the factors of a position are complete two positions ahead of the step.
        const int s = wv - NC - NW - RX;
        constexpr std::integral_constant<int, 2> two;
        ChainWalk walk = start;
        int at[3];                                         // positions whose factors come next
        unsigned ask = walk.tile();
        auto advance = [&](int set) {                      // requests `ask`, whose successor becomes the walk's position
            walk.next();
            __builtin_amdgcn_sched_barrier(0);
            request(set, 2 * s, two, ask, walk.tile());
            ask = walk.tile();
            __builtin_amdgcn_sched_barrier(0);
        };
        auto leave = [&](int buf, int set, int p) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4 f[2];
                factors(set, j, p, f);
                factor_lds[buf][2 * s + j][0][lane] = f[0];
                factor_lds[buf][2 * s + j][1][lane] = f[1];
            }
        };
        if (n_steps > 0) {
            request_first_c(2 * s, two, ask);
            const int p0 = walk.p;
            advance(0);
            const int p1 = walk.p;
            advance(1);
            at[0] = walk.p;
            leave(0, 0, p0);
            advance(0);
            at[1] = walk.p;
            leave(1, 1, p1);
            advance(1);
            at[2] = walk.p;
            lds_barrier();                                 // both complete
            lds_barrier();                                 // the first one taken by the chain waves
        }
        alternate(n_steps, [&](auto u) {
            constexpr int U = decltype(u)::value;
            leave(U, U, at[0]);
            advance(U);
            at[0] = at[1];
            at[1] = at[2];
            at[2] = walk.p;
            lds_barrier();
            __builtin_amdgcn_sched_barrier(0);
        });
    } else {
        // =========================== dx waves ===========================
        const int s = wv - NC - NW;                        // 16-row tile of x
        constexpr int NT = HTE / 2;                        // pairs of unit tiles
        u32x4 w[NT][3];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const u32x2 *src = a.wpack + (((size_t)s * HTE + 2 * t) * 3 + q) * 64 + lane;
                const u32x2 w0 = src[0], w1 = src[3 * 64];
                w[t][q] = u32x4{w0[0], w0[1], w1[0], w1[1]};
            }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 3; ++q) arrived(w[t][q]);
        // S: the wave's number, a compile-time constant so that it knows which tiles it stores
        auto role = [&](auto sc) {
            constexpr int S = decltype(sc)::value;
            auto work = [&](int buf, unsigned tile, auto &&aside) {
                // accumulators for terms of like size: small sums do not round the large one, and consecutive products do
                // not wait for each other
                f32x4 acc[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                u32x4 b[2][3];                             // one pair of unit tiles ahead
                auto read_pair = [&](int t) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const char *at = da_lds[buf] + da_at(2 * t, q) + own;
                        const u32x2 b0 = *reinterpret_cast<const u32x2 *>(at);
                        const u32x2 b1 = 2 * t + 1 < HT ? *reinterpret_cast<const u32x2 *>(at + kPartBytes) : u32x2{0u, 0u};
                        b[t & 1][q] = u32x4{b0[0], b0[1], b1[0], b1[1]};
                    }
                };
                if constexpr (kReadAhead) read_pair(0);
                aside();
                static_for<0, NT>([&](auto tc) {
                    constexpr int t = decltype(tc)::value;
                    if constexpr (!kReadAhead) read_pair(t);
                    else if constexpr (t + 1 < NT) read_pair(t + 1);
                    static_for<0, 6>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        constexpr TtPair m = tt_group_rising(i);
                        constexpr int size = i < 2 ? 0 : i < 5 ? 1 : 2;   // hi lo, lo hi; mid mid, hi mid, mid hi; hi hi
                        acc[size] = mfma_bf16(w[t][m.a], b[t & 1][m.b], acc[size]);
                    });
                    if constexpr (kReadAhead) __builtin_amdgcn_sched_barrier(0);
                });
                const f32x4 dx = acc[0] + acc[1] + acc[2];
                const buf_rsrc r_dx = make_rsrc(tile_at(a.gdst, tile, xtile));
                static_for<0, 4>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    if constexpr (4 * S + r < KXT) buf_store(r_dx, lane4, (4 * S + r) * 256, dx[r]);
                });
                static_for<0, ML>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (S == RX - 1 - i % RX) {
                        float t = 0.0f;
#pragma unroll
                        for (int k = 0; k < NC; ++k) t += part_lds[buf][k][HT + i][lane];
                        buf_store(r_dx, lane4, (4 * RX + i) * 256, t);
                    }
                });
            };
            consumer(std::integral_constant<bool, (NW + S < MB)>{}, NW + S, work);
        };
        static_for<0, RX>([&](auto sc) {
            if (s == decltype(sc)::value) role(sc);
        });
    }
}

template <int HT, int KXT>
hipError_t run_bwd(const LstmBwdArgs &a, int chains, hipStream_t st)
{
    constexpr int threads = 64 * bwd_waves(HT, KXT);
    if (a.sc) lstm_backward_kernel<HT, KXT, true><<<dim3(a.NB, chains), threads, 0, st>>>(a);
    else lstm_backward_kernel<HT, KXT, false><<<dim3(a.NB, chains), threads, 0, st>>>(a);
    return hipGetLastError();
}

inline LstmBwdArgs backward_args(const Plan &pl, int layer, const LstmBwdSources &src, const int32_t *lengths, float *ws)
{
    const LayerPlan &lp = pl.layer[layer];
    const bool cp = lp.first_in_block && pl.cfg.lambda_cs != 0.0f;
    return LstmBwdArgs{reinterpret_cast<const u32x2 *>(ws + lp.wpack_bwd), ws + lp.xsrc, ws + lp.gates, ws + lp.c,
                       ws + lp.hid, {src.g[0], src.g[1]}, src.n, ws + lp.gdst, ws + lp.dw_partial, ws + lp.db_partial,
                       pl.NB, lp.dil, reinterpret_cast<const int32_t *>(ws + pl.pmax), lengths,
                       cp ? reinterpret_cast<const Scalars *>(ws + pl.scalars) : nullptr, 2.0f * pl.cfg.lambda_cs, pl.B, pl.T,
                       pl.I, pl.H};
}

}  // namespace

}  // namespace esrnn
