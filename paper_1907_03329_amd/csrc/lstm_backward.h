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
// Three kinds of waves, one barrier per position:
//   chain waves (two unit tiles each) carry the recurrence: A, and B for the h rows, split over the waves along the
//     contraction, so that a wave multiplies what it has just computed in registers; the partial results meet in
//     LDS and every wave sums those of its own units.  Whatever of A does not depend on the recurrent gradient is
//     formed one position ahead, so that between the barrier and the first product there are a dozen dependent
//     instructions.  They also leave the three parts of da in LDS.
//   dx waves (one 16-row tile each) do B for the x rows, which nothing in the recurrence waits for, one position
//     behind, from the parts in LDS.  If the last tile of h rows has room for the x tiles that do not fill a tile of
//     their own, the chain waves' products carry them, and a dx wave sums and stores them.
//   dW waves (two rows of tiles each) do C one position behind.  They bring [x ; h], two positions ahead; both
//     operands are needed transposed (series along the contraction) and are read with the LDS transpose load.
// Chain waves only load, dx waves only store (a dx wave brings a tile of [x ; h] where the dW waves do not suffice),
// so that no wait for a request covers a store.
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
    int P, NB, d;
    const int32_t *pmax;  // [NB] positions the longest series of a tile has: the tile's chains stop there
    // cell-state penalty (Section 8.4) of a block's first layer, kernels instantiated with CP only
    const int32_t *lengths;
    const Scalars *sc;
    float two_lambda_cs;
    int B, T, I, H;
};

// The positions of a workgroup in order: residue classes r, r + step, ..., each from its last position down.  Scalar,
// without branches.
struct ChainWalk {
    int p, r, step, d, top, top_mod, classes;
    __device__ ChainWalk(int first, int step_, int d_, int positions)
        : r(first), step(step_), d(d_), top(positions - 1), top_mod((positions - 1) % d_), classes(min(d_, positions))
    {
        p = first < classes ? last(first) : 0;
    }
    __device__ int last(int rr) const { return top - (top_mod - rr + (top_mod >= rr ? 0 : d)); }
    __device__ int count() const        // (of a walk at its start)
    {
        if (r >= classes) return 0;
        const int n = (classes - 1 - r) / step + 1, longer = r <= top_mod ? (top_mod - r) / step + 1 : 0;
        return n * (top / d) + longer;
    }
    __device__ void next()              // stays at the last one
    {
        const int r2 = r + step, below = p - d, over = r2 < classes ? last(r2) : p;
        r = below < 0 && r2 < classes ? r2 : r;
        p = below >= 0 ? below : over;
    }
};
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

constexpr int kPartBytes = 64 * 8 + 32;                    // LDS home of one part of 16 rows x 16 series

typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 lds_read_transposed(const char *at)
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at)));
}

// Workgroups are alone on their compute unit (for their registers), so the waves of one fill it: three or four per SIMD.
template <int HT, int KXT, bool CP>
__global__ void __launch_bounds__(64 * bwd_waves(HT, KXT), (bwd_waves(HT, KXT) + 3) / 4) lstm_backward_kernel(LstmBwdArgs a)
{
    constexpr int KT = KXT + HT, MB = (KT + 3) / 4;        // unit tiles and 16-column tiles of [x ; h]
    constexpr int RX = bwd_x_row_tiles(HT, KXT), RH = bwd_h_row_tiles(HT), ML = bwd_merged_tiles(HT, KXT);
    constexpr int NC = bwd_chain_waves(HT), NW = bwd_dw_waves(HT), HTE = 2 * NC;
    constexpr int HM = HT + ML;                            // unit tiles the chain waves' products give
    constexpr bool kTail = HT % 2 != 0;                    // a last row of dW tiles, dealt to the dW waves by columns
    constexpr int XC = (MB + NW - 1) / NW;                 // columns of it per wave
    constexpr int D = HT <= 10 ? 2 : 1;                    // positions the stash is requested ahead
    static_assert(MB <= NW + RX, "every column tile needs a wave that brings it");

    __shared__ __align__(16) char da_lds[2][HTE * 3 * kPartBytes];   // [pair of unit tiles][part][unit tile of the pair]
    __shared__ __align__(16) char xh_lds[2][MB * 3 * kPartBytes];
    __shared__ float part_lds[2][NC][HM][64];
    static_assert(sizeof(da_lds) + sizeof(xh_lds) + sizeof(part_lds) <= 128 * 1024, "LDS budget of the reverse kernel");

    const int lane = threadIdx.x & 63, bt = blockIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index, known to be uniform
    const int g = lane >> 4, n = lane & 15;
    const int Pt = a.pmax[bt];      // the chains of this tile stop at its longest series
    const size_t part = (size_t)bt * gridDim.y + blockIdx.y;
    constexpr size_t xtile = (size_t)KXT * 64, htile = (size_t)HT * 64;
    const unsigned lane4 = 4 * lane, lane16 = 16 * lane;
    auto da_at = [](int mt, int q) { return ((mt >> 1) * 6 + 2 * q + (mt & 1)) * kPartBytes; };
    const int own = 8 * lane + 32 * (lane >> 5);           // this lane's chunk inside a part
    const ChainWalk start(blockIdx.y, gridDim.y, a.d, Pt);
    const int n_steps = start.count();

    // ---- [x ; h] of one position, column tile nb: requested two positions ahead, split, left in LDS.
    float xraw[2][4];
    auto request_xh = [&](int set, int nb, int p) {
        const size_t pb = (size_t)p * a.NB + bt;
        const size_t pbd = (size_t)(p >= a.d ? p - a.d : p) * a.NB + bt;
        // scalar choices of a base, no branch around a request; tiles past the end alias the last one
        const char *x = reinterpret_cast<const char *>(a.xsrc + pb * xtile);
        const char *h = reinterpret_cast<const char *>(a.hid + pbd * htile) - KXT * 256;
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
        const Parts p0 = split_pair(v[0], v[1]), p1 = split_pair(v[2], v[3]);
        char *dst = xh_lds[buf] + nb * 3 * kPartBytes + own;
        *reinterpret_cast<u32x2 *>(dst) = u32x2{p0.hi, p1.hi};
        *reinterpret_cast<u32x2 *>(dst + kPartBytes) = u32x2{p0.mid, p1.mid};
        *reinterpret_cast<u32x2 *>(dst + 2 * kPartBytes) = u32x2{p0.lo, p1.lo};
    };
    // A wave that consumes what the chain waves leave: `work(buf, p)` after the barrier that completes position p.
    // LOAD: it also brings column tile nb.  Every wave of the workgroup meets the same barriers.
    auto consumer = [&](auto load, int nb, auto &&work) {
        constexpr bool LOAD = decltype(load)::value;
        if (n_steps == 0) return;
        ChainWalk now = start, bring = start, ask = start;
        if constexpr (LOAD) {
            request_xh(0, nb, ask.p);
            ask.next();
            __builtin_amdgcn_sched_barrier(0);
            request_xh(1, nb, ask.p);
            ask.next();
            store_xh(0, 0, nb, bring.p >= a.d);
            __builtin_amdgcn_sched_barrier(0);
            request_xh(0, nb, ask.p);
        }
        alternate(n_steps, [&](auto u) {
            constexpr int U = decltype(u)::value;
            lds_barrier();
            if constexpr (LOAD) {
                bring.next();
                store_xh(U ^ 1, U ^ 1, nb, bring.p >= a.d);
                __builtin_amdgcn_sched_barrier(0);
                ask.next();
                request_xh(U ^ 1, nb, ask.p);
            }
            work(U, now.p);
            now.next();
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    if (wv < NC) {
        // =========================== chain waves ===========================
        __builtin_amdgcn_s_setprio(3);
        const int s = wv;
        auto chains = [&](auto njc) {
            constexpr int NJ = decltype(njc)::value;       // unit tiles 2 s .. 2 s + NJ - 1
            u32x4 w[RH][3];
#pragma unroll
            for (int mb = 0; mb < RH; ++mb)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const u32x2 *src = a.wpack + ((((size_t)RX + mb) * HTE + 2 * s) * 3 + q) * 64 + lane;
                    const u32x2 w0 = src[0], w1 = src[3 * 64];
                    w[mb][q] = u32x4{w0[0], w0[1], w1[0], w1[1]};
                }
#pragma unroll
            for (int mb = 0; mb < RH; ++mb)
#pragma unroll
                for (int q = 0; q < 3; ++q) arrived(w[mb][q]);
            const float g2_scale = a.n_gsrc >= 2 ? 1.0f : 0.0f;
            int n_valid = 0;            // positions below this take part in the loss for this lane's series (CP only)
            float pen = 0.0f;
            if constexpr (CP) {
                const int col = bt * kTileN + n;
                const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
                n_valid = len - a.I - a.H + 1;
                pen = a.two_lambda_cs * a.sc->inv_n_cs;
            }
            // what is requested for a position: gates, arriving gradients, and the cell state of the position that
            // follows in the walk - inside a chain that is the predecessor's, which this position needs too
            f32x4 gt[D][2];
            float cnext[D][2], ga[D][2], gb[D][2], ccur[2];
            auto request = [&](int set, int p, int p_next) {
                const size_t pb = (size_t)p * a.NB + bt, pn = (size_t)p_next * a.NB + bt;
                const buf_rsrc r_g = make_rsrc(a.gates + pb * htile * 4), r_c = make_rsrc(a.c + pn * htile);
                const buf_rsrc r_a = make_rsrc(a.gsrc[0] + pb * htile), r_b = make_rsrc(a.gsrc[1] + pb * htile);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int mt = 2 * s + j;
                    gt[set][j] = buf_load4(r_g, lane16, mt * 1024);
                    cnext[set][j] = buf_load(r_c, lane4, mt * 256);
                    ga[set][j] = buf_load(r_a, lane4, mt * 256);
                    gb[set][j] = buf_load(r_b, lane4, mt * 256);
                }
            };
            // factors of a position that do not depend on the recurrent gradient:
            // dc = dcreg + dh ad + pc;  da = (dc ki, dc kf, dc kg, dh ko);  dcreg = dc f
            float gs[2], ad[2], ki[2], kf[2], kg[2], ko[2], ff[2], pc[2];
            auto factors = [&](int set, int p) {
                const bool has_prev = p >= a.d;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const f32x4 v = gt[set][j];            // input, forget, candidate, output gate
                    const float tc = tanh_f(ccur[j]), cp = has_prev ? cnext[set][j] : 0.0f;
                    gs[j] = own_register(ga[set][j]) + g2_scale * gb[set][j];
                    ad[j] = v[3] * (1.0f - tc * tc);
                    ki[j] = v[0] * v[2] * (1.0f - v[0]);
                    kf[j] = v[1] * cp * (1.0f - v[1]);
                    kg[j] = v[0] * (1.0f - v[2] * v[2]);
                    ko[j] = v[3] * tc * (1.0f - v[3]);
                    ff[j] = own_register(v[1]);
                    if constexpr (CP) pc[j] = p < n_valid ? pen * ccur[j] : 0.0f;
                    ccur[j] = own_register(cnext[set][j]);
                }
            };
            float dhreg[2] = {0.f, 0.f}, dcreg[2] = {0.f, 0.f};
            float db[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            // `now`: the position whose factors are ready; `ask`, `after`: the next one to request and its successor
            ChainWalk now = start, ask = start, after = start;
            if (n_steps > 0) {
                after.next();
                const buf_rsrc r_c = make_rsrc(a.c + ((size_t)start.p * a.NB + bt) * htile);
#pragma unroll
                for (int j = 0; j < NJ; ++j) ccur[j] = buf_load(r_c, lane4, (2 * s + j) * 256);
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    request(i, ask.p, after.p);
                    ask.next();
                    after.next();
                    __builtin_amdgcn_sched_barrier(0);
                }
                factors(0, now.p);
                __builtin_amdgcn_sched_barrier(0);
                request(0, ask.p, after.p);
                ask.next();
                after.next();
            }
            alternate(n_steps, [&](auto u) {
                constexpr int U = decltype(u)::value, set = (U + 1) % D;
                // A: gate gradients, their parts to LDS and into the operand of B
                u32x4 b[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) b[q] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const float dh = gs[j] + dhreg[j];
                    float dc = dcreg[j] + dh * ad[j];
                    if constexpr (CP) dc += pc[j];
                    const float da[4] = {dc * ki[j], dc * kf[j], dc * kg[j], dh * ko[j]};
                    dcreg[j] = dc * ff[j];
                    const Parts p0 = split_pair(da[0], da[1]), p1 = split_pair(da[2], da[3]);
                    char *dst = da_lds[U] + da_at(2 * s + j, 0) + own;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        b[q][2 * j] = part_of(p0, q);
                        b[q][2 * j + 1] = part_of(p1, q);
                        *reinterpret_cast<u32x2 *>(dst + 2 * q * kPartBytes) = u32x2{part_of(p0, q), part_of(p1, q)};
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) db[j][r] += da[r];
                }
                // (The scheduler sees one position at a time.  Left alone it moves the uses of what was requested two
                // positions ago to the top of a position, and requests in between the uses of the registers they
                // fill, which then are copied at the end: both wait for requests that have just gone out.)
                __builtin_amdgcn_sched_barrier(0);
                // B: the h rows (and merged x rows), this wave's share of the contraction
                f32x4 acc[RH];
#pragma unroll
                for (int mb = 0; mb < RH; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                static_for<0, 6>([&](auto ic) {
                    constexpr TtPair t = tt_mfma(4, decltype(ic)::value);
#pragma unroll
                    for (int mb = 0; mb < RH; ++mb) acc[mb] = mfma_bf16(w[mb][t.a], b[t.b], acc[mb]);
                });
                const bool last_of_chain = now.p < a.d;
                now.next();
                factors(set, now.p);
                __builtin_amdgcn_sched_barrier(0);
                request(set, ask.p, after.p);
                ask.next();
                after.next();
#pragma unroll
                for (int mb = 0; mb < RH; ++mb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * mb + r < HM) part_lds[U][s][4 * mb + r][lane] = acc[mb][r];
                lds_barrier();          // da, [x ; h] and partial results of the position complete
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float t = 0.0f;
#pragma unroll
                    for (int i = 0; i < NC; i += 2)
                        t += i + 1 < NC ? part_lds[U][i][2 * s + j][lane] + part_lds[U][i + 1][2 * s + j][lane]
                                        : part_lds[U][i][2 * s + j][lane];
                    dhreg[j] = last_of_chain ? 0.0f : t;
                    dcreg[j] = last_of_chain ? 0.0f : dcreg[j];
                }
            });
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float tot = group16_sum(db[j][r]);
                    if (n == 0) a.db_partial[(part * HT + 2 * s + j) * 16 + g * 4 + r] = tot;
                }
        };
        if (kTail && s == NC - 1) chains(std::integral_constant<int, 1>{});
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
        auto work = [&](int buf, int) {
            u32x4 ar[2][3];                                // (hi | hi), (mid | mid), (hi | lo) of da
            auto read_row = [&](int row, u32x4 (&v)[3]) {
                const char *base = da_lds[buf] + da_at(row, 0);
                v[0] = quad(base + tr);
                v[1] = quad(base + tr + 2 * kPartBytes);
                v[2] = quad(base + hl);
            };
            read_row(2 * s, ar[0]);
            read_row(2 * s + 1, ar[1]);
#pragma unroll
            for (int nb = 0; nb < MB; ++nb) {
                const char *base = xh_lds[buf] + nb * 3 * kPartBytes;
                const u32x4 b_hm = quad(base + hm), b_lh = quad(base + lh);
                auto product = [&](const u32x4 (&v)[3], f32x4 acc) {
                    acc = mfma_bf16(v[0], b_hm, acc);
                    acc = mfma_bf16(v[1], b_hm, acc);
                    return mfma_bf16(v[2], b_lh, acc);
                };
                dw[0][nb] = product(ar[0], dw[0][nb]);
                dw[1][nb] = product(ar[1], dw[1][nb]);
                if constexpr (kTail)
                    if (nb % NW == s) {
                        u32x4 at[3];
                        read_row(HT - 1, at);
                        dwt[nb / NW] = product(at, dwt[nb / NW]);
                    }
            }
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
    } else {
        // =========================== dx waves ===========================
        const int s = wv - NC - NW;                        // 16-row tile of x
        u32x4 w[NC][3];
#pragma unroll
        for (int t = 0; t < NC; ++t)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const u32x2 *src = a.wpack + (((size_t)s * HTE + 2 * t) * 3 + q) * 64 + lane;
                const u32x2 w0 = src[0], w1 = src[3 * 64];
                w[t][q] = u32x4{w0[0], w0[1], w1[0], w1[1]};
            }
#pragma unroll
        for (int t = 0; t < NC; ++t)
#pragma unroll
            for (int q = 0; q < 3; ++q) arrived(w[t][q]);
        // S: the wave's number, a compile-time constant so that it knows which tiles it stores
        auto role = [&](auto sc) {
            constexpr int S = decltype(sc)::value;
            auto work = [&](int buf, int p) {
                f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
                static_for<0, NC>([&](auto tc) {
                    constexpr int t = decltype(tc)::value;
                    u32x4 b[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const char *at = da_lds[buf] + da_at(2 * t, q) + own;
                        const u32x2 b0 = *reinterpret_cast<const u32x2 *>(at);
                        const u32x2 b1 = 2 * t + 1 < HT ? *reinterpret_cast<const u32x2 *>(at + kPartBytes) : u32x2{0u, 0u};
                        b[q] = u32x4{b0[0], b0[1], b1[0], b1[1]};
                    }
                    static_for<0, 6>([&](auto ic) {
                        constexpr TtPair m = tt_mfma(4, decltype(ic)::value);
                        acc[t & 1] = mfma_bf16(w[t][m.a], b[m.b], acc[t & 1]);
                    });
                });
                const f32x4 dx = acc[0] + acc[1];
                const buf_rsrc r_dx = make_rsrc(a.gdst + ((size_t)p * a.NB + bt) * xtile);
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
                       ws + lp.hid, {src.g[0], src.g[1]}, src.n, ws + lp.gdst, ws + lp.dw_partial, ws + lp.db_partial, pl.P,
                       pl.NB, lp.dil, reinterpret_cast<const int32_t *>(ws + pl.pmax), lengths,
                       cp ? reinterpret_cast<const Scalars *>(ws + pl.scalars) : nullptr, 2.0f * pl.cfg.lambda_cs, pl.B, pl.T,
                       pl.I, pl.H};
}

}  // namespace

}  // namespace esrnn
