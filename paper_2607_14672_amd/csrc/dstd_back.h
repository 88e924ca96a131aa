// dstd_back.h -- the backward contraction over one sample's events (device
// code shared by the dense and conv backward passes).
//
// G[m][i] = dL/dw^_m of one sample's neurons i (dense: a batch element; conv:
// an output position of one) lives in LDS as a table of rows r = m + 1, lanes
// = neurons. A wave owns some inputs and NT neurons per lane; the dW sums and
// the weights of those pairs stay in its registers over all samples of the
// block. An input's event (row, L, R, dL, dR) is the same for every lane: a
// few vector loads bring a wave's events, an item ahead, with 16 lanes = inputs
// of one field; an active input's fields are row_newbcast operands of the
// instructions that use them (read into scalars first, an input took five more
// instructions: 5 % of the whole pass at 4096 -> 4096).
//   - An input without events, or whose row lies past the last spike that
//     passes gradient, costs one scalar branch (the causal half of the pairs
//     and the silent inputs are never multiplied);
//   - its two G rows are one conflict-free two-address LDS read;
//   - dW takes 2 and dt_in 3 multiply-adds per lane, neuron and tap from those
//     reads, and no weight is loaded again. (dt_in's dL G[r-1] + dR G[r] nearly
//     cancels where dt is small: formed per neuron, before the weight. Summing
//     w G[r-1] and w G[r] apart over a lane's pairs, one multiply-add less for
//     three taps, rounds two to three times as often at that size.)
//   - dt_in's sum over the lanes is taken once per input, for all its taps.
// What bounds it is the vector ALU.
#pragma once

#include "dstd_internal.h"

#include <utility>

namespace dstd {

// Rows of one neuron's G from its triple (gK, gE, q) = (gamma K(t - T_q),
// gamma e^{-(t - T_q)/ti}, q): with d = q - m >= 0,
//   G[m] = gamma K(t - T_q + d dt) = a_d gK + k_d gE,
// a_d = e^{-d dt/tv}, k_d = K(d dt) (terms of one sign: no cancellation).
// The pairs (a_d, k_d) are tabulated in LDS for d = -(M+2) .. M, zero for
// d < 0, once per block.
__host__ __device__ __forceinline__ int g_table_len(int M) { return 2 * M + 4; }

// Every thread of the block calls it: the entries are shared out over the
// threads and any wave reads all of them, so it ends with the block barrier
// that stands between (what was written to LDS before the call is seen after it
// too).
__device__ __forceinline__ void g_table_fill(const LifConst &C, float2 *tab) {
    for (int k = threadIdx.x; k < g_table_len(C.M); k += blockDim.x) {
        const int d = k - (C.M + 2);
        const float u = static_cast<float>(d) * C.dt;
        tab[k] = (d >= 0) ? make_float2(expf(-u * C.inv_tv), kern(C, u)) : make_float2(0.f, 0.f);
    }
    __syncthreads();
}

struct GradTriple { float gK, gE; int q; };

// q <= M also where the caller's interval index is not (the table has no entry
// past it): such a neuron is taken to fire after the last grid point.
__device__ __forceinline__ GradTriple grad_triple(const LifConst &C, float t, float slope, int q,
                                                  float g) {
    const GradPrep p = grad_prep(C, t, slope, min(q, C.M), g);
    if (p.q < 0) return GradTriple{0.f, 0.f, -1};
    return GradTriple{p.gam * kern(C, p.uq), p.gam * expf(-p.uq * C.inv_ti), p.q};
}

template <int NT> struct GTri { float gK[NT], gE[NT]; int q[NT]; };

// NT consecutive floats in LDS as one read or write
template <int NT> __device__ __forceinline__ void lds_get(const float *p, float (&v)[NT]) {
    if constexpr (NT == 4) {
        const float4 x = *reinterpret_cast<const float4 *>(p);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else if constexpr (NT == 2) {
        const float2 x = *reinterpret_cast<const float2 *>(p);
        v[0] = x.x; v[1] = x.y;
    } else {
        v[0] = p[0];
    }
}
template <int NT> __device__ __forceinline__ void lds_put(float *p, const float (&v)[NT]) {
    if constexpr (NT == 4) *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    else if constexpr (NT == 2) *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    else p[0] = v[0];
}

// rows 1 .. r_end + 1 of one sample's G (row 0 is zero for good), wave w of nw
// taking rows 1 + w, 1 + w + nw, ..., four at a time (their table reads in
// flight together); gl = the table + NT * lane, its rows kRow floats apart
template <int NT, int kRow = NT * kWave>
__device__ __forceinline__ void g_rows(int M, const float2 *tab, const GTri<NT> &t, int r_end,
                                       int w, int nw, float *gl) {
    for (int r0 = 1 + w; r0 <= r_end + 1; r0 += 4 * nw) {
        float2 e[4][NT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = min(r0 + u * nw, r_end + 1);
#pragma unroll
            for (int c = 0; c < NT; ++c) e[u][c] = tab[t.q[c] + M + 3 - r];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + u * nw;
            if (r > r_end + 1) break;
            float v[NT];
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const float x = fmaf(t.gK[c], e[u][c].x, t.gE[c] * e[u][c].y);
                v[c] = (t.q[c] >= r - 1) ? x : 0.f;
            }
            lds_put<NT>(gl + r * kRow, v);
        }
    }
}

// f(0), ..., f(N - 1) with compile-time arguments: array elements named by
// them are registers from the start (a loop unrolled later had left the
// accumulators of skipped inputs behind as 8-wide vector copies).
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// x is in its register here
__device__ __forceinline__ void settle(float &x) { asm volatile("" : "+v"(x)); }

__device__ __forceinline__ void opaque(unsigned &x) { asm volatile("" : "+s"(x)); }

// A wave's events of one item: lane l of register e[h] holds x = 16 h + l % 16,
// field x / TJ (row as int bits, L, R, dL, dR) of input x % TJ, so that an
// input's field reaches every lane as the row_newbcast operand of the
// instruction that uses it.
constexpr int kBackGroup = 8;
constexpr int kEvFields = 5;
template <int TJ> constexpr int ev_regs() { return (kEvFields * TJ + 15) / 16; }
template <int TJ> struct EvRegs { float e[ev_regs<TJ>()]; };

// Offsets (floats) of a lane's events from the first input's row, the fields fs
// floats apart; lanes past the fields, or inputs past nj >= 1, take a field or
// input that exists.
template <int TJ> struct EvOffs { unsigned o[ev_regs<TJ>()]; };
template <int TJ> __device__ __forceinline__ EvOffs<TJ> ev_offs(int fs, int nj, int lane) {
    EvOffs<TJ> r;
#pragma unroll
    for (int h = 0; h < ev_regs<TJ>(); ++h) {
        const int x = h * 16 + (lane & 15);
        r.o[h] = static_cast<unsigned>(min(x / TJ, kEvFields - 1) * fs + min(x % TJ, nj - 1));
    }
    return r;
}
// p: the first input's row (scalar)
template <int TJ>
__device__ __forceinline__ EvRegs<TJ> ev_load(const float *p, const EvOffs<TJ> &o) {
    EvRegs<TJ> r;
#pragma unroll
    for (int h = 0; h < ev_regs<TJ>(); ++h) r.e[h] = p[o.o[h]];
    return r;
}
// lane N of each 16 lanes, to all of them (every lane active)
template <int N> __device__ __forceinline__ int row_bcast(int x) {
    return __builtin_amdgcn_update_dpp(0, x, 0x150 + N, 0xf, 0xf, true);  // row_newbcast:N
}
template <int TJ> constexpr int ev_reg(int f, int k) { return (f * TJ + k) / 16; }
template <int TJ> constexpr int ev_lane(int f, int k) { return (f * TJ + k) % 16; }

// acc[c] += bcast(L) x[c] + bcast(R) y[c] from lanes NL and NR of each 16, the
// broadcasts being operands of the multiply-adds (the compiler folds a row
// broadcast into a product but leaves it a move of its own before a
// multiply-add). s_nop: a register written by the vector ALU may be read as a
// row broadcast two cycles later at the earliest. (&: the sums are written
// before the last operand is read; without it an operand that starts out equal
// to a sum is given the sum's own register.)
template <int NL, int NR, int NT>
__device__ __forceinline__ void fma_bcast(float (&acc)[NT], float L, float R, const float (&x)[NT],
                                          const float (&y)[NT]) {
#define FB(d, e, s, n) "v_fmac_f32_dpp " d ", " e ", " s " row_newbcast:" n " row_mask:0xf bank_mask:0xf\n"
    if constexpr (NT == 4)
        asm("s_nop 1\n" FB("%0", "%5", "%11", "%15") FB("%1", "%5", "%12", "%15")
                FB("%2", "%5", "%13", "%15") FB("%3", "%5", "%14", "%15") FB("%0", "%4", "%7", "%6")
                    FB("%1", "%4", "%8", "%6") FB("%2", "%4", "%9", "%6") FB("%3", "%4", "%10", "%6")
            : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
            : "v"(L), "v"(R), "n"(NL), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(y[0]),
              "v"(y[1]), "v"(y[2]), "v"(y[3]), "n"(NR));
    else if constexpr (NT == 2)
        asm("s_nop 1\n" FB("%0", "%3", "%7", "%9") FB("%1", "%3", "%8", "%9") FB("%0", "%2", "%5", "%4")
                FB("%1", "%2", "%6", "%4")
            : "+&v"(acc[0]), "+&v"(acc[1])
            : "v"(L), "v"(R), "n"(NL), "v"(x[0]), "v"(x[1]), "v"(y[0]), "v"(y[1]), "n"(NR));
    else
        asm("s_nop 1\n" FB("%0", "%2", "%5", "%6") FB("%0", "%1", "%4", "%3")
            : "+&v"(acc[0])
            : "v"(L), "v"(R), "n"(NL), "v"(x[0]), "v"(y[0]), "n"(NR));
}
// v[c] = bcast(p) a[c] + bcast(q) b[c]
template <int NP, int NQ, int NT>
__device__ __forceinline__ void dot_bcast(float (&v)[NT], float p, float q, const float (&a)[NT],
                                          const float (&b)[NT]) {
#define MB(d, e, s, n) "v_mul_f32_dpp " d ", " e ", " s " row_newbcast:" n " row_mask:0xf bank_mask:0xf\n"
    if constexpr (NT == 4)
        asm("s_nop 1\n" MB("%0", "%5", "%10", "%15") MB("%1", "%5", "%11", "%15")
                MB("%2", "%5", "%12", "%15") MB("%3", "%5", "%13", "%15") FB("%0", "%4", "%6", "%14")
                    FB("%1", "%4", "%7", "%14") FB("%2", "%4", "%8", "%14") FB("%3", "%4", "%9", "%14")
            : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
            : "v"(p), "v"(q), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]),
              "v"(b[2]), "v"(b[3]), "n"(NP), "n"(NQ));
    else if constexpr (NT == 2)
        asm("s_nop 1\n" MB("%0", "%3", "%6", "%9") MB("%1", "%3", "%7", "%9") FB("%0", "%2", "%4", "%8")
                FB("%1", "%2", "%5", "%8")
            : "=&v"(v[0]), "=&v"(v[1])
            : "v"(p), "v"(q), "v"(a[0]), "v"(a[1]), "v"(b[0]), "v"(b[1]), "n"(NP), "n"(NQ));
    else
        asm("s_nop 1\n" MB("%0", "%2", "%4", "%6") FB("%0", "%1", "%3", "%5")
            : "=&v"(v[0])
            : "v"(p), "v"(q), "v"(a[0]), "v"(b[0]), "n"(NP), "n"(NQ));
#undef MB
#undef FB
}

// Inputs 8 G .. 8 G + 7 of a wave, act: bit k set where input k's row is in
// 0 .. r_end. gl[i]: the G table of tap i + NT * lane. acc += dW contributions;
// returns (dt_in) the wave's sum over its neurons and taps of input 8 G + k on
// lanes 8k .. 8k + 7. The empty asm keeps each skip a branch (selects would do
// the work anyway). kB inputs' reads are in flight before their sums.
template <int NT, int KW, int TJ, int G, bool DW, bool DT>
__device__ __forceinline__ float back_group(const float *(&gl)[KW], int lane, unsigned act,
                                            const EvRegs<TJ> &ev,
                                            const float (&w)[kBackGroup][KW][NT],
                                            float (&acc)[kBackGroup][KW][NT]) {
    constexpr int kB = (NT * KW == 1) ? 8 : (NT * KW <= 3) ? 4 : 2;
    float v[kBackGroup];
    // an input's row in the table, in bytes
    const int row_at = __float_as_int(ev.e[0]) * (NT * kWave * 4);
    static_for<kBackGroup / kB>([&](auto h) {
        float g0[kB][KW][NT], g1[kB][KW][NT];
        opaque(act);  // tested bit by bit where it is used, no masks kept
        static_for<kB>([&](auto j) {
            constexpr int k = G * kBackGroup + h * kB + j;
            if (act & (1u << k)) {
                const int o = row_bcast<k>(row_at);
                static_for<KW>([&](auto i) {
                    const float *q = reinterpret_cast<const float *>(reinterpret_cast<const char *>(gl[i]) + o);
                    lds_get<NT>(q, g0[j][i]);
                    lds_get<NT>(q + NT * kWave, g1[j][i]);
                });
                asm volatile("");
            }
        });
        opaque(act);
        static_for<kB>([&](auto j) {
            constexpr int kl = h * kB + j, k = G * kBackGroup + kl;
            v[kl] = 0.f;
            if (act & (1u << k)) {
                asm volatile("");
                static_for<KW>([&](auto i) {
                    if constexpr (DW)
                        fma_bcast<ev_lane<TJ>(1, k), ev_lane<TJ>(2, k)>(
                            acc[kl][i], ev.e[ev_reg<TJ>(1, k)], ev.e[ev_reg<TJ>(2, k)], g0[j][i], g1[j][i]);
                    if constexpr (DT) {
                        float d[NT];
                        dot_bcast<ev_lane<TJ>(3, k), ev_lane<TJ>(4, k)>(
                            d, ev.e[ev_reg<TJ>(3, k)], ev.e[ev_reg<TJ>(4, k)], g0[j][i], g1[j][i]);
                        static_for<NT>([&](auto c) {
                            v[kl] = (i == 0 && c == 0) ? w[kl][i][c] * d[c] : fmaf(w[kl][i][c], d[c], v[kl]);
                        });
                    }
                });
            }
        });
    });
    if constexpr (DT) return wave_sum8(v, lane);
    return 0.f;
}

}  // namespace dstd
