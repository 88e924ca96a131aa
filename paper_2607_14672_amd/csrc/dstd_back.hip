// dstd_back.hip -- the backward contraction of a dense layer on gfx950
// (dstd_back.h with one tap per input): dL/dW and dL/dt_in of the TTFS layer
// and of the multi-spike layer.
//
// A block holds one tile of NT * 64 neurons, up to kBackWavesMax waves of TJ
// inputs each, and walks a share of the batch. Items are (sample, input spike
// f) pairs (f < F; F = 1 for the TTFS layer); a wave's TJ events of an item are
// loaded during the item before. G of the sample S ahead is written to a ring of
// 2 S LDS tables meanwhile -- from the neurons' gradient triples, or (multi-
// spike) copied from memory -- with one barrier per S samples, so that waves
// with many and with few active inputs average out. A sample's table reaches the
// last grid point at which a neuron of the tile passes gradient; inputs after
// it are skipped.
// dW: each block's sums, to grad_W or (batch split) to partial sums added in
// split order. dt_in: each tile's sums over its neurons go to a buffer of its
// own, the first of them grad_t_in itself; launches with more tiles than buffers
// add to theirs, in order, and back_sum_kernel adds the buffers in order.
// Bound: the vector ALU and, as its chains are short, waits (about half the wave
// cycles at 4 waves per SIMD). Against the kernels before it (dW with lanes =
// inputs, two G rows gathered from LDS per lane and neuron; dt_in with a weight
// row loaded and a block reduced per record), forward and backward of a layer:
// 4096 -> 4096, batch 256, M = 64, bf16 weights 3.20 -> 2.06 ms; 6000 -> 1000,
// batch 100 585 -> 406 us; 784 -> 1000, batch 128 114 -> 105 us; the
// multi-spike layer 784 x 4 -> 1000, batch 128 754 -> 347 us. dW alone of larger
// TTFS layers has back_dw_kernel: there the LDS reads bound this one.
#include "dstd_back.h"
#include "dstd_internal.h"
#include "dstd_kernels.h"
#include "dstd_profile.h"

#include <algorithm>

namespace dstd {

constexpr int kBackWavesMax = 16;
constexpr int kBackAhead = 4;  // most samples between barriers

// lanes' maximum of v
__device__ __forceinline__ int wave_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xF, 0xF, false));  // row_mirror
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// four consecutive weights, 8 (bf16) or 16 byte aligned
__device__ __forceinline__ void load4(const float *p, float (&x)[4]) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
}
__device__ __forceinline__ void load4(const uint16_t *p, float (&x)[4]) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    x[0] = __uint_as_float(v.x << 16);
    x[1] = __uint_as_float(v.x & 0xffff0000u);
    x[2] = __uint_as_float(v.y << 16);
    x[3] = __uint_as_float(v.y & 0xffff0000u);
}

struct BackArgs {
    int B, N_in, N_out, F;
    int b_per_split;
    int tile0, add;      // first tile of the launch; add to its dt_in buffers
    int ahead;           // samples between barriers
    const float *ev;     // events [B][F][5][N_in] (row as int bits, L, R, dL, dR)
    const float *g;      // triples [B][3][N_out], or G [B][M + 1][N_out]
    const void *W;
    float *dt_in, *P;    // dt_in buffer of the launch's tile 0, and of tile t + 1 at P + t n
    float *dW;           // grad_W or partial sums [nsplit][N_out][N_in]
    const float *dq;     // dead-neuron term per neuron, added to dW (one split), or NULL
    bool vec, w_vec;     // dW rows are 16-byte, W rows four elements aligned
};

template <typename WT, int NT, int TJ, bool DW, bool DT, bool MEMG>
__global__ __launch_bounds__(kBackWavesMax * kWave) void back_dense_kernel(LifConst C, BackArgs a) {
    constexpr int kG = TJ / kBackGroup;
    constexpr int kRow = NT * kWave;
    extern __shared__ float gs[];  // G [2 S][R][kRow], pairs (a_d, k_d)
    const int R = rows_of(C);
    const int ts = R * kRow;
    const int S = a.ahead;
    float2 *tab = reinterpret_cast<float2 *>(gs + 2 * S * ts);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int nw = static_cast<int>(blockDim.x) >> 6;
    const int tile = a.tile0 + static_cast<int>(blockIdx.y);
    const int j0 = (static_cast<int>(blockIdx.x) * nw + wave) * TJ;
    const int nj = max(0, min(TJ, a.N_in - j0));
    const int i0 = tile * kRow + NT * lane;  // this lane's neurons i0 .. i0 + NT - 1
    const int b0 = static_cast<int>(blockIdx.z) * a.b_per_split;
    const int b1 = min(a.B, b0 + a.b_per_split);
    // rows 0 and R - 1 hold no grid point (R - 1 is also a triple's table's last
    // row: written after a barrier)
    for (int k = threadIdx.x; k < 2 * S * kRow; k += blockDim.x) {
        float *t = gs + (k / kRow) * ts + k % kRow;
        t[0] = 0.f;
        t[(R - 1) * kRow] = 0.f;
    }
    if constexpr (MEMG) __syncthreads();
    else g_table_fill(C, tab);
    float acc[kG][kBackGroup][1][NT], w[kG][kBackGroup][1][NT];
    static_for<TJ>([&](auto j) {
        static_for<NT>([&](auto c) {
            acc[j / kBackGroup][j % kBackGroup][0][c] = 0.f;
            w[j / kBackGroup][j % kBackGroup][0][c] = 0.f;
        });
    });
    if constexpr (DT) {
        const WT *wp = static_cast<const WT *>(a.W);
        static_for<NT>([&](auto c) {
            if (i0 + c >= a.N_out) return;
            const WT *row = wp + static_cast<int64_t>(i0 + c) * a.N_in + j0;
            if (a.w_vec && nj == TJ) {
                static_for<TJ / 4>([&](auto k) {
                    float x[4];
                    load4(row + 4 * k, x);
                    static_for<4>([&](auto u) {
                        constexpr int jj = 4 * k + u;
                        w[jj / kBackGroup][jj % kBackGroup][0][c] = x[u];
                    });
                });
            } else {
                static_for<TJ>([&](auto j) {
                    if (j < nj) w[j / kBackGroup][j % kBackGroup][0][c] = WLoad<WT>::get(row, j);
                });
            }
        });
    }
    // this lane's neurons: offsets clamped into the tile, neurons past N_out
    // without gradient
    unsigned no[NT];
    bool nok[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        no[c] = static_cast<unsigned>(min(i0 + c, a.N_out - 1));
        nok[c] = i0 + c < a.N_out;
    }
    auto load_tri = [&](int b) {
        const float *p = a.g + static_cast<int64_t>(min(b, a.B - 1)) * 3 * a.N_out;
        GTri<NT> t;
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            t.gK[c] = p[no[c]];
            t.gE[c] = (p + a.N_out)[no[c]];
            t.q[c] = __float_as_int((p + 2 * a.N_out)[no[c]]);
        }
        return t;
    };
    // the table of sample b; returns the last event row that meets gradient
    auto write_tri = [&](GTri<NT> t, int slot) {
        int qm = -1;
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            t.gK[c] = nok[c] ? t.gK[c] : 0.f;
            t.gE[c] = nok[c] ? t.gE[c] : 0.f;
            t.q[c] = nok[c] ? t.q[c] : -1;
            qm = max(qm, t.q[c]);
        }
        const int top = min(R - 2, wave_max(qm) + 1);
        if (top <= 0) return -1;
        g_rows<NT>(C.M, tab, t, top, wave, nw, gs + slot * ts + NT * lane);
        return top;
    };
    auto write_mem = [&](int b, int slot) {
        const float *p = a.g + static_cast<int64_t>(b) * (C.M + 1) * a.N_out;
        float *gl = gs + slot * ts + NT * lane;
        constexpr int kU = 16 / NT;  // rows in flight: a one-sample block waits for little else
        for (int r0 = 1 + wave; r0 <= C.M + 1; r0 += kU * nw) {
            float v[kU][NT];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if (r0 + u * nw > C.M + 1) break;
                const float *q = p + static_cast<int64_t>(r0 + u * nw - 1) * a.N_out;
#pragma unroll
                for (int c = 0; c < NT; ++c) v[u][c] = q[no[c]];
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if (r0 + u * nw > C.M + 1) break;
#pragma unroll
                for (int c = 0; c < NT; ++c) v[u][c] = nok[c] ? v[u][c] : 0.f;
                lds_put<NT>(gl + (r0 + u * nw) * kRow, v[u]);
            }
        }
        return R - 2;
    };
    const EvOffs<TJ> ev_o = ev_offs<TJ>(a.N_in, max(nj, 1), lane);
    auto item_ev = [&](int b, int d) {
        return ev_load<TJ>(a.ev + (static_cast<int64_t>(min(b, a.B - 1)) * a.F + d) * kEvFields * a.N_in +
                               (nj > 0 ? j0 : 0), ev_o);
    };
    // lane 8j + h of a dt_in store holds input 8h + j of the wave
    const int p_off = (lane & 7) < kG ? 4 * a.F * ((lane & 7) * kBackGroup + (lane >> 3)) : 1 << 30;
    float *p_buf = blockIdx.y == 0 ? a.dt_in
                                   : a.P + static_cast<int64_t>(blockIdx.y - 1) * a.B * a.N_in * a.F;
    if (b0 < b1) {
        // sample b's table is in slot (b - b0) % (2 S); r[k]: r_end of sample b + k
        int b = b0, d = 0, r[kBackAhead];
        EvRegs<TJ> ev[2];
        ev[0] = item_ev(b0, 0);
#pragma unroll
        for (int k = 0; k < kBackAhead; ++k) {
            r[k] = -1;
            if (k < S && b0 + k < b1) {
                if constexpr (MEMG) r[k] = write_mem(b0 + k, k);
                else r[k] = write_tri(load_tri(b0 + k), k);
            }
        }
        // the weights are here before the loop (its waits count its own loads), but
        // only now: they were on their way together with the first tables
        if constexpr (DT)
            static_for<TJ>([&](auto j) {
                static_for<NT>([&](auto c) { settle(w[j / kBackGroup][j % kBackGroup][0][c]); });
            });
        __syncthreads();
        int slot = 0;
        bool more = true;
        auto item = [&](auto par) {
            constexpr int p = par;
            const bool last_d = d + 1 == a.F;
            ev[p ^ 1] = item_ev(last_d ? b + 1 : b, last_d ? 0 : d + 1);
            GTri<NT> t_n;
            if constexpr (!MEMG) t_n = load_tri(b + S);
            float tot[kG];
            static_for<kG>([&](auto h) { tot[h] = 0.f; });
            if (r[0] >= 0) {
                const float *gl[1] = {gs + slot * ts + NT * lane};
                const unsigned act = static_cast<unsigned>(__ballot(
                    lane < nj && static_cast<unsigned>(__float_as_int(ev[p].e[0])) <= static_cast<unsigned>(r[0])));
                static_for<kG>([&](auto h) {
                    if ((act >> (h * kBackGroup)) & 0xffu)
                        tot[h] = back_group<NT, 1, TJ, h, DW, DT>(gl, lane, act, ev[p], w[h], acc[h]);
                });
            }
            if constexpr (DT) {
                float v = tot[0];
                static_for<kG>([&](auto x) { v = ((lane & 7) == x) ? tot[x] : v; });
                float *out = p_buf + (static_cast<int64_t>(b) * a.N_in + (nj > 0 ? j0 : 0)) * a.F + d;
                const __amdgpu_buffer_rsrc_t pr =
                    make_rsrc(out, nj > 0 ? static_cast<uint32_t>((nj - 1) * a.F + 1) * 4u : 0u);
                if (a.add) v += BufLoad<float>::get(pr, p_off, 0);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), pr, p_off, 0, 0);
            }
            ++d;
            if (last_d) {
                int rn = -1;
                if (b + S < b1) {
                    const int sn = slot + S < 2 * S ? slot + S : slot - S;
                    if constexpr (MEMG) rn = write_mem(b + S, sn);
                    else rn = write_tri(t_n, sn);
                }
#pragma unroll
                for (int k = 0; k < kBackAhead; ++k)
                    r[k] = k + 1 < S ? r[min(k + 1, kBackAhead - 1)] : rn;
                ++b;
                d = 0;
                more = b < b1;
                slot = slot + 1 < 2 * S ? slot + 1 : 0;
                if (slot == 0 || slot == S) __syncthreads();
            }
        };
        while (true) {
            item(std::integral_constant<int, 0>{});
            if (!more) break;
            item(std::integral_constant<int, 1>{});
            if (!more) break;
        }
    }
    if constexpr (DW) {
        float *out = a.dW + static_cast<int64_t>(blockIdx.z) * a.N_out * a.N_in + j0;
        const bool vec = a.vec && nj == TJ;
        static_for<NT>([&](auto c) {
            if (!nok[c]) return;
            float *o = out + static_cast<int64_t>(i0 + c) * a.N_in;
            const float q = a.dq ? a.dq[i0 + c] : 0.f;
            auto at = [&](auto jj) {
                const float x = acc[jj / kBackGroup][jj % kBackGroup][0][c];
                return a.dq ? x + q : x;
            };
            if (vec) {
                static_for<TJ / 4>([&](auto k) {
                    constexpr int x = 4 * k;
                    reinterpret_cast<float4 *>(o)[k] =
                        make_float4(at(std::integral_constant<int, x>{}), at(std::integral_constant<int, x + 1>{}),
                                    at(std::integral_constant<int, x + 2>{}), at(std::integral_constant<int, x + 3>{}));
                });
            } else {
                static_for<TJ>([&](auto jj) {
                    if (jj < nj) o[jj] = at(jj);
                });
            }
        });
    }
}

// dW alone with lanes = inputs: a block takes 256 * IPT inputs and 64 neurons,
// a thread IPT inputs and all the tile's sums. Against the kernel above, whose
// two LDS reads per input and lane are covered by the dt_in products only if
// there are any: a thread reads four neurons of a row at a time, and lanes whose
// inputs have the same event row read the same words at once (few intervals:
// most of them). G of the next sample goes to the other of two tables meanwhile.
// Same sums in the same order. Bound: LDS reads.
constexpr int kDwIn = 256;
constexpr int kDwRow = kWave + 4;  // a row's floats: 16-byte reads, neighbouring rows 4 banks apart
template <int IPT>
__global__ __launch_bounds__(kDwIn) void back_dw_kernel(LifConst C, BackArgs a) {
    extern __shared__ float gs[];  // G [2][R + 1][kDwRow], pairs (a_d, k_d)
    const int R = rows_of(C);
    const int ts = (R + 1) * kDwRow;
    float2 *tab = reinterpret_cast<float2 *>(gs + 2 * ts);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int jb = static_cast<int>(blockIdx.x) * kDwIn * IPT + static_cast<int>(threadIdx.x);
    const int i0 = static_cast<int>(blockIdx.y) * kWave;
    const int b0 = static_cast<int>(blockIdx.z) * a.b_per_split;
    const int b1 = min(a.B, b0 + a.b_per_split);
    // row 0 holds no grid point; rows R - 1 and R are zero for inputs without
    // events (or past the last spike)
    for (int k = threadIdx.x; k < 2 * kDwRow; k += kDwIn) {
        float *t = gs + (k / kDwRow) * ts + k % kDwRow;
        t[0] = 0.f;
        t[(R - 1) * kDwRow] = 0.f;
        t[R * kDwRow] = 0.f;
    }
    g_table_fill(C, tab);
    float acc[IPT][kWave];
#pragma unroll
    for (int k = 0; k < IPT; ++k)
#pragma unroll
        for (int i = 0; i < kWave; ++i) acc[k][i] = 0.f;
    const unsigned no = static_cast<unsigned>(min(i0 + lane, a.N_out - 1));
    const bool nok = i0 + lane < a.N_out;
    auto load_tri = [&](int b) {
        const float *p = a.g + static_cast<int64_t>(min(b, a.B - 1)) * 3 * a.N_out;
        GTri<1> t;
        t.gK[0] = p[no];
        t.gE[0] = (p + a.N_out)[no];
        t.q[0] = __float_as_int((p + 2 * a.N_out)[no]);
        return t;
    };
    auto write_tri = [&](GTri<1> t, int slot) {
        t.gK[0] = nok ? t.gK[0] : 0.f;
        t.gE[0] = nok ? t.gE[0] : 0.f;
        t.q[0] = nok ? t.q[0] : -1;
        const int top = min(R - 2, wave_max(t.q[0]) + 1);
        if (top <= 0) return -1;
        g_rows<1, kDwRow>(C.M, tab, t, top, wave, kDwIn / kWave, gs + slot * ts + lane);
        return top;
    };
    struct Ev { int row[IPT]; float L[IPT], R[IPT]; };
    auto load_ev = [&](int b) {
        const float *p = a.ev + static_cast<int64_t>(min(b, a.B - 1)) * kEvFields * a.N_in;
        Ev e;
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            const unsigned j = static_cast<unsigned>(min(jb + k * kDwIn, a.N_in - 1));
            e.row[k] = __float_as_int(p[j]);
            e.L[k] = (p + a.N_in)[j];
            e.R[k] = (p + 2 * static_cast<int64_t>(a.N_in))[j];
        }
        return e;
    };
    if (b0 < b1) {
        Ev ev = load_ev(b0);
        int top = write_tri(load_tri(b0), 0);
        GTri<1> tri = load_tri(b0 + 1);
        __syncthreads();
        for (int b = b0; b < b1; ++b) {
            const Ev next = load_ev(b + 1);
            const int cur = (b - b0) & 1;
            int top_n = -1;
            if (b + 1 < b1) top_n = write_tri(tri, cur ^ 1);
            tri = load_tri(b + 2);
            if (top >= 0) {
#pragma unroll
                for (int k = 0; k < IPT; ++k) {
                    const bool on = static_cast<unsigned>(ev.row[k]) <= static_cast<unsigned>(top);
                    const float L = on ? ev.L[k] : 0.f, Rv = on ? ev.R[k] : 0.f;
                    const float4 *p = reinterpret_cast<const float4 *>(gs + cur * ts + (on ? ev.row[k] : R - 1) * kDwRow);
#pragma unroll
                    for (int i = 0; i < kWave; i += 4) {
                        const float4 x = p[i / 4], y = p[(i + kDwRow) / 4];
                        acc[k][i] = fmaf(L, x.x, fmaf(Rv, y.x, acc[k][i]));
                        acc[k][i + 1] = fmaf(L, x.y, fmaf(Rv, y.y, acc[k][i + 1]));
                        acc[k][i + 2] = fmaf(L, x.z, fmaf(Rv, y.z, acc[k][i + 2]));
                        acc[k][i + 3] = fmaf(L, x.w, fmaf(Rv, y.w, acc[k][i + 3]));
                    }
                }
            }
            ev = next;
            top = top_n;
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
        const int j = jb + k * kDwIn;
        if (j >= a.N_in) continue;
        float *o = a.dW + (static_cast<int64_t>(blockIdx.z) * a.N_out + i0) * a.N_in + j;
#pragma unroll
        for (int i = 0; i < kWave; ++i)
            if (i0 + i < a.N_out)
                o[static_cast<int64_t>(i) * a.N_in] = a.dq ? acc[k][i] + a.dq[i0 + i] : acc[k][i];
    }
}

// Sums in order, four outputs per thread (one 16-byte load per summand where
// they are aligned to it), eight summands in flight: what bounds a small layer's
// many partial sums is the chain of their loads.
// blocks [0, n_dw) add the dW partial sums (+ the row's dead-neuron term), the
// rest the dt_in buffers.
struct SumJob {
    int64_t n;
    int count;
    const float *first, *rest;
    float *out;
    const float *dq;
    int row_len;
    bool vec;  // every summand is 16-byte aligned, n a multiple of 4
};

template <bool VEC> __device__ __forceinline__ void sum4(const SumJob &s, int64_t k) {
    constexpr int kAhead = 8;
    auto load = [&](int z, float (&y)[4]) {
        const float *p = (z == 0 ? s.first : s.rest + static_cast<int64_t>(z - 1) * s.n) + k;
        if constexpr (VEC) {
            const float4 x = *reinterpret_cast<const float4 *>(p);
            y[0] = x.x; y[1] = x.y; y[2] = x.z; y[3] = x.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) y[c] = p[k + c < s.n ? c : 0];
        }
    };
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (s.count > 0) load(0, v);
    for (int z = 1; z < s.count; z += kAhead) {
        float y[kAhead][4];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (z + u < s.count) load(z + u, y[u]);
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (z + u < s.count)
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] += y[u][c];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (k + c < s.n) s.out[k + c] = s.dq ? v[c] + s.dq[(k + c) / s.row_len] : v[c];
}

__device__ __forceinline__ void sum_block(const SumJob &s, int64_t blk) {
    const int64_t k = 4 * (blk * 256 + threadIdx.x);
    if (k >= s.n) return;
    if (s.vec) sum4<true>(s, k);
    else sum4<false>(s, k);
}

__global__ __launch_bounds__(256) void back_sum_kernel(SumJob dw, int n_dw, SumJob dt) {
    const int64_t blk = blockIdx.x;
    if (blk < n_dw) sum_block(dw, blk);
    else sum_block(dt, blk - n_dw);
}

// ------------------------------------------------------------- launcher --
// The shape of a call: NT neurons per lane (2 only past 64 neurons, as far as
// their two tables fit kBackLdsDense), TJ = 8 or 16 inputs per wave, the waves
// per block, the blocks over the inputs and the batch split, by the time they
// predict. A block takes a fixed start and, per sample, its barrier, its share of
// the table's rows (copied ones: a load each) and its wave's inputs, in cycles of
// a wave alone on its CU; waves that share a CU slow each other down by kShare
// each. The last, partly filled round of blocks counts with the waves that it
// has. Partial sums are written and read once more, in order.
// The constants are a fit to 6,500 timed shapes of 143 layers, dW alone, dt_in
// alone and both: batch 4 to 256, 16 to 6000 inputs of 1 to 8 spikes, 4 to 4096
// neurons, M 8 to 250. The predicted best is 4 % above the timed best on average;
// one fixed shape (16 inputs, two neurons, at least four samples per block) was
// 54 % above it, and small layers left most of the chip idle with it:
// 400 -> 120, batch 24, M = 64, both gradients 47.5 -> 21.1 us.
constexpr int kBackLdsDense = 152 * 1024;
constexpr int kBackCUs = 256;
constexpr int kLdsBytes = 160 * 1024;

// Waves per SIMD that the kernel's registers leave (at least)
static int back_occupancy(int pairs, bool both) {
    if (both) return pairs >= 32 ? 4 : pairs >= 16 ? 5 : 8;
    return pairs >= 32 ? 5 : pairs >= 16 ? 7 : 8;
}

static int back_lds(int M, int nt, int ahead) {
    return 2 * ahead * (M + 3) * nt * kWave * 4 + g_table_len(M) * static_cast<int>(sizeof(float2));
}

// nt, b_per_split: given, or 0
static BackPlan back_search(const BackSize &z, int M, bool dw, bool dt, int nt_given, int bps_given) {
    constexpr double kStart = 3600., kStartM = 10.5, kBarrier = 1000., kRow = 52., kRowMem = 980.;
    constexpr double kPerUs = 2400., kShare = 0.053, kWide = 1.27;
    constexpr double kSumUs = 3., kSumUsPerMB = 0.68, kSumUsPerPart = 0.18;
    const double k_input = (dw && dt) ? 109. : dt ? 105. : 57.;
    const int Bn = static_cast<int>(std::max<int64_t>(z.B, 1));
    const double dw_mb = 4e-6 * static_cast<double>(z.N_in) * static_cast<double>(z.N_out);
    const double dt_mb = 4e-6 * static_cast<double>(z.B) * static_cast<double>(z.N_in * z.F);
    const int most_split = dw ? std::max(1, std::min(static_cast<int>(z.cap), Bn)) : std::min(Bn, 256);
    // (one tile needs no dt_in buffers to add up: 64 < N_out <= 128 takes NT = 2)
    const int nt_most = (z.N_out > kWave && back_lds(M, 2, 1) <= kBackLdsDense) ? 2 : 1;
    if (nt_most == 2 && z.N_out <= 2 * kWave) nt_given = 2;
    BackPlan p{};
    double best = -1.;
    for (int nt = nt_given ? nt_given : nt_most; nt >= (nt_given ? nt_given : 1); --nt) {
        const int tiles = static_cast<int>((z.N_out + nt * kWave - 1) / (nt * kWave));
        const int launches = dt ? static_cast<int>((tiles + z.n_buf) / (1 + z.n_buf)) : 1;
        const int per_launch = launches > 0 ? (tiles + launches - 1) / launches : 0;
        const int by_lds = std::max(1, kLdsBytes / back_lds(M, nt, 1));
        for (int tj = 16; tj >= 8; tj -= 8) {
            const int chunks = static_cast<int>((z.N_in + tj - 1) / tj);
            const int slots = 4 * back_occupancy(nt * tj, dw && dt);
            const double item = static_cast<double>(z.F) * tj * k_input * (nt == 2 ? kWide : 1.);
            for (const int most : {kBackWavesMax, 12, 8, 6, 4, 2}) {
                const int groups = std::max(1, (chunks + most - 1) / most);
                // (one block over the inputs: also with waves that only write table rows)
                const int even = std::max(1, (chunks + groups - 1) / groups);
                const int w = groups == 1 ? most : even;
                const int per = std::max(1, std::min(slots / w, by_lds));
                const int64_t blocks = static_cast<int64_t>(groups) * std::max(1, per_launch);
                const double sample = item + kBarrier + (z.mem_g ? kRowMem : kRow) * nt * (M + 3) / w;
                const double start = kStart + kStartM * M / w;
                for (int want = 1;; want = std::min(2 * want, most_split)) {
                    const int bps = bps_given ? bps_given : (Bn + want - 1) / want;
                    const int ns = (Bn + bps - 1) / bps;
                    const int64_t tot = blocks * ns, full = tot < kBackCUs * per ? 0 : tot / (kBackCUs * per);
                    const int64_t rest = tot - full * kBackCUs * per;
                    const double alone = start + static_cast<double>(bps) * sample;
                    double us = static_cast<double>(full) * (1. + kShare * per * w);
                    if (rest > 0) us += 1. + kShare * static_cast<double>((static_cast<int>(rest) + kBackCUs - 1) / kBackCUs) * w;
                    us *= alone * std::max(1, launches) / kPerUs;
                    if (dw && ns > 1)
                        us += kSumUs + std::max(kSumUsPerMB * static_cast<double>(ns + 1) * dw_mb,
                                                kSumUsPerPart * static_cast<double>(ns));
                    else if (dt && per_launch > 1) us += kSumUs;
                    if (dt && per_launch > 1) us += kSumUsPerMB * (per_launch + 1) * dt_mb;
                    if (best < 0. || us < best) {
                        best = us;
                        p.nt = nt;
                        p.tj = tj;
                        p.tiles = tiles;
                        p.groups = groups;
                        p.waves = w;
                        p.nsplit = ns;
                        p.b_per_split = bps;
                    }
                    if (bps_given || want >= most_split) break;
                }
            }
        }
    }
    // tables ahead as far as the CU still holds its blocks
    const int room = kBackLdsDense / std::max(1, kBackWavesMax / p.waves);
    p.ahead = 1;
    while (p.ahead < kBackAhead && back_lds(M, p.nt, 2 * p.ahead) <= room) p.ahead *= 2;
    p.lds = static_cast<size_t>(back_lds(M, p.nt, p.ahead));
    return p;
}

// One gradient alone keeps what the order of its sums depends on (dW: the batch
// split; dt_in: the neurons per lane) as both together have it, so that it comes
// out the same to the bit; that costs it 0 and 2 % of its time.
BackPlan plan_back(const BackSize &z, int M, bool dw, bool dt) {
    const BackPlan p = back_search(z, M, true, true, 0, 0);
    if (dw && dt) return p;
    return dw ? back_search(z, M, true, false, 0, p.b_per_split) : back_search(z, M, false, true, p.nt, 0);
}

// Room for partial sums and dt_in buffers by their bytes: at most 64 splits and
// 48 MiB of partials; a dt_in buffer for each 64 neurons past the first, as far
// as 32 MiB or about the weights' size (2 + N_out / B buffers) hold them.
int64_t back_split_cap(int64_t B, int64_t N_in, int64_t N_out) {
    const int64_t n = std::max<int64_t>(1, N_in * N_out);
    return std::max<int64_t>(1, std::min<int64_t>({B, 64, (int64_t{48} << 20) / (4 * n)}));
}
int64_t back_buf_cap(int64_t B, int64_t N_in, int64_t F, int64_t N_out) {
    const int64_t n = std::max<int64_t>(1, B * N_in * F);
    const int64_t most = std::max<int64_t>(2 + N_out / std::max<int64_t>(B, 1), (int64_t{32} << 20) / (4 * n));
    return std::max<int64_t>(0, std::min<int64_t>((N_out + kWave - 1) / kWave - 1, most));
}

// ---- end of the launch rules of back_dense_kernel ----

// dW alone (TTFS layer): inputs or neurons along the lanes? back_dw_kernel from
// 2.5 million pairs over the batch, 96 inputs, and as far as a CU holds two of its
// blocks (M <= 128); two inputs per thread where that still leaves two blocks per
// CU, and the table's rows are many enough to be worth sharing. back_dense_kernel
// -> back_dw_kernel, prep and sums with it:
//   4096 -> 4096, batch 256, M = 8, 32, 64, 128   891, 1010, 1105, 1418 -> 427, 593, 713, 918 us
//     (one input per thread                       427, 618, 767, 1337)
//   6000 -> 1000, batch 100 203 -> 131; 784 -> 1000, batch 128 63 -> 49 (two inputs: 55)
//   below the line: 24 x 400 -> 120 19.9 -> 21.0, 8 x 784 -> 100 18.0 -> 18.8
static size_t dw_lds(int M) {
    return 2 * static_cast<size_t>(M + 4) * kDwRow * sizeof(float) +
           static_cast<size_t>(g_table_len(M)) * sizeof(float2);
}
static bool dw_by_input(const BackJob &j, int M) {
    return !j.mem_g && M <= 128 && j.N_in >= 96 && j.B * j.N_in * j.N_out >= 2500000;
}
static int dw_ipt(const BackJob &j, int M, int nsplit) {
    const int64_t blocks = ((j.N_in + 2 * kDwIn - 1) / (2 * kDwIn)) * ((j.N_out + kWave - 1) / kWave) * nsplit;
    return (M >= 16 && blocks >= 2 * kBackCUs) ? 2 : 1;
}

hipError_t launch_back(const LifConst &C, const BackJob &j, hipStream_t st) {
    const bool dw = j.grad_W && j.N_out * j.N_in > 0;
    const bool dt = j.grad_t_in && j.B * j.N_in > 0;
    const int64_t n_dt = j.B * j.N_in * j.F;
    if (!dw && !dt) return hipSuccess;
    const BackPlan p = plan_back(BackSize{j.B, j.N_in, j.N_out, j.F, j.mem_g,
                                          back_split_cap(j.B, j.N_in, j.N_out), j.n_buf},
                                 C.M, dw, dt);
    const bool split = dw && p.nsplit > 1;
    BackArgs a{static_cast<int>(j.B), static_cast<int>(j.N_in), static_cast<int>(j.N_out),
               static_cast<int>(j.F), p.b_per_split, 0, 0, p.ahead, j.ev, j.g, j.W,
               j.grad_t_in, j.P, split ? j.part : j.grad_W, split ? nullptr : j.dq, false, false};
    auto al16 = [](const void *x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; };
    a.vec = (j.N_in & 3) == 0 && al16(a.dW);
    a.w_vec = (j.N_in & 3) == 0 && (reinterpret_cast<uintptr_t>(j.W) & (j.bf16 ? 7 : 15)) == 0;
    const int launches = dt ? (p.tiles + j.n_buf) / (1 + j.n_buf) : 1;
    const int bufs = launches > 0 ? (p.tiles + launches - 1) / launches : 0;
    if (dw && !dt && dw_by_input(j, C.M)) {
        ProfScope prof("back_dw", st);
        const int ipt = dw_ipt(j, C.M, p.nsplit);
        const dim3 grid(static_cast<unsigned>((j.N_in + kDwIn * ipt - 1) / (kDwIn * ipt)),
                        static_cast<unsigned>((j.N_out + kWave - 1) / kWave),
                        static_cast<unsigned>(p.nsplit));
        if (ipt == 2) hipLaunchKernelGGL((back_dw_kernel<2>), grid, dim3(kDwIn), dw_lds(C.M), st, C, a);
        else hipLaunchKernelGGL((back_dw_kernel<1>), grid, dim3(kDwIn), dw_lds(C.M), st, C, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    } else {
        // tiles per launch: all, or with dt_in as evenly as its buffers allow
        ProfScope prof(j.mem_g ? "ms_back" : "back_dense", st);
        for (int t = 0; t < p.tiles; t += bufs) {
            a.tile0 = t;
            a.add = dt && t > 0;
            const dim3 grid(static_cast<unsigned>(p.groups),
                            static_cast<unsigned>(std::min(bufs, p.tiles - t)),
                            static_cast<unsigned>(p.nsplit));
            const dim3 block(static_cast<unsigned>(p.waves * kWave));
#define BD(WTY, NTV, TJV, DWV, DTV, MG)                                                          \
    hipLaunchKernelGGL((back_dense_kernel<WTY, NTV, TJV, DWV, DTV, MG>), grid, block, p.lds, st, C, a)
#define BD_M(WTY, NTV, TJV, MG)                               \
    do {                                                      \
        if (dw && dt) BD(WTY, NTV, TJV, true, true, MG);      \
        else if (dw) BD(float, NTV, TJV, true, false, MG);    \
        else BD(WTY, NTV, TJV, false, true, MG);              \
    } while (0)
#define BD_T(WTY, NTV, MG)                       \
    do {                                         \
        if (p.tj == 16) BD_M(WTY, NTV, 16, MG);  \
        else BD_M(WTY, NTV, 8, MG);              \
    } while (0)
#define BD_N(WTY, MG)                     \
    do {                                  \
        if (p.nt == 2) BD_T(WTY, 2, MG);  \
        else BD_T(WTY, 1, MG);            \
    } while (0)
            if (j.bf16) {
                if (j.mem_g) BD_N(uint16_t, true);
                else BD_N(uint16_t, false);
            } else {
                if (j.mem_g) BD_N(float, true);
                else BD_N(float, false);
            }
#undef BD_N
#undef BD_T
#undef BD_M
#undef BD
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    const int64_t n_dw = j.N_out * j.N_in;
    const int used = bufs;
    const SumJob sw{split ? n_dw : 0, p.nsplit, j.part, j.part + n_dw, j.grad_W, j.dq,
                    static_cast<int>(j.N_in), (n_dw & 3) == 0 && al16(j.part)};
    // (no neurons: dt_in = 0)
    const SumJob sd{dt && used != 1 ? n_dt : 0, used, j.grad_t_in, j.P, j.grad_t_in, nullptr, 1,
                    (n_dt & 3) == 0 && al16(j.grad_t_in) && al16(j.P)};
    const int64_t nb_w = (sw.n + 1023) / 1024, nb_d = (sd.n + 1023) / 1024;
    if (nb_w + nb_d > 0) {
        ProfScope prof(j.mem_g ? "ms_sum" : "back_sum", st);
        hipLaunchKernelGGL(back_sum_kernel, dim3(static_cast<unsigned>(nb_w + nb_d)), dim3(256), 0, st,
                           sw, static_cast<int>(nb_w), sd);
    }
    return hipGetLastError();
}

}  // namespace dstd
