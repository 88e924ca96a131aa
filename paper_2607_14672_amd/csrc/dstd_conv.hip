// dstd_conv.hip -- DSTD-LIF convolutional-layer kernels for gfx950.
//
// A conv layer is the dense layer of App. B.1 whose weight matrix is the
// convolution's shared, local connectivity: w^_{(c,p), m} sums w_ij s_jm over
// the receptive field of position p. Event pooling (2x2 or global) averages
// the input events before the convolution; being linear, it is folded into
// the weights (W / P) with every raw input of a pooled cell kept as its own
// event source.
//
// Input ordering used by every kernel here ("cell-major"): the (pooled) map
// has Hp x Wp cells, each with PC = P * C_in raw inputs j' = d * C_in + ci
// (d = raw pixel inside the cell). Index ((b * Hp + py) * Wp + px) * PC + j'.
//
// The inputs of one cell row (b, py) that have events are bucketed by (event
// row r, cell column px) -- a counting sort, stable in j' -- so the records
// of row r under the KW cells of an output position's kernel row form ONE
// contiguous segment, and the forward walks, per output position, the event
// rows in grid order and reads KH segments per row: lanes = output channels;
// row sums feed the interval scan as rows close (the weighted events never
// exist in memory).
// The backward needs no order: it takes the cell-major events as they are
// (dstd_back.h; conv_back_kernel for both gradients or dt_in alone, conv_dw_kernel
// for dW alone), dW summed over the (b, position) samples in splits of the output
// rows, dt_in stored as one entry per (input, kernel row, tap group, channel tile)
// and gathered in that order afterwards.
#include "dstd_back.h"
#include "dstd_internal.h"
#include "dstd_kernels.h"
#include "dstd_profile.h"

#include <algorithm>

namespace dstd {

// raw pixel (y, x) of input j' = d * C_in + ci in cell (py, px)
__device__ __forceinline__ void raw_pixel(const ConvGeom &g, int py, int px, int d, int &y,
                                          int &x) {
    if (g.pool == 2) {
        y = 2 * py + (d >> 1);
        x = 2 * px + (d & 1);
    } else if (g.pool == 0) {
        y = d / g.W;
        x = d % g.W;
    } else {
        y = py;
        x = px;
    }
}

__device__ __forceinline__ int64_t nchw_index(const ConvGeom &g, int b, int ci, int y, int x) {
    return ((static_cast<int64_t>(b) * g.C_in + ci) * g.H + y) * g.W + x;
}

// Raw input v = ((ky * KW + kx) * P + d) * C_in + ci (v < 64) of the
// receptive field of an output position of image b whose window starts at
// cell row py0 = oy * stride - pad and cell column x0: its NCHW index, or -1
// where the cell lies in the padding; wrow = its weight row k * C_in + ci.
__device__ __forceinline__ int64_t rf_input(const ConvGeom &g, int b, int py0, int x0, int v,
                                            int &wrow) {
    const int t1 = fdiv(v, g.dv_cin), ci = v - t1 * g.C_in;
    const int k = fdiv(t1, g.dv_p), d = t1 - k * g.P;
    const int ky = fdiv(k, g.dv_kw), kx = k - ky * g.KW;
    const int py = py0 + ky, px = x0 + kx;
    wrow = k * g.C_in + ci;
    if (py < 0 || py >= g.Hp || px < 0 || px >= g.Wp) return -1;
    int y, x;
    raw_pixel(g, py, px, d, y, x);
    return nchw_index(g, b, ci, y, x);
}

// Events of the raw inputs [1024 blk, 1024 blk + 1024) in NCHW order (layers
// whose forward bins its receptive fields directly, plain input): key = event
// row (-1: none), L, R where the row is >= 0. Every position that reads an
// input then loads its event instead of binning it again.
constexpr int kBinPerBlock = 1024;
__device__ void bin_block(const LifConst &C, int64_t n_in, const float *__restrict__ t_in,
                          const ConvSorted &cs, int blk) {
    const int64_t i0 = static_cast<int64_t>(blk) * kBinPerBlock + threadIdx.x;
    float v[kBinPerBlock / 256];
#pragma unroll
    for (int u = 0; u < kBinPerBlock / 256; ++u) {
        const int64_t i = i0 + u * 256;
        v[u] = (i < n_in) ? t_in[i] : INFINITY;
    }
#pragma unroll
    for (int u = 0; u < kBinPerBlock / 256; ++u) {
        const int64_t i = i0 + u * 256;
        if (i < n_in) {
            const Event e = bin_event(C, v[u]);
            cs.key[i] = e.row;
            if (e.row >= 0) {
                cs.L[i] = e.L;
                cs.R[i] = e.R;
            }
        }
    }
}

// The t-th raw input of cell row (b, py) in NCHW order (channel-major, so
// consecutive t are mostly consecutive addresses): its NCHW index, and its
// cell-major slot px * PC + j' in `slot`.
__device__ __forceinline__ int64_t cell_row_input(const ConvGeom &g, int b, int py, int t,
                                                  int &slot) {
    const int per_ch = g.Wp * g.P;
    const int ci = fdiv(t, g.dv_pch), rem = t - ci * per_ch;  // t < 2^30
    int y, x, px, d;
    if (g.pool == 2) {
        const int dy = fdiv(rem, g.dv_w);
        x = rem - dy * g.W;
        y = 2 * py + dy;
        px = x >> 1;
        d = dy * 2 + (x & 1);
    } else if (g.pool == 0) {
        d = rem;
        y = fdiv(d, g.dv_w);
        x = d - y * g.W;
        px = 0;
    } else {
        x = rem;
        y = py;
        px = rem;
        d = 0;
    }
    slot = px * g.PC + d * g.C_in + ci;
    return nchw_index(g, b, ci, y, x);
}

// ------------------------------------------------------------ cell sort --
// One block of 256 threads per cell row (b, py).
// LDS: hist[r][px] (later the next free slot of bucket (r, px)), the 256
// per-thread partial sums of the prefix scan, then (when they fit) the cell
// row's input spike times in cell-major order, read once in NCHW order, and
// (when they fit too) the four waves' lists of inputs with events.
// Wave w owns cells px = w, w + 4, ... (each bucket is ranked by one wave
// only); where a cell has fewer than 64 inputs a wave takes several of its
// cells per pass. Records of a bucket keep the input order (j' ascending).
// With ev set the cell row's events are written too: every input's row, and
// the halves and their derivatives where the row is >= 0.
__host__ __device__ __forceinline__ int sort_stage_floats(int M, const ConvGeom &g) {
    const int per = g.Wp * g.PC;
    return ((M + 3) * g.Wp + 256 + per) * 4 <= 64 * 1024 ? per : 0;
}

// With the row staged: ints of the four waves' lists of event inputs (each
// wave owns the cell columns px = wave mod 4, at most ceil(Wp / 4) * PC
// inputs), or 0 where they do not fit beside the staging in 64 KB.
constexpr int kSortWaves = 4;  // the sort runs in blocks of 256 threads
__host__ __device__ __forceinline__ int sort_list_ints(int M, const ConvGeom &g) {
    const int stage = sort_stage_floats(M, g);
    const int cap = (g.Wp + kSortWaves - 1) / kSortWaves * g.PC * kSortWaves;
    return (stage > 0 && ((M + 3) * g.Wp + 256 + stage + cap) * 4 <= 64 * 1024) ? cap : 0;
}

// the event of cell-major input slot k = cell * PC + d * C_in + ci: its row
// (int bits), and the halves and their derivatives (read only where it is >= 0)
__device__ __forceinline__ float *event_at(const CellEv &ev, const ConvGeom &g, int64_t cell, int j) {
    const int d = fdiv(j, g.dv_cin);
    return ev.ev + (cell * g.P + d) * 5 * g.C_in + (j - d * g.C_in);
}
__device__ __forceinline__ void put_event(const CellEv &ev, const ConvGeom &g, int64_t cell, int j,
                                          const Event &e) {
    float *p = event_at(ev, g, cell, j);
    p[g.C_in] = e.L;
    p[2 * g.C_in] = e.R;
    p[3 * g.C_in] = e.dL;
    p[4 * g.C_in] = e.dR;
}

__device__ void sort_cell_row(const LifConst &C, const ConvGeom &g, const float *__restrict__ t_in,
                              const ConvSorted &cs, const CellEv &ev, int cr, int *sh) {
    const int R = rows_of(C);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int b = cr / g.Hp, py = cr % g.Hp;
    const int nb = R * g.Wp;  // buckets, flat f = r * Wp + px
    const int noff = conv_off_stride(R, g);
    int *hist = sh;
    int *part = sh + nb;
    float *tl = sort_stage_floats(C.M, g) > 0 ? reinterpret_cast<float *>(part + 256) : nullptr;
    for (int k = threadIdx.x; k < nb; k += blockDim.x) hist[k] = 0;
    if (tl) {
        // staged rows are checked for events as they are read: a row without
        // any (the deep layers at random initialisation) skips the
        // histogram pass. The test is a window 0.001 dt wider at both ends
        // than the one bin_row keeps, [T_0 - dt, T_M + dt) (a superset:
        // bin_row's rounding moves its bounds far less), so it costs two
        // compares; NaN and +-inf fail it.
        const int per = g.Wp * g.PC;
        const float w_lo = C.t0 - 1.001f * C.dt;
        const float w_hi = fmaf(static_cast<float>(C.M) + 1.001f, C.dt, C.t0);
        bool any = false;
        // four inputs per pass, their loads issued together
        for (int t4 = threadIdx.x; t4 < per; t4 += 4 * blockDim.x) {
            int slot[4];
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t4 + u * static_cast<int>(blockDim.x);
                const int64_t src = cell_row_input(g, b, py, min(t, per - 1), slot[u]);
                v[u] = (t < per) ? t_in[src] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (t4 + u * static_cast<int>(blockDim.x) < per) {
                    tl[slot[u]] = v[u];
                    any = any || (v[u] >= w_lo && v[u] < w_hi);
                }
            }
        }
        if (!__syncthreads_or(any)) {
            if (ev.ev && threadIdx.x == 0) ev.live[cr] = 0;
            int *off0 = cs.off + static_cast<int64_t>(cr) * noff;
            for (int f = threadIdx.x; f < noff; f += blockDim.x) off0[f] = 0;
            return;
        }
    } else {
        __syncthreads();
    }
    auto t_at = [&](int px, int j) {
        if (tl) return tl[px * g.PC + j];
        int y, x;
        const int d = fdiv(j, g.dv_cin);
        raw_pixel(g, py, px, d, y, x);
        return t_in[nchw_index(g, b, j - d * g.C_in, y, x)];
    };
    const int cpi = (g.PC < kWave) ? kWave / g.PC : 1;  // cells per pass
    const int lsub = (g.PC < kWave) ? lane / g.PC : 0;
    const int lj = (g.PC < kWave) ? lane % g.PC : lane;
    const int64_t cb = static_cast<int64_t>(cr) * g.Wp, rb = cb * g.PC;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // List form (the row staged and the lists fitting): the histogram pass
    // also appends each event input (slot px * PC + j, row r) to its wave's
    // list in pass order and writes every input's event row; the placement
    // then visits only the listed inputs. A wave's buckets (r, px) hold only
    // its own cell columns, so list order is the pass order within each.
    const int lcap = (tl && nw == kSortWaves) ? sort_list_ints(C.M, g) / kSortWaves : 0;
    int *lst = lcap > 0 ? reinterpret_cast<int *>(tl + sort_stage_floats(C.M, g)) + wave * lcap
                        : nullptr;
    int nq = 0;
    bool has = false;
    for (int i0 = 0; wave + nw * i0 < g.Wp; i0 += cpi) {
        const int px = wave + nw * (i0 + lsub);
        const bool cell_ok = lsub < cpi && px < g.Wp;
        for (int j0 = 0; j0 < g.PC; j0 += kWave) {
            const int j = j0 + lj;
            int r = -1;
            if (cell_ok && j < g.PC) {
                r = bin_row(C, t_at(px, j));
                if (lst && ev.ev) *event_at(ev, g, cb + px, j) = __int_as_float(r);
                if (r >= 0) {
                    atomicAdd(&hist[r * g.Wp + px], 1);
                    has = true;
                }
            }
            if (lst) {
                const uint64_t m = __ballot(r >= 0);
                if (r >= 0) lst[nq + __popcll(m & below)] = ((px * g.PC + j) << 9) | r;
                nq += __popcll(m);
            }
        }
    }
    has = __syncthreads_or(has);
    if (ev.ev && threadIdx.x == 0) ev.live[cr] = has;
    if (!has) {
        // no input of this cell row has events: empty buckets
        int *off0 = cs.off + static_cast<int64_t>(cr) * noff;
        for (int f = threadIdx.x; f < noff; f += blockDim.x) off0[f] = 0;
        return;
    }
    // exclusive prefix over the buckets in (r, px) order: per-thread chunk
    // sums, scanned by wave 0 (four per lane), then each chunk in order
    const int chunk = (nb + blockDim.x - 1) / blockDim.x;
    const int lo = min(nb, static_cast<int>(threadIdx.x) * chunk), hi = min(nb, lo + chunk);
    int s = 0;
    for (int f = lo; f < hi; ++f) s += hist[f];
    part[threadIdx.x] = s;
    __syncthreads();
    if (wave == 0) {
        const int v0 = part[4 * lane], v1 = part[4 * lane + 1], v2 = part[4 * lane + 2],
                  v3 = part[4 * lane + 3];
        const int tot = v0 + v1 + v2 + v3;
        int inc = tot;
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) {
            const int o = __shfl_up(inc, m);
            if (lane >= m) inc += o;
        }
        const int ex = inc - tot;
        part[4 * lane] = ex;
        part[4 * lane + 1] = ex + v0;
        part[4 * lane + 2] = ex + v0 + v1;
        part[4 * lane + 3] = ex + v0 + v1 + v2;
        if (lane == kWave - 1) {
            // the last row's end and the record count
            int *off = cs.off + static_cast<int64_t>(cr) * noff;
            off[g.Wp * R + R - 1] = inc;
            off[noff - 1] = inc;
        }
    }
    __syncthreads();
    int run = part[threadIdx.x];
    int *off = cs.off + static_cast<int64_t>(cr) * noff;
    int r = lo / g.Wp, px = lo - r * g.Wp;  // bucket f = r * Wp + px, advanced with f
    for (int f = lo; f < hi; ++f) {
        const int v = hist[f];
        off[px * R + r] = run;
        if (px == 0 && r > 0) off[g.Wp * R + r - 1] = run;  // the end of row r - 1
        hist[f] = run;
        run += v;
        if (++px == g.Wp) {
            px = 0;
            ++r;
        }
    }
    __syncthreads();
    // placement: lanes of one bucket are ranked by lane (j' ascending). The
    // lanes of one pass that share a bucket are found by matching the bits of
    // a per-pass bucket key k = row * cpi + lsub (one ballot per bit, a cost
    // independent of how many buckets the pass touches); the highest lane of
    // each group then moves the bucket's next free slot.
    if (lst) {
        // list form: 64 listed inputs per pass, key row * ncw + px / 4
        // (ncw = the wave's cell columns); entries are in pass order, so each
        // bucket's records keep the input order
        const int ncw = (g.Wp + kSortWaves - 1) / kSortWaves;
        const int kb2 = uniform(R * ncw > 1 ? 32 - __clz(R * ncw - 1) : 0);
        for (int c0 = 0; c0 < nq; c0 += kWave) {
            const bool ok = c0 + lane < nq;
            const int en = ok ? lst[c0 + lane] : 0;
            const int slot = en >> 9, r = en & 511;
            const int px = fdiv(slot, g.dv_pc), j = slot - px * g.PC;
            Event e{-1, 0.f, 0.f, 0.f, 0.f};
            if (ok) e = bin_event(C, tl[slot]);  // its row is r
            const int kb = ok ? r * ncw + px / kSortWaves : 0;
            uint64_t same = __ballot(ok);
            for (int bit = 0; bit < kb2; ++bit) {
                const bool on = (kb >> bit) & 1;
                const uint64_t bal = __ballot(on);
                same &= on ? bal : ~bal;
            }
            const int f = r * g.Wp + px;
            int pos = 0;
            if (ok) {
                const int base = hist[f];
                pos = base + __popcll(same & below);
                if ((same >> lane) == 1ull) hist[f] = base + __popcll(same);
            }
            __builtin_amdgcn_wave_barrier();
            if (ok) {
                if (ev.ev) put_event(ev, g, cb + px, j, e);
                const int64_t o = rb + pos;
                cs.key[o] = px * g.C_in + (j - fdiv(j, g.dv_cin) * g.C_in);
                cs.L[o] = e.L;
                cs.R[o] = e.R;
            }
        }
        return;
    }
    const int kbits = uniform(R * cpi > 1 ? 32 - __clz(R * cpi - 1) : 0);
    for (int i0 = 0; wave + nw * i0 < g.Wp; i0 += cpi) {
        const int px = wave + nw * (i0 + lsub);
        const bool cell_ok = lsub < cpi && px < g.Wp;
        for (int j0 = 0; j0 < g.PC; j0 += kWave) {
            const int j = j0 + lj;
            Event e{-1, 0.f, 0.f, 0.f, 0.f};
            int f = -1;
            if (cell_ok && j < g.PC) {
                e = bin_event(C, t_at(px, j));
                if (ev.ev) {
                    *event_at(ev, g, cb + px, j) = __int_as_float(e.row);
                    if (e.row >= 0) put_event(ev, g, cb + px, j, e);
                }
                if (e.row >= 0) f = e.row * g.Wp + px;
            }
            const int kb = (f >= 0) ? e.row * cpi + lsub : 0;
            uint64_t same = __ballot(f >= 0);
            for (int bit = 0; bit < kbits; ++bit) {
                const bool on = (kb >> bit) & 1;
                const uint64_t bal = __ballot(on);
                same &= on ? bal : ~bal;
            }
            int pos = 0;
            if (f >= 0) {
                const int base = hist[f];
                pos = base + __popcll(same & below);
                if ((same >> lane) == 1ull) hist[f] = base + __popcll(same);
            }
            __builtin_amdgcn_wave_barrier();
            if (f >= 0) {
                const int64_t o = rb + pos;
                cs.key[o] = px * g.C_in + (j - fdiv(j, g.dv_cin) * g.C_in);
                cs.L[o] = e.L;
                cs.R[o] = e.R;
            }
        }
    }
}

// The events of one cell row without the sort (the backward without a kept
// forward): read in NCHW order, staged in LDS where the row fits, written in
// cell-major order (both coalesced). A row without events writes only its flag.
__host__ __device__ __forceinline__ int events_stage_floats(const ConvGeom &g) {
    return g.Wp * g.PC * 4 <= 48 * 1024 ? g.Wp * g.PC : 0;
}

__device__ void events_cell_row(const LifConst &C, const ConvGeom &g,
                                const float *__restrict__ t_in, const CellEv &ev, int cr,
                                float *tl) {
    const int b = cr / g.Hp, py = cr % g.Hp;
    const int per = g.Wp * g.PC;
    const int64_t cb = static_cast<int64_t>(cr) * g.Wp;
    const bool staged = events_stage_floats(g) > 0;
    bool has = false;
    for (int t = threadIdx.x; t < per; t += blockDim.x) {
        int slot;
        const float v = t_in[cell_row_input(g, b, py, t, slot)];
        has = has || bin_row(C, v) >= 0;
        if (staged) tl[slot] = v;
    }
    has = __syncthreads_or(has);
    if (threadIdx.x == 0) ev.live[cr] = has;
    if (!has) return;
    for (int t = threadIdx.x; t < per; t += blockDim.x) {
        int slot = t;
        const float v = staged ? tl[t] : t_in[cell_row_input(g, b, py, t, slot)];
        const Event e = bin_event(C, v);
        const int px = fdiv(slot, g.dv_pc), j = slot - px * g.PC;
        *event_at(ev, g, cb + px, j) = __int_as_float(e.row);
        if (e.row >= 0) put_event(ev, g, cb + px, j, e);
    }
}

// ------------------------------------------------------ weight layout ----
// WT[(k * C_in + ci) * C_out + co] = W[co, ci, k] / P (k = ky*KW + kx): W seen
// as [C_out][C_in * KT] (u = ci * KT + k) is transposed in 32 x 32 tiles
// through LDS (reads along u and writes along co coalesced); block blk takes
// tile (co0, u0) = ((blk / ntu) * 32, (blk % ntu) * 32).
constexpr int kWtLdsBytes = 32 * 33 * static_cast<int>(sizeof(float));

__host__ __device__ __forceinline__ int64_t weight_tiles(const ConvGeom &g) {
    const int64_t nu = static_cast<int64_t>(g.C_in) * g.KH * g.KW;
    return ((nu + 31) / 32) * ((g.C_out + 31) / 32);
}

template <typename WT>
__device__ void weights_block(const ConvGeom &g, const WT *__restrict__ W, float *__restrict__ out,
                              int64_t blk, float (*buf)[33]) {
    const int KT = g.KH * g.KW;
    const int NU = g.C_in * KT;
    const int ntu = (NU + 31) / 32;
    const int u0 = static_cast<int>(blk % ntu) * 32, c0 = static_cast<int>(blk / ntu) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int r = ty; r < 32; r += blockDim.x >> 5) {
        const int co = c0 + r, u = u0 + tx;
        if (co < g.C_out && u < NU) buf[r][tx] = WLoad<WT>::get(W, static_cast<int64_t>(co) * NU + u);
    }
    __syncthreads();
    for (int r = ty; r < 32; r += blockDim.x >> 5) {
        const int u = u0 + r, co = c0 + tx;
        if (u < NU && co < g.C_out) {
            const int ci = u / KT, k = u % KT;
            out[(static_cast<int64_t>(k) * g.C_in + ci) * g.C_out + co] = buf[tx][r] * g.inv_P;
        }
    }
}

// ------------------------------------------------------ position walk ----
// The records an output position (b, oy, ox) reads: for event row r and
// kernel row ky, the segment [off[r][xa], off[r][xb]) of cell row
// py = oy*stride - pad + ky; a record's key px*C_in + ci plus the segment
// constant (ky*KW - x0)*C_in is its row in WT. The bucket starts of the KH
// cell rows are held one event row per lane (64 rows at a time).
constexpr int kCBatch = 8;

template <int KHT>
struct PosWalk {
    int b, pos, x0, xa, xb, nb1, wlim;
    int64_t recb[KHT], offb[KHT];
    int wofs[KHT];
    bool vky[KHT];
    int oa[KHT], ob[KHT];

    // geometry of position p (no memory reads)
    __device__ __forceinline__ void init(const LifConst &C, const ConvGeom &g, int64_t p) {
        const int HoWo = g.Ho * g.Wo;
        const int pi = static_cast<int>(p);  // B * Ho * Wo < 2^31 (checked at the boundary)
        b = uniform(pi / HoWo);
        pos = uniform(pi % HoWo);
        const int oy = pos / g.Wo, ox = pos % g.Wo;
        x0 = ox * g.stride - g.pad;
        xa = max(0, x0);
        xb = max(xa, min(g.Wp, x0 + g.KW));
        nb1 = conv_off_stride(rows_of(C), g);
        wlim = g.KH * g.KW * g.C_in - 1;
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky) {
            const int py = oy * g.stride - g.pad + ky;
            vky[ky] = ky < g.KH && py >= 0 && py < g.Hp && xa < xb;
            const int64_t cr = static_cast<int64_t>(b) * g.Hp + (vky[ky] ? py : 0);
            recb[ky] = cr * g.Wp * g.PC;
            offb[ky] = cr * nb1;
            wofs[ky] = (ky * g.KW - x0) * g.C_in;
        }
    }

    // the number of records in the KH cell rows (0: nothing to read)
    __device__ __forceinline__ int cell_records(const ConvSorted &cs) const {
        int any = 0;
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky)
            if (vky[ky]) any += *as_const(cs.off + offb[ky] + nb1 - 1);
        return any;
    }

    __device__ __forceinline__ void load_offs(const ConvGeom &g, const ConvSorted &cs, int R,
                                              int r0, int lane) {
        const int r = min(r0 + lane, R - 1);
        // bucket starts are clamped to the cell row's slots; lanes read one
        // column of the table each, contiguously
        const int per = g.Wp * g.PC;
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky) {
            const int *o = cs.off + offb[ky] + r;
            oa[ky] = vky[ky] ? min(max(o[xa * R], 0), per) : 0;
            ob[ky] = vky[ky] ? min(max(o[xb * R], oa[ky]), per) : 0;
        }
    }
};

// -------------------------------------------------------------- forward --
// Wave = one output position, lane = output channel of a 64-wide tile.
// The position's records, in the order the sums need them (event row, then
// kernel row, then bucket order), form a virtual list: lanes = event rows
// hold the KH segment bounds of their row and an exclusive prefix of the
// row counts; for 64 list entries at a time each lane finds its entry's row
// (binary search over the prefix with lane shuffles), its segment and its
// record, and loads the record's fields with one vector load each; the
// decoded entries (weight-row offset, row, L, R) go to a small LDS area of
// the wave. The entries are then summed in batches of up to 8 entries of one
// event row (a batch's entries read back with one LDS read, its weight rows
// loaded together), and rows close into the interval scan as the
// row changes. Sums and their order are those of a row-by-row walk.
struct FwdEntry { int wb, row; float L, R; };
// kDirect (receptive fields of at most 64 raw inputs, at most 64 event rows,
// pooled or plain input): no cell-row sort; lane v takes raw input
// v = ((ky * KW + kx) * P + d) * C_in + ci of the receptive field, bins its
// spike time itself, and the lanes are ranked by event row (stable in v, so
// within a row the order is kernel row, cell column, input slot: the sorted
// walk's order) from ballots of the row's bits; the ranked entries go to the
// same LDS list as one chunk of the walk.
// A block takes kFwdWaves consecutive output positions of one 64-channel
// tile, one per wave. Before its own position, every wave of the sorted walk
// makes the same block-level test from scalar loads (no barrier): where the
// block's positions lie in one image and the cell rows their receptive
// fields span hold no records at all, the waves write the block's silent
// outputs together, as runs of kFwdWaves consecutive positions per channel,
// instead of 64 single floats 4 * Ho * Wo bytes apart per position (such
// scattered stores bound the forward of layers without input events).
// (At most 72 VGPRs, seven waves per SIMD, where that needs no spill: conv9
// 0.819 -> 0.795 ms against six; else at most 80. Eight would spill.)
constexpr int kFwdWaves = 4;
// Sums of up to kCBatch list entries: lane l holds entry l % 8 of the batch (one
// LDS read of the lanes' entries instead of a broadcast read of each), and an
// entry's fields are row_newbcast operands: of the add that makes its weight's
// offset and of its two multiply-adds. What bounds the walk is the vector ALU:
// 64 -> 64 channels, 32 x 32, 3,873 -> 3,068 vector, 898 -> 143 LDS and (the second
// half of a batch not loaded where the row ends before it) 453 -> 393 vector
// memory instructions per wave; forward and backward of that layer 1321 -> 1281 us,
// the forward of 64 -> 128, 28 x 28, stride 2 220 -> 199 us. Offsets read into
// scalars instead cost a wait each (forward 15 % slower), and groups of 8 loaded
// ahead across rows more scalar branches than the unused loads they save (28 %).
// s_nop: a register written by the vector ALU may be read as a row broadcast two
// cycles later at the earliest.
#define FWD_FMA(q, w)                                                                   \
    "v_fmac_f32_dpp %0, %2, " w " row_newbcast:" q " row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %1, %3, " w " row_newbcast:" q " row_mask:0xf bank_mask:0xf\n"
template <int Q>
__device__ __forceinline__ void sum_entry(float &aL, float &aR, float L, float R, float w) {
    asm("s_nop 1\n" FWD_FMA("%5", "%4") : "+&v"(aL), "+&v"(aR) : "v"(L), "v"(R), "v"(w), "n"(Q));
}
__device__ __forceinline__ void sum_entries4(float &aL, float &aR, float L, float R,
                                             const float *w) {
    asm("s_nop 1\n" FWD_FMA("0", "%4") FWD_FMA("1", "%5") FWD_FMA("2", "%6") FWD_FMA("3", "%7")
        : "+&v"(aL), "+&v"(aR)
        : "v"(L), "v"(R), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]));
}
__device__ __forceinline__ void sum_entries8(float &aL, float &aR, float L, float R,
                                             const float (&w)[kCBatch]) {
    static_assert(kCBatch == 8, "one asm operand per entry");
    asm("s_nop 1\n" FWD_FMA("0", "%4") FWD_FMA("1", "%5") FWD_FMA("2", "%6") FWD_FMA("3", "%7")
            FWD_FMA("4", "%8") FWD_FMA("5", "%9") FWD_FMA("6", "%10") FWD_FMA("7", "%11")
        : "+&v"(aL), "+&v"(aR)
        : "v"(L), "v"(R), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]),
          "v"(w[6]), "v"(w[7]));
}
#undef FWD_FMA
// the weights of entries Q .. Q + 3 of a batch, their byte offsets row broadcasts of wb
template <int Q>
__device__ __forceinline__ void load_entries(__amdgpu_buffer_rsrc_t wr, int voff, int wb,
                                             float (&w)[kCBatch]) {
    static_for<kCBatch / 2>([&](auto q) { w[Q + q] = BufLoad<float>::get(wr, voff + row_bcast<Q + q>(wb), 0); });
}
template <int KHT, int KS, bool kDirect>
constexpr int fwd_min_waves() {
    return (KHT <= 3 && (kDirect || KS != kAnyKind)) ? 7 : 6;
}
template <int KHT, int KS, bool kDirect>
__global__ __launch_bounds__(kFwdWaves * kWave) __attribute__((amdgpu_waves_per_eu(fwd_min_waves<KHT, KS, kDirect>(), 8))) void conv_fwd_kernel(LifConst C, ConvGeom g, int64_t n_pos,
                                                       const float *__restrict__ Wt,
                                                       ConvSorted cs, const float *__restrict__ t_in,
                                                       float *__restrict__ t_out,
                                                       float *__restrict__ slope,
                                                       int *__restrict__ q_idx, int pre) {
    // a wave's list, padded so that a batch starting at any entry stays inside
    __shared__ FwdEntry ent[kFwdWaves][kWave + kCBatch];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int64_t p0 = static_cast<int64_t>(xcd_block(blockIdx.x, gridDim.x)) * kFwdWaves;
    const int64_t p = p0 + wave;
    const int HoWo = g.Ho * g.Wo;
    if constexpr (!kDirect) {
        // positions p0 .. pl (p0 < n_pos: the grid holds no empty block);
        // B * Ho * Wo < 2^31 (checked at the boundary)
        const int q0 = static_cast<int>(p0), ql = static_cast<int>(min(p0 + kFwdWaves, n_pos) - 1);
        const int b0 = q0 / HoWo;
        if (b0 == ql / HoWo) {
            const int y_lo = max(0, (q0 - b0 * HoWo) / g.Wo * g.stride - g.pad);
            const int y_hi = min(g.Hp - 1, (ql - b0 * HoWo) / g.Wo * g.stride - g.pad + g.KH - 1);
            const int nb1 = conv_off_stride(rows_of(C), g);
            int recs = 0;
            for (int y = y_lo; y <= y_hi; ++y)
                recs |= *as_const(cs.off + (static_cast<int64_t>(b0) * g.Hp + y) * nb1 + nb1 - 1);
            if (recs == 0) {
                // element e = wave * 64 + lane: channel e / kFwdWaves,
                // position e % kFwdWaves
                const int e = wave * kWave + lane;
                const int64_t ps = p0 + e % kFwdWaves;
                const int o = blockIdx.y * kWave + e / kFwdWaves;
                if (ps < n_pos && o < g.C_out) {
                    const int pi = static_cast<int>(ps);
                    const int bb = pi / HoWo;
                    const int64_t idx = (static_cast<int64_t>(bb) * g.C_out + o) * HoWo + (pi - bb * HoWo);
                    t_out[idx] = INFINITY;
                    slope[idx] = 0.f;
                    q_idx[idx] = -1;
                }
                return;
            }
        }
    }
    if (p >= n_pos) return;  // wave-uniform; no block barrier below
    FwdEntry *my = ent[wave];
    if (lane < kCBatch) my[kWave + lane] = FwdEntry{0, 0, 0.f, 0.f};
    const int co = blockIdx.y * kWave + lane;
    const bool row_ok = co < g.C_out;
    const int R = rows_of(C);
    PosWalk<KHT> wk;
    wk.init(C, g, p);
    const int64_t o_out = (static_cast<int64_t>(wk.b) * g.C_out + co) * HoWo + wk.pos;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(
        Wt, static_cast<uint32_t>(static_cast<int64_t>(wk.wlim + 1) * g.C_out * sizeof(float)));
    const int voff = (row_ok ? co : 0) * static_cast<int>(sizeof(float));
    const int rstride = g.C_out * static_cast<int>(sizeof(float));
    Scan<KS> sc;
    float aL = 0.f, aR = 0.f, carry = 0.f;
    int cur = 0;  // row being summed
    // close rows cur .. target-1: point r-1 gets row r's L sums plus row
    // r-1's R sums. A record's row is at most R-2, so closing up to it never
    // reaches grid point M (the last interval, tested only at the end).
    auto close_to_mid = [&](int target) {
        while (cur < target) {
            if (cur >= 1) sc.template step_k<false>(C, cur - 1, aL + carry);
            carry = aR;
            aL = 0.f;
            aR = 0.f;
            ++cur;
        }
    };
    auto close_to_end = [&](int target) {
        while (cur < target) {
            if (cur >= 1) sc.step(C, cur - 1, aL + carry);
            carry = aR;
            aL = 0.f;
            aR = 0.f;
            ++cur;
        }
    };
    // (direct path) the sums of a batch of nk <= kCBatch list entries in
    // order; true once every lane has found its interval. A full batch inside
    // one event row (rows never decrease along the list) is summed without
    // per-entry tests.
    auto sum_batch = [&](const FwdEntry (&e)[kCBatch], const float (&w)[kCBatch], int nk) {
        const int ra = uniform(e[0].row);
        if (nk == kCBatch && ra == uniform(e[kCBatch - 1].row)) {
            if (ra != cur) {
                close_to_mid(ra);
                if (__all(sc.found() || !row_ok)) return true;
            }
#pragma unroll
            for (int q = 0; q < kCBatch; ++q) {
                aL = fmaf(w[q], e[q].L, aL);
                aR = fmaf(w[q], e[q].R, aR);
            }
            return false;
        }
#pragma unroll
        for (int q = 0; q < kCBatch; ++q) {
            if (q < nk) {
                const int row = uniform(e[q].row);
                if (row != cur) {
                    close_to_mid(row);
                    if (__all(sc.found() || !row_ok)) return true;
                }
                aL = fmaf(w[q], e[q].L, aL);
                aR = fmaf(w[q], e[q].R, aR);
            }
        }
        return false;
    };
    bool done = false, started = false;
    if constexpr (kDirect) {
        const int F = g.KH * g.KW * g.PC;
        bool has = false;
        FwdEntry me{0, -1, 0.f, 0.f};
        if (lane < F) {
            int wrow;
            const int64_t src = rf_input(g, wk.b, (wk.pos / g.Wo) * g.stride - g.pad, wk.x0,
                                         lane, wrow);
            if (src >= 0) {
                if (pre) {  // binned once per input by the set-up launch
                    const int r = cs.key[src];
                    const float Lv = cs.L[src], Rv = cs.R[src];
                    if (r >= 0) {
                        has = true;
                        me = FwdEntry{wrow * rstride, r, Lv, Rv};
                    }
                } else {
                    const Event e = bin_event<KS>(C, t_in[src]);
                    if (e.row >= 0) {
                        has = true;
                        me = FwdEntry{wrow * rstride, e.row, e.L, e.R};
                    }
                }
            }
        }
        const uint64_t hm = __ballot(has);
        const int total = __popcll(hm);
        if (total == 0) {  // no events in the receptive field: silent
            if (row_ok) {
                t_out[o_out] = INFINITY;
                slope[o_out] = 0.f;
                q_idx[o_out] = -1;
            }
            return;
        }
        // stable rank by event row: lanes with a smaller row, then lanes
        // with the same row and a lower index
        uint64_t lt = 0, eq = hm;
        const int kbits = uniform(32 - __clz(max(R - 2, 1)));
        for (int bit = kbits - 1; bit >= 0; --bit) {
            const bool on = has && ((me.row >> bit) & 1);
            const uint64_t bal = __ballot(on);
            if (on) lt |= eq & ~bal;
            eq &= on ? bal : (hm & ~bal);
        }
        const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        if (has) my[__popcll(lt) + __popcll(eq & below)] = me;
        __builtin_amdgcn_wave_barrier();
        cur = uniform(my[0].row);  // the scan starts at the first row with records
        started = true;
        for (int s0 = 0; s0 < total; s0 += kCBatch) {
            FwdEntry e[kCBatch];
            float w[kCBatch];
#pragma unroll
            for (int q = 0; q < kCBatch; ++q) e[q] = my[s0 + q];  // LDS broadcasts
#pragma unroll
            for (int q = 0; q < kCBatch; ++q) w[q] = BufLoad<float>::get(wr, voff + e[q].wb, 0);
            if (sum_batch(e, w, min(kCBatch, total - s0))) {
                done = true;
                break;
            }
        }
    } else {
    // the KH cell rows' record counts (scalar loads) rule out most positions
    // without events in their receptive field before any vector load
    if (wk.cell_records(cs) == 0) {
        if (row_ok) {
            t_out[o_out] = INFINITY;
            slope[o_out] = 0.f;
            q_idx[o_out] = -1;
        }
        return;
    }
    for (int r0 = 0; r0 <= R - 2 && !done; r0 += kWave) {
        wk.load_offs(g, cs, R, r0, lane);
        const bool rvalid = r0 + lane <= R - 2;
        int n0[KHT];
        int nr = 0;
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky) {
            n0[ky] = rvalid ? wk.ob[ky] - wk.oa[ky] : 0;
            nr += n0[ky];
        }
        int inc = nr;
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) {
            const int o = __shfl_up(inc, m);
            if (lane >= m) inc += o;
        }
        const int start = inc - nr;
        const int start_eff = rvalid ? start : 0x7fffffff;
        const int total = uniform(__builtin_amdgcn_readlane(inc, kWave - 1));
        if (!started && total > 0) {
            // rows before the first one with records add nothing to a zero
            // state: the scan starts there
            cur = r0 + __ffsll(static_cast<unsigned long long>(__ballot(nr > 0))) - 1;
            started = true;
        }
        for (int c0 = 0; c0 < total && !done; c0 += kWave) {
            const int v = c0 + lane;
            const bool rec_ok = v < total;
            // row lane lo: the last row whose prefix start is <= v
            int lo = 0;
#pragma unroll
            for (int step = kWave / 2; step >= 1; step >>= 1) {
                const int cand = lo + step;
                const int sv = __shfl(start_eff, cand & (kWave - 1));
                if (cand < kWave && sv <= v) lo = cand;
            }
            int kk = v - __shfl(start, lo);
            int sel = -1, ridx = 0;
#pragma unroll
            for (int ky = 0; ky < KHT; ++ky) {
                const int a = __shfl(wk.oa[ky], lo), nn = __shfl(n0[ky], lo);
                if (sel < 0) {
                    if (kk < nn) {
                        sel = ky;
                        ridx = a + kk;
                    } else {
                        kk -= nn;
                    }
                }
            }
            int64_t gi = 0;
            int wof = 0;
#pragma unroll
            for (int ky = 0; ky < KHT; ++ky) {
                if (sel == ky) {
                    gi = wk.recb[ky] + ridx;
                    wof = wk.wofs[ky];
                }
            }
            const bool ok = rec_ok && sel >= 0;
            const int key = ok ? cs.key[gi] : 0;
            const float Lv = ok ? cs.L[gi] : 0.f;
            const float Rv = ok ? cs.R[gi] : 0.f;
            const int wb = min(max(key + wof, 0), wk.wlim) * rstride;
            // the entry's row, and how many entries of that row the list holds
            // from this one on (itself included): row | nrem << 16 (rows < 2^16)
            const int nrem = min(__shfl(inc, lo) - v, kWave);
            my[lane] = FwdEntry{wb, (r0 + lo) | (nrem << 16), Lv, Rv};
            __builtin_amdgcn_wave_barrier();
            const int nc = min(kWave, total - c0);
            // batches never cross a row: up to kCBatch entries of the head
            // entry's row, summed without per-entry row tests; entries past
            // the row are read (and, in the batch's first half, and in its
            // second where it has entries, their weights loaded) but not summed
            for (int s0 = 0; s0 < nc;) {
                const FwdEntry e = my[s0 + (lane & (kCBatch - 1))];
                float w[kCBatch];
                load_entries<0>(wr, voff, e.wb, w);
                const int hd = uniform(e.row);
                const int ra = hd & 0xffff;
                const int nk = max(1, min(min(kCBatch, hd >> 16), nc - s0));  // always advances
                if (nk > kCBatch / 2) load_entries<kCBatch / 2>(wr, voff, e.wb, w);
                if (ra != cur) {
                    close_to_mid(ra);
                    if (__all(sc.found() || !row_ok)) {
                        done = true;
                        break;
                    }
                }
                if (nk == kCBatch) {
                    sum_entries8(aL, aR, e.L, e.R, w);
                } else if (nk >= kCBatch / 2) {
                    sum_entries4(aL, aR, e.L, e.R, w);
                    if (nk > 4) sum_entry<4>(aL, aR, e.L, e.R, w[4]);
                    if (nk > 5) sum_entry<5>(aL, aR, e.L, e.R, w[5]);
                    if (nk > 6) sum_entry<6>(aL, aR, e.L, e.R, w[6]);
                } else {
                    sum_entry<0>(aL, aR, e.L, e.R, w[0]);
                    if (nk > 1) sum_entry<1>(aL, aR, e.L, e.R, w[1]);
                    if (nk > 2) sum_entry<2>(aL, aR, e.L, e.R, w[2]);
                }
                s0 += nk;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    }  // kDirect
    if (!started) {  // no events in the receptive field: silent
        if (row_ok) {
            t_out[o_out] = INFINITY;
            slope[o_out] = 0.f;
            q_idx[o_out] = -1;
        }
        return;
    }
    if (!done) {
        // the last row's sums reach grid points cur-1 and cur; after them no
        // input arrives: the rest of the window is one free-decay segment
        close_to_end(min(cur + 2, R - 1));
        if (cur < R - 1) sc.tail(C, cur - 1);
    }
    if (!row_ok) return;
    float to, sl;
    int q;
    sc.finish(C, to, sl, q);
    t_out[o_out] = to;
    slope[o_out] = sl;
    q_idx[o_out] = q;
}

// NP output positions per wave, LP = 64 / NP lanes each (one channel per
// lane; with NP = 1 a grid row per 64-channel tile). Needs at most LP event
// rows (R - 1 <= LP) and at most kListMaxRec raw inputs per receptive field
// (E = KH * KW * PC). Each position's lanes decode its records -- in the
// order of the chunked walk: event row, kernel row, bucket order -- into the
// wave's LDS list; then the positions sum the event rows in lockstep, one row
// at a time (a position with fewer records in the row adds zero-weight
// entries, which leave its sums unchanged), and close each row into the
// interval scan together, so the scan runs on all 64 lanes and the row
// structure needs no per-record test. Every neuron's sums and their order
// are those of the chunked walk.
constexpr int kListMaxRec = 640;

// LDS ints of one wave's list of ne records: the weight rows as 16-bit
// indices (a list layer's receptive field has at most kListMaxRec / 2 raw
// inputs, so its weight rows fit), then the (L, R) pairs, 8-byte aligned
__host__ __device__ __forceinline__ int list_wave_ints(int ne) {
    const int ne4 = (ne + 3) & ~3;
    return ne4 / 2 + 2 * ne4;
}

// K consecutive records of a row from the LDS list at idx, of which the lane's
// position has `left` (entries past them add zero weight): weights loaded as
// one batch, then summed in order. kFull: every position of the wave has all
// K (no masking).
template <int K, bool kFull = false>
__device__ __forceinline__ void list_batch(const uint16_t *erow, const float2 *eLR, int idx,
                                           int left, __amdgpu_buffer_rsrc_t wr, int voff,
                                           int rstride, int l8, float &aL, float &aR) {
    // l8 = lane % 8: lanes l and l + 8 of each 16 hold record l of the lane's position
    // (32 -> 32 channels, 28 x 28, batch 128: the layer's pass 1340 -> 1297 us)
    const bool ok = (K == 8 || l8 < K) && (kFull || l8 < left);
    const int wb = ok ? static_cast<int>(__umul24(erow[idx + l8], rstride)) : 0;  // both < 2^24
    const float2 lr = ok ? eLR[idx + l8] : make_float2(0.f, 0.f);
    float w[K];
    static_for<K>([&](auto q) { w[q] = BufLoad<float>::get(wr, voff + row_bcast<q>(wb), 0); });
    if constexpr (K == 8) sum_entries8(aL, aR, lr.x, lr.y, w);
    else if constexpr (K == 4) sum_entries4(aL, aR, lr.x, lr.y, w);
    else static_for<K>([&](auto q) { sum_entry<q>(aL, aR, lr.x, lr.y, w[q]); });
}

// kDirect (E <= LP): as in the chunked walk, no cell-row sort: lane li of a
// position takes raw input li of its receptive field and bins it; the row
// counts come from LDS integer atomics, and each record's place in its row
// from ballots of the row bits (stable in li: the sorted walk's order).
template <int KHT, int KS, int NP, bool kDirect>
__global__ __launch_bounds__(256) void conv_fwd_list_kernel(LifConst C, ConvGeom g, int64_t n_pos,
                                                            const float *__restrict__ Wt,
                                                            ConvSorted cs,
                                                            const float *__restrict__ t_in,
                                                            float *__restrict__ t_out,
                                                            float *__restrict__ slope,
                                                            int *__restrict__ q_idx, int pre) {
    constexpr int LP = kWave / NP;
    extern __shared__ int list_lds[];  // per wave: weight rows [NP][E] (16-bit), then (L, R)[NP][E]
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int half = lane / LP, li = lane % LP, hb = half * LP;  // hb: the position's first lane
    const int nwb = blockDim.x >> 6;
    const int64_t pb = static_cast<int64_t>(xcd_block(blockIdx.x, gridDim.x)) * nwb * NP;
    const int64_t p0 = pb + wave * NP;
    if constexpr (!kDirect) {
        // the block's positions pb .. (nwb * NP of them; pb < n_pos): where
        // they lie in one image and the cell rows their receptive fields span
        // hold no records, the waves write the block's silent outputs
        // together, as runs of nwb * NP positions per channel (the same test
        // in every wave, from scalar loads: no barrier)
        const int HoWo = g.Ho * g.Wo, npb = nwb * NP;
        const int q0 = static_cast<int>(pb), ql = static_cast<int>(min(pb + npb, n_pos) - 1);
        const int b0 = q0 / HoWo;
        if (b0 == ql / HoWo) {
            const int y_lo = max(0, (q0 - b0 * HoWo) / g.Wo * g.stride - g.pad);
            const int y_hi = min(g.Hp - 1, (ql - b0 * HoWo) / g.Wo * g.stride - g.pad + g.KH - 1);
            const int nb1 = conv_off_stride(rows_of(C), g);
            int recs = 0;
            for (int y = y_lo; y <= y_hi; ++y)
                recs |= *as_const(cs.off + (static_cast<int64_t>(b0) * g.Hp + y) * nb1 + nb1 - 1);
            if (recs == 0) {
                // element e = wave * 64 + lane: channel e / npb, position e % npb
                for (int e = wave * kWave + lane; e < npb * LP; e += static_cast<int>(blockDim.x)) {
                    const int64_t ps = pb + e % npb;
                    const int o = blockIdx.y * LP + e / npb;
                    if (ps < n_pos && o < g.C_out) {
                        const int pi = static_cast<int>(ps);
                        const int bb = pi / HoWo;
                        const int64_t idx = (static_cast<int64_t>(bb) * g.C_out + o) * HoWo + (pi - bb * HoWo);
                        t_out[idx] = INFINITY;
                        slope[idx] = 0.f;
                        q_idx[idx] = -1;
                    }
                }
                return;
            }
        }
    }
    if (p0 >= n_pos) return;  // wave-uniform; no block barrier below
    const int64_t p = p0 + half;
    const bool pos_ok = p < n_pos;
    const int E = g.KH * g.KW * g.PC;
    const int ebase = half * E;  // the position's part of the wave's list
    const int WI = list_wave_ints(NP * E);
    uint16_t *erow = reinterpret_cast<uint16_t *>(list_lds + wave * WI);
    // (L, R) of a record: one 8-byte read
    float2 *eLR = reinterpret_cast<float2 *>(list_lds + wave * WI + ((NP * E + 3) & ~3) / 2);
    const int co = blockIdx.y * LP + li;
    const bool row_ok = pos_ok && co < g.C_out;
    const int HoWo = g.Ho * g.Wo;
    const int R = rows_of(C);
    const int64_t pp = pos_ok ? p : p0;
    const int b = static_cast<int>(pp) / HoWo, pos = static_cast<int>(pp) % HoWo;
    const int oy = pos / g.Wo, ox = pos % g.Wo;
    const int x0 = ox * g.stride - g.pad;
    const int xa = max(0, x0), xb = max(xa, min(g.Wp, x0 + g.KW));
    const int nb1 = conv_off_stride(R, g);
    const int wlim = g.KH * g.KW * g.C_in - 1;
    int64_t recb[KHT], offb[KHT];
    int wofs[KHT];
    bool vky[KHT];
    const int64_t o_out = (static_cast<int64_t>(b) * g.C_out + co) * HoWo + pos;
    auto write_silent = [&]() {
        if (row_ok) {
            t_out[o_out] = INFINITY;
            slope[o_out] = 0.f;
            q_idx[o_out] = -1;
        }
    };
    // lane li of a position = its event row li: the row's record count (and
    // on the sorted path its segment bounds), then an exclusive prefix of
    // the counts within the position's lanes
    const bool rvalid = li <= R - 2;
    int oa[KHT], n0[KHT];
    int nr = 0;
    // direct path: this lane's own record
    bool dhas = false;
    int drow = 0, dwb = 0;
    float2 dlr = make_float2(0.f, 0.f);
    if constexpr (kDirect) {
        int *hist = list_lds + (blockDim.x >> 6) * WI + wave * kWave;  // [NP][LP] row counts
        hist[lane] = 0;
        __builtin_amdgcn_wave_barrier();
        if (pos_ok && li < E) {
            int wrow;
            const int64_t src = rf_input(g, b, oy * g.stride - g.pad, x0, li, wrow);
            if (src >= 0) {
                int r;
                float Lv, Rv;
                if (pre) {  // binned once per input by the set-up launch
                    r = cs.key[src];
                    Lv = cs.L[src];
                    Rv = cs.R[src];
                } else {
                    const Event e = bin_event<KS>(C, t_in[src]);
                    r = e.row;
                    Lv = e.L;
                    Rv = e.R;
                }
                if (r >= 0) {
                    dhas = true;
                    drow = r;
                    dwb = wrow;  // weight row
                    dlr = make_float2(Lv, Rv);
                    atomicAdd(&hist[hb + r], 1);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (!__any(dhas)) {  // no events in any receptive field
            write_silent();
            return;
        }
        nr = rvalid ? hist[lane] : 0;
    } else {
        int any = 0;
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky) {
            const int py = oy * g.stride - g.pad + ky;
            vky[ky] = pos_ok && ky < g.KH && py >= 0 && py < g.Hp && xa < xb;
            const int64_t cr = static_cast<int64_t>(b) * g.Hp + (vky[ky] ? py : 0);
            recb[ky] = cr * g.Wp * g.PC;
            offb[ky] = cr * nb1;
            wofs[ky] = (ky * g.KW - x0) * g.C_in;
            if (vky[ky]) any += cs.off[offb[ky] + nb1 - 1];
        }
        if (!__any(any > 0)) {  // no receptive field's cell rows hold records
            write_silent();
            return;
        }
        const int rr = min(li, R - 2);
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky) {
            const int *o = cs.off + offb[ky] + rr;
            const int a = vky[ky] ? o[xa * R] : 0, e = vky[ky] ? o[xb * R] : 0;
            oa[ky] = a;
            n0[ky] = rvalid ? e - a : 0;
            nr += n0[ky];
        }
    }
    int inc = nr;
#pragma unroll
    for (int m = 1; m < LP; m <<= 1) {
        const int o = __shfl_up(inc, m, LP);
        if (li >= m) inc += o;
    }
    const int start = inc - nr;
    const int start_eff = rvalid ? start : 0x7fffffff;
    int tot = 0, tmax = 0;
#pragma unroll
    for (int h = 0; h < NP; ++h) {
        const int th = uniform(__builtin_amdgcn_readlane(inc, h * LP + LP - 1));
        if (h == half) tot = th;
        tmax = max(tmax, th);
    }
    const int rstride = g.C_out * static_cast<int>(sizeof(float));
    if constexpr (kDirect) {
        // place = the row's start + the records of the same row in lower lanes
        const uint64_t half_mask = (((1ull << (LP - 1)) << 1) - 1) << hb;
        const uint64_t hm = __ballot(dhas) & half_mask;
        uint64_t eq = hm;
        const int kbits = uniform(32 - __clz(max(R - 2, 1)));
        for (int bit = 0; bit < kbits; ++bit) {
            const bool on = dhas && ((drow >> bit) & 1);
            const uint64_t bal = __ballot(on);
            eq &= on ? bal : (hm & ~bal);
        }
        const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        const int rs = __shfl(start, hb + (dhas ? drow : 0));
        if (dhas) {
            const int at = ebase + rs + __popcll(eq & below);
            erow[at] = static_cast<uint16_t>(dwb);
            eLR[at] = dlr;
        }
    } else
    // decode LP records per position at a time into the LDS list
    for (int c0 = 0; c0 < tmax; c0 += LP) {
        const int v = c0 + li;
        int lo = 0;  // the position's last row whose start is <= v
#pragma unroll
        for (int step = LP / 2; step >= 1; step >>= 1) {
            const int cand = lo + step;
            const int sv = __shfl(start_eff, hb + (cand & (LP - 1)));
            if (cand < LP && sv <= v) lo = cand;
        }
        int kk = v - __shfl(start, hb + lo);
        int sel = -1, ridx = 0;
#pragma unroll
        for (int ky = 0; ky < KHT; ++ky) {
            const int a = __shfl(oa[ky], hb + lo), nn = __shfl(n0[ky], hb + lo);
            if (sel < 0) {
                if (kk < nn) {
                    sel = ky;
                    ridx = a + kk;
                } else {
                    kk -= nn;
                }
            }
        }
        if (v < tot && sel >= 0) {
            int64_t gi = 0;
            int wof = 0;
#pragma unroll
            for (int ky = 0; ky < KHT; ++ky) {
                if (sel == ky) {
                    gi = recb[ky] + ridx;
                    wof = wofs[ky];
                }
            }
            erow[ebase + v] = static_cast<uint16_t>(min(max(cs.key[gi] + wof, 0), wlim));
            eLR[ebase + v] = make_float2(cs.L[gi], cs.R[gi]);
        }
    }
    __builtin_amdgcn_wave_barrier();
    uint64_t rows_any = __ballot(nr > 0);
#pragma unroll
    for (int h = 1; h < NP; ++h) rows_any |= rows_any >> (h * LP);
    if (NP > 1) rows_any &= (1ull << LP) - 1;
    if (rows_any == 0) {  // no records in any receptive field
        write_silent();
        return;
    }
    // rows before the first one with records add nothing to a zero state
    const int r_first = __ffsll(static_cast<unsigned long long>(rows_any)) - 1;
    const int r_last = 63 - __clzll(static_cast<long long>(rows_any));
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(
        Wt, static_cast<uint32_t>(static_cast<int64_t>(wlim + 1) * g.C_out * sizeof(float)));
    const int voff = (row_ok ? co : 0) * static_cast<int>(sizeof(float));
    Scan<KS> sc;
    float aL = 0.f, aR = 0.f, carry = 0.f;
    for (int r = r_first; r <= R - 2; ++r) {
        if (r <= r_last) {
            int n = 0, nmin = 0x7fffffff, my_n = 0, my_s = ebase;
#pragma unroll
            for (int h = 0; h < NP; ++h) {
                const int nh = uniform(__builtin_amdgcn_readlane(nr, h * LP + r));
                const int sh = uniform(__builtin_amdgcn_readlane(start, h * LP + r));
                n = max(n, nh);
                nmin = min(nmin, nh);
                if (h == half) {
                    my_n = nh;
                    my_s += sh;
                }
            }
            // batches of 8 (unmasked while every position has them), then
            // 4, then single records: no load or sum past the row's largest
            // count
            int i0 = 0;
            for (; i0 + 8 <= nmin; i0 += 8)
                list_batch<8, true>(erow, eLR, my_s + i0, my_n - i0, wr, voff, rstride, li & 7, aL, aR);
            for (; i0 + 8 <= n; i0 += 8)
                list_batch<8>(erow, eLR, my_s + i0, my_n - i0, wr, voff, rstride, li & 7, aL, aR);
            if (i0 + 4 <= n) {
                list_batch<4>(erow, eLR, my_s + i0, my_n - i0, wr, voff, rstride, li & 7, aL, aR);
                i0 += 4;
            }
            for (; i0 < n; ++i0) list_batch<1>(erow, eLR, my_s + i0, my_n - i0, wr, voff, rstride, li & 7, aL, aR);
        } else if (r == r_last + 2) {
            // every record is in: grid points r-1 .. M see no input, the rest
            // of the window is one free-decay segment
            sc.tail(C, r - 1);
            break;
        }
        // grid point r-1: this row's L sums plus the previous row's R sums
        if (r >= 1) sc.step(C, r - 1, aL + carry);
        carry = aR;
        aL = 0.f;
        aR = 0.f;
        if (__all(sc.found() || !row_ok)) break;
    }
    if (!row_ok) return;
    float to, sl;
    int q;
    sc.finish(C, to, sl, q);
    t_out[o_out] = to;
    slope[o_out] = sl;
    q_idx[o_out] = q;
}

// --------------------------------------------------------- backward ------
// Gradient triples (gK, gE, q) of grad_triple for kGradPos output
// positions s = b * Ho*Wo + p and one tile of kGradCh channels (block blk =
// position group * tiles + tile): read from the NCHW outputs with positions
// along the lanes, staged in LDS and written position-major [s][3][co] (gK, gE
// and q as int bits; each position's channels contiguous).
// rend[s] = min(R-2, max q + 1) over the channels of s that pass gradient
// (G[m] vanishes for m > q, and a record of event row r reads G[r-1] and
// G[r]), -1 if none does.
constexpr int kGradPos = 16, kGradCh = 64;
constexpr int kGradLdsBytes = (3 * kGradCh * (kGradPos + 1) + kGradPos) * 4;

__device__ void grad_block(const LifConst &C, const ConvGeom &g, int64_t n_pos, int64_t blk,
                           const float *__restrict__ t_out, const float *__restrict__ slope,
                           const int *__restrict__ q_idx, const float *__restrict__ grad_t,
                           const Synfire &sf, float *__restrict__ tri,
                           int *__restrict__ rend, int *sh) {
    constexpr int kS = kGradPos + 1;
    float *sg = reinterpret_cast<float *>(sh);
    float *su = sg + kGradCh * kS;
    int *sq = reinterpret_cast<int *>(su + kGradCh * kS);
    int *sl = sq + kGradCh * kS;
    const int HoWo = g.Ho * g.Wo;
    const int ntile = (g.C_out + kGradCh - 1) / kGradCh;
    const int tile = static_cast<int>(blk % ntile);
    const int64_t s0 = (blk / ntile) * kGradPos;
    if (threadIdx.x < kGradPos) sl[threadIdx.x] = -1;
    __syncthreads();
    // Only positions through which gradient passes are written (the dW and
    // dt_in kernels read no others); with more than one channel tile their
    // largest q over all channels is found first (by every tile's block).
    const bool tiles = ntile > 1;
    // each thread keeps one position (blockDim is a multiple of kGradPos):
    // its NCHW offset at channel 0, decoded once
    const int pl = static_cast<int>(threadIdx.x) % kGradPos;
    const int cstep = static_cast<int>(blockDim.x) / kGradPos;
    const bool pos_ok = s0 + pl < n_pos;
    int64_t obase = 0;
    if (pos_ok) {
        const int si = static_cast<int>(s0 + pl);  // B * Ho * Wo < 2^31 (checked at the boundary)
        const int b = si / HoWo;
        obase = static_cast<int64_t>(b) * g.C_out * HoWo + (si - b * HoWo);
    }
    if (tiles) {
        if (pos_ok) {
            // four channels per pass, their loads issued together
            for (int c4 = static_cast<int>(threadIdx.x) / kGradPos; c4 < g.C_out; c4 += 4 * cstep) {
                int q[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int co = c4 + u * cstep;
                    q[u] = (co < g.C_out) ? q_idx[obase + static_cast<int64_t>(co) * HoWo] : -1;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (q[u] >= 0) {
                        const int64_t o = obase + static_cast<int64_t>(c4 + u * cstep) * HoWo;
                        float gt = grad_t[o];
                        if (sf.on) gt += synfire_dt(sf, t_out[o]);
                        if (gt != 0.f) atomicMax(&sl[pl], min(q[u], C.M));
                    }
                }
            }
        }
        __syncthreads();
    }
    {
        // a thread's kCh channels of its position (256 threads: 16 positions
        // x 4 channel rows): each load stage is issued for all of them before
        // the next, so the dependent loads (q, then the upstream gradient,
        // then the spike time and slope) overlap across channels
        constexpr int kCh = kGradCh * kGradPos / 256;
        const int c0 = tile * kGradCh;
        const int cl0 = static_cast<int>(threadIdx.x) / kGradPos;
        int64_t o[kCh];
        int q[kCh];
        float gt[kCh];
        // with channel tiles the pass above found whether any channel of the
        // position passes gradient; a position without writes nothing
        const bool live = pos_ok && (!tiles || sl[pl] >= 0);
#pragma unroll
        for (int u = 0; u < kCh; ++u) {
            const int co = c0 + cl0 + u * cstep;
            o[u] = obase + static_cast<int64_t>(co) * HoWo;
            q[u] = (co < g.C_out && live) ? q_idx[o[u]] : -1;
        }
#pragma unroll
        for (int u = 0; u < kCh; ++u) gt[u] = (q[u] >= 0) ? grad_t[o[u]] : 0.f;  // silent: no load
#pragma unroll
        for (int u = 0; u < kCh; ++u) {
            GradTriple gp{0.f, 0.f, -1};
            if (q[u] >= 0) {
                // the spike time only where it is used (no gradient: no load)
                const float t = (sf.on || gt[u] != 0.f) ? t_out[o[u]] : 0.f;
                float gu = gt[u];
                if (sf.on) gu += synfire_dt(sf, t);
                if (gu != 0.f) gp = grad_triple(C, t, slope[o[u]], q[u], gu);
            }
            const int cl = cl0 + u * cstep;
            sg[cl * kS + pl] = gp.gK;
            su[cl * kS + pl] = gp.gE;
            sq[cl * kS + pl] = gp.q;
            if (!tiles && gp.q >= 0) atomicMax(&sl[pl], gp.q);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < kGradPos * kGradCh; e += blockDim.x) {
            const int pw = e / kGradCh, cl = e % kGradCh;
            const int co = c0 + cl;
            const int64_t sp = s0 + pw;
            if (co < g.C_out && sp < n_pos && sl[pw] >= 0) {
                float *d = tri + sp * 3 * g.C_out + co;
                d[0] = sg[cl * kS + pw];
                d[g.C_out] = su[cl * kS + pw];
                d[2 * g.C_out] = __int_as_float(sq[cl * kS + pw]);
            }
        }
        __syncthreads();
    }
    if (rend && tile == 0 && threadIdx.x < kGradPos && s0 + threadIdx.x < n_pos) {
        const int qm = sl[threadIdx.x];
        rend[s0 + threadIdx.x] = qm < 0 ? -1 : min(rows_of(C) - 2, qm + 1);
    }
}

// Dead-neuron term of output channel co: dq[co] = -gamma_q * scale * (number
// of silent (b, position) outputs of the channel); integer counts, so the
// block sum is exact.
__device__ void dead_channel_block(const ConvGeom &g, int64_t B, const int *__restrict__ q_idx,
                                   const Synfire &sf, int co, int *sh) {
    const int HoWo = g.Ho * g.Wo;
    const int64_t n = B * HoWo;
    int cnt = 0;
    for (int64_t e = threadIdx.x; e < n; e += blockDim.x) {
        const int64_t b = e / HoWo;
        const int p = static_cast<int>(e % HoWo);
        cnt += (q_idx[(b * g.C_out + co) * HoWo + p] < 0) ? 1 : 0;
    }
    sh[threadIdx.x] = cnt;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if (static_cast<int>(threadIdx.x) < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) sf.dq[co] = -(sf.gq * sf.scale * static_cast<float>(sh[0]));
}

// dt_in of the raw inputs of cell row cr, slots [s0, s0 + ns) of its
// cell-major order (kGatherSlots at most; a block per slice). Each input sums
// its partials P[cell][entry][slot] (entry = (ky, tap group, tile)) over the
// (ky, tap group)s with a position that passes gradient (the ones written); the
// sums are staged in LDS, and the slice is written in NCHW order, so
// consecutive threads read and write consecutive addresses. A cell row without
// events, or none of whose output rows passes gradient, writes zeros at once.
constexpr int kGatherSlots = 4096;
struct ConvGatherArgs { const int *cr_live, *rend; const float *P; int kwt, kg, n_tile; };

__device__ void dt_gather_block(const ConvGeom &g, const ConvGatherArgs &a,
                                float *__restrict__ dt_in, int cr, int s0, float *buf) {
    const int per = g.Wp * g.PC;
    const int ns = min(kGatherSlots, per - s0);
    const int b = cr / g.Hp, py = cr % g.Hp;
    // the kernel rows ky (bit mask) whose output row exists and passes gradient
    unsigned kys = 0;
    if (a.cr_live[cr])
        for (int ky = 0; ky < g.KH; ++ky) {
            const int y = py + g.pad - ky, oy = y / g.stride;
            if (y < 0 || oy * g.stride != y || oy >= g.Ho) continue;
            bool any = false;
            for (int x = threadIdx.x; x < g.Wo; x += blockDim.x)
                any = any || a.rend[(static_cast<int64_t>(b) * g.Ho + oy) * g.Wo + x] >= 0;
            if (__syncthreads_or(any)) kys |= 1u << ky;
        }
    if (kys == 0) {
        for (int t = threadIdx.x; t < per; t += blockDim.x) {
            int slot;
            const int64_t dst = cell_row_input(g, b, py, t, slot);
            if (slot >= s0 && slot < s0 + ns) dt_in[dst] = 0.f;
        }
        return;
    }
    const int entries = g.KH * a.kg * a.n_tile;
    for (int t = threadIdx.x; t < ns; t += blockDim.x) {
        const int slot = s0 + t;
        const int px = fdiv(slot, g.dv_pc), j = slot - px * g.PC;
        const float *pc = a.P + (static_cast<int64_t>(cr) * g.Wp + px) * entries * g.PC + j;
        float acc = 0.f;
        for (int ky = 0; ky < g.KH; ++ky) {
            if (!((kys >> ky) & 1u)) continue;
            const int *rr = a.rend + (static_cast<int64_t>(b) * g.Ho + (py + g.pad - ky) / g.stride) * g.Wo;
            for (int kg = 0; kg < a.kg; ++kg) {
                // the group's first tap meets position x / stride (one-tap
                // groups), or its taps meet positions x - kwt + 1 .. x
                const int x = px + g.pad - kg * a.kwt, ox = x / g.stride;
                bool on = false;
                if (a.kwt == 1)
                    on = x >= 0 && ox * g.stride == x && ox < g.Wo && rr[ox] >= 0;
                else
                    for (int i = 0; i < a.kwt; ++i)
                        on = on || (x - i >= 0 && x - i < g.Wo && rr[x - i] >= 0);
                if (!on) continue;
                for (int ti = 0; ti < a.n_tile; ++ti)
                    acc += pc[static_cast<int64_t>((ky * a.kg + kg) * a.n_tile + ti) * g.PC];
            }
        }
        buf[t] = acc;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < per; t += blockDim.x) {
        int slot;
        const int64_t dst = cell_row_input(g, b, py, t, slot);
        if (slot >= s0 && slot < s0 + ns) dt_in[dst] = buf[slot - s0];
    }
}

// dW and the dt_in partials of one layer (dstd_back.h). A block walks output
// rows (b, oy) that pass gradient, position by position; its waves share the
// positions' G tables and own one kernel row ky, KWT neighbouring taps of it
// and TJ input channels each. At step n the table of position ox = n is new,
// and a wave's cell px = n stride - pad + kx0 meets the KWT tables n, n - 1, ...
// at once (stride 1): its events are read once and its inputs' lane sums taken
// once for KWT taps. The waves write the next position's table meanwhile, into a
// ring, one barrier per step. KWT = 1 (other strides, 1-wide kernels, and grids
// whose ring would not fit) gives every tap its own waves.
// Only the runs of steps whose tables include one with gradient are walked (a
// row's positions without gradient further than KWT from one with it cost
// nothing); inside a run a position without gradient is a table of zeros, so a
// tap needs no test of its own. Tables reach the row's largest rend.
// dW: partial sums part[z][co][k * C_in + ci] per split z of the rows. dt_in:
// P[cell][entry][slot], entry = (ky, tap group, channel tile of the launch),
// written for the walked cells whose row has events; the gather adds the
// entries. Further launches (more tiles than entries fit) add to theirs, in
// order.
// Against the forms before it (dW with lanes = inputs and G gathered from LDS;
// dt_in with a weight row loaded and a wave reduced per (record, position)):
// a 64 -> 64 channel 32 x 32 layer, batch 64, M = 32: 2.10 ms -> 0.77 ms; with its
// set-up and sums 2.33 -> 0.87 ms. dW alone has conv_dw_kernel.
struct ConvBackArgs {
    int n_rows, rows_per_split;  // output rows (b, oy)
    int cpt, n_chunk;        // input-channel chunks per (ky, tap group); chunks in all
    int kg;                  // tap groups per kernel row
    int tile0, n_tile, add;  // channel tiles tile0 .. + n_tile - 1; add to P
    const float *tri;
    const int *rend, *cr_live;
    const float *ev, *Wt;
    float *P, *part;
    int *zlive;
};
constexpr int kBackWaves = 12;
constexpr int kBackRowList = 256;  // output rows listed at a time

// G tables: those of a step and the next one's
constexpr int back_ring(int kwt) { return kwt == 1 ? 2 : 4; }

// What a wave of conv_back_kernel leaves out: its taps kx0 .. kx0 + taps - 1 of
// kernel row ky with an infinite or NaN weight to one of channels co0 .. co0 + nco
// - 1, each added to the input's entry where the tap's own position passes gradient
// to the input's event row. By one wave, input by input, from memory.
__device__ __forceinline__ void odd_weights(const LifConst &C, const ConvGeom &g, const ConvBackArgs &a,
                                         const float2 *tab, int r_lo, int r_hi, int ky, int kx0, int taps,
                                         int ci0, int nj, int co0, int nco, int entries, int entry) {
    const int lane = threadIdx.x & (kWave - 1);
    __threadfence_block();  // the entries that the other lanes wrote
    for (int x = 0; x < nj * taps; ++x) {
        const int kx = kx0 + x % taps, ci = ci0 + x / taps;
        const float *wp = a.Wt + (static_cast<int64_t>(ky * g.KW + kx) * g.C_in + ci) * g.C_out;
        bool bad = false;
        for (int c = co0 + lane; c < min(co0 + nco, g.C_out); c += kWave) bad = bad || !(fabsf(wp[c]) < INFINITY);
        if (!__any(bad)) continue;
        for (int s = r_lo * g.Wo; s < r_hi * g.Wo; ++s) {
            const int rw = s / g.Wo, b = rw / g.Ho;
            const int py = (rw - b * g.Ho) * g.stride - g.pad + ky, px = (s - rw * g.Wo) * g.stride - g.pad + kx;
            const int last = a.rend[s];
            if (last < 0 || py < 0 || py >= g.Hp || px < 0 || px >= g.Wp || !a.cr_live[b * g.Hp + py]) continue;
            const int64_t cell = (static_cast<int64_t>(b) * g.Hp + py) * g.Wp + px;
            for (int d = 0; d < g.P; ++d) {
                const float *ev = a.ev + (cell * g.P + d) * kEvFields * g.C_in + ci;
                const int r = __float_as_int(ev[0]);
                if (r < 0 || r > last) continue;
                const float dL = ev[3 * g.C_in], dR = ev[4 * g.C_in];
                float v = 0.f;
                for (int c = co0 + lane; c < min(co0 + nco, g.C_out); c += kWave) {
                    if (fabsf(wp[c]) < INFINITY) continue;
                    const float *t = a.tri + static_cast<int64_t>(s) * 3 * g.C_out + c;
                    const int q = __float_as_int(t[2 * g.C_out]);
                    auto at = [&](int row) {  // as g_rows writes it
                        const float2 e = tab[q + C.M + 3 - row];
                        return row >= 1 && q >= row - 1 ? fmaf(t[0], e.x, t[g.C_out] * e.y) : 0.f;
                    };
                    v += wp[c] * fmaf(dL, at(r), dR * at(r + 1));
                }
                for (int o = kWave / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o);
                if (lane == 0) a.P[(cell * entries + entry) * g.PC + d * g.C_in + ci] += v;
            }
        }
    }
}

template <int KWT, int NT, int TJ, bool DW, bool DT>
__global__ __launch_bounds__(kBackWaves * kWave) void conv_back_kernel(LifConst C, ConvGeom g,
                                                                       ConvBackArgs a) {
    constexpr int kG = TJ / kBackGroup;
    constexpr int kRow = NT * kWave;
    constexpr int kRing = back_ring(KWT);
    extern __shared__ float gs[];  // G [kRing][R][kRow], pairs (a_d, k_d)
    __shared__ int row_top[kBackRowList];  // largest rend of each listed row
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int nw = static_cast<int>(blockDim.x) >> 6;
    const int z = blockIdx.y;
    const int tile = a.tile0 + static_cast<int>(blockIdx.z);
    const int r_lo = z * a.rows_per_split;
    const int r_hi = min(a.n_rows, r_lo + a.rows_per_split);
    // the largest rend of rows rl .. rl + nl - 1 (rows of -1 are skipped);
    // returns whether any passes gradient
    auto list_rows = [&](int rl, int nl) {
        bool any = false;
        for (int l = wave; l < nl; l += nw) {
            int m = -1;
            for (int x = lane; x < g.Wo; x += kWave)
                m = max(m, a.rend[static_cast<int64_t>(rl + l) * g.Wo + x]);
#pragma unroll
            for (int o = kWave / 2; o >= 1; o >>= 1) m = max(m, __shfl_xor(m, o));
            if (lane == 0) row_top[l] = m;
            any = any || m >= 0;
        }
        return __syncthreads_or(any) != 0;
    };
    // the first rows with gradient; a split without any writes no partials (the
    // reduction skips it)
    int rl = r_lo;
    bool any_row = false;
    for (; rl < r_hi; rl += kBackRowList) {
        any_row = list_rows(rl, min(kBackRowList, r_hi - rl));
        if (any_row) break;
        __syncthreads();  // the list is rewritten
    }
    if (DW && threadIdx.x == 0 && blockIdx.x == 0 && tile == 0) a.zlive[z] = any_row;
    if (!any_row) return;
    const int R = rows_of(C);
    const int ts = R * kRow;  // floats of a G table
    float2 *tab = reinterpret_cast<float2 *>(gs + kRing * ts);
    // this wave's chunk: kernel row ky, taps kx0 .. kx0 + KWT - 1, channels
    // ci0 .. ci0 + nj - 1
    const int chunk = static_cast<int>(blockIdx.x) * nw + wave;
    const bool mine = chunk < a.n_chunk;
    const int tg = mine ? chunk / a.cpt : 0;
    const int ci0 = (mine ? chunk - tg * a.cpt : 0) * TJ;
    const int nj = mine ? min(TJ, g.C_in - ci0) : 0;
    const int ky = tg / a.kg, kx0 = (tg - ky * a.kg) * KWT;
    const int co = tile * kRow + NT * lane;  // this lane's channels co .. co + NT - 1
    for (int k = threadIdx.x; k < kRing * kRow; k += blockDim.x) gs[(k / kRow) * ts + k % kRow] = 0.f;
    g_table_fill(C, tab);
    // channels past C_out: weight 0 and no gradient
    float acc[kG][kBackGroup][KWT][NT], w[kG][kBackGroup][KWT][NT];
    static_for<kG>([&](auto h) {
        static_for<kBackGroup>([&](auto j) {
            static_for<KWT>([&](auto i) {
                static_for<NT>([&](auto c) {
                    acc[h][j][i][c] = 0.f;
                    w[h][j][i][c] = 0.f;
                    if constexpr (DT) {
                        const int ci = min(ci0 + h * kBackGroup + j, g.C_in - 1);
                        const int k = ky * g.KW + kx0 + i;
                        if (kx0 + i < g.KW && co + c < g.C_out)
                            w[h][j][i][c] = a.Wt[static_cast<int64_t>(k * g.C_in + ci) * g.C_out + co + c];
                    }
                });
            });
        });
    });
    // loaded before the loops (a load still pending at their entry would make
    // every step wait for its own prefetches)
    static_for<kG>([&](auto h) {
        static_for<kBackGroup>([&](auto j) {
            static_for<KWT>([&](auto i) {
                static_for<NT>([&](auto c) { settle(w[h][j][i][c]); });
            });
        });
    });
    // Infinite and NaN weights: a table without gradient is multiplied like any
    // other, and 0 times such a weight would reach inputs that no position passes
    // gradient to. A wave that has any takes them as 0 and adds them at the end
    // (odd_weights). (One tap per wave visits only positions with gradient.)
    bool odd = false;
    if constexpr (DT && KWT > 1) {
        static_for<TJ>([&](auto j) {
            static_for<KWT>([&](auto i) {
                static_for<NT>([&](auto c) {
                    odd = odd || !(fabsf(w[j / kBackGroup][j % kBackGroup][i][c]) < INFINITY);
                });
            });
        });
        odd = __any(odd);
        if (odd)
            static_for<TJ>([&](auto j) {
                static_for<KWT>([&](auto i) {
                    static_for<NT>([&](auto c) {
                        float &x = w[j / kBackGroup][j % kBackGroup][i][c];
                        x = fabsf(x) < INFINITY ? x : 0.f;
                    });
                });
            });
    }
    // gradient triples of the position whose triples start at p (scalar)
    unsigned tri_o[NT];
    bool ch_ok[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        tri_o[c] = static_cast<unsigned>(min(co + c, g.C_out - 1));
        ch_ok[c] = co + c < g.C_out;
    }
    auto load_tri = [&](const float *p) {
        GTri<NT> t;
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            t.gK[c] = p[tri_o[c]];
            t.gE[c] = (p + g.C_out)[tri_o[c]];
            t.q[c] = __float_as_int((p + 2 * g.C_out)[tri_o[c]]);
        }
        return t;
    };
    auto write_rows = [&](GTri<NT> t, int top, int slot) {
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            t.gK[c] = ch_ok[c] ? t.gK[c] : 0.f;
            t.gE[c] = ch_ok[c] ? t.gE[c] : 0.f;
            t.q[c] = ch_ok[c] ? t.q[c] : -1;
        }
        g_rows<NT>(C.M, tab, t, top, wave, nw, gs + slot * ts + NT * lane);
    };
    // a table without gradient: rows 1 .. top + 1
    auto zero_rows = [&](int top, int slot) {
        float *zt = gs + slot * ts + kRow;
        for (int k = threadIdx.x; k < (top + 1) * kRow; k += blockDim.x) zt[k] = 0.f;
    };
    // steps of a row: positions 0 .. Wo - 1, and (KWT > 1) the cells after them
    const int steps = (KWT == 1) ? g.Wo : min(g.Wp + g.pad, g.Wo + KWT - 1);
    const int entries = g.KH * a.kg * a.n_tile;
    const int entry = tg * a.n_tile + static_cast<int>(blockIdx.z);
    // lane 8j + h of a partial store holds input 8h + j of the wave
    const int p_off = (lane & 7) < kG ? 4 * ((lane & 7) * kBackGroup + (lane >> 3)) : 1 << 30;
    const EvOffs<TJ> ev_o = ev_offs<TJ>(g.C_in, max(nj, 1), lane);
    const int64_t ev_cell = static_cast<int64_t>(kEvFields) * g.PC, p_cell = static_cast<int64_t>(entries) * g.PC;
    while (true) {
        const int nl = min(kBackRowList, r_hi - rl);
        for (int l = 0; l < nl; ++l) {
            const int top = uniform(row_top[l]);
            if (top < 0) continue;  // block-uniform
            const int rw = rl + l;
            const int b = rw / g.Ho, py = (rw - b * g.Ho) * g.stride - g.pad + ky;
            const int cr = b * g.Hp + py;
            const bool live = mine && py >= 0 && py < g.Hp && *as_const(a.cr_live + (py >= 0 && py < g.Hp ? cr : 0));
            const float *ev_row = a.ev + static_cast<int64_t>(live ? cr : 0) * g.Wp * ev_cell + ci0;
            float *p_row = a.P + static_cast<int64_t>(live ? cr : 0) * g.Wp * p_cell + static_cast<int64_t>(entry) * g.PC + ci0;
            // rend of position x, held 64 positions at a time (lane = x mod 64)
            int er = 0, er0 = -1;
            auto rend_at = [&](int x) {
                if (x >= g.Wo) return -1;
                if ((x >> 6) != er0) {
                    er0 = x >> 6;
                    er = a.rend[static_cast<int64_t>(rw) * g.Wo + min(er0 * kWave + lane, g.Wo - 1)];
                }
                return __builtin_amdgcn_readlane(er, x & (kWave - 1));
            };
            int n = 0;
            while (true) {
                // the run's first step: the next position with gradient
                int e[KWT];  // rend of the step's tables
                static_for<KWT>([&](auto i) { e[i] = -1; });
                for (; n < g.Wo && (e[0] = rend_at(n)) < 0; ++n) {}
                if (n >= g.Wo || n >= steps) break;
                // items: (step n, raw pixel d), the events of one, and the triples
                // of the position after its step, loaded during the one before.
                // Loads and the store are issued whether they are needed or not
                // (addresses clamped, the store's range empty): a wait then counts
                // what was issued since, and prefetches stay in flight
                int d = 0, px = n * g.stride - g.pad + kx0, r_end = e[0];
                const float *tri_p = a.tri + (static_cast<int64_t>(rw) * g.Wo + n) * 3 * g.C_out;
                auto here = [&](int x) { return live && x >= 0 && x < g.Wp; };
                auto item_ev = [&](int x, int dd) {
                    return ev_load<TJ>(ev_row + min(max(x, 0), g.Wp - 1) * ev_cell + dd * kEvFields * g.C_in, ev_o);
                };
                EvRegs<TJ> ev[2];
                ev[0] = item_ev(px, 0);
                write_rows(load_tri(tri_p), top, n & (kRing - 1));
                static_for<KWT - 1>([&](auto i) { zero_rows(top, (n - 1 - i) & (kRing - 1)); });
                __syncthreads();
                bool more = true;
                auto item = [&](auto par) {
                    constexpr int p = par;
                    const bool last_d = d + 1 == g.P;
                    ev[p ^ 1] = item_ev(last_d ? px + g.stride : px, last_d ? 0 : d + 1);
                    const GTri<NT> t_n = load_tri(tri_p + (n + 1 < g.Wo ? 3 * g.C_out : 0));
                    float tot[kG];
                    static_for<kG>([&](auto h) { tot[h] = 0.f; });
                    if (here(px)) {
                        const float *gl[KWT];
                        static_for<KWT>([&](auto i) { gl[i] = gs + ((n - i) & (kRing - 1)) * ts + NT * lane; });
                        const unsigned act = static_cast<unsigned>(__ballot(
                            lane < nj && static_cast<unsigned>(__float_as_int(ev[p].e[0])) <= static_cast<unsigned>(r_end)));
                        static_for<kG>([&](auto h) {
                            if ((act >> (h * kBackGroup)) & 0xffu)
                                tot[h] = back_group<NT, KWT, TJ, h, DW, DT>(gl, lane, act, ev[p], w[h], acc[h]);
                        });
                    }
                    if constexpr (DT) {
                        float v = tot[0];
                        static_for<kG>([&](auto x) { v = ((lane & 7) == x) ? tot[x] : v; });
                        float *out = p_row + min(max(px, 0), g.Wp - 1) * p_cell + d * g.C_in;
                        const __amdgpu_buffer_rsrc_t pr = make_rsrc(out, here(px) ? static_cast<uint32_t>(nj) * 4u : 0u);
                        if (a.add) v += BufLoad<float>::get(pr, p_off, 0);
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), pr, p_off, 0, 0);
                    }
                    ++d;
                    if (last_d) {
                        ++n;
                        static_for<KWT - 1>([&](auto i) { e[KWT - 1 - i] = e[KWT - 2 - i]; });
                        e[0] = rend_at(n);
                        r_end = e[0];
                        static_for<KWT>([&](auto i) { r_end = max(r_end, e[i]); });
                        more = n < steps && r_end >= 0;
                        if (more) {
                            if (KWT == 1 || e[0] >= 0) write_rows(t_n, top, n & (kRing - 1));
                            else zero_rows(top, n & (kRing - 1));
                        }
                        tri_p += 3 * g.C_out;
                        px += g.stride;
                        d = 0;
                        __syncthreads();
                    }
                };
                while (true) {
                    item(std::integral_constant<int, 0>{});
                    if (!more) break;
                    item(std::integral_constant<int, 1>{});
                    if (!more) break;
                }
            }
        }
        rl += kBackRowList;
        if (rl >= r_hi) break;
        __syncthreads();  // the list's readers
        list_rows(rl, min(kBackRowList, r_hi - rl));
    }
    if constexpr (DW) {
        const int NJ = g.KH * g.KW * g.C_in;
        static_for<NT>([&](auto c) {
            if (co + c >= g.C_out) return;
            static_for<KWT>([&](auto i) {
                if (kx0 + i >= g.KW) return;
                float *out = a.part + (static_cast<int64_t>(z) * g.C_out + co + c) * NJ +
                             (ky * g.KW + kx0 + i) * g.C_in + ci0;
                static_for<TJ>([&](auto jj) {
                    if (jj < nj) out[jj] = acc[jj / kBackGroup][jj % kBackGroup][i][c];
                });
            });
        });
    }
    if constexpr (DT && KWT > 1) {
        if (odd) odd_weights(C, g, a, tab, r_lo, r_hi, ky, kx0, min(KWT, g.KW - kx0), ci0, nj, tile * kRow, kRow, entries, entry);
    }
}

// dW alone with lanes = (tap, input) pairs: a block takes 256 of a layer's pairs
// and TI channels, whose sums stay in registers over its output rows, position by
// position. The contraction above gives an input a wave and its taps a table read
// each; where a kernel row has few inputs (a first layer's one to three) a wave
// spends its position on one of them, and without dt_in nothing covers the reads.
// Here lanes whose inputs have the same event row read the same words of it at
// once. Positions without gradient are skipped 64 at a time; the next position's
// table goes to the other of two meanwhile, its triples and the next events are on
// their way. Same sums in the same order.
constexpr int kDwPairs = 256;

template <int TI>
__global__ __launch_bounds__(kDwPairs) void conv_dw_kernel(LifConst C, ConvGeom g, ConvBackArgs a) {
    constexpr int kRow = TI + 4;            // a row's floats: 16-byte reads
    constexpr int kParts = kWave / TI;      // rows that a wave writes at a time
    extern __shared__ float gs[];  // G [2][R + 1][kRow], pairs (a_d, k_d)
    const int R = rows_of(C);
    const int ts = (R + 1) * kRow;
    float2 *tab = reinterpret_cast<float2 *>(gs + 2 * ts);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int z = blockIdx.y;
    const int s_lo = z * a.rows_per_split * g.Wo;
    const int s_hi = min(a.n_rows, (z + 1) * a.rows_per_split) * g.Wo;
    // the split's positions that pass gradient, in order (-1: none left), and the
    // last event row that meets it there
    int base = s_lo - kWave, er = -1;
    uint64_t mask = 0;
    auto next = [&](int &top) {
        while (mask == 0) {
            if (s_hi - base <= kWave) return -1;
            base += kWave;
            er = base + lane < s_hi ? a.rend[base + lane] : -1;
            mask = __ballot(er >= 0);
        }
        const int bit = __builtin_ctzll(mask);
        mask &= mask - 1;
        top = __builtin_amdgcn_readlane(er, bit);
        return base + bit;
    };
    int top0 = -1, top1 = -1, top2 = -1;
    int s0 = next(top0);
    // (a split without any writes no partials: the reduction skips it)
    if (threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.z == 0) a.zlive[z] = s0 >= 0;
    if (s0 < 0) return;  // block-uniform
    int s1 = next(top1);
    const int NJ = g.KH * g.KW * g.C_in;
    const int jj = static_cast<int>(blockIdx.x) * kDwPairs + static_cast<int>(threadIdx.x);
    const bool j_ok = jj < NJ;
    const int k = (j_ok ? jj : 0) / g.C_in, ci = (j_ok ? jj : 0) - k * g.C_in;
    const int ky = k / g.KW, kx = k - ky * g.KW;
    const int c0 = static_cast<int>(blockIdx.z) * TI;
    // row 0 holds no grid point; rows R - 1 and R are zero for inputs without
    // events (or past the last spike)
    for (int t = threadIdx.x; t < 2 * kRow; t += kDwPairs) {
        float *q = gs + (t / kRow) * ts + t % kRow;
        q[0] = 0.f;
        q[(R - 1) * kRow] = 0.f;
        q[R * kRow] = 0.f;
    }
    g_table_fill(C, tab);
    float acc[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i) acc[i] = 0.f;
    const int cl = lane % TI, part = lane / TI;
    const unsigned co = static_cast<unsigned>(min(c0 + cl, g.C_out - 1));
    const bool c_ok = c0 + cl < g.C_out;
    auto load_tri = [&](int s) {
        const float *p = a.tri + static_cast<int64_t>(s) * 3 * g.C_out;
        GTri<1> t;
        t.gK[0] = p[co];
        t.gE[0] = (p + g.C_out)[co];
        t.q[0] = __float_as_int((p + 2 * g.C_out)[co]);
        return t;
    };
    auto write_tri = [&](GTri<1> t, int top, int slot) {
        t.gK[0] = c_ok ? t.gK[0] : 0.f;
        t.gE[0] = c_ok ? t.gE[0] : 0.f;
        t.q[0] = c_ok ? t.q[0] : -1;
        g_rows<1, kRow>(C.M, tab, t, top, wave * kParts + part, kDwPairs / TI, gs + slot * ts + cl);
    };
    // this lane's cell at position s (-1: outside, or no events in its cell row)
    struct Ev { int row; float L, R; };
    const int HoWo = g.Ho * g.Wo;
    auto cell_at = [&](int s, int &live) {
        const int b = s / HoWo, p = s - b * HoWo, oy = p / g.Wo, ox = p - oy * g.Wo;
        const int py = oy * g.stride - g.pad + ky, px = ox * g.stride - g.pad + kx;
        const bool in = j_ok && py >= 0 && py < g.Hp && px >= 0 && px < g.Wp;
        const int cr = in ? b * g.Hp + py : 0;
        live = in ? a.cr_live[cr] : 0;
        return static_cast<int64_t>(cr) * g.Wp + (in ? px : 0);
    };
    auto load_ev = [&](int64_t cell, int d) {
        const float *p = a.ev + (cell * g.P + d) * kEvFields * g.C_in + ci;
        return Ev{__float_as_int(p[0]), p[g.C_in], p[2 * g.C_in]};
    };
    int live0 = 0, live1 = 0;
    int64_t cell0 = cell_at(s0, live0), cell1 = cell0;
    Ev ev = load_ev(cell0, 0);
    write_tri(load_tri(s0), top0, 0);
    GTri<1> tri = load_tri(s1 >= 0 ? s1 : s0);
    __syncthreads();
    for (int cur = 0;; cur ^= 1) {
        const int s2 = s1 >= 0 ? next(top2) : -1;
        if (s1 >= 0) {
            cell1 = cell_at(s1, live1);
            write_tri(tri, top1, cur ^ 1);
            tri = load_tri(s2 >= 0 ? s2 : s1);
        }
        for (int d = 0; d < g.P; ++d) {
            const Ev n = d + 1 < g.P ? load_ev(cell0, d + 1) : load_ev(cell1, 0);
            const bool on = live0 != 0 && static_cast<unsigned>(ev.row) <= static_cast<unsigned>(top0);
            if (__any(on)) {
                const float L = on ? ev.L : 0.f, Rv = on ? ev.R : 0.f;
                const float4 *p = reinterpret_cast<const float4 *>(gs + cur * ts + (on ? ev.row : R - 1) * kRow);
#pragma unroll
                for (int i = 0; i < TI; i += 4) {
                    const float4 x = p[i / 4], y = p[(i + kRow) / 4];
                    acc[i] = fmaf(L, x.x, fmaf(Rv, y.x, acc[i]));
                    acc[i + 1] = fmaf(L, x.y, fmaf(Rv, y.y, acc[i + 1]));
                    acc[i + 2] = fmaf(L, x.z, fmaf(Rv, y.z, acc[i + 2]));
                    acc[i + 3] = fmaf(L, x.w, fmaf(Rv, y.w, acc[i + 3]));
                }
            }
            ev = n;
        }
        if (s1 < 0) break;
        s0 = s1; top0 = top1; cell0 = cell1; live0 = live1;
        s1 = s2; top1 = top2;
        __syncthreads();
    }
    if (!j_ok) return;
    float *out = a.part + (static_cast<int64_t>(z) * g.C_out + c0) * NJ + jj;
#pragma unroll
    for (int i = 0; i < TI; ++i)
        if (c0 + i < g.C_out) out[static_cast<int64_t>(i) * NJ] = acc[i];
}

// dW[co, ci, ky, kx] = (1/P) sum_z part[z][co][k * C_in + ci]. Threads follow
// the partial-sum layout (coalesced reads); a block takes groups of 256 / G
// consecutive entries x G split groups (G from red_groups: more groups where
// there are many splits; at most 512 blocks, each taking every nblk-th entry
// group): group h sums z = h, h + G, ...; the G group sums are added in
// group order (fixed order: deterministic) and written to the [co][ci][ky][kx]
// slot. Splits without gradient-carrying samples wrote no partials and are
// skipped (their sums would be +0, which leaves every partial sum unchanged);
// where no split has any, the block writes the dead-neuron term (or 0) at once.
__host__ __device__ __forceinline__ int red_groups(int nsplit) {
    int G = 8;
    while (G < 64 && G * 16 < nsplit) G *= 2;
    return G;
}

__device__ void dw_reduce_block(const ConvGeom &g, int nsplit, const float *__restrict__ part,
                                const int *__restrict__ zlive, const float *__restrict__ dq,
                                float *__restrict__ dW, int blk, int nblk, float *red) {
    const int KT = g.KH * g.KW;
    const int NJ = KT * g.C_in;
    const int64_t n = static_cast<int64_t>(g.C_out) * NJ;
    const int G = red_groups(nsplit), O = static_cast<int>(blockDim.x) / G;
    const int lo = threadIdx.x % O, h = threadIdx.x / O;
    bool any = false;
    for (int z = threadIdx.x; z < nsplit; z += blockDim.x) any = any || zlive[z] != 0;
    any = __syncthreads_or(any);
    if (!any) {
        // no split carries gradient (the same for every block of the layer):
        // dW is the dead-neuron term or 0, written in dW's own order
        // (coalesced)
        for (int64_t i = static_cast<int64_t>(blk) * blockDim.x + threadIdx.x; i < n;
             i += static_cast<int64_t>(nblk) * blockDim.x)
            dW[i] = dq ? 0.f + dq[i / NJ] : 0.f;
        return;
    }
    // groups of O outputs, nblk blocks apart (block-uniform trip count)
    const int64_t ngrp = (n + O - 1) / O;
    for (int64_t grp = blk; grp < ngrp; grp += nblk) {
        const int64_t src = grp * O + lo;  // [co][k][ci]
        float s = 0.f;
        if (src < n) {
#pragma unroll 8
            for (int z = h; z < nsplit; z += G)
                if (zlive[z]) s += part[static_cast<int64_t>(z) * n + src];
        }
        red[h * O + lo] = s;
        __syncthreads();
        float tot = 0.f;
        if (h == 0)
            for (int q = 0; q < G; ++q) tot += red[q * O + lo];
        __syncthreads();  // red is rewritten by the next group
        if (h == 0 && src < n) {
            const int co = static_cast<int>(src / NJ);
            const int rem = static_cast<int>(src % NJ);
            const int k = rem / g.C_in, ci = rem % g.C_in;
            const float v = tot * g.inv_P;
            dW[(static_cast<int64_t>(co) * g.C_in + ci) * KT + k] = dq ? v + dq[co] : v;
        }
    }
}

// --------------------------------------------------------- fused launches --
// Independent per-call work shares one launch by block role (a launch costs
// several microseconds even when its work is tiny).
// Forward set-up: blocks [0, n_sort) sort cell rows (with ev set, keeping
// the cell-major events for the backward too), the next n_bin bin the raw
// inputs of a direct layer once (bin_block), the next n_ev keep a direct
// layer's cell-major events, the rest lay out WT.
template <typename WT>
__global__ __launch_bounds__(256) void conv_fprep_kernel(LifConst C, ConvGeom g, int n_sort,
                                                         int n_bin, int n_ev, int64_t n_in,
                                                         const float *__restrict__ t_in,
                                                         ConvSorted cs, CellEv ev,
                                                         const WT *__restrict__ W,
                                                         float *__restrict__ Wt) {
    extern __shared__ int sh[];
    const int blk = static_cast<int>(blockIdx.x);
    if (blk < n_sort)
        sort_cell_row(C, g, t_in, cs, ev, blk, sh);
    else if (blk < n_sort + n_bin)
        bin_block(C, n_in, t_in, cs, blk - n_sort);
    else if (blk < n_sort + n_bin + n_ev)
        events_cell_row(C, g, t_in, ev, blk - n_sort - n_bin, reinterpret_cast<float *>(sh));
    else
        weights_block<WT>(g, W, Wt, blk - n_sort - n_bin - n_ev, reinterpret_cast<float (*)[33]>(sh));
}

// Backward set-up: [0, n_cr) cell rows' events, then n_gr blocks of gradient
// triples and per-position gradient rows (rend), n_dq blocks of dead-neuron
// terms (one per channel, synfire terms on) and the WT layout.
template <typename WT>
__global__ __launch_bounds__(256) void conv_bprep_kernel(
    LifConst C, ConvGeom g, int n_cr, int n_gr, int n_dq, const float *__restrict__ t_in,
    CellEv ev, int64_t n_pos, const float *__restrict__ t_out,
    const float *__restrict__ slope, const int *__restrict__ q_idx,
    const float *__restrict__ grad_t, Synfire sf, float *__restrict__ tri,
    int *__restrict__ rend,
    const WT *__restrict__ W, float *__restrict__ Wt) {
    extern __shared__ int sh[];
    // XCD-aware order: neighbouring gradient blocks read the two halves of
    // the same cache lines of the NCHW outputs
    int blk = xcd_block(blockIdx.x, gridDim.x);
    if (blk < n_cr) {
        events_cell_row(C, g, t_in, ev, blk, reinterpret_cast<float *>(sh));
        return;
    }
    blk -= n_cr;
    if (blk < n_gr) {
        grad_block(C, g, n_pos, blk, t_out, slope, q_idx, grad_t, sf, tri, rend, sh);
        return;
    }
    blk -= n_gr;
    if (blk < n_dq) {
        dead_channel_block(g, n_pos / (g.Ho * g.Wo), q_idx, sf, blk, sh);
        return;
    }
    weights_block<WT>(g, W, Wt, blk - n_dq, reinterpret_cast<float (*)[33]>(sh));
}

// Backward finish: [0, n_red) dW split reduction, the rest gathers dt_in
// (nsl blocks per cell row, one per slice of kGatherSlots slots).
__global__ __launch_bounds__(256) void conv_bfin_kernel(ConvGeom g, int n_red, int nsplit,
                                                        const float *__restrict__ part,
                                                        const int *__restrict__ zlive,
                                                        const float *__restrict__ dq,
                                                        float *__restrict__ dW, int nsl,
                                                        ConvGatherArgs ga,
                                                        float *__restrict__ dt_in) {
    static_assert(kGatherSlots >= 256, "the reduction shares the gather's LDS");
    __shared__ float lds[kGatherSlots];
    const int blk = static_cast<int>(blockIdx.x);
    if (blk < n_red) {
        dw_reduce_block(g, nsplit, part, zlive, dq, dW, blk, n_red, lds);
    } else {
        const int t = blk - n_red;
        dt_gather_block(g, ga, dt_in, t / nsl, (t % nsl) * kGatherSlots, lds);
    }
}

// ------------------------------------------------------------ launchers --
// positions per wave of the list forward (its LDS list stays within 30 KB
// per block): 2 for at most 32 channels, 32 event rows and kListMaxRec / 2
// raw inputs per receptive field, else 0 (the chunked walk). One position
// per wave (64-channel tiles) was measured slower than the chunked walk
// (conv9's forward 0.81 against 0.68 ms): with few records per event row
// the row-by-row batches stay short, where the chunked walk's batches run
// across rows.
// the forward bins its inputs itself (no sort) where a receptive field holds
// at most as many raw inputs as a position has lanes (64; 32 with two
// positions per wave)
bool conv_fwd_direct(const ConvGeom &g, int np) {
    return g.KH * g.KW * g.PC <= (np == 2 ? kWave / 2 : kWave);
}

int conv_fwd_list_np(int M, const ConvGeom &g) {
    const int E = g.KH * g.KW * g.PC;
    return (g.C_out <= 32 && M + 2 <= 32 && 2 * E <= kListMaxRec) ? 2 : 0;
}

int conv_sort_lds_bytes(int M, const ConvGeom &g) {
    return ((M + 3) * g.Wp + 256 + sort_stage_floats(M, g) + sort_list_ints(M, g)) *
           static_cast<int>(sizeof(int));
}

hipError_t launch_conv_forward(const LifConst &C, const ConvGeom &g, int64_t B, const void *W,
                               bool bf16, float *Wt, ConvSorted cs, CellEv ev, const float *t_in,
                               float *t_out, float *slope, int *q_idx, hipStream_t st) {
    const int np = conv_fwd_list_np(C.M, g);
    const bool direct = conv_fwd_direct(g, np);
    const bool keep = ev.ev != nullptr;
    // the direct walk bins its inputs itself: no cell-row sort (a keeping
    // call leaves the events for the backward all the same)
    const int n_sort = direct ? 0 : static_cast<int>(B * g.Hp);
    const int n_ev = (direct && keep) ? static_cast<int>(B * g.Hp) : 0;
    // a direct layer on plain input has its raw inputs
    // binned once here, in NCHW order, in the sort's key/L/R arrays (as many
    // slots as raw inputs), and its positions load those events
    const int64_t n_in = B * g.C_in * g.H * g.W;
    const int pre = (direct && g.pool == 1) ? 1 : 0;
    const int n_bin = pre ? static_cast<int>((n_in + kBinPerBlock - 1) / kBinPerBlock) : 0;
    {
        ProfScope prof("conv_fprep", st);
        const unsigned blocks = static_cast<unsigned>(n_sort + n_bin + n_ev + weight_tiles(g));
        const int lds = std::max({n_sort > 0 ? conv_sort_lds_bytes(C.M, g) : 0, kWtLdsBytes,
                                  n_ev > 0 ? events_stage_floats(g) * static_cast<int>(sizeof(float)) : 0});
        if (bf16)
            hipLaunchKernelGGL(conv_fprep_kernel<uint16_t>, dim3(blocks), dim3(256), lds, st, C, g,
                               n_sort, n_bin, n_ev, n_in, t_in, cs, ev, static_cast<const uint16_t *>(W),
                               Wt);
        else
            hipLaunchKernelGGL(conv_fprep_kernel<float>, dim3(blocks), dim3(256), lds, st, C, g,
                               n_sort, n_bin, n_ev, n_in, t_in, cs, ev, static_cast<const float *>(W), Wt);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int64_t n_pos = B * g.Ho * g.Wo;
    constexpr int waves = 4;
    ProfScope prof("conv_fwd", st);
    if (np > 0) {
        const size_t lds =
            static_cast<size_t>(waves) * (list_wave_ints(np * g.KH * g.KW * g.PC) + (direct ? kWave : 0)) *
            sizeof(int);
        dim3 lgrid(static_cast<unsigned>((n_pos + np * waves - 1) / (np * waves)));
#define CFL(KHV, KSV, DV)                                                                         \
    hipLaunchKernelGGL((conv_fwd_list_kernel<KHV, KSV, 2, DV>), lgrid, dim3(waves * kWave), lds,  \
                       st, C, g, n_pos, Wt, cs, t_in, t_out, slope, q_idx, pre)
#define CFL_D(KHV, KSV)                                                   \
    do {                                                                  \
        if (direct) CFL(KHV, KSV, true);                                  \
        else CFL(KHV, KSV, false);                                        \
    } while (0)
#define CFL_K(KHV)                                                        \
    do {                                                                  \
        if (C.kind == kGeneral) CFL_D(KHV, kGeneral);                     \
        else CFL_D(KHV, kAnyKind);                                        \
    } while (0)
        if (g.KH == 1) CFL_K(1);
        else if (g.KH <= 3) CFL_K(3);
        else CFL_K(kConvMaxK);
#undef CFL_K
#undef CFL_D
#undef CFL
        return hipGetLastError();
    }
    dim3 grid(static_cast<unsigned>((n_pos + kFwdWaves - 1) / kFwdWaves),
              static_cast<unsigned>((g.C_out + kWave - 1) / kWave));
#define CFW(KHV, KSV, DV)                                                                        \
    hipLaunchKernelGGL((conv_fwd_kernel<KHV, KSV, DV>), grid, dim3(kFwdWaves * kWave), 0, st, C, \
                       g, n_pos, Wt, cs, t_in, t_out, slope, q_idx, pre)
#define CFW_D(KHV, KSV)                                                   \
    do {                                                                  \
        if (direct) CFW(KHV, KSV, true);                                  \
        else CFW(KHV, KSV, false);                                        \
    } while (0)
#define CFW_K(KHV)                                                        \
    do {                                                                  \
        if (C.kind == kGeneral) CFW_D(KHV, kGeneral);                     \
        else CFW_D(KHV, kAnyKind);                                        \
    } while (0)
    if (g.KH == 1) CFW_K(1);
    else if (g.KH <= 3) CFW_K(3);
    else CFW_K(kConvMaxK);
#undef CFW_K
#undef CFW_D
#undef CFW
    return hipGetLastError();
}

// The shape of the backward contraction: KWT = 3 taps per wave (kernels wider
// than 1 at stride 1; a 5- or 7-wide kernel row takes 2 or 3 such groups) or 1,
// NT = 1 or 2 channels per lane (2 only past 64), each as far as their G tables fit
// kBackLds, TJ = 8 or 16 inputs per wave (KWT NT TJ <= 48 pairs per lane: their
// sums and weights are two thirds of the 168 registers that three waves per SIMD
// leave), up to 12, 8 or 4 waves per block, and splits of the output
// rows (at most 4096, 64 MiB of partial sums), by the time they predict. A block
// takes a fixed start and its weights, and per position its barrier, its share of
// the table's rows, and per raw pixel a fixed part and its wave's inputs, in cycles
// of a wave alone on its CU; waves that share a CU slow each other down by kShare
// each, and a block of w waves needs ceil(w / 4) on every SIMD (blocks of three to
// six waves fill a CU less than their waves would). Partial sums and dt_in entries
// are written and read once more.
// The constants are a fit to 2,700 timed shapes of 98 layers: batch 4 to 128, 1 to
// 256 channels in, 8 to 256 out, maps of 4 to 32, kernels 1, 3 and 5, strides,
// pooling, M 8 to 128, dW alone, dt_in alone and both. The predicted best is 2 %
// above the timed best on average; one fixed shape per layer with at least 16
// positions per split was 66 % above it: 16 -> 32, 8 x 8, batch 16, both gradients
// 71.9 -> 39 us, 53 -> 101, 10 x 10 pooled, 1 x 1, batch 4 177 -> 42,
// 32 -> 32, 28 x 28, batch 128 1007 -> 743.
constexpr int kBackLds = 152 * 1024;
constexpr int kConvCUs = 256;
constexpr int kConvMaxSplit = 4096;

static int conv_back_lds(int M, int kwt, int nt) {
    return back_ring(kwt) * (M + 3) * nt * kWave * 4 + g_table_len(M) * static_cast<int>(sizeof(float2));
}

// waves per SIMD that the kernel's registers leave
static int conv_back_occupancy(int kwt, int pairs, bool dw, bool dt) {
    if (dw && dt) return pairs > 24 ? 3 : pairs > 8 ? 4 : 6;
    if (dw) return pairs > 32 ? 4 : pairs > 16 ? 5 : 7;
    return pairs > 32 ? 3 : pairs > 16 ? 4 : kwt == 1 && pairs <= 8 ? 7 : 6;
}

// kwt and nt, rows_per_split: given, or 0
static ConvBackPlan conv_back_search(const ConvGeom &g, int64_t B, int M, bool dw, bool dt, int kwt_given,
                                     int nt_given, int rows_given) {
    constexpr double kStart = 2720., kStartPair = 294., kStep = 750., kRow = 79., kItem = 831., kInput = 49.5;
    constexpr double kPerUs = 2400., kShare = 0.0346, kPartUsPerMB = 1.92, kPartUsPerSplit = 0.0134, kEntryUsPerMB = 0.76;
    const double k_pair = (dw && dt) ? 38. : dt ? 33.7 : 10.1;
    const int64_t nw = static_cast<int64_t>(g.KH) * g.KW * g.C_in * g.C_out;
    const int rows = static_cast<int>(std::max<int64_t>(1, B * g.Ho));
    const double dw_mb = 4e-6 * static_cast<double>(nw);
    const double in_mb = 4e-6 * static_cast<double>(B * g.Hp) * g.Wp * g.PC;
    int most_split = std::min(rows, kConvMaxSplit);
    if (dw) most_split = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(most_split, (int64_t{64} << 20) / (4 * std::max<int64_t>(nw, 1)))));
    // (dW alone of a layer whose pairs are one block of conv_dw_kernel needs 1024
    // splits, of 16 positions at least, to fill the chip: 1 -> 32, 5 x 5, 28 x 28, batch 64 250 -> 122 us, both
    // gradients 324 -> 360)
    const int least_split =
        (dw && g.KH * g.KW * g.C_in <= kDwPairs && g.C_out <= kWave)
            ? static_cast<int>(std::max<int64_t>(1, std::min<int64_t>({1024, most_split, static_cast<int64_t>(rows) * g.Wo / 16}))) : 1;
    ConvBackPlan p{};
    double best = -1.;
    for (int kwt = 3; kwt >= 1; kwt -= 2) {
        if (kwt_given ? kwt != kwt_given : (kwt == 3 && (g.KW == 1 || g.stride != 1))) continue;
        if (conv_back_lds(M, kwt, 1) > kBackLds) continue;
        for (int nt = 2; nt >= 1; --nt) {
            if (nt_given ? nt != nt_given : (nt == 2 && (g.C_out <= kWave || conv_back_lds(M, kwt, 2) > kBackLds))) continue;
            const int kg = (g.KW + kwt - 1) / kwt;
            const int tiles = (g.C_out + nt * kWave - 1) / (nt * kWave);
            // dt_in entries per input: at most KH * KW + 1 at a time, or 32 MiB of them
            // (132 -> 238, 6 x 6, stride 2, batch 54: one launch of both tiles for two)
            const int64_t by_bytes = (int64_t{32} << 20) / std::max<int64_t>(1, 4 * B * g.Hp * g.Wp * g.PC * g.KH * kg);
            const int tiles_dt = static_cast<int>(std::max<int64_t>(
                1, std::min<int64_t>(tiles, std::max<int64_t>((g.KH * g.KW + 1) / (g.KH * kg), by_bytes))));
            const int launches = dt ? (tiles + tiles_dt - 1) / tiles_dt : 1;
            const int by_lds = std::max(1, (160 * 1024) / (conv_back_lds(M, kwt, nt) + 1024));
            const double steps = g.Wo + kwt - 1;
            for (int tj = 16; tj >= 8; tj -= 8) {
                if (kwt * nt * tj > 48) continue;
                const int cpt = (g.C_in + tj - 1) / tj, chunks = cpt * g.KH * kg;
                const int occ = conv_back_occupancy(kwt, kwt * nt * tj, dw, dt);
                const double item = kItem + static_cast<double>(g.C_in) / cpt * (kwt * nt * k_pair + kInput);
                const double start = kStart + kStartPair * kwt * nt * tj;
                for (const int most : {kBackWaves, 8, 4}) {
                    const int groups = (chunks + most - 1) / most;
                    const int even = (chunks + groups - 1) / groups;
                    // (one block over the chunks: also with waves that only write table
                    // rows; 1 -> 22, 1 x 1, 24 x 24, batch 7, M = 66 112 -> 51 us)
                    for (const int w : {even, most}) {
                        if (w != even && groups > 1) continue;
                        const int per = std::max(1, std::min(w <= 2 ? 4 * occ / w : occ / ((w + 3) / 4), by_lds));
                        const double step = g.P * item + kStep + kRow * nt * (M + 3) / w;
                        const int64_t blocks = static_cast<int64_t>(groups) * ((tiles + launches - 1) / launches);
                        for (int want = least_split;; want = std::min(2 * want, most_split)) {
                            const int rps = rows_given ? rows_given : (rows + want - 1) / want;
                            const int ns = (rows + rps - 1) / rps;
                            const int64_t tot = blocks * ns, full = tot < kConvCUs * per ? 0 : tot / (kConvCUs * per);
                            const int64_t rest = tot - full * kConvCUs * per;
                            double us = static_cast<double>(full) * (1. + kShare * per * w);
                            if (rest > 0) us += 1. + kShare * static_cast<double>((static_cast<int>(rest) + kConvCUs - 1) / kConvCUs) * w;
                            us *= launches * (start + static_cast<double>(rps) * steps * step) / kPerUs;
                            if (dw) us += std::max(kPartUsPerMB * static_cast<double>(ns) * dw_mb,
                                                   kPartUsPerSplit * static_cast<double>(ns));
                            if (dt) us += kEntryUsPerMB * g.KH * kg * tiles * in_mb;
                            if (best < 0. || us < best) {
                                best = us;
                                p = ConvBackPlan{kwt, nt, tj, kg, tiles, tiles_dt, cpt, chunks, groups, w,
                                                 ns, rps,
                                                 static_cast<size_t>(conv_back_lds(M, kwt, nt))};
                            }
                            if (rows_given || want >= most_split) break;
                        }
                    }
                }
            }
        }
    }
    return p;
}

// One gradient alone keeps what the order of its sums depends on (dW: the splits;
// dt_in: taps and channels per lane) as both together have it, so that it comes out
// the same to the bit; the workspace is laid out for both.
ConvBackPlan plan_conv_back(const ConvGeom &g, int64_t B, int M, bool dw, bool dt) {
    const ConvBackPlan p = conv_back_search(g, B, M, true, true, 0, 0, 0);
    if (dw == dt) return p;
    return dw ? conv_back_search(g, B, M, true, false, 0, 0, p.rows_per_split)
              : conv_back_search(g, B, M, false, true, p.kwt, p.nt, 0);
}
// ---- end of the launch rules of conv_back_kernel ----

// dW alone: pairs along the lanes (conv_dw_kernel) where a position has enough of
// them for the lanes, 64 (tap, input) pairs times raw pixels, or 18 with at most 64
// channels out (below: 3 -> 64, 1 x 1, 32 x 32, batch 64 149 us, 171 with pairs
// along the lanes; 1 -> 38, 18 x 18, batch 11 44 and 53). 32 channels per block past
// M = 88, where two tables of 64 would leave two blocks per CU or less.
// conv_back_kernel -> conv_dw_kernel, set-up and sums with it: 64 -> 64, 32 x 32,
// batch 64 656 -> 589 us; 128 -> 128, 16 x 16, stride 2, batch 64 341 -> 263;
// 17 -> 140, 26 x 26, stride 2, batch 20 146 -> 79; 1 -> 32, 5 x 5, 28 x 28,
// batch 64 285 -> 122.
static bool conv_dw_by_pair(const ConvGeom &g) {
    return static_cast<int64_t>(g.KH) * g.KW * g.C_in * g.P >= (g.C_out <= kWave ? 18 : 64);
}
static int conv_dw_ti(const ConvGeom &g, int M) { return (g.C_out <= 32 || M > 88) ? 32 : 64; }
static size_t conv_dw_lds(int M, int ti) {
    return 2 * static_cast<size_t>(M + 4) * (ti + 4) * sizeof(float) +
           static_cast<size_t>(g_table_len(M)) * sizeof(float2);
}

template <int KWT, int NT, int TJ>
static void launch_back(const LifConst &C, const ConvGeom &g, const ConvBackArgs &a,
                        const ConvBackPlan &p, int tiles, bool dw, bool dt, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(p.groups), static_cast<unsigned>(p.nsplit),
                    static_cast<unsigned>(tiles));
    const dim3 block(static_cast<unsigned>(p.waves * kWave));
    if (dw && dt) hipLaunchKernelGGL((conv_back_kernel<KWT, NT, TJ, true, true>), grid, block, p.lds, st, C, g, a);
    else if (dw) hipLaunchKernelGGL((conv_back_kernel<KWT, NT, TJ, true, false>), grid, block, p.lds, st, C, g, a);
    else hipLaunchKernelGGL((conv_back_kernel<KWT, NT, TJ, false, true>), grid, block, p.lds, st, C, g, a);
}

hipError_t launch_conv_backward(const LifConst &C, const ConvGeom &g, int64_t B, const void *W,
                                bool bf16, const float *t_in, const float *t_out,
                                const float *slope, const int *q_idx, const float *grad_t,
                                ConvBwdWs ws, float *grad_W, float *grad_t_in, const Synfire &sf,
                                bool reuse, hipStream_t st) {
    const int64_t n_in = B * g.Hp * g.Wp * g.PC;
    const int64_t n_pos = B * g.Ho * g.Wo;
    const int64_t nj = static_cast<int64_t>(g.KH) * g.KW * g.C_in;
    const bool dt = grad_t_in && n_in > 0;
    hipError_t e;
    {
        // cell rows' events, gradient triples + gradient rows, and the WT
        // layout for dt_in: one launch (after a keeping forward only the
        // gradient roles)
        const int n_cr = (!reuse && n_in > 0 && (grad_W || dt)) ? static_cast<int>(B * g.Hp) : 0;
        const int n_gr = static_cast<int>((n_pos + kGradPos - 1) / kGradPos) *
                         ((g.C_out + kGradCh - 1) / kGradCh);
        const int n_wt = (dt && !reuse) ? static_cast<int>(weight_tiles(g)) : 0;
        // dead-neuron terms only where dW is written
        const bool dead = sf.on && sf.dq && grad_W;
        const int n_dq = dead ? g.C_out : 0;
        const int lds = std::max({kGradLdsBytes, 256 * static_cast<int>(sizeof(int)),
                                  n_cr > 0 ? events_stage_floats(g) * static_cast<int>(sizeof(float)) : 0});
        const unsigned blocks = static_cast<unsigned>(n_cr + n_gr + n_dq + n_wt);
        ProfScope prof("conv_bprep", st);
        if (blocks > 0) {
            if (bf16)
                hipLaunchKernelGGL(conv_bprep_kernel<uint16_t>, dim3(blocks), dim3(256), lds, st, C,
                                   g, n_cr, n_gr, n_dq, t_in, ws.ev, n_pos, t_out, slope,
                                   q_idx, grad_t, sf, ws.tri, ws.rend,
                                   static_cast<const uint16_t *>(W), ws.wt);
            else
                hipLaunchKernelGGL(conv_bprep_kernel<float>, dim3(blocks), dim3(256), lds, st, C,
                                   g, n_cr, n_gr, n_dq, t_in, ws.ev, n_pos, t_out, slope,
                                   q_idx, grad_t, sf, ws.tri, ws.rend,
                                   static_cast<const float *>(W), ws.wt);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const bool dtl = dt && n_pos > 0;
    const ConvBackPlan p = plan_conv_back(g, B, C.M, grad_W != nullptr, dtl);
    if (grad_W || dtl) {
        ConvBackArgs a{static_cast<int>(B * g.Ho), p.rows_per_split, p.cpt, p.n_chunk, p.kg, 0, 0, 0,
                       ws.tri, ws.rend, ws.ev.live, ws.ev.ev, ws.wt, ws.P, ws.part,
                       ws.zlive};
        if (grad_W && !dtl && conv_dw_by_pair(g)) {
            ProfScope prof("conv_dw", st);
            const int ti = conv_dw_ti(g, C.M);
            const dim3 grid(static_cast<unsigned>((nj + kDwPairs - 1) / kDwPairs), static_cast<unsigned>(p.nsplit),
                            static_cast<unsigned>((g.C_out + ti - 1) / ti));
            if (ti == 64) hipLaunchKernelGGL((conv_dw_kernel<64>), grid, dim3(kDwPairs), conv_dw_lds(C.M, 64), st, C, g, a);
            else hipLaunchKernelGGL((conv_dw_kernel<32>), grid, dim3(kDwPairs), conv_dw_lds(C.M, 32), st, C, g, a);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        } else {
            ProfScope prof("conv_back", st);
            const int step = dtl ? p.tiles_dt : p.tiles;
            a.n_tile = step;
            for (int t = 0; t < p.tiles; t += step) {
                a.tile0 = t;
                a.add = t > 0;
                const int nt = std::min(step, p.tiles - t);
                const bool dw = grad_W != nullptr;
                if (p.kwt == 3 && p.nt == 2) launch_back<3, 2, 8>(C, g, a, p, nt, dw, dtl, st);
                else if (p.kwt == 3 && p.tj == 16) launch_back<3, 1, 16>(C, g, a, p, nt, dw, dtl, st);
                else if (p.kwt == 3) launch_back<3, 1, 8>(C, g, a, p, nt, dw, dtl, st);
                else if (p.nt == 2 && p.tj == 16) launch_back<1, 2, 16>(C, g, a, p, nt, dw, dtl, st);
                else if (p.nt == 2) launch_back<1, 2, 8>(C, g, a, p, nt, dw, dtl, st);
                else if (p.tj == 16) launch_back<1, 1, 16>(C, g, a, p, nt, dw, dtl, st);
                else launch_back<1, 1, 8>(C, g, a, p, nt, dw, dtl, st);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        }
    }
    {
        // dW split reduction and dt_in gather: one launch
        const int64_t n = static_cast<int64_t>(g.C_out) * nj;
        // reduction blocks: one per red_out outputs, at most 512 (each then
        // takes every 512th group; two blocks per CU)
        const int red_out = 256 / red_groups(p.nsplit);
        const int n_red = grad_W ? static_cast<int>(std::min<int64_t>((n + red_out - 1) / red_out, 512)) : 0;
        const int per = g.Wp * g.PC;
        const int nsl = (per + kGatherSlots - 1) / kGatherSlots;
        const int n_ga = dt ? static_cast<int>(B * g.Hp) * nsl : 0;
        ProfScope prof("conv_bfin", st);
        if (n_red + n_ga > 0)
            hipLaunchKernelGGL(conv_bfin_kernel, dim3(static_cast<unsigned>(n_red + n_ga)),
                               dim3(256), 0, st, g, n_red, p.nsplit, ws.part, ws.zlive,
                               (sf.on && sf.dq) ? sf.dq : nullptr, grad_W, nsl,
                               ConvGatherArgs{ws.ev.live, ws.rend, ws.P, p.kwt, p.kg, p.tiles_dt},
                               grad_t_in);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace dstd
