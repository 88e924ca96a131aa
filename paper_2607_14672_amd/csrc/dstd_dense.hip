// dstd_dense.hip -- DSTD-LIF dense-layer kernels for gfx950.
//
// The event matrix S[b, m, j] has at most two nonzeros per (b, j): the DSTD
// kernel has two-point support (App. B.3). The contraction
// w^[b, m, i] = sum_j W[i, j] S[b, m, j] therefore runs over each sample's
// inputs sorted by event row: a wavefront (lanes = neurons) adds W[i, j] L and
// W[i, j] R of every input to the running sums of its row and feeds each
// closed row to the interval scan, instead of a dense (M+1)-row GEMM that
// would spend (M+1)/2 times the method's multiply-adds on zeros. The weighted
// events never go to HBM. The backward contraction (dstd_back.hip) takes the
// events in input order.
#include "dstd_back.h"
#include "dstd_internal.h"
#include "dstd_kernels.h"
#include "dstd_lif.h"
#include "dstd_walk.h"
#include "dstd_rows.h"
#include "dstd_profile.h"

#include <algorithm>

namespace dstd {

// ----------------------------------------------------------- event sort --
// Per sample, the inputs that have events, sorted by event row (stable: j
// ascending within a row), as structure-of-arrays records {j, row, L, R}, plus
// the row starts.
// One block of kSortWaves wavefronts per sample; wave w owns a contiguous
// range of inputs. Row histograms per wave (integer LDS atomics, order-free)
// give every (row, wave) pair its start offset (wave 0 scans the row totals
// across its lanes); each wave then places its inputs 64 at a time: a lane's
// rank among the lanes of its batch with the same row comes from a match
// mask built bit by bit from ballots of the row index, and the lowest lane
// of each row advances that row's slot. The fixed order keeps every sum of
// the forward pass bitwise reproducible.
constexpr int kSortWaves = 8;
constexpr int kPrepThreads = kSortWaves * 64;
constexpr int kRowBits = 9;  // row + 1 < 512 covers R = M + 3 rows for every M <= 256
static_assert(DSTD_MAX_M + 3 < (1 << kRowBits), "row keys must fit kRowBits");

template <int KS>
__device__ void sort_sample(const LifConst &C, int b, int N_in, const float *__restrict__ t_in,
                            SortedEv srt, int *__restrict__ n_valid, int *sh) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int R = rows_of(C);
    int *hist = sh;  // [kSortWaves][R], then rowstart [R + 1]
    int *rowstart = sh + kSortWaves * R;
    const float *tb = t_in + static_cast<int64_t>(b) * N_in;
    const int per = ((N_in + kSortWaves * kWave - 1) / (kSortWaves * kWave)) * kWave;
    const int j_lo = wave * per, j_hi = min(N_in, j_lo + per);
    for (int k = threadIdx.x; k < kSortWaves * R + R + 1; k += blockDim.x) sh[k] = 0;
    __syncthreads();
    for (int j0 = j_lo; j0 < j_hi; j0 += kWave) {
        const int j = j0 + lane;
        const int r = (j < j_hi) ? bin_row(C, tb[j]) : -1;
        if (r >= 0) atomicAdd(&hist[wave * R + r], 1);
    }
    __syncthreads();
    if (wave == 0) {
        // rowstart[r + 1] = events in rows <= r: an inclusive scan of the row
        // totals, 64 rows per pass
        int acc = 0;
        for (int r0 = 0; r0 < R; r0 += kWave) {
            const int r = r0 + lane;
            int v = 0;
            if (r < R)
                for (int w = 0; w < kSortWaves; ++w) v += hist[w * R + r];
#pragma unroll
            for (int m = 1; m < kWave; m <<= 1) {
                const int o = __shfl_up(v, m);
                if (lane >= m) v += o;
            }
            if (r < R) rowstart[r + 1] = acc + v;
            acc += __shfl(v, kWave - 1);
        }
        if (lane == 0) n_valid[b] = acc;
    }
    __syncthreads();
    for (int r = threadIdx.x; r <= R; r += blockDim.x)
        srt.rs[static_cast<int64_t>(b) * (R + 1) + r] = rowstart[r];
    for (int r = threadIdx.x; r < R; r += blockDim.x) {
        int base = rowstart[r];
        for (int w = 0; w < kSortWaves; ++w) {
            const int h = hist[w * R + r];
            hist[w * R + r] = base;  // becomes this wave's next slot in row r
            base += h;
        }
    }
    __syncthreads();
    const int64_t ob = static_cast<int64_t>(b) * srt.stride;
    int *next = hist + wave * R;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int j0 = j_lo; j0 < j_hi; j0 += kWave) {
        const int j = j0 + lane;
        Event e{-1, 0.f, 0.f, 0.f, 0.f};
        if (j < j_hi) e = bin_event<KS>(C, tb[j]);
        const int r = e.row;
        // lanes with the same row: agree with this lane on every bit of r + 1
        // (lanes without an event, r + 1 = 0, match only each other)
        const unsigned key = static_cast<unsigned>(r + 1);
        uint64_t same = ~0ull;
#pragma unroll
        for (int bit = 0; bit < kRowBits; ++bit) {
            const uint64_t ones = __ballot((key >> bit) & 1u);
            same &= ((key >> bit) & 1u) ? ones : ~ones;
        }
        const int rank = __popcll(same & below);
        int pos = 0;
        if (r >= 0) {
            const int base = next[r];
            pos = base + rank;
            if (rank == 0) next[r] = base + __popcll(same);
        }
        if (r >= 0) {
            const int64_t o = ob + pos;
            srt.j[o] = j;
            srt.r[o] = r;
            srt.L[o] = e.L;
            srt.R[o] = e.R;
        }
    }
}

// Set-up of a forward call in one launch, by block role: blocks [0, n_sort)
// sort one sample's n_rec records each, the rest transpose one weight tile each. One launch
// instead of two: every launch costs a few microseconds even when its work is
// tiny.
template <typename WT, int KS>
__global__ __launch_bounds__(kPrepThreads) void prep_kernel(LifConst C, int n_sort, int n_rec,
                                                            int N_in, int N_out,
                                                            const float *__restrict__ t_in,
                                                            SortedEv srt, int *__restrict__ n_valid,
                                                            const WT *__restrict__ W,
                                                            WT *__restrict__ Wt) {
    extern __shared__ int sh[];
    __shared__ WT buf[32][33];
    const int blk = blockIdx.x;
    if (blk < n_sort) sort_sample<KS>(C, blk, n_rec, t_in, srt, n_valid, sh);
    else transpose_tile<WT, kPrepThreads>(N_out, N_in, W, Wt, blk - n_sort, buf);
}

// Set-up of a backward call, by block role: n_ev blocks per sample write the
// events of kBackPrep inputs each, ev[b][field][j]; then n_gr blocks per sample
// the gradient triples of kBackPrep neurons each, tri[b][field][i]; then (with
// the synfire terms on) blocks counting each neuron's silent samples into sf.dq.
constexpr int kBackPrep = 256;
template <int KS>
__global__ __launch_bounds__(kBackPrep) void back_prep_kernel(LifConst C, int B, int n_ev, int n_gr,
                                                              int N_in, int N_out,
                                                              const float *__restrict__ t_in,
                                                              float *__restrict__ ev,
                                                              const float *__restrict__ t_out,
                                                              const float *__restrict__ slope,
                                                              const int *__restrict__ q_idx,
                                                              const float *__restrict__ grad_t,
                                                              float *__restrict__ tri, Synfire sf) {
    int blk = blockIdx.x;
    if (blk < n_ev * B) {
        const int b = blk / n_ev, j = (blk - b * n_ev) * kBackPrep + static_cast<int>(threadIdx.x);
        if (j < N_in) {
            const Event e = bin_event<KS>(C, t_in[static_cast<int64_t>(b) * N_in + j]);
            float *o = ev + static_cast<int64_t>(b) * kEvFields * N_in + j;
            o[0] = __int_as_float(e.row);
            o[N_in] = e.L;
            o[2 * static_cast<int64_t>(N_in)] = e.R;
            o[3 * static_cast<int64_t>(N_in)] = e.dL;
            o[4 * static_cast<int64_t>(N_in)] = e.dR;
        }
        return;
    }
    blk -= n_ev * B;
    if (blk < n_gr * B) {
        const int b = blk / n_gr, i = (blk - b * n_gr) * kBackPrep + static_cast<int>(threadIdx.x);
        if (i < N_out) {
            const int64_t k = static_cast<int64_t>(b) * N_out + i;
            const int q = q_idx[k];
            GradTriple gp{0.f, 0.f, -1};
            if (q >= 0) {  // silent neurons: no further loads
                float g = grad_t[k];
                // the spike time only where it is used (no gradient: no load)
                const float t = (sf.on || g != 0.f) ? t_out[k] : 0.f;
                if (sf.on) g += synfire_dt(sf, t);
                if (g != 0.f) gp = grad_triple(C, t, slope[k], q, g);
            }
            float *o = tri + static_cast<int64_t>(b) * 3 * N_out + i;
            o[0] = gp.gK;
            o[N_out] = gp.gE;
            o[2 * static_cast<int64_t>(N_out)] = __int_as_float(gp.q);
        }
        return;
    }
    // silent-sample count of neuron i over the batch (dead-neuron term)
    const int i = (blk - n_gr * B) * kBackPrep + static_cast<int>(threadIdx.x);
    if (i < N_out) {
        int cnt = 0;
        for (int b = 0; b < B; ++b) cnt += (q_idx[static_cast<int64_t>(b) * N_out + i] < 0) ? 1 : 0;
        sf.dq[i] = -(sf.gq * sf.scale * static_cast<float>(cnt));
    }
}

// --------------------------------------------------------------- forward --
// Lane = neuron i of a 64-neuron tile, one sample per wavefront (4 per block).
// The wave walks its sample's events in grid order: each record adds
// W[i, j] L and W[i, j] R to the running sums of its row (WT row j is one
// coalesced 256-byte load with a scalar base). When a row closes, grid point
// m = row - 1 is complete (its L parts come from this row, its R parts from
// the previous one) and goes straight into the interval scan: the weighted
// events never exist in memory. Once every lane has found its crossing
// interval, later events cannot change the outputs and the wave stops.

template <typename WT, int KS>
__global__ __launch_bounds__(256) void fwd_sorted_kernel(LifConst C, int B, int N_in, int N_out,
                                                         const WT *__restrict__ Wt,
                                                         SortedEv srt,
                                                         const int *__restrict__ n_valid,
                                                         float *__restrict__ t_out,
                                                         float *__restrict__ slope,
                                                         int *__restrict__ q_idx) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int i = blockIdx.x * kWave + lane;
    const bool row_ok = i < N_out;
    const int b = uniform(blockIdx.y * waves + wave);
    if (b >= B) return;  // wave-uniform; the kernel has no block barrier
    const int n = *as_const(n_valid + b);
    Scan<KS> sc;
    walk_sorted_rows<WT, false>(C, N_in, N_out, Wt, srt, b, n, i, row_ok, 1, sc);
    if (!row_ok) return;
    float to, sl;
    int q;
    sc.finish(C, to, sl, q);
    const int64_t o = static_cast<int64_t>(b) * N_out + i;
    t_out[o] = to;
    slope[o] = sl;
    q_idx[o] = q;
}


// ---------------------------------------------------------------- losses --
// One block per sample; block reductions run over a fixed LDS tree, so the
// per-sample losses (loss[1 + b]) and their fixed-order sum (loss[0]) are
// deterministic.
constexpr int kLossThreads = 256;

__device__ __forceinline__ float block_reduce(float v, float *red, bool is_max) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = kLossThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w)
            red[threadIdx.x] = is_max ? fmaxf(red[threadIdx.x], red[threadIdx.x + w])
                                      : red[threadIdx.x] + red[threadIdx.x + w];
        __syncthreads();
    }
    const float r = red[0];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kLossThreads) void softmax_ce_kernel(int B, int N,
                                                                  const float *__restrict__ t,
                                                                  const int *__restrict__ labels,
                                                                  float tau_soft, float t_cap,
                                                                  float *__restrict__ grad,
                                                                  float *__restrict__ loss) {
    __shared__ float red[kLossThreads];
    const int b = blockIdx.x;
    const float inv = 1.f / tau_soft;
    const float *tb = t + static_cast<int64_t>(b) * N;
    float *gb = grad + static_cast<int64_t>(b) * N;
    float mx = -INFINITY;
    for (int k = threadIdx.x; k < N; k += kLossThreads) {
        const float tk = isfinite(tb[k]) ? tb[k] : t_cap;
        mx = fmaxf(mx, -tk * inv);
    }
    mx = block_reduce(mx, red, true);
    float z = 0.f;
    for (int k = threadIdx.x; k < N; k += kLossThreads) {
        const float tk = isfinite(tb[k]) ? tb[k] : t_cap;
        z += expf(-tk * inv - mx);
    }
    z = block_reduce(z, red, false);
    const int lab = labels[b];
    const float lz = logf(z) + mx;
    for (int k = threadIdx.x; k < N; k += kLossThreads) {
        const bool fired = isfinite(tb[k]);
        const float tk = fired ? tb[k] : t_cap;
        const float sk = expf(-tk * inv - lz);
        const float dl = (sk - (k == lab ? 1.f : 0.f)) * (-inv) / static_cast<float>(B);
        gb[k] = fired ? dl : 0.f;
    }
    if (threadIdx.x == 0) {
        const float tl = isfinite(tb[lab]) ? tb[lab] : t_cap;
        loss[1 + b] = (lz + tl * inv) / static_cast<float>(B);
    }
}

__global__ __launch_bounds__(kLossThreads) void mse_kernel(int B, int N, const float *__restrict__ t,
                                                           const float *__restrict__ y,
                                                           float *__restrict__ grad,
                                                           float *__restrict__ loss) {
    __shared__ float red[kLossThreads];
    const int b = blockIdx.x;
    float acc = 0.f;
    for (int k = threadIdx.x; k < N; k += kLossThreads) {
        const int64_t o = static_cast<int64_t>(b) * N + k;
        const bool fired = isfinite(t[o]);
        const float d = fired ? (t[o] - y[o]) : 0.f;
        grad[o] = d / static_cast<float>(B);
        acc += 0.5f * d * d / static_cast<float>(B);
    }
    acc = block_reduce(acc, red, false);
    if (threadIdx.x == 0) loss[1 + b] = acc;
}

// loss[0] = sum_b loss[1 + b] in a fixed order
__global__ __launch_bounds__(kLossThreads) void loss_total_kernel(int B, float *__restrict__ loss) {
    __shared__ float red[kLossThreads];
    float acc = 0.f;
    for (int b = threadIdx.x; b < B; b += kLossThreads) acc += loss[1 + b];
    acc = block_reduce(acc, red, false);
    if (threadIdx.x == 0) loss[0] = acc;
}

// ------------------------------------------------------------- launchers --
static int tiles32(int64_t N_in, int64_t N_out) {
    return static_cast<int>(((N_in + 31) / 32) * ((N_out + 31) / 32));
}

static size_t sort_lds_bytes(const LifConst &C) {
    const int R = C.M + 3;
    return static_cast<size_t>(kSortWaves * R + R + 1) * sizeof(int);
}

hipError_t launch_sort_transpose(const LifConst &C, int64_t B, int64_t n_rec, int64_t N_in,
                                 int64_t N_out, const float *t_in, SortedEv srt, int *n_valid,
                                 const void *W, bool bf16, void *Wt, const char *name,
                                 hipStream_t st) {
    const int64_t blocks = B + (N_in * N_out > 0 ? tiles32(N_in, N_out) : 0);
    if (blocks == 0) return hipSuccess;
    ProfScope prof(name, st);
#define PREP(WTY, KSV)                                                                             \
    hipLaunchKernelGGL((prep_kernel<WTY, KSV>), dim3(static_cast<unsigned>(blocks)),              \
                       dim3(kPrepThreads), sort_lds_bytes(C), st, C, static_cast<int>(B),          \
                       static_cast<int>(n_rec), static_cast<int>(N_in), static_cast<int>(N_out),   \
                       t_in, srt, n_valid, static_cast<const WTY *>(W), static_cast<WTY *>(Wt))
    const bool gen = C.kind == kGeneral;
    if (bf16) {
        if (gen) PREP(uint16_t, kGeneral); else PREP(uint16_t, kAnyKind);
    } else {
        if (gen) PREP(float, kGeneral); else PREP(float, kAnyKind);
    }
#undef PREP
    return hipGetLastError();
}

hipError_t launch_forward(const LifConst &C, int64_t B, int64_t N_in, int64_t N_out, const void *W,
                          bool bf16, void *Wt, SortedEv srt, int *n_valid, const float *t_in,
                          float *t_out, float *slope, int *q_idx, hipStream_t st) {
    const int R = C.M + 3;
    hipError_t e = launch_sort_transpose(C, B, N_in, N_in, N_out, t_in, srt, n_valid, W, bf16, Wt,
                                         "sort_transpose", st);
    if (e != hipSuccess) return e;
    ProfScope prof("fwd_dense", st);
    if (C.M <= kRowsMaxM) {
        const int nt = rows_nt(N_out, R);
        const int tiles = static_cast<int>((N_out + kWave - 1) / kWave);
        dim3 grid(static_cast<unsigned>((tiles + nt - 1) / nt), static_cast<unsigned>(B));
        const size_t lds = rows_lds(nt, R);
        // NT neighbouring neurons per lane where rows keep NT-wide loads aligned
        const bool vec = (N_out % nt) == 0;
#define FWR_KV(WTY, NTV, KSV, VECV)                                                               \
    hipLaunchKernelGGL((fwd_rows_kernel<WTY, NTV, KSV, VECV, RowOutTtfs>), grid,                 \
                       dim3(kRowWaves * kWave), lds, st, C, static_cast<int>(N_in),               \
                       static_cast<int>(N_out), static_cast<const WTY *>(Wt), srt,                \
                       RowOutTtfs{t_out, slope, q_idx})
#define FWR_K(WTY, NTV, KSV)                      \
    do {                                          \
        if (vec) FWR_KV(WTY, NTV, KSV, true);     \
        else FWR_KV(WTY, NTV, KSV, false);        \
    } while (0)
#define FWR(WTY, NTV)                                                     \
    do {                                                                  \
        if (C.kind == kGeneral) FWR_K(WTY, NTV, kGeneral);                \
        else FWR_K(WTY, NTV, kAnyKind);                                   \
    } while (0)
        if (bf16) {
            if (nt == 4) FWR(uint16_t, 4);
            else if (nt == 2) FWR(uint16_t, 2);
            else FWR(uint16_t, 1);
        } else {
            if (nt == 4) FWR(float, 4);
            else if (nt == 2) FWR(float, 2);
            else FWR(float, 1);
        }
#undef FWR
#undef FWR_K
#undef FWR_KV
        return hipGetLastError();
    }
    constexpr int waves = 4;
    dim3 grid(static_cast<unsigned>((N_out + kWave - 1) / kWave),
              static_cast<unsigned>((B + waves - 1) / waves));
#define FWS(WTY, KSV)                                                                           \
    hipLaunchKernelGGL((fwd_sorted_kernel<WTY, KSV>), grid, dim3(waves * kWave), 0, st, C,      \
                       static_cast<int>(B), static_cast<int>(N_in), static_cast<int>(N_out),     \
                       static_cast<const WTY *>(Wt), srt, n_valid, t_out, slope, q_idx)
    const bool gen = C.kind == kGeneral;
    if (bf16) {
        if (gen) FWS(uint16_t, kGeneral); else FWS(uint16_t, kAnyKind);
    } else {
        if (gen) FWS(float, kGeneral); else FWS(float, kAnyKind);
    }
#undef FWS
    return hipGetLastError();
}

hipError_t launch_backward(const LifConst &C, int64_t B, int64_t N_in, int64_t N_out,
                           const void *W, bool bf16, const float *t_in, const float *t_out,
                           const float *slope, const int *q_idx, const float *grad_t,
                           DenseBwdWs ws, float *grad_W, float *grad_t_in, const Synfire &sf,
                           hipStream_t st) {
    const bool run_dw = grad_W && N_out * N_in > 0;
    // the dead-neuron term needs dW; without dW only dT/dt is used
    Synfire sfp = sf;
    if (!run_dw) sfp.dq = nullptr;
    const float *dq = (sfp.on && sfp.dq) ? sfp.dq : nullptr;
    const int n_ev = static_cast<int>((N_in + kBackPrep - 1) / kBackPrep);
    const int n_gr = static_cast<int>((N_out + kBackPrep - 1) / kBackPrep);
    const int64_t blocks = B * (n_ev + n_gr) + (dq ? n_gr : 0);
    if (blocks > 0) {
        ProfScope prof("bwd_prep", st);
#define BPREP(KSV)                                                                                 \
    hipLaunchKernelGGL((back_prep_kernel<KSV>), dim3(static_cast<unsigned>(blocks)),               \
                       dim3(kBackPrep), 0, st, C, static_cast<int>(B), n_ev, n_gr,                 \
                       static_cast<int>(N_in), static_cast<int>(N_out), t_in, ws.ev, t_out, slope, \
                       q_idx, grad_t, ws.tri, sfp)
        if (C.kind == kGeneral) BPREP(kGeneral);
        else BPREP(kAnyKind);
#undef BPREP
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_back(C, BackJob{B, N_in, N_out, 1, ws.ev, ws.tri, false, W, bf16, ws.P, ws.n_buf, ws.part,
                                  dq, grad_W, grad_t_in}, st);
}

hipError_t launch_softmax_ce(int64_t B, int64_t N, const float *t, const int *labels,
                             float tau_soft, float t_cap, float *grad, float *loss,
                             hipStream_t st) {
    ProfScope prof("softmax_ce", st);
    if (B > 0)
        hipLaunchKernelGGL(softmax_ce_kernel, dim3(static_cast<unsigned>(B)), dim3(kLossThreads), 0,
                           st, static_cast<int>(B), static_cast<int>(N), t, labels, tau_soft,
                           t_cap, grad, loss);
    hipLaunchKernelGGL(loss_total_kernel, dim3(1), dim3(kLossThreads), 0, st, static_cast<int>(B),
                       loss);
    return hipGetLastError();
}

hipError_t launch_mse(int64_t B, int64_t N, const float *t, const float *y, float *grad,
                      float *loss, hipStream_t st) {
    ProfScope prof("mse", st);
    if (B > 0)
        hipLaunchKernelGGL(mse_kernel, dim3(static_cast<unsigned>(B)), dim3(kLossThreads), 0, st,
                           static_cast<int>(B), static_cast<int>(N), t, y, grad, loss);
    hipLaunchKernelGGL(loss_total_kernel, dim3(1), dim3(kLossThreads), 0, st, static_cast<int>(B),
                       loss);
    return hipGetLastError();
}

}  // namespace dstd
