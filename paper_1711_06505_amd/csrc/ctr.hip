// ctr.hip -- the worker side of one joint training step (Algorithm 1,
// WORKERITERATION) next to the image path:
//   ams_bag_fwd      per sample and ID table, the sum of the table rows of its
//                    behaviors' IDs and of its ad's ID (sparse ID features
//                    embedded from key-value tables, section 4.1);
//   ams_bag_bwd      the gradient of every touched row: the bag gradient of
//                    each occurrence's sample, summed per unique ID in
//                    ascending occurrence order (the segmented reduction of
//                    the SUM aggregator's backward);
//   ams_ctr_fwd_bwd  the CTR MLP on the concatenated input fields, softmax over
//                    the classes and mean cross-entropy with the click labels
//                    (section 3.1), and its backward: the worker's weight
//                    gradients and the gradient of every input field (among
//                    them delta_e of the image path);
//   ams_adagrad_rows sparse Adagrad on the touched rows of an ID table.
// No float atomics: every sum runs in a fixed order.
#include "ams_device.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / AMS_WAVE;
constexpr int kCtrBS = 16;                  // samples per block of the CTR kernel
constexpr int kCtrThreads = 512;            // threads per block of the CTR and tower kernels (2 waves per SIMD)
constexpr int kCtrMaxIn = 128, kCtrMaxHidden = 256, kCtrMaxC = 8, kTowerMaxOut = 64;
constexpr int kCtrMaxLayers = 3, kCtrMaxFields = 8;

// ------------------------------------------------------------ bag forward

// One wave per sample: lane l adds the rows of behaviors l, l + 64, ... in
// that order; the lanes' partial rows are summed by a fixed butterfly, then
// the ad row.  Behaviors go in rounds of U per lane (8 for rows up to 16
// floats, else 4) with every ID load, then every row load, of a round in
// flight together.  An ID outside [0, n_rows) reads as a zero row (dedup
// reports it).
template <int DM>
__global__ __launch_bounds__(kThreads) void bag_fwd_k(int B, int D, const int32_t *__restrict__ seg_off,
                                                      int64_t n_beh, const int32_t *__restrict__ ids,
                                                      const float *__restrict__ table, int64_t n_rows,
                                                      float *__restrict__ bag)
{
    const int lane = ams_lane();
    const int i = blockIdx.x * kWaves + threadIdx.x / AMS_WAVE;
    if (i >= B) return;
    const int j0 = seg_off[i], j1 = seg_off[i + 1];
    float acc[DM];
#pragma unroll
    for (int d = 0; d < DM; ++d) acc[d] = 0.f;
    const bool vec4 = (D & 3) == 0 && ((uintptr_t)table & 15) == 0;
    constexpr int kBagU = DM <= 16 ? 8 : 4;
    // every load of a round unconditional (a position past the sample reads
    // its last ID, an ID outside the table reads row 0), masked once all are
    // in flight; no table rows at all: nothing to read
    if (n_rows > 0) {
        for (int jr = j0; jr < j1; jr += kBagU * AMS_WAVE) {
            int id[kBagU];
#pragma unroll
            for (int u = 0; u < kBagU; ++u) {
                const int j = jr + u * AMS_WAVE + lane;
                id[u] = ids[j < j1 ? j : j1 - 1];
            }
            bool ok[kBagU];
#pragma unroll
            for (int u = 0; u < kBagU; ++u) {
                const int j = jr + u * AMS_WAVE + lane;
                ok[u] = j < j1 && id[u] >= 0 && (int64_t)id[u] < n_rows;
            }
            if (vec4) {
                float4 v[kBagU][DM / 4];
#pragma unroll
                for (int u = 0; u < kBagU; ++u) {
                    const float *r = table + (size_t)(ok[u] ? id[u] : 0) * D;
#pragma unroll
                    for (int d4 = 0; d4 < DM / 4; ++d4) v[u][d4] = *(const float4 *)(r + (4 * d4 < D ? 4 * d4 : 0));
                }
#pragma unroll
                for (int u = 0; u < kBagU; ++u)
#pragma unroll
                    for (int d4 = 0; d4 < DM / 4; ++d4) {
                        const bool take = ok[u] && 4 * d4 < D;
                        acc[4 * d4] += take ? v[u][d4].x : 0.f;
                        acc[4 * d4 + 1] += take ? v[u][d4].y : 0.f;
                        acc[4 * d4 + 2] += take ? v[u][d4].z : 0.f;
                        acc[4 * d4 + 3] += take ? v[u][d4].w : 0.f;
                    }
            } else {
                float v[kBagU][DM];
#pragma unroll
                for (int u = 0; u < kBagU; ++u) {
                    const float *r = table + (size_t)(ok[u] ? id[u] : 0) * D;
#pragma unroll
                    for (int d = 0; d < DM; ++d) v[u][d] = r[d < D ? d : 0];
                }
#pragma unroll
                for (int u = 0; u < kBagU; ++u)
#pragma unroll
                    for (int d = 0; d < DM; ++d) acc[d] += (ok[u] && d < D) ? v[u][d] : 0.f;
            }
        }
    }
    float mine = 0.f;
#pragma unroll
    for (int d = 0; d < DM; ++d) {
        const float s = ams_wave_sum(acc[d]);
        if (lane == d) mine = s;
    }
    if (lane < D) {
        const int id = ids[n_beh + i];
        const float a = (id >= 0 && (int64_t)id < n_rows) ? table[(size_t)id * D + lane] : 0.f;
        bag[(size_t)i * D + lane] = mine + a;
    }
}

// ---------------------------------------------------------------- CTR MLP

struct CtrArgs {
    int L;                                   // layers (1 to 3)
    int dims[kCtrMaxLayers + 1];
    int n_fields;
    int fdim[kCtrMaxFields];
    const float *field[kCtrMaxFields];
    float *dfield[kCtrMaxFields];
    const float *W[kCtrMaxLayers];
    const float *b[kCtrMaxLayers];
    const float *slope[kCtrMaxLayers];       // PReLU slopes after layer l < L-1; NULL: ReLU
};

// A block's partial row holds, per layer, dW [O x K], db [O] and, below the
// last layer, the slope gradient [O], each layer's part starting on a
// 16-byte boundary (padded to 4 floats); after the net(s) come 4 floats
// whose first is the loss sum, so rows are 16-byte multiples.
__host__ __device__ inline int net_layer_size(const CtrArgs &a, int l)
{
    return (a.dims[l + 1] * a.dims[l] + a.dims[l + 1] * (l < a.L - 1 ? 2 : 1) + 3) & ~3;
}

__host__ __device__ inline int net_part_size(const CtrArgs &a)
{
    int n = 0;
    for (int l = 0; l < a.L; ++l) n += net_layer_size(a, l);
    return n;
}

// The nets' layers run on float32 MFMA (v_mfma_f32_16x16x4_f32): the block's
// 16 samples are one side of every tile.  Lane l holds row l % 16 of the
// first operand and column l % 16 of the second, each at k = l / 16, and of
// the 16 x 16 result rows 4 (l / 16) .. + 3 of column l % 16.  Which k a step
// takes is free as long as both operands agree, so four steps take
// k = 16 g + 4 (l / 16) + e, e = 0..3: one 16-byte read per operand feeds
// them.  Where a lane's quad runs along the result's columns instead (the W
// rows of the backward, a layer's input in the weight gradient), its four
// elements belong to four tiles whose columns are 4 (l % 16) + e: one read
// feeds four tiles, and the results are stored as 16-byte quads.
// What bounds these kernels: a dozen dependent phases of a barrier, an L2 round
// trip and a few tens of MFMAs per wave (counters on the 72-200-80-2 net: a
// wave waits half of its time and issues a third of it), and last the partial
// rows' stores (31 MB at 4096 samples, 8 us).  4096 samples with PReLU, whole
// call: that net 60.8 us with the layers as vector FMA loops, 56.8 us so; a
// pair of 48-64-32 towers 62.3 and 33.4 us (side by side, four waves each).
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // any float address

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Barrier that orders LDS accesses only: global loads issued ahead of it and
// the partial row's stores stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Reads one word of each of the first N 64-byte lines of the kernel's
// arguments, all in flight together: the layers come to them one by one, and
// each line's first read is a miss to memory.
template <int N>
__device__ __forceinline__ void net_args_touch()
{
    typedef const __attribute__((address_space(4))) int kint;
    kint *p = (kint *)__builtin_amdgcn_kernarg_segment_ptr();
    int x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = p[16 * i];
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" ::"s"(x[i]));
}

// LDS row length of a layer w wide: whole quads (the pad columns are zero),
// and an odd number of them, so that 16 rows' quads fall in distinct banks.
__host__ __device__ inline int net_ld(int w) { return 4 * (((w + 3) / 4) | 1); }

// A row's quad at column k for a group of 16 that may pass the row's end at w:
// zero there.
__device__ __forceinline__ f4 net_quad(const float *row, int k, int w)
{
    const bool in = k < w;
    const f4 v = *(const f4 *)(row + (in ? k : 0));
    return in ? v : (f4){0.f, 0.f, 0.f, 0.f};
}

// Data gradient of a layer K wide into O by nw waves: blocks of 64 inputs
// times parts of the contraction over O (in groups of 16).
__host__ __device__ inline int net_kblocks(int K) { return (K + 63) / 64; }
__host__ __device__ inline int net_bwd_parts(int K, int O, int nw)
{
    const int p = nw / net_kblocks(K), groups = (O + 15) / 16;
    return p < 1 ? 1 : p < groups ? p : groups;
}

// LDS of one net for a block of kCtrBS samples: act (every layer's
// activations, the input fields first), grd (the loss gradient of each
// act[l]; with PReLU a hidden layer's slot holds its pre-activations between
// the forward and the backward) and the parts of the data gradients.

// net_off: where layer l's activations (and gradients) start.
__host__ __device__ inline int net_off(const CtrArgs &a, int l)
{
    int n = 0;
    for (int x = 0; x < l; ++x) n += kCtrBS * net_ld(a.dims[x]);
    return n;
}

__host__ __device__ inline int net_act_floats(const CtrArgs &a) { return net_off(a, a.L + 1); }

__host__ __device__ inline int net_scr_floats(const CtrArgs &a, int nw)
{
    int n = 0;
    for (int l = 0; l < a.L; ++l) {
        const int x = net_bwd_parts(a.dims[l], a.dims[l + 1], nw) * kCtrBS * 64 * net_kblocks(a.dims[l]);
        if (x > n) n = x;
    }
    return n;
}

// One net and the waves of the block that run it.
struct NetRun {
    float *act, *grd, *scr;
    int w, nw, t, nt;                        // this wave of nw, this thread of nt
};

__device__ __forceinline__ NetRun net_run(const CtrArgs &a, float *base, float *scr, int w, int nw)
{
    NetRun n;
    n.act = base;
    n.grd = base + net_act_floats(a);
    n.scr = scr;
    n.w = w;
    n.nw = nw;
    n.t = w * AMS_WAVE + ams_lane();
    n.nt = nw * AMS_WAVE;
    return n;
}

// The field that column k of the concatenated input lies in, at k's place in
// row i (out: the gradient's arrays; NULL where that field's is not wanted).
__device__ __forceinline__ float *net_field(const CtrArgs &a, int k, int64_t i, bool out)
{
    float *p = nullptr;
    int w = 0, at = 0, c0 = 0;
#pragma unroll
    for (int f = 0; f < kCtrMaxFields; ++f) {
        if (f >= a.n_fields) break;
        if (k >= c0) {
            p = out ? a.dfield[f] : const_cast<float *>(a.field[f]);
            w = a.fdim[f];
            at = k - c0;
        }
        c0 += a.fdim[f];
    }
    return p ? p + i * w + at : nullptr;
}

// Input fields, concatenated (rows past B read 0), and the zero pad columns
// of every layer.  A thread's loads are all in flight together.
constexpr int kLoadBatch = 4;
__device__ __forceinline__ void net_load(const CtrArgs &a, const NetRun &n, int b0, int B)
{
    const int K0 = a.dims[0], ld0 = net_ld(K0);
    for (int e0 = n.t; e0 < kCtrBS * K0; e0 += kLoadBatch * n.nt) {
        float v[kLoadBatch];
#pragma unroll
        for (int i = 0; i < kLoadBatch; ++i) {
            const int e = e0 + i * n.nt, s = e / K0, k = e - s * K0;
            const bool in = s < kCtrBS && b0 + s < B;
            const float x = *net_field(a, in ? k : 0, in ? b0 + s : b0, false);
            v[i] = in ? x : 0.f;
        }
#pragma unroll
        for (int i = 0; i < kLoadBatch; ++i) {
            const int e = e0 + i * n.nt, s = e / K0, k = e - s * K0;
            if (s < kCtrBS) n.act[s * ld0 + k] = v[i];
        }
    }
    int off = 0;
    for (int l = 0; l <= a.L; ++l) {
        const int w = a.dims[l], ld = net_ld(w), pad = ld - w;
        for (int e = n.t; e < kCtrBS * pad; e += n.nt) {
            const int x = off + (e / pad) * ld + w + e % pad;
            n.act[x] = 0.f;
            n.grd[x] = 0.f;
        }
        off += kCtrBS * ld;
    }
}

// Activation of a hidden unit: ReLU, or PReLU with slope a (z for z > 0,
// a z otherwise).
__device__ __forceinline__ float ctr_act(float v, const float *slope, float a) 
{
    return v > 0.f ? v : slope ? a * v : 0.f;
}

// This lane's W operands of output tile ot of a layer, groups g0 .. g0 + 3:
// row 16 ot + lane % 16 (rows past O read the last one, their results are
// dropped), group g's quad k = 16 g + 4 (lane / 16) .. + 3 (zero past K).
constexpr int kFwdBatch = 4;
__device__ __forceinline__ void net_fwd_load(const float *__restrict__ W, int K, int O, int ot, int g0,
                                             f4 (&w)[kFwdBatch])
{
    const int lane = ams_lane(), o = min(16 * ot + (lane & 15), O - 1), k0 = 16 * g0 + 4 * (lane >> 4);
    const float *wr = W + (size_t)o * K;
    if (16 * (g0 + kFwdBatch) <= K) {
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i) w[i] = *(const f4u *)(wr + k0 + 16 * i);
    } else if ((K & 3) == 0) {
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i) {
            const bool in = k0 + 16 * i < K;
            const f4 v = *(const f4u *)(wr + (in ? k0 + 16 * i : 0));
            w[i] = in ? v : (f4){0.f, 0.f, 0.f, 0.f};
        }
    } else {
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + 16 * i + e;
                const float v = wr[min(k, K - 1)];
                w[i][e] = k < K ? v : 0.f;
            }
    }
}

// The four lanes of a column (l, l + 16, l + 32, l + 48) as a 4 x 4 matrix of
// their four elements, transposed: element j of lane quarter q was element q of
// quarter j.  A quad read per lane so becomes the operands of four steps whose
// k are four consecutive ones.
__device__ __forceinline__ f4 quarters_transposed(f4 v)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
    const u2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
    const u2 c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const u2 d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    return (f4){__uint_as_float(c[0]), __uint_as_float(c[1]), __uint_as_float(d[0]), __uint_as_float(d[1])};
}

// Width of the parts that a forward sum is added up in: each part's terms in
// the order of k, the parts in order onto the bias.  A unit whose sum is within
// rounding of zero takes the side that this order gives it, so the order is
// part of the results: it is that of 512 threads that share a layer's outputs
// and, for narrow layers, its K in quads.
__device__ __forceinline__ int net_fwd_part(int K, int O)
{
    int P = 512 / O;
    if (P < 1) P = 1;
    if (P > (K + 15) / 16) P = (K + 15) / 16;
    return (((K + P - 1) / P) + 3) & ~3;
}

// out[s][o] = act(b[o] + sum_k in[s][k] W[o][k]): output tile ot (w: its
// first operands, afterwards those of tile next); the result's rows are
// outputs, so a lane holds four consecutive outputs of one sample.  An MFMA
// adds its four products in the order of k, each with a rounding of its own
// (as four fused multiply-adds), so one chain of them is net_fwd_part's order.
// The calls measured above with other forwards: four interleaved chains, in an
// order of their own, 47.4 and 30.4 us; operands by 4-byte reads 67.8 and 37.8;
// batches that follow the parts, with no test per step, 59.1 and 36.8.  With
// PReLU the pre-activations go to zout.
__device__ __forceinline__ void net_fwd_tile(const float *in, int ldi, int K, float *out, float *zout, int ldo, int O,
                                             int ot, int next, f4 (&w)[kFwdBatch], const float *__restrict__ W,
                                             const float *__restrict__ bias, bool hidden,
                                             const float *__restrict__ slope)
{
    const int lane = ams_lane(), s = lane & 15, q = lane >> 4, o0 = 16 * ot + 4 * q, groups = (K + 15) / 16;
    const int part = net_fwd_part(K, O);
    f4 v, acc = (f4){0.f, 0.f, 0.f, 0.f};
    float sl[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = bias[min(o0 + e, O - 1)];
        sl[e] = slope ? slope[min(o0 + e, O - 1)] : 0.f;
    }
    const float *x0 = in + s * ldi;
    int end = part;
#pragma unroll 1
    for (int g = 0; g < groups; g += kFwdBatch) {
        f4 nx[kFwdBatch];
        if (g + kFwdBatch < groups) net_fwd_load(W, K, O, ot, g + kFwdBatch, nx);
        else if (16 * next < O) net_fwd_load(W, K, O, next, 0, nx);
        f4 x[kFwdBatch];
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i) x[i] = net_quad(x0, 16 * (g + i) + 4 * q, K);
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i) {
            x[i] = quarters_transposed(x[i]);
            w[i] = quarters_transposed(w[i]);
        }
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 16 * (g + i) + 4 * j;
                if (k >= K) break;
                if (k == end) {
                    v += acc;
                    acc = (f4){0.f, 0.f, 0.f, 0.f};
                    end += part;
                }
                acc = mfma4(w[i][j], x[i][j], acc);
            }
#pragma unroll
        for (int i = 0; i < kFwdBatch; ++i) w[i] = nx[i];
    }
    v += acc;
    f4 z, y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        z[e] = o0 + e < O ? v[e] : 0.f;
        y[e] = hidden ? ctr_act(z[e], slope, sl[e]) : z[e];
    }
    if (o0 < O) {
        *(f4 *)(out + s * ldo + o0) = y;
        if (hidden && slope) *(f4 *)(zout + s * ldo + o0) = z;
    }
}

// Layer l of the forward (w holds the first operands of this wave's first
// tile, and afterwards those of the next layer's).
__device__ __forceinline__ void net_fwd_layer(const CtrArgs &a, const NetRun &n, int l, f4 (&w)[kFwdBatch])
{
    const int K = a.dims[l], O = a.dims[l + 1], tiles = (O + 15) / 16;
    const int oi = net_off(a, l), oo = oi + kCtrBS * net_ld(K);
    const bool hidden = l < a.L - 1;
#pragma unroll 1
    for (int ot = n.w; ot < tiles; ot += n.nw) {
        net_fwd_tile(n.act + oi, net_ld(K), K, n.act + oo, n.grd + oo, net_ld(O), O, ot, ot + n.nw, w, a.W[l], a.b[l],
                     hidden, hidden ? a.slope[l] : nullptr);
    }
    if (hidden && 16 * n.w < a.dims[l + 2]) net_fwd_load(a.W[l + 1], O, a.dims[l + 2], n.w, 0, w);
}

// dW[o][k] = sum_s gout[s][o] in[s][k] over the block's samples: 16 outputs x
// 64 inputs per wave and turn, written to the partial row at p; then
// db[o] = sum_s gout[s][o].
__device__ __forceinline__ void net_bwd_weight(const float *gout, int ldg, int O, const float *in, int ldi, int K,
                                               float *__restrict__ p, const NetRun &n)
{
    const int lane = ams_lane(), c = lane & 15, q = lane >> 4;
    const int kbs = net_kblocks(K), jobs = ((O + 15) / 16) * kbs;
#pragma unroll 1
    for (int j = n.w; j < jobs; j += n.nw) {
        const int ot = j / kbs, k = 64 * (j % kbs) + 4 * c;
        const float *gp = gout + 4 * q * ldg + 16 * ot + c, *xp = in + 4 * q * ldi + min(k, ldi - 4);
        f4 acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = (f4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < 4; ++st) {                  // samples 4 q + st
            const float g = gp[st * ldg];
            const f4 x = *(const f4 *)(xp + st * ldi);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = mfma4(g, x[e], acc[e]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 16 * ot + 4 * q + r;
            if (o >= O) continue;
            float *dst = p + o * K + k;
            if (k + 3 < K) *(f4u *)dst = (f4){acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e < K) dst[e] = acc[e][r];
        }
    }
    for (int o = n.t; o < O; o += n.nt) {
        float acc = 0.f;
#pragma unroll
        for (int s = 0; s < kCtrBS; ++s) acc += gout[s * ldg + o];
        p[O * K + o] = acc;
    }
}

// This lane's W operands of the data gradient's groups g0, g0 + 1 (outputs
// 16 g + 4 (lane / 16) + e, zero past O) for the inputs k .. k + 3.
constexpr int kBwdBatch = 2;
__device__ __forceinline__ void net_bwd_load(const float *__restrict__ W, int K, int O, int k, int g0, int g1,
                                             f4 (&w)[kBwdBatch][4])
{
    // inputs past K: any address of the row, their columns are dropped
    const int q = ams_lane() >> 4;
    const bool vec = (K & 3) == 0 || (k | 63) < K;         // (the same for the whole wave)
#pragma unroll
    for (int i = 0; i < kBwdBatch; ++i) {
        if (g0 + i >= g1) break;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *wr = W + (size_t)min(16 * (g0 + i) + 4 * q + e, O - 1) * K;
            if (vec) w[i][e] = *(const f4u *)(wr + (k < K ? k : 0));
            else
#pragma unroll
                for (int c = 0; c < 4; ++c) w[i][e][c] = wr[min(k + c, K - 1)];
        }
        if (16 * (g0 + i) + 16 > O)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (16 * (g0 + i) + 4 * q + e >= O) w[i][e] = (f4){0.f, 0.f, 0.f, 0.f};
    }
}

// The layer's data gradient, through the activation that produced its input
// (act, below the first layer): d[s][k] = sum_o gout[s][o] W[o][k] in parts
// over O, added in part order; ReLU takes d where in > 0; PReLU reads its
// pre-activation z from gin (left there by the forward) and takes d for
// z > 0, slope[k] d otherwise, and adds d min(z, 0) over the block's samples
// (ascending) into the slope gradient dsl[k].
__device__ __forceinline__ void net_bwd_parts_out(const float *__restrict__ W, int K, int O, const float *gout, int ldg,
                                                  const NetRun &n, f4 (&w)[kBwdBatch][4])
{
    const int lane = ams_lane(), c = lane & 15, q = lane >> 4;
    const int kbs = net_kblocks(K), P = net_bwd_parts(K, O, n.nw), groups = (O + 15) / 16;
#pragma unroll 1
    for (int j = n.w; j < kbs * P; j += n.nw) {
        const int kb = j % kbs, pp = j / kbs, k = 64 * kb + 4 * c;
        const int g0 = pp * groups / P, g1 = (pp + 1) * groups / P;
        f4 acc[2][4];                                      // even and odd e: two chains
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][e] = acc[1][e] = (f4){0.f, 0.f, 0.f, 0.f};
        if (j != n.w) net_bwd_load(W, K, O, k, g0, g1, w);
#pragma unroll 1
        for (int g = g0; g < g1; g += kBwdBatch) {
            f4 nx[kBwdBatch][4];
            if (g + kBwdBatch < g1) net_bwd_load(W, K, O, k, g + kBwdBatch, g1, nx);
            f4 x[kBwdBatch];
#pragma unroll
            for (int i = 0; i < kBwdBatch; ++i) x[i] = net_quad(gout + c * ldg, 16 * (g + i) + 4 * q, O);
#pragma unroll
            for (int i = 0; i < kBwdBatch; ++i) {
                if (g + i >= g1) break;
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) acc[e & 1][e2] = mfma4(x[i][e], w[i][e][e2], acc[e & 1][e2]);
            }
#pragma unroll
            for (int i = 0; i < kBwdBatch; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) w[i][e] = nx[i][e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][e] += acc[1][e];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *(f4 *)(n.scr + (pp * kCtrBS + 4 * q + r) * 64 * kbs + k) =
                (f4){acc[0][0][r], acc[0][1][r], acc[0][2][r], acc[0][3][r]};
    }
}

// The sum of the parts: TS threads (adjacent lanes) per input k, each with
// 16 / TS of the samples.
template <int TS>
__device__ __forceinline__ void net_bwd_combine(float *gin, const float *in, int ldi, int K, int O, bool act,
                                                const float *__restrict__ slope, float *dsl, const NetRun &n)
{
    constexpr int NS = kCtrBS / TS;
    const int lds = 64 * net_kblocks(K), P = net_bwd_parts(K, O, n.nw), s0 = (n.t % TS) * NS;
    for (int k = n.t / TS; k < K; k += n.nt / TS) {
        const float a = slope ? slope[k] : 0.f;
        float d[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) d[s] = 0.f;
        for (int pp = 0; pp < P; ++pp)
#pragma unroll
            for (int s = 0; s < NS; ++s) d[s] += n.scr[(pp * kCtrBS + s0 + s) * lds + k];
        float ds = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int x = (s0 + s) * ldi + k;
            if (act) {
                const float z = slope ? gin[x] : in[x];
                const bool pos = z > 0.f;
                ds = fmaf(pos ? 0.f : z, d[s], ds);
                d[s] = pos ? d[s] : slope ? a * d[s] : 0.f;
            }
            gin[x] = d[s];
        }
        if (act) {
#pragma unroll
            for (int o = 1; o < TS; o <<= 1) ds += __shfl_xor(ds, o, AMS_WAVE);
            if (n.t % TS == 0) dsl[k] = slope ? ds : 0.f;
        }
    }
}

// The data gradients run down the layers first, two halves per layer with a
// barrier after each (the parts, then their sum); the weight gradients, whose
// stores a later load's wait would have to sit out, come after all of them
// (every layer's activations and gradients stay in LDS).
__device__ __forceinline__ void net_bwd_preload(const CtrArgs &a, const NetRun &n, int l, f4 (&w)[kBwdBatch][4])
{
    const int K = a.dims[l], O = a.dims[l + 1], kbs = net_kblocks(K), P = net_bwd_parts(K, O, n.nw);
    if (n.w < kbs * P) {
        const int pp = n.w / kbs, groups = (O + 15) / 16;
        net_bwd_load(a.W[l], K, O, 64 * (n.w % kbs) + 4 * (ams_lane() & 15), pp * groups / P, (pp + 1) * groups / P, w);
    }
}

__device__ __forceinline__ void net_bwd_first(const CtrArgs &a, const NetRun &n, int l, f4 (&w)[kBwdBatch][4])
{
    const int K = a.dims[l], O = a.dims[l + 1];
    net_bwd_parts_out(a.W[l], K, O, n.grd + net_off(a, l + 1), net_ld(O), n, w);
    if (l > 0) net_bwd_preload(a, n, l - 1, w);
}

__device__ __forceinline__ void net_bwd_weights(const CtrArgs &a, const NetRun &n, float *p)
{
#pragma unroll 1
    for (int l = 0; l < a.L; ++l) {
        const int K = a.dims[l], O = a.dims[l + 1], oi = net_off(a, l);
        net_bwd_weight(n.grd + oi + kCtrBS * net_ld(K), net_ld(O), O, n.act + oi, net_ld(K), K, p, n);
        p += net_layer_size(a, l);
    }
}

__device__ __forceinline__ void net_bwd_second(const CtrArgs &a, const NetRun &n, int l, float *p)
{
    const int K = a.dims[l];
    // the activation below layer l belongs to layer l - 1: its slot follows
    // that layer's dW and db
    float *dsl = p;
    if (l > 0) {
        for (int x = 0; x < l - 1; ++x) dsl += net_layer_size(a, x);
        dsl += K * a.dims[l - 1] + K;
    }
    const int oi = net_off(a, l);
    const float *slope = l > 0 ? a.slope[l - 1] : nullptr;
    if (4 * K <= n.nt) net_bwd_combine<4>(n.grd + oi, n.act + oi, net_ld(K), K, a.dims[l + 1], l > 0, slope, dsl, n);
    else net_bwd_combine<2>(n.grd + oi, n.act + oi, net_ld(K), K, a.dims[l + 1], l > 0, slope, dsl, n);
}

__device__ __forceinline__ void net_store_dfields(const CtrArgs &a, const NetRun &n, int b0, int B)
{
    const int K0 = a.dims[0], ld0 = net_ld(K0);
    for (int e = n.t; e < kCtrBS * K0; e += n.nt) {
        const int s = e / K0, k = e - s * K0;
        if (b0 + s >= B) continue;
        float *p = net_field(a, k, b0 + s, true);
        if (p) *p = n.grd[s * ld0 + k];
    }
}

constexpr int kCtrWaves = kCtrThreads / AMS_WAVE;

// LDS of a block: per net act and grd, then the samples' losses and the parts
// of the data gradients.
inline size_t ctr_lds_bytes(const CtrArgs &a)
{
    return (size_t)(2 * net_act_floats(a) + kCtrBS + net_scr_floats(a, kCtrWaves)) * 4;
}

// Which widths the calls take: the sum of the nets' activations, twice, and of
// the parts of a 512-thread block's widest layer has to fit the LDS.  What the
// kernels themselves need, with rows padded to whole quads and parts of whole
// 64-column blocks, is a little more (72-200-80-2: 79,936 bytes where this says
// 77,632) and is checked beside it; the widest CTR net takes 117,824 bytes, so on
// a device with 160 KB for a block only this rule refuses one.
inline size_t net_width_bytes(const CtrArgs *const *nets, int count)
{
    int act = 0, parts = 0;
    for (int i = 0; i < count; ++i) {
        const CtrArgs &a = *nets[i];
        for (int l = 0; l <= a.L; ++l) act += kCtrBS * a.dims[l];
        for (int l = 0; l < a.L; ++l) {
            const int K = a.dims[l], O = a.dims[l + 1];
            const int pf = min(max(kCtrThreads / O, 1), (K + 15) / 16), pb = min(max(kCtrThreads / K, 1), (O + 7) / 8);
            if (pf > 1) parts = max(parts, pf * kCtrBS * O);
            if (pb > 1) parts = max(parts, pb * kCtrBS * K);
        }
    }
    return (size_t)(2 * act + parts + kCtrBS) * 4;
}

// The towers run side by side, each with its own parts; where that does not
// fit the LDS (tight), their backwards take turns with one area for both,
// which every pair of widths that the call takes fits.
inline size_t dssm_lds_bytes(const CtrArgs &u, const CtrArgs &v, bool tight)
{
    const int su = net_scr_floats(u, kCtrWaves / 2), sv = net_scr_floats(v, kCtrWaves / 2);
    return (size_t)(2 * (net_act_floats(u) + net_act_floats(v)) + kCtrBS + (tight ? max(su, sv) : su + sv)) * 4;
}

// One block = kCtrBS samples: forward through every layer in LDS, softmax
// and cross-entropy, then the backward; the block's gradient and loss sums
// (over its samples, ascending) go to its partial row.
__global__ __launch_bounds__(kCtrThreads) void ctr_fb_k(CtrArgs a, int B, const int32_t *__restrict__ labels,
                                                     float *__restrict__ prob, float *__restrict__ part, int PS)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    net_args_touch<sizeof(CtrArgs) / 64 + 1>();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / AMS_WAVE);
    float *lossv = lds + 2 * net_act_floats(a);
    const NetRun n = net_run(a, lds, lossv + kCtrBS, wave, kCtrWaves);
    const int t = threadIdx.x;
    const int b0 = blockIdx.x * kCtrBS;
    const int L = a.L, C = a.dims[L];
    f4 w[kFwdBatch];
    if (16 * wave < a.dims[1]) net_fwd_load(a.W[0], a.dims[0], a.dims[1], wave, 0, w);
    const int y = t < kCtrBS && b0 + t < B ? labels[b0 + t] : -1;
    net_load(a, n, b0, B);
    lds_barrier();
#pragma unroll 1
    for (int l = 0; l < L; ++l) {
        net_fwd_layer(a, n, l, w);
        lds_barrier();
    }
    f4 wb[kBwdBatch][4];
    net_bwd_preload(a, n, L - 1, wb);
    // softmax, cross-entropy, dlogits = (p - onehot(y)) / B
    if (t < kCtrBS) {
        const int s = t, i = b0 + s;
        const int oz = net_off(a, L) + s * net_ld(C);
        const float *z = n.act + oz;
        float *gz = n.grd + oz;
        float ls = 0.f;
        if (i < B && y >= 0 && y < C) {
            float m = z[0];
            for (int c = 1; c < C; ++c) m = fmaxf(m, z[c]);
            float se = 0.f;
            for (int c = 0; c < C; ++c) se += expf(z[c] - m);
            const float lse = m + logf(se);
            for (int c = 0; c < C; ++c) {
                const float pc = expf(z[c] - lse);
                if (prob) prob[(size_t)i * C + c] = pc;
                gz[c] = (pc - (c == y ? 1.f : 0.f)) / (float)B;
            }
            ls = lse - z[y];
        } else {
            for (int c = 0; c < C; ++c) gz[c] = 0.f;
            if (i < B && prob)
                for (int c = 0; c < C; ++c) prob[(size_t)i * C + c] = 0.f;
        }
        lossv[s] = ls;
    }
    lds_barrier();
    float *p = part + (size_t)blockIdx.x * PS;
#pragma unroll 1
    for (int l = L - 1; l >= 0; --l) {
        net_bwd_first(a, n, l, wb);
        lds_barrier();
        net_bwd_second(a, n, l, p);
        lds_barrier();
    }
    net_store_dfields(a, n, b0, B);
    net_bwd_weights(a, n, p);
    if (t == 0) {
        float ls = 0.f;
        for (int s = 0; s < kCtrBS; ++s) ls += lossv[s];
        p[PS - 4] = ls;
    }
}

// Pre-rank model (section 6): a user tower and an ad tower on their own
// fields, score s = <u, a> of their outputs, click probability sigmoid(s),
// logistic loss softplus(s) - y s for y in {0, 1} (other labels add
// nothing), divided by B.  Same block layout as the CTR kernel with both
// towers in LDS, four waves each side by side; the partial row holds the user
// tower's gradients, then the ad tower's, then the loss sum.
struct TowerArgs {
    CtrArgs n[2];                            // user, ad
};

__global__ __launch_bounds__(kCtrThreads) void dssm_fb_k(TowerArgs a2, int tight, int B, const int32_t *__restrict__ labels,
                                                      float *__restrict__ prob, float *__restrict__ part, int PS)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    constexpr int half = kCtrWaves / 2;
    net_args_touch<sizeof(TowerArgs) / 64 + 1>();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / AMS_WAVE);
    const int ad = wave / half;
    const CtrArgs &a = a2.n[ad], &u = a2.n[0], &v = a2.n[1];
    const int fu = 2 * net_act_floats(u);
    float *lossv = lds + fu + 2 * net_act_floats(v), *scr = lossv + kCtrBS;
    const NetRun n = net_run(a, lds + (ad ? fu : 0), scr + (ad && !tight ? net_scr_floats(u, half) : 0), wave % half, half);
    const int t = threadIdx.x;
    const int b0 = blockIdx.x * kCtrBS;
    const int R = u.dims[u.L], Lmax = max(u.L, v.L);
    f4 w[kFwdBatch];
    if (16 * n.w < a.dims[1]) net_fwd_load(a.W[0], a.dims[0], a.dims[1], n.w, 0, w);
    const int y = t < kCtrBS && b0 + t < B ? labels[b0 + t] : -1;
    net_load(a, n, b0, B);
    lds_barrier();
#pragma unroll 1
    for (int l = 0; l < Lmax; ++l) {
        if (l < a.L) net_fwd_layer(a, n, l, w);
        lds_barrier();
    }
    f4 wb[kBwdBatch][4];
    net_bwd_preload(a, n, a.L - 1, wb);
    if (t < kCtrBS) {
        const int s = t, i = b0 + s;
        const int ld = net_ld(R), ou = net_off(u, u.L) + s * ld, ov = fu + net_off(v, v.L) + s * ld;
        const float *zu = lds + ou, *zv = lds + ov;
        float sc = 0.f;
        for (int r = 0; r < R; ++r) sc = fmaf(zu[r], zv[r], sc);
        const float pr = 1.f / (1.f + expf(-sc));
        float ls = 0.f, g = 0.f;
        if (i < B) {
            if (prob) prob[i] = pr;
            if (y == 0 || y == 1) {
                ls = fmaxf(sc, 0.f) + log1pf(expf(-fabsf(sc))) - (float)y * sc;
                g = (pr - (float)y) / (float)B;
            }
        }
        float *gu = lds + net_act_floats(u) + ou, *gv = lds + net_act_floats(v) + ov;
        for (int r = 0; r < R; ++r) {
            gu[r] = g * zv[r];
            gv[r] = g * zu[r];
        }
        lossv[s] = ls;
    }
    lds_barrier();
    float *p = part + (size_t)blockIdx.x * PS;
    float *pn = p + (ad ? net_part_size(u) : 0);
#pragma unroll 1
    for (int i = 0; i < (tight ? 2 : 1) * Lmax; ++i) {
        const int l = a.L - 1 - i % Lmax;
        const bool mine = l >= 0 && (!tight || i / Lmax == ad);
        if (mine) net_bwd_first(a, n, l, wb);
        lds_barrier();
        if (mine) net_bwd_second(a, n, l, pn);
        lds_barrier();
    }
    net_store_dfields(a, n, b0, B);
    net_bwd_weights(a, n, pn);
    if (t == 0) {
        float ls = 0.f;
        for (int s = 0; s < kCtrBS; ++s) ls += lossv[s];
        p[PS - 4] = ls;
    }
}

// Where the reduced partial rows go: per layer (of one net, or of the two
// towers one after the other) dW, db and, below a net's last layer, the
// slope gradient (NULL: not stored), at the offsets of the partial row; the loss sum sits at PS - 4.
struct RedLayer {
    int off, K, O, hidden;
    float *dW, *db, *ds;
};

struct CtrOut {
    int nl;
    RedLayer ly[2 * kCtrMaxLayers];
    float *loss;
    int B;
};

// Fixed-order sum of the blocks' partial rows, scattered into the gradients
// and the mean loss.  A block takes 64 elements; each of its 16 waves sums a
// sixteenth of the G rows (eight running chains over g = 8 i + r, added
// r = 0..7), and the sixteenths are added in order.  4096 samples of the
// 72-200-80-2 net (31 MB of partial rows): with four waves per 64 elements
// 8.5 us, 8.1 us so; the towers' 9 k elements 6.4 and 5.0 us (more loads in
// flight).
constexpr int kRedCols = AMS_WAVE, kRedWaves = 16, kRedThreads = kRedWaves * AMS_WAVE;

__global__ __launch_bounds__(kRedThreads) void ctr_reduce_k(const float *__restrict__ part, int G, int PS, CtrOut o)
{
    __shared__ float q16[kRedWaves][kRedCols];
    const int c = threadIdx.x % kRedCols, qt = threadIdx.x / kRedCols;
    const int e = blockIdx.x * kRedCols + c;
    const int g0 = (int)((int64_t)qt * G / kRedWaves), g1 = (int)((int64_t)(qt + 1) * G / kRedWaves);
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (e < PS) {
        int g = g0;
        for (; g + 8 <= g1; g += 8)
#pragma unroll
            for (int r = 0; r < 8; ++r) s[r] += part[(size_t)(g + r) * PS + e];
        for (int r = 0; g + r < g1; ++r) s[r] += part[(size_t)(g + r) * PS + e];
    }
    float sub = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) sub += s[r];
    q16[qt][c] = sub;
    __syncthreads();
    if (qt != 0 || e >= PS) return;
    float tot = q16[0][c];
#pragma unroll
    for (int q = 1; q < kRedWaves; ++q) tot += q16[q][c];
    if (e == PS - 4) {
        *o.loss = tot / (float)o.B;
        return;
    }
    for (int l = 0; l < o.nl; ++l) {
        const RedLayer &y = o.ly[l];
        int x = e - y.off;
        if (x < 0) return;                     // padding before this layer
        const int nw = y.O * y.K;
        if (x < nw) {
            y.dW[x] = tot;
            return;
        }
        x -= nw;
        if (x < y.O) {
            y.db[x] = tot;
            return;
        }
        x -= y.O;
        if (y.hidden && x < y.O) {
            if (y.ds) y.ds[x] = tot;
            return;
        }
    }
}

// ---------------------------------------------------------------- Adagrad

// One thread per 4 elements of a touched row when D % 4 == 0 and the arrays
// are 16-byte aligned (vec4), else per element; a grid-stride loop over the
// n_u rows the device counted (the grid is sized for at most kAdaBlocks, not
// for the host cap, whose blocks past n_u would each still be dispatched).
constexpr int kAdaBlocks = 2048;
__device__ __forceinline__ float ada_one(float p, float g, float &a, float lr, float eps)
{
    a = a + g * g;
    return p - lr * g / (sqrtf(a) + eps);
}

__global__ __launch_bounds__(kThreads) void adagrad_k(int D, const int32_t *__restrict__ uniq,
                                                      const int32_t *__restrict__ n_uniq_p, int cap,
                                                      const float *__restrict__ grad, float *__restrict__ table,
                                                      int64_t n_rows, float *__restrict__ accum, float lr, float eps,
                                                      int vec4)
{
    const int n_u = min(*n_uniq_p, cap);
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    if (vec4) {
        const int D4 = D / 4;
        const int64_t n4 = (int64_t)n_u * D4;
        for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n4; e += stride) {
            const int u = (int)(e / D4), d = (int)(e % D4) * 4;
            const int r = uniq[u];
            if (r < 0 || (int64_t)r >= n_rows) continue;
            const float4 g = *(const float4 *)(grad + (size_t)u * D + d);
            const size_t x = (size_t)r * D + d;
            float4 a = *(const float4 *)(accum + x), t = *(const float4 *)(table + x);
            t.x = ada_one(t.x, g.x, a.x, lr, eps);
            t.y = ada_one(t.y, g.y, a.y, lr, eps);
            t.z = ada_one(t.z, g.z, a.z, lr, eps);
            t.w = ada_one(t.w, g.w, a.w, lr, eps);
            *(float4 *)(accum + x) = a;
            *(float4 *)(table + x) = t;
        }
    } else {
        const int64_t n = (int64_t)n_u * D;
        for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += stride) {
            const int u = (int)(e / D), d = (int)(e % D);
            const int r = uniq[u];
            if (r < 0 || (int64_t)r >= n_rows) continue;
            const size_t x = (size_t)r * D + d;
            float a = accum[x];
            table[x] = ada_one(table[x], grad[e], a, lr, eps);
            accum[x] = a;
        }
    }
}

// ------------------------------------------------------------------- Adam

struct AdamK {
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float adam_one(float p, float g, float &m, float &v, const AdamK &k)
{
    m = k.b1 * m + (1.f - k.b1) * g;
    v = k.b2 * v + (1.f - k.b2) * g * g;
    return p - k.lr * (m / k.c1) / (sqrtf(v / k.c2) + k.eps);
}

// Scalar form: any alignment.
__global__ __launch_bounds__(kThreads) void adam_k(int64_t n, float *__restrict__ param,
                                                   const float *__restrict__ grad, float *__restrict__ m,
                                                   float *__restrict__ v, AdamK k, uint16_t *__restrict__ pb)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        float mi = m[i], vi = v[i];
        const float p = adam_one(param[i], grad[i], mi, vi, k);
        m[i] = mi;
        v[i] = vi;
        param[i] = p;
        if (pb) pb[i] = ams_f32_to_bf16(p);
    }
}

// 16-byte form (param, grad, m, v 16-byte aligned, the bf16 copy 8-byte
// aligned): quad q = elements 4q..4q+3; the n % 4 last elements go to the
// first threads of the grid.  Same arithmetic per element as adam_k.
__global__ __launch_bounds__(kThreads) void adam4_k(int64_t n, float *__restrict__ param,
                                                    const float *__restrict__ grad, float *__restrict__ m,
                                                    float *__restrict__ v, AdamK k, uint16_t *__restrict__ pb)
{
    const int64_t nq = n / 4, t0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t q = t0; q < nq; q += (int64_t)gridDim.x * kThreads) {
        const float4 g = ((const float4 *)grad)[q];
        float4 p = ((float4 *)param)[q], mm = ((float4 *)m)[q], vv = ((float4 *)v)[q];
        p.x = adam_one(p.x, g.x, mm.x, vv.x, k);
        p.y = adam_one(p.y, g.y, mm.y, vv.y, k);
        p.z = adam_one(p.z, g.z, mm.z, vv.z, k);
        p.w = adam_one(p.w, g.w, mm.w, vv.w, k);
        ((float4 *)param)[q] = p;
        ((float4 *)m)[q] = mm;
        ((float4 *)v)[q] = vv;
        if (pb)
            ((uint2 *)pb)[q] = make_uint2((uint32_t)ams_f32_to_bf16(p.x) | ((uint32_t)ams_f32_to_bf16(p.y) << 16),
                                          (uint32_t)ams_f32_to_bf16(p.z) | ((uint32_t)ams_f32_to_bf16(p.w) << 16));
    }
    const int64_t i = 4 * nq + t0;
    if (i < n) {
        float mi = m[i], vi = v[i];
        const float p = adam_one(param[i], grad[i], mi, vi, k);
        m[i] = mi;
        v[i] = vi;
        param[i] = p;
        if (pb) pb[i] = ams_f32_to_bf16(p);
    }
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// Widths a net of the CTR kind accepts: 1..kCtrMaxLayers layers, inputs up
// to kCtrMaxIn, hidden widths up to kCtrMaxHidden; the output width is
// checked by the caller (classes, or a tower's representation).
bool net_dims_ok(const ams_ctr *net, int min_layers)
{
    if (!net || net->n_layers < min_layers || net->n_layers > kCtrMaxLayers) return false;
    if (net->dims[0] < 1 || net->dims[0] > kCtrMaxIn) return false;
    for (int l = 1; l < net->n_layers; ++l)
        if (net->dims[l] < 1 || net->dims[l] > kCtrMaxHidden) return false;
    return true;
}

bool ctr_ok(const ams_ctr *net)
{
    if (!net_dims_ok(net, 2)) return false;
    const int C = net->dims[net->n_layers];
    return C >= 2 && C <= kCtrMaxC;
}

bool tower_ok(const ams_ctr *net)
{
    if (!net_dims_ok(net, 1)) return false;
    const int R = net->dims[net->n_layers];
    return R >= 1 && R <= kTowerMaxOut;
}

// LDS a block may have on the current device (gfx950's 160 KiB if it cannot
// be asked).
size_t lds_limit()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || n <= 0)
        n = 160 * 1024;
    return (size_t)n;
}

// Fill a net's arguments; NULL pointers where the ABI requires them give NULL.
ams_status net_args(const ams_ctr *net, int32_t n_fields, const float *const *fields, const int32_t *field_dims,
                    const float *const *W, const float *const *b, const float *const *slope,
                    float *const *dfields, CtrArgs &a)
{
    if (!fields || !field_dims || !W || !b) return AMS_ERR_NULL;
    if (n_fields < 1 || n_fields > kCtrMaxFields) return AMS_ERR_DIMS;
    a = CtrArgs{};
    a.L = net->n_layers;
    for (int l = 0; l <= a.L; ++l) a.dims[l] = net->dims[l];
    a.n_fields = n_fields;
    int width = 0;
    for (int f = 0; f < n_fields; ++f) {
        if (field_dims[f] < 1) return AMS_ERR_DIMS;
        if (!fields[f]) return AMS_ERR_NULL;
        a.fdim[f] = field_dims[f];
        a.field[f] = fields[f];
        a.dfield[f] = dfields ? dfields[f] : nullptr;
        width += field_dims[f];
    }
    if (width != a.dims[0]) return AMS_ERR_DIMS;
    for (int l = 0; l < a.L; ++l) {
        if (!W[l] || !b[l]) return AMS_ERR_NULL;
        a.W[l] = W[l];
        a.b[l] = b[l];
        a.slope[l] = (slope && l < a.L - 1) ? slope[l] : nullptr;
    }
    return AMS_OK;
}

// Reduction targets of one net's layers, appended to o.
// base: where this net's part of the partial row starts.
ams_status net_out(const CtrArgs &a, float *const *dW, float *const *db, float *const *dslope, int base, CtrOut &o)
{
    if (!dW || !db) return AMS_ERR_NULL;
    for (int l = 0; l < a.L; ++l) {
        if (!dW[l] || !db[l]) return AMS_ERR_NULL;
        RedLayer &y = o.ly[o.nl++];
        y.off = base;
        base += net_layer_size(a, l);
        y.K = a.dims[l];
        y.O = a.dims[l + 1];
        y.hidden = l < a.L - 1;
        y.dW = dW[l];
        y.db = db[l];
        y.ds = (y.hidden && dslope && a.slope[l]) ? dslope[l] : nullptr;
    }
    return AMS_OK;
}

}  // namespace

extern "C" ams_status ams_bag_fwd(int32_t B, int32_t D, const int32_t *seg_off, int64_t n_beh,
                                  const int32_t *ids, const float *table, int64_t n_rows, float *bag, void *stream)
{
    if (B < 0 || n_beh < 0 || n_beh > INT32_MAX || n_rows < 0) return AMS_ERR_SIZE;
    if (D < 1 || D > 32) return AMS_ERR_DIMS;
    if (B == 0) return AMS_OK;
    if (!seg_off || !ids || !table || !bag) return AMS_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    const int grid = (B + kWaves - 1) / kWaves;
    if (D <= 16)
        AMS_LAUNCH("bag_fwd", st, bag_fwd_k<16><<<grid, kThreads, 0, st>>>(B, D, seg_off, n_beh, ids, table, n_rows, bag));
    else
        AMS_LAUNCH("bag_fwd", st, bag_fwd_k<32><<<grid, kThreads, 0, st>>>(B, D, seg_off, n_beh, ids, table, n_rows, bag));
    return ams_launch_status();
}

extern "C" size_t ams_bag_workspace(int32_t B, int64_t n_beh, int32_t D, int32_t n_uniq_cap)
{
    return ams_pool_workspace(AMS_POOL_SUM, B, n_beh, D, n_uniq_cap);
}

extern "C" ams_status ams_bag_bwd(int32_t B, int32_t D, const int32_t *seg_off, int64_t n_beh, const int32_t *inv,
                                  const int32_t *occ_perm, const int32_t *uniq_off, const int32_t *n_uniq,
                                  int32_t n_uniq_cap, const float *dbag, const float *dad, float *grad, void *ws,
                                  size_t ws_bytes, void *stream)
{
    (void)n_uniq;
    if (B > 0 && !dbag) return AMS_ERR_NULL;
    // the SUM aggregator's backward with the bag gradient as the upstream
    // gradient of behaviors and ads alike, the ads also taking dad
    return pool_bwd_sum_ads(B, D, seg_off, n_beh, inv, occ_perm, uniq_off, n_uniq_cap, dbag, dbag, dad, grad, ws,
                            ws_bytes, stream);
}

extern "C" size_t ams_ctr_workspace(const ams_ctr *net, int32_t B)
{
    if (!ctr_ok(net) || B < 0) return 0;
    CtrArgs a{};
    a.L = net->n_layers;
    for (int l = 0; l <= a.L; ++l) a.dims[l] = net->dims[l];
    const int G = (B + kCtrBS - 1) / kCtrBS;
    return al256((size_t)(G > 0 ? G : 1) * (net_part_size(a) + 4) * 4);
}

extern "C" ams_status ams_ctr_fwd_bwd(const ams_ctr *net, int32_t B, int32_t n_fields, const float *const *fields,
                                      const int32_t *field_dims, const int32_t *labels, const float *const *W,
                                      const float *const *b, const float *const *slope, float *loss, float *prob,
                                      float *const *dW, float *const *db, float *const *dslope,
                                      float *const *dfields, void *ws, size_t ws_bytes, void *stream)
{
    if (!net) return AMS_ERR_NULL;
    if (!ctr_ok(net)) return AMS_ERR_DIMS;
    if (B < 1) return AMS_ERR_SIZE;
    CtrArgs a;
    ams_status s = net_args(net, n_fields, fields, field_dims, W, b, slope, dfields, a);
    if (s != AMS_OK) return s;
    CtrOut o{};
    s = net_out(a, dW, db, dslope, 0, o);
    if (s != AMS_OK) return s;
    if (!labels || !loss) return AMS_ERR_NULL;
    const CtrArgs *nets[] = {&a};
    if (net_width_bytes(nets, 1) > lds_limit()) return AMS_ERR_DIMS;
    const size_t lds = ctr_lds_bytes(a);
    if (lds > lds_limit()) return AMS_ERR_DIMS;
    const int G = (B + kCtrBS - 1) / kCtrBS;
    const int PS = net_part_size(a) + 4;
    if (!ws || ws_bytes < (size_t)G * PS * 4) return AMS_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    float *part = (float *)ws;
    AMS_LAUNCH("ctr_fwd_bwd", st, ctr_fb_k<<<G, kCtrThreads, lds, st>>>(a, B, labels, prob, part, PS));
    o.loss = loss;
    o.B = B;
    AMS_LAUNCH("ctr_reduce", st, ctr_reduce_k<<<(PS + kRedCols - 1) / kRedCols, kRedThreads, 0, st>>>(part, G, PS, o));
    return ams_launch_status();
}

extern "C" size_t ams_dssm_workspace(const ams_ctr *user_net, const ams_ctr *ad_net, int32_t B)
{
    if (!tower_ok(user_net) || !tower_ok(ad_net) || B < 0) return 0;
    CtrArgs u{}, v{};
    u.L = user_net->n_layers;
    v.L = ad_net->n_layers;
    for (int l = 0; l <= u.L; ++l) u.dims[l] = user_net->dims[l];
    for (int l = 0; l <= v.L; ++l) v.dims[l] = ad_net->dims[l];
    const int G = (B + kCtrBS - 1) / kCtrBS;
    return al256((size_t)(G > 0 ? G : 1) * (net_part_size(u) + net_part_size(v) + 4) * 4);
}

extern "C" ams_status ams_dssm_fwd_bwd(const ams_ctr *user_net, const ams_ctr *ad_net, int32_t B,
                                       int32_t n_user_fields, const float *const *user_fields,
                                       const int32_t *user_field_dims, int32_t n_ad_fields,
                                       const float *const *ad_fields, const int32_t *ad_field_dims,
                                       const int32_t *labels, const float *const *Wu, const float *const *bu,
                                       const float *const *slope_u, const float *const *Wa,
                                       const float *const *ba, const float *const *slope_a, float *loss,
                                       float *prob, float *const *dWu, float *const *dbu,
                                       float *const *dslope_u, float *const *dWa, float *const *dba,
                                       float *const *dslope_a, float *const *duser_fields,
                                       float *const *dad_fields, void *ws, size_t ws_bytes, void *stream)
{
    if (!user_net || !ad_net) return AMS_ERR_NULL;
    if (!tower_ok(user_net) || !tower_ok(ad_net)) return AMS_ERR_DIMS;
    if (user_net->dims[user_net->n_layers] != ad_net->dims[ad_net->n_layers]) return AMS_ERR_DIMS;
    if (B < 1) return AMS_ERR_SIZE;
    CtrArgs u, v;
    ams_status s = net_args(user_net, n_user_fields, user_fields, user_field_dims, Wu, bu, slope_u, duser_fields, u);
    if (s != AMS_OK) return s;
    s = net_args(ad_net, n_ad_fields, ad_fields, ad_field_dims, Wa, ba, slope_a, dad_fields, v);
    if (s != AMS_OK) return s;
    CtrOut o{};
    s = net_out(u, dWu, dbu, dslope_u, 0, o);
    if (s != AMS_OK) return s;
    s = net_out(v, dWa, dba, dslope_a, net_part_size(u), o);
    if (s != AMS_OK) return s;
    if (!labels || !loss) return AMS_ERR_NULL;
    const CtrArgs *nets[] = {&u, &v};
    if (net_width_bytes(nets, 2) > lds_limit()) return AMS_ERR_DIMS;
    const bool tight = dssm_lds_bytes(u, v, false) > lds_limit();
    const size_t lds = dssm_lds_bytes(u, v, tight);
    if (lds > lds_limit()) return AMS_ERR_DIMS;
    const int G = (B + kCtrBS - 1) / kCtrBS;
    const int PS = net_part_size(u) + net_part_size(v) + 4;
    if (!ws || ws_bytes < (size_t)G * PS * 4) return AMS_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    float *part = (float *)ws;
    AMS_LAUNCH("dssm_fwd_bwd", st, dssm_fb_k<<<G, kCtrThreads, lds, st>>>(TowerArgs{{u, v}}, tight, B, labels, prob, part,
                                                                           PS));
    o.loss = loss;
    o.B = B;
    AMS_LAUNCH("ctr_reduce", st, ctr_reduce_k<<<(PS + kRedCols - 1) / kRedCols, kRedThreads, 0, st>>>(part, G, PS, o));
    return ams_launch_status();
}

extern "C" ams_status ams_adagrad_rows(int32_t D, const int32_t *uniq, const int32_t *n_uniq, int32_t n_uniq_cap,
                                       const float *grad, float *table, int64_t n_rows, float *accum, float lr,
                                       float eps, void *stream)
{
    if (D < 1 || n_uniq_cap < 0 || n_rows < 0) return AMS_ERR_SIZE;
    if (n_uniq_cap == 0) return AMS_OK;
    if (!uniq || !n_uniq || !grad || !table || !accum) return AMS_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    const int vec4 = (D % 4 == 0) && ((((uintptr_t)grad) | ((uintptr_t)table) | ((uintptr_t)accum)) & 15) == 0;
    const int64_t n = (int64_t)n_uniq_cap * (vec4 ? D / 4 : D);
    const int64_t g = (n + kThreads - 1) / kThreads;
    AMS_LAUNCH("adagrad_rows", st, adagrad_k<<<(unsigned)(g < kAdaBlocks ? g : kAdaBlocks), kThreads, 0, st>>>(
                                       D, uniq, n_uniq, n_uniq_cap, grad, table, n_rows, accum, lr, eps, vec4));
    return ams_launch_status();
}

extern "C" ams_status ams_adam_update(int64_t n, float *param, const float *grad, float *m, float *v, float lr,
                                      float b1, float b2, float eps, int64_t t, uint16_t *param_bf16, void *stream)
{
    if (n < 0 || t < 1) return AMS_ERR_SIZE;
    if (n == 0) return AMS_OK;
    if (!param || !grad || !m || !v) return AMS_ERR_NULL;
    // bias corrections of step t, formed in double on the host
    AdamK k{lr, b1, b2, eps, (float)(1.0 - pow((double)b1, (double)t)), (float)(1.0 - pow((double)b2, (double)t))};
    hipStream_t st = (hipStream_t)stream;
    const bool v4 = ((((uintptr_t)param | (uintptr_t)grad | (uintptr_t)m | (uintptr_t)v) & 15) == 0) &&
                    (((uintptr_t)param_bf16 & 7) == 0);
    const int64_t work = v4 ? (n + 3) / 4 : n;
    int64_t g = (work + kThreads - 1) / kThreads;
    if (g > 4096) g = 4096;
    if (v4)
        AMS_LAUNCH("adam_update", st, adam4_k<<<(unsigned)g, kThreads, 0, st>>>(n, param, grad, m, v, k, param_bf16));
    else
        AMS_LAUNCH("adam_update", st, adam_k<<<(unsigned)g, kThreads, 0, st>>>(n, param, grad, m, v, k, param_bf16));
    return ams_launch_status();
}
