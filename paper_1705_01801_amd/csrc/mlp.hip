// Surrogate MLP: dense layers with tanh hidden activations and a linear
// output, BF16 weights and activations, FP32 accumulation on MFMA, FP32
// master weights updated by Adam.  Trained on spectra produced by the batched
// LBM to map horn-profile parameters to resonant frequencies.
//
// Precision points (the CPU check follows the same ones): the input x, the
// weights used in products and the hidden activations are rounded to BF16;
// products accumulate in FP32; biases, pre-activations, loss and gradients
// are FP32; the output-layer gradient and the hidden-layer gradients are
// rounded to BF16 before they enter a product.
//
// Networks of up to 8 layers of at most 256 units (the surrogate's are 3-256-
// 256-256-10) run in few launches, because at these sizes a launch costs more
// than a layer:
//  - rows_kernel takes 4 to 64 rows of the batch through all layers, the
//    activations in LDS, and when training on through the loss and the
//    gradients with respect to every layer's pre-activations, which are as
//    local to a row as the forward pass is;
//  - weights_kernel forms every layer's weight and bias gradient (sums over
//    the batch) and applies Adam to them in its epilogue.
// A forward pass is one launch, a training step two.  Both read every operand
// with 16-byte loads: the weights are kept as two BF16 copies in the order in
// which the forward and the backward products take them (frag_place),
// and rows_kernel writes activations and gradients transposed, so that the
// batch, over which weights_kernel sums, is contiguous.  The next layer's
// weights are loaded while a layer's epilogue runs.  Both issue the products
// of gemm_kernel below in its order, so the results are the same bits.
// (The loss, a sum of FP32 shares, is added up in another order.)
// Forward of 10,000 rows, 3-256-256-256-10: 74 us with a launch per layer, 13.6
// so, most of it the tanh of 7.7 million activations.  A training
// step of 512 rows: 72 us in nine launches; 17 + 10 us in two.  rows_kernel is
// bound by each CU reading every weight (0.85 us per 256 x 256 layer at 64
// bytes a cycle) and by the chain of layers, weights_kernel by a trip to
// memory for its operands.  Loading two layers ahead, and workgroups that only
// warm the caches, made no difference.
//
// Larger networks: every product is one kernel, gemm_kernel, with the
// elementwise work of the layer fused into its epilogue: bias + tanh (hidden
// forward), bias (output forward), bias + squared-error loss with the output
// gradient (training forward), tanh backward (hidden gradient), and the bias
// gradient as the row sums of the weight-gradient product.  A launch may carry two independent
// products (a layer's weight gradient and its input gradient), so a training
// step is L forward launches, L backward launches and one Adam launch.
//
// MFMA layout (v_mfma_f32_16x16x32_bf16): a wave computes one 16 x 16 tile
// of C = A B over K in steps of 32; lane l supplies row/column l % 16 and
// eight consecutive k values of group l / 16; the accumulator holds rows
// 4 (l / 16) + j, column l % 16.  A workgroup of four waves covers 32 x 32.
// The matrices are small (at most max_batch x 4096) and read with arbitrary
// strides: where an operand's k index is contiguous and its rows 16-byte
// aligned a lane reads its eight values with one 16-byte load, otherwise with
// eight 2-byte loads.  Loads are branch-free (an out-of-range element reads
// element 0 and is replaced by zero), and four K steps are loaded before
// their products, so a K of 128 costs one memory latency.
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "host_util.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

using lbw::fail;
using lbw::hip_fail;

namespace {

constexpr int kEpiNone = -1;         // no second product
constexpr int kEpiBias = 0;          // outf = acc + bias
constexpr int kEpiBiasTanh = 1;      // outb = bf16(tanh(acc + bias))
constexpr int kEpiBiasLoss = 2;      // outf = y = acc + bias; dz, partial loss (below)
constexpr int kEpiWeightGrad = 3;    // outf = acc; rowsum[m] = sum_k A(m, k)
constexpr int kEpiTanhBack = 4;      // outb = bf16(acc (1 - y^2)), y = act[m][n]
constexpr int kKSteps = 4;           // K steps of 32 loaded before their products

// C[m][n] = sum_k A(m, k) B(k, n) over m < M, n < N, k < K, with
// A(m, k) = A[m sam + k sak] and B(k, n) = B[k sbk + n sbn]; C row stride ldo.
struct Gemm {
    const __bf16* A;
    int64_t sam, sak;
    const __bf16* B;
    int64_t sbk, sbn;
    int M, N, K;
    int64_t ldo;
    int tiles_m;           // ceil(M / 32); tile id = tile_n * tiles_m + tile_m
    const float* bias;     // [N]
    float* outf;           // FP32 output
    __bf16* outb;          // BF16 output
    const __bf16* act;     // tanh backward: stored activation, layout of C
    float* rowsum;         // weight gradient: bias gradient [M]
    const float* t;        // loss: targets, layout of C
    const float* w;        // loss: weights, layout of C, NULL = 1
    float inv;             // loss: 1 / sum of weights
    __bf16* dz;            // loss: bf16(2 w (y - t) inv), layout of C
    float* partial;        // loss: sum of w (y - t)^2 per tile
};

// Work done once per launch by workgroup 0 besides its tile.
struct Extra {
    int64_t* counter;           // += 1 (training step counter), or NULL
    const float* fin_partial;   // loss = inv * sum of fin_partial[0, fin_n), or NULL
    int fin_n;
    float fin_inv;
    float* fin_loss;
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Eight consecutive k values kb .. kb + 7 of row `row` of an operand with
// element (row, k) at P[row s_row + k s_k]; zero outside row < nrow, k < K.
// VEC: s_k == 1, K % 8 == 0 and every row start 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ bf16x8 fragment(const __bf16* __restrict__ P, int64_t s_row, int64_t s_k, int row,
                                           int nrow, int kb, int K) {
    if constexpr (VEC) {
        const bool ok = row < nrow && kb < K;
        const int64_t idx = ok ? (int64_t)row * s_row + kb : 0;
        uint4 raw = *reinterpret_cast<const uint4*>(P + idx);
        raw.x = ok ? raw.x : 0u;
        raw.y = ok ? raw.y : 0u;
        raw.z = ok ? raw.z : 0u;
        raw.w = ok ? raw.w : 0u;
        return __builtin_bit_cast(bf16x8, raw);
    } else {
        bf16x8 out;
        const bool rok = row < nrow;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool ok = rok && kb + j < K;
            const int64_t idx = ok ? (int64_t)row * s_row + (int64_t)(kb + j) * s_k : 0;
            const __bf16 v = P[idx];
            out[j] = ok ? v : (__bf16)0.0f;
        }
        return out;
    }
}

template <int EPI, bool AV, bool BV>
__device__ __forceinline__ void gemm_tile(const Gemm& g, int tm, int tn) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, grp = lane >> 4;
    const int m0 = tm * 32 + (wave & 1) * 16, n0 = tn * 32 + (wave >> 1) * 16;
    const int am = m0 + r, bn = n0 + r;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f}, accs = {0.f, 0.f, 0.f, 0.f};
    // the waves holding column 0 also multiply A by ones: row sums of A
    const bool sums = EPI == kEpiWeightGrad && g.rowsum && n0 == 0;
    bf16x8 ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = sums ? (__bf16)1.0f : (__bf16)0.0f;
    // epilogue operands, loaded branch-free before the products
    const int n = n0 + r;
    const bool nok = n < g.N;
    float bias = 0.f, e1[4] = {0.f, 0.f, 0.f, 0.f}, e2[4] = {1.f, 1.f, 1.f, 1.f};
    if constexpr (EPI == kEpiBias || EPI == kEpiBiasTanh || EPI == kEpiBiasLoss) {
        const float bv = g.bias[nok ? n : 0];
        bias = nok ? bv : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = m0 + 4 * grp + j;
        const bool ok = nok && m < g.M;
        const int64_t o = ok ? (int64_t)m * g.ldo + n : 0;
        if constexpr (EPI == kEpiTanhBack) e1[j] = (float)g.act[o];
        if constexpr (EPI == kEpiBiasLoss) {
            e1[j] = g.t[o];
            if (g.w) e2[j] = g.w[o];
        }
    }
    for (int k0 = 0; k0 < g.K; k0 += 32 * kKSteps) {
        bf16x8 a[kKSteps], b[kKSteps];
#pragma unroll
        for (int u = 0; u < kKSteps; ++u) {
            const int kb = k0 + 32 * u + 8 * grp;
            a[u] = fragment<AV>(g.A, g.sam, g.sak, am, g.M, kb, g.K);
            b[u] = fragment<BV>(g.B, g.sbn, g.sbk, bn, g.N, kb, g.K);
        }
#pragma unroll
        for (int u = 0; u < kKSteps; ++u) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[u], acc, 0, 0, 0);
            if constexpr (EPI == kEpiWeightGrad) accs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], ones, accs, 0, 0, 0);
        }
    }
    float lsum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = m0 + 4 * grp + j;
        if (m < g.M && nok) {
            const int64_t o = (int64_t)m * g.ldo + n;
            const float v = acc[j];
            if constexpr (EPI == kEpiBias) {
                g.outf[o] = v + bias;
            } else if constexpr (EPI == kEpiBiasTanh) {
                g.outb[o] = (__bf16)tanhf(v + bias);
            } else if constexpr (EPI == kEpiBiasLoss) {
                const float y = v + bias;
                g.outf[o] = y;
                const float d = y - e1[j];
                const float ww = e2[j];
                lsum += ww * d * d;
                g.dz[o] = (__bf16)(2.0f * ww * d * g.inv);
            } else if constexpr (EPI == kEpiWeightGrad) {
                g.outf[o] = v;
            } else if constexpr (EPI == kEpiTanhBack) {
                const float y = e1[j];
                g.outb[o] = (__bf16)(v * (1.0f - y * y));
            }
        }
        if constexpr (EPI == kEpiWeightGrad)
            if (sums && r == 0 && m < g.M) g.rowsum[m] = accs[j];
    }
    if constexpr (EPI == kEpiBiasLoss) {
        __shared__ float red[4];
        lsum = wave_sum(lsum);
        if (lane == 0) red[wave] = lsum;
        __syncthreads();
        if (threadIdx.x == 0) g.partial[tn * g.tiles_m + tm] = ((red[0] + red[1]) + red[2]) + red[3];
    }
}

// Tiles [0, n1) of the grid compute g1, tiles [n1, n1 + n2) compute g2.
template <int E1, bool AV1, bool BV1, int E2, bool AV2, bool BV2>
__global__ __launch_bounds__(256) void gemm_kernel(Gemm g1, int n1, Gemm g2, Extra x) {
    const int id = blockIdx.x;
    if (id < n1) {
        gemm_tile<E1, AV1, BV1>(g1, id % g1.tiles_m, id / g1.tiles_m);
    } else if constexpr (E2 != kEpiNone) {
        const int id2 = id - n1;
        gemm_tile<E2, AV2, BV2>(g2, id2 % g2.tiles_m, id2 / g2.tiles_m);
    }
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        if (x.counter && threadIdx.x == 0) *x.counter += 1;
        if (x.fin_partial) {
            float s = 0.f;
            for (int i = threadIdx.x; i < x.fin_n; i += 64) s += x.fin_partial[i];
            s = wave_sum(s);
            if (threadIdx.x == 0) x.fin_loss[0] = s * x.fin_inv;
        }
    }
}

// ---- networks of few, small layers ----

// Barrier that orders LDS accesses only: __syncthreads also waits for every
// global load and store in flight, here the next layer's weights and the
// transposed results.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kFewLayers = 8;
constexpr int kFewWidth = 256;
constexpr int kRowWaves = 16;              // waves of rows_kernel, one 16-column tile each

// Offsets of layer l: off parameters (W then b), fwd / bwd the two BF16
// weight copies, xt its transposed input [w_l][Bp], dzt the transposed
// gradient of its pre-activations [w_{l+1}][Bp] (Bp = B rounded up to 32).
struct Net {
    int L;
    int w[kFewLayers + 1];
    int64_t off[kFewLayers], fwd[kFewLayers], bwd[kFewLayers], xt[kFewLayers], dzt[kFewLayers];
};

// The kernel's first argument, a Net, copied to LDS by the workgroup (at
// least 128 threads).
__device__ __forceinline__ void net_to_lds(Net& out) {
    constexpr int words = sizeof(Net) / 4;
    static_assert(sizeof(Net) % 4 == 0 && words <= 128, "one word per thread");
    const int* arg = (const int*)__builtin_amdgcn_kernarg_segment_ptr();
    if (threadIdx.x < words) reinterpret_cast<int*>(&out)[threadIdx.x] = arg[threadIdx.x];
}

// Place of W[n][k] in the copies: 1 KB blocks of the 64 lanes' eight values of
// one MFMA operand, (contraction step, output tile) in row-major order, so
// that the steps beyond a layer's last lie beyond its copy.
__host__ __device__ inline int64_t frag_place(int out, int con, int tiles) {
    return (((int64_t)(con >> 5) * tiles + (out >> 4)) * 64 + ((con >> 3) & 3) * 16 + (out & 15)) * 8 + (con & 7);
}
__host__ __device__ inline int64_t frag_size(int out, int con) {
    return (int64_t)((out + 15) / 16) * ((con + 31) / 32) * 512;
}
__device__ inline void put_weight(const Net& net, int l, int n, int k, float v, __bf16* __restrict__ wf) {
    const int N = net.w[l + 1], K = net.w[l];
    wf[net.fwd[l] + frag_place(n, k, (N + 15) / 16)] = (__bf16)v;
    wf[net.bwd[l] + frag_place(k, n, (K + 15) / 16)] = (__bf16)v;
}

// Work of a training step that one thread does for all: the step counter,
// and the learning rate and bias corrections of the step it now counts
// (out[0..2]).  The rate follows the cosine schedule lr0 (1 + cos(pi s /
// total)) / 2 + lr_floor with s = t - 1 - done0 the step within this run, and
// the bias corrections are 1 - beta^t, in double.
struct Schedule {
    int64_t* counter;  // NULL: none
    double lr0, lr_floor;
    int64_t total, done0;
    float b1, b2;
    float* out;
};
__device__ inline void schedule_step(const Schedule& s) {
    const int64_t t = *s.counter + 1;
    *s.counter = t;
    const double sfrac = (double)(t - 1 - s.done0) / (double)s.total;
    s.out[0] = (float)(s.lr0 * 0.5 * (1.0 + cos(3.14159265358979323846 * sfrac)) + s.lr_floor);
    s.out[1] = 1.0f - (float)pow((double)s.b1, (double)t);
    s.out[2] = 1.0f - (float)pow((double)s.b2, (double)t);
}

// Rows [RV MT b, RV MT (b + 1)) of the batch, b = blockIdx.x, through all
// layers.  An MFMA tile has 16 rows; with RV = 8 or 4 the rows repeat in it, and
// the lanes that hold the same row divide the epilogue among them: it costs
// more vector instructions (tanh) than the products do matrix ones, so a batch
// that leaves CUs idle is better spread over them so.  TRAIN: t, w, inv as in Gemm; xt and dzt receive what
// weights_kernel sums, partial[b] the block's share of the loss.  Else y
// receives the outputs.
// W: waves, of 16 columns each.  Four or eight serve networks of at most 64 or
// 128 units and leave room for several workgroups on a CU, where a batch beyond
// one round of workgroups would otherwise wait for sixteen waves of which few
// have a tile.  400,000 rows, sixteen waves and so: 3-10 110 and 27 us, 3-32-10
// 140 and 36, 128-128-128 363 and 209; one layer alone in half the rows again,
// 72-72 195 and 74.
template <bool TRAIN, int RV, int MT, int W = kRowWaves>
__global__ __launch_bounds__(64 * W) void rows_kernel(Net net, const __bf16* __restrict__ wf,
                                                              const float* __restrict__ par,
                                                              const float* __restrict__ x, int B,
                                                              float* __restrict__ y, const float* __restrict__ t,
                                                              const float* __restrict__ w, float inv, int Bp,
                                                              __bf16* __restrict__ tr, float* __restrict__ partial,
                                                              Schedule sched) {
    // activations and gradients of every layer when training, else the
    // activations of two
    constexpr int ROWS = RV * MT, J = RV / 4;  // J: values of a lane in a tile
    constexpr int kWide = 16 * W, kLdw = kWide + 8;  // columns, and the LDS row (padded: rows 4 banks apart)
    constexpr int kFragSteps = kWide / 32;
    static_assert(RV == 16 || MT == 1, "one tile of repeated rows");
    __shared__ __align__(16) __bf16 act[TRAIN ? kFewLayers : 2][ROWS][kLdw];
    __shared__ __align__(16) __bf16 grad[TRAIN ? kFewLayers : 1][TRAIN ? ROWS : 1][kLdw];
    __shared__ float red[W];
    __shared__ Net nets;
    __shared__ int4 desc[2 * kFewLayers + 1];
    __shared__ float biases[kFewLayers][kWide];
    const int lane = threadIdx.x & 63, r = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int b0 = blockIdx.x * ROWS;
    // this lane's J rows of a tile are row0 .. row0 + J - 1, held in
    // accumulator places j0 .. j0 + J - 1
    const int j0 = RV == 16 ? 0 : RV == 8 ? 2 * (grp >> 1) : grp;
    const int row0 = (4 * grp + j0) % RV;
    const auto value = [&](const floatx4& a, int j) {
        if constexpr (RV == 16) return a[j];
        if constexpr (RV == 8) return grp < 2 ? a[j] : a[j + 2];
        const float lo = grp & 1 ? a[1] : a[0], hi = grp & 1 ? a[3] : a[2];
        return grp < 2 ? lo : hi;
    };
    if (TRAIN && b0 >= Bp) {
        // one workgroup more than the batch takes: the schedule
        if (threadIdx.x == 0) schedule_step(sched);
        return;
    }

    // Phase p < L: layer p forward; phase L + i, when training: the gradient
    // through layer L - 1 - i.  A phase's operand is this wave's column tile of
    // a weight copy, loaded during the phase before: all eight steps, or two
    // where those are enough (a CU takes 64 bytes a cycle from its cache, which
    // is 0.85 us for a 256 x 256 layer whatever the number of rows; a load
    // or a step behind a branch of its own is waited for at the join, 7.1 for
    // 5.4 ms of 200 training steps, so the steps beyond a copy read as zero
    // and are multiplied).
    // The network's description, in LDS for indexing by phase:
    net_to_lds(nets);
    lds_barrier();
    const int L = __builtin_amdgcn_readfirstlane(nets.L), phases = TRAIN ? 2 * L - 1 : L;
    const int NO = __builtin_amdgcn_readfirstlane(nets.w[L]), rows = B - b0;
    if (threadIdx.x < 2 * kFewLayers + 1) {
        // phase -> bytes to its weight copy, bytes of it, columns, terms
        const int p = threadIdx.x, q = p < phases ? p : phases - 1, l = q < L ? q : 2 * L - 1 - q;
        const int N = nets.w[l + 1], K = nets.w[l], out = q < L ? N : K, con = q < L ? K : N;
        desc[p] = make_int4(2 * (int)(q < L ? nets.fwd[l] : nets.bwd[l]), p < phases ? 2 * (int)frag_size(out, con) : 0,
                            out, con);
    }
    // all biases
    for (int i = threadIdx.x; i < L * kWide; i += 64 * W) {
        const int l = i / kWide, n = i % kWide, N = nets.w[l + 1];
        if (n < N) biases[l][n] = par[nets.off[l] + (int64_t)N * nets.w[l] + n];
    }
    lds_barrier();
    struct Operand {
        bf16x8 fr[kFragSteps];
        int out, steps;
    };
    const auto load = [&](Operand& o, int p) {
        const int4 d = desc[p];
        const int out = __builtin_amdgcn_readfirstlane(d.z), tiles = (out + 15) / 16;
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(reinterpret_cast<const char*>(wf)) + __builtin_amdgcn_readfirstlane(d.x), (short)0,
            __builtin_amdgcn_readfirstlane(d.y), 0x00020000);
        o.out = out;
        o.steps = wave < tiles ? (__builtin_amdgcn_readfirstlane(d.w) + 31) / 32 : 0;
        const int at = wave * 1024 + lane * 16;
        const auto block = [&](int s) {
            o.fr[s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, at, s * tiles * 1024, 0));
        };
        if (kFragSteps > 2 && o.steps > 2) {
#pragma unroll
            for (int s = 0; s < kFragSteps; ++s) block(s);
        } else if (o.steps > 0) {
            block(0);
            block(1);
        }
    };
    Operand o;
    load(o, 0);
    const int k0 = __builtin_amdgcn_readfirstlane(nets.w[0]);
    // (the first product reads the columns of two steps, or all)
    const auto inputs = [&](auto columns) {
        constexpr int C = decltype(columns)::value;
#pragma unroll 4
        for (int i = threadIdx.x; i < ROWS * C; i += 64 * W) {
            const int m = i / C, k = i % C;
            const bool ok = b0 + m < B && k < k0;
            const float v = x[ok ? (int64_t)(b0 + m) * k0 + k : 0];
            act[0][m][k] = ok ? (__bf16)v : (__bf16)0.0f;
        }
    };
    if (k0 <= 64) inputs(std::integral_constant<int, 64>{});
    else inputs(std::integral_constant<int, kWide>{});
    // this lane's column, and the loss's targets and weights there
    const int n = wave * 16 + r;
    float tv[MT][J], wv[MT][J];
    if constexpr (TRAIN)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int row = 16 * m + row0 + j;
                const int64_t at = n < NO && row < rows ? (int64_t)(b0 + row) * NO + n : 0;
                tv[m][j] = t[at];
                wv[m][j] = 1.0f;
                if (w) wv[m][j] = w[at];
            }
    lds_barrier();
    float lsum = 0.f;
    for (int p = 0; p < phases; ++p) {
        const int l = p < L ? p : 2 * L - 1 - p;
        const int out = o.out;
        const __bf16(*in)[kLdw] = p < L ? act[TRAIN ? l : l & 1] : grad[TRAIN ? l : 0];
        floatx4 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
        const auto step = [&](int s) {
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(&in[16 * m + r % RV][32 * s + 8 * grp]);
                acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, o.fr[s], acc[m], 0, 0, 0);
            }
        };
        if (kFragSteps > 2 && o.steps > 2) {
#pragma unroll
            for (int s = 0; s < kFragSteps; ++s) step(s);
        } else if (o.steps > 0) {
            step(0);
            step(1);
        }
        load(o, p + 1);
        // (every wave writes its columns, zeros beyond the layer's)
        const bool nok = n < out;
        if (p + 1 < L) {
            const float bias = biases[l][n];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    float z = 0.f;
                    if (wave * 16 < out) z = tanhf(value(acc[m], j) + bias);
                    act[TRAIN ? l + 1 : (l + 1) & 1][16 * m + row0 + j][n] =
                        nok && 16 * m + row0 + j < rows ? (__bf16)z : (__bf16)0.0f;
                }
        } else if (p < L) {
            const float bias = biases[l][n];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int row = 16 * m + row0 + j;
                    const bool ok = nok && row < rows;
                    const float yy = value(acc[m], j) + bias;
                    if constexpr (TRAIN) {
                        const float d = yy - tv[m][j];
                        const float ww = wv[m][j];
                        lsum += ok ? ww * d * d : 0.f;
                        grad[l][row][n] = ok ? (__bf16)(2.0f * ww * d * inv) : (__bf16)0.0f;
                    } else if (ok) {
                        y[(int64_t)(b0 + row) * NO + n] = yy;
                    }
                }
        } else if constexpr (TRAIN) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int row = 16 * m + row0 + j;
                    const float yy = (float)act[l][row][n];
                    const float v = value(acc[m], j);
                    grad[l - 1][row][n] = nok && row < rows ? (__bf16)(v * (1.0f - yy * yy)) : (__bf16)0.0f;
                }
        }
        lds_barrier();
    }
    if constexpr (TRAIN) {
        // everything transposed: ROWS batch values of a column at a time
        typedef __bf16 bf16xr __attribute__((ext_vector_type(ROWS)));
        for (int l = 0; l < L; ++l)
            for (int i = threadIdx.x; i < nets.w[l] + nets.w[l + 1]; i += 64 * W) {
                const bool x_part = i < nets.w[l];
                const int c = x_part ? i : i - nets.w[l];
                bf16xr q;
#pragma unroll
                for (int row = 0; row < ROWS; ++row) q[row] = x_part ? act[l][row][c] : grad[l][row][c];
                *reinterpret_cast<bf16xr*>(tr + (x_part ? nets.xt[l] : nets.dzt[l]) + (int64_t)c * Bp + b0) = q;
            }
        lsum = wave_sum(lsum);
        if (lane == 0) red[wave] = lsum;
        lds_barrier();
        if (threadIdx.x == 0) {
            float s = 0.f;
            for (int i = 0; i < W; ++i) s += red[i];
            partial[blockIdx.x] = s;
        }
    }
}

// One Adam update (FP32): parameter p, moments m and v (updated), gradient gi;
// returns the new parameter.
__device__ __forceinline__ float adam_value(float p, float& m, float& v, float gi, float lr, float b1, float b2,
                                            float eps, float c1, float c2) {
    const float mi = b1 * m + (1.0f - b1) * gi;
    const float vi = b2 * v + (1.0f - b2) * gi * gi;
    m = mi;
    v = vi;
    return p - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// The update of parameter i in memory.
__device__ __forceinline__ float adam_update(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                                             int64_t i, float gi, float lr, float b1, float b2, float eps, float c1,
                                             float c2) {
    float mi = m[i], vi = v[i];
    const float pi = adam_value(p[i], mi, vi, gi, lr, b1, b2, eps, c1, c2);
    m[i] = mi;
    v[i] = vi;
    p[i] = pi;
    return pi;
}

// Weight and bias gradients of every layer, dW = dz^T X and db = row sums of
// dz^T over the batch (B rounded up to 32), one 32 x 32 tile per workgroup;
// with `rate` (learning rate and bias corrections of this step) Adam follows
// at once.  Workgroup 0 also adds up the loss.
__global__ __launch_bounds__(256) void weights_kernel(Net net, const __bf16* __restrict__ tr, int Bp,
                                                      float* __restrict__ g, float* __restrict__ p,
                                                      float* __restrict__ m1, float* __restrict__ v1,
                                                      __bf16* __restrict__ wf, const float* __restrict__ rate,
                                                      float b1, float b2, float eps, Extra x) {
    constexpr int kSteps = 16;
    __shared__ Net nets;
    net_to_lds(nets);
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, grp = lane >> 4;
    int l = 0, id = blockIdx.x, tm = (nets.w[1] + 31) / 32;
    for (; l + 1 < nets.L; ++l, tm = (nets.w[l + 1] + 31) / 32) {
        const int n = tm * ((nets.w[l] + 31) / 32);
        if (id < n) break;
        id -= n;
    }
    l = __builtin_amdgcn_readfirstlane(l);
    id = __builtin_amdgcn_readfirstlane(id);
    tm = __builtin_amdgcn_readfirstlane(tm);
    const int M = __builtin_amdgcn_readfirstlane(nets.w[l + 1]), N = __builtin_amdgcn_readfirstlane(nets.w[l]);
    const int64_t off = nets.off[l];
    const int m0 = (id % tm) * 32 + (wave & 1) * 16, n0 = (id / tm) * 32 + (wave >> 1) * 16;
    // rows m0 + r of dz^T and n0 + r of X^T, eight batch values of group grp
    const bool aok = m0 + r < M, bok = n0 + r < N;
    const __bf16* __restrict__ A = tr + nets.dzt[l] + (int64_t)(aok ? m0 + r : 0) * Bp + 8 * grp;
    const __bf16* __restrict__ X = tr + nets.xt[l] + (int64_t)(bok ? n0 + r : 0) * Bp + 8 * grp;
    const bool sums = n0 == 0;
    bf16x8 ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.0f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f}, accs = {0.f, 0.f, 0.f, 0.f};
    const auto masked = [](uint4 v, bool ok) {
        v.x = ok ? v.x : 0u;
        v.y = ok ? v.y : 0u;
        v.z = ok ? v.z : 0u;
        v.w = ok ? v.w : 0u;
        return __builtin_bit_cast(bf16x8, v);
    };
    const int steps = Bp / 32;
    uint4 ra[kSteps], rb[kSteps];
    const auto load = [&](int s0) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const int s = s0 + u < steps ? s0 + u : steps - 1;  // (past the end: loaded, not used)
            ra[u] = *reinterpret_cast<const uint4*>(A + 32 * s);
            rb[u] = *reinterpret_cast<const uint4*>(X + 32 * s);
        }
    };
    load(0);
    // Adam's operands, on their way during the products
    const int n = n0 + r;
    float pv[4], mv[4], vv[4], lr = 0.f, c1 = 1.f, c2 = 1.f;
    if (rate) {
        lr = rate[0];
        c1 = rate[1];
        c2 = rate[2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = m0 + 4 * grp + j;
            const int64_t i = m < M && n < N ? off + (int64_t)m * N + n : 0;
            pv[j] = p[i];
            mv[j] = m1[i];
            vv[j] = v1[i];
        }
    }
    for (int s0 = 0; s0 < steps; s0 += kSteps) {
        bf16x8 a[kSteps], b[kSteps];
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            a[u] = masked(ra[u], aok);
            b[u] = masked(rb[u], bok);
        }
        if (s0 + kSteps < steps) load(s0 + kSteps);
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            if (s0 + u < steps) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[u], acc, 0, 0, 0);
                if (sums) accs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], ones, accs, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = m0 + 4 * grp + j;
        if (m < M && n < N) {
            const int64_t i = off + (int64_t)m * N + n;
            g[i] = acc[j];
            if (rate) {
                const float pi = adam_value(pv[j], mv[j], vv[j], acc[j], lr, b1, b2, eps, c1, c2);
                p[i] = pi;
                m1[i] = mv[j];
                v1[i] = vv[j];
                put_weight(nets, l, m, n, pi, wf);
            }
        }
        if (m < M && sums && r == 0) {
            const int64_t i = off + (int64_t)M * N + m;
            g[i] = accs[j];
            if (rate) adam_update(p, m1, v1, i, accs[j], lr, b1, b2, eps, c1, c2);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < 64 && x.fin_partial) {
        float s = 0.f;
        for (int i = threadIdx.x; i < x.fin_n; i += 64) s += x.fin_partial[i];
        s = wave_sum(s);
        if (threadIdx.x == 0) x.fin_loss[0] = s * x.fin_inv;
    }
}

// The weight copies from the FP32 parameters (n of them); with grad, after an
// Adam update of each.
__global__ void copies_kernel(Net net, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                              float* __restrict__ v, __bf16* __restrict__ wf, int64_t n, float lr, float b1, float b2,
                              float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float pi = g ? adam_update(p, m, v, i, g[i], lr, b1, b2, eps, c1, c2) : p[i];
    int l = 0;
    while (l + 1 < net.L && i >= net.off[l + 1]) ++l;
    const int64_t q = i - net.off[l];
    const int K = net.w[l];
    if (q < (int64_t)net.w[l + 1] * K) put_weight(net, l, (int)(q / K), (int)(q % K), pi, wf);
}

__global__ void to_bf16_kernel(const float* __restrict__ in, __bf16* __restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (__bf16)in[i];
}

// Adam on the FP32 master parameters, bias corrections passed in; refreshes
// the BF16 copy used by the products.
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, __bf16* __restrict__ pb, int64_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    pb[i] = (__bf16)adam_update(p, m, v, i, g[i], lr, b1, b2, eps, c1, c2);
}

// The same update inside a replayed training step: the step index t (from 1)
// is read from the device counter, the learning rate follows the cosine
// schedule lr0 (1 + cos(pi s / total)) / 2 + lr_floor with s = t - 1 - done0
// the step within this run, and the bias corrections are 1 - beta^t.
__global__ void adam_sched_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                  float* __restrict__ v, __bf16* __restrict__ pb, int64_t n, double lr0,
                                  double lr_floor, int64_t total, int64_t done0, float b1, float b2, float eps,
                                  const int64_t* __restrict__ counter) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t t = *counter;
    const double sfrac = (double)(t - 1 - done0) / (double)total;
    const float lr = (float)(lr0 * 0.5 * (1.0 + cos(3.14159265358979323846 * sfrac)) + lr_floor);
    const float c1 = 1.0f - (float)pow((double)b1, (double)t);
    const float c2 = 1.0f - (float)pow((double)b2, (double)t);
    pb[i] = (__bf16)adam_update(p, m, v, i, g[i], lr, b1, b2, eps, c1, c2);
}

__global__ void count_set_kernel(int64_t* c, int64_t value) {
    if (threadIdx.x == 0) *c = value;
}

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// Operand (row, k) at P[row s_row + k s_k] can take 16-byte loads.
inline bool vec_ok(const __bf16* P, int64_t s_row, int64_t s_k, int K) {
    return s_k == 1 && K % 8 == 0 && s_row % 8 == 0 && aligned16(P);
}

Gemm make_gemm(const __bf16* A, int64_t sam, int64_t sak, const __bf16* B, int64_t sbk, int64_t sbn, int M, int N,
               int K, int64_t ldo) {
    Gemm g{};
    g.A = A;
    g.sam = sam;
    g.sak = sak;
    g.B = B;
    g.sbk = sbk;
    g.sbn = sbn;
    g.M = M;
    g.N = N;
    g.K = K;
    g.ldo = ldo;
    g.tiles_m = (M + 31) / 32;
    return g;
}

inline int tiles(const Gemm& g) { return g.tiles_m * ((g.N + 31) / 32); }

template <int E1, bool AV1, bool BV1, int E2, bool AV2, bool BV2>
hipError_t launch(const Gemm& g1, const Gemm* g2, const Extra& x, hipStream_t st) {
    const int n1 = tiles(g1), n2 = g2 ? tiles(*g2) : 0;
    hipLaunchKernelGGL((gemm_kernel<E1, AV1, BV1, E2, AV2, BV2>), dim3(n1 + n2), dim3(256), 0, st, g1, n1,
                       g2 ? *g2 : g1, x);
    return hipGetLastError();
}

// One product with epilogue EPI; the two load paths picked from the operands.
template <int EPI>
hipError_t gemm1(const Gemm& g, const Extra& x, hipStream_t st) {
    const bool av = vec_ok(g.A, g.sam, g.sak, g.K), bv = vec_ok(g.B, g.sbn, g.sbk, g.K);
    if (av && bv) return launch<EPI, true, true, kEpiNone, false, false>(g, nullptr, x, st);
    if (av) return launch<EPI, true, false, kEpiNone, false, false>(g, nullptr, x, st);
    if (bv) return launch<EPI, false, true, kEpiNone, false, false>(g, nullptr, x, st);
    return launch<EPI, false, false, kEpiNone, false, false>(g, nullptr, x, st);
}

}  // namespace

struct lbw_mlp {
    std::vector<int> w;     // widths, n_layers + 1
    int L = 0;              // layers
    int max_batch = 0;
    hipStream_t stream = nullptr;
    std::vector<int64_t> off;  // parameter offset of layer l (W then b)
    int64_t P = 0;
    float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;  // FP32 master, grad, Adam moments
    __bf16* wb = nullptr;        // BF16 copy of the weights (same offsets, biases unused)
    __bf16* act = nullptr;       // BF16 input and hidden activations, layer l at act_off[l]
    std::vector<int64_t> act_off;
    float* yout = nullptr;       // FP32 output of the last training forward
    __bf16* dz[2] = {nullptr, nullptr};  // BF16 gradients w.r.t. pre-activations (alternating layers)
    float* partial = nullptr;    // per-tile loss sums of the output product
    int n_partial = 0;
    float* loss_dev = nullptr;
    int64_t* d_steps = nullptr;  // Adam steps taken, on the device (scheduled training)
    // networks of few, small layers: the weight copies, the transposed
    // activations and gradients of a training step (offsets for batch Bp),
    // and the rate and bias corrections of the step
    bool few = false;
    int cus = 256, widest = 0;
    Net net{};
    __bf16* wf = nullptr;
    int64_t wf_size = 0;
    __bf16* tr = nullptr;
    float* rate = nullptr;
    int64_t steps = 0;
    bool have_grad = false;
};

namespace {

hipError_t refresh_bf16(lbw_mlp* M) {
    if (M->few) {
        hipLaunchKernelGGL(copies_kernel, dim3(nblk(M->P)), dim3(256), 0, M->stream, M->net, M->p, nullptr, nullptr,
                           nullptr, M->wf, M->P, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(to_bf16_kernel, dim3(nblk(M->P)), dim3(256), 0, M->stream, M->p, M->wb, M->P);
    return hipGetLastError();
}

hipError_t cast_input(lbw_mlp* M, const float* x, int B, hipStream_t st) {
    hipLaunchKernelGGL(to_bf16_kernel, dim3(nblk((int64_t)B * M->w[0])), dim3(256), 0, st, x,
                       M->act + M->act_off[0], (int64_t)B * M->w[0]);
    return hipGetLastError();
}

// Layers 0 .. L-1 on the cast input.  The output layer writes y_out (FP32,
// [B][w_L]) when t is NULL, else the loss gradient and per-tile loss sums.
hipError_t forward_layers(lbw_mlp* M, int B, float* y_out, const float* t, const float* w, float inv,
                          int64_t* counter, hipStream_t st) {
    hipError_t e = hipSuccess;
    for (int l = 0; l < M->L && e == hipSuccess; ++l) {
        const int K = M->w[l], N = M->w[l + 1];
        Gemm g = make_gemm(M->act + M->act_off[l], K, 1, M->wb + M->off[l], 1, K, B, N, K, N);
        g.bias = M->p + M->off[l] + (int64_t)N * K;
        Extra x{};
        x.counter = l == 0 ? counter : nullptr;
        if (l + 1 < M->L) {
            g.outb = M->act + M->act_off[l + 1];
            e = gemm1<kEpiBiasTanh>(g, x, st);
        } else if (!t) {
            g.outf = y_out;
            e = gemm1<kEpiBias>(g, x, st);
        } else {
            g.outf = M->yout;
            g.t = t;
            g.w = w;
            g.inv = inv;
            g.dz = M->dz[0];
            g.partial = M->partial;
            M->n_partial = tiles(g);
            e = gemm1<kEpiBiasLoss>(g, x, st);
        }
    }
    return e;
}

// Gradients after a training forward: per layer (last first) one launch with
// dW = dz^T X and the bias gradient (row sums of dz^T), and, below the
// output layer, the next dz = (dz W) (1 - X^2) from the stored activation X.
// The first launch also reduces the loss.
hipError_t backward(lbw_mlp* M, int B, float inv, hipStream_t st) {
    hipError_t e = hipSuccess;
    int cur = 0;
    for (int l = M->L - 1; l >= 0 && e == hipSuccess; --l, cur ^= 1) {
        const int K = M->w[l], N = M->w[l + 1];
        const __bf16* X = M->act + M->act_off[l];
        const __bf16* dz = M->dz[cur];
        Gemm gw = make_gemm(dz, 1, N, X, K, 1, N, K, B, K);
        gw.outf = M->g + M->off[l];
        gw.rowsum = gw.outf + (int64_t)N * K;
        Extra x{};
        if (l == M->L - 1) {
            x.fin_partial = M->partial;
            x.fin_n = M->n_partial;
            x.fin_inv = inv;
            x.fin_loss = M->loss_dev;
        }
        if (l == 0) {
            e = launch<kEpiWeightGrad, false, false, kEpiNone, false, false>(gw, nullptr, x, st);
        } else {
            Gemm gy = make_gemm(dz, N, 1, M->wb + M->off[l], K, 1, B, K, N, K);
            gy.act = X;
            gy.outb = M->dz[cur ^ 1];
            if (vec_ok(gy.A, gy.sam, gy.sak, gy.K))
                e = launch<kEpiWeightGrad, false, false, kEpiTanhBack, true, false>(gw, &gy, x, st);
            else
                e = launch<kEpiWeightGrad, false, false, kEpiTanhBack, false, false>(gw, &gy, x, st);
        }
    }
    return e;
}

int rows32(int B) { return (B + 31) / 32 * 32; }

// Offsets of the transposed arrays for a batch of B rows.
Net net_for(const lbw_mlp* M, int B) {
    Net net = M->net;
    const int64_t Bp = rows32(B);
    int64_t at = 0;
    for (int l = 0; l < net.L; ++l) {
        net.xt[l] = at;
        at += net.w[l] * Bp;
        net.dzt[l] = at;
        at += net.w[l + 1] * Bp;
    }
    return net;
}

// Outputs y of B rows of x, one launch: as many rows per workgroup, 4 to 64,
// as give each CU one workgroup (each reads all the weights, and a second
// round of workgroups costs as much as the first).  Beyond that, workgroups of as
// few waves as the widest layer needs, of 64 rows, or 32 where a single layer of
// up to 128 units leaves mostly memory to wait for (8-128, 400,000 rows: 55 us
// against 67).
template <int RV, int MT, int W = kRowWaves>
void launch_rows(lbw_mlp* M, const float* x, int B, float* y) {
    hipLaunchKernelGGL((rows_kernel<false, RV, MT, W>), dim3((B + RV * MT - 1) / (RV * MT)), dim3(64 * W), 0,
                       M->stream, M->net, M->wf, M->p, x, B, y, nullptr, nullptr, 0.f, 0, nullptr, nullptr,
                       Schedule{});
}
hipError_t few_forward(lbw_mlp* M, const float* x, int B, float* y) {
    const int cus = M->cus;
    if (B <= 4 * cus) launch_rows<4, 1>(M, x, B, y);
    else if (B <= 8 * cus) launch_rows<8, 1>(M, x, B, y);
    else if (B <= 16 * cus) launch_rows<16, 1>(M, x, B, y);
    else if (B <= 32 * cus) launch_rows<16, 2>(M, x, B, y);
    else if (B <= 48 * cus) launch_rows<16, 3>(M, x, B, y);
    else if (M->widest <= 64) launch_rows<16, 4, 4>(M, x, B, y);
    else if (M->widest <= 128 && M->L == 1) launch_rows<16, 2, 8>(M, x, B, y);
    else if (M->widest <= 128) launch_rows<16, 4, 8>(M, x, B, y);
    else launch_rows<16, 4>(M, x, B, y);
    return hipGetLastError();
}

// Loss and gradients, and with a schedule the Adam step: two launches.
hipError_t few_train(lbw_mlp* M, const Net& net, const float* x, const float* t, const float* w, int B, float inv,
                     const Schedule& sched, float eps) {
    const int Bp = rows32(B);
    int rows = 16;  // per workgroup, as few_forward
    const auto launch = [&](auto rv) {
        constexpr int RV = decltype(rv)::value;
        rows = RV;
        hipLaunchKernelGGL((rows_kernel<true, RV, 1>), dim3(Bp / RV + (sched.counter ? 1 : 0)), dim3(64 * kRowWaves),
                           0, M->stream, net, M->wf, M->p, x, B, nullptr, t, w, inv, Bp, M->tr, M->partial, sched);
    };
    if (Bp <= 4 * M->cus) launch(std::integral_constant<int, 4>{});
    else if (Bp <= 8 * M->cus) launch(std::integral_constant<int, 8>{});
    else launch(std::integral_constant<int, 16>{});
    int tiles = 0;
    for (int l = 0; l < net.L; ++l) tiles += ((net.w[l + 1] + 31) / 32) * ((net.w[l] + 31) / 32);
    Extra fin{};
    fin.fin_partial = M->partial;
    fin.fin_n = Bp / rows;
    fin.fin_inv = inv;
    fin.fin_loss = M->loss_dev;
    hipLaunchKernelGGL(weights_kernel, dim3(tiles), dim3(256), 0, M->stream, net, M->tr, Bp, M->g, M->p, M->m, M->v,
                       M->wf, sched.counter ? M->rate : nullptr, sched.b1, sched.b2, eps, fin);
    return hipGetLastError();
}

}  // namespace

extern "C" {

int lbw_mlp_create(const int32_t* widths, int n_layers, int max_batch, void* stream, lbw_mlp_t* out) {
    if (!out) return fail(LBW_EINVAL, "out is NULL");
    *out = nullptr;
    if (!widths || n_layers < 1 || n_layers > 16 || max_batch < 1) return fail(LBW_EINVAL, "invalid MLP shape");
    for (int l = 0; l <= n_layers; ++l)
        if (widths[l] < 1 || widths[l] > 4096) return fail(LBW_EINVAL, "layer width outside [1, 4096]");
    lbw_mlp* M = new lbw_mlp();
    M->w.assign(widths, widths + n_layers + 1);
    M->L = n_layers;
    M->max_batch = max_batch;
    M->stream = (hipStream_t)stream;
    int64_t P = 0, A = 0, maxw = 0;
    for (int l = 0; l < n_layers; ++l) {
        M->off.push_back(P);
        P += (int64_t)M->w[l] * M->w[l + 1] + M->w[l + 1];
    }
    for (int l = 0; l <= n_layers; ++l) {
        M->act_off.push_back(A);
        A += ((int64_t)max_batch * M->w[l] + 7) / 8 * 8;  // 16-byte aligned layers
        if (M->w[l] > maxw) maxw = M->w[l];
    }
    M->P = P;
    M->widest = (int)maxw;
    const int64_t bw = (int64_t)max_batch * maxw;
    // (the last bound: offsets of rows x width elements stay within 32 bits)
    M->few = n_layers <= kFewLayers && maxw <= kFewWidth && max_batch <= (1 << 22);
    int64_t T = 0;
    if (M->few) {
        if (lbw::device_cus(&M->cus) != LBW_OK) M->cus = 256;
        M->net.L = n_layers;
        for (int l = 0; l <= n_layers; ++l) M->net.w[l] = M->w[l];
        for (int l = 0; l < n_layers; ++l) {
            M->net.off[l] = M->off[l];
            M->net.fwd[l] = M->wf_size;
            M->wf_size += frag_size(M->w[l + 1], M->w[l]);
            M->net.bwd[l] = M->wf_size;
            M->wf_size += frag_size(M->w[l], M->w[l + 1]);
            T += (int64_t)(M->w[l] + M->w[l + 1]) * rows32(max_batch);
        }
    }
    hipError_t e = hipMalloc(&M->p, sizeof(float) * P);
    if (e == hipSuccess) e = hipMalloc(&M->g, sizeof(float) * P);
    if (e == hipSuccess) e = hipMalloc(&M->m, sizeof(float) * P);
    if (e == hipSuccess) e = hipMalloc(&M->v, sizeof(float) * P);
    if (M->few) {
        if (e == hipSuccess) e = hipMalloc(&M->wf, sizeof(__bf16) * M->wf_size);
        if (e == hipSuccess) e = hipMemsetAsync(M->wf, 0, sizeof(__bf16) * M->wf_size, M->stream);
        if (e == hipSuccess) e = hipMalloc(&M->tr, sizeof(__bf16) * T);
        if (e == hipSuccess) e = hipMalloc(&M->rate, sizeof(float) * 3);
        // one loss sum per 4 rows or more
        if (e == hipSuccess) e = hipMalloc(&M->partial, sizeof(float) * (rows32(max_batch) / 4));
    } else {
        if (e == hipSuccess) e = hipMalloc(&M->wb, sizeof(__bf16) * P);
        if (e == hipSuccess) e = hipMalloc(&M->act, sizeof(__bf16) * A);
        if (e == hipSuccess) e = hipMalloc(&M->yout, sizeof(float) * (int64_t)max_batch * M->w[n_layers]);
        if (e == hipSuccess) e = hipMalloc(&M->dz[0], sizeof(__bf16) * bw);
        if (e == hipSuccess) e = hipMalloc(&M->dz[1], sizeof(__bf16) * bw);
        // one loss sum per 32 x 32 output tile
        if (e == hipSuccess)
            e = hipMalloc(&M->partial,
                          sizeof(float) * (((int64_t)max_batch + 31) / 32) * ((M->w[n_layers] + 31) / 32));
    }
    if (e == hipSuccess) e = hipMalloc(&M->loss_dev, sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&M->d_steps, sizeof(int64_t));
    if (e == hipSuccess) e = hipMemsetAsync(M->p, 0, sizeof(float) * P, M->stream);
    if (e == hipSuccess) e = hipMemsetAsync(M->m, 0, sizeof(float) * P, M->stream);
    if (e == hipSuccess) e = hipMemsetAsync(M->v, 0, sizeof(float) * P, M->stream);
    if (e == hipSuccess) e = refresh_bf16(M);
    if (e != hipSuccess) {
        lbw_mlp_free(M);
        return hip_fail(e, "lbw_mlp_create");
    }
    *out = M;
    return LBW_OK;
}

int lbw_mlp_param_count(lbw_mlp_t M, int64_t* count) {
    if (!M || !count) return fail(LBW_EINVAL, "NULL argument");
    *count = M->P;
    return LBW_OK;
}

int lbw_mlp_set_params(lbw_mlp_t M, const float* host) {
    if (!M || !host) return fail(LBW_EINVAL, "NULL argument");
    HIP_TRY(hipMemcpyAsync(M->p, host, sizeof(float) * M->P, hipMemcpyHostToDevice, M->stream), "lbw_mlp_set_params");
    HIP_TRY(hipMemsetAsync(M->m, 0, sizeof(float) * M->P, M->stream), "lbw_mlp_set_params");
    HIP_TRY(hipMemsetAsync(M->v, 0, sizeof(float) * M->P, M->stream), "lbw_mlp_set_params");
    HIP_TRY(refresh_bf16(M), "lbw_mlp_set_params");
    HIP_TRY(hipStreamSynchronize(M->stream), "lbw_mlp_set_params");
    M->steps = 0;
    M->have_grad = false;
    return LBW_OK;
}

int lbw_mlp_get_params(lbw_mlp_t M, float* host) {
    if (!M || !host) return fail(LBW_EINVAL, "NULL argument");
    HIP_TRY(hipMemcpyAsync(host, M->p, sizeof(float) * M->P, hipMemcpyDeviceToHost, M->stream), "lbw_mlp_get_params");
    HIP_TRY(hipStreamSynchronize(M->stream), "lbw_mlp_get_params");
    return LBW_OK;
}

int lbw_mlp_forward(lbw_mlp_t M, const float* x, int B, float* y) {
    if (!M || !x || !y) return fail(LBW_EINVAL, "NULL argument");
    if (B < 1 || B > M->max_batch) return fail(LBW_EINVAL, "batch %d outside [1, %d]", B, M->max_batch);
    if (M->few) {
        // the rows of x are read while other rows of y are written: where the
        // two overlap, the narrower goes through the workspace of a training
        // step (two bytes for each input and output, and more)
        const size_t nx = sizeof(float) * (size_t)B * M->w[0], ny = sizeof(float) * (size_t)B * M->w[M->L];
        const uintptr_t x0 = (uintptr_t)x, y0 = (uintptr_t)y;
        const bool overlap = x0 < y0 + ny && y0 < x0 + nx;
        float* const work = reinterpret_cast<float*>(M->tr);
        if (overlap && nx <= ny) {
            HIP_TRY(hipMemcpyAsync(work, x, nx, hipMemcpyDeviceToDevice, M->stream), "lbw_mlp_forward");
            x = work;
        }
        HIP_TRY(few_forward(M, x, B, overlap && x != work ? work : y), "lbw_mlp_forward");
        if (overlap && x != work)
            HIP_TRY(hipMemcpyAsync(y, work, ny, hipMemcpyDeviceToDevice, M->stream), "lbw_mlp_forward");
        return LBW_OK;
    }
    HIP_TRY(cast_input(M, x, B, M->stream), "lbw_mlp_forward");
    HIP_TRY(forward_layers(M, B, y, nullptr, nullptr, 0.f, nullptr, M->stream), "lbw_mlp_forward");
    return LBW_OK;
}

int lbw_mlp_loss_grad(lbw_mlp_t M, const float* x, const float* t, const float* w, int B, float weight_sum,
                      float* loss, float* grad) {
    if (!M || !x || !t) return fail(LBW_EINVAL, "NULL argument");
    if (B < 1 || B > M->max_batch) return fail(LBW_EINVAL, "batch %d outside [1, %d]", B, M->max_batch);
    if (!(weight_sum > 0.0f)) return fail(LBW_EINVAL, "weight_sum must be > 0");
    const float inv = 1.0f / weight_sum;
    if (M->few) {
        HIP_TRY(few_train(M, net_for(M, B), x, t, w, B, inv, Schedule{}, 0.f), "lbw_mlp_loss_grad");
    } else {
        HIP_TRY(cast_input(M, x, B, M->stream), "lbw_mlp_loss_grad");
        HIP_TRY(forward_layers(M, B, nullptr, t, w, inv, nullptr, M->stream), "lbw_mlp_loss_grad");
        HIP_TRY(backward(M, B, inv, M->stream), "lbw_mlp_loss_grad");
    }
    if (loss) HIP_TRY(hipMemcpyAsync(loss, M->loss_dev, sizeof(float), hipMemcpyDeviceToDevice, M->stream), "loss");
    if (grad) HIP_TRY(hipMemcpyAsync(grad, M->g, sizeof(float) * M->P, hipMemcpyDeviceToDevice, M->stream), "grad");
    M->have_grad = true;
    return LBW_OK;
}

int lbw_mlp_adam_step(lbw_mlp_t M, float lr, float beta1, float beta2, float eps) {
    if (!M) return fail(LBW_EINVAL, "NULL argument");
    if (!M->have_grad) return fail(LBW_ESTATE, "no gradient: call lbw_mlp_loss_grad first");
    if (!(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return fail(LBW_EINVAL, "invalid Adam hyper-parameters");
    M->steps += 1;
    const float c1 = 1.0f - (float)std::pow((double)beta1, (double)M->steps);
    const float c2 = 1.0f - (float)std::pow((double)beta2, (double)M->steps);
    if (M->few)
        hipLaunchKernelGGL(copies_kernel, dim3(nblk(M->P)), dim3(256), 0, M->stream, M->net, M->p, M->g, M->m, M->v,
                           M->wf, M->P, lr, beta1, beta2, eps, c1, c2);
    else
        hipLaunchKernelGGL(adam_kernel, dim3(nblk(M->P)), dim3(256), 0, M->stream, M->p, M->g, M->m, M->v, M->wb,
                           M->P, lr, beta1, beta2, eps, c1, c2);
    HIP_TRY(hipGetLastError(), "lbw_mlp_adam_step");
    return LBW_OK;
}

int lbw_mlp_train(lbw_mlp_t M, const float* x, const float* t, const float* w, int B, float weight_sum, int steps,
                  double lr, double lr_floor, float beta1, float beta2, float eps, float* loss) {
    if (!M || !x || !t) return fail(LBW_EINVAL, "NULL argument");
    if (B < 1 || B > M->max_batch) return fail(LBW_EINVAL, "batch %d outside [1, %d]", B, M->max_batch);
    if (!(weight_sum > 0.0f)) return fail(LBW_EINVAL, "weight_sum must be > 0");
    if (steps < 1) return fail(LBW_EINVAL, "steps must be >= 1");
    if (!(lr > 0.0) || !(lr_floor >= 0.0) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) ||
        !(eps > 0.f))
        return fail(LBW_EINVAL, "invalid Adam hyper-parameters");
    // the input is cast once and the device counter starts at the network's
    // step count; one training step (forward with the counter increment and
    // the loss, backward, Adam with the BF16 refresh) is captured on a
    // private stream and replayed on the network's stream
    const float inv = 1.0f / weight_sum;
    if (!M->few) HIP_TRY(cast_input(M, x, B, M->stream), "lbw_mlp_train");
    hipLaunchKernelGGL(count_set_kernel, dim3(1), dim3(64), 0, M->stream, M->d_steps, M->steps);
    HIP_TRY(hipGetLastError(), "lbw_mlp_train");
    if (M->few) {
        // two launches per step, queued directly: they take longer to run
        // than to queue
        const Schedule sched{M->d_steps, lr, lr_floor, (int64_t)steps, M->steps, beta1, beta2, M->rate};
        const Net net = net_for(M, B);
        hipError_t e = hipSuccess;
        for (int i = 0; i < steps && e == hipSuccess; ++i) e = few_train(M, net, x, t, w, B, inv, sched, eps);
        if (e == hipSuccess && loss)
            e = hipMemcpyAsync(loss, M->loss_dev, sizeof(float), hipMemcpyDeviceToDevice, M->stream);
        const hipError_t es = hipStreamSynchronize(M->stream);
        if (e == hipSuccess) e = es;
        if (e != hipSuccess) return hip_fail(e, "lbw_mlp_train");
        M->steps += steps;
        M->have_grad = true;
        return LBW_OK;
    }
    hipStream_t cap = nullptr;
    HIP_TRY(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking), "lbw_mlp_train");
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        hipError_t le = forward_layers(M, B, nullptr, t, w, inv, M->d_steps, cap);
        if (le == hipSuccess) le = backward(M, B, inv, cap);
        if (le == hipSuccess) {
            hipLaunchKernelGGL(adam_sched_kernel, dim3(nblk(M->P)), dim3(256), 0, cap, M->p, M->g, M->m, M->v, M->wb,
                               M->P, lr, lr_floor, (int64_t)steps, M->steps, beta1, beta2, eps, M->d_steps);
            le = hipGetLastError();
        }
        e = hipStreamEndCapture(cap, &graph);
        if (e == hipSuccess) e = le;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    for (int i = 0; i < steps && e == hipSuccess; ++i) e = hipGraphLaunch(exec, M->stream);
    if (e == hipSuccess && loss) e = hipMemcpyAsync(loss, M->loss_dev, sizeof(float), hipMemcpyDeviceToDevice, M->stream);
    const hipError_t es = hipStreamSynchronize(M->stream);  // before the graph is destroyed
    if (e == hipSuccess) e = es;
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamDestroy(cap);
    if (e != hipSuccess) return hip_fail(e, "lbw_mlp_train");
    M->steps += steps;
    M->have_grad = true;
    return LBW_OK;
}

int lbw_mlp_free(lbw_mlp_t M) {
    if (!M) return LBW_OK;
    (void)hipStreamSynchronize(M->stream);
    for (void* ptr : {(void*)M->p, (void*)M->g, (void*)M->m, (void*)M->v, (void*)M->wb, (void*)M->act,
                      (void*)M->yout, (void*)M->dz[0], (void*)M->dz[1], (void*)M->partial, (void*)M->loss_dev,
                      (void*)M->d_steps, (void*)M->wf, (void*)M->tr, (void*)M->rate})
        (void)hipFree(ptr);
    delete M;
    return LBW_OK;
}

}  // extern "C"
