// Resonant frequencies from probe traces, FP64 on the device.
//
// The paper locates resonances by driven frequency sweeps (Sec. IV.A and
// IV.C); for a freely ringing field the same peaks appear in the power
// spectrum of the probe signal.  Rule: per probe subtract the mean, apply
// the symmetric Hann window 1/2 - 1/2 cos(2 pi t / (T - 1)), zero-pad to
// nfft = 4 * nextpow2(T), FFT,
// P_k = sum over a group's probes of |X_k|^2 for k in [0, nfft/2]; peaks are
// bins b in [16, nfft/2 - 1] with P[b-1] < P[b] >= P[b+1] and
// P[b] > 1e-3 max P[16:], refined by a parabola through ln P (no refinement
// when a neighbour is 0).  Bin 16 is the first bin outside the Hann window's
// DC main lobe (half-width 2/T cycles per step = at most 16 bins), where the
// leakage of a slow baseline drift would otherwise show up as a peak.
//
// A "group" is the set of probes of one geometry: consecutive columns of a
// trace whose rows hold `stride` values.  Groups are processed in chunks so
// that the work space stays bounded.
//
// The work is moving FP64 data, so the passes over memory are what counts.
//  - Two real columns a, b make one complex one, z = a + i b: the sum of
//    their powers is (|Z_k|^2 + |Z_{n-k}|^2) / 2, so nothing has to be
//    separated, and a single last column is z = a by the same formula.
//  - n = n1 n2 (j = j1 n2 + j2, k = k1 + n1 k2): `cols_kernel` does the n1
//    point transforms over j1 in LDS straight from the (transposed) trace,
//    whose rows beyond T are not there to be read: they are the upper three
//    quarters of every transform, so its first radix-4 pass is a copy.
//    `rows_kernel` does the n2 point transforms over j2 and adds |Z|^2 of a
//    group's pairs in registers.  One complex array is written and read
//    once, where radix-2 passes over memory wrote and read it log2 n times.
//  - Chunks of whole groups keep that array below 96 MiB (kCacheBytes), so
//    it is read back from the 256 MiB Infinity Cache.
// Spectra of 64 groups of 8 probes over 30,000 rows (nfft 131,072, 123 MB of
// traces): 6.9 ms with radix-2 passes over memory (177 us each), 0.63 ms so:
// rows_kernel 253 us (537 MB read), cols_kernel 199 us (537 MB written),
// transpose 97 us, power 37 us, peaks 11 us.
#include <algorithm>
#include <mutex>
#include <vector>

#include "lbw_internal.h"

namespace lbw {
namespace {

constexpr int kBlock = 256;
constexpr int kPeakBlock = 1024;
constexpr int64_t kFirstBin = 16;
constexpr size_t kChunkBytes = size_t(1) << 30;  // bound of the columns of one spectrum (32 nfft bytes each)
constexpr size_t kCacheBytes = size_t(96) << 20; // complex array of one chunk of groups
constexpr size_t kSpectrumBytes = size_t(256) << 20;  // power spectra kept before their peaks are read off
constexpr int kMaxLog = 13;      // longest line held in LDS: 8192 points
constexpr int kRowTile = 256;    // trace rows per block of the transpose
constexpr int kColTile = 16;     // trace columns per block of the transpose
constexpr int kPairBlock = 4;    // pairs whose power one block of rows_kernel adds up
constexpr int kMostPairs = 65532;  // pairs of a chunk: the grid's limit, in whole blocks
constexpr int kTileK1 = 64, kTileK2 = 16;  // bins per block of the power kernel

// Transform of one length: n = n1 n2.
struct Split {
    int64_t T, n, n2;
    int n1, log1, log2;
};

// n1 = 64 where that leaves rows of at most 8192 points (which fit the LDS):
// 64-point columns let a block read and write 16 to 32 neighbouring columns
// at a time.  Longer transforms take longer columns, short ones sqrt(n).
// Beyond 2^26 points (traces of more than 2^24 rows) neither line would fit:
// n1 = 1, and the transform is done in radix-2 passes over memory.
Split split_for(int64_t T) {
    Split s{};
    s.T = T;
    s.n = modes_nfft(T);
    int m = 0;
    while ((int64_t(1) << m) < s.n) ++m;
    s.log1 = m > 2 * kMaxLog ? 0 : std::max(std::min(6, m / 2), m - kMaxLog);
    s.log2 = m - s.log1;
    s.n1 = 1 << s.log1;
    s.n2 = s.n >> s.log1;
    return s;
}

// The groups of one chunk.  cpg > 0: every group has cpg columns, and pairs,
// blocks of pairs and groups follow by arithmetic; else they are listed
// (device): pair -> (column, second column or -1), block -> (first pair,
// pairs), group -> (first block, blocks).
struct Groups {
    int cpg, ppg, bpg;
    const int2 *pair, *block, *group;
};

__device__ inline int2 pair_of(const Groups& g, int p) {
    if (g.cpg == 0) return g.pair[p];
    const int h = p / g.ppg, q = p - h * g.ppg, a = h * g.cpg + 2 * q;
    return make_int2(a, 2 * q + 1 < g.cpg ? a + 1 : -1);
}
__device__ inline int2 block_of(const Groups& g, int b) {
    if (g.cpg == 0) return g.block[b];
    const int h = b / g.bpg, i = b - h * g.bpg;
    return make_int2(h * g.ppg + i * kPairBlock, min(kPairBlock, g.ppg - i * kPairBlock));
}
__device__ inline int2 group_of(const Groups& g, int h) {
    return g.cpg == 0 ? g.group[h] : make_int2(h * g.bpg, g.bpg);
}

// Trace rows to columns xt[c][t] (Tp values each), the sums of kRowTile rows
// of each column (part[row tile][c]) and the twiddles exp(-2 pi i j / n2).
__global__ __launch_bounds__(kBlock) void transpose_kernel(const double* __restrict__ trace, int64_t T,
                                                           int64_t stride, int64_t col0, int cols, int64_t Tp,
                                                           double* __restrict__ xt, double* __restrict__ part,
                                                           double2* __restrict__ tw, int64_t n2) {
    __shared__ double tile[kColTile][kRowTile + 1];
    const int64_t t0 = (int64_t)blockIdx.x * kRowTile;
    const int c0 = blockIdx.y * kColTile, nc = min(kColTile, cols - c0);
    if (blockIdx.y == 0)
        for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n2; j += (int64_t)gridDim.x * kBlock) {
            double sn, cs;
            sincospi(-2.0 * (double)j / (double)n2, &sn, &cs);
            tw[j] = make_double2(cs, sn);
        }
    const int c = threadIdx.x % kColTile;
#pragma unroll 4
    for (int r = threadIdx.x / kColTile; r < kRowTile; r += kBlock / kColTile) {
        const int64_t t = t0 + r;
        tile[c][r] = c < nc && t < T ? trace[t * stride + col0 + c0 + c] : 0.0;
    }
    __syncthreads();
    for (int q = 0; q < nc; ++q) {
        const int64_t t = t0 + threadIdx.x;
        if (t < T) xt[(int64_t)(c0 + q) * Tp + t] = tile[q][threadIdx.x];
    }
    const int lane = threadIdx.x & 63;
    for (int q = threadIdx.x >> 6; q < nc; q += kBlock / 64) {
        double s = (tile[q][lane] + tile[q][lane + 64]) + (tile[q][lane + 128] + tile[q][lane + 192]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) part[(int64_t)blockIdx.x * cols + c0 + q] = s;
    }
}

__device__ inline double2 cmul(double2 a, double2 w) {
    return make_double2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}

// Radix-4 butterfly of the forward transform.
__device__ inline void radix4(double2 (&v)[4]) {
    const double2 s0 = make_double2(v[0].x + v[2].x, v[0].y + v[2].y);
    const double2 d0 = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
    const double2 s1 = make_double2(v[1].x + v[3].x, v[1].y + v[3].y);
    const double2 d1 = make_double2(v[1].x - v[3].x, v[1].y - v[3].y);
    v[0] = make_double2(s0.x + s1.x, s0.y + s1.y);
    v[1] = make_double2(d0.x + d1.y, d0.y - d1.x);
    v[2] = make_double2(s0.x - s1.x, s0.y - s1.y);
    v[3] = make_double2(d0.x - d1.y, d0.y + d1.x);
}

// Stockham passes of C = 8 NT / L transforms of length L = 2^logL held in
// LDS (element i of transform c at s[at(i, c)]), after the first radix-4
// pass (Ns = 1) has been stored.  Every thread does two radix-4 butterflies
// per pass (the last pass of an odd logL four radix-2 ones) in place, with a
// barrier between its reads and its writes.  The last pass's results stay in
// v; out(u, r) names the place of v[u][r].  Butterfly b is transform
// c = b / (L/4), or b % C with CFIRST (neighbouring lanes on neighbouring
// transforms).  tw holds exp(-2 pi i j / (L << tshift)).
template <int NT, bool CFIRST>
struct Lines {
    int logL, logC;
    __device__ int at(int i, int c) const { return CFIRST ? (i << logC) + c : (c << logL) + i; }
    __device__ void split(int b, int logB, int& c, int& j) const {
        if (CFIRST) {
            c = b & ((1 << logC) - 1);
            j = b >> logC;
        } else {
            c = b >> logB;
            j = b & ((1 << logB) - 1);
        }
    }
    __device__ bool odd() const { return (logL & 1) != 0; }
    // transform and index of result v[u][r]
    __device__ void out(int u, int r, int& c, int& k) const {
        int j;
        if (odd()) {
            split((int)threadIdx.x + (2 * u + (r >> 1)) * NT, logL - 1, c, j);
            k = j + ((r & 1) << (logL - 1));
        } else {
            split((int)threadIdx.x + u * NT, logL - 2, c, j);
            k = j + (r << (logL - 2));
        }
    }
    __device__ void passes(double2* __restrict__ s, double2 (&v)[2][4], const double2* __restrict__ tw,
                           int tshift) const {
        const int q4 = logL - 2;
        for (int ls = 2; ls + 2 <= logL; ls += 2) {  // Ns = 1 << ls
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                int c, j;
                split((int)threadIdx.x + u * NT, q4, c, j);
                const int step = (j & ((1 << ls) - 1)) << (logL - 2 - ls + tshift);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[u][r] = s[at(j + (r << q4), c)];
                    if (r > 0) v[u][r] = cmul(v[u][r], tw[step * r]);
                }
                radix4(v[u]);
            }
            if (ls + 2 == logL) return;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                int c, j;
                split((int)threadIdx.x + u * NT, q4, c, j);
                const int k = j & ((1 << ls) - 1), o = ((j >> ls) << (ls + 2)) + k;
#pragma unroll
                for (int r = 0; r < 4; ++r) s[at(o + (r << ls), c)] = v[u][r];
            }
        }
        if (!odd()) return;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int c, j;
            split((int)threadIdx.x + i * NT, logL - 1, c, j);
            const double2 a = s[at(j, c)];
            const double2 b = cmul(s[at(j + (1 << (logL - 1)), c)], tw[j << tshift]);
            v[i >> 1][(i & 1) * 2] = make_double2(a.x + b.x, a.y + b.y);
            v[i >> 1][(i & 1) * 2 + 1] = make_double2(a.x - b.x, a.y - b.y);
        }
    }
};

// Column transforms of one pair: windowed values from xt, transforms over
// j1 of C = 8 NT / n1 neighbouring j2, twiddled by exp(-2 pi i j2 k1 / n),
// to A[pair][k1][j2].
template <int NT>
__global__ __launch_bounds__(NT) void cols_kernel(Split sp, Groups g, const double* __restrict__ xt, int64_t Tp,
                                                  const double* __restrict__ part, int cols,
                                                  const double2* __restrict__ tw, double2* __restrict__ A) {
    __shared__ double2 s[8 * NT];
    __shared__ double red[2][NT / 64];
    constexpr int logE = NT == 256 ? 11 : NT == 512 ? 12 : 13;
    const Lines<NT, true> ln{sp.log1, logE - sp.log1};
    const int2 pc = pair_of(g, blockIdx.y);
    const int C = 1 << ln.logC;
    const int jb = blockIdx.x * C;
    // the two columns' means, from the row tiles' sums
    double ma = 0.0, mb = 0.0;
    const int tiles = (int)((sp.T + kRowTile - 1) / kRowTile);
    for (int i = threadIdx.x; i < tiles; i += NT) {
        ma += part[(int64_t)i * cols + pc.x];
        if (pc.y >= 0) mb += part[(int64_t)i * cols + pc.y];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        ma += __shfl_xor(ma, off, 64);
        mb += __shfl_xor(mb, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = ma;
        red[1][threadIdx.x >> 6] = mb;
    }
    __syncthreads();
    ma = mb = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        ma += red[0][i];
        mb += red[1][i];
    }
    ma /= (double)sp.T;
    mb /= (double)sp.T;
    double2 v[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        int c, j;
        ln.split((int)threadIdx.x + u * NT, sp.log1 - 2, c, j);
        const int64_t t = ((int64_t)j << sp.log2) + jb + c;
        double2 x = make_double2(0.0, 0.0);
        if (jb + c < sp.n2 && t < sp.T) {
            const double win = 0.5 - 0.5 * cospi(2.0 * (double)t / (double)(sp.T - 1));
            x.x = (xt[(int64_t)pc.x * Tp + t] - ma) * win;
            if (pc.y >= 0) x.y = (xt[(int64_t)pc.y * Tp + t] - mb) * win;
        }
        // first radix-4 pass: the inputs n/4 .. n - 1 are the zero padding
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[u][r] = x;
            if (sp.log1 > 2) s[ln.at(4 * j + r, c)] = x;
        }
    }
    ln.passes(s, v, tw, sp.log2 - sp.log1);
    double2* Ap = A + (int64_t)blockIdx.y * sp.n;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int c, k1;
            ln.out(u, r, c, k1);
            const int j2 = jb + c;
            if (j2 >= sp.n2) continue;
            double sn, cs;
            sincospi(-2.0 * (double)((int64_t)j2 * k1) / (double)sp.n, &sn, &cs);
            Ap[((int64_t)k1 << sp.log2) + j2] = cmul(v[u][r], make_double2(cs, sn));
        }
}

// Row transforms of a block of pairs: Q[block][k1][k2] = sum over its pairs
// of |Z_{k1 + n1 k2}|^2 (added to what is there when `add`).  blockIdx.x:
// C = 8 NT / n2 rows.
template <int NT>
__global__ __launch_bounds__(NT) void rows_kernel(Split sp, Groups g, const double2* __restrict__ A, int add,
                                                  const double2* __restrict__ tw, double* __restrict__ Q) {
    __shared__ double2 s[8 * NT];
    constexpr int logE = NT == 256 ? 11 : NT == 512 ? 12 : 13;
    const Lines<NT, false> ln{sp.log2, logE - sp.log2};
    const int2 pb = block_of(g, blockIdx.y);
    const int k1b = (int)blockIdx.x << ln.logC;
    double* Qb = Q + (int64_t)blockIdx.y * sp.n;
    double acc[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int c, k2;
            ln.out(u, r, c, k2);
            acc[u][r] = add && k1b + c < sp.n1 ? Qb[((int64_t)(k1b + c) << sp.log2) + k2] : 0.0;
        }
    for (int p = 0; p < pb.y; ++p) {
        const double2* Ap = A + (int64_t)(pb.x + p) * sp.n;
        double2 v[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            int c, j;
            ln.split((int)threadIdx.x + u * NT, sp.log2 - 2, c, j);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[u][r] = k1b + c < sp.n1 ? Ap[((int64_t)(k1b + c) << sp.log2) + j + (r << (sp.log2 - 2))]
                                          : make_double2(0.0, 0.0);
            radix4(v[u]);
        }
        if (p > 0) __syncthreads();  // the previous pair's last reads
        if (sp.log2 > 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                int c, j;
                ln.split((int)threadIdx.x + u * NT, sp.log2 - 2, c, j);
#pragma unroll
                for (int r = 0; r < 4; ++r) s[ln.at(4 * j + r, c)] = v[u][r];
            }
        }
        ln.passes(s, v, tw, 0);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[u][r] += v[u][r].x * v[u][r].x + v[u][r].y * v[u][r].y;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int c, k2;
            ln.out(u, r, c, k2);
            if (k1b + c < sp.n1) Qb[((int64_t)(k1b + c) << sp.log2) + k2] = acc[u][r];
        }
}

// The transforms of pairs too long for LDS: windowed values of pair
// pair0 + blockIdx.y to x, a radix-2 Stockham pass (Ns: size of the
// transforms already formed) and Q of one block of pairs.
__device__ double block_sum(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}
__global__ __launch_bounds__(kBlock) void long_fill_kernel(Split sp, Groups g, const double* __restrict__ xt,
                                                           int64_t Tp, const double* __restrict__ part, int cols,
                                                           double2* __restrict__ x) {
    __shared__ double red[kBlock / 64];
    const int2 pc = pair_of(g, blockIdx.y);
    const int64_t tiles = (sp.T + kRowTile - 1) / kRowTile;
    double ma = 0.0, mb = 0.0;
    for (int64_t i = threadIdx.x; i < tiles; i += kBlock) {
        ma += part[i * cols + pc.x];
        if (pc.y >= 0) mb += part[i * cols + pc.y];
    }
    ma = block_sum(ma, red) / (double)sp.T;
    mb = block_sum(mb, red) / (double)sp.T;
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < sp.n; t += (int64_t)gridDim.x * kBlock) {
        double2 v = make_double2(0.0, 0.0);
        if (t < sp.T) {
            const double win = 0.5 - 0.5 * cospi(2.0 * (double)t / (double)(sp.T - 1));
            v.x = (xt[pc.x * Tp + t] - ma) * win;
            if (pc.y >= 0) v.y = (xt[pc.y * Tp + t] - mb) * win;
        }
        x[blockIdx.y * sp.n + t] = v;
    }
}
__global__ __launch_bounds__(kBlock) void long_pass_kernel(const double2* __restrict__ in, double2* __restrict__ out,
                                                           int64_t n, int64_t Ns) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x, half = n / 2, k = j & (Ns - 1);
    in += blockIdx.y * n;
    out += blockIdx.y * n;
    double2 w;
    sincospi(-(double)k / (double)Ns, &w.y, &w.x);
    const double2 a = in[j], b = cmul(in[j + half], w);
    const int64_t o = 2 * j - k;
    out[o] = make_double2(a.x + b.x, a.y + b.y);
    out[o + Ns] = make_double2(a.x - b.x, a.y - b.y);
}
__global__ __launch_bounds__(kBlock) void long_sum_kernel(Split sp, Groups g, const double2* __restrict__ X, int add,
                                                          double* __restrict__ Q) {
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int2 pb = block_of(g, blockIdx.y);
    double* Qk = Q + blockIdx.y * sp.n + k;
    double s = add ? *Qk : 0.0;
    for (int p = 0; p < pb.y; ++p) {
        const double2 v = X[(int64_t)(pb.x + p) * sp.n + k];
        s += v.x * v.x + v.y * v.y;
    }
    *Qk = s;
}

// P[group][k] = sum over the group's blocks of (Q_k + Q_{n-k}) / 2, k in
// [0, n/2] (added to what is there when `add`), and the largest value of
// each block's bins from kFirstBin on.  A block covers kTileK1 x kTileK2 bins
// k1 + n1 k2, read along k2 and written along k1.
__global__ __launch_bounds__(kBlock) void power_kernel(Split sp, Groups g, const double* __restrict__ Q, int add,
                                                       double* __restrict__ Pall, double* __restrict__ pmax) {
    __shared__ double tile[kTileK2][kTileK1 + 1];
    __shared__ double red[kBlock / 64];
    const int tiles1 = (sp.n1 + kTileK1 - 1) / kTileK1;
    const int k1b = (blockIdx.x % tiles1) * kTileK1;
    const int64_t k2b = (int64_t)(blockIdx.x / tiles1) * kTileK2;
    const int2 gb = group_of(g, blockIdx.y);
    const int64_t half = sp.n / 2;
    double* P = Pall + (int64_t)blockIdx.y * (half + 1);
    const int c2 = threadIdx.x % kTileK2;
    const int64_t k2 = k2b + c2;
    for (int r1 = threadIdx.x / kTileK2; r1 < kTileK1; r1 += kBlock / kTileK2) {
        const int k1 = k1b + r1;
        double v = 0.0;
        if (k1 < sp.n1 && k2 < sp.n2 && k1 + (k2 << sp.log1) <= half) {
            // bin n - k (mod n)
            const int m1 = k1 == 0 ? 0 : sp.n1 - k1;
            const int64_t m2 = k1 == 0 ? (k2 == 0 ? 0 : sp.n2 - k2) : sp.n2 - 1 - k2;
            const int64_t i = ((int64_t)k1 << sp.log2) + k2, j = ((int64_t)m1 << sp.log2) + m2;
            v = add ? P[k1 + (k2 << sp.log1)] : 0.0;
            for (int b = gb.x; b < gb.x + gb.y; ++b) v += 0.5 * (Q[b * sp.n + i] + Q[b * sp.n + j]);
        }
        tile[c2][r1] = v;
    }
    __syncthreads();
    double m = 0.0;
    const int w1 = min(kTileK1, sp.n1);  // a power of two
    for (int i = threadIdx.x; i < w1 * kTileK2; i += kBlock) {
        const int r1 = i & (w1 - 1), q2 = i / w1;
        const int64_t k = k1b + r1 + ((k2b + q2) << sp.log1);
        if (k > half) continue;
        P[k] = tile[q2][r1];
        if (k >= kFirstBin) m = fmax(m, tile[q2][r1]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
        pmax[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// One block per group: the largest value from the power kernel's blocks,
// then an ordered scan.
__global__ __launch_bounds__(kPeakBlock) void peaks_kernel(const double* __restrict__ Pall,
                                                           const double* __restrict__ pmax, int nmax, int64_t nfft,
                                                           int k, double* __restrict__ freq,
                                                           double* __restrict__ power) {
    constexpr int W = kPeakBlock / 64;
    __shared__ double red[W];
    __shared__ int cnt[2][W];
    const int64_t last = nfft / 2;
    const double* P = Pall + (size_t)blockIdx.x * (last + 1);
    freq += (size_t)blockIdx.x * k;
    power += (size_t)blockIdx.x * k;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double m = 0.0;
    for (int i = threadIdx.x; i < nmax; i += kPeakBlock) m = fmax(m, pmax[(size_t)blockIdx.x * nmax + i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if (lane == 0) red[wave] = m;
    for (int i = threadIdx.x; i < k; i += kPeakBlock) {
        freq[i] = __longlong_as_double(0x7ff8000000000000LL);
        power[i] = __longlong_as_double(0x7ff8000000000000LL);
    }
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int i = 1; i < W; ++i) m = fmax(m, red[i]);
    const double thr = 1e-3 * m;
    int found = 0, bank = 0;
    for (int64_t base = kFirstBin; base < last && found < k; base += kPeakBlock, bank ^= 1) {
        const int64_t b = base + threadIdx.x;
        const bool flag = b < last && P[b - 1] < P[b] && P[b] >= P[b + 1] && P[b] > thr;
        const uint64_t votes = __ballot(flag);
        if (lane == 0) cnt[bank][wave] = __popcll(votes);
        __syncthreads();  // (the other bank is free again after the next barrier)
        int before = 0, all = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            before += i < wave ? cnt[bank][i] : 0;
            all += cnt[bank][i];
        }
        const int slot = found + before + __popcll(votes & ((uint64_t(1) << lane) - 1));
        if (flag && slot < k) {
            const double pm = P[b - 1], p0 = P[b], pp = P[b + 1];
            const double l0 = log(p0);
            double delta = 0.0, lm = 0.0, lp = 0.0;
            if (pm > 0.0 && pp > 0.0) {
                lm = log(pm);
                lp = log(pp);
                const double den = lm - 2.0 * l0 + lp;
                delta = den != 0.0 ? 0.5 * (lm - lp) / den : 0.0;
            }
            freq[slot] = ((double)b + delta) / (double)nfft;
            power[slot] = exp(l0 - 0.25 * (lm - lp) * delta);
        }
        found += all;
    }
}

// Work space of the allocation-free spectrum: a fixed array in device
// memory, one per GPU the library runs on, kept until the process ends.
// Host code never passes `scratch` itself to a kernel (on the host the name
// is only a stand-in for the symbol); it uses the device address that
// hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[kModesScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

hipError_t modes_scratch(void** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

int64_t modes_nfft(int64_t T) {
    int64_t p = 1;
    while (p < T) p *= 2;
    return 4 * p;
}

int modes_max_cols(int64_t T) {
    const size_t per_col = 2 * (size_t)modes_nfft(T) * sizeof(double2);
    return (int)std::max<size_t>(1, kChunkBytes / per_col);
}

namespace {

// Work space of one chunk: `cols` columns in `pairs` pairs, `blocks` blocks
// and `groups` groups.
struct Work {
    double2 *A, *B, *tw;  // B: second array of a transform in passes
    double *xt, *part, *Q, *P, *pmax;
    int64_t Tp;
    int nmax;  // blocks of the power kernel per group
    size_t bytes;
};

Work layout(const Split& sp, void* base, int64_t cols, int64_t pairs, int64_t blocks, int64_t groups) {
    Work w{};
    unsigned char* const p0 = static_cast<unsigned char*>(base);
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t o = at;
        at += (bytes + 255) / 256 * 256;
        return p0 ? p0 + o : nullptr;
    };
    w.Tp = (sp.T + 15) / 16 * 16;
    w.nmax = ((sp.n1 + kTileK1 - 1) / kTileK1) * (int)((sp.n2 / 2 + 1 + kTileK2 - 1) / kTileK2);
    w.A = reinterpret_cast<double2*>(take(sizeof(double2) * (size_t)(pairs * sp.n)));
    if (sp.n1 == 1) w.B = reinterpret_cast<double2*>(take(sizeof(double2) * (size_t)(pairs * sp.n)));
    w.tw = reinterpret_cast<double2*>(take(sp.n1 == 1 ? 0 : sizeof(double2) * (size_t)sp.n2));
    w.xt = reinterpret_cast<double*>(take(sizeof(double) * (size_t)(cols * w.Tp)));
    w.part = reinterpret_cast<double*>(take(sizeof(double) * (size_t)(cols * ((sp.T + kRowTile - 1) / kRowTile))));
    w.Q = reinterpret_cast<double*>(take(sizeof(double) * (size_t)(blocks * sp.n)));
    w.P = reinterpret_cast<double*>(take(sizeof(double) * (size_t)(groups * (sp.n / 2 + 1))));
    w.pmax = reinterpret_cast<double*>(take(sizeof(double) * (size_t)(groups * w.nmax)));
    w.bytes = at;
    return w;
}

// Transforms `pairs` pairs of columns from col0 on and leaves Q of their
// `blocks` blocks.
void launch_transforms(const Split& sp, const Groups& g, const Work& w, const double* trace, int64_t stride,
                       int64_t col0, int cols, int pairs, int blocks, int add, hipStream_t st) {
    hipLaunchKernelGGL(transpose_kernel,
                       dim3((unsigned)((sp.T + kRowTile - 1) / kRowTile), (unsigned)((cols + kColTile - 1) / kColTile)),
                       dim3(kBlock), 0, st, trace, sp.T, stride, col0, cols, w.Tp, w.xt, w.part, w.tw,
                       sp.n1 == 1 ? 0 : sp.n2);
    if (sp.n1 == 1) {
        const dim3 half((unsigned)(sp.n / 2 / kBlock), (unsigned)pairs);
        hipLaunchKernelGGL(long_fill_kernel, dim3(4096, (unsigned)pairs), dim3(kBlock), 0, st, sp, g, w.xt, w.Tp,
                           w.part, cols, w.A);
        double2 *src = w.A, *dst = w.B;
        for (int64_t Ns = 1; Ns < sp.n; Ns *= 2) {
            hipLaunchKernelGGL(long_pass_kernel, half, dim3(kBlock), 0, st, src, dst, sp.n, Ns);
            std::swap(src, dst);
        }
        hipLaunchKernelGGL(long_sum_kernel, dim3((unsigned)(sp.n / kBlock), (unsigned)blocks), dim3(kBlock), 0, st, sp,
                           g, src, add, w.Q);
        return;
    }
    // 8 values per thread; the block is the smallest of 256, 512 and 1024
    // threads that holds a whole line
    const auto grid = [&](int nt, int64_t line, int64_t lines, int y) {
        const int64_t per = std::max<int64_t>(1, 8 * nt / line);
        return dim3((unsigned)((lines + per - 1) / per), (unsigned)y);
    };
    if (sp.n1 <= 2048)
        hipLaunchKernelGGL(cols_kernel<256>, grid(256, sp.n1, sp.n2, pairs), dim3(256), 0, st, sp, g, w.xt, w.Tp,
                           w.part, cols, w.tw, w.A);
    else if (sp.n1 <= 4096)
        hipLaunchKernelGGL(cols_kernel<512>, grid(512, sp.n1, sp.n2, pairs), dim3(512), 0, st, sp, g, w.xt, w.Tp,
                           w.part, cols, w.tw, w.A);
    else
        hipLaunchKernelGGL(cols_kernel<1024>, grid(1024, sp.n1, sp.n2, pairs), dim3(1024), 0, st, sp, g, w.xt, w.Tp,
                           w.part, cols, w.tw, w.A);
    if (sp.n2 <= 2048)
        hipLaunchKernelGGL(rows_kernel<256>, grid(256, sp.n2, sp.n1, blocks), dim3(256), 0, st, sp, g, w.A, add, w.tw,
                           w.Q);
    else if (sp.n2 <= 4096)
        hipLaunchKernelGGL(rows_kernel<512>, grid(512, sp.n2, sp.n1, blocks), dim3(512), 0, st, sp, g, w.A, add, w.tw,
                           w.Q);
    else
        hipLaunchKernelGGL(rows_kernel<1024>, grid(1024, sp.n2, sp.n1, blocks), dim3(1024), 0, st, sp, g, w.A, add,
                           w.tw, w.Q);
}

// Power spectra of `groups` groups, the first at place `at` of w.P.
void launch_power(const Split& sp, const Groups& g, const Work& w, int at, int groups, int add, hipStream_t st) {
    hipLaunchKernelGGL(power_kernel, dim3((unsigned)w.nmax, (unsigned)groups), dim3(kBlock), 0, st, sp, g, w.Q, add,
                       w.P + (int64_t)at * (sp.n / 2 + 1), w.pmax + (int64_t)at * w.nmax);
}

inline int pairs_of(int cols) { return (cols + 1) / 2; }
inline int blocks_of(int cols) { return (pairs_of(cols) + kPairBlock - 1) / kPairBlock; }

// A single group of `cols` columns.
Groups one_group(int cols) {
    Groups g{};
    g.cpg = cols;
    g.ppg = pairs_of(cols);
    g.bpg = blocks_of(cols);
    return g;
}

// Groups whose power spectra are kept before their peaks are read off.
int64_t spectra_kept(const Split& sp) {
    return std::max<int64_t>(1, (int64_t)(kSpectrumBytes / (sizeof(double) * (size_t)(sp.n / 2 + 1))));
}

// Whole groups [g0, g1) of one chunk: at most the columns of one spectrum
// and, with more than one group, at most kCacheBytes of transforms.  A group of
// more than kMostPairs pairs is a chunk for every so many of them (part of
// `parts`), whose powers are added up in the order of the pairs.
struct Chunk {
    int g0, g1, cols, pairs, blocks, part, parts;
};
Chunk next_chunk(const Split& sp, const int* group_ncols, int groups, int g0, int cap) {
    Chunk c{g0, g0, 0, 0, 0, 0, 1};
    while (c.g1 < groups) {
        const int n = group_ncols[c.g1], pairs = c.pairs + pairs_of(n);
        if (c.cols + n > cap) break;
        if (c.g1 > g0 && (size_t)pairs * (size_t)sp.n * sizeof(double2) > kCacheBytes) break;
        if (pairs > kMostPairs && c.g1 > g0) break;
        if (c.g1 - g0 >= std::min<int64_t>(65535, spectra_kept(sp))) break;  // grid limit
        c.cols += n;
        c.pairs = pairs;
        c.blocks += blocks_of(n);
        c.g1 += 1;
    }
    return c;
}

}  // namespace

// Pairs of columns that the fixed work space holds (0: the trace is too long).
static int static_pairs(const Split& sp) {
    // the columns of one pass are bounded as the 32 nfft bytes of work space
    // per column that the entry point documents
    if (sp.n > 4 * (int64_t)LBW_MODES_NOALLOC_MAX_ROWS) return 0;
    int pairs = 0;
    while (pairs < 32 * kPairBlock &&
           layout(sp, nullptr, 2 * (pairs + 1), pairs + 1, (pairs + kPairBlock) / kPairBlock, 1).bytes <=
               kModesScratchBytes)
        ++pairs;
    return pairs > kPairBlock ? pairs / kPairBlock * kPairBlock : pairs;
}

int modes_static_cols(int64_t T) { return 2 * static_pairs(split_for(T)); }

hipError_t launch_modes_static(void* scratch_ptr, const double* trace, int64_t T, int64_t stride, int ncols, int k,
                               double* freq, double* power, hipStream_t st) {
    const Split sp = split_for(T);
    const int per_pass = static_pairs(sp);
    if (per_pass < 1 || ncols < 1) return hipErrorInvalidValue;
    const int pairs = pairs_of(ncols);
    const Work w = layout(sp, scratch_ptr, 2 * std::min(per_pass, pairs), std::min(per_pass, pairs),
                          (std::min(per_pass, pairs) + kPairBlock - 1) / kPairBlock, 1);
    // passes of whole blocks of pairs, or of parts of one block: the power of
    // a block is added up in the order of its pairs either way
    int add = 0;
    for (int p0 = 0; p0 < pairs;) {
        int np = std::min(per_pass, pairs - p0);
        const int in_block = p0 % kPairBlock;
        if (per_pass < kPairBlock) np = std::min(np, kPairBlock - in_block);
        const int c0 = 2 * p0, cols = std::min(2 * np, ncols - c0);
        const Groups g = one_group(cols);
        launch_transforms(sp, g, w, trace, stride, c0, cols, np, g.bpg, in_block > 0 ? 1 : 0, st);
        p0 += np;
        if (p0 == pairs || p0 % kPairBlock == 0) {
            launch_power(sp, g, w, 0, 1, add, st);
            add = 1;
        }
    }
    hipLaunchKernelGGL(peaks_kernel, dim3(1), dim3(kPeakBlock), 0, st, w.P, w.pmax, w.nmax, sp.n, k, freq, power);
    return hipGetLastError();
}

namespace {

// The chunks of a call, their largest work space (with the spectra kept) and
// the entries of their lists.
struct Plan {
    std::vector<Chunk> chunks;
    int64_t cols = 0, pairs = 0, blocks = 0, groups = 0;  // most of any chunk; groups: spectra kept
    int64_t list = 0;
    bool ok = true;
};
Plan plan_chunks(const Split& sp, const int* group_ncols, int groups, int cap) {
    Plan p;
    for (int g0 = 0; g0 < groups;) {
        const Chunk c = next_chunk(sp, group_ncols, groups, g0, cap);
        if (c.g1 == g0) {
            p.ok = false;
            break;
        }
        g0 = c.g1;
        if (c.pairs > kMostPairs) {  // (one group)
            const int parts = (c.pairs + kMostPairs - 1) / kMostPairs;
            for (int i = 0; i < parts; ++i) {
                const int cols = std::min(2 * kMostPairs, c.cols - i * 2 * kMostPairs);
                p.chunks.push_back(Chunk{c.g0, c.g1, cols, pairs_of(cols), blocks_of(cols), i, parts});
            }
            p.cols = std::max<int64_t>(p.cols, 2 * kMostPairs);
            p.pairs = std::max<int64_t>(p.pairs, kMostPairs);
            p.blocks = std::max<int64_t>(p.blocks, kMostPairs / kPairBlock);
            continue;
        }
        p.chunks.push_back(c);
        p.cols = std::max<int64_t>(p.cols, c.cols);
        p.pairs = std::max<int64_t>(p.pairs, c.pairs);
        p.blocks = std::max<int64_t>(p.blocks, c.blocks);
        p.list += c.pairs + c.blocks + (c.g1 - c.g0);
    }
    p.groups = std::min<int64_t>(groups, std::min<int64_t>(65535, spectra_kept(sp)));
    return p;
}

}  // namespace

size_t modes_work_bytes(int64_t T, const int* group_ncols, int groups) {
    const Split sp = split_for(T);
    const Plan p = plan_chunks(sp, group_ncols, groups, modes_max_cols(T));
    if (!p.ok) return 0;
    return layout(sp, nullptr, p.cols, p.pairs, p.blocks, p.groups).bytes + sizeof(int2) * (size_t)p.list;
}

hipError_t launch_modes_grouped(const double* trace, int64_t T, int64_t stride, const int* group_ncols, int groups,
                                int k, double* work, size_t work_bytes, double* freq, double* power,
                                hipStream_t st) {
    const Split sp = split_for(T);
    const Plan plan = plan_chunks(sp, group_ncols, groups, modes_max_cols(T));
    if (!plan.ok || work_bytes < modes_work_bytes(T, group_ncols, groups)) return hipErrorInvalidValue;
    const Work w = layout(sp, work, plan.cols, plan.pairs, plan.blocks, plan.groups);
    bool uniform = group_ncols[0] > 0;
    for (int g = 1; g < groups; ++g)
        if (group_ncols[g] != group_ncols[0]) uniform = false;
    // groups of different sizes: the lists of pairs, blocks and groups, chunk
    // after chunk, numbered within their chunk, behind the work space
    std::vector<int2> list;
    int2* const d_list = reinterpret_cast<int2*>(reinterpret_cast<unsigned char*>(work) + w.bytes);
    if (!uniform) {
        list.reserve((size_t)plan.list);
        for (const Chunk& c : plan.chunks) {
            if (c.parts > 1) continue;
            int col = 0, pair = 0, block = 0;
            for (int g = c.g0; g < c.g1; col += group_ncols[g++])
                for (int q = 0; q < group_ncols[g]; q += 2)
                    list.push_back(make_int2(col + q, q + 1 < group_ncols[g] ? col + q + 1 : -1));
            for (int g = c.g0; g < c.g1; pair += pairs_of(group_ncols[g++]))
                for (int q = 0; q < pairs_of(group_ncols[g]); q += kPairBlock)
                    list.push_back(make_int2(pair + q, std::min(kPairBlock, pairs_of(group_ncols[g]) - q)));
            for (int g = c.g0; g < c.g1; block += blocks_of(group_ncols[g++]))
                list.push_back(make_int2(block, blocks_of(group_ncols[g])));
        }
        const hipError_t e = hipMemcpyAsync(d_list, list.data(), sizeof(int2) * list.size(), hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return e;
    }
    const int2* next = d_list;
    int64_t col0 = 0;
    int kept0 = 0;  // first group whose spectrum is kept
    for (size_t i = 0; i < plan.chunks.size(); ++i) {
        const Chunk& c = plan.chunks[i];
        Groups g = one_group(c.parts > 1 ? c.cols : group_ncols[0]);
        if (!uniform && c.parts == 1) {
            g.cpg = 0;
            g.pair = next;
            g.block = g.pair + c.pairs;
            g.group = g.block + c.blocks;
            next = g.group + (c.g1 - c.g0);
        }
        if (c.cols > 0) launch_transforms(sp, g, w, trace, stride, col0, c.cols, c.pairs, c.blocks, 0, st);
        launch_power(sp, g, w, c.g0 - kept0, c.g1 - c.g0, c.part > 0 ? 1 : 0, st);
        if (i + 1 == plan.chunks.size() || plan.chunks[i + 1].g1 - kept0 > plan.groups) {
            hipLaunchKernelGGL(peaks_kernel, dim3(c.g1 - kept0), dim3(kPeakBlock), 0, st, w.P, w.pmax, w.nmax, sp.n, k,
                               freq + (size_t)kept0 * k, power + (size_t)kept0 * k);
            kept0 = c.g1;
        }
        col0 += c.cols;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || list.empty()) return e;
    return hipStreamSynchronize(st);  // the host list goes out of scope
}

}  // namespace lbw
