// Several time steps per launch of a 2-D grid (D2Q5), the state on chip.
//
// A 2-D grid is small (64 x 64 to a few million nodes): one step per launch
// costs a launch and a round trip to memory per step, whatever the grid.
// Here a workgroup takes a tile with a halo of two nodes per step (a node's
// next state depends on S two nodes away), keeps it in registers, and writes
// the tile back after the last step:
//  - a wave owns a strip of R rows of 64 nodes along axis 0, one lane per
//    column: axis-0 neighbours come by a wave-wide lane shift (DPP, no LDS),
//    axis-1 neighbours are registers of the same lane;
//  - strips are stacked along axis 1.  After a collision a wave sends, for
//    each side, its outgoing populations and what its neighbour needs to form
//    the new S = sum_l f_l of the adjoining row itself: one exchange of five
//    values per lane through LDS, and one barrier, per step;
//  - a probe node's populations are put aside in LDS and summed and divided
//    by sqrt(g) in FP64 by the whole workgroup when there are many (done by
//    the owning wave at every step, the division held up all the others).
//    Each lane knows its own probe nodes, as one bit a row: with every wave
//    going through the list of places at every step, 64 probes on 64 x 64 nodes
//    took 6.8 us a step, so 2.4 (1.2 without probes);
//  - a node next to the tile's outer edge has no neighbour there; what it
//    computes is wrong, and the error moves in by two nodes per step, so after
//    k steps exactly the halo is spoilt, which is not written;
//  - an axis that fits the tile whole has no halo (a walled axis 0 of at
//    most 64 nodes; axis 1, periodic or walled, in one column of strips), and
//    a grid that fits whole along both takes any number of steps.
// Every node is computed by collide_2d, the one-step kernel's routine, and
// wall rules and streaming move the same values, so results are those of
// single steps bit for bit.
//
// The vector instructions (272 for eight rows with walls on axis 0, 210 without,
// of which 188 are arithmetic) bound a grid that fits whole, and a third of a
// tiled one, whose launch, first loads and last stores are the rest.  64 x 64
// nodes: 3.9 us a step with one step per launch, 1.25 so, 1.27 with a probe (one
// workgroup, no launches in between); 701 x 503: 10.4 and 2.8 to 3.15 (234 tiles
// of 64 x 64 nodes, five or six steps per launch).
#include <type_traits>

#include "march_common.h"

namespace lbw {
namespace {

using namespace march;

constexpr int kLanes = 64;
constexpr int kMaxWaves = 16;
constexpr int kTileProbes = 64;
constexpr int kHeld = 1024;

// lane i receives lane i - 1's (shr) or lane i + 1's (shl) value, the end lane 0
__device__ __forceinline__ float lane_shr(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_shl(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

// i on a periodic axis of n nodes (a halo may go round a short axis more
// than once)
__device__ inline int wrapped(int i, int n) {
    while (i < 0) i += n;
    while (i >= n) i -= n;
    return i;
}

// Tile `i` of `tiles` along an axis of n nodes (shares of n / tiles nodes, the
// first n % tiles of them one more): own nodes [a, b) and the nodes [lo, hi)
// held for `k` steps (coordinates beyond a periodic axis wrap).
struct Span {
    int a, b, lo, hi;
};
__host__ __device__ inline Span tile_span(int i, int share, int more, int n, bool periodic, bool whole, int k) {
    Span s;
    s.a = i * share + (i < more ? i : more);
    s.b = s.a + share + (i < more ? 1 : 0);
    s.lo = s.a - 2 * k;
    s.hi = s.b + 2 * k;
    if (!periodic) {
        s.lo = s.lo < 0 ? 0 : s.lo;
        s.hi = s.hi > n ? n : s.hi;
    }
    if (whole) {
        s.lo = 0;
        s.hi = n;
    }
    return s;
}

struct Tile2Lds {
    // per bank and wave: the first row's f_0 + f_1 + f_2, f_4 and outgoing
    // f*_4 (for the wave below), the last row's f_0 + .. + f_3 and outgoing
    // f*_3 (for the wave above)
    float down[2][3][kMaxWaves][kLanes];
    float up[2][2][kMaxWaves][kLanes];
    // probes: trace column, thread << 3 | row, sqrt(g)
    int probe[kTileProbes], place[kTileProbes];
    double sqrtg[kTileProbes];
    // the rows of a thread that hold probe nodes, the number of its first; and
    // the populations of up to kHeld recordings of a node
    unsigned mask[kLanes * kMaxWaves];
    int base[kLanes * kMaxWaves];
    float held[kHeld][5];
    int count, nodes;
};

// fout may be fin, and pr.tout pr.tin, where the grid is one workgroup's.
// FREE: a wall may be a free one (its rule returns the node's own
// population; the others scale the outgoing one).
template <int R, bool FREE>
__global__ __launch_bounds__(kLanes* kMaxWaves) void step_tile2_kernel(GeomDev g, ProbeArgs pr, Tile2Plan plan,
                                                                       int steps, int share0, int more0, int share1,
                                                                       int more1, const float* fin,
                                                                       float* fout) {
#pragma clang fp contract(off)
    __shared__ Tile2Lds L;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n0 = g.n0, n1 = g.n1;
    const uint32_t N = (uint32_t)g.N;
    const bool per0 = g.bc_lo[0] == LBW_BC_PERIODIC, per1 = g.bc_lo[1] == LBW_BC_PERIODIC;
    const bool whole1 = plan.nty == 1;
    const Span sx = tile_span(blockIdx.x, share0, more0, n0, per0, plan.ntx == 1 && !per0, steps);
    const Span sy = tile_span(blockIdx.y, share1, more1, n1, per1, whole1, steps);
    const int EX = sx.hi - sx.lo, EY = sy.hi - sy.lo;
    const int row0 = wave * R;
    const int nr = min(max(EY - row0, 0), R);  // rows of this strip
    const int last = (EY - 1) / R;             // the last wave with rows
    const bool ring = whole1 && per1;          // the strips close into a ring
    // the ends of the strip: a neighbouring wave, a wall, or the tile's edge
    const bool wall_b = wave == 0 && !per1 && sy.lo == 0;
    const bool wall_t = wave == last && !per1 && sy.hi == n1;
    const int below = wave > 0 ? wave - 1 : ring ? last : 0;
    const int above = wave < last ? wave + 1 : 0;
    const bool have_b = wave > 0 ? wave <= last : ring, have_t = wave < last || (ring && wave == last);

    const int x = sx.lo + lane;
    const bool act = lane < EX;
    const int xg = act ? (per0 ? wrapped(x, n0) : x) : 0;
    const bool wall_l = !per0 && x == 0, wall_r = !per0 && x == n0 - 1;
    const bool walls0 = !per0 && (sx.lo == 0 || sx.hi == n0);  // some lane has an axis-0 wall
    const float* te = g.tab + (size_t)xg * kTabF32;
    const float cM00 = te[0], cM11 = te[3], hG0 = te[4];
    const float c2 = g.c2, two_w0 = g.two_w0, damp = g.damp;
    const int lo0 = g.bc_lo[0], hi0 = g.bc_hi[0], lo1 = g.bc_lo[1], hi1 = g.bc_hi[1];
    // what a wall returns: a factor times the outgoing population (or, free,
    // the node's own opposite one)
    const auto factor = [&](int wall) { return wall == LBW_BC_BOUNCEBACK ? damp : -1.0f; };
    const float m_l = factor(lo0), m_r = factor(hi0), m_b = factor(lo1), m_t = factor(hi1);
    const auto back = [&](int wall, float m, float out, float own) {
        if constexpr (FREE) return wall == LBW_BC_FREE ? own : m * out;
        return m * out;
    };

    float f[R][5], S[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = sy.lo + row0 + r;
        const bool on = act && r < nr;
        const uint32_t n = on ? (uint32_t)xg + (uint32_t)n0 * (uint32_t)(per1 ? wrapped(y, n1) : y) : 0u;
#pragma unroll
        for (int l = 0; l < 5; ++l) {
            const float v = fin[(uint32_t)l * N + n];
            f[r][l] = on ? v : 0.f;
        }
        S[r] = f[r][0] + f[r][1] + f[r][2] + f[r][3] + f[r][4];
    }

    // the tile's probes
    const int64_t t = *pr.tin;
    L.mask[threadIdx.x] = 0;
    if (threadIdx.x == 0) L.count = L.nodes = 0;
    __syncthreads();
    if (t >= 0 && t < pr.t_max)
        for (int p = threadIdx.x; p < pr.n; p += blockDim.x) {
            const int node = (int)pr.nodes[p];
            const int i0 = node % n0, i1 = node / n0;
            if (i0 < sx.a || i0 >= sx.b || i1 < sy.a || i1 >= sy.b) continue;
            const int slot = atomicAdd(&L.count, 1);
            if (slot < kTileProbes) {
                const int row = i1 - sy.lo, who = row / R * kLanes + i0 - sx.lo;
                L.probe[slot] = p;
                L.place[slot] = who << 3 | row % R;
                L.sqrtg[slot] = g.sqrtg[i0];
                atomicOr(&L.mask[who], 1u << (row % R));
            }
        }

    // S of the rows next to the strip, from bank 1 (first written by step 1)
    L.down[1][0][wave][lane] = S[0];
    {
        float top = S[0];
#pragma unroll
        for (int r = 1; r < R; ++r) top = r == nr - 1 ? S[r] : top;
        L.up[1][0][wave][lane] = top;
    }
    __syncthreads();
    const int probes = __builtin_amdgcn_readfirstlane(min(L.count, kTileProbes));
    const unsigned mask = L.mask[threadIdx.x];
    unsigned wave_mask = 0;  // (uniform) rows of the strip with a probe node
    int base = 0, nodes = 0;
    if (probes > 0) {
        if (mask) {
            base = atomicAdd(&L.nodes, __popc(mask));
            L.base[threadIdx.x] = base;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (__builtin_amdgcn_ballot_w64((mask >> r) & 1u)) wave_mask |= 1u << r;
        __syncthreads();
        nodes = __builtin_amdgcn_readfirstlane(L.nodes);
        wave_mask = (unsigned)__builtin_amdgcn_readfirstlane((int)wave_mask);
    }
    float Sb = L.up[1][0][below][lane], St = L.down[1][0][above][lane];

    // One step of the strip: collision and streaming, up to what the
    // neighbouring strips send.  FULL: all R rows exist; WALLS: lanes with an
    // axis-0 wall.
    float up3 = 0.f, upS = 0.f, down4 = 0.f;
    const auto advance = [&](auto full, auto walls) {
        constexpr bool FULL = decltype(full)::value, WALLS = decltype(walls)::value;
        float fs[R][5], a11[R];
#pragma unroll
        for (int r = 0; r < R; ++r) a11[r] = cM11 * S[r];
        const float a11b = wall_b ? ghost(lo1, a11[0]) : cM11 * Sb;
        const float a11t = cM11 * St;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float a00 = cM00 * S[r];
            float a00p = lane_shl(a00), a00m = lane_shr(a00);
            if constexpr (WALLS) {
                a00p = wall_r ? ghost(hi0, a00) : a00p;
                a00m = wall_l ? ghost(lo0, a00) : a00m;
            }
            const bool top = FULL ? r == R - 1 : r == nr - 1;
            const float a11p = top ? (wall_t ? ghost(hi1, a11[r]) : a11t) : a11[r + 1 < R ? r + 1 : r];
            const float a11m = r == 0 ? a11b : a11[r > 0 ? r - 1 : r];
            collide_2d(f[r], S[r], a00p, a00m, a11p, a11m, hG0, c2, two_w0, fs[r]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool top = FULL ? r == R - 1 : r == nr - 1;
            f[r][0] = fs[r][0];
            f[r][1] = lane_shr(fs[r][1]);
            f[r][2] = lane_shl(fs[r][2]);
            if constexpr (WALLS) {
                f[r][1] = wall_l ? back(lo0, m_l, fs[r][2], fs[r][1]) : f[r][1];
                f[r][2] = wall_r ? back(hi0, m_r, fs[r][1], fs[r][2]) : f[r][2];
            }
            f[r][3] = r > 0 ? fs[r > 0 ? r - 1 : r][3] : back(lo1, m_b, fs[r][4], fs[r][3]);
            f[r][4] = top ? back(hi1, m_t, fs[r][3], fs[r][4]) : fs[r + 1 < R ? r + 1 : r][4];
            S[r] = f[r][0] + f[r][1] + f[r][2];
            if (top) {
                up3 = fs[r][3];
                upS = S[r] + f[r][3];
            }
        }
        down4 = fs[0][4];
    };
    // recordings held in LDS: the probes of steps s0 .. s - 1
    int s0 = 0;
    const auto flush = [&](int s) {
        const int64_t most = pr.t_max - (t + s0);
        const int rows = (int)min((int64_t)(s - s0), most < 0 ? 0 : most);
        for (int i = threadIdx.x; i < rows * probes; i += blockDim.x) {
            const int p = i % probes, who = L.place[p] >> 3, row = L.place[p] & 7;
            const int at = i / probes * nodes + L.base[who] + __popc(L.mask[who] & ((1u << row) - 1u));
            double sum = 0.0;
#pragma unroll
            for (int l = 0; l < 5; ++l) sum += (double)L.held[at][l];
            pr.trace[(t + s0 + i / probes) * pr.n + L.probe[p]] = sum / L.sqrtg[p];
        }
        s0 = s;
    };

    for (int s = 0; s < steps; ++s) {
        if (probes > 0) {
            if ((s - s0 + 1) * nodes > kHeld) {
                // (the last step's barrier made its recordings visible)
                flush(s);
                __syncthreads();
            }
            // (a loop over the strip's probe rows: unrolled, with a branch for
            // each row, R = 8 takes 45 registers more than there are)
            if (wave_mask) {
                const int at = (s - s0) * nodes + base;
                for (unsigned w = wave_mask; w; w &= w - 1) {
                    const int row = __builtin_ctz(w);
                    float v[5];
#pragma unroll
                    for (int l = 0; l < 5; ++l) v[l] = f[0][l];
#pragma unroll
                    for (int r = 1; r < R; ++r)
                        if (r == row)
#pragma unroll
                            for (int l = 0; l < 5; ++l) v[l] = f[r][l];
                    if ((mask >> row) & 1u)
#pragma unroll
                        for (int l = 0; l < 5; ++l) L.held[at + __popc(mask & ((1u << row) - 1u))][l] = v[l];
                }
            }
        }
        if (nr == R) {
            if (walls0) advance(std::true_type{}, std::true_type{});
            else advance(std::true_type{}, std::false_type{});
        } else if (nr > 0) {
            advance(std::false_type{}, std::true_type{});
        }
        const int bank = s & 1;
        L.down[bank][0][wave][lane] = S[0];
        L.down[bank][1][wave][lane] = f[0][4];
        L.down[bank][2][wave][lane] = down4;
        L.up[bank][0][wave][lane] = upS;
        L.up[bank][1][wave][lane] = up3;
        __syncthreads();  // (the other bank is written only after the next one)
        if (have_b) {
            f[0][3] = L.up[bank][1][below][lane];
            Sb = L.up[bank][0][below][lane] + down4;
        }
        if (have_t) {
            const float in = L.down[bank][2][above][lane];
            St = (L.down[bank][0][above][lane] + up3) + L.down[bank][1][above][lane];
            if (nr == R) {
                f[R - 1][4] = in;
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) f[r][4] = r == nr - 1 ? in : f[r][4];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) S[r] = (S[r] + f[r][3]) + f[r][4];
    }
    if (probes > 0) flush(steps);

#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = sy.lo + row0 + r;
        if (r < nr && x >= sx.a && x < sx.b && y >= sy.a && y < sy.b) {
            const uint32_t n = (uint32_t)x + (uint32_t)n0 * (uint32_t)y;
#pragma unroll
            for (int l = 0; l < 5; ++l) fout[(uint32_t)l * N + n] = f[r][l];
        }
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *pr.tout = t + steps;
}

}  // namespace

int tile2_probes() { return kTileProbes; }

// The tiling with the lowest modelled cost per step.  A launch costs
// kLaunch, plus what it loads (halos included) and stores at kBytes; a step
// costs, for each round of workgroups (one per CU), kRow for every row of a
// strip (about 45 wave instructions) and half a row for its exchange, on the
// busiest of the four SIMDs, and at least kStep.
// The constants are from sweeps of rows, strips and k on 64 x 64 and 701 x
// 503 nodes, which the model meets within 12 %: 701 x 503 in 4 x 16 rows 3.58
// us a step at k = 4, 3.06 at 5, 2.82 at 6 (7 needs a second round of
// workgroups); 64 x 64 whole 1.40, in 8 tiles of 24 rows and k = 4 1.71.  On
// other sizes it gives, and long blocks take: 30 x 40 1.01 and 0.97 us a step, 60
// x 128 1.37 and 1.39, 150 x 300 1.68 and 1.57, 1600 x 1600 12.9 and 12.2.
Tile2Plan make_tile2_plan(const GeomDev& g, int cus) {
    constexpr double kLaunch = 4.5, kStep = 0.3, kRow = 0.0186;  // microseconds
    constexpr double kBytes = 5e6;                               // bytes per microsecond
    const bool per0 = g.bc_lo[0] == LBW_BC_PERIODIC, per1 = g.bc_lo[1] == LBW_BC_PERIODIC;
    Tile2Plan best{};
    double best_cost = 1e30;
    for (int rows : {2, 3, 4, 8})
        for (int k : {2, 3, 4, 5, 6, 7, 8, 10, 12, 1024}) {
            const bool whole0 = !per0 && g.n0 <= kLanes;
            const bool all = k == 1024;  // the whole grid in one workgroup
            if (all && !whole0) continue;
            int ntx = 1;
            while (!whole0 && kLanes > 4 * k) {
                int most = 0;  // (tile 0 has the larger share, tile 1 both halos)
                for (int i = 0; i < 3 && i < ntx; ++i) {
                    const Span s = tile_span(i, g.n0 / ntx, g.n0 % ntx, g.n0, per0, false, k);
                    most = s.hi - s.lo > most ? s.hi - s.lo : most;
                }
                if (most <= kLanes) break;
                ntx += 1;
                if (ntx > g.n0) break;
            }
            if (!whole0 && (kLanes <= 4 * k || ntx > g.n0)) continue;
            for (int waves = 1; waves <= kMaxWaves; ++waves) {
                const int held = rows * waves;
                // axis 1 whole (closing into a ring of strips when periodic,
                // which takes two rows in the last one), or tiles with halos
                int nty = 1;
                if (g.n1 > held || (per1 && (g.n1 < 2 || g.n1 % rows == 1))) {
                    if (all || held <= 4 * k + 1) continue;
                    nty = (g.n1 + held - 4 * k - 2) / (held - 4 * k - 1);
                    if (nty == 1) nty = 2;
                    if (nty > g.n1) continue;
                }
                const int64_t groups = (int64_t)ntx * nty;
                if (nty > 65535) continue;  // grid limit
                const int64_t rounds = (groups + cus - 1) / cus;
                const int used = nty == 1 ? (g.n1 + rows - 1) / rows * rows : held;
                const double row = kRow * 4 * (rows + 0.5) * ((used / rows + 3) / 4);
                // (few tall strips: half the waves to hide latencies with,
                // 3.13 against 2.82 us a step at 701 x 503)
                const double step = (row > kStep ? row : kStep) * (rows == 8 && waves <= 8 && !all ? 1.1 : 1.0);
                const double bytes = 20.0 * ((double)groups * kLanes * used + (double)g.N);
                const double cost = (kLaunch + bytes / kBytes) / k + (double)rounds * step;
                if (cost < best_cost) {
                    best_cost = cost;
                    best = Tile2Plan{rows, used / rows, ntx, nty, k};
                }
            }
        }
    return best;
}

hipError_t launch_step_tile2(const GeomDev& g, const ProbeArgs& pr, const Tile2Plan& plan, int steps,
                             const float* fin, float* fout, hipStream_t st) {
    if (fin == fout && plan.ntx * plan.nty != 1) return hipErrorInvalidValue;
    if (g.dim != 2 || steps < 1 || steps > plan.k || plan.waves < 1 || plan.waves > kMaxWaves) return hipErrorInvalidValue;
    const dim3 grid((unsigned)plan.ntx, (unsigned)plan.nty), block(kLanes * plan.waves);
    bool free = false;
    for (int a = 0; a < 2; ++a) free = free || g.bc_lo[a] == LBW_BC_FREE || g.bc_hi[a] == LBW_BC_FREE;
    const auto launch = [&](auto rows) {
        constexpr int R = decltype(rows)::value;
        if (free)
            hipLaunchKernelGGL((step_tile2_kernel<R, true>), grid, block, 0, st, g, pr, plan, steps,
                               g.n0 / plan.ntx, g.n0 % plan.ntx, g.n1 / plan.nty, g.n1 % plan.nty, fin, fout);
        else
            hipLaunchKernelGGL((step_tile2_kernel<R, false>), grid, block, 0, st, g, pr, plan, steps,
                               g.n0 / plan.ntx, g.n0 % plan.ntx, g.n1 / plan.nty, g.n1 % plan.nty, fin, fout);
    };
    if (plan.rows == 2) launch(std::integral_constant<int, 2>{});
    else if (plan.rows == 3) launch(std::integral_constant<int, 3>{});
    else if (plan.rows == 4) launch(std::integral_constant<int, 4>{});
    else if (plan.rows == 8) launch(std::integral_constant<int, 8>{});
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace lbw
