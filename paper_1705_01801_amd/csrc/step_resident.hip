// Many steps per launch for batches of small D3Q7 geometries: one workgroup
// holds a whole geometry on chip.
//
// A geometry of some ten thousand nodes fits one CU (28 bytes of populations
// a node, 512 KB of registers), and nothing but its own workgroup ever needs
// its state.  So a workgroup loads a geometry once, takes up to
// kResidentSteps steps, and stores it once; the one-step kernel reads and
// writes every population on every step and pays a launch for it.
//  - A thread owns R (or R - 1) consecutive planes of one (axis 0, axis 1)
//    column: its populations stay in registers, those that move along axis 2
//    pass from node to node without leaving them, and only the two ends of a
//    thread's run go through LDS.
//  - The runs are walked plane by plane, all threads together, with one
//    barrier a plane: S of the next plane and the four populations that leave
//    the present one along axes 0 and 1 go into LDS on one side of it and are
//    read by the neighbours on the other (two buffers each).
//  - Walls need no selection in the loop: a link across a wall reads the
//    node's own slot, the table of coefficients carries a border whose records
//    are the node's own (negated for a fixed wall, where the mirrored S is),
//    and what a wall returns is an own slot times 1, damp or -1.
//  - Per node the arithmetic is collide() of march_common.h, so the results
//    are the same bits as those of single steps.
//  - Driven nodes: at most one per thread; the sines of all steps are taken
//    before the first.  Probes are added up in double as they pass, kept in
//    LDS and written with the state.
//  - The coefficients sit in LDS as six planes of floats.  Lanes of a wave
//    that share a column along axis 1 read the same record, and the LDS serves
//    equal addresses in one pass only for reads of 4 bytes: with 8-byte reads
//    of the same table a step took 19.6 us, with these 7.0.
// 119 driven pipes of 20 x 5 x 100: 7.5 us per step against 20.8 (tuned) with
// a launch per step, whose 67 MB a step pass through the caches; 476 of them
// 15.4 against 75.  What bounds it is the one CU that a geometry has: half
// of the time its vector units (43 instructions per plane and wave), most of
// it its LDS (16).  768 threads with up to 16 planes each hold more than 1024
// with 10, whose registers do not suffice (128 a thread).  Up to 12 planes fit
// the 168 registers that 768 threads leave a lane; from 13 on part of the state is
// in scratch, 8 to 52 bytes a lane at 13 and 14 planes, 52 and 92 (axis 1 walled)
// at 15, 96 and 116 at 16, which still pays: walled pipes of 15 and 16 planes take
// 7.1 and 7.6 us per step against 20.7 and 21.7.
#include "march_common.h"

namespace lbw {
namespace {

using namespace march;

constexpr int kThreads = 768;
constexpr int kRecords = 2816;  // of the table with its border
constexpr int kProbeSlots = 32, kDriven = 32;

struct Lds {
    float X[2][4][kThreads];  // populations leaving along +0, -0, +1, -1
    float S[2][kThreads];
    float E[4 * kThreads + 1];    // S of a run's first and last node, f*_6 leaving its bottom, f*_5 its top
    float tab[6 * kRecords];  // planes c2M00, c2M02, c2M22, c2M11, c2G0/2, c2G2/2
    double rec[kResidentSteps][kProbeSlots];
    double sine[kResidentSteps][kDriven];
    BatchSource src[kDriven];
    uint32_t mask[kThreads];  // probe nodes of a thread's run (bit: plane of the run)
    int base[kThreads];       // slot of the first of them
    int probes, driven;
};

// A value the compiler takes as new: what is derived from it in the unrolled
// planes is not computed before the loop over steps and held there (one
// register a plane each).
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// what a wall returns, as a slot of X and a factor: `same` / `opp` are the
// populations that enter from it and leave towards it
__device__ __forceinline__ void wall_slot(int wall, float damp, int same, int opp, int tid, int& slot, float& fac) {
    slot = (wall == LBW_BC_FREE ? same : opp) * kThreads + tid;
    fac = wall == LBW_BC_BOUNCEBACK ? damp : wall == LBW_BC_FREE ? 1.f : -1.f;
}

template <int R, bool PERY>
__global__ __launch_bounds__(kThreads) void resident_kernel(const BatchItem* __restrict__ items, int n_items,
                                                            BatchProbeArgs bp, int steps, const float* fin,
                                                            float* fout) {
    __shared__ Lds L;
    const int h = blockIdx.x, tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const BatchItem& it = items[h];
    const int n0 = it.n0, n1 = it.n1, n2 = it.n2, C = n0 * n1;
    const uint32_t N = it.N;
    const float c2 = it.c2, two_w0 = it.two_w0, damp = it.damp;
    const int64_t t = bp.tcount[(size_t)bp.parity * n_items + h];
    // runs: `full` of R planes, the others of R - 1
    const int G = (n2 + R - 1) / R, full = n2 - G * (R - 1);
    const int g = tid / C, c = tid - g * C;
    const bool on = g < G;
    const bool whole = g < full;  // (a run of R planes)
    const int z0 = on ? g * (R - 1) + min(g, full) : 0;
    const int y = c / n0, x = c - y * n0;

    // ---- table with its border: planes -1 .. n2, columns -1 .. n0 ----
    const int pitch = n0 + 2;
    const float4* tab4 = bp.tab4 + 2 * (size_t)it.tab_off;
    for (int i = tid; i < pitch * (n2 + 2); i += nt) {
        const int pz = i / pitch - 1, px = i - (pz + 1) * pitch - 1;
        int qx = px, qz = pz;
        float s0 = 1.f, s2 = 1.f;
        if (px < 0 || px >= n0) {
            const int wall = px < 0 ? it.bc_lo[0] : it.bc_hi[0];
            qx = wall == LBW_BC_PERIODIC ? (px < 0 ? n0 - 1 : 0) : (px < 0 ? 0 : n0 - 1);
            if (wall == LBW_BC_FIXED) s0 = -1.f;
        }
        if (pz < 0 || pz >= n2) {
            const int wall = pz < 0 ? it.bc_lo[2] : it.bc_hi[2];
            qz = wall == LBW_BC_PERIODIC ? (pz < 0 ? n2 - 1 : 0) : (pz < 0 ? 0 : n2 - 1);
            if (wall == LBW_BC_FIXED) s2 = -1.f;
        }
        const size_t e = (size_t)(qx + n0 * qz);
        const float4 lo = tab4[2 * e], hi = tab4[2 * e + 1];
        float* w = &L.tab[i];
        w[0] = s0 * lo.x;
        w[kRecords] = s0 * s2 * lo.y;
        w[2 * kRecords] = s2 * lo.z;
        w[3 * kRecords] = lo.w;
        w[4 * kRecords] = hi.x;
        w[5 * kRecords] = hi.y;
    }

    // ---- slots of the neighbours ----
    int nx_p, nx_m, ny_p, ny_m, ix1, ix2, ix3, ix4, ez_m, ez_p;
    float fc1 = 1.f, fc2 = 1.f, fc3 = 1.f, fc4 = 1.f, f5 = 1.f, f6 = 1.f, sy_p = 1.f, sy_m = 1.f;
    bool own5 = false, own6 = false;  // the run's end stores what a free wall returns
    {
        int wall = 0;
        int j = link_coord(x, +1, n0, it.bc_lo[0], it.bc_hi[0], &wall);
        nx_p = on && j >= 0 ? tid + j - x : tid;
        ix2 = kThreads + nx_p;
        if (j < 0) wall_slot(wall, damp, 1, 0, tid, ix2, fc2);
        j = link_coord(x, -1, n0, it.bc_lo[0], it.bc_hi[0], &wall);
        nx_m = on && j >= 0 ? tid + j - x : tid;
        ix1 = nx_m;
        if (j < 0) wall_slot(wall, damp, 0, 1, tid, ix1, fc1);
        j = link_coord(y, +1, n1, it.bc_lo[1], it.bc_hi[1], &wall);
        ny_p = on && j >= 0 ? tid + (j - y) * n0 : tid;
        ix4 = 3 * kThreads + ny_p;
        if (j < 0) {
            wall_slot(wall, damp, 3, 2, tid, ix4, fc4);
            if (wall == LBW_BC_FIXED) sy_p = -1.f;
        }
        j = link_coord(y, -1, n1, it.bc_lo[1], it.bc_hi[1], &wall);
        ny_m = on && j >= 0 ? tid + (j - y) * n0 : tid;
        ix3 = 2 * kThreads + ny_m;
        if (j < 0) {
            wall_slot(wall, damp, 2, 3, tid, ix3, fc3);
            if (wall == LBW_BC_FIXED) sy_m = -1.f;
        }
        if constexpr (PERY) {  // every link of axis 1 is there
            ix3 = 2 * kThreads + ny_m;
            ix4 = 3 * kThreads + ny_p;
        }
        // along axis 2, between runs: S of the run's end beyond (E[0], E[1]),
        // and 2 kThreads further what arrives from there
        const bool perz = it.bc_lo[2] == LBW_BC_PERIODIC;
        ez_m = tid;
        ez_p = kThreads + tid;
        if (on) {
            if (g > 0 || perz) {
                ez_m = kThreads + (g > 0 ? tid - C : tid + (G - 1) * C);
            } else {
                own5 = it.bc_lo[2] == LBW_BC_FREE;
                f5 = it.bc_lo[2] == LBW_BC_BOUNCEBACK ? damp : own5 ? 1.f : -1.f;
            }
            if (g < G - 1 || perz) {
                ez_p = g < G - 1 ? tid + C : c;
            } else {
                own6 = it.bc_hi[2] == LBW_BC_FREE;
                f6 = it.bc_hi[2] == LBW_BC_BOUNCEBACK ? damp : own6 ? 1.f : -1.f;
            }
        }
    }
    L.mask[tid] = 0;
    if (tid == 0) L.probes = L.driven = 0;
    __syncthreads();

    // ---- state, probes, driven nodes ----
    float f[R][7];
    {
        const __amdgpu_buffer_rsrc_t rin = make_rsrc(fin + it.f_off, 28u * N);
#pragma unroll
        for (int j = 0; j < R; ++j)
            bload7(rin, 4u * N, on && (j < R - 1 || whole), 4u * (uint32_t)(c + C * (z0 + j)), f[j]);
    }
    const bool record = bp.t_max > 0;
    const auto place = [&](uint32_t node, int& j) {  // thread and plane of its run that hold a node
        const int pz = (int)(node / (uint32_t)C), pc = (int)node - pz * C;
        const int pg = pz < full * R ? pz / R : full + (pz - full * R) / max(R - 1, 1);
        j = pz - (pg * (R - 1) + min(pg, full));
        return pg * C + pc;
    };
    for (int p = tid; record && p < it.n_probes; p += nt) {
        int j;
        const int who = place((uint32_t)bp.nodes[it.probe_off + p], j);
        atomicOr(&L.mask[who], 1u << j);
    }
    int dj = -1, dslot = 0;
    if (bp.src && it.src_count > 0) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int z = z0 + j;
            if (on && (j < R - 1 || whole) && z >= it.src_zlo && z <= it.src_zhi) {
                const int hit = bp.src_map[it.src_map + (uint32_t)((z - it.src_zlo) * C + c)];
                if (hit >= 0) {
                    dj = j;
                    dslot = min(atomicAdd(&L.driven, 1), kDriven - 1);
                    L.src[dslot] = bp.src[hit];
                }
            }
        }
    }
    __syncthreads();
    const uint32_t mask = L.mask[tid];
    int slot0 = 0;
    if (mask) {
        slot0 = atomicAdd(&L.probes, __popc(mask));
        L.base[tid] = slot0;
    }
    {
        const int D = min(L.driven, kDriven);
        for (int i = tid; i < D * steps; i += nt) {
            const int d = i % D, s = i / D;
            L.sine[s][d] = sin(L.src[d].omega * (double)(t + s));
        }
    }
    // (uniform) planes of the runs at which the wave's lanes hold probes or
    // driven nodes
    uint32_t wave_probes = 0, wave_driven = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (__builtin_amdgcn_ballot_w64((mask >> j) & 1u)) wave_probes |= 1u << j;
        if (__builtin_amdgcn_ballot_w64(dj == j)) wave_driven |= 1u << j;
    }
    __syncthreads();

    Links k{};  // every link present: walls are in the slots and the table
    int tab0 = ((on ? z0 + 1 : 1) * pitch + x + 1);
    float* const X = &L.X[0][0][0];
    float* const E = &L.E[0];
    for (int s = 0; s < steps; ++s) {
        if (wave_driven) {
            const int dj_s = opaque(dj);
#pragma unroll
            for (int j = 0; j < R; ++j)
                if ((wave_driven >> j) & 1u) {
                    if (dj_s == j) {
                        const BatchSource& e = L.src[dslot];
                        drive_value<7>(e.kind, e.a0, e.a1, L.sine[s][dslot], f[j]);
                    }
                }
        }
        if (wave_probes) {
            const uint32_t m = (uint32_t)opaque((int)mask);
#pragma unroll
            for (int j = 0; j < R; ++j)
                if ((wave_probes >> j) & 1u) {
                    const int slot = slot0 + __popc(m & ((1u << j) - 1u));
                    if (((m >> j) & 1u) && slot < kProbeSlots) {
                        double sum = 0.0;
#pragma unroll
                        for (int l = 0; l < 7; ++l) sum += (double)f[j][l];
                        L.rec[s][slot] = sum;
                    }
                }
        }
        float S = sum7(f[0]), Sm, Send;
        E[tid] = S;
        {
            const float a = sum7(f[R - 1]), b = sum7(f[R - 2]);
            E[kThreads + tid] = whole ? a : b;
        }
        L.S[0][tid] = S;
        int at = opaque(tab0);
        const float* tp = &L.tab[at];
        float2 ea = make_float2(tp[0], tp[kRecords]), eb = make_float2(tp[2 * kRecords], tp[3 * kRecords]);
        float em02 = (tp - pitch)[kRecords], em22 = (tp - pitch)[2 * kRecords];
        float up = 0.f;  // f*_5 of the plane below
        __syncthreads();
        Sm = E[ez_m];
        Send = E[ez_p];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float* Ls = L.S[j & 1];
            if (j > 0) {
                __syncthreads();
                // populations that reached plane j - 1 along axes 0 and 1
                const float* Xj = X + ((j - 1) & 1) * 4 * kThreads;
                f[j - 1][1] = fc1 * Xj[ix1];
                f[j - 1][2] = fc2 * Xj[ix2];
                f[j - 1][3] = PERY ? Xj[ix3] : fc3 * Xj[ix3];
                f[j - 1][4] = PERY ? Xj[ix4] : fc4 * Xj[ix4];
            }
            float Sp;
            if (j == R - 1) {
                Sp = Send;
            } else {
                Sp = sum7(f[j + 1]);
                if (j == R - 2) Sp = whole ? Sp : Send;
                L.S[(j + 1) & 1][tid] = Sp;
            }
            const float2 ec = make_float2(tp[4 * kRecords], tp[5 * kRecords]), xp = make_float2(tp[1], tp[kRecords + 1]), xm = make_float2(tp[-1], tp[kRecords - 1]);
            at = opaque(at + pitch);
            tp = &L.tab[at];
            // (the plane above a run of R - 1 planes at j = R - 1 is not used)
            const float2 na = make_float2(tp[0], tp[kRecords]), nb = make_float2(tp[2 * kRecords], tp[3 * kRecords]);
            const float Syp = PERY ? Ls[ny_p] : sy_p * Ls[ny_p], Sym = PERY ? Ls[ny_m] : sy_m * Ls[ny_m];
            float fs[7];
            collide(f[j], S, make_float4(ea.x, ea.y, eb.x, eb.y), make_float4(ec.x, ec.y, 0.f, 0.f),
                    make_float4(xp.x, xp.y, 0.f, 0.f), make_float4(xm.x, xm.y, 0.f, 0.f),
                    make_float4(0.f, na.y, nb.x, 0.f), make_float2(em02, em22), Ls[nx_p], Ls[nx_m], Syp, Sym, Sp, Sm,
                    k, c2, two_w0, fs);
            float* Xw = X + (j & 1) * 4 * kThreads + tid;
            Xw[0] = fs[1];
            Xw[kThreads] = fs[2];
            Xw[2 * kThreads] = fs[3];
            Xw[3 * kThreads] = fs[4];
            f[j][0] = fs[0];
            if (j == 0) E[2 * kThreads + tid] = own5 ? fs[5] : fs[6];
            else f[j][5] = up;
            if (j > 0) f[j - 1][6] = j < R - 1 || whole ? fs[6] : f[j - 1][6];
            // (no branch: the compiler would move arithmetic of all planes past it)
            if (j == R - 2) E[3 * kThreads + tid] = own6 ? fs[6] : fs[5];
            if (j == R - 1) E[whole ? 3 * kThreads + tid : 4 * kThreads] = own6 ? fs[6] : fs[5];
            up = fs[5];
            em02 = ea.y;
            em22 = eb.x;
            ea = na;
            eb = nb;
            Sm = S;
            S = Sp;
        }
        __syncthreads();
        const float* Xj = X + ((R - 1) & 1) * 4 * kThreads;
        f[R - 1][1] = fc1 * Xj[ix1];
        f[R - 1][2] = fc2 * Xj[ix2];
        f[R - 1][3] = PERY ? Xj[ix3] : fc3 * Xj[ix3];
        f[R - 1][4] = PERY ? Xj[ix4] : fc4 * Xj[ix4];
        f[0][5] = f5 * E[ez_m + 2 * kThreads];
        const float top = f6 * E[ez_p + 2 * kThreads];
        f[R - 1][6] = top;
        f[R - 2][6] = whole ? f[R - 2][6] : top;
    }

    // ---- results ----
    {
        const uint32_t first = (uint32_t)opaque(4 * (c + C * z0));
        const __amdgpu_buffer_rsrc_t rout = make_rsrc(fout + it.f_off, 28u * N);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint32_t at = on && (j < R - 1 || whole) ? first + 4u * (uint32_t)(C * j) : kOff;
#pragma unroll
            for (int l = 0; l < 7; ++l) bst(rout, at + (uint32_t)l * (4u * N), f[j][l]);
        }
    }
    for (int i = tid; record && i < it.n_probes * steps; i += nt) {
        const int s = i / it.n_probes, p = i - s * it.n_probes;
        const uint32_t node = (uint32_t)bp.nodes[it.probe_off + p];
        int j;
        const int who = place(node, j);
        const int slot = L.base[who] + __popc(L.mask[who] & ((1u << j) - 1u));
        if (t + s >= 0 && t + s < bp.t_max && slot < kProbeSlots)
            bp.trace[(t + s) * bp.stride + it.probe_off + p] =
                L.rec[s][slot] / bp.sqrtg[it.sg_off + node % (uint32_t)n0 + (uint32_t)n0 * (node / (uint32_t)C)];
    }
    // (this block alone reads and writes the geometry's counters)
    if (tid == 0) bp.tcount[(size_t)((bp.parity + steps) & 1) * n_items + h] = t + steps;
}

template <int R>
void launch_of(bool pery, int n_items, int threads, const BatchItem* items, const BatchProbeArgs& bp, int steps,
               const float* fin, float* fout, hipStream_t st) {
    if (pery)
        hipLaunchKernelGGL((resident_kernel<R, true>), dim3(n_items), dim3(threads), 0, st, items, n_items, bp, steps,
                           fin, fout);
    else
        hipLaunchKernelGGL((resident_kernel<R, false>), dim3(n_items), dim3(threads), 0, st, items, n_items, bp,
                           steps, fin, fout);
}

}  // namespace

bool resident_fits(int n0, int n1, int n2, int n_probes, int run, int* threads) {
    const int64_t C = (int64_t)n0 * n1;
    const int64_t G = ((int64_t)n2 + run - 1) / run;
    if (run < 2 || run > kResidentRun || C * G > kThreads || n2 < G * (run - 1) || n_probes > kProbeSlots) return false;
    if ((int64_t)(n0 + 2) * (n2 + 2) + 2 * (n0 + 2) > kRecords) return false;
    *threads = (int)((C * G + 63) / 64 * 64);
    return true;
}

int resident_slot(int n0, int n1, int n2, int run, int64_t node) {
    const int64_t C = (int64_t)n0 * n1, z = node / C, G = ((int64_t)n2 + run - 1) / run, full = n2 - G * (run - 1);
    const int64_t g = z < full * run ? z / run : full + (z - full * run) / (run - 1);
    return (int)(g * C + node % C);
}

int resident_driven() { return kDriven; }

hipError_t launch_step_resident(const BatchItem* items, int n_items, int run, int threads, bool pery,
                                const BatchProbeArgs& bp, int steps, const float* fin, float* fout, hipStream_t st) {
    if (steps < 1 || steps > kResidentSteps || threads < 64 || threads > kThreads) return hipErrorInvalidValue;
    switch (run) {
        case 2: launch_of<2>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 3: launch_of<3>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 4: launch_of<4>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 5: launch_of<5>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 6: launch_of<6>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 7: launch_of<7>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 8: launch_of<8>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 9: launch_of<9>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 10: launch_of<10>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 11: launch_of<11>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 12: launch_of<12>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 13: launch_of<13>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 14: launch_of<14>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 15: launch_of<15>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        case 16: launch_of<16>(pery, n_items, threads, items, bp, steps, fin, fout, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace lbw
