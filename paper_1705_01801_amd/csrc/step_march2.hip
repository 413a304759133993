// Two time steps per pass of the D3Q7 z-march (temporal blocking).
//
// The one-step kernels read every population once and write it once per
// step, 56 bytes per node update, and on grids that do not fit the caches
// that is the whole cost.  This kernel advances a tile from t to t+2 in one
// pass over memory, so the populations are read and written once per two
// updates:
//  - a workgroup of TX x (TY + 2) threads owns TY whole axis-0 rows (the
//    grid's walled axis 0 fits one row of TX lanes) over a chunk of planes
//    along axis 2;
//  - step A (t -> t+1) runs plane by plane on the tile and one halo row on
//    either side (TY + 2 rows), with the one-step kernel's data movement:
//    the own column's populations of planes z and z+1 in registers (plane
//    z+2 in flight), S of the plane staged in LDS for the axis-0 and axis-1
//    neighbours.  Its post-collision populations are not stored: along
//    axis 2 they stay in the thread that owns the column (a register carries
//    the +e2 one to the next plane, the -e2 one completes the plane below),
//    along axes 0 and 1 they are handed over through LDS.  The two rows
//    beyond the halo rows send one population each into them (+e1 into the
//    lower halo row, -e1 into the upper one); the first 2 TX threads load
//    those rows and run their collision too, the next 2 TX load the rows
//    beyond them for S only;
//  - a plane's state at t+1 is complete once step A has passed the plane
//    above it, and step B (t+1 -> t+2) also needs S(t+1) of the plane
//    above, so step B runs two planes behind step A, on the tile's own rows,
//    and pushes its populations to memory as the one-step kernel does;
//  - per node both steps call collide() of march_common.h in the same
//    order as a one-step launch would, so the result is that of two single
//    steps, bit for bit;
//  - probes: block 0 records time t from the input; the thread that owns a
//    probe node records time t+1 from the state it assembled.
// What bounds it: on a 96 x 256 x 512 torus a launch moves 1135 MB in 203 us
// (45.1 bytes per update; 28 if nothing were read twice), 5.6 TB/s, more than a
// copy of the same bytes reaches, while a plane (about 4900 cycles for 12 waves)
// keeps the vector unit busy 28 % and the LDS 23 % of its time.  The extra bytes
// are the price of equal shares, whose neighbours do not march in step: whole
// chunks move 31 bytes per update, but the best of them (103 planes) takes 107 us
// per step against 100.
// Offsets in memory are a lane constant plus a uniform part, and the walls of
// axis 0 lane constants: 112 vector instructions per plane and wave instead of
// 178, 100 us per step instead of 104.  Loads of the own column and the ring two
// planes ahead did not fit the registers (spills, 110 us); as built the variants
// take 137 to 150 of the 168 that three waves per SIMD have, and spill 70 to 114
// scalar registers to lanes (the batch's: 165 to 167, and 34 to 49).
// Chunks along axis 2 are extended by two planes of step A either side (the
// state at t+1 of planes z0-1 and z1 is needed), which is the price of the
// chunking besides the two halo rows.
#include "march_common.h"

namespace lbw {
namespace {

using namespace march;

constexpr int kTileProbes = 16;

// RT: the tile is run-time, whole rows of n0 <= TX columns, as many as fit the
// threads; TX x TY then only sizes the LDS arrays (kRtSlots bounds the padded
// tile, checked by the host).
constexpr int kRtSlots = 1400;
template <int TX, int TY, bool RT = false>
struct M2 {
    static constexpr int NT = TX * (TY + 2);
    static constexpr int W = TX + 2;          // LDS row: one pad entry either side of the axis-0 row
    static constexpr int S = RT ? kRtSlots : (TY + 6) * W;   // S(t) of extended rows -2 .. TY+3
    static constexpr int X = RT ? kRtSlots : (TY + 4) * W;   // populations handed over by rows -1 .. TY+2
    static constexpr int S1 = RT ? kRtSlots : (TY + 4) * W;  // S(t+1) of rows -1 .. TY+2 (the outer two unused)
    static constexpr int B = RT ? NT : TY * TX;
};

template <int TX, int TY, bool RT = false>
struct M2Lds {
    using C = M2<TX, TY, RT>;
    float S[2][C::S + 1];      // + a sink slot
    float X[4][C::X + 1];      // (the last slot takes what nobody reads)
    float S1[2][C::S1 + 1];
    // coefficient rows, slot = (plane - za0) mod 6: c^2 Mhat00, 02, 22, 11,
    // c^2 Gamh0 / 2, c^2 Gamh2 / 2, an array each (96 x 256 x 512 torus: 104 us
    // per step; with records of 16 bytes, whose ten reads per plane and wave
    // were most of the LDS's time, 120)
    float E[6][6 * C::W + 1];  // + a sink slot
    float B[2][2][C::B + 1];   // step B: +-e0 populations along the row (2 planes)
    int pnode[kTileProbes], px[kTileProbes], py[kTileProbes], pz[kTileProbes];
    int pcount;
};

__device__ inline int wrap(int i, int n) { return ((i % n) + n) % n; }

// The lane's link indices along axis 1 passed through an empty asm statement
// once per plane: the compiler then derives the lane masks it selects with
// where they are used, instead of keeping them all in scalar registers for the
// whole march (more than the scalar file holds: the rest would be spilled to
// vector lanes and read back twice per use).
__device__ __forceinline__ void opaque_jy(Links& k) { asm volatile("" : "+v"(k.jy_p), "+v"(k.jy_m)); }

// Loads and stores with a lane part (kOff in disabled lanes) and a uniform
// part of the offset: a plane's address costs the vector unit nothing.  The
// uniform part is below 7 N4 < 2^31, so a disabled lane's sum stays out of
// range and does not wrap.
__device__ __forceinline__ float bldu(__amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t uni) {
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)lane, (int)uni, 0));
}
__device__ __forceinline__ void bstu(__amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t uni, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, (int)lane, (int)uni, 0);
}
__device__ __forceinline__ void bload7u(__amdgpu_buffer_rsrc_t r, uint32_t N4, uint32_t lane, uint32_t uni,
                                        float v[7]) {
#pragma unroll
    for (int l = 0; l < 7; ++l) v[l] = bldu(r, lane, uni + (uint32_t)l * N4);
}

// PERY, PERZ: axis 1, axis 2 is periodic (every link along it present;
// the wall rules of that axis are compiled out).
// rows: the tile's rows (RT; else TY); stride: the trace's row length.
template <int TX, int TY, bool PERY, bool PERZ, bool RT = false>
__device__ __forceinline__ void march2_tile(const GeomDev& g, const ProbeArgs& pr, int64_t stride, int64_t t, int ty,
                                            int rows, int z0, int z1, const float* __restrict__ fin,
                                            float* __restrict__ fout, M2Lds<TX, TY, RT>& L) {
    using C = M2<TX, TY, RT>;
    const int TXr = RT ? g.n0 : TX, TYr = RT ? rows : TY;
    const int W = TXr + 2;
    const int n0 = g.n0, n1 = g.n1, n2 = g.n2;
    const uint32_t N = (uint32_t)g.N;
    const uint32_t plane = (uint32_t)n0 * (uint32_t)n1;
    const float c2 = g.c2, two_w0 = g.two_w0, damp = g.damp;
    const int lx = (int)(threadIdx.x % (unsigned)TXr), ly = (int)(threadIdx.x / (unsigned)TXr);
    // row tile ty (rows ty TYr ..), planes [z0, z1) with 0 <= z0 < z1 <= n2
    const int y0 = ty * TYr;
    const int hgt = min(TYr, n1 - y0);
    const bool perz = g.bc_lo[2] == LBW_BC_PERIODIC;
    const bool pery = PERY || (RT && g.bc_lo[1] == LBW_BC_PERIODIC);  // (a batch may mix both)
    // step A runs on march planes [za0, za1); the march runs on [za0, z1 + 2)
    const int za0 = perz ? z0 - 2 : max(z0 - 2, 0);
    const int za1 = perz ? z1 + 2 : min(z1 + 2, n2);

    // this thread's node: x = lx on the row of extended row ly (tile row ly - 1)
    const int yr = y0 - 1 + ly;
    const bool ypres = pery || (yr >= 0 && yr < n1);
    const int ya = pery ? wrap(yr, n1) : yr;
    const bool idle = RT && ly > TYr + 1;  // (threads beyond the halo rows)
    const bool actA = lx < n0 && ypres && !idle;
    const bool actB = actA && ly >= 1 && ly <= hgt;
    // waves with no lane on the tile's own rows (all in the halo rows) skip
    // step B altogether (it has no barrier; its hand-over slots are read
    // only by lanes of the same row, which are on the tile's rows)
    const bool waveB = __builtin_amdgcn_ballot_w64(actB) != 0;
    Links kl{};
    kl.jx_p = link_coord(lx, +1, n0, g.bc_lo[0], g.bc_hi[0], &kl.wx_p);
    kl.jx_m = link_coord(lx, -1, n0, g.bc_lo[0], g.bc_hi[0], &kl.wx_m);
    kl.jy_p = ypres ? link_coord(ya, +1, n1, g.bc_lo[1], g.bc_hi[1], &kl.wy_p) : -1;
    kl.jy_m = ypres ? link_coord(ya, -1, n1, g.bc_lo[1], g.bc_hi[1], &kl.wy_m) : -1;
    const uint32_t col4 = actA ? ((uint32_t)lx + (uint32_t)n0 * (uint32_t)ya) * 4u : 0u;
    const int bcy_lo = g.bc_lo[1], bcy_hi = g.bc_hi[1];
    // byte offsets to the axis-1 neighbours' columns (used where the link exists)
    const uint32_t dyp4 = (uint32_t)((kl.jy_p - ya) * n0) * 4u, dym4 = (uint32_t)((kl.jy_m - ya) * n0) * 4u;

    // ring loader: rows -1 and TY+2 (loaded and collided: they send +e1 / -e1
    // into the halo rows), rows -2 and TY+3 (loaded for S only)
    const int rid = ly;  // 0..3 for loaders
    const int re = rid == 0 ? -1 : rid == 1 ? TYr + 2 : rid == 2 ? -2 : TYr + 3;
    const int ryr = y0 - 1 + re;
    const bool rpres = rid < 4 && (pery || (ryr >= 0 && ryr < n1));
    const int rya = pery ? wrap(ryr, n1) : ryr;
    const bool ring_on = rpres && lx < n0;
    const bool ring_col = ring_on && rid < 2;  // collides its ring node
    Links kr{};
    kr.jy_p = rpres ? link_coord(rya, +1, n1, g.bc_lo[1], g.bc_hi[1], &kr.wy_p) : -1;
    kr.jy_m = rpres ? link_coord(rya, -1, n1, g.bc_lo[1], g.bc_hi[1], &kr.wy_m) : -1;
    const uint32_t ring4 = ring_on ? ((uint32_t)lx + (uint32_t)n0 * (uint32_t)rya) * 4u : 0u;
    const int my_s = (ly + 2) * W + lx + 1;                  // own S(t) slot
    const int ring_s = ring_on ? (re + 2) * W + lx + 1 : C::S;
    const int xo = my_s - W;                                 // own slot of X and S1
    const int my_w = idle ? C::S : my_s, xw = idle ? C::X : xo;  // written (idle threads: the sinks)

    // The walls of axis 0 as lane constants instead of selections per plane:
    // across a wall a lane reads its own S (negated for a fixed wall) and
    // coefficients, and what the wall returns is a slot of its own in the
    // hand-over times 1, damp or -1 (free walls: the population itself, else
    // the opposite one)
    const bool xp = kl.jx_p >= 0, xm = kl.jx_m >= 0;
    const int sxp = my_s + (xp ? 1 : 0), sxm = my_s - (xm ? 1 : 0);
    const int exo = lx + 1, exp = exo + (xp ? 1 : 0), exm = exo - (xm ? 1 : 0);
    const bool free_p = g.bc_hi[0] == LBW_BC_FREE, free_m = g.bc_lo[0] == LBW_BC_FREE;
    const float sg_p = !xp && g.bc_hi[0] == LBW_BC_FIXED ? -1.f : 1.f;
    const float sg_m = !xm && g.bc_lo[0] == LBW_BC_FIXED ? -1.f : 1.f;
    const float fac1 = xm || free_m ? 1.f : g.bc_lo[0] == LBW_BC_BOUNCEBACK ? damp : -1.f;
    const float fac2 = xp || free_p ? 1.f : g.bc_hi[0] == LBW_BC_BOUNCEBACK ? damp : -1.f;
    constexpr int XS = C::X + 1, BS = C::B + 1;
    const int ix1 = xm ? xo - 1 : free_m ? xo : XS + xo, ix2 = xp ? XS + xo + 1 : free_p ? XS + xo : xo;
    const int bo = actB ? (ly - 1) * TXr + lx : C::B;        // step B hand-over slot
    const int ib1 = !actB ? C::B : xm ? bo - 1 : free_m ? bo : BS + bo;
    const int ib2 = !actB ? C::B : xp ? BS + bo + 1 : free_p ? BS + bo : bo;

    // lane parts of the offsets in memory
    const uint32_t N4 = N * 4u, plane4 = plane * 4u;
    const uint32_t ownA = actA ? col4 : kOff, ownR = ring_on ? ring4 : kOff, ownB = actB ? col4 : kOff;
    const uint32_t to3 = !actB ? kOff : kl.jy_p >= 0 ? 3u * N4 + col4 + dyp4 : 4u * N4 + col4;
    const uint32_t to4 = !actB ? kOff : kl.jy_m >= 0 ? 4u * N4 + col4 + dym4 : 3u * N4 + col4;

    // coefficient-row loader: a row is n0 records of 8 floats, 6 of them used;
    // thread t loads and stages float t mod 6 of record t / 6
    const int erec = (int)(threadIdx.x / 6u), ecoef = (int)(threadIdx.x % 6u);
    const bool erow_on = erec < n0;
    const uint32_t erow4 = erow_on ? (uint32_t)(erec * 32 + ecoef * 4) : kOff;
    const int erow_s = erow_on ? ecoef * W + erec + 1 : 6 * C::W;

    const __amdgpu_buffer_rsrc_t rin = make_rsrc(fin, 7u * N4);
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(fout, 7u * N4);
    const __amdgpu_buffer_rsrc_t rtab = make_rsrc(g.tab, (uint32_t)n0 * (uint32_t)n2 * 32u);

    // march plane -> real plane (-1 beyond a wall); in the plane loop the
    // real planes of z - 2, z, z + 2 and z + 3 are carried along and
    // advanced by one plane each (radv: one compare and select, no division)
    auto rplane = [&](int z) -> int { return perz ? wrap(z, n2) : (z >= 0 && z < n2 ? z : -1); };
    // r: real plane of march plane zn - 1; returns that of zn
    auto radv = [&](int r, int zn) -> int {
        const int up = r + 1 == n2 ? 0 : r + 1;
        return perz ? up : (zn >= 0 && zn < n2 ? zn : -1);
    };
    // axis-2 links of real plane r (as link_coord gives them), from the two
    // ends' rules computed once
    const int bz_lo = g.bc_lo[2], bz_hi = g.bc_hi[2];
    const int jzp_end = bz_hi == LBW_BC_PERIODIC ? 0 : -1, wzp_end = bz_hi == LBW_BC_PERIODIC ? 0 : bz_hi;
    const int jzm_end = bz_lo == LBW_BC_PERIODIC ? n2 - 1 : -1, wzm_end = bz_lo == LBW_BC_PERIODIC ? 0 : bz_lo;
    auto zlinks = [&](int r, Links& k) {
        const bool up = r + 1 < n2, dn = r > 0;
        k.jz_p = up ? r + 1 : jzp_end;
        k.wz_p = up ? 0 : wzp_end;
        k.jz_m = dn ? r - 1 : jzm_end;
        k.wz_m = dn ? 0 : wzm_end;
    };
    // (a row beyond a wall is not read: any row does)
    const uint32_t erow_bytes = (uint32_t)n0 * 32u;
    auto erow_r = [&](int zr) { return bldu(rtab, erow4, (uint32_t)max(zr, 0) * erow_bytes); };
    auto elo = [&](int slot, int i) {
        const float* e = &L.E[slot][i];
        return make_float4(e[0], e[W], e[2 * W], e[3 * W]);
    };
    auto ehi = [&](int slot, int i) {
        const float* e = &L.E[slot][i];
        return make_float4(e[4 * W], e[5 * W], 0.f, 0.f);
    };

    // tile probes: those on the tile's own rows and planes record time t+1
    if (threadIdx.x == 0) L.pcount = 0;
    __syncthreads();
    if (t + 1 >= 0 && t + 1 < pr.t_max) {
        for (int p = threadIdx.x; p < pr.n; p += blockDim.x) {
            const int64_t node = pr.nodes[p];
            const int i0 = (int)(node % n0);
            const int i1 = (int)((node / n0) % n1);
            const int i2 = (int)(node / ((int64_t)n0 * n1));
            if (i1 >= y0 && i1 < y0 + hgt && i2 >= z0 && i2 < z1) {
                const int slot = atomicAdd(&L.pcount, 1);
                if (slot < kTileProbes) {
                    L.pnode[slot] = p;
                    L.px[slot] = i0;
                    L.py[slot] = i1;
                    L.pz[slot] = i2;
                }
            }
        }
    }

    __syncthreads();  // the tile's probe list complete
    const int tile_probes = __builtin_amdgcn_readfirstlane(min(L.pcount, kTileProbes));
    // the plane of the thread's probe (-1: none in its column; -2: several,
    // looked up on every plane), so that a plane costs one comparison: with the
    // list walked on every plane a batch of 96 horns with 8 probes each took 190
    // us per step instead of 173
    int probe_z = -1;
    for (int i = 0; i < tile_probes; ++i)
        if (actB && L.py[i] == ya && L.px[i] == lx) probe_z = probe_z == -1 ? L.pz[i] : -2;

    // ---- prologue: planes za0 - 1 (S only) and za0 (own column, ring,
    // staged S); coefficient rows za0 - 1 .. za0 + 1; in flight into the
    // loop: own column of plane za0 + 1, ring of plane za0 + 1, coefficient
    // row za0 + 2 ----
    float fA[7], fB[7], fC[7], rA[7], rB[7], rC[7], tmp[7];
    float Sm = 0.f, Sc = 0.f, Sp = 0.f;
    {
        const int zm = rplane(za0 - 1), zc = rplane(za0);
        bload7(rin, N4, actA && zm >= 0, col4 + (uint32_t)zm * plane4, tmp);
        bload7(rin, N4, actA && zc >= 0, col4 + (uint32_t)zc * plane4, fA);
        bload7(rin, N4, ring_on && zc >= 0, ring4 + (uint32_t)zc * plane4, rA);
        const float e0 = erow_r(rplane(za0 - 1)), e1 = erow_r(rplane(za0)), e2 = erow_r(rplane(za0 + 1));
        Sm = sum7(tmp);
        Sc = sum7(fA);
        L.E[5][erow_s] = e0;  // plane za0 - 1
        L.E[0][erow_s] = e1;
        L.E[1][erow_s] = e2;
        L.S[0][my_w] = Sc;
        L.S[0][ring_s] = sum7(rA);
    }
    {
        // plane za1 itself is loaded where it exists: S(t) of the plane above
        // the last step-A plane
        const int zn = rplane(za0 + 1);
        const bool on = za0 + 1 <= za1 && zn >= 0;
        bload7(rin, N4, actA && on, col4 + (uint32_t)zn * plane4, fB);
        bload7(rin, N4, ring_on && on, ring4 + (uint32_t)zn * plane4, rB);
    }
    // coefficient rows in flight: eA holds row za0 + 2 for the first plane;
    // each plane stages the row loaded one plane earlier and loads the next
    // into the following slot (period three, by argument order, so no
    // register holding a load in flight is ever copied)
    float eA = erow_r(rplane(za0 + 2)), eB = 0.f, eC = 0.f;
    // real planes of march planes z, z + 2, z + 3 and z - 2 (carried along)
    int zrr = rplane(za0), zr2 = rplane(za0 + 2), zr3 = rplane(za0 + 3), zrb = rplane(za0 - 2);

    // state at t+1 of planes z-2 (for step B), z-1 and z (being assembled),
    // and S(t+1) of planes z-3 .. z-1
    float fa[7], fb[7], fz[7];
#pragma unroll
    for (int l = 0; l < 7; ++l) fa[l] = fb[l] = fz[l] = 0.f;
    float carry5 = 0.f;
    float S1a = 0.f, S1b = 0.f, S1c = 0.f;  // S(t+1) of planes z-3, z-2, z-1
    // step B's +-e0 stores of the previous plane, done after the next barrier
    // (the row hand-over through LDS then needs no barrier of its own)
    bool pend = false;
    uint32_t pend_z4 = 0;  // offset of that plane
    int pend_slot = 0;     // (the loop passes it as a constant)
    auto flush_pending = [&](int slot) {
        const float* Bx = &L.B[slot][0][0];
        bstu(rout, ownB, 1u * N4 + pend_z4, fac1 * Bx[ib1]);
        bstu(rout, ownB, 2u * N4 + pend_z4, fac2 * Bx[ib2]);
    };

    const int zend = z1 + 2;
    // One march plane z: step A on z (when z < za1), completion of plane z-1,
    // step B on z-2 (when it is one of the tile's planes).  f2 receives the
    // state at t+1 of plane z, f1 holds plane z-1, f0 plane z-2; fc / fnx /
    // fnn hold the own column at time t of planes z, z+1 and (loading) z+2,
    // rc / rn / rnn the ring's; the caller rotates all of them by argument
    // order (period three), so no register is copied.
    auto march_plane = [&](float (&f0)[7], float (&f1)[7], float (&f2)[7], float (&fc)[7], float (&fnx)[7],
                           float (&fnn)[7], float (&rc)[7], float (&rn)[7], float (&rnn)[7], float& en, float& e3,
                           int z, auto kc) {
        constexpr int K = decltype(kc)::value;  // z - za0 modulo 6 (the loop runs six planes per turn)
        const int sb = K & 1;
        const bool doA = z < za1;
        const int zr = zrr;
        Links kp = kl, krp = kr;
        // (the walls of axis 0 are in the slots: every link is there.)  A wall
        // code matters only where the link is missing, and there it is that
        // end's code: every lane takes the end codes, uniform, so the wall
        // rules are tested on the scalar unit
        kp.jx_p = kp.jx_m = kp.wx_p = kp.wx_m = 0;
        if constexpr (PERY) {
            kp.jy_p = kp.jy_m = kp.wy_p = kp.wy_m = 0;
            krp.jy_p = krp.jy_m = krp.wy_p = krp.wy_m = 0;
        } else {
            kp.wy_p = krp.wy_p = bcy_hi;
            kp.wy_m = krp.wy_m = bcy_lo;
            opaque_jy(kp);
            opaque_jy(krp);
        }
        // loads consumed later: own column and ring of plane z+2 (S(t) of
        // plane z+1 comes from fnx), coefficient row z+3; beyond the last
        // plane that is needed, plane z once more (not used)
        {
            const uint32_t zq4 = (uint32_t)(z + 2 <= za1 && zr2 >= 0 ? zr2 : max(zr, 0)) * plane4;
            bload7u(rin, N4, ownA, zq4, fnn);
            bload7u(rin, N4, ownR, zq4, rnn);
        }
        e3 = erow_r(zr3);
        Sp = sum7(fnx);
        const float Srp = sum7(rn);
        __syncthreads();  // S(t) of plane z, coefficient rows up to z+2, step B's hand-over visible
        if (pend) flush_pending((K + 1) & 1);  // uniform
        pend = false;

        if (doA) {
            // (a step-A plane is always a real one: zr >= 0)
            Links k = kp;
            zlinks(zr, k);
            if constexpr (PERZ) k.jz_p = k.jz_m = 0;  // (step A uses only their presence)
            const float* Ls = L.S[sb];
            const float4 e_lo = elo(K % 6, exo), e_hi = ehi(K % 6, exo);
            const float4 enp = elo(K % 6, exp), enm = elo(K % 6, exm);
            const float4 ezp = elo((K + 1) % 6, exo);
            const float4 ezm = elo((K + 5) % 6, exo);
            float fs[7];
            collide(fc, Sc, e_lo, e_hi, enp, enm, ezp, make_float2(ezm.y, ezm.z), sg_p * Ls[sxp], sg_m * Ls[sxm],
                    Ls[my_s + W], Ls[my_s - W], Sp, Sm, k, c2, two_w0, fs);
            L.X[0][xw] = fs[1];
            L.X[1][xw] = fs[2];
            L.X[2][xw] = fs[3];
            L.X[3][xw] = fs[4];
            // the ring rows -1 and TY+2 (threads of the first 2 TX, whole
            // waves) send f*_3 (row -1, into row 0) and f*_4 (row TY+2, into
            // row TY+1): the axis-1 part of their collision
            // (where 2 TX is no multiple of 64, the last of these waves holds
            // other lanes too: row -1's slots, and the sink)
            if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) < 2 * TXr) {
                const int ri = (RT && rid > 1 ? 1 : re + 2) * W + lx + 1;
                float rs3, rs4;
                collide_axis1(rc[3], rc[4], sum7(rc), e_lo.w, Ls[ri + W], Ls[ri - W], krp, c2, rs3, rs4);
                const int ro = (re + 1) * W + lx + 1;
                // (row -1 sends f*_3 through X[2], row TY+2 f*_4 through X[3];
                // one store by index, no branch)
                (&L.X[0][0])[(rid == 0 ? 2 * XS : 3 * XS) + (ring_col ? ro : C::X)] = rid == 0 ? rs3 : rs4;
            }
            __syncthreads();  // handed-over populations visible
            f2[0] = fs[0];
            f2[1] = fac1 * (&L.X[0][0])[ix1];
            f2[2] = fac2 * (&L.X[0][0])[ix2];
            f2[3] = k.jy_m >= 0 ? L.X[2][xo - W] : bounce(k.wy_m, damp, fs[4], fs[3]);
            f2[4] = k.jy_p >= 0 ? L.X[3][xo + W] : bounce(k.wy_p, damp, fs[3], fs[4]);
            f2[5] = k.jz_m >= 0 ? carry5 : bounce(k.wz_m, damp, fs[6], fs[5]);
            f2[6] = k.jz_p >= 0 ? 0.f : bounce(k.wz_p, damp, fs[5], fs[6]);
            if (k.jz_m >= 0) f1[6] = fs[6];
            carry5 = fs[5];
        }
        // plane z-1 is complete: its S(t+1) for step B's neighbours
        if (z - 1 >= za0 && z - 1 < za1) {
            S1c = sum7(f1);
            L.S1[(K + 1) & 1][xw] = S1c;  // plane z - 1
        }

        // step B on plane zb = z - 2
        const int zb = z - 2;
        if (zb >= z0 && zb < z1 && waveB) {
            const int zbr = zrb;
            Links k = kp;
            zlinks(zbr, k);
            const int jzp = k.jz_p, jzm = k.jz_m;  // the stores' planes
            if constexpr (PERZ) k.jz_p = k.jz_m = 0;
            const float* L1 = L.S1[K & 1];  // plane z - 2
            const float4 e_lo = elo((K + 4) % 6, exo), e_hi = ehi((K + 4) % 6, exo);
            const float4 enp = elo((K + 4) % 6, exp), enm = elo((K + 4) % 6, exm);
            const float4 ezp = elo((K + 5) % 6, exo);
            const float4 ezm = elo((K + 3) % 6, exo);
            float fs[7];
            collide(f0, S1b, e_lo, e_hi, enp, enm, ezp, make_float2(ezm.y, ezm.z), sg_p * L1[sxp - W],
                    sg_m * L1[sxm - W], L1[xo + W], L1[xo - W], S1c, S1a, k, c2, two_w0, fs);
            // probes at t+1 on this plane (the state f0 before step B)
            const bool probed = probe_z == zbr || probe_z == -2;
            if (__builtin_amdgcn_ballot_w64(probed) != 0) {
                for (int i = 0; i < tile_probes; ++i) {
                    if (probed && L.pz[i] == zbr && L.py[i] == ya && L.px[i] == lx) {
                        double s = 0.0;
                        for (int l = 0; l < 7; ++l) s += (double)f0[l];
                        pr.trace[(t + 1) * stride + L.pnode[i]] = s / g.sqrtg[lx + (int64_t)n0 * zbr];
                    }
                }
            }
            // push: +-e0 along the row through LDS, stored after the next
            // barrier (aligned stores); the rest to their destinations (or the
            // wall rules) now
            pend_slot = K & 1;
            L.B[K & 1][0][bo] = fs[1];
            L.B[K & 1][1][bo] = fs[2];
            const uint32_t z4 = (uint32_t)zbr * plane4;
            pend = true;
            pend_z4 = z4;
            const uint32_t u5 = jzp >= 0 ? 5u * N4 + (uint32_t)jzp * plane4 : 6u * N4 + z4;
            const uint32_t u6 = jzm >= 0 ? 6u * N4 + (uint32_t)jzm * plane4 : 5u * N4 + z4;
            const float v3 = k.jy_p >= 0 ? fs[3] : bounce(k.wy_p, damp, fs[3], fs[4]);
            const float v4 = k.jy_m >= 0 ? fs[4] : bounce(k.wy_m, damp, fs[4], fs[3]);
            const float v5 = k.jz_p >= 0 ? fs[5] : bounce(k.wz_p, damp, fs[5], fs[6]);
            const float v6 = k.jz_m >= 0 ? fs[6] : bounce(k.wz_m, damp, fs[6], fs[5]);
            bstu(rout, ownB, z4, fs[0]);
            bstu(rout, to3, z4, v3);
            bstu(rout, to4, z4, v4);
            bstu(rout, ownB, u5, v5);
            bstu(rout, ownB, u6, v6);
        }
        S1a = S1b;
        S1b = S1c;

        // stage S(t) of plane z+1 and the coefficient row z+2 for the next
        // march plane (their slots were last read two barriers ago)
        if (z + 1 < zend) {
            L.S[sb ^ 1][my_w] = Sp;
            L.S[sb ^ 1][ring_s] = Srp;
            L.E[(K + 2) % 6][erow_s] = en;
        }
        Sm = Sc;
        Sc = Sp;
        zrr = radv(zr, z + 1);
        zr2 = radv(zr2, z + 3);
        zr3 = radv(zr3, z + 4);
        zrb = radv(zrb, z - 1);
    };
    for (int z = za0;;) {
        if (z >= zend) break;
        march_plane(fa, fb, fz, fA, fB, fC, rA, rB, rC, eA, eB, z, std::integral_constant<int, 0>{});
        if (++z >= zend) break;
        march_plane(fb, fz, fa, fB, fC, fA, rB, rC, rA, eB, eC, z, std::integral_constant<int, 1>{});
        if (++z >= zend) break;
        march_plane(fz, fa, fb, fC, fA, fB, rC, rA, rB, eC, eA, z, std::integral_constant<int, 2>{});
        if (++z >= zend) break;
        march_plane(fa, fb, fz, fA, fB, fC, rA, rB, rC, eA, eB, z, std::integral_constant<int, 3>{});
        if (++z >= zend) break;
        march_plane(fb, fz, fa, fB, fC, fA, rB, rC, rA, eB, eC, z, std::integral_constant<int, 4>{});
        if (++z >= zend) break;
        march_plane(fz, fa, fb, fC, fA, fB, rC, rA, rB, eC, eA, z, std::integral_constant<int, 5>{});
        ++z;
    }
    __syncthreads();  // the last plane's hand-over visible
    if (pend) flush_pending(pend_slot);
    __syncthreads();  // LDS reuse by the next tile
}

template <int TX, int TY, bool PERY, bool PERZ>
__global__ __launch_bounds__(TX * (TY + 2)) void step_march2_kernel(GeomDev g, ProbeArgs pr, MarchPlan plan,
                                                                    const float* __restrict__ fin,
                                                                    float* __restrict__ fout) {
    __shared__ M2Lds<TX, TY> L;
    const int64_t t = *pr.tin;
    if (blockIdx.x == 0) record_probes<7>(g, pr, 2, fin);  // time t, from the input
    if (plan.lz > 0) {
        // tiles of chunk_z planes, XCD-contiguous ranges of the tile list
        const int xcd = blockIdx.x % kXcds;
        const int per_xcd_blocks = gridDim.x / kXcds;
        const int t_begin = (int)(plan.tiles * xcd / kXcds);
        const int t_end = (int)(plan.tiles * (xcd + 1) / kXcds);
        for (int tile = t_begin + (int)blockIdx.x / kXcds; tile < t_end; tile += per_xcd_blocks) {
            const int ty = tile % plan.nty, z0 = (tile / plan.nty) * plan.lz;
            if (z0 < g.n2) march2_tile<TX, TY, PERY, PERZ>(g, pr, pr.n, t, ty, TY, z0, min(z0 + plan.lz, g.n2), fin, fout, L);
        }
    } else {
        // balanced: this workgroup's share of the (row tile, plane) pairs,
        // marched as one segment per row tile it touches
        int64_t a = 0, e = 0;
        march2_share(plan.tiles, (int)gridDim.x, (int)blockIdx.x, &a, &e);
        while (a < e) {
            const int ty = (int)(a / g.n2), z0 = (int)(a % g.n2);
            const int z1 = (int)min((int64_t)g.n2, (int64_t)z0 + (e - a));
            march2_tile<TX, TY, PERY, PERZ>(g, pr, pr.n, t, ty, TY, z0, z1, fin, fout, L);
            a += z1 - z0;
        }
    }
}

// The geometries of a batch, two steps per launch: row tiles of it.rty2 whole
// axis-0 rows, marched in the segments that the host dealt out (equal shares of
// the planes: tiles of 24 planes, the best of fixed lengths, cost 13 us a step
// more).  96 horns of about 20 x 52 x 184: 173 us per step; single steps, bound by
// memory at 4.9 TB/s, 203.  Nine waves of a row tile's 28 x 20 threads leave the
// latency of a plane less hidden than in step_march2_kernel.
template <bool PERY>
__global__ __launch_bounds__(768) void step_batch2_kernel(const BatchItem* __restrict__ items,
                                                          const BatchSegment* __restrict__ seg,
                                                          const int32_t* __restrict__ seg_begin, int n_items,
                                                          BatchProbeArgs bp, const float* __restrict__ fin,
                                                          float* __restrict__ fout) {
    __shared__ M2Lds<96, 6, true> L;
    const int64_t* __restrict__ t_now = bp.tcount + (size_t)bp.parity * n_items;
    const auto geom = [&](const BatchItem& it, GeomDev& g, ProbeArgs& pr) {
        g.dim = 3;
        g.n0 = it.n0;
        g.n1 = it.n1;
        g.n2 = it.n2;
        g.N = it.N;
        for (int a = 0; a < 3; ++a) {
            g.bc_lo[a] = it.bc_lo[a];
            g.bc_hi[a] = it.bc_hi[a];
        }
        g.c2 = it.c2;
        g.two_w0 = it.two_w0;
        g.damp = it.damp;
        g.tab = reinterpret_cast<const float*>(bp.tab4 + 2 * (size_t)it.tab_off);
        g.sqrtg = bp.sqrtg + it.sg_off;
        g.sg_node = 0;
        pr.nodes = bp.nodes + it.probe_off;
        pr.n = it.n_probes;
        pr.trace = bp.trace + it.probe_off;
        pr.t_max = bp.t_max;
    };
    // time t, from the input; the next time into the other bank
    for (int h = blockIdx.x; h < n_items; h += gridDim.x) {
        GeomDev g{};
        ProbeArgs pr{};
        geom(items[h], g, pr);
        const int64_t t = t_now[h];
        if (t >= 0 && t < pr.t_max) {
            const float* f = fin + items[h].f_off;
            for (int p = threadIdx.x; p < pr.n; p += blockDim.x) {
                const uint32_t node = (uint32_t)pr.nodes[p];
                const uint32_t e = node % (uint32_t)g.n0 + (uint32_t)g.n0 * (node / ((uint32_t)g.n0 * (uint32_t)g.n1));
                double s = 0.0;
                for (int l = 0; l < 7; ++l) s += (double)f[(uint32_t)l * (uint32_t)g.N + node];
                pr.trace[t * bp.stride + p] = s / g.sqrtg[e];
            }
        }
        if (threadIdx.x == 0) bp.tcount[(size_t)(bp.parity ^ 1) * n_items + h] = t + 2;
    }
    // the shares of an XCD's workgroups (those equal modulo 8) follow each other
    const int share = (int)(blockIdx.x % kXcds) * (int)(gridDim.x / kXcds) + (int)(blockIdx.x / kXcds);
    for (int i = seg_begin[share]; i < seg_begin[share + 1]; ++i) {
        const BatchSegment sg = seg[i];
        const BatchItem& it = items[sg.item];
        GeomDev g{};
        ProbeArgs pr{};
        geom(it, g, pr);
        march2_tile<96, 6, PERY, false, true>(g, pr, bp.stride, t_now[sg.item], sg.ty, it.rty2, sg.z0, sg.z1,
                                              fin + it.f_off, fout + it.f_off, L);
    }
}

template <int TX, int TY>
int blocks_per_cu2() {
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, step_march2_kernel<TX, TY, false, false>, TX * (TY + 2), 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}

}  // namespace

bool march2_shape_ok(int tx, int ty) {
    // 768 threads: the shapes whose registers fit three waves per SIMD
    // without spilling (taller tiles spill at four)
    return (tx == 96 && ty == 6) || (tx == 128 && ty == 4);
}

bool march2_fits(const GeomDev& g, int tx) {
    return g.dim == 3 && !g.sg_node && g.n0 <= tx && g.bc_lo[0] != LBW_BC_PERIODIC;
}

int march2_tile_probes() { return kTileProbes; }

int march2_blocks_per_cu(int tx, int ty) {
    return tx == 96 ? blocks_per_cu2<96, 6>() : blocks_per_cu2<128, 4>();
}

MarchPlan make_march2_plan(const GeomDev& g, int tx, int ty, int lz, int blocks) {
    MarchPlan p{};
    p.tx = tx;
    p.ty = ty;
    p.lz = lz < 0 ? 0 : lz;
    p.ntx = 1;
    p.nty = (g.n1 + ty - 1) / ty;
    // balanced (lz 0): tiles counts the (row tile, plane) pairs shared out
    p.nchunks = p.lz > 0 ? (g.n2 + p.lz - 1) / p.lz : 0;
    p.tiles = p.lz > 0 ? (int64_t)p.nty * p.nchunks : (int64_t)p.nty * g.n2;
    int b = blocks < kXcds ? kXcds : blocks;
    b = (b / kXcds) * kXcds;
    const int64_t cap = ((p.tiles + kXcds - 1) / kXcds) * kXcds;
    if (b > cap) b = (int)cap;
    if (b < kXcds) b = kXcds;
    p.blocks = b;
    return p;
}

namespace {
template <int TX, int TY>
void launch2_of(bool pery, bool perz, dim3 grid, dim3 block, hipStream_t st, const GeomDev& g, const ProbeArgs& pr,
                const MarchPlan& plan, const float* fin, float* fout) {
    if (pery && perz)
        hipLaunchKernelGGL((step_march2_kernel<TX, TY, true, true>), grid, block, 0, st, g, pr, plan, fin, fout);
    else if (pery)
        hipLaunchKernelGGL((step_march2_kernel<TX, TY, true, false>), grid, block, 0, st, g, pr, plan, fin, fout);
    else if (perz)
        hipLaunchKernelGGL((step_march2_kernel<TX, TY, false, true>), grid, block, 0, st, g, pr, plan, fin, fout);
    else
        hipLaunchKernelGGL((step_march2_kernel<TX, TY, false, false>), grid, block, 0, st, g, pr, plan, fin, fout);
}
}  // namespace

int batch2_rows(int n0, int n1) {
    // rows with their two halo rows fit the threads, four of them load rings;
    // equal shares of the axis-1 rows
    if (n0 < 4 || n0 > 96) return 0;
    const int most = 768 / n0 - 2;
    if (most < 2) return 0;
    const int tiles = (n1 + most - 1) / most, rows = (n1 + tiles - 1) / tiles;
    // the slots that any thread, idle ones included, reads or writes
    const int last = 767 / n0 > rows + 3 ? 767 / n0 : rows + 3;
    return (last + 4) * (n0 + 2) <= kRtSlots ? rows : 0;
}

int batch2_threads(int n0, int n1) {
    // the tile with its halo rows, and a coefficient row by one thread a value
    const int rows = batch2_rows(n0, n1), need = (rows + 2 > 6 ? rows + 2 : 6) * n0;
    return (need + 63) / 64 * 64;
}

hipError_t launch_step_batch2(const BatchItem* items, const BatchSegment* seg, const int32_t* seg_begin, int n_items,
                              int blocks, int threads, bool pery, const BatchProbeArgs& bp, const float* fin,
                              float* fout, hipStream_t st) {
    if (blocks < kXcds || blocks % kXcds || threads < 64 || threads > 768) return hipErrorInvalidValue;
    const dim3 grid(blocks), block(threads);
    if (pery)
        hipLaunchKernelGGL((step_batch2_kernel<true>), grid, block, 0, st, items, seg, seg_begin, n_items, bp, fin,
                           fout);
    else
        hipLaunchKernelGGL((step_batch2_kernel<false>), grid, block, 0, st, items, seg, seg_begin, n_items, bp, fin,
                           fout);
    return hipGetLastError();
}

hipError_t launch_step_march2(const GeomDev& g, const ProbeArgs& pr, const MarchPlan& plan, const float* fin,
                              float* fout, hipStream_t st) {
    if (!march2_shape_ok(plan.tx, plan.ty) || !march2_fits(g, plan.tx)) return hipErrorInvalidValue;
    const dim3 grid(plan.blocks), block(plan.tx * (plan.ty + 2));
    const bool pery = g.bc_lo[1] == LBW_BC_PERIODIC, perz = g.bc_lo[2] == LBW_BC_PERIODIC;
    if (plan.tx == 96)
        launch2_of<96, 6>(pery, perz, grid, block, st, g, pr, plan, fin, fout);
    else
        launch2_of<128, 4>(pery, perz, grid, block, st, g, pr, plan, fin, fout);
    return hipGetLastError();
}

}  // namespace lbw
