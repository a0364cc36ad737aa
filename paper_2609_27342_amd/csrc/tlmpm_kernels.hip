// tlmpm_kernels.hip -- gfx950 kernels of one TLMPM cutting substep.
//
// Work decomposition.  Particles are sorted into bricks of 4x4x4 reference cells;
// inside a brick by cell parity class (8 classes of 8 cells that share no grid node)
// and then by cell.  One 512-thread workgroup owns one brick: wave w holds parity
// class w, lane (i, j) holds particle j of cell i of that class, where the bits of
// j sit at lane bits 0, 1 and 4 and those of i at lane bits 2, 3 and 5 (a cell's 8
// lanes are two quads in rows 2q and 2q+1 of the wave).  A brick touches the 5x5x5
// box of nodes around it.
//
// Particle-to-grid sums are gathers with a fixed order, without float atomics:
//   1. every lane forms its particle's contribution to the 8 corner nodes of its
//      cell;
//   2. an 8-lane butterfly reduce-scatter leaves in lane (i, k) the sum of cell i's
//      particles for corner k (the j bit 2 stage swaps rows with
//      v_permlane16_swap, the other two add across the quad with DPP);
//   3. every lane writes its sum to its place in LDS, and the quad of lanes that owns a
//      node adds the 8 places that touch it (one cell of each class), class by class;
//   4. the box sums are written as this brick's partial; a node's total is the sum
//      of the partials of the (up to 8) bricks around it, formed in fixed order by
//      the kernel that consumes it.
// (Step 3 with the waves adding into one LDS box in turn took 9 barriers a round instead
// of 2 and a slot lookup per lane, corner and component.)
//
// Each node holds one slot (logical grid, Sec. III-D) per side code present in its
// 8 incident cells, in ascending code order; coupling (Eq. 8) is done per node when
// a box is finalized, by the node's quad, a component per lane.
//
// What bounds P2G and G2P: in a large scene vector issue and memory together (14M
// particles: P2G about 80 % of the issue slots at 3.8 TB/s, G2P 60 % at 3.9, where a device
// copy reaches 5.1), in a small one the chain of dependent phases in a workgroup (brick record,
// cell index and partial gather, coupling, particle stage, sums); at three workgroups per
// CU (80 registers, 43 to 53 KB of LDS).  Geometry that depends on the thread alone comes
// from tables, rows of particles at 32-bit offsets from the brick's first (1250 -> 1050
// vector instructions per wave of P2G: 183k particles on a cut 23.7 -> 22.9 us, 64 scenes
// 301 -> 287 us, 14M particles 572 -> 564 us, the plastic P2G 58.9 -> 54.6 us and 37 since
// its eigen-decomposition is cheaper).  The registers hold only because a round recomputes
// its lane geometry (`late`): hoisted out of the round loop it spills 20 and more words a
// lane.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "tlmpm_common.h"
#include "tlmpm_band.h"
#include "tlmpm_reach.h"
#include "tlmpm_device.h"


// A value that is the same in every lane, kept in a scalar register
DEV float scalar(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }

DEV int box_index(int X, int Y, int Z) { return (Z * 5 + Y) * 5 + X; }

// Global node id of box node (X, Y, Z) of cell brick (bx, by, bz); -1 outside the grid.
DEV long long box_gid(const SceneK& S, int bx, int by, int bz, int X, int Y, int Z)
{
    int gx = bx * TL_B + X, gy = by * TL_B + Y, gz = bz * TL_B + Z;
    if (gx > S.cx || gy > S.cy || gz > S.cz) return -1;
    long long nb = ((long long)(gz >> 2) * S.nby + (gy >> 2)) * S.nbx + (gx >> 2);
    return (nb << 6) | ((gz & 3) * 16 + (gy & 3) * 4 + (gx & 3));
}

// ------------------------------------------------------------------- box slot table
// Slots of the 125 box nodes, packed: node bn holds slots [base, base + count), their
// codes ascending; one word base | count << 16 per node.
struct BoxTab {
    int meta[TL_BOXN];
    uint32_t code[TL_BOX_SLOTS];
};

// A node's packed word and what a lane knows of its own node
DEV int tab_base(int meta) { return meta & 0xFFFF; }
DEV int tab_count(int meta) { return meta >> 16; }

// LDS words written by lanes of this wave are read by other lanes of it from here on
// (a wave's LDS operations run in order; this only keeps the compiler from moving them)
DEV void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Inclusive scan over the 64 lanes by DPP row shifts and row broadcasts
DEV int wave_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false); // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false); // row_bcast 15 to rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false); // row_bcast 31 to rows 2, 3
    return x;
}

// The counts of box nodes 2 l and 2 l + 1 in lane l (every wave loads all of them).
struct BoxCounts {
    int a, b;
    DEV void load(const SceneK& S, const uint8_t* cnt, int bx, int by, int bz)
    {
        const int l = threadIdx.x & 63;
        a = node_count(S, cnt, bx, by, bz, 2 * l);
        b = node_count(S, cnt, bx, by, bz, 2 * l + 1);
    }
    static DEV int node_count(const SceneK& S, const uint8_t* cnt, int bx, int by, int bz, int n)
    {
        if (n >= TL_BOXN) return 0;
        const long long g = box_gid(S, bx, by, bz, n % 5, (n / 5) % 5, n / 25);
        return g >= 0 ? (int)cnt[g] : 0;
    }
    // Packed words of all nodes: wave 0 writes them to T (read after the next barrier);
    // returns the total (every wave alike) and in `own` the word of node bn (no barrier:
    // every wave scans for itself).
    DEV int scan(BoxTab& T, int bn, int& own) const
    {
        const int l = threadIdx.x & 63;
        const int incl = wave_scan(a + b), base = incl - a - b;
        if (threadIdx.x < 64) {
            if (2 * l < TL_BOXN) T.meta[2 * l] = base | (a << 16);
            if (2 * l + 1 < TL_BOXN) T.meta[2 * l + 1] = (base + a) | (b << 16);
        }
        const int pair = __shfl(base | (a << 16) | (b << 24), bn >> 1, 64);
        const int pb = pair & 0xFFFF, pa = (pair >> 16) & 0xFF, pc = (pair >> 24) & 0xFF;
        own = (bn & 1) ? (pb + pa) | (pc << 16) : pb | (pa << 16);
        return __builtin_amdgcn_readlane(incl, 63);
    }
};

// Codes of the slots of node bn, loaded by the quad that owns it: lane u takes slots u,
// u + 4, ...; the first one is loaded ahead (pre) so that it is in flight with the
// partial gather.
DEV uint32_t codes_pre(const SceneK& S, const uint32_t* scode, int meta, long long gid, int u)
{
    return u < tab_count(meta) ? scode[(long long)u * S.NN + gid] : 0u;
}

DEV void codes_put(const SceneK& S, const uint32_t* scode, BoxTab& T, int meta, long long gid, int u, uint32_t pre)
{
    const int c = tab_count(meta), b0 = tab_base(meta);
    if (u < c) T.code[b0 + u] = pre;
    for (int s = u + 4; s < c; s += 4) T.code[b0 + s] = scode[(long long)s * S.NN + gid];
}

DEV int find_slot(const BoxTab& T, int bn, uint32_t key)
{
    const int m = T.meta[bn], c = tab_count(m), b0 = tab_base(m);
    for (int s = 0; s < c; s++)
        if (T.code[b0 + s] == key) return b0 + s;
    return -1;
}

// Partial arrays hold every active brick's sums over its 5x5x5 box of nodes:
// [active brick][slot][box node][QP floats], the Q components of one node-slot
// contiguous (QP = Q rounded up to 4 floats).  A node's slot index is global (the
// node's slot table), so all bricks that share the node use the same slot.
template <int Q>
struct QPad {
    static constexpr int value = (Q + 3) & ~3;
};

// The two contributors of box node bn that lane u of its quad loads: contributor d is
// the brick at home - (d & 1, d >> 1 & 1, d >> 2 & 1), which holds the node at box
// position (l + 4 * offset); lane u takes d = u and u + 4.  nb: the active indices of the
// 27 bricks around in lanes 0..26; every lane of the wave calls this.  Which of the 27 and
// which of its nodes are a table per thread.
struct ContribTable {
    uint16_t from[TL_WG][2]; // 4 x index into the 27 (a byte address across lanes), or 4 x 63: none
    uint16_t node[TL_WG][2];
    constexpr ContribTable() : from(), node()
    {
        for (int t = 0; t < TL_WG; t++)
            for (int e = 0; e < 2; e++) {
                const int bn = t >> 2, d = (t & 3) + 4 * e;
                const int N[3] = {bn % 5, (bn / 5) % 5, bn / 25};
                int at = 0, pn = 0, f27 = 1, f5 = 1;
                bool in = bn < TL_BOXN;
                for (int a = 0; a < 3; a++) {
                    const int o = (d >> a) & 1, l = N[a] & 3;
                    if (o && l) in = false;
                    at += f27 * ((N[a] >> 2) - o + 1);
                    pn += f5 * (l + 4 * o);
                    f27 *= 3;
                    f5 *= 5;
                }
                from[t][e] = (uint16_t)(4 * (in ? at : 63));
                node[t][e] = (uint16_t)(in ? pn : 0);
            }
    }
};
static __device__ const ContribTable k_contrib __attribute__((aligned(16))) = ContribTable();

struct Contrib {
    int ai[2];       // active index, -1: none
    unsigned rec[2]; // record of slot 0 (in nodes)
    DEV void set(const SceneK& S, int nb, int tid)
    {
        const uint32_t from = *(const uint32_t*)k_contrib.from[tid], node = *(const uint32_t*)k_contrib.node[tid];
#pragma unroll
        for (int e = 0; e < 2; e++) {
            // (lanes 27 .. 63 hold -1)
            ai[e] = __builtin_amdgcn_ds_bpermute((int)(e ? from >> 16 : from & 0xFFFFu), nb);
            rec[e] = (unsigned)ai[e] * (unsigned)(S.scap * TL_BOXN) + (e ? node >> 16 : node & 0xFFFFu);
        }
    }
};

// One slot's two loads of a lane and their sum over the quad: (own pair), then lanes
// ^ 1, then ^ 2.  The order is fixed: results are bitwise reproducible.  Every lane of
// the quad gets the sum.
template <int QP>
struct Gather {
    float4 v[2][QP / 4];
    DEV void load(const float* __restrict__ part, const Contrib& C, int s, bool on)
    {
#pragma unroll
        for (int e = 0; e < 2; e++) {
#pragma unroll
            for (int q = 0; q < QP / 4; q++) v[e][q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (on && C.ai[e] >= 0) {
                const float4* pp = (const float4*)(part + (size_t)(C.rec[e] + (unsigned)(s * TL_BOXN)) * QP);
#pragma unroll
                for (int q = 0; q < QP / 4; q++) v[e][q] = pp[q];
            }
        }
    }
    // a split brick's second partial, added to its first (xbox: see split_offset).  Its word
    // is read where it is used: kept from slot to slot, the words of both contributors cost
    // G2P of a batch six more spilled registers (256 scenes: 0.85 -> 0.88 ms).
    DEV void add(const float* __restrict__ xpart, const int* __restrict__ xbox, const Contrib& C, int s)
    {
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const int ai = late(C.ai[e]);
            const unsigned x = ai < 0 ? 0u : (unsigned)xbox[ai];
            if (!x) continue;
            const float4* xp = (const float4*)(xpart + (size_t)(C.rec[e] + x - 1u + (unsigned)(s * TL_BOXN)) * QP);
#pragma unroll
            for (int q = 0; q < QP / 4; q++) {
                const float4 x4 = xp[q];
                v[e][q].x += x4.x;
                v[e][q].y += x4.y;
                v[e][q].z += x4.z;
                v[e][q].w += x4.w;
            }
        }
    }
    template <int Q>
    DEV void sum(float (&acc)[Q]) const
    {
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const float4 a = v[0][q / 4], b = v[1][q / 4];
            acc[q] = (q % 4 == 0) ? a.x + b.x : (q % 4 == 1) ? a.y + b.y : (q % 4 == 2) ? a.z + b.z : a.w + b.w;
            acc[q] += lane_xor<1>(acc[q]);
            acc[q] += lane_xor<2>(acc[q]);
        }
    }
};

// Compatibility coupling of component `off` of a node with slots [b0, b0 + c) (Eq. 8):
// f_a += (1/M) sum_{b != a, compatible} (m_a f_b - m_b f_a), M = sum of all slot masses;
// src[slot * Q] the masses, src[slot * Q + off] the field, all pre-exchange values.
// Calls put(slot, m, f_bar).
template <int Q, class Put>
DEV void couple_component(const BoxTab& T, int b0, int c, const float* src, int off, Put&& put)
{
    float M = 0.0f;
    for (int a = 0; a < c; a++) M += src[(b0 + a) * Q];
    const float invM = M > 0.0f ? 1.0f / M : 0.0f;
    for (int a = 0; a < c; a++) {
        const uint32_t ca = T.code[b0 + a];
        const float ma = src[(b0 + a) * Q], fa = src[(b0 + a) * Q + off];
        float acc = 0.0f;
        for (int b = 0; b < c; b++) {
            if (b == a || codes_conflict(ca, T.code[b0 + b])) continue;
            const float mb = src[(b0 + b) * Q];
            acc += ma * src[(b0 + b) * Q + off] - mb * fa;
        }
        put(b0 + a, ma, fa + acc * invM);
    }
}

// ------------------------------------------------------------- particle geometry
struct Lane {
    int w, lane, i, j;
    int cxl, cyl, czl; // cell inside the brick
    int beg, count;    // particles of the cell
};

// Place of thread tid in its brick
DEV Lane lane_at(int tid)
{
    Lane L;
    L.w = tid >> 6;
    L.lane = tid & 63;
    L.i = ((L.lane >> 2) & 3) | ((L.lane >> 3) & 4); // lane bits 2, 3, 5
    L.j = (L.lane & 3) | ((L.lane >> 2) & 4);        // lane bits 0, 1, 4
    L.cxl = 2 * (L.i & 1) + (L.w & 1);
    L.cyl = 2 * ((L.i >> 1) & 1) + ((L.w >> 1) & 1);
    L.czl = 2 * ((L.i >> 2) & 1) + ((L.w >> 2) & 1);
    L.beg = L.count = 0;
    return L;
}

DEV void lane_cell(const SceneD& D, int brick, Lane& L)
{
    const int* cs = D.cell_start + (long long)brick * TL_CELLS + L.w * 8 + L.i;
    L.beg = cs[0];
    L.count = cs[1] - cs[0];
}

// Arrays from a brick's first particle on: rows of the brick's particles at 32-bit offsets
// from a scalar base.
struct Local {
    int p0; // first particle of the brick
    long long N;
    DEV Local(const SceneK& S, const SceneD& D, int brick)
        : p0(D.cell_start[(long long)brick * TL_CELLS]), N(S.N)
    {
    }
    DEV float* row(float* a, int p) const { return (float*)((char*)(a + 3 * (size_t)p0) + 12u * (unsigned)(p - p0)); }
    DEV float* row(float* a, int r, int p) const // row r of a matrix
    {
        return (float*)((char*)(a + 3 * ((size_t)r * (size_t)N + (size_t)p0)) + 12u * (unsigned)(p - p0));
    }
    template <class T>
    DEV T* one(T* a, int p) const
    {
        return (T*)((char*)(a + (size_t)p0) + 4u * (unsigned)(p - p0));
    }
    DEV void get(float* a, int p, float* v) const
    {
        const float* q = row(a, p);
        v[0] = q[0];
        v[1] = q[1];
        v[2] = q[2];
    }
    DEV void get9(float* a, int p, float* v) const
    {
#pragma unroll
        for (int r = 0; r < 3; r++) {
            const float* q = row(a, r, p);
            v[3 * r] = q[0];
            v[3 * r + 1] = q[1];
            v[3 * r + 2] = q[2];
        }
    }
    DEV void put9(float* a, int p, const float* v) const
    {
#pragma unroll
        for (int r = 0; r < 3; r++) {
            float* q = row(a, r, p);
            q[0] = v[3 * r];
            q[1] = v[3 * r + 1];
            q[2] = v[3 * r + 2];
        }
    }
};

// Particle of this lane in round r.  Bricks whose cells each hold one code take
// particle 8 r + j of the lane's cell; bricks with a mixed cell take particle j of
// the cell's r-th same-code group (group table built when the codes change).
DEV bool lane_particle(const SceneD& D, int bi, bool grouped, const Lane& L, int r, int& p)
{
    if (!grouped) {
        const int jj = 8 * r + L.j;
        p = L.beg + (jj < L.count ? jj : 0);
        return jj < L.count;
    }
    p = L.beg;
    if (r >= TL_GMAX) return false;
    const int m = D.gmeta[((long long)bi * TL_CELLS + L.w * 8 + L.i) * TL_GMAX + r];
    const int cnt = m & 15, off = m >> 4;
    if (L.j >= cnt) return false;
    p = D.gperm[L.beg + off + L.j];
    return true;
}

// fractional position inside the base cell (reading R1), in [0, 1]
DEV void frac_of(const SceneK& S, const float* X, int gxc, int gyc, int gzc, float t[3])
{
    double q0 = ((double)X[0] - S.ox) * S.inv_dx_d - (double)gxc;
    double q1 = ((double)X[1] - S.oy) * S.inv_dx_d - (double)gyc;
    double q2 = ((double)X[2] - S.oz) * S.inv_dx_d - (double)gzc;
    t[0] = fminf(fmaxf((float)q0, 0.0f), 1.0f);
    t[1] = fminf(fmaxf((float)q1, 0.0f), 1.0f);
    t[2] = fminf(fmaxf((float)q2, 0.0f), 1.0f);
}

// ... of the lane's particle, as P2G takes it: from the scene's T, or (FRAC false) from X
// where a scene of the launch has no T.  A kernel of its own: a branch on D.T keeps the
// scalars of both ways in registers (a 1.3 % slower pass of a 14M-particle scene).
template <bool FRAC>
DEV void cell_position(const SceneK& S, const SceneD& D, const Local& loc, const int4 info, const Lane& L, int p,
                       float t[3])
{
    if constexpr (FRAC) {
        loc.get(D.T, p, t);
    } else {
        float X[3];
        loc.get(D.X, p, X);
        frac_of(S, X, info.y * TL_B + L.cxl, info.z * TL_B + L.cyl, info.w * TL_B + L.czl, t);
    }
}

// The positions inside the reference cells, once per scene: P2G reads them in place of X
// (the same bytes, and no FP64 chain per particle and substep)
__global__ __launch_bounds__(256) void k_frac(SceneK S, SceneD D)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= S.N) return;
    const long long cs = D.pcell[p], brick = cs / TL_CELLS;
    const int w = (int)(cs & 63) >> 3, i = (int)cs & 7;
    const int bx = (int)(brick % S.cbx), by = (int)((brick / S.cbx) % S.cby), bz = (int)(brick / (S.cbx * S.cby));
    const float X[3] = {D.X[at3(p, 0)], D.X[at3(p, 1)], D.X[at3(p, 2)]};
    float t[3];
    frac_of(S, X, bx * TL_B + 2 * (i & 1) + (w & 1), by * TL_B + 2 * ((i >> 1) & 1) + ((w >> 1) & 1),
            bz * TL_B + 2 * ((i >> 2) & 1) + ((w >> 2) & 1), t);
    for (int a = 0; a < 3; a++) D.T[at3(p, a)] = t[a];
}

DEV void corner_weights(const float t[3], int k, float& wx, float& wy, float& wz)
{
    wx = (k & 1) ? t[0] : 1.0f - t[0];
    wy = (k & 2) ? t[1] : 1.0f - t[1];
    wz = (k & 4) ? t[2] : 1.0f - t[2];
}

// --------------------------------------------------------- butterfly reduce-scatter
// Weights of the 8 corners of a lane's cell in the order the relative butterfly
// takes them: corner r has x bit (r & 1) and y bit (r >> 1 & 1) relative to the
// lane's own corner j (clear: j's side, set: the other side) and z bit (r >> 2)
// absolute, so its absolute index is r ^ (j & 3).  Each factor is the one
// corner_weights gives for the absolute corner.
struct CornerW {
    float wx[2], wy[2], wz[2];
};

DEV CornerW corner_table(const float t[3], int j)
{
    CornerW c;
    const bool bx = j & 1, by = (j >> 1) & 1;
    const float ox = 1.0f - t[0], oy = 1.0f - t[1];
    c.wx[0] = bx ? t[0] : ox;
    c.wx[1] = bx ? ox : t[0];
    c.wy[0] = by ? t[1] : oy;
    c.wy[1] = by ? oy : t[1];
    c.wz[0] = 1.0f - t[2];
    c.wz[1] = t[2];
    return c;
}

// gen(r, out) produces this lane's contribution to corner r of its cell, r in the order of
// CornerW (x and y bits relative to the lane's own corner j).  Result: res[Q] = sum over the
// 8 lanes of the cell group of their values for corner j.  Stage 1 pairs j with j ^ 4 (lane
// ^ 16): v_permlane16_swap of (z = 0, z = 1) leaves in the even row (z bit of j clear) its
// own and its partner's z = 0 values, in the odd row the z = 1 values; stages 2 and 3 pair
// j ^ 2 and j ^ 1 within the quad, each lane sending its other-side value (the partner's
// side: no select).  The sum tree is ((j, j^4), (j^2, j^6)), ((j^1, j^5), (j^3, j^7)), own
// operand first, for every lane order.  Corners are generated in (z = 0, z = 1) pairs, so at
// most 4 x Q partial sums are live.
template <int Q, class Gen>
DEV void reduce_scatter8(Gen&& gen, float (&res)[Q])
{
    float c1[4][Q];
#pragma unroll
    for (int rr = 0; rr < 4; rr++) {
        float lo[Q], hi[Q];
        gen(rr, lo);
        gen(rr | 4, hi);
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo[q]), __float_as_uint(hi[q]), false,
                                                             false);
            c1[rr][q] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
    }
    float c2[2][Q];
#pragma unroll
    for (int rr = 0; rr < 2; rr++)
#pragma unroll
        for (int q = 0; q < Q; q++) c2[rr][q] = c1[rr][q] + lane_xor<2>(c1[rr | 2][q]);
#pragma unroll
    for (int q = 0; q < Q; q++) res[q] = c2[0][q] + lane_xor<1>(c2[1][q]);
}

// ------------------------------------------------------- history-based friction
// Tangential spring transported to the current tangent plane (length kept), trial
// force -k_t u - c_t v_t, stick below mu_s f_n, else slip at mu_d f_n with the
// spring reset to match the applied force (Eq. 12).
DEV void friction(const SceneK& S, const float vrel[3], const float n[3], float fn, float meff, float u[3],
                  float ft[3])
{
    float dt = S.dt;
    float un = u[0] * n[0] + u[1] * n[1] + u[2] * n[2];
    float up[3] = {u[0] - un * n[0], u[1] - un * n[1], u[2] - un * n[2]};
    float lu = sqrtf(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    float lp = sqrtf(up[0] * up[0] + up[1] * up[1] + up[2] * up[2]);
    float sc = lp > 0.0f ? lu / lp : 0.0f;
    float ut[3] = {up[0] * sc, up[1] * sc, up[2] * sc};
    float vn = vrel[0] * n[0] + vrel[1] * n[1] + vrel[2] * n[2];
    float vt[3] = {vrel[0] - vn * n[0], vrel[1] - vn * n[1], vrel[2] - vn * n[2]};
    float kt = S.gamma_k * meff / (dt * dt);
    float ct = 2.0f * S.gamma_c * sqrtf(meff * kt);
    float ftr[3] = {-kt * ut[0] - ct * vt[0], -kt * ut[1] - ct * vt[1], -kt * ut[2] - ct * vt[2]};
    float lf = sqrtf(ftr[0] * ftr[0] + ftr[1] * ftr[1] + ftr[2] * ftr[2]);
    if (lf <= S.mu_s * fn) {
        for (int a = 0; a < 3; a++) {
            ft[a] = ftr[a];
            u[a] = ut[a] + dt * vt[a];
        }
    } else {
        float sl = S.mu_d * fn / lf;
        for (int a = 0; a < 3; a++) {
            ft[a] = ftr[a] * sl;
            u[a] = -(ft[a] + ct * vt[a]) / kt;
        }
    }
}

// One rigid body against one particle (Eqs. 14-16, 5).  body 0 = floor, else tool.
// Returns the impulse on the particle in J (added), updates D and the wrench sums.
// The contact geometry (closest point, gap, normal, front-band coordinates) is
// formed in FP64 from the exact current position x = X + u: the normal impulse is
// s_n m / dt times the gap, and for a particle close to the zero-thickness blade
// the normal is (x - x_c) / |x - x_c| of a short vector, so FP32 rounding of the
// positions (1e-8 m at 0.2 m) would shift the gap and turn the normal by far more
// than the FP32 state error.
DEV void rigid_one(const SceneK& S, const SceneD& D, const DevTool* T, int slot, long long p, const double x[3],
                   const float v[3], float m, float V0, float R, int stamp, double jdt, float J[3], float& Dp,
                   float Dstart, float* wr)
{
    const float dt = S.dt;
    double adv = (T && (T->flags & TL_TOOL_ADVANCE)) ? jdt : 0.0;
    float nB[3], phi, vB[3] = {0.0f, 0.0f, 0.0f}, arm[3] = {0.0f, 0.0f, 0.0f};
    float invm = 0.0f;
    double r[3] = {0.0, 0.0, 0.0}; // x - x_e of a tool
    if (!T) {
        nB[0] = 0.0f;
        nB[1] = 0.0f;
        nB[2] = 1.0f;
        phi = (float)((x[2] - (double)S.floor_z) - (double)R);
    } else {
        const DevBlade& B = T->b;
        for (int a = 0; a < 3; a++) r[a] = x[a] - (B.xe[a] + adv * B.ve[a]);
        double al = r[0] * B.e[0] + r[1] * B.e[1] + r[2] * B.e[2];
        double be = -(r[0] * B.d[0] + r[1] * B.d[1] + r[2] * B.d[2]);
        al = fmin(fmax(al, -B.half_len), B.half_len);
        be = fmin(fmax(be, 0.0), B.b_back);
        double df[3];
        for (int a = 0; a < 3; a++) df[a] = r[a] - al * B.e[a] + be * B.d[a]; // x - x_c
        const double dist = sqrt(df[0] * df[0] + df[1] * df[1] + df[2] * df[2]);
        if (dist > 0.0)
            for (int a = 0; a < 3; a++) nB[a] = (float)(df[a] / dist);
        else
            for (int a = 0; a < 3; a++) nB[a] = (float)B.n[a];
        phi = (float)(dist - (double)R);
        for (int a = 0; a < 3; a++)
            arm[a] = (float)((x[a] - df[a]) - (T->xB[a] + adv * T->vB[a])); // x_c - x_B
        float wxr[3] = {T->wB[1] * arm[2] - T->wB[2] * arm[1], T->wB[2] * arm[0] - T->wB[0] * arm[2],
                        T->wB[0] * arm[1] - T->wB[1] * arm[0]};
        for (int a = 0; a < 3; a++) vB[a] = (float)T->vB[a] + wxr[a];
        // inverse effective mass of the tool at xc along nB: w_B + 1/M + (r x n) . I^-1 (r x n)
        const float cr[3] = {arm[1] * nB[2] - arm[2] * nB[1], arm[2] * nB[0] - arm[0] * nB[2],
                             arm[0] * nB[1] - arm[1] * nB[0]};
        float ang = 0.0f;
        for (int a = 0; a < 3; a++)
            ang += cr[a] * (T->iinv[3 * a] * cr[0] + T->iinv[3 * a + 1] * cr[1] + T->iinv[3 * a + 2] * cr[2]);
        invm = T->invm + T->imass + ang;
    }
    float vrel[3] = {v[0] - vB[0], v[1] - vB[1], v[2] - vB[2]};
    float vrn = vrel[0] * nB[0] + vrel[1] * nB[1] + vrel[2] * nB[2];
    float phihat = phi + dt * fminf(vrn, 0.0f);
    float meff = 1.0f / (1.0f / m + invm);
    float Jn = S.s_n * meff / dt * fmaxf(-phihat, 0.0f);
    if (!(Jn > 0.0f)) return;
    float* h = D.hist + (long long)slot * 4 * S.N;
    float u[3] = {0.0f, 0.0f, 0.0f};
    if (__float_as_int(h[3 * S.N + p]) == stamp - 1) {
        u[0] = h[p];
        u[1] = h[S.N + p];
        u[2] = h[2 * S.N + p];
    }
    float ft[3];
    friction(S, vrel, nB, Jn / dt, meff, u, ft);
    h[p] = u[0];
    h[S.N + p] = u[1];
    h[2 * S.N + p] = u[2];
    h[3 * S.N + p] = __int_as_float(stamp);
    float JpB[3] = {Jn * nB[0] + ft[0] * dt, Jn * nB[1] + ft[1] * dt, Jn * nB[2] + ft[2] * dt};
    if (T && (T->flags & TL_TOOL_CUTTING)) {
        const DevBlade& B = T->b;
        const double sv = r[0] * B.n[0] + r[1] * B.n[1] + r[2] * B.n[2];
        const double lv = r[0] * B.e[0] + r[1] * B.e[1] + r[2] * B.e[2];
        const double fv = r[0] * B.d[0] + r[1] * B.d[1] + r[2] * B.d[2];
        float uc = ((float)B.ve[0] - v[0]) * (float)B.d[0] + ((float)B.ve[1] - v[1]) * (float)B.d[1] +
                   ((float)B.ve[2] - v[2]) * (float)B.d[2];
        if (fabs(sv) <= B.half_width && fabs(lv) <= B.half_len && fv >= 0.0 && fv <= B.b_lead && uc > S.u_min) {
            float dd[3] = {(float)B.d[0], (float)B.d[1], (float)B.d[2]};
            float Jc = fmaxf(JpB[0] * dd[0] + JpB[1] * dd[1] + JpB[2] * dd[2], 0.0f);
            if (Dstart < 1.0f) {
                float Wth = S.G_c * powf(V0, 2.0f / 3.0f) * (1.0f - S.zeta) / S.zeta;
                Dp = fminf(Dp + Jc * uc / Wth, 1.0f);
            } else {
                for (int a = 0; a < 3; a++) JpB[a] -= Jc * dd[a];
            }
        }
    }
    for (int a = 0; a < 3; a++) J[a] += JpB[a];
    if (wr) {
        float Fb[3] = {-JpB[0] / dt, -JpB[1] / dt, -JpB[2] / dt};
        wr[0] += Fb[0];
        wr[1] += Fb[1];
        wr[2] += Fb[2];
        wr[3] += arm[1] * Fb[2] - arm[2] * Fb[1];
        wr[4] += arm[2] * Fb[0] - arm[0] * Fb[2];
        wr[5] += arm[0] * Fb[1] - arm[1] * Fb[0];
    }
}

// --------------------------------------------------------------------------- K_A
// P2G kernel (one brick per workgroup).  If f_pending: finalize the remapped
// velocities of the previous substep's MUSL re-scatter on the box (tables rs),
// apply the deformation-gradient update and write F.  Then, if do_p2g: stress,
// tool/floor contact, and the label-masked P2G of (m, p, dp) (Eq. 2 with external
// and contact impulses, Eqs. 13, 16) into this brick's partials (tables cur).
struct KA_Args {
    int do_p2g;      // 0: only the pending F update
    int tabs_differ; // cur != rsb (applies to scenes with a pending F update)
    int cur;         // current slot table buffer
    int rsb;         // slot table buffer of the pending re-scatter
};

// --------------------------------------------------------------------- rigid contact
// Floor and tool contact of every particle of bricks whose AABB can reach a rigid
// body this substep (Eqs. 14-16, 5): impulses to Jrig, cutting progress D, contact
// springs, and per-brick wrench sums added to those of the call (wave tree, then
// waves in order).  Bound by the FP64 chain per particle and the loads around it where
// a body is near, by the number of workgroups elsewhere.
#define TL_GROUP 16   // most bricks per workgroup of these passes
#define TL_BODIES (TL_MAX_TOOLS + 1)

// Rigid contact of a brick within reach of the bodies of mask `near` (bit 0 the floor, bit
// 1 + b tool b), whole block.
DEV void rigid_brick(const SceneK& S, const SceneD& D, int bi, int brick, int near)
{
    __shared__ float s_wr[4][TL_MAX_TOOLS * 6];
    const int n_tools = D.tinfo[0];
    const int stamp = D.ctr[0];
    const double jdt = (double)D.ctr[2] * S.dt_d; // substep of the call (TL_TOOL_ADVANCE poses)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const bool want_wrench = D.tinfo[1] != 0;
    const int beg = D.cell_start[(long long)brick * TL_CELLS], end = D.cell_start[(long long)(brick + 1) * TL_CELLS];
    if (lane < TL_MAX_TOOLS * 6) s_wr[wv][lane] = 0.0f;
    for (int p0 = beg; p0 < end; p0 += 256) {
        const int p = p0 + tid;
        const bool valid = p < end;
        double x[3] = {0.0, 0.0, 0.0};
        float v[3] = {0.0f, 0.0f, 0.0f}, m = 0.0f, V0 = 0.0f, R = 0.0f, Dp = 0.0f;
        float Jc[3] = {0.0f, 0.0f, 0.0f};
        if (valid) {
            for (int a = 0; a < 3; a++) {
                x[a] = (double)D.X[at3(p, a)] + (double)D.u[at3(p, a)];
                v[a] = D.v[at3(p, a)];
            }
            m = S.m_uniform ? S.m0 : D.m[p];
            V0 = S.v_uniform ? S.V0 : D.V0[p];
            R = 0.5f * S.s_R * cbrtf(V0);
            Dp = D.D[p];
        }
        const float Ds = Dp;
        if (valid && (near & 1)) rigid_one(S, D, nullptr, 0, p, x, v, m, V0, R, stamp, jdt, Jc, Dp, Dp, nullptr);
        for (int b = 0; b < n_tools; b++) {
            if (!((near >> (b + 1)) & 1)) continue;
            float wr[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            if (valid) rigid_one(S, D, &D.tools[b], 1 + b, p, x, v, m, V0, R, stamp, jdt, Jc, Dp, Ds, wr);
            bool nz = wr[0] != 0.0f || wr[1] != 0.0f || wr[2] != 0.0f;
            if (want_wrench && __any(nz)) {
                for (int q = 0; q < 6; q++) {
                    float val = wr[q];
                    for (int o = 32; o >= 1; o >>= 1) val += __shfl_xor(val, o, 64);
                    if (lane == 0) s_wr[wv][b * 6 + q] += val;
                }
            }
        }
        if (valid) {
            D.Jrig[at3(p, 0)] = Jc[0];
            D.Jrig[at3(p, 1)] = Jc[1];
            D.Jrig[at3(p, 2)] = Jc[2];
            if (Dp != Ds) D.D[p] = Dp;
        }
    }
    if (want_wrench) { // bricks out of reach add nothing to the call's sums
        __syncthreads();
        if (tid < n_tools * 6) {
            float acc = 0.0f;
            for (int w = 0; w < 4; w++) acc += s_wr[w][tid];
            D.wpart[(long long)tid * D.n_active + bi] += (double)acc;
        }
    }
}

// Bodies (mask as in rigid_brick) that can reach a brick this substep, one test per lane
DEV bool body_near(const SceneK& S, const SceneD& D, int bi, int brick, int body)
{
    if (body == 0 ? !S.floor_on : (body > D.tinfo[0] || !(D.tools[body - 1].flags & TL_TOOL_CONTACT))) return false;
    float bb[7];
    brick_aabb(S, D, bi, brick, bb);
    if (body == 0) return brick_near_floor(bb, S.floor_z, S.Rmax, S.dt);
    return brick_near_tool(bb, D.tools[body - 1], S.Rmax, S.dt, (double)D.ctr[2] * S.dt_d);
}

// The work items of a brick pass: the bricks of one scene, or (scene, brick) pairs
struct BricksOfScene {
    const SceneK& S;
    const SceneD& D;
    int n;
    DEV const SceneK& scene(int) const { return S; }
    DEV const SceneD& data(int) const { return D; }
    DEV int brick(int i) const { return i; }
};
struct BricksOfBatch {
    const SceneK* Ks;
    const SceneD* Ds;
    const int2* it;
    int n;
    DEV const SceneK& scene(int i) const { return Ks[it[i].x]; }
    DEV const SceneD& data(int i) const { return Ds[it[i].x]; }
    DEV int brick(int i) const { return it[i].y; }
};

// Rigid contact of nb bricks per workgroup, bricks w, w + G, w + 2 G, ... (G workgroups:
// neighbours near one body fall to different ones): the first lanes test every body
// against every brick at once, then the workgroup goes through the bricks within reach.
template <class Items>
DEV void rigid_group(const Items& I, int w, int G, int nb)
{
    __shared__ int s_near[TL_GROUP * 8];
    const int t = threadIdx.x;
    if (t < nb * 8) {
        const int i = w + (t >> 3) * G, body = t & 7;
        bool nr = false;
        if (i < I.n && body < TL_BODIES) {
            const SceneD& D = I.data(i);
            const int bi = I.brick(i);
            nr = body_near(I.scene(i), D, bi, D.active[bi], body);
        }
        // the mask of a brick from its 8 lanes
        const unsigned long long all = __ballot(nr);
        const int mask = (int)((all >> (t & 56)) & 0xFF);
        if (body == 0) {
            s_near[t >> 3] = mask;
            if (i < I.n && (I.scene(i).floor_on || I.data(i).tinfo[1])) {
                const SceneD& D = I.data(i);
                D.brig[D.active[I.brick(i)]] = mask != 0;
            }
        }
    }
    __syncthreads();
    for (int k = 0; k < nb; k++) {
        const int m = s_near[k];
        if (!m) continue;
        const int i = w + k * G;
        const SceneD& D = I.data(i);
        const int bi = I.brick(i);
        rigid_brick(I.scene(i), D, bi, D.active[bi], m);
        __syncthreads(); // the brick's LDS words are reused by the next one
    }
}

// ------------------------------------------------------- particle stage of P2G
// Gradient Lg of the field v(k) at the corners k of a particle's cell.  A zero weight
// contributes nothing (reading R7); where no particle of the wave has a weight at or near
// zero along an axis (nearly every wave), no product of three is zero and the tests are
// left out.  The other waves go over the corners once more, one by one (a second unrolled
// copy would share its products with the first across the branch, and spill them).
template <class V>
DEV void grad_of(const SceneK& S, const float* t, V&& v, float* Lg)
{
    auto add = [&](int k, bool test) {
        float wx, wy, wz;
        corner_weights(t, k, wx, wy, wz);
        const float4 v4 = v(k);
        float g0 = ((k & 1) ? S.inv_dx : -S.inv_dx) * wy * wz;
        float g1 = ((k & 2) ? S.inv_dx : -S.inv_dx) * wx * wz;
        float g2 = ((k & 4) ? S.inv_dx : -S.inv_dx) * wx * wy;
        if (test && wx * wy * wz == 0.0f) g0 = g1 = g2 = 0.0f;
        const float va[3] = {v4.x, v4.y, v4.z};
#pragma unroll
        for (int a = 0; a < 3; a++) {
            Lg[3 * a + 0] = test || k ? Lg[3 * a + 0] + va[a] * g0 : va[a] * g0;
            Lg[3 * a + 1] = test || k ? Lg[3 * a + 1] + va[a] * g1 : va[a] * g1;
            Lg[3 * a + 2] = test || k ? Lg[3 * a + 2] + va[a] * g2 : va[a] * g2;
        }
    };
#pragma unroll
    for (int k = 0; k < 8; k++) add(k, false);
    const float lo = fminf(fminf(t[0], t[1]), t[2]), hi = fmaxf(fmaxf(t[0], t[1]), t[2]);
    if (__any(lo < 1e-12f || 1.0f - hi < 1e-12f)) {
#pragma unroll
        for (int a = 0; a < 9; a++) Lg[a] = 0.0f;
#pragma unroll 1
        for (int k = 0; k < 8; k++) add(k, true);
    }
}

// F update from the gradient Lg of the remapped velocities (MUSL), stored; a particle
// whose code changed in this substep's label pass used its previous code for it and drops
// that mark.  A state that is not finite sets the status: here with `check`, else by the
// stress that follows (no entry of H that is not finite leaves J finite).
DEV void store_F(const SceneD& D, const Local& loc, int p, float dt, const float* Lg, bool check, float* H,
                 uint32_t& code)
{
#pragma unroll
    for (int a = 0; a < 9; a++) H[a] += dt * Lg[a];
    loc.put9(D.H, p, H);
    if (check) {
        bool fin = true;
        for (int a = 0; a < 9; a++) fin = fin && isfinite(H[a]);
        if (!fin) atomicOr(D.status, TL_ST_NONFINITE);
    }
    if (code & TL_PREV_BIT) {
        code &= ~TL_PREV_BIT;
        *loc.one(D.code, p) = code;
    }
}

// MAT 1: plastic projection after an F update, and the rate of F for the viscosity
// (kept for the substeps whose P2G has no pending update: the first, or after a
// state read)
template <int MAT>
DEV void plastic_rate(const SceneK& S, const SceneD& D, const Local& loc, int p, bool updated, const float* H,
                      float* Lg, float* Gp)
{
    if constexpr (MAT == 1) {
        // plasticity: F_p^{-1} = I + Gp; projection after each F update
        if (S.ystress > 0.0f) {
            loc.get9(D.Gp, p, Gp);
            if (updated) {
                float K[9]; // F_e - I = H + Gp + H Gp
#pragma unroll
                for (int i = 0; i < 3; i++)
#pragma unroll
                    for (int j = 0; j < 3; j++) {
                        float k = H[3 * i + j] + Gp[3 * i + j];
#pragma unroll
                        for (int m = 0; m < 3; m++) k += H[3 * i + m] * Gp[3 * m + j];
                        K[3 * i + j] = k;
                    }
                float mu, lam;
                lame(S, S.e_uniform ? 0.0f : *loc.one(D.E, p), mu, lam);
                if (vm_project(mu, S.ystress, K, Gp)) loc.put9(D.Gp, p, Gp);
            }
        }
        if (S.visc > 0.0f) {
            if (updated)
                loc.put9(D.Fdot, p, Lg);
            else
                loc.get9(D.Fdot, p, Lg);
        }
    }
}

// First Piola-Kirchhoff stress of a particle (zero with the status bit set where J <= 0
// or the state is not finite)
template <int MAT>
DEV void particle_stress(const SceneK& S, const SceneD& D, float E, const float* H, const float* Lg, const float* Gp,
                         float* Pk)
{
    bool ok;
    float mu, lam;
    lame(S, E, mu, lam);
    if constexpr (MAT == 1) {
        if (S.ystress > 0.0f) {
            // P = P_fcr(F_e) F_p^{-T}, F_e - I = H + Gp + H Gp, F_p^{-1} = I + Gp
            float K[9], Pe[9];
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    float k = H[3 * i + j] + Gp[3 * i + j];
#pragma unroll
                    for (int m = 0; m < 3; m++) k += H[3 * i + m] * Gp[3 * m + j];
                    K[3 * i + j] = k;
                }
            ok = fixed_corotated(mu, lam, K, Pe);
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    float a = Pe[3 * i + j];
#pragma unroll
                    for (int m = 0; m < 3; m++) a += Pe[3 * i + m] * Gp[3 * j + m];
                    Pk[3 * i + j] = a;
                }
        } else {
            ok = S.material == 1 ? fixed_corotated(mu, lam, H, Pk) : neo_hookean(mu, lam, H, Pk);
        }
    } else {
        ok = neo_hookean(mu, lam, H, Pk);
    }
    if (ok && MAT == 1 && S.visc > 0.0f) add_viscous(S.visc, H, Lg, Pk);
    if (!ok) {
        atomicOr(D.status, TL_ST_NONFINITE);
        for (int a = 0; a < 9; a++) Pk[a] = 0.0f;
    }
}

// What a particle adds to the 8 corners of its cell: w (m, m v) and A grad N + w ext
// with A = -dt V0 P (Eq. 2); a zero weight contributes nothing (reading R7).  Corners in
// the order of CornerW; the gradient's sign along x and y is that of the lane's own corner
// on its side and the opposite one on the other.
struct Scatter {
    CornerW c;
    float A[9], ext[3], vel[3], m, inv_dx, sx, sy;
    DEV void mp(int r, float* o) const // mass and momentum
    {
        const float wx = c.wx[r & 1], wy = c.wy[(r >> 1) & 1], wz = c.wz[r >> 2];
        float wm = wx * wy * wz * m;
        o[0] = wm;
        o[1] = wm * vel[0];
        o[2] = wm * vel[1];
        o[3] = wm * vel[2];
    }
    DEV void dp(int r, float* o) const // internal, external and contact impulse
    {
        const float wx = c.wx[r & 1], wy = c.wy[(r >> 1) & 1], wz = c.wz[r >> 2];
        float w = wx * wy * wz;
        float g0 = ((r & 1) ? -sx : sx) * wy * wz;
        float g1 = ((r & 2) ? -sy : sy) * wx * wz;
        float g2 = ((r & 4) ? inv_dx : -inv_dx) * wx * wy;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            float f = A[3 * a] * g0 + A[3 * a + 1] * g1 + A[3 * a + 2] * g2 + w * ext[a];
            o[a] = w != 0.0f ? f : 0.0f;
        }
    }
    // The sums over the cell's particles for the lane's corner: impulses first (their
    // butterfly then runs while fewer values are live)
    DEV void sums(float (&d)[3], float (&q)[4]) const
    {
        reduce_scatter8<3>([&](int r, float* o) { dp(r, o); }, d);
        reduce_scatter8<4>([&](int r, float* o) { mp(r, o); }, q);
    }
};

// Stress and external impulses of the lane's particle, ready to scatter (a lane without
// a particle adds zeros)
template <int MAT>
DEV void scatter_setup(const SceneK& S, const SceneD& D, const Local& loc, int p, bool valid, bool rig, uint32_t code,
                       const float* H, const float* Lg, const float* Gp, const float* t, int j, Scatter& C)
{
    const float dt = S.dt;
    float m = 0.0f, V0 = 0.0f;
    C.c = corner_table(t, j);
    C.inv_dx = S.inv_dx;
    C.sx = (j & 1) ? S.inv_dx : -S.inv_dx;
    C.sy = (j & 2) ? S.inv_dx : -S.inv_dx;
    for (int a = 0; a < 3; a++) C.vel[a] = C.ext[a] = 0.0f;
    if (valid) {
        // (loaded here, not with the rest: in flight during the stress)
        float jr[3] = {0.0f, 0.0f, 0.0f}, jm[3] = {0.0f, 0.0f, 0.0f};
        loc.get(D.v, p, C.vel);
        m = S.m_uniform ? S.m0 : *loc.one(D.m, p);
        V0 = S.v_uniform ? S.V0 : *loc.one(D.V0, p);
        const float E = S.e_uniform ? S.E0 : *loc.one(D.E, p);
        if (rig) loc.get(D.Jrig, p, jr); // floor and tool impulses of this substep (k_rigid)
        if (S.material_contact && (code & TL_CAND_BIT)) loc.get(D.Jmat, p, jm);
        particle_stress<MAT>(S, D, E, H, Lg, Gp, C.A);
        C.ext[0] = (jr[0] + jm[0]) + dt * m * S.gx;
        C.ext[1] = (jr[1] + jm[1]) + dt * m * S.gy;
        C.ext[2] = (jr[2] + jm[2]) + dt * m * S.gz;
    } else {
        for (int a = 0; a < 9; a++) C.A[a] = 0.0f;
    }
    const float sA = -dt * V0;
#pragma unroll
    for (int a = 0; a < 9; a++) C.A[a] *= sA;
    C.m = valid ? m : 0.0f;
}

// --------------------------------------------------------------- one-code bricks
// Most bricks lie away from every cut: all particles of the 27 bricks around them hold
// one side code.  The nodes of such a brick's box then hold one slot each, number 0, in
// every table, so P2G and G2P need no slot tables there: a box value is indexed by its
// node, the coupling is the identity, and the sum of a node over the 8 parity classes
// reads 8 known places (one cell of each class touches a node) instead of taking the
// classes one after another.  The sums keep the order of the general path, so a
// brick's results are bitwise the same on either path.  Box of 14.2M particles with three
// cuts (about a quarter of the bricks near one): P2G 746 -> 570 us, G2P 598 -> 422 us; a
// block of 4 bricks, where one workgroup's chain is all: 13.0 -> 8.6 and 11.7 -> 7.1 us.

// Whether brick (bx, by, bz) is such a brick; every wave decides by itself from the
// same words, without a barrier.  nb: in lanes 0..26 the active index of the brick at
// offset (l % 3 - 1, l / 3 % 3 - 1, l / 9 - 1), -1 if it holds no particle.  STAMP: also
// require that no label pass changed the codes of these bricks since the last G2P
// (`changed` false: the pending re-scatter sums then have the same slots).
template <bool STAMP>
DEV bool one_code(const SceneK& S, const SceneD& D, int bx, int by, int bz, int& nb, bool& changed)
{
    const int l = threadIdx.x & 63;
    nb = -1;
    uint32_t key = 0u;
    bool ch = false;
    if (l < 27) {
        const int x = bx + l % 3 - 1, y = by + (l / 3) % 3 - 1, z = bz + l / 9 - 1;
        if (x >= 0 && y >= 0 && z >= 0 && x < S.cbx && y < S.cby && z < S.cbz) {
            const int b = (z * S.cby + y) * S.cbx + x;
            nb = D.bact[b];
            key = D.bkey[b];
            if (STAMP) ch = D.bdirty[b] == D.ctr[0];
        }
    }
    changed = STAMP && __any(nb >= 0 && ch);
    const uint32_t own = __builtin_amdgcn_readlane(key, 13);
    return own != TL_CC_MIXED && !changed && __all(nb < 0 || key == own);
}

#define TL_ONE_PLACES (TL_WG + 1) // a wave's 64 (cell, corner) sums for 8 classes, and a zero

// Where node bn finds its sum of class w = (px, py, pz): of the two cells that touch it
// along an axis one has parity p; place = wave p bits << 6 | lane bits of the cell's i
// and the corner's j (lane layout of Lane).  Classes without a cell of the brick there
// read the zero at place TL_WG.  A table, 16 bytes per node (forming the 8 places took
// about 60 instructions).
struct PlaceTable {
    uint16_t at[TL_WG / 4][8];
    constexpr PlaceTable() : at()
    {
        for (int bn = 0; bn < TL_WG / 4; bn++)
            for (int w = 0; w < 8; w++) {
                const int N[3] = {bn % 5, (bn / 5) % 5, bn / 25};
                const int cell_bit[3] = {2, 3, 5}, corner_bit[3] = {0, 1, 4};
                int s = 0;
                bool in = bn < TL_BOXN;
                for (int a = 0; a < 3; a++) {
                    const int p = (w >> a) & 1, c = (N[a] ^ p) & 1, cell = N[a] - c; // corner bit, cell
                    if (cell < 0 || cell > 3) in = false;
                    s |= ((cell >> 1) << cell_bit[a]) | (c << corner_bit[a]) | (p << (6 + a));
                }
                at[bn][w] = (uint16_t)(in ? s : TL_WG);
            }
    }
};
static __device__ const PlaceTable k_places __attribute__((aligned(16))) = PlaceTable();

struct NodePlaces {
    uint4 t;
    DEV void set(int bn) { t = *(const uint4*)k_places.at[bn]; }
    DEV int operator()(int w) const
    {
        const uint32_t x = w < 2 ? t.x : w < 4 ? t.y : w < 6 ? t.z : t.w;
        return (w & 1) ? (int)(x >> 16) : (int)(x & 0xFFFFu);
    }
};

// Rounds of 8 particles per cell that the cells of this wave need; the largest of the
// block's waves (after the barrier that follows put) is the brick's.
DEV void put_rounds(const Lane& L, int* s_rw)
{
    int r = 0;
    while (__any(L.count > 8 * r)) r++;
    if (L.lane == 0) s_rw[L.w] = r;
}

DEV int get_rounds(const int* s_rw)
{
    int r = s_rw[0];
#pragma unroll
    for (int w = 1; w < 8; w++) r = max(r, s_rw[w]);
    return r;
}

// P2G of a one-code brick.  s_v: the box's remapped velocities (float4 per node); s_part:
// TL_ONE_PLACES places of 8 floats.
template <int MAT, bool SPLIT, bool FRAC>
DEV void p2g_one(const SceneK& S, const SceneD& D, int bi, const int4 info, int nb, KA_Args A, bool fp, float* s_v,
                 float* s_part, int* s_rw)
{
    const int tid = threadIdx.x, bn = tid >> 2, u = tid & 3;
    const Local loc(S, D, info.x);
    Contrib con;
    con.set(S, nb, tid);
    Gather<4> G;
    if (fp) G.load(D.rs, con, 0, true);
    Lane L = lane_at(tid);
    lane_cell(D, info.x, L);
    const bool rig = A.do_p2g && (S.floor_on || D.tinfo[1]) && D.brig[info.x] != 0;
    int p = L.beg;
    bool valid = lane_particle(D, bi, false, L, 0, p);
    float t[3] = {0.0f, 0.0f, 0.0f}, H[9];
    uint32_t code = 0;
    auto load_particle = [&]() {
        cell_position<FRAC>(S, D, loc, info, L, p, t);
        code = *loc.one(D.code, p);
        loc.get9(D.H, p, H);
    };
    if (valid) load_particle();
    put_rounds(L, s_rw);
    if (tid < 8) s_part[TL_WG * 8 + tid] = 0.0f;
    if (fp) { // node velocities v~ = p~ / m (Eq. 8 with one slot: no exchange)
        float acc[4];
        G.sum(acc);
        const float im = acc[0] > 0.0f ? 1.0f / acc[0] : 0.0f;
        const float pu = u == 0 ? acc[1] : u == 1 ? acc[2] : acc[3];
        if (bn < TL_BOXN) s_v[tid] = pu * im;
    }
    lds_barrier();
    const int rounds = get_rounds(s_rw);
    float sum[2] = {0.0f, 0.0f};
    for (int r = 0; r < rounds; r++) {
        const int tl = late(tid);
        L = lane_at(tl);
        if (r > 0) {
            lane_cell(D, info.x, L);
            valid = lane_particle(D, bi, false, L, r, p);
            if (valid) load_particle();
        }
        if (!valid) t[0] = t[1] = t[2] = 0.0f;
        float Lg[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}; // dF/dt of the update
        float Gp[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        const float4* vb = (const float4*)s_v + box_index(L.cxl, L.cyl, L.czl);
        if (valid) {
            if (fp) {
                grad_of(S, t, [&](int k) { return vb[(k & 1) + 5 * ((k >> 1) & 1) + 25 * (k >> 2)]; }, Lg);
                store_F(D, loc, p, S.dt, Lg, !A.do_p2g, H, code);
            }
            plastic_rate<MAT>(S, D, loc, p, fp, H, Lg, Gp);
        }
        if (!A.do_p2g) continue;
        Scatter C;
        scatter_setup<MAT>(S, D, loc, p, valid, rig, code, H, Lg, Gp, t, L.j, C);
        float dp[3], mp[4];
        C.sums(dp, mp);
        if (r > 0) lds_barrier(); // the places of the last round have been read
        float4* pl = (float4*)(s_part + tl * 8);
        pl[0] = make_float4(mp[0], mp[1], mp[2], mp[3]);
        pl[1] = make_float4(dp[0], dp[1], dp[2], 0.0f);
        lds_barrier();
        NodePlaces np;
        np.set(late(tid) >> 2);
        if (bn < TL_BOXN)
#pragma unroll
            for (int w = 0; w < 8; w++) {
                const float2 c = *(const float2*)(s_part + np(w) * 8 + 2 * u);
                sum[0] += c.x;
                sum[1] += c.y;
            }
    }
    if (!A.do_p2g) return;
    if (SPLIT && tid == 0) D.xp2g[bi] = 0;
    if (bn < TL_BOXN) *(float2*)(D.p2g + (size_t)bi * (unsigned)(S.scap * TL_BOXN * 8) + 2 * tid) = make_float2(sum[0], sum[1]);
}

// ------------------------------------------------- rounds of bricks with several codes
#define TL_NO_SLOT 0xFFFFu

// The slots of the 8 corners of a lane's cell, from the wave's places of s_slot (the
// lane of corner j found the slot of its own corner): corner k at bits 16 (k & 3) of
// word k >> 2.
struct CellSlots {
    unsigned long long w[2];
    DEV void read(const uint16_t* s_slot, int tid)
    {
        const int b = tid & ~0x13; // j = 0 of the lane's cell
        w[0] = *(const unsigned long long*)(s_slot + b);
        w[1] = *(const unsigned long long*)(s_slot + b + 16);
    }
    DEV int operator()(int k) const { return (int)(((k & 4 ? w[1] : w[0]) >> (16 * (k & 3))) & 0xFFFFu); }
};

// Every 8-lane group of a round holds particles of one code (bricks with a mixed cell are
// processed in same-code groups): lane j looks the slot of corner j of its cell up, once
// for the whole group, and writes it to its place.  A group without particles, or a
// failed lookup, has none.  The launches of a mid-size scene last as long as these bricks
// do: 183k particles on a cut, P2G 29.2 -> 24.0 us, G2P 26.5 -> 21.4 us.
DEV void find_corner_slot(const SceneD& D, const BoxTab& T, const Lane& L, int tid, bool valid, uint32_t key,
                          uint16_t* s_slot)
{
    const int leader = L.lane & ~0x13; // j = 0 of the lane's cell
    const uint32_t lkey = __shfl(key, leader, 64);
    const bool gvalid = __shfl((int)valid, leader, 64) != 0;
    if (__any(valid && key != lkey) && L.lane == 0) atomicOr(D.status, TL_ST_LOOKUP);
    int sl = TL_NO_SLOT;
    if (gvalid) {
        const int bn = box_index(L.cxl + (L.j & 1), L.cyl + ((L.j >> 1) & 1), L.czl + ((L.j >> 2) & 1));
        const int f = find_slot(T, bn, lkey);
        if (f < 0)
            atomicOr(D.status, TL_ST_LOOKUP);
        else
            sl = f;
    }
    s_slot[tid] = (uint16_t)sl;
}

// Adds a round's places to the sums of the slots of a node's owner lane (components C u
// .. C u + C - 1): per slot the 8 classes in order after the sums of the rounds before.
// Sums of earlier rounds wait in s_acc (Q components per slot); the last round's go to
// the brick's partial [slot][box node][4 C].
template <int C, int Q>
DEV void add_places(const NodePlaces& np, int meta, int bn, int u, const float* s_part, const uint16_t* s_slot,
                    float* s_acc, bool first, bool last, float* __restrict__ part)
{
    float v[8][C];
    int sl[8];
#pragma unroll
    for (int w = 0; w < 8; w++) {
        const int at = np(w);
        sl[w] = s_slot[at];
#pragma unroll
        for (int q = 0; q < C; q++) v[w][q] = s_part[at * 4 * C + C * u + q];
    }
    const int c = tab_count(meta), b0 = tab_base(meta);
    for (int s = 0; s < c; s++) {
        float sum[C];
        float* wait = s_acc + (b0 + s) * Q + C * u;
#pragma unroll
        for (int q = 0; q < C; q++) sum[q] = (first || C * u + q >= Q) ? 0.0f : wait[q];
#pragma unroll
        for (int w = 0; w < 8; w++)
#pragma unroll
            for (int q = 0; q < C; q++) sum[q] += sl[w] == b0 + s ? v[w][q] : 0.0f;
        if (last) {
            float* out = part + ((size_t)s * TL_BOXN + bn) * 4 * C + C * u;
#pragma unroll
            for (int q = 0; q < C; q++) out[q] = sum[q];
        } else {
#pragma unroll
            for (int q = 0; q < C; q++)
                if (C * u + q < Q) wait[q] = sum[q];
        }
    }
}

// Word of a split brick in xp2g and xrs, written by its second workgroup: 1 + what the
// records of its second box, `boxes` further on, are away from those of its first, modulo
// 2^32.  Never 0: distances are multiples of a box.
DEV int split_offset(const SceneK& S, int boxes)
{
    return (int)((unsigned)boxes * (unsigned)(S.scap * TL_BOXN) + 1u);
}

// MAT 0: Neo-Hookean only; MAT 1: the scene's material (Neo-Hookean or
// fixed-corotated) with Newtonian viscosity.
// part 0 takes the brick's first same-code round (all rounds unless the brick is
// split), part 1 the later rounds of a split brick (a brick whose cells hold two
// codes and need more than one round): the two run as separate workgroups, each
// with its own box partial (box: its index in p2g or p2g_x), so that such bricks do not
// lengthen the launch.
template <int MAT, bool SPLIT, bool FRAC>
DEV void p2g_body(const SceneK& S, const SceneD& D, int bi, KA_Args A, int part, int box)
{
    __shared__ BoxTab Tc;
    __shared__ BoxTab Tr;
    __shared__ __align__(16) float s_vt[(TL_BOX_SLOTS + 1) * 4];  // v~ of the slots, and a zero
    __shared__ __align__(16) float s_part[TL_ONE_PLACES * 8];      // first the node sums of the re-scatter
    __shared__ __align__(16) float s_acc[TL_BOX_SLOTS * 7];
    __shared__ __align__(8) uint16_t s_cs[TL_ONE_PLACES + 7], s_cr[TL_ONE_PLACES + 7];
    __shared__ int s_rw[8];
    float* const s_rsum = s_part;
    static_assert(TL_ONE_PLACES * 8 >= TL_BOX_SLOTS * 4, "node sums in the places");

    const int nround = SPLIT ? D.bround[bi] : 0; // rounds of a brick with a mixed cell, else 0
    if (SPLIT && part == 1 && nround <= 1) return;
    const int4 info = D.binfo[bi];
    const int brick = info.x, bx = info.y, by = info.z, bz = info.w;
    const bool fp = D.ctr[1] != 0; // F update of the last substep pending
    int nbv;
    bool changed;
    if (one_code<true>(S, D, bx, by, bz, nbv, changed)) {
        p2g_one<MAT, SPLIT, FRAC>(S, D, bi, info, nbv, A, fp, s_vt, s_part, s_rw);
        return;
    }
    const bool grouped = D.bmixed[brick] != 0; // a cell holds two codes: same-code groups
    // (all mixed bricks split, or none: the decision does not depend on list order)
    const bool split = SPLIT && grouped && nround > 1 && S.xcap > 0 && D.ctr[3] <= S.xcap;
    const int r0 = part; // first round of this workgroup
    const int tid = threadIdx.x, bn = tid >> 2, u = tid & 3;
    const Local loc(S, D, brick);
    const bool use_r = fp; // finalize v~ (tables rs)
    // separate P2G tables, where a label pass changed the codes around (the two buffers
    // agree elsewhere)
    const bool use_c = A.do_p2g && ((A.tabs_differ && fp && changed) || !fp);
    const bool xg_rs = SPLIT && D.xg[0] != 0; // the last G2P split bricks: their second re-scatter sums

    // ---- phase 1: counts, cell index, codes and partials of the own node, particle loads
    BoxCounts nr, nc;
    if (use_r) nr.load(S, D.cnt[A.rsb], bx, by, bz);
    if (use_c) nc.load(S, D.cnt[A.cur], bx, by, bz);
    Lane L = lane_at(tid);
    lane_cell(D, brick, L);
    // floor/tool impulses were computed for this brick by k_rigid
    const bool rig = A.do_p2g && (S.floor_on || D.tinfo[1]) && D.brig[brick] != 0;
    int p = L.beg;
    bool valid = lane_particle(D, bi, grouped, L, r0, p);
    float t[3] = {0.0f, 0.0f, 0.0f}, H[9];
    uint32_t code = 0;
    auto load_particle = [&]() {
        cell_position<FRAC>(S, D, loc, info, L, p, t);
        code = *loc.one(D.code, p);
        loc.get9(D.H, p, H);
    };
    int mr = 0, mc = 0;
    const int total_r = use_r ? nr.scan(Tr, bn, mr) : 0;
    const int total_c = use_c ? nc.scan(Tc, bn, mc) : total_r;
    if (total_r > TL_BOX_SLOTS || total_c > TL_BOX_SLOTS) {
        if (tid == 0) atomicOr(D.status, TL_ST_BOX);
        return;
    }
    if (bn >= TL_BOXN) mr = mc = 0;
    const long long gid = bn < TL_BOXN ? box_gid(S, bx, by, bz, bn % 5, (bn / 5) % 5, bn / 25) : -1;
    Contrib C;
    C.set(S, nbv, tid);
    const int cr = tab_count(mr), br = tab_base(mr);
    Gather<4> g0, g1;
    uint32_t pre_r = 0, pre_c = 0;
    if (use_r) {
        pre_r = codes_pre(S, D.scode[A.rsb], mr, gid, u);
        g0.load(D.rs, C, 0, cr > 0);
        g1.load(D.rs, C, 1, cr > 1);
    }
    if (use_c) pre_c = codes_pre(S, D.scode[A.cur], mc, gid, u);
    if (valid) load_particle();
    put_rounds(L, s_rw);
    if (tid < 8) s_part[TL_WG * 8 + tid] = 0.0f;
    if (tid < 4) s_vt[TL_BOX_SLOTS * 4 + tid] = 0.0f;
    if (tid == 0) s_cs[TL_WG] = TL_NO_SLOT;
    // ---- phase 2: re-scatter sums of the own node, coupling, v~ (Eq. 8, MUSL)
    if (use_r) {
        codes_put(S, D.scode[A.rsb], Tr, mr, gid, u, pre_r);
        for (int s = 0; s < cr; s += 2) {
            if (s > 0) {
                g0.load(D.rs, C, s, true);
                g1.load(D.rs, C, s + 1, s + 1 < cr);
            }
            if (xg_rs) {
                g0.add(D.rs_x, D.xrs, C, s);
                if (s + 1 < cr) g1.add(D.rs_x, D.xrs, C, s + 1);
            }
            float a0[4], a1[4];
            g0.sum(a0);
            g1.sum(a1);
            if (cr == 1) { // one slot: no exchange
                const float im = a0[0] > 0.0f ? 1.0f / a0[0] : 0.0f;
                s_vt[br * 4 + u] = (u == 0 ? a0[1] : u == 1 ? a0[2] : a0[3]) * im;
            } else {
                s_rsum[(br + s) * 4 + u] = u == 0 ? a0[0] : u == 1 ? a0[1] : u == 2 ? a0[2] : a0[3];
                if (s + 1 < cr) s_rsum[(br + s + 1) * 4 + u] = u == 0 ? a1[0] : u == 1 ? a1[1] : u == 2 ? a1[2] : a1[3];
            }
        }
        wave_lds_fence();
        if (cr > 1 && u < 3)
            couple_component<4>(Tr, br, cr, s_rsum, 1 + u, [&](int sl, float m, float f) {
                const float im = m > 0.0f ? 1.0f / m : 0.0f;
                s_vt[sl * 4 + u] = f * im;
            });
    }
    if (use_c) codes_put(S, D.scode[A.cur], Tc, mc, gid, u, pre_c);
    lds_barrier();
    const BoxTab& T = use_c ? Tc : Tr;
    const int mt = use_c ? mc : mr;
    const int rounds = (split && part == 0) ? 1 : grouped ? D.bround[bi] : get_rounds(s_rw);
    const float4* const vt = (const float4*)s_vt;

    for (int r = r0; r < rounds; r++) {
        const int tl = late(tid);
        L = lane_at(tl);
        if (r > r0) {
            lane_cell(D, brick, L);
            valid = lane_particle(D, bi, grouped, L, r, p);
            if (valid) load_particle();
        }
        if (!valid) t[0] = t[1] = t[2] = 0.0f;
        const uint32_t key = valid ? slot_key(S, code) : 0u;
        if (r > r0) lds_barrier(); // the places of the last round have been read
        if (A.do_p2g) find_corner_slot(D, T, L, tl, valid, key, s_cs);
        // ---- deformation-gradient update from the remapped velocities (MUSL)
        float Lg[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}; // dF/dt of the update
        float Gp[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (use_r) {
            // particles labelled in this substep's pass use their previous code; their
            // wave looks every corner up by itself
            const bool fresh = __any(valid && (code & TL_PREV_BIT) != 0u);
            const bool same = !use_c && A.do_p2g;
            if (!fresh && !same) find_corner_slot(D, Tr, L, tl, valid, key, s_cr);
            wave_lds_fence();
            CellSlots cs;
            cs.read(same ? s_cs : s_cr, tl);
            if (fresh && valid) {
                const uint32_t kprev = (code & TL_PREV_BIT) ? slot_key(S, D.code_prev[p]) : key;
                auto half = [&](int h) {
                    unsigned long long x = 0;
#pragma unroll 1
                    for (int k = 4 * h + 3; k >= 4 * h; k--) {
                        float wx, wy, wz;
                        corner_weights(t, k, wx, wy, wz);
                        int sl = TL_NO_SLOT;
                        if (wx * wy * wz != 0.0f) {
                            const int f = find_slot(
                                Tr, box_index(L.cxl + (k & 1), L.cyl + ((k >> 1) & 1), L.czl + (k >> 2)), kprev);
                            if (f < 0)
                                atomicOr(D.status, TL_ST_LOOKUP);
                            else
                                sl = f;
                        }
                        x = (x << 16) | (unsigned)sl;
                    }
                    return x;
                };
                cs.w[0] = half(0);
                cs.w[1] = half(1);
            }
            if (valid) {
                grad_of(S, t, [&](int k) { return vt[cs(k) < TL_BOX_SLOTS ? cs(k) : TL_BOX_SLOTS]; }, Lg);
                store_F(D, loc, p, S.dt, Lg, !A.do_p2g, H, code);
            }
        }
        if (valid) plastic_rate<MAT>(S, D, loc, p, use_r, H, Lg, Gp);
        if (!A.do_p2g) continue;
        Scatter W;
        scatter_setup<MAT>(S, D, loc, p, valid, rig, code, H, Lg, Gp, t, L.j, W);
        float dp[3], mp[4];
        W.sums(dp, mp);
        float4* pl = (float4*)(s_part + tl * 8);
        pl[0] = make_float4(mp[0], mp[1], mp[2], mp[3]);
        pl[1] = make_float4(dp[0], dp[1], dp[2], 0.0f);
        lds_barrier();
        NodePlaces np;
        np.set(late(tid) >> 2);
        if (bn < TL_BOXN)
            add_places<2, 7>(np, mt, bn, u, s_part, s_cs, s_acc, r == r0, r + 1 == rounds,
                          (part ? D.p2g_x : D.p2g) + (size_t)box * (unsigned)(S.scap * TL_BOXN * 8));
    }
    if (!A.do_p2g) return;
    if (SPLIT && tid == 0 && (part || !split)) D.xp2g[bi] = part ? split_offset(S, box - bi) : 0;
}

// --------------------------------------------------------------------------- K_B
// Grid update and G2P kernel (one brick per workgroup): finalize the box from the
// P2G partials (sum over contributing bricks, coupling Eq. 8, velocities Eq. 9),
// PIC/FLIP G2P of v and x (Eq. 17), then the MUSL re-scatter of m_p v_p^{n+1} into
// this brick's partials.  Also records the brick's current AABB and speed bound.

// PIC/FLIP update of the lane's particle from the interpolated increments av and ax;
// joins x^{n+1}, the speed and |u^{n+1} - a| into bb.
DEV void move_particle(const SceneK& S, const SceneD& D, const Local& loc, int p, const float* Xp, const float* v,
                       const float* u, const float* av, const float* ax, const float* ap, float* vn1, float* bb)
{
    const float dt = S.dt, beta = S.beta;
    float *vo = loc.row(D.v, p), *uo = loc.row(D.u, p);
    for (int a = 0; a < 3; a++) {
        vn1[a] = beta * v[a] + av[a];
        float un = u[a] + dt * ax[a];
        vo[a] = vn1[a];
        uo[a] = un;
        float xa = Xp[a] + un;
        bb[a] = fmaxf(bb[a], -xa);
        bb[3 + a] = fmaxf(bb[3 + a], xa);
        bb[7] = fmaxf(bb[7], fabsf(un - ap[a]));
    }
    bb[6] = fmaxf(bb[6], sqrtf(vn1[0] * vn1[0] + vn1[1] * vn1[1] + vn1[2] * vn1[2]));
}

// Brick AABB of x^{n+1} and speed bound (used to skip distant contact work), from each
// lane's bb; a split brick's second workgroup keeps the box of its particles apart
// (brick_aabb joins the two).  With track also the displacement anchor.
DEV void put_box(const SceneK& S, const SceneD& D, int bi, int brick, int part, bool track, const float* ap,
                 const float* bb, float (*s_bb)[8])
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // maxima of 8 values over 64 lanes: three stages that halve the values a lane keeps
    // (its bit chooses which half, the partner gets the other), then three on the one left
    float m4[4], m2[2];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const float send = (lane & 1) ? bb[q] : bb[q + 4], keep = (lane & 1) ? bb[q + 4] : bb[q];
        m4[q] = fmaxf(keep, lane_xor<1>(send));
    }
#pragma unroll
    for (int q = 0; q < 2; q++) {
        const float send = (lane & 2) ? m4[q] : m4[q + 2], keep = (lane & 2) ? m4[q + 2] : m4[q];
        m2[q] = fmaxf(keep, lane_xor<2>(send));
    }
    float m = fmaxf((lane & 4) ? m2[1] : m2[0], lane_xor<4>((lane & 4) ? m2[0] : m2[1]));
    // lane bits 0, 1, 2 now hold value 4 b0 + 2 b1 + b2
    m = fmaxf(m, __shfl_xor(m, 8, 64));
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if (lane < 8) s_bb[w][((lane & 1) << 2) | (lane & 2) | (lane >> 2)] = m;
    lds_barrier();
    if (tid < 7) {
        float val = s_bb[0][tid];
        for (int wv = 1; wv < 8; wv++) val = fmaxf(val, s_bb[wv][tid]);
        (part ? D.aabb_x : D.aabb)[(long long)brick * 8 + tid] = tid < 3 ? -val : val;
        // the next binning's bin edge needs the largest speed bound; the maximum
        // of non-negative floats is taken on their bit patterns (order-independent)
        if (tid == 6 && S.material_contact && val > 0.0f)
            atomicMax(D.hmax + (bi & (TL_HSLOTS - 1)) * TL_HSTRIDE, __float_as_int(val));
    } else if (tid == 7 && track) {
        float dv = s_bb[0][7];
        for (int wv = 1; wv < 8; wv++) dv = fmaxf(dv, s_bb[wv][7]);
        put_anchor(D, bi, brick, part, ap, dv);
    }
}

// G2P of a one-code brick.  s_g: per box node (1 - beta) v^n + dv and v^n + dv (two
// float4); s_part: TL_ONE_PLACES places of 4 floats.
template <bool SPLIT>
DEV void g2p_one(const SceneK& S, const SceneD& D, int bi, const int4 info, int nb, bool track, const float* ap,
                 float* s_g, float* s_part, int* s_rw, float (*s_bb)[8])
{
    const int tid = threadIdx.x, bn = tid >> 2, u4 = tid & 3;
    const Local loc(S, D, info.x);
    const float beta = S.beta;
    Contrib con;
    con.set(S, nb, tid);
    Gather<8> G;
    G.load(D.p2g, con, 0, true);
    Lane L = lane_at(tid);
    lane_cell(D, info.x, L);
    int p = L.beg;
    bool valid = lane_particle(D, bi, false, L, 0, p);
    float Xp[3] = {0.0f, 0.0f, 0.0f}, v[3] = {0.0f, 0.0f, 0.0f}, u[3] = {0.0f, 0.0f, 0.0f};
    auto load_particle = [&]() {
        loc.get(D.X, p, Xp);
        loc.get(D.v, p, v);
        loc.get(D.u, p, u);
    };
    if (valid) load_particle();
    put_rounds(L, s_rw);
    if (tid < 4) s_part[TL_WG * 4 + tid] = 0.0f;
    { // node velocities and increments (Eq. 9; Eq. 8 with one slot: no exchange)
        float acc[7];
        G.sum(acc);
        const float im = acc[0] > 0.0f ? 1.0f / acc[0] : 0.0f;
        const float pu = u4 == 0 ? acc[1] : u4 == 1 ? acc[2] : acc[3];
        const float du = u4 == 0 ? acc[4] : u4 == 1 ? acc[5] : acc[6];
        const float vn = pu * im, dv = du * im;
        if (bn < TL_BOXN) {
            s_g[bn * 8 + u4] = (1.0f - beta) * vn + dv;
            s_g[bn * 8 + 4 + u4] = vn + dv;
        }
    }
    lds_barrier();
    const int rounds = get_rounds(s_rw);
    float sum = 0.0f;
    // box of x^{n+1} (its lower faces negated), speed bound, and the largest |u^{n+1} - a| about the anchor a
    // (for the pair-search skip)
    float bb[8] = {-1e30f, -1e30f, -1e30f, -1e30f, -1e30f, -1e30f, 0.0f, 0.0f};
    for (int r = 0; r < rounds; r++) {
        const int tl = late(tid);
        L = lane_at(tl);
        if (r > 0) {
            lane_cell(D, info.x, L);
            valid = lane_particle(D, bi, false, L, r, p);
            if (valid) load_particle();
        }
        float t[3] = {0.0f, 0.0f, 0.0f};
        float m = 0.0f, vn1[3] = {0.0f, 0.0f, 0.0f};
        if (valid) {
            frac_of(S, Xp, info.y * TL_B + L.cxl, info.z * TL_B + L.cyl, info.w * TL_B + L.czl, t);
            const float4* gb = (const float4*)s_g + 2 * box_index(L.cxl, L.cyl, L.czl);
            float av[3] = {0.0f, 0.0f, 0.0f}, ax[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 8; k++) { // (a zero weight adds zero: node values are finite or unused)
                float wx, wy, wz;
                corner_weights(t, k, wx, wy, wz);
                const float w = wx * wy * wz;
                const int o = 2 * ((k & 1) + 5 * ((k >> 1) & 1) + 25 * (k >> 2));
                const float4 fv = gb[o], fx = gb[o + 1];
                av[0] += w * fv.x;
                av[1] += w * fv.y;
                av[2] += w * fv.z;
                ax[0] += w * fx.x;
                ax[1] += w * fx.y;
                ax[2] += w * fx.z;
            }
            move_particle(S, D, loc, p, Xp, v, u, av, ax, ap, vn1, bb);
            m = S.m_uniform ? S.m0 : *loc.one(D.m, p);
        }
        const float mm = valid ? m : 0.0f;
        const CornerW cw = corner_table(t, L.j);
        float res[4];
        reduce_scatter8<4>(
            [&](int q, float* o) {
                const float wx = cw.wx[q & 1], wy = cw.wy[(q >> 1) & 1], wz = cw.wz[q >> 2];
                float w = wx * wy * wz * mm;
                o[0] = w;
                o[1] = w * vn1[0];
                o[2] = w * vn1[1];
                o[3] = w * vn1[2];
            },
            res);
        if (r > 0) lds_barrier(); // the places of the last round have been read
        *(float4*)(s_part + tl * 4) = make_float4(res[0], res[1], res[2], res[3]);
        lds_barrier();
        NodePlaces np;
        np.set(late(tid) >> 2);
        if (bn < TL_BOXN)
#pragma unroll
            for (int w = 0; w < 8; w++) sum += s_part[np(w) * 4 + u4];
    }
    if (SPLIT && tid == 0) D.xrs[bi] = 0;
    if (bn < TL_BOXN) D.rs[(size_t)bi * (unsigned)(S.scap * TL_BOXN * 4) + tid] = sum;
    put_box(S, D, bi, info.x, 0, track, ap, bb, s_bb);
}

template <bool SPLIT>
DEV void g2p_body(const SceneK& S, const SceneD& D, int bi, int cur, int part, int box)
{
    __shared__ BoxTab T;
    __shared__ __align__(16) float s_grid[(TL_BOX_SLOTS + 1) * 8]; // per slot (1 - beta) v^n + dv, v^n + dv; a zero
    __shared__ __align__(16) float s_work[TL_ONE_PLACES * 4 + TL_BOX_SLOTS * 4];
    __shared__ __align__(8) uint16_t s_cs[TL_ONE_PLACES + 7];
    __shared__ int s_rw[8];
    __shared__ float s_bb[8][8];
    float* const s_sum = s_work;                      // the node sums of nodes with several slots, then
    float* const s_part = s_work;                     // the places of a round and
    float* const s_acc = s_work + TL_ONE_PLACES * 4; // the sums of earlier rounds
    static_assert(TL_ONE_PLACES * 4 + TL_BOX_SLOTS * 4 >= TL_BOX_SLOTS * 7, "node sums in the places");

    const int nround = SPLIT ? D.bround[bi] : 0; // rounds of a brick with a mixed cell, else 0
    if (SPLIT && part == 1 && nround <= 1) return; // (split bricks as in the P2G)
    const int4 info = D.binfo[bi];
    const int brick = info.x, bx = info.y, by = info.z, bz = info.w;
    if (bi == 0 && part == 0 && threadIdx.x == 0) {
        // end of the substep for this scene: next history stamp, F update pending
        // (no other kernel of the substep reads these after this point); whether this
        // G2P splits its mixed bricks (read by the next P2G and box tests)
        D.tstamp[cur] = D.ctr[0]; // (the slot tables in use are up to date)
        D.ctr[0] += 1;
        D.ctr[1] = 1;
        D.ctr[2] += 1;
        if (SPLIT) D.xg[0] = (S.xcap > 0 && D.ctr[3] > 0 && D.ctr[3] <= S.xcap) ? 1 : 0;
    }
    // displacement anchor of this workgroup's particles (pair-search skip), kept for
    // bricks with contact candidates (only candidates can be partners): the centre of
    // the brick's box after the last G2P minus the centre of its particles' reference
    // box.  A split brick's second workgroup reads the first one's record, which that
    // one may rewrite in this launch; either value is a valid anchor, since the spread
    // is measured against the anchor taken.
    const bool track = S.pair_skip && D.bcand[bi] > 0;
    float ap[3] = {0.0f, 0.0f, 0.0f};
    if (track) {
        g2p_anchor(D, D.aabb + (long long)brick * 8, brick, ap);
        for (int a = 0; a < 3; a++) ap[a] = scalar(ap[a]);
    }
    int nbv;
    bool changed;
    if (one_code<false>(S, D, bx, by, bz, nbv, changed)) {
        g2p_one<SPLIT>(S, D, bi, info, nbv, track, ap, s_grid, s_part, s_rw, s_bb);
        return;
    }
    const bool grouped = D.bmixed[brick] != 0; // a cell holds two codes: same-code groups
    // this substep's P2G split its mixed bricks (a scene without split workgroups never)
    const bool xsplit = SPLIT && S.xcap > 0 && D.ctr[3] > 0 && D.ctr[3] <= S.xcap;
    const bool split = grouped && nround > 1 && xsplit;
    const int r0 = part;
    const int tid = threadIdx.x, bn = tid >> 2, u4 = tid & 3;
    const Local loc(S, D, brick);
    const float beta = S.beta;

    // ---- phase 1: counts, cell index, codes and partials of the own node, particle loads
    BoxCounts nc;
    nc.load(S, D.cnt[cur], bx, by, bz);
    Lane L = lane_at(tid);
    lane_cell(D, brick, L);
    int p = L.beg;
    bool valid = lane_particle(D, bi, grouped, L, r0, p);
    float Xp[3] = {0.0f, 0.0f, 0.0f}, v[3] = {0.0f, 0.0f, 0.0f}, u[3] = {0.0f, 0.0f, 0.0f};
    uint32_t code = 0;
    auto load_particle = [&]() {
        loc.get(D.X, p, Xp);
        loc.get(D.v, p, v);
        loc.get(D.u, p, u);
        code = *loc.one(D.code, p);
    };
    int mt = 0;
    const int total = nc.scan(T, bn, mt);
    if (total > TL_BOX_SLOTS) {
        if (tid == 0) atomicOr(D.status, TL_ST_BOX);
        return;
    }
    if (bn >= TL_BOXN) mt = 0;
    const int c = tab_count(mt), b0 = tab_base(mt);
    const long long gid = bn < TL_BOXN ? box_gid(S, bx, by, bz, bn % 5, (bn / 5) % 5, bn / 25) : -1;
    Contrib C;
    C.set(S, nbv, tid);
    const uint32_t pre = codes_pre(S, D.scode[cur], mt, gid, u4);
    Gather<8> g0, g1;
    g0.load(D.p2g, C, 0, c > 0);
    g1.load(D.p2g, C, 1, c > 1);
    if (valid) load_particle();
    put_rounds(L, s_rw);
    if (tid < 8) s_grid[TL_BOX_SLOTS * 8 + tid] = 0.0f;
    if (tid == 0) s_cs[TL_WG] = TL_NO_SLOT;
    // ---- phase 2: P2G sums of the own node, coupling (Eq. 8), v^n and dv (Eq. 9)
    codes_put(S, D.scode[cur], T, mt, gid, u4, pre);
    for (int s = 0; s < c; s += 2) {
        if (s > 0) {
            g0.load(D.p2g, C, s, true);
            g1.load(D.p2g, C, s + 1, s + 1 < c);
        }
        if (xsplit) {
            g0.add(D.p2g_x, D.xp2g, C, s);
            if (s + 1 < c) g1.add(D.p2g_x, D.xp2g, C, s + 1);
        }
        float a0[7], a1[7];
        g0.sum(a0);
        g1.sum(a1);
        if (c == 1) { // one slot: no exchange
            const float im = a0[0] > 0.0f ? 1.0f / a0[0] : 0.0f;
            const float vn = (u4 == 0 ? a0[1] : u4 == 1 ? a0[2] : a0[3]) * im;
            const float dv = (u4 == 0 ? a0[4] : u4 == 1 ? a0[5] : a0[6]) * im;
            s_grid[b0 * 8 + u4] = (1.0f - beta) * vn + dv;
            s_grid[b0 * 8 + 4 + u4] = vn + dv;
        } else {
            float* o = s_sum + (b0 + s) * 7;
            if (u4 == 0)
#pragma unroll
                for (int q = 0; q < 7; q++) o[q] = a0[q];
            if (u4 == 1 && s + 1 < c)
#pragma unroll
                for (int q = 0; q < 7; q++) o[7 + q] = a1[q];
        }
    }
    wave_lds_fence();
    if (c > 1 && u4 < 3) {
        couple_component<7>(T, b0, c, s_sum, 1 + u4, [&](int sl, float m, float f) {
            const float im = m > 0.0f ? 1.0f / m : 0.0f;
            s_grid[sl * 8 + u4] = f * im;
        });
        couple_component<7>(T, b0, c, s_sum, 4 + u4, [&](int sl, float m, float f) {
            const float im = m > 0.0f ? 1.0f / m : 0.0f;
            const float vn = s_grid[sl * 8 + u4], dv = f * im;
            s_grid[sl * 8 + u4] = (1.0f - beta) * vn + dv;
            s_grid[sl * 8 + 4 + u4] = vn + dv;
        });
    }
    lds_barrier();
    const int rounds = (split && part == 0) ? 1 : grouped ? D.bround[bi] : get_rounds(s_rw);
    const float4* const gr = (const float4*)s_grid;
    // box of x^{n+1} (its lower faces negated), speed bound, and the largest |u^{n+1} - a| about the anchor a
    // (for the pair-search skip)
    float bb[8] = {-1e30f, -1e30f, -1e30f, -1e30f, -1e30f, -1e30f, 0.0f, 0.0f};
    for (int r = r0; r < rounds; r++) {
        const int tl = late(tid);
        L = lane_at(tl);
        if (r > r0) {
            lane_cell(D, brick, L);
            valid = lane_particle(D, bi, grouped, L, r, p);
            if (valid) load_particle();
        }
        float t[3] = {0.0f, 0.0f, 0.0f};
        uint32_t key = 0;
        float m = 0.0f, vn1[3] = {0.0f, 0.0f, 0.0f};
        if (valid) {
            frac_of(S, Xp, info.y * TL_B + L.cxl, info.z * TL_B + L.cyl, info.w * TL_B + L.czl, t);
            key = slot_key(S, code);
        }
        if (r > r0) lds_barrier(); // the places of the last round have been read
        find_corner_slot(D, T, L, tl, valid, key, s_cs);
        wave_lds_fence();
        CellSlots cs;
        cs.read(s_cs, tl);
        if (valid) {
            float av[3] = {0.0f, 0.0f, 0.0f}, ax[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 8; k++) { // (a zero weight adds zero: node values are finite)
                float wx, wy, wz;
                corner_weights(t, k, wx, wy, wz);
                const float w = wx * wy * wz;
                const int sl = cs(k) < TL_BOX_SLOTS ? cs(k) : TL_BOX_SLOTS;
                const float4 fv = gr[2 * sl], fx = gr[2 * sl + 1];
                av[0] += w * fv.x;
                av[1] += w * fv.y;
                av[2] += w * fv.z;
                ax[0] += w * fx.x;
                ax[1] += w * fx.y;
                ax[2] += w * fx.z;
            }
            move_particle(S, D, loc, p, Xp, v, u, av, ax, ap, vn1, bb);
            m = S.m_uniform ? S.m0 : *loc.one(D.m, p);
        }
        const float mm = valid ? m : 0.0f;
        const CornerW cw = corner_table(t, L.j);
        float res[4];
        reduce_scatter8<4>(
            [&](int q, float* o) {
                const float wx = cw.wx[q & 1], wy = cw.wy[(q >> 1) & 1], wz = cw.wz[q >> 2];
                float w = wx * wy * wz * mm;
                o[0] = w;
                o[1] = w * vn1[0];
                o[2] = w * vn1[1];
                o[3] = w * vn1[2];
            },
            res);
        *(float4*)(s_part + tl * 4) = make_float4(res[0], res[1], res[2], res[3]);
        lds_barrier();
        NodePlaces np;
        np.set(late(tid) >> 2);
        if (bn < TL_BOXN)
            add_places<1, 4>(np, mt, bn, u4, s_part, s_cs, s_acc, r == r0, r + 1 == rounds,
                          (part ? D.rs_x : D.rs) + (size_t)box * (unsigned)(S.scap * TL_BOXN * 4));
    }
    if (SPLIT && tid == 0 && (part || !split)) D.xrs[bi] = part ? split_offset(S, box - bi) : 0;
    put_box(S, D, bi, brick, part, track, ap, bb, s_bb);
}

// ------------------------------------------------------------- mixed-code bricks
// Per cell of a brick whose codes changed (or of every brick, when forced): the
// one slot key of its particles (or empty / mixed).  A brick with a mixed cell
// gets a group table: each of its cells lists its particles by ascending key
// (input order within a key) in gperm over the cell's range, cut into groups of at
// most 8 same-key particles; P2G and G2P then take one group per cell and round.
DEV void cell_summaries(const SceneK& S, const SceneD& D, int bi, int brick)
{
    __shared__ int s_rounds;
    __shared__ uint32_t s_bor;
    if (threadIdx.x == 0) {
        s_rounds = 1;
        s_bor = 0u;
    }
    __syncthreads();
    bool mixed = false, some = false;
    uint32_t key = 0u, done = TL_CODE_MASK; // cuts with a digit in all particles
    for (int c = threadIdx.x; c < TL_CELLS; c += blockDim.x) {
        const long long cs = (long long)brick * TL_CELLS + c;
        const int b0 = D.cell_start[cs], b1 = D.cell_start[cs + 1];
        if (b1 <= b0) {
            D.ccode[cs] = TL_CC_EMPTY;
            if (S.material_contact) D.cmask[cs] = 0;
            continue;
        }
        const uint32_t c0 = D.code[b0], k0 = slot_key(S, c0);
        done &= c0 | ((c0 & TL_CODE_MASK) >> 15);
        uint32_t orm = k0; // OR of the codes of the cell (material contact candidates)
        uint32_t ks[TL_CKEYS] = {k0, 0u, 0u, 0u};
        int nk = 1;
        bool many = false;
#pragma unroll 4
        for (int p = b0 + 1; p < b1; p++) {
            const uint32_t cp = D.code[p], k = slot_key(S, cp);
            done &= cp | ((cp & TL_CODE_MASK) >> 15);
            orm |= k;
            // distinct keys in ascending order (insertion; at most TL_CKEYS kept)
            bool seen = false;
#pragma unroll
            for (int q = 0; q < TL_CKEYS; q++) seen |= q < nk && ks[q] == k;
            if (seen) continue;
            if (nk == TL_CKEYS) {
                many = true;
                continue;
            }
#pragma unroll
            for (int q = TL_CKEYS - 1; q > 0; q--)
                if (q <= nk && ks[q - 1] > k) {
                    ks[q] = ks[q - 1];
                    ks[q - 1] = k;
                } else if (q == nk) {
                    ks[q] = k;
                }
            nk++;
        }
        const bool cm = nk > 1 || many;
        D.ccode[cs] = !cm ? k0 : (many ? TL_CC_MIXED : (TL_CC_FEW | (uint32_t)nk));
        if (cm && !many)
            for (int q = 0; q < nk; q++) D.ckeys[cs * TL_CKEYS + q] = ks[q];
        if (S.material_contact) D.cmask[cs] = orm;
        if (S.pair_skip && orm) atomicOr(&s_bor, orm);
        some = true;
        key = k0;
        mixed |= cm;
    }
    // the key of a one-code brick: the first wave holds its cells, one per lane
    if (threadIdx.x < TL_CELLS) {
        const unsigned long long cells = __ballot(some);
        const uint32_t k0 = __shfl(key, cells ? __ffsll(cells) - 1 : 0, 64);
        key = __any(some && key != k0) ? TL_CC_MIXED : k0;
        for (int o = 32; o >= 1; o >>= 1) done &= (uint32_t)__shfl_xor((int)done, o, 64);
    }
    const int m = __syncthreads_or(mixed);
    if (threadIdx.x == 0) {
        if (S.pair_skip) D.bor[brick] = s_bor; // (the barrier above ordered the LDS ORs)
        D.bkey[brick] = m ? TL_CC_MIXED : key;
        D.ball[brick] = done & 0x7FFFu;
        D.bmixed[brick] = m;
        if (!m) {
            D.bround[bi] = 0; // no split workgroup for this brick
        } else if (S.xcap > 0 && !D.xin[bi]) { // (codes only gain digits: once mixed, always mixed)
            D.xin[bi] = 1;
            D.xlist[atomicAdd(D.ctr + 3, 1)] = bi;
        }
    }
    if (!m) return;
    if (threadIdx.x < TL_CELLS) {
        const int c = threadIdx.x; // cell slot w * 8 + i
        const long long cs = (long long)brick * TL_CELLS + c;
        const int b0 = D.cell_start[cs], b1 = D.cell_start[cs + 1];
        int* meta = D.gmeta + ((long long)bi * TL_CELLS + c) * TL_GMAX;
        const int n = b1 - b0;
        // the keys of the cell's first TL_KC particles, loaded once (registers: every
        // index below is a compile-time constant); the rest are read when needed
        constexpr int TL_KC = 8;
        uint32_t kc[TL_KC];
#pragma unroll
        for (int q = 0; q < TL_KC; q++) kc[q] = q < n ? slot_key(S, D.code[b0 + q]) : 0u;
        int ng = 0, pos = 0, gstart = 0;
        uint32_t last = 0;
        bool first = true;
        auto place = [&](int p) {
            D.gperm[b0 + pos] = p;
            pos++;
            if (pos - gstart == 8) {
                if (ng < TL_GMAX) meta[ng] = (gstart << 4) | 8;
                ng++;
                gstart = pos;
            }
        };
        while (pos < n) {
            uint32_t kmin = 0xFFFFFFFFu; // smallest key above the last one
#pragma unroll
            for (int q = 0; q < TL_KC; q++)
                if (q < n && (first || kc[q] > last) && kc[q] < kmin) kmin = kc[q];
            for (int q = TL_KC; q < n; q++) {
                const uint32_t k = slot_key(S, D.code[b0 + q]);
                if ((first || k > last) && k < kmin) kmin = k;
            }
            gstart = pos;
#pragma unroll
            for (int q = 0; q < TL_KC; q++)
                if (q < n && kc[q] == kmin) place(b0 + q);
            for (int q = TL_KC; q < n; q++)
                if (slot_key(S, D.code[b0 + q]) == kmin) place(b0 + q);
            if (pos > gstart) {
                if (ng < TL_GMAX) meta[ng] = (gstart << 4) | (pos - gstart);
                ng++;
            }
            last = kmin;
            first = false;
        }
        for (int g = ng; g < TL_GMAX; g++) meta[g] = 0;
        if (ng > TL_GMAX) atomicOr(D.status, TL_ST_BOX);
        atomicMax(&s_rounds, ng < TL_GMAX ? ng : TL_GMAX);
    }
    __syncthreads();
    if (threadIdx.x == 0) D.bround[bi] = s_rounds;
}

DEV void mixed_body(const SceneK& S, const SceneD& D, int bi, int force)
{
    const int brick = D.active[bi];
    if (!force && D.bdirty[brick] != D.ctr[0]) return;
    cell_summaries(S, D, bi, brick);
}

// ------------------------------------------------------------------------ labels
// Side-label pass (Eqs. 3, 4, 6) with the predicates of tlmpm_band.h (FP64, a
// fixed evaluation order, no contraction: the order of the CPU reference), on
// x = X + u and v.  One brick per workgroup; a brick whose box cannot meet any band
// exits at once.
// Blade of tool b at this substep (TL_TOOL_ADVANCE translates the edge).
DEV DevBlade blade_at(const DevTool& T, double jdt)
{
    DevBlade B = T.b;
    if (T.flags & TL_TOOL_ADVANCE)
        for (int a = 0; a < 3; a++) B.xe[a] = T.b.xe[a] + jdt * T.b.ve[a];
    return B;
}

// Whether the band of tool b can give a digit to a particle of active brick bi (= brick)
// this substep: it labels, some particle has no digit of its cut yet (an assigned digit
// never changes), and its band can meet the brick's box (brick_near_band, conservative).
DEV bool band_near(const SceneK& S, const SceneD& D, int bi, int brick, int b, double jdt)
{
    if (b >= D.tinfo[0] || !(D.tools[b].flags & TL_TOOL_LABELS)) return false;
    if ((D.ball[brick] >> D.tools[b].b.cut) & 1u) return false;
    float bb[7];
    brick_aabb(S, D, bi, brick, bb);
    return brick_near_band(bb, blade_at(D.tools[b], jdt), S.dt_d);
}

// Label pass of one brick within reach of the blades of mask m (whole block).
DEV void labels_brick(const SceneK& S, const SceneD& D, int bi, int brick, int m, double jdt)
{
    const bool mark_prev = D.ctr[1] != 0; // keep the codes the pending F update needs
    __shared__ DevBlade s_bl[TL_MAX_TOOLS];
    __shared__ int s_nb;
    if (threadIdx.x == 0) {
        int nb = 0;
        for (int b = 0; b < TL_MAX_TOOLS; b++)
            if ((m >> b) & 1) s_bl[nb++] = blade_at(D.tools[b], jdt);
        s_nb = nb;
    }
    __syncthreads();
    const int beg = D.cell_start[(long long)brick * TL_CELLS], end = D.cell_start[(long long)(brick + 1) * TL_CELLS];
    bool any = false;
    for (int p = beg + threadIdx.x; p < end; p += blockDim.x) {
        uint32_t code = D.code[p];
        uint32_t nc = code;
        double x[3] = {(double)D.X[at3(p, 0)] + (double)D.u[at3(p, 0)], (double)D.X[at3(p, 1)] + (double)D.u[at3(p, 1)],
                       (double)D.X[at3(p, 2)] + (double)D.u[at3(p, 2)]};
        double v[3] = {(double)D.v[at3(p, 0)], (double)D.v[at3(p, 1)], (double)D.v[at3(p, 2)]};
        for (int b = 0; b < s_nb; b++) {
            const DevBlade& B = s_bl[b];
            uint32_t bit1 = 1u << B.cut, bit2 = 1u << (15 + B.cut);
            if (nc & (bit1 | bit2)) continue; // persistence: an assigned digit never changes
            int dg = label_digit(x, v, B, S.dt_d);
            if (dg == 1) nc |= bit1;
            if (dg == 2) nc |= bit2;
        }
        if (nc != code) {
            if (mark_prev && !(code & TL_PREV_BIT)) {
                D.code_prev[p] = code & TL_CODE_MASK;
                nc |= TL_PREV_BIT;
            }
            D.code[p] = nc;
            any = true;
        }
    }
    if (__syncthreads_or(any)) {
        // label-change flags carry the substep stamp: no clearing pass needed
        if (threadIdx.x == 0) D.bdirty[brick] = D.ctr[0];
        __syncthreads(); // the new codes of the brick, visible to the whole block
        cell_summaries(S, D, bi, brick);
    }
}

// Label pass of nb bricks per workgroup (as rigid_group): four lanes per brick test the
// bands at once, then the workgroup labels the bricks within reach one after another.
template <class Items>
DEV void labels_group(const Items& I, int w, int G, int nb)
{
    __shared__ int s_m[TL_GROUP];
    const int t = threadIdx.x;
    if (t < nb * TL_MAX_TOOLS) {
        const int i = w + (t / TL_MAX_TOOLS) * G;
        bool nr = false;
        if (i < I.n) {
            const SceneK& S = I.scene(i);
            const SceneD& D = I.data(i);
            const int bi = I.brick(i);
            nr = band_near(S, D, bi, D.active[bi], t % TL_MAX_TOOLS, (double)D.ctr[2] * S.dt_d);
        }
        const unsigned long long all = __ballot(nr);
        if (t % TL_MAX_TOOLS == 0) s_m[t / TL_MAX_TOOLS] = (int)((all >> (t & 60)) & 0xF);
    }
    __syncthreads();
    for (int k = 0; k < nb; k++) {
        const int m = s_m[k];
        if (!m) continue;
        const int i = w + k * G;
        const SceneK& S = I.scene(i);
        const SceneD& D = I.data(i);
        const int bi = I.brick(i);
        labels_brick(S, D, bi, D.active[bi], m, (double)D.ctr[2] * S.dt_d);
        __syncthreads(); // the brick's LDS words are reused by the next one
    }
}

// Bricks per workgroup of these two passes for n bricks (a batch: work items): one each
// below 4096, where a workgroup per brick starts about as fast as the tests run; beyond
// that most workgroups only test, and bricks share them so that their number stays near
// 2048, up to TL_GROUP.  2.5k bricks: labels 45 us in groups of 16, 17 us one each.  28k
// bricks in groups of 14: labels 48 us with one lane testing all bands, 42 us with a lane
// per band; rigid contact 120 us one each, 66 us in groups.
static int group_of(int n) { return n < 4096 ? 1 : n / 2048 > TL_GROUP ? TL_GROUP : n / 2048; }

__global__ __launch_bounds__(256) void k_labels(SceneK S, SceneD D, int nb)
{
    labels_group(BricksOfScene{S, D, D.n_active}, blockIdx.x, gridDim.x, nb);
}
__global__ __launch_bounds__(256) void k_labels_b(const SceneK* __restrict__ Ks, const SceneD* __restrict__ Ds,
                                                    const int2* __restrict__ it, int n, int nb)
{
    labels_group(BricksOfBatch{Ks, Ds, it, n}, blockIdx.x, gridDim.x, nb);
}
__global__ __launch_bounds__(256) void k_rigid(SceneK S, SceneD D, int nb)
{
    rigid_group(BricksOfScene{S, D, D.n_active}, blockIdx.x, gridDim.x, nb);
}
__global__ __launch_bounds__(256) void k_rigid_b(const SceneK* __restrict__ Ks, const SceneD* __restrict__ Ds,
                                                   const int2* __restrict__ it, int n, int nb)
{
    rigid_group(BricksOfBatch{Ks, Ds, it, n}, blockIdx.x, gridDim.x, nb);
}

// The label pass and rigid contact of one scene in one launch: blocks below nl take the
// label pass of a brick, the others its rigid contact.  Rigid contact reads only the last
// substep's motion, the tools and the cutting progress, none of which the label pass
// writes, and the label pass reads nothing rigid contact writes.
__global__ __launch_bounds__(256) void k_labels_rigid(SceneK S, SceneD D, int nl)
{
    const BricksOfScene I{S, D, D.n_active};
    if ((int)blockIdx.x < nl)
        labels_group(I, blockIdx.x, nl, 1);
    else
        rigid_group(I, blockIdx.x - nl, nl, 1);
}

// --------------------------------------------------------------- small kernels
// D := 0 for a new cut (Sec. III-A), over particle block bi
DEV void resetD_body(const SceneK& S, const SceneD& D, int bi)
{
    if (!D.tinfo[2]) return;
    long long i = (long long)bi * blockDim.x + threadIdx.x;
    if (i < S.N) D.D[i] = 0.0f;
}

// start of a call: substep index 0 and (with tool contact) a cleared interval
// wrench accumulator
DEV void call_start_body(const SceneK& S, const SceneD& D, int bi)
{
    if (threadIdx.x == 0) D.ctr[2] = 0;
    if (D.tinfo[1] && threadIdx.x < TL_MAX_TOOLS * 6) D.wacc[threadIdx.x] = 0.0;
}

// Workspace of the batches that allocate no device memory (tlmpm_batch_create_static):
// one array per GPU, held by at most one such batch at a time, for the life of the
// process.  Its size bounds their footprint (TL_STATIC_SCRATCH_BYTES).
static __device__ __align__(256) unsigned char scratch[TL_STATIC_SCRATCH_BYTES];

// Ternary code sum_k d_k 3^k of side masks (Eq. 7)
DEV unsigned long long ternary(uint32_t c, int K)
{
    unsigned long long v = 0, w = 1;
    for (int k = 0; k < K; k++) {
        const int dg = (c >> k) & 1 ? 1 : ((c >> (15 + k)) & 1 ? 2 : 0);
        v += (unsigned long long)dg * w;
        w *= 3;
    }
    return v;
}

// State fields in the caller's particle order and layout (array of structs), for the copy
// to the host: particles [o0, o1) of that order, field f at out + at[f] bytes (negative:
// not wanted).  A row per lane is read in the device order and written to its place; the
// host then only receives (permuting 14M particles there took 0.1 s for u and v alone).
__global__ __launch_bounds__(256) void k_export(SceneK S, SceneD D, TlExport E, char* out, int o0, int o1, int K)
{
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= S.N) return;
    const int o = D.perm[q];
    if (o < o0 || o >= o1) return;
    const size_t r = (size_t)(o - o0);
    auto row3 = [&](int f, const float* src) {
        if (E.at[f] < 0) return;
        float* d = (float*)(out + E.at[f]) + 3 * r;
        for (int a = 0; a < 3; a++) d[a] = src[at3(q, a)];
    };
    row3(0, D.X);
    row3(1, D.u);
    row3(2, D.v);
    for (int f = 3; f <= 7; f += 4) { // F = I + H, or H itself
        if (E.at[f] < 0) continue;
        float* d = (float*)(out + E.at[f]) + 9 * r;
        for (int a = 0; a < 9; a++) {
            float val = D.H[at9(S.N, q, a)];
            if (f == 3 && a % 4 == 0) val += 1.0f;
            d[a] = val;
        }
    }
    if (E.at[4] >= 0) ((unsigned long long*)(out + E.at[4]))[r] = ternary(D.code[q], K);
    if (E.at[5] >= 0) ((float*)(out + E.at[5]))[r] = D.D[q];
    if (E.at[6] >= 0) {
        const uint32_t c = D.code[q];
        uint8_t* d = (uint8_t*)(out + E.at[6]) + (size_t)K * r;
        for (int k = 0; k < K; k++) d[k] = (c >> k) & 1 ? 1 : ((c >> (15 + k)) & 1 ? 2 : 0);
    }
}

__global__ void k_fill_f32(float* p, long long n, float v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_i32(int* p, long long n, int v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// brick AABB from the current state (scene creation, after a state write); with the
// pair-search skip also the centre of the box of the reference positions and the
// displacement anchor (exact spread: a second pass over the particles)
DEV void aabb_body(const SceneK& S, const SceneD& D, int bi)
{
    __shared__ float s_bb[4][13];
    __shared__ float s_a[3];
    const int brick = D.active[bi];
    const int beg = D.cell_start[(long long)brick * TL_CELLS], end = D.cell_start[(long long)(brick + 1) * TL_CELLS];
    // current box (0-5), speed (6), reference box (7-12)
    float bb[13] = {1e30f, 1e30f, 1e30f, -1e30f, -1e30f, -1e30f, 0.0f, 1e30f, 1e30f, 1e30f, -1e30f, -1e30f, -1e30f};
    for (int p = beg + threadIdx.x; p < end; p += blockDim.x) {
        float sp = 0.0f;
        for (int a = 0; a < 3; a++) {
            const float X = D.X[at3(p, a)];
            float xa = X + D.u[at3(p, a)];
            bb[a] = fminf(bb[a], xa);
            bb[3 + a] = fmaxf(bb[3 + a], xa);
            bb[7 + a] = fminf(bb[7 + a], X);
            bb[10 + a] = fmaxf(bb[10 + a], X);
            sp += D.v[at3(p, a)] * D.v[at3(p, a)];
        }
        bb[6] = fmaxf(bb[6], sqrtf(sp));
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    auto is_min = [](int q) { return q < 3 || (q >= 7 && q < 10); };
    for (int q = 0; q < 13; q++) {
        float val = bb[q];
        for (int o = 32; o >= 1; o >>= 1) {
            float other = __shfl_xor(val, o, 64);
            val = is_min(q) ? fminf(val, other) : fmaxf(val, other);
        }
        if (lane == 0) s_bb[w][q] = val;
    }
    __syncthreads();
    if (threadIdx.x < 13) {
        int q = threadIdx.x;
        float val = s_bb[0][q];
        for (int wv = 1; wv < 4; wv++) val = is_min(q) ? fminf(val, s_bb[wv][q]) : fmaxf(val, s_bb[wv][q]);
        if (q < 7) D.aabb[(long long)brick * 8 + q] = val;
        if (q == 6 && S.material_contact && val > 0.0f)
            atomicMax(D.hmax + (bi & (TL_HSLOTS - 1)) * TL_HSTRIDE, __float_as_int(val));
        s_bb[0][q] = val;
    }
    if (!S.pair_skip) return;
    __syncthreads();
    if (threadIdx.x < 3) { // (the anchor g2p_anchor would form from this box)
        const int a = threadIdx.x;
        const float rc = 0.5f * (s_bb[0][7 + a] + s_bb[0][10 + a]);
        D.uref[(long long)brick * 4 + a] = rc;
        s_a[a] = 0.5f * (s_bb[0][a] + s_bb[0][3 + a]) - rc;
    }
    __syncthreads();
    // spread about the anchor: exact, from a second pass over the particles
    float dv = 0.0f;
    for (int p = beg + threadIdx.x; p < end; p += blockDim.x)
        for (int a = 0; a < 3; a++) dv = fmaxf(dv, fabsf(D.u[at3(p, a)] - s_a[a]));
    for (int o = 32; o >= 1; o >>= 1) dv = fmaxf(dv, __shfl_xor(dv, o, 64));
    __syncthreads();
    if (lane == 0) s_bb[w][7] = dv;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int wv = 1; wv < 4; wv++) dv = fmaxf(dv, s_bb[wv][7]);
        const float a[3] = {s_a[0], s_a[1], s_a[2]};
        put_anchor(D, bi, brick, 0, a, dv);
    }
}

// Once per call: sum of the per-brick wrench partials accumulated over the call's
// substeps, in fixed order (one workgroup per force or torque component: four
// running sums per thread, a tree over the workgroup), added to the interval
// accumulator; the partials are cleared for the next call.
DEV void wrench_body(const SceneK& S, const SceneD& D, int bi)
{
    __shared__ double s[256];
    const int q = bi;
    if (!D.tinfo[1] || q >= D.tinfo[0] * 6) return;
    double* w = D.wpart + (long long)q * D.n_active;
    const int n = D.n_active, T = blockDim.x;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int b = threadIdx.x;
    for (; b + 3 * T < n; b += 4 * T) {
        a0 += w[b];
        a1 += w[b + T];
        a2 += w[b + 2 * T];
        a3 += w[b + 3 * T];
        w[b] = 0.0;
        w[b + T] = 0.0;
        w[b + 2 * T] = 0.0;
        w[b + 3 * T] = 0.0;
    }
    for (; b < n; b += T) {
        a0 += w[b];
        w[b] = 0.0;
    }
    s[threadIdx.x] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) D.wacc[q] += s[0];
}

// ------------------------------------------------------------------- kernels
// Every body runs either for one scene (parameters by value, block = item) or for
// a batch (block -> (scene, item) from a list).
#define TL_WRAP(NAME, BOUNDS, PARAMS, ARGS)                                                                   \
    __global__ __launch_bounds__(BOUNDS) void k_##NAME(SceneK S, SceneD D PARAMS)                           \
    {                                                                                                       \
        NAME##_body(S, D, blockIdx.x ARGS);                                                                 \
    }                                                                                                       \
    __global__ __launch_bounds__(BOUNDS) void k_##NAME##_b(const SceneK* __restrict__ Ks,                    \
                                                           const SceneD* __restrict__ Ds,                    \
                                                           const int2* __restrict__ it PARAMS)               \
    {                                                                                                       \
        const int2 t = it[blockIdx.x];                                                                      \
        NAME##_body(Ks[t.x], Ds[t.x], t.y ARGS);                                                            \
    }

#define TL_COMMA ,
TL_WRAP(slots, 256, TL_COMMA int dst TL_COMMA int src TL_COMMA int force, TL_COMMA dst TL_COMMA src TL_COMMA force)
TL_WRAP(mixed, 256, TL_COMMA int force, TL_COMMA force)
TL_WRAP(aabb, 256, , )
TL_WRAP(wrench, 256, , )
TL_WRAP(resetD, 256, , )
TL_WRAP(call_start, 64, , )

// at most 80 VGPRs: three 512-thread workgroups per CU
// Neo-Hookean: at most 80 VGPRs (three workgroups per CU); the general path (polar
// decomposition) at most 128 (two)
// P2G and G2P launch, ahead of the one workgroup per brick, S.xcap workgroups for the
// later rounds of the bricks in xlist (dispatched first so that these long ones start
// early).  Bricks are split only while all mixed bricks of the scene have such a
// workgroup (at most S.xcap of them); otherwise every brick keeps all its rounds, so
// the results do not depend on the order of xlist.  Block b -> (active index, part);
// -1: nothing to do.
// Brick of workgroup j of the split launches (j < S.xcap, part 1); -1: nothing to do
DEV int split_brick(const SceneK& S, const SceneD& D, int j)
{
    const int count = D.ctr[3];
    return (j < count && count <= S.xcap) ? D.xlist[j] : -1;
}

// SPLIT false: one workgroup per brick, every brick keeps all its rounds (scenes with
// S.xcap = 0, and batches of such scenes); true: the xcap extra workgroups first.
template <int MAT, bool SPLIT, bool FRAC>
__global__ __launch_bounds__(TL_WG) __attribute__((amdgpu_waves_per_eu(MAT == 0 ? 6 : 4))) void k_p2g(SceneK S,
                                                                                                     SceneD D,
                                                                                                     KA_Args A)
{
    const int b = blockIdx.x, nx = SPLIT ? S.xcap : 0;
    const int bi = SPLIT && b < nx ? split_brick(S, D, b) : b - nx;
    if (SPLIT && bi < 0) return;
    p2g_body<MAT, SPLIT, FRAC>(S, D, bi, A, SPLIT && b < nx, SPLIT && b < nx ? b : bi);
}
template <int MAT, bool SPLIT, bool FRAC>
__global__ __launch_bounds__(TL_WG) __attribute__((amdgpu_waves_per_eu(MAT == 0 ? 6 : 4))) void k_p2g_b(
    const SceneK* __restrict__ Ks, const SceneD* __restrict__ Ds, const int2* __restrict__ it,
    const int2* __restrict__ xit, int nx, KA_Args A)
{
    const int b = blockIdx.x;
    const int2 t = SPLIT && b < nx ? xit[b] : it[xcd_order(b - (SPLIT ? nx : 0), gridDim.x - (SPLIT ? nx : 0))];
    const SceneK& S = Ks[t.x];
    const SceneD& D = Ds[t.x];
    const int bi = SPLIT && b < nx ? split_brick(S, D, t.y) : t.y;
    if (SPLIT && bi < 0) return;
    p2g_body<MAT, SPLIT, FRAC>(S, D, bi, A, SPLIT && b < nx, SPLIT && b < nx ? t.y : bi);
}
template <bool SPLIT>
__global__ __launch_bounds__(TL_WG) __attribute__((amdgpu_waves_per_eu(6))) void k_g2p(SceneK S, SceneD D, int cur)
{
    const int b = blockIdx.x, nx = SPLIT ? S.xcap : 0;
    const int bi = SPLIT && b < nx ? split_brick(S, D, b) : b - nx;
    if (SPLIT && bi < 0) return;
    g2p_body<SPLIT>(S, D, bi, cur, SPLIT && b < nx, SPLIT && b < nx ? b : bi);
}
template <bool SPLIT>
__global__ __launch_bounds__(TL_WG) __attribute__((amdgpu_waves_per_eu(6))) void k_g2p_b(
    const SceneK* __restrict__ Ks, const SceneD* __restrict__ Ds, const int2* __restrict__ it,
    const int2* __restrict__ xit, int nx, int cur)
{
    const int b = blockIdx.x;
    const int2 t = SPLIT && b < nx ? xit[b] : it[xcd_order(b - (SPLIT ? nx : 0), gridDim.x - (SPLIT ? nx : 0))];
    const SceneK& S = Ks[t.x];
    const SceneD& D = Ds[t.x];
    const int bi = SPLIT && b < nx ? split_brick(S, D, t.y) : t.y;
    if (SPLIT && bi < 0) return;
    g2p_body<SPLIT>(S, D, bi, cur, SPLIT && b < nx, SPLIT && b < nx ? t.y : bi);
}

// ------------------------------------------------------------------- launchers
template <class KP, class KB, class... Args>
static hipError_t tl_run(const TlLaunch& L, int kind, int plain_blocks, int threads, KP kp, KB kb, Args... args)
{
    if (L.S) {
        if (plain_blocks <= 0) return hipSuccess;
        hipLaunchKernelGGL(kp, dim3(plain_blocks), dim3(threads), 0, L.st, *L.S, *L.D, args...);
    } else {
        if (L.n_items[kind] <= 0) return hipSuccess;
        hipLaunchKernelGGL(kb, dim3(L.n_items[kind]), dim3(threads), 0, L.st, L.Ks, L.Ds, L.items[kind], args...);
    }
    return hipGetLastError();
}

// one workgroup per brick, plus (split kernels) the workgroups of the split bricks'
// later rounds
template <class KP, class KB, class KPX, class KBX, class... Args>
static hipError_t tl_run_split(const TlLaunch& L, KP kp, KB kb, KPX kpx, KBX kbx, Args... args)
{
    if (L.S) {
        if (L.D->n_active <= 0) return hipSuccess;
        if (L.S->xcap > 0)
            hipLaunchKernelGGL(kpx, dim3(L.S->xcap + L.D->n_active), dim3(TL_WG), 0, L.st, *L.S, *L.D, args...);
        else
            hipLaunchKernelGGL(kp, dim3(L.D->n_active), dim3(TL_WG), 0, L.st, *L.S, *L.D, args...);
    } else {
        if (L.n_items[IT_BRICK] <= 0) return hipSuccess;
        const int nx = L.n_items[IT_XBRICK];
        if (nx > 0)
            hipLaunchKernelGGL(kbx, dim3(nx + L.n_items[IT_BRICK]), dim3(TL_WG), 0, L.st, L.Ks, L.Ds,
                               L.items[IT_BRICK], L.items[IT_XBRICK], nx, args...);
        else
            hipLaunchKernelGGL(kb, dim3(L.n_items[IT_BRICK]), dim3(TL_WG), 0, L.st, L.Ks, L.Ds, L.items[IT_BRICK],
                               L.items[IT_XBRICK], 0, args...);
    }
    return hipGetLastError();
}

template <int MAT, bool FRAC>
static hipError_t run_p2g(const TlLaunch& L, KA_Args A)
{
    return tl_run_split(L, k_p2g<MAT, false, FRAC>, k_p2g_b<MAT, false, FRAC>, k_p2g<MAT, true, FRAC>,
                        k_p2g_b<MAT, true, FRAC>, A);
}

static int blocks_of(long long n, int per) { return (int)((n + per - 1) / per); }
static int plain_bricks(const TlLaunch& L) { return L.S ? L.D->n_active : 0; }
static int plain_nodes(const TlLaunch& L) { return L.S ? blocks_of(L.S->NN, 256) : 0; }
static int plain_parts(const TlLaunch& L) { return L.S ? blocks_of(L.S->N, 256) : 0; }

// the label pass and rigid contact: group_of(n) bricks per workgroup
template <class KP, class KB>
static hipError_t run_groups(const TlLaunch& L, KP kp, KB kb)
{
    const int n = L.S ? L.D->n_active : L.n_items[IT_BRICK];
    if (n <= 0) return hipSuccess;
    const int nb = group_of(n), G = (n + nb - 1) / nb;
    if (L.S)
        hipLaunchKernelGGL(kp, dim3(G), dim3(256), 0, L.st, *L.S, *L.D, nb);
    else
        hipLaunchKernelGGL(kb, dim3(G), dim3(256), 0, L.st, L.Ks, L.Ds, L.items[IT_BRICK], n, nb);
    return hipGetLastError();
}

extern "C" {
hipError_t tl_launch_rigid(const TlLaunch* L)
{
    return run_groups(*L, k_rigid, k_rigid_b);
}

hipError_t tl_launch_p2g(const TlLaunch* L, int do_p2g, int tabs_differ, int cur, int rsb)
{
    KA_Args A;
    A.do_p2g = do_p2g;
    A.tabs_differ = tabs_differ;
    A.cur = cur;
    A.rsb = rsb;
    if (L->frac) return L->general ? run_p2g<1, true>(*L, A) : run_p2g<0, true>(*L, A);
    return L->general ? run_p2g<1, false>(*L, A) : run_p2g<0, false>(*L, A);
}

hipError_t tl_launch_g2p(const TlLaunch* L, int cur)
{
    return tl_run_split(*L, k_g2p<false>, k_g2p_b<false>, k_g2p<true>, k_g2p_b<true>, cur);
}

hipError_t tl_launch_labels(const TlLaunch* L)
{
    return run_groups(*L, k_labels, k_labels_b);
}

hipError_t tl_launch_labels_rigid(const TlLaunch* L)
{
    const int n = plain_bricks(*L); // (single scenes only)
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_labels_rigid, dim3(2 * n), dim3(256), 0, L->st, *L->S, *L->D, n);
    return hipGetLastError();
}

hipError_t tl_launch_slots(const TlLaunch* L, int dst, int src, int force)
{
    return tl_run(*L, IT_NODE, plain_nodes(*L), 256, k_slots, k_slots_b, dst, src, force);
}

hipError_t tl_launch_mixed(const TlLaunch* L, int force)
{
    return tl_run(*L, IT_BRICK, plain_bricks(*L), 256, k_mixed, k_mixed_b, force);
}

hipError_t tl_launch_aabb(const TlLaunch* L)
{
    return tl_run(*L, IT_BRICK, plain_bricks(*L), 256, k_aabb, k_aabb_b);
}

hipError_t tl_launch_wrench(const TlLaunch* L)
{
    return tl_run(*L, IT_WRENCH, L->S ? TL_MAX_TOOLS * 6 : 0, 256, k_wrench, k_wrench_b);
}

hipError_t tl_launch_resetD(const TlLaunch* L)
{
    return tl_run(*L, IT_PART, plain_parts(*L), 256, k_resetD, k_resetD_b);
}

hipError_t tl_launch_call_start(const TlLaunch* L)
{
    return tl_run(*L, IT_SCENE, L->S ? 1 : 0, 64, k_call_start, k_call_start_b);
}

hipError_t tl_launch_frac(const SceneK* S, const SceneD* D, hipStream_t st)
{
    if (S->N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_frac, dim3(blocks_of(S->N, 256)), dim3(256), 0, st, *S, *D);
    return hipGetLastError();
}

hipError_t tl_launch_export(const TlLaunch* L, const TlExport* E, void* out, int o0, int o1, int max_cuts)
{
    if (L->S->N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_export, dim3(blocks_of(L->S->N, 256)), dim3(256), 0, L->st, *L->S, *L->D, *E, (char*)out, o0,
                       o1, max_cuts);
    return hipGetLastError();
}

hipError_t tl_launch_fill_f32(float* p, long long n, float v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t tl_launch_fill_i32(int* p, long long n, int v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

// Device address of this GPU's copy of `scratch` (the batch workspace of
// tlmpm_batch_create_static), looked up once per device with that device current
// and kept: in host code the array's name is only a stand-in, never a device
// address.
hipError_t tl_static_scratch(int dev, void** ptr)
{
    static std::mutex m;
    static void* addr[TL_STATIC_DEVICES] = {};
    if (dev < 0 || dev >= TL_STATIC_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(m);
    if (!addr[dev]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != dev) return hipErrorInvalidDevice;
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}
}
