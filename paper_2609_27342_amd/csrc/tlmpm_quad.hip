// tlmpm_quad.hip -- gfx950 kernels of the quadratic B-spline variant of the
// transfers (27-node stencil, reading R33): P2G, grid update, G2P with the MUSL
// re-scatter, velocity remap and deformation-gradient update.  Labels, contact,
// cutting work and the wrench are shared with the trilinear path.
//
// A particle at reference coordinate q = (X - origin)/dx (in cells) touches the
// nodes base .. base + 2 per axis, base = floor(q - 1/2); a brick of 4x4x4 cells
// therefore touches the 7x7x7 box of nodes from (4 b - 1) to (4 b + 5).
//
// Logical grids (Sec. III-D) are slots of a per-node table of side keys, built each
// substep from the keys that reach the node: two tables alternate by substep
// parity, the table of one substep cleared during the next.
//
// Lanes.  Thread h * 64 + l of a brick workgroup holds, in each round, a particle
// of the brick's cell l whose position inside the cell has half pattern h (bit a
// set: upper half along axis a); the host builds this map once (reference
// positions do not move), with more rounds where a cell holds two particles of
// one pattern.  A wave's particles then lie in distinct cells with one pattern, so
// their base nodes, and the nodes of any one stencil offset, are distinct, and
// all of them lie in a 6x6x6 region fixed by the pattern.  Each wave adds into its own LDS
// region with plain read-modify-writes (no atomics, no barriers), one side key of the
// brick at a time (bricks on a cut hold two or three); the regions are summed in wave
// order when the box goes out: to the brick's own partials, one box per side key, and the
// node kernels add up the (at most 8) boxes that hold a node in a fixed order.  Keys of a
// brick beyond the slot capacity go to the node slots with floating-point atomics (with
// them for every key the 1.5M atomics of 586 bricks kept the P2G waiting 18 us per box,
// up to 50 us, of 85 us).
#include <hip/hip_runtime.h>
#include <hip/amd_detail/amd_hip_unsafe_atomics.h>
#include <math.h>
#include <stdint.h>

#include "tlmpm_common.h"
#include "tlmpm_device.h"

#define TL_QBOX 7
#define TL_QBOXN 343      // nodes of a brick's 7x7x7 box
#define TL_QWG 512        // threads of a brick workgroup
#define TL_QNODE 256      // threads of a workgroup of the node kernels (8 per node)
#define TL_QEMPTY 0xFFFFFFFFu
// LDS places of a wave's 6x6x6 region and of a brick's 7x7x7 box, in 16-byte units: two z
// planes side by side, and pitches that put the 16 cells of two parity classes (a quarter
// of a wave's lanes) in 16 different bank groups whatever the stencil offset
#define TL_QREG 224
#define TL_QBOXP 403
DEV int q_reg_at(int x, int y, int z) { return (z >> 1) * 76 + y * 12 + (z & 1) * 6 + x; }
DEV int q_box_at(int x, int y, int z) { return (z >> 1) * 104 + y * 14 + (z & 1) * 7 + x; }

// brick-major id of grid node (gx, gy, gz); -1 outside the grid
DEV long long q_gid(const SceneK& S, int gx, int gy, int gz)
{
    if (gx < 0 || gy < 0 || gz < 0 || gx > S.cx || gy > S.cy || gz > S.cz) return -1;
    const long long nb = ((long long)(gz >> 2) * S.nby + (gy >> 2)) * S.nbx + (gx >> 2);
    return (nb << 6) | ((gz & 3) * 16 + (gy & 3) * 4 + (gx & 3));
}

// box node of a brick: (X, Y, Z) in 0..6 stands for grid node 4 b - 1 + (X, Y, Z)
DEV long long q_box_gid(const SceneK& S, int bx, int by, int bz, int bn)
{
    return q_gid(S, bx * TL_B - 1 + bn % TL_QBOX, by * TL_B - 1 + (bn / TL_QBOX) % TL_QBOX, bz * TL_B - 1 + bn / 49);
}

// grid cell of cell slot l (0..63, sorted order: parity class, cell) of brick (bx, by, bz)
DEV void q_cell(int bx, int by, int bz, int l, int c[3])
{
    const int w = l >> 3, i = l & 7;
    c[0] = bx * TL_B + 2 * (i & 1) + (w & 1);
    c[1] = by * TL_B + 2 * ((i >> 1) & 1) + ((w >> 1) & 1);
    c[2] = bz * TL_B + 2 * ((i >> 2) & 1) + ((w >> 2) & 1);
}

// Quadratic B-spline weights and derivatives per axis (reading R33).  The half of
// the cell the particle lies in (decided once on the host, in FP64) gives the base
// node; f = q - base lies in [1/2, 3/2) and the node distances are f, f - 1, f - 2:
//   N = (3/2 - f)^2 / 2,  3/4 - (f - 1)^2,  (f - 1/2)^2 / 2.
struct QStencil {
    int lo[3];        // base node per axis
    float w[3][3];    // [axis][node]
    float g[3][3];    // derivative / dx
    // some weight is zero (the middle ones are at least 1/2): its nodes take no part (R7)
    DEV bool zero() const
    {
        return w[0][0] == 0.0f || w[0][2] == 0.0f || w[1][0] == 0.0f || w[1][2] == 0.0f || w[2][0] == 0.0f ||
               w[2][2] == 0.0f;
    }
};
// a gather with tests for zero weights, or without (waves that hold none)
template <bool B>
struct QGuard {
    static constexpr bool value = B;
};

DEV void q_stencil(const SceneK& S, const float* X, const int c[3], int h, QStencil& Q)
{
    const double o[3] = {S.ox, S.oy, S.oz};
#pragma unroll
    for (int a = 0; a < 3; a++) {
        double t = ((double)X[a] - o[a]) * S.inv_dx_d - (double)c[a];
        t = fmin(fmax(t, 0.0), 1.0);
        const bool low = ((h >> a) & 1) == 0; // the host's FP64 decision t < 1/2
        Q.lo[a] = low ? c[a] - 1 : c[a];
        const float f = (float)(low ? t + 1.0 : t);
        const float d0 = 1.5f - f, d1 = f - 1.0f, d2 = f - 0.5f;
        Q.w[a][0] = 0.5f * d0 * d0;
        Q.w[a][1] = 0.75f - d1 * d1;
        Q.w[a][2] = 0.5f * d2 * d2;
        Q.g[a][0] = -d0 * S.inv_dx;
        Q.g[a][1] = -2.0f * d1 * S.inv_dx;
        Q.g[a][2] = d2 * S.inv_dx;
    }
}

// index of a side key in the brick's LDS key list (inserted on first use); -1 full
DEV int q_key_index(uint32_t* s_keys, uint32_t key)
{
    for (int k = 0; k < TL_SCAP_MAX; k++) {
        if (s_keys[k] == key) return k; // (most lanes find it: no serial exchanges)
        const uint32_t old = atomicCAS(&s_keys[k], TL_QEMPTY, key);
        if (old == TL_QEMPTY || old == key) return k;
    }
    return -1;
}

// place of slot s of node g in the arrays of sums: slot by slot, so that the first slots,
// nearly all there are, lie side by side
DEV size_t q_at(const SceneK& S, long long g, int s) { return (size_t)s * (size_t)S.NN + (size_t)g; }

// slot of key at node g in a table (slots fill from 0; the first empty one ends
// the list); -1 if absent
DEV int q_find(const SceneK& S, const uint32_t* tab, long long g, uint32_t key)
{
    for (int s = 0; s < S.scap; s++) {
        const uint32_t c = tab[(long long)s * S.NN + g];
        if (c == key) return s;
        if (c == TL_QEMPTY) return -1;
    }
    return -1;
}

DEV uint32_t* q_table(const SceneK& S, const SceneD& D, int par)
{
    return D.qcode + (size_t)par * (size_t)S.scap * (size_t)S.NN;
}

// Compatibility coupling of one 3-vector field over the c slots of a node (Eq. 8):
// f_a + (1/M) sum_{b != a, compatible} (m_a f_b - m_b f_a), M = sum of the masses,
// from the pre-exchange values; written over f.
DEV void q_couple(int c, const float* m, const uint32_t* codes, float (*f)[3])
{
    float M = 0.0f;
    for (int a = 0; a < c; a++) M += m[a];
    const float invM = M > 0.0f ? 1.0f / M : 0.0f;
    float out[TL_SCAP_MAX][3];
    for (int a = 0; a < c; a++) {
        float acc[3] = {0.0f, 0.0f, 0.0f};
        for (int b = 0; b < c; b++) {
            if (b == a || codes_conflict(codes[a], codes[b])) continue;
            for (int j = 0; j < 3; j++) acc[j] += m[a] * f[b][j] - m[b] * f[a][j];
        }
        for (int j = 0; j < 3; j++) out[a][j] = f[a][j] + acc[j] * invM;
    }
    for (int a = 0; a < c; a++)
        for (int j = 0; j < 3; j++) f[a][j] = out[a][j];
}

// the same for two slots, in registers (nearly every node with more than one)
DEV void q_couple2(float m0, float m1, bool compatible, float (&f0)[3], float (&f1)[3])
{
    const float M = m0 + m1, invM = M > 0.0f ? 1.0f / M : 0.0f;
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const float a = f0[j], b = f1[j];
        f0[j] = a + (compatible ? m0 * b - m1 * a : 0.0f) * invM;
        f1[j] = b + (compatible ? m1 * a - m0 * b : 0.0f) * invM;
    }
}

// particle of this thread in round r of active brick bi (-1: none)
DEV int q_particle(const SceneD& D, int bi, int r)
{
    return D.qmap[(size_t)(D.qround[bi] + r) * TL_QWG + threadIdx.x];
}

DEV int q_rounds(const SceneD& D, int bi) { return D.qround[bi + 1] - D.qround[bi]; }

// Particle of this thread in round r, its code and reference position.  Round 0, nearly
// always the only one, is loaded before a brick's box, so that the two chains of loads
// overlap.
struct QFirst {
    int p;
    uint32_t code;
    float X[3];
    DEV QFirst(const SceneD& D, int bi, int rounds, int r = 0)
    {
        p = r < rounds ? q_particle(D, bi, r) : -1;
        code = 0u;
        X[0] = X[1] = X[2] = 0.0f;
        if (p < 0) return;
        code = D.code[p];
        X[0] = D.X[at3(p, 0)];
        X[1] = D.X[at3(p, 1)];
        X[2] = D.X[at3(p, 2)];
    }
};

// registers the side keys of a brick's particles in its LDS key list (call between
// barriers)
DEV void q_register_keys(const SceneK& S, const SceneD& D, int bi, uint32_t* s_keys)
{
    const int rounds = q_rounds(D, bi);
    for (int r = 0; r < rounds; r++) {
        const int p = q_particle(D, bi, r);
        if (p < 0) continue;
        if (q_key_index(s_keys, slot_key(S, D.code[p])) < 0) atomicOr(D.status, TL_ST_BOX);
    }
}

// ------------------------------------------------------------------ slot tables
// Per active brick: clears the other parity's table over its box, then inserts the
// side key of every (box node, key) reached by a particle with a non-zero weight
// into this parity's table (atomic compare-and-swap per slot); a new slot's sums
// are zeroed by the thread that created it.
__global__ __launch_bounds__(TL_QWG) void k_q_slots(SceneK S, SceneD D, int par)
{
    __shared__ uint32_t s_keys[TL_SCAP_MAX];
    __shared__ uint32_t s_pres[TL_QBOXN];
    const int bi = blockIdx.x, tid = threadIdx.x;
    const int brick = D.active[bi];
    const int bx = brick % S.cbx, by = (brick / S.cbx) % S.cby, bz = brick / (S.cbx * S.cby);
    uint32_t* tab = q_table(S, D, par);
    uint32_t* other = q_table(S, D, 1 - par);
    for (int t = tid; t < TL_QBOXN; t += TL_QWG) {
        s_pres[t] = 0u;
        const long long g = q_box_gid(S, bx, by, bz, t);
        if (g < 0) continue;
        for (int s = 0; s < S.scap; s++) {
            const long long i = (long long)s * S.NN + g;
            if (other[i] == TL_QEMPTY) break;
            other[i] = TL_QEMPTY;
        }
    }
    if (tid < TL_SCAP_MAX) s_keys[tid] = TL_QEMPTY;
    __syncthreads();
    const int rounds = q_rounds(D, bi), h = tid >> 6;
    int c[3];
    q_cell(bx, by, bz, tid & 63, c);
    for (int r = 0; r < rounds; r++) {
        const int p = q_particle(D, bi, r);
        if (p < 0) continue;
        const uint32_t key = slot_key(S, D.code[p]);
        const int k = q_key_index(s_keys, key);
        if (k < 0) {
            atomicOr(D.status, TL_ST_BOX);
            continue;
        }
        const float X[3] = {D.X[at3(p, 0)], D.X[at3(p, 1)], D.X[at3(p, 2)]};
        QStencil Q;
        q_stencil(S, X, c, h, Q);
        const int ox = Q.lo[0] - (bx * TL_B - 1), oy = Q.lo[1] - (by * TL_B - 1), oz = Q.lo[2] - (bz * TL_B - 1);
#pragma unroll
        for (int cz = 0; cz < 3; cz++)
#pragma unroll
            for (int cy = 0; cy < 3; cy++)
#pragma unroll
                for (int cx = 0; cx < 3; cx++) {
                    if (Q.w[0][cx] * Q.w[1][cy] * Q.w[2][cz] == 0.0f) continue; // reading R7
                    atomicOr(&s_pres[((oz + cz) * TL_QBOX + oy + cy) * TL_QBOX + ox + cx], 1u << k);
                }
    }
    __syncthreads();
    for (int t = tid; t < TL_QBOXN; t += TL_QWG) {
        uint32_t pm = s_pres[t];
        if (!pm) continue;
        const long long g = q_box_gid(S, bx, by, bz, t);
        if (g < 0) {
            atomicOr(D.status, TL_ST_BOX);
            continue;
        }
        while (pm) {
            const int k = __ffs(pm) - 1;
            pm &= pm - 1u;
            const uint32_t key = s_keys[k];
            int s = 0;
            for (; s < S.scap; s++) {
                const uint32_t old = atomicCAS(&tab[(long long)s * S.NN + g], TL_QEMPTY, key);
                if (old == TL_QEMPTY) {
                    float4* a = (float4*)(D.qacc + q_at(S, g, s) * 8);
                    a[0] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    a[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    *(float4*)(D.qrs + q_at(S, g, s) * 4) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    break;
                }
                if (old == key) break;
            }
            if (s == S.scap) atomicOr(D.status, TL_ST_SLOT);
        }
    }
}

// The 8 wave regions of the P2G: {m, m v} and the impulse per node (28 bytes: with 32 a CU
// holds two workgroups instead of three)
struct QRegions {
    float4 a[8 * TL_QREG];
    float2 b[8 * TL_QREG];
    float c[8 * TL_QREG];
    DEV void zero()
    {
        for (int t = late(threadIdx.x); t < 8 * TL_QREG; t += TL_QWG) {
            a[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            b[t] = make_float2(0.0f, 0.0f);
            c[t] = 0.0f;
        }
    }
    DEV void sum(int at, float v[7]) const
    {
        const float4 x = a[at];
        const float2 y = b[at];
        const float z = c[at];
        v[0] += x.x;
        v[1] += x.y;
        v[2] += x.z;
        v[3] += x.w;
        v[4] += y.x;
        v[5] += y.y;
        v[6] += z;
    }
};
// ... and of the re-scatter: m v^{n+1}
struct QRegions3 {
    float4 a[8 * TL_QREG];
    DEV void zero()
    {
        for (int t = late(threadIdx.x); t < 8 * TL_QREG; t += TL_QWG) a[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    DEV void sum(int at, float v[3]) const
    {
        const float4 x = a[at];
        v[0] += x.x;
        v[1] += x.y;
        v[2] += x.z;
    }
};

// A brick's partials: boxes of its first slot-capacity side keys (8 floats per node, 4 in
// the re-scatter), and the keys.  They use the arrays that the trilinear transfers keep
// their partials in (12000 bytes per brick and slot; a box takes 10976, the keys 64 per
// brick).
DEV float* q_part(const SceneK& S, const SceneD& D, int bi, int k)
{
    static_assert(TL_QBOXN * 8 * 4 + TL_SCAP_MAX * 4 <= TL_BOXN * 24 * 4, "the box fits the trilinear partials");
    return D.p2g + ((size_t)k * D.n_active + bi) * (TL_QBOXN * 8); // (boxes of one k side by side: nearly all are k = 0)
}
DEV uint32_t* q_part_keys(const SceneK& S, const SceneD& D, int bi)
{
    return (uint32_t*)(D.p2g + (size_t)D.n_active * S.scap * (TL_QBOXN * 8)) + (size_t)bi * TL_SCAP_MAX;
}

// One of the 8 boxes around node g, by the lane's place d in its group of 8 (a lane per box:
// its loads run side by side, and the code stays short; with a thread per node a scene of a
// few bricks waited longer for the code than for the data): the active brick (-1: none) and
// the node's place in its box.  Per axis a node lies in the box of its own brick, and the
// lower two of four also in that of the brick below, the last one in that of the brick above.
struct QAround {
    int bi, bn;
    uint4 key; // the box's first four side keys
    DEV void set(const SceneK& S, const SceneD& D, long long g, int d)
    {
        const int nb = (int)(g >> 6), l[3] = {(int)g & 3, ((int)g >> 2) & 3, ((int)g >> 4) & 3};
        const int h[3] = {nb % S.nbx, (nb / S.nbx) % S.nby, nb / S.nbx / S.nby};
        const int n[3] = {S.cbx, S.cby, S.cbz};
        int b[3], x[3];
        bool in = true;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const bool other = (d >> a) & 1;
            b[a] = !other ? h[a] : l[a] == 3 ? h[a] + 1 : h[a] - 1;
            x[a] = !other ? l[a] + 1 : l[a] == 3 ? 0 : l[a] + 5;
            in = in && b[a] >= 0 && b[a] < n[a] && x[a] < TL_QBOX;
        }
        bn = (x[2] * TL_QBOX + x[1]) * TL_QBOX + x[0];
        bi = in ? D.bact[((long long)b[2] * S.cby + b[1]) * S.cbx + b[0]] : -1;
        key = bi >= 0 ? *(const uint4*)q_part_keys(S, D, bi)
                      : make_uint4(TL_QEMPTY, TL_QEMPTY, TL_QEMPTY, TL_QEMPTY);
    }
    // adds the boxes' sums of one side key (NV float4 per node) to v in all 8 lanes (in a
    // fixed order)
    template <int NV>
    DEV void sum(const SceneK& S, const SceneD& D, uint32_t want, float4 (&v)[NV]) const
    {
        int k = key.x == want ? 0 : key.y == want ? 1 : key.z == want ? 2 : key.w == want ? 3 : -1;
        if (k < 0 && key.w != TL_QEMPTY) // (a brick of more than four keys)
            for (int j = 4; j < S.scap; j++)
                if (q_part_keys(S, D, bi)[j] == want) k = j;
        if (k >= S.scap) k = -1; // (in the node's slots already)
#pragma unroll
        for (int n = 0; n < NV; n++) {
            float4 w = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k >= 0) w = *((const float4*)q_part(S, D, bi, k) + bn * NV + n);
            v[n].x += all8(w.x);
            v[n].y += all8(w.y);
            v[n].z += all8(w.z);
            v[n].w += all8(w.w);
        }
    }
    DEV static float all8(float w)
    {
        w += lane_xor<1>(w);
        w += lane_xor<2>(w);
        return w + lane_xor<4>(w);
    }
};

// puts a brick's LDS sums of its side key k into its partials (Q values per node; a key
// beyond the slot capacity: into the node slots in HBM, stride
// QS floats per slot): the 8 wave regions in wave order
// (wave h holds box node (X, Y, Z) at region (X, Y, Z) - 1 + low(h), low = 1 on the
// axes of the lower half)
template <int Q, int QS, class R>
DEV void q_flush(const SceneK& S, const SceneD& D, const uint32_t* tab, float* dst, int bi, int bx, int by, int bz,
                 int k, uint32_t key, const R& reg)
{
    for (int bn = late(threadIdx.x); bn < TL_QBOXN; bn += TL_QWG) {
        const int X = bn % TL_QBOX, Y = (bn / TL_QBOX) % TL_QBOX, Z = bn / 49;
        float v[Q];
#pragma unroll
        for (int c = 0; c < Q; c++) v[c] = 0.0f;
#pragma unroll
        for (int h = 0; h < 8; h++) {
            const int rx = X - (h & 1), ry = Y - ((h >> 1) & 1), rz = Z - ((h >> 2) & 1);
            if (rx < 0 || ry < 0 || rz < 0 || rx > 5 || ry > 5 || rz > 5) continue;
            reg.sum(h * TL_QREG + q_reg_at(rx, ry, rz), v);
        }
        if (k < S.scap) {
            float4* o = (float4*)q_part(S, D, bi, k) + bn * (QS / 4);
            o[0] = make_float4(v[0], v[1], v[2], Q > 3 ? v[Q > 3 ? 3 : 0] : 0.0f);
            if constexpr (Q == 7) o[1] = make_float4(v[4], v[5], v[6], 0.0f);
            continue;
        }
        bool any = false;
#pragma unroll
        for (int c = 0; c < Q; c++) any = any || v[c] != 0.0f;
        if (!any) continue;
        const long long g = q_box_gid(S, bx, by, bz, bn);
        const int s = g >= 0 ? q_find(S, tab, g, key) : -1;
        if (s < 0) {
            atomicOr(D.status, TL_ST_LOOKUP);
            continue;
        }
        float* o = dst + q_at(S, g, s) * QS;
#pragma unroll
        for (int c = 0; c < Q; c++)
            if (v[c] != 0.0f) unsafeAtomicAdd(o + c, v[c]);
    }
}

// ---------------------------------------------------------------------------- P2G
// Per active brick: stress (Neo-Hookean, or the fixed-corotated family with
// viscosity and plasticity for MAT 1), gravity and contact impulses, and the
// label-masked scatter of m, m v and the impulse (Eq. 2) to the 27 nodes.  Bound by the
// chain of 27 LDS read-modify-writes of a brick's one round; three workgroups per CU (28
// bytes per node, 80 registers), so that a scene of 586 bricks runs in one go.  There: 125
// us with LDS atomics for every key after the first and node atomics at the end, 84 us
// with a pass per key, 35 us with partials too.
template <int MAT>
__global__ __launch_bounds__(TL_QWG, MAT == 0 ? 6 : 4) void k_q_p2g(SceneK S, SceneD D, int par)
{
    __shared__ uint32_t s_keys[TL_SCAP_MAX];
    __shared__ QRegions s_wv;
    const int bi = blockIdx.x, tid = threadIdx.x;
    const int brick = D.active[bi];
    const int bx = brick % S.cbx, by = (brick / S.cbx) % S.cby, bz = brick / (S.cbx * S.cby);
    const uint32_t* tab = q_table(S, D, par);
    if (tid < TL_SCAP_MAX) s_keys[tid] = TL_QEMPTY;
    s_wv.zero();
    __syncthreads();
    q_register_keys(S, D, bi, s_keys);
    __syncthreads();
    if (tid < TL_SCAP_MAX) q_part_keys(S, D, bi)[tid] = s_keys[tid]; // for the other passes of the substep
    const long long N = S.N;
    const float dt = S.dt;
    const bool rig = (S.floor_on || D.tinfo[1]) && D.brig[brick] != 0;
    const int rounds = q_rounds(D, bi);
    for (int k = 0; k < TL_SCAP_MAX && s_keys[k] != TL_QEMPTY; k++) {
        const uint32_t key = s_keys[k];
        if (k > 0) {
            s_wv.zero();
            __syncthreads();
        }
        for (int r = 0; r < rounds; r++) {
            const int p = q_particle(D, bi, r);
            if (p < 0) continue;
            const uint32_t code = D.code[p];
            if (slot_key(S, code) != key) continue;
            float m, vel[3], ext[3], Pk[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            float H[9];
            const float X[3] = {D.X[at3(p, 0)], D.X[at3(p, 1)], D.X[at3(p, 2)]};
#pragma unroll
            for (int a = 0; a < 9; a++) H[a] = D.H[at9(N, p, a)];
#pragma unroll
            for (int a = 0; a < 3; a++) vel[a] = D.v[at3(p, a)];
            m = S.m_uniform ? S.m0 : D.m[p];
            const float V0 = S.v_uniform ? S.V0 : D.V0[p];
            float mu, lam;
            lame(S, S.e_uniform ? 0.0f : D.E[p], mu, lam);
            bool ok;
            if constexpr (MAT == 1) {
                if (S.ystress > 0.0f) {
                    // P = P_fcr(F_e) F_p^{-T}, F_e - I = H + Gp + H Gp, F_p^{-1} = I + Gp
                    float Gp[9], K[9], Pe[9];
#pragma unroll
                    for (int a = 0; a < 9; a++) Gp[a] = D.Gp[at9(N, p, a)];
#pragma unroll
                    for (int i = 0; i < 3; i++)
#pragma unroll
                        for (int j = 0; j < 3; j++) {
                            float kk = H[3 * i + j] + Gp[3 * i + j];
#pragma unroll
                            for (int l = 0; l < 3; l++) kk += H[3 * i + l] * Gp[3 * l + j];
                            K[3 * i + j] = kk;
                        }
                    ok = fixed_corotated(mu, lam, K, Pe);
#pragma unroll
                    for (int i = 0; i < 3; i++)
#pragma unroll
                        for (int j = 0; j < 3; j++) {
                            float a = Pe[3 * i + j];
#pragma unroll
                            for (int l = 0; l < 3; l++) a += Pe[3 * i + l] * Gp[3 * j + l];
                            Pk[3 * i + j] = a;
                        }
                } else {
                    ok = S.material == 1 ? fixed_corotated(mu, lam, H, Pk) : neo_hookean(mu, lam, H, Pk);
                }
                if (ok && S.visc > 0.0f) {
                    float Fd[9];
#pragma unroll
                    for (int a = 0; a < 9; a++) Fd[a] = D.Fdot[at9(N, p, a)];
                    add_viscous(S.visc, H, Fd, Pk);
                }
            } else {
                ok = neo_hookean(mu, lam, H, Pk);
            }
            if (!ok) {
                atomicOr(D.status, TL_ST_NONFINITE);
#pragma unroll
                for (int a = 0; a < 9; a++) Pk[a] = 0.0f;
            }
            float Jc[3] = {0.0f, 0.0f, 0.0f};
            if (rig) {
                Jc[0] += D.Jrig[at3(p, 0)];
                Jc[1] += D.Jrig[at3(p, 1)];
                Jc[2] += D.Jrig[at3(p, 2)];
            }
            if (S.material_contact && (code & TL_CAND_BIT)) {
                Jc[0] += D.Jmat[at3(p, 0)];
                Jc[1] += D.Jmat[at3(p, 1)];
                Jc[2] += D.Jmat[at3(p, 2)];
            }
#pragma unroll
            for (int a = 0; a < 3; a++) ext[a] = Jc[a] + dt * m * (a == 0 ? S.gx : a == 1 ? S.gy : S.gz);
            const float sA = -dt * V0;
#pragma unroll
            for (int a = 0; a < 9; a++) Pk[a] *= sA;
            int c[3];
            const int h = late(tid) >> 6;
            q_cell(bx, by, bz, late(tid) & 63, c);
            QStencil Q;
            q_stencil(S, X, c, h, Q);
            // own region of this wave: the lanes' nodes of one offset are distinct
            const int r0 = h * TL_QREG + (c[1] - by * TL_B) * 12 + c[0] - bx * TL_B, rz = c[2] - bz * TL_B;
#pragma unroll
            for (int cz = 0; cz < 3; cz++)
#pragma unroll
                for (int cy = 0; cy < 3; cy++) {
                    const int row = r0 + q_reg_at(0, 0, rz + cz) + cy * 12;
                    const float wyz = Q.w[1][cy] * Q.w[2][cz];
                    if (wyz == 0.0f) continue; // reading R7: a zero weight contributes nothing
                    // node (cx, cy, cz) gets w {m, m v} and A grad N + w ext, w = wx wyz,
                    // grad N = (gx wyz, wx gy wz, wx wy gz): what the row shares
                    const float gywz = Q.g[1][cy] * Q.w[2][cz], wygz = Q.w[1][cy] * Q.g[2][cz];
                    const float wm = wyz * m;
                    const float mv[3] = {wm * vel[0], wm * vel[1], wm * vel[2]};
                    float A[3], B[3];
#pragma unroll
                    for (int a = 0; a < 3; a++) {
                        A[a] = Pk[3 * a] * wyz;
                        B[a] = Pk[3 * a + 1] * gywz + Pk[3 * a + 2] * wygz + wyz * ext[a];
                    }
#pragma unroll
                    for (int cx = 0; cx < 3; cx++) {
                        const float wx = Q.w[0][cx], gx = Q.g[0][cx];
                        if (cx != 1 && wx == 0.0f) continue; // (the middle weight is at least 1/2)
                        const int at = row + cx;
                        float4 a = s_wv.a[at];
                        float2 b = s_wv.b[at];
                        float c2 = s_wv.c[at];
                        a.x += wx * wm;
                        a.y += wx * mv[0];
                        a.z += wx * mv[1];
                        a.w += wx * mv[2];
                        b.x += gx * A[0] + wx * B[0];
                        b.y += gx * A[1] + wx * B[1];
                        c2 += gx * A[2] + wx * B[2];
                        s_wv.a[at] = a;
                        s_wv.b[at] = b;
                        s_wv.c[at] = c2;
                        // one node at a time: another lane adds to it at its next offset
                        asm volatile("" ::: "memory");
                    }
                }
        }
        __syncthreads();
        q_flush<7, 8>(S, D, tab, D.qacc, bi, bx, by, bz, k, key, s_wv);
        __syncthreads();
    }
}

// ---------------------------------------------------------------- node kernels
// Grid update (bound by its chain of loads: 12 us with sums made by atomics, 16 us with a lane
// per box, 20 us with a thread per node, for 48k nodes): per node, the sums of its slots from the boxes around it (and of keys beyond
// them, added by atomics), coupling of momentum and impulse (Eq. 8), then
// v^n = pbar / m and dv = dpbar / m (Eq. 9) over the slot's sums.
__global__ __launch_bounds__(TL_QNODE) void k_q_grid(SceneK S, SceneD D, int par)
{
    const int i = (blockIdx.x * TL_QNODE + threadIdx.x) >> 3, d = threadIdx.x & 7;
    if (i >= D.n_qnodes) return;
    const long long g = D.qnodes[i];
    const uint32_t* tab = q_table(S, D, par);
    const uint32_t key0 = tab[g], key1 = S.scap > 1 ? tab[S.NN + g] : TL_QEMPTY;
    const uint32_t key2 = S.scap > 2 ? tab[2 * S.NN + g] : TL_QEMPTY;
    QAround A;
    A.set(S, D, g, d);
    if (key0 == TL_QEMPTY) return;
    const bool one = key1 == TL_QEMPTY, more = key2 != TL_QEMPTY;
    auto at = [&](int s) { return (float4*)(D.qacc + q_at(S, g, s) * 8); };
    float4 v[2] = {}, u[2] = {}; // the first two slots
#pragma unroll 1
    for (int s = 0; s < (one ? 1 : 2); s++) {
        u[0] = v[0];
        u[1] = v[1];
        v[0] = at(s)[0];
        v[1] = at(s)[1];
        A.sum<2>(S, D, s ? key1 : key0, v);
    }
    if (one) {
        if (d) return;
        const float m = v[0].x, im = m > 0.0f ? 1.0f / m : 0.0f;
        at(0)[0] = make_float4(m, v[0].y * im, v[0].z * im, v[0].w * im);
        at(0)[1] = make_float4(v[1].x * im, v[1].y * im, v[1].z * im, 0.0f);
        return;
    }
    if (!more) {
        if (d) return;
        const float m0 = u[0].x, m1 = v[0].x;
        float p0[3] = {u[0].y, u[0].z, u[0].w}, p1[3] = {v[0].y, v[0].z, v[0].w};
        float d0[3] = {u[1].x, u[1].y, u[1].z}, d1[3] = {v[1].x, v[1].y, v[1].z};
        const bool compatible = !codes_conflict(key0, key1);
        q_couple2(m0, m1, compatible, p0, p1);
        q_couple2(m0, m1, compatible, d0, d1);
        const float i0 = m0 > 0.0f ? 1.0f / m0 : 0.0f, i1 = m1 > 0.0f ? 1.0f / m1 : 0.0f;
        at(0)[0] = make_float4(m0, p0[0] * i0, p0[1] * i0, p0[2] * i0);
        at(0)[1] = make_float4(d0[0] * i0, d0[1] * i0, d0[2] * i0, 0.0f);
        at(1)[0] = make_float4(m1, p1[0] * i1, p1[1] * i1, p1[2] * i1);
        at(1)[1] = make_float4(d1[0] * i1, d1[1] * i1, d1[2] * i1, 0.0f);
        return;
    }
    float m[TL_SCAP_MAX], p[TL_SCAP_MAX][3], dp[TL_SCAP_MAX][3];
    uint32_t codes[TL_SCAP_MAX];
    int c = 0;
#pragma unroll 1
    for (; c < S.scap; c++) {
        codes[c] = tab[(long long)c * S.NN + g];
        if (codes[c] == TL_QEMPTY) break;
        v[0] = at(c)[0];
        v[1] = at(c)[1];
        A.sum<2>(S, D, codes[c], v);
        m[c] = v[0].x;
        p[c][0] = v[0].y;
        p[c][1] = v[0].z;
        p[c][2] = v[0].w;
        dp[c][0] = v[1].x;
        dp[c][1] = v[1].y;
        dp[c][2] = v[1].z;
    }
    if (d) return;
    q_couple(c, m, codes, p);
    q_couple(c, m, codes, dp);
    for (int s = 0; s < c; s++) {
        const float im = m[s] > 0.0f ? 1.0f / m[s] : 0.0f;
        at(s)[0] = make_float4(m[s], p[s][0] * im, p[s][1] * im, p[s][2] * im);
        at(s)[1] = make_float4(dp[s][0] * im, dp[s][1] * im, dp[s][2] * im, 0.0f);
    }
}

// Velocity remap of the MUSL re-scatter: per node, the sums as above, coupling of m v^{n+1}
// (Eq. 8), then v~ = ptbar / m.
__global__ __launch_bounds__(TL_QNODE) void k_q_remap(SceneK S, SceneD D, int par)
{
    const int i = (blockIdx.x * TL_QNODE + threadIdx.x) >> 3, d = threadIdx.x & 7;
    if (i >= D.n_qnodes) return;
    const long long g = D.qnodes[i];
    const uint32_t* tab = q_table(S, D, par);
    const uint32_t key0 = tab[g], key1 = S.scap > 1 ? tab[S.NN + g] : TL_QEMPTY;
    const uint32_t key2 = S.scap > 2 ? tab[2 * S.NN + g] : TL_QEMPTY;
    QAround A;
    A.set(S, D, g, d);
    if (key0 == TL_QEMPTY) return;
    const bool one = key1 == TL_QEMPTY, more = key2 != TL_QEMPTY;
    auto mass = [&](int s) { return D.qacc[q_at(S, g, s) * 8]; };
    auto at = [&](int s) { return (float4*)(D.qrs + q_at(S, g, s) * 4); };
    float4 v[1] = {}, u = {}; // the first two slots
#pragma unroll 1
    for (int s = 0; s < (one ? 1 : 2); s++) {
        u = v[0];
        v[0] = *at(s);
        A.sum<1>(S, D, s ? key1 : key0, v);
    }
    if (one) {
        if (d) return;
        const float m = mass(0), im = m > 0.0f ? 1.0f / m : 0.0f;
        *at(0) = make_float4(v[0].x * im, v[0].y * im, v[0].z * im, 0.0f);
        return;
    }
    if (!more) {
        if (d) return;
        const float m0 = mass(0), m1 = mass(1);
        float p0[3] = {u.x, u.y, u.z}, p1[3] = {v[0].x, v[0].y, v[0].z};
        q_couple2(m0, m1, !codes_conflict(key0, key1), p0, p1);
        const float i0 = m0 > 0.0f ? 1.0f / m0 : 0.0f, i1 = m1 > 0.0f ? 1.0f / m1 : 0.0f;
        *at(0) = make_float4(p0[0] * i0, p0[1] * i0, p0[2] * i0, 0.0f);
        *at(1) = make_float4(p1[0] * i1, p1[1] * i1, p1[2] * i1, 0.0f);
        return;
    }
    float m[TL_SCAP_MAX], pt[TL_SCAP_MAX][3];
    uint32_t codes[TL_SCAP_MAX];
    int c = 0;
#pragma unroll 1
    for (; c < S.scap; c++) {
        codes[c] = tab[(long long)c * S.NN + g];
        if (codes[c] == TL_QEMPTY) break;
        v[0] = *at(c);
        A.sum<1>(S, D, codes[c], v);
        m[c] = mass(c);
        pt[c][0] = v[0].x;
        pt[c][1] = v[0].y;
        pt[c][2] = v[0].z;
    }
    if (d) return;
    q_couple(c, m, codes, pt);
    for (int s = 0; s < c; s++) {
        const float im = m[s] > 0.0f ? 1.0f / m[s] : 0.0f;
        *at(s) = make_float4(pt[s][0] * im, pt[s][1] * im, pt[s][2] * im, 0.0f);
    }
}

// ---------------------------------------------------------------------------- G2P
// Per active brick and side key: the box's grid velocities (v^n, dv) into LDS, PIC/FLIP
// update of v and x (Eq. 17), the MUSL re-scatter (69 us, now 40 us for 586 bricks) of
// m_p v_p^{n+1}, and the brick's AABB and speed bound.
__global__ __launch_bounds__(TL_QWG, 6) void k_q_g2p(SceneK S, SceneD D, int par)
{
    __shared__ uint32_t s_keys[TL_SCAP_MAX];
    __shared__ float4 s_grid[2][TL_QBOXP]; // {(1 - beta) v^n + dv} and {v^n + dv} per box node
    __shared__ QRegions3 s_wv;
    __shared__ float s_bb[TL_QWG / 64][7];
    const int bi = blockIdx.x, tid = threadIdx.x;
    const int brick = D.active[bi];
    if (bi == 0 && tid == 0) {
        // end of the substep for this scene: next history stamp and substep index
        // (no later kernel of the substep reads them)
        D.ctr[0] += 1;
        D.ctr[2] += 1;
    }
    const int bx = brick % S.cbx, by = (brick / S.cbx) % S.cby, bz = brick / (S.cbx * S.cby);
    const uint32_t* tab = q_table(S, D, par);
    const int rounds = q_rounds(D, bi);
    const QFirst first(D, bi, rounds);
    if (tid < TL_SCAP_MAX) s_keys[tid] = q_part_keys(S, D, bi)[tid]; // (of the P2G)
    __syncthreads();
    const float dt = S.dt, beta = S.beta;
    float bb[7] = {1e30f, 1e30f, 1e30f, -1e30f, -1e30f, -1e30f, 0.0f};
    for (int k = 0; k < TL_SCAP_MAX && s_keys[k] != TL_QEMPTY; k++) {
        const uint32_t key = s_keys[k];
        s_wv.zero();
        for (int bn = late(tid); bn < TL_QBOXN; bn += TL_QWG) { // absent slots read as zero
            const long long g = q_box_gid(S, bx, by, bz, bn);
            float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
            if (g >= 0) {
                // {m, v^n}, {dv}: the first slot's with its key, nearly always the one
                const float4* q = (const float4*)(D.qacc + (size_t)g * 8);
                const float4 a0 = q[0], b0 = q[1];
                const int s = q_find(S, tab, g, key);
                if (s == 0) {
                    a = a0;
                    b = b0;
                } else if (s > 0) {
                    q = (const float4*)(D.qacc + q_at(S, g, s) * 8);
                    a = q[0];
                    b = q[1];
                } else if (k < S.scap) {
                    // no slot for a sum that the P2G put into this box (its other keys
                    // report that where they are added to the slots)
                    q = (const float4*)q_part(S, D, bi, k) + 2 * bn;
                    const float4 m = q[0], f = q[1];
                    if (m.x != 0.0f || m.y != 0.0f || m.z != 0.0f || m.w != 0.0f || f.x != 0.0f || f.y != 0.0f ||
                        f.z != 0.0f)
                        atomicOr(D.status, TL_ST_LOOKUP);
                }
            }
            const int at = q_box_at(bn % TL_QBOX, (bn / TL_QBOX) % TL_QBOX, bn / 49);
            s_grid[0][at] = make_float4((1.0f - beta) * a.y + b.x, (1.0f - beta) * a.z + b.y, (1.0f - beta) * a.w + b.z, 0.0f);
            s_grid[1][at] = make_float4(a.y + b.x, a.z + b.y, a.w + b.z, 0.0f);
        }
        __syncthreads();
        for (int r = 0; r < rounds; r++) {
            const QFirst q = r ? QFirst(D, bi, rounds, r) : first;
            const int p = q.p;
            if (p < 0 || slot_key(S, q.code) != key) continue;
            const float (&X)[3] = q.X;
            float v[3], u[3];
#pragma unroll
            for (int j = 0; j < 3; j++) {
                v[j] = D.v[at3(p, j)];
                u[j] = D.u[at3(p, j)];
            }
            const float m = S.m_uniform ? S.m0 : D.m[p];
            int c[3];
            const int h = late(tid) >> 6;
            q_cell(bx, by, bz, late(tid) & 63, c);
            QStencil Q;
            q_stencil(S, X, c, h, Q);
            float av[3] = {0.0f, 0.0f, 0.0f}, ax[3] = {0.0f, 0.0f, 0.0f};
            const int ox = Q.lo[0] - (bx * TL_B - 1), oy = Q.lo[1] - (by * TL_B - 1), oz = Q.lo[2] - (bz * TL_B - 1);
            auto gather = [&](auto guard) {
#pragma unroll
                for (int cz = 0; cz < 3; cz++)
#pragma unroll
                    for (int cy = 0; cy < 3; cy++) {
                        const int row = q_box_at(ox, oy, oz + cz) + cy * 14;
                        const float wyz = Q.w[1][cy] * Q.w[2][cz];
                        if (guard.value && wyz == 0.0f) continue;
#pragma unroll
                        for (int cx = 0; cx < 3; cx++) {
                            if (guard.value && Q.w[0][cx] == 0.0f) continue;
                            const float w = Q.w[0][cx] * wyz;
                            const float4 a = s_grid[0][row + cx], b = s_grid[1][row + cx];
                            av[0] += w * a.x;
                            av[1] += w * a.y;
                            av[2] += w * a.z;
                            ax[0] += w * b.x;
                            ax[1] += w * b.y;
                            ax[2] += w * b.z;
                        }
                    }
            };
            if (__any(Q.zero()))
                gather(QGuard<true>{});
            else
                gather(QGuard<false>{});
            float vn1[3];
#pragma unroll
            for (int j = 0; j < 3; j++) {
                vn1[j] = beta * v[j] + av[j];
                const float un = u[j] + dt * ax[j];
                D.v[at3(p, j)] = vn1[j];
                D.u[at3(p, j)] = un;
                const float xa = X[j] + un;
                bb[j] = fminf(bb[j], xa);
                bb[3 + j] = fmaxf(bb[3 + j], xa);
            }
            bb[6] = fmaxf(bb[6], sqrtf(vn1[0] * vn1[0] + vn1[1] * vn1[1] + vn1[2] * vn1[2]));
            // MUSL re-scatter of m v^{n+1} (wave regions as in the P2G)
            const int r0 = h * TL_QREG + (c[1] - by * TL_B) * 12 + c[0] - bx * TL_B, rz = c[2] - bz * TL_B;
#pragma unroll
            for (int cz = 0; cz < 3; cz++)
#pragma unroll
                for (int cy = 0; cy < 3; cy++) {
                    const int row = r0 + q_reg_at(0, 0, rz + cz) + cy * 12;
                    const float wm = Q.w[1][cy] * Q.w[2][cz] * m;
                    if (wm == 0.0f) continue;
                    const float mv[3] = {wm * vn1[0], wm * vn1[1], wm * vn1[2]};
#pragma unroll
                    for (int cx = 0; cx < 3; cx++) {
                        const float wx = Q.w[0][cx];
                        if (cx != 1 && wx == 0.0f) continue;
                        float4 a = s_wv.a[row + cx];
                        a.x += wx * mv[0];
                        a.y += wx * mv[1];
                        a.z += wx * mv[2];
                        s_wv.a[row + cx] = a;
                        asm volatile("" ::: "memory"); // one node at a time, as in the P2G
                    }
                }
        }
        __syncthreads();
        q_flush<3, 4>(S, D, tab, D.qrs, bi, bx, by, bz, k, key, s_wv);
        __syncthreads();
    }
    // brick AABB of x^{n+1} and speed bound (used to skip distant contact work)
    const int lane = tid & 63, wv = tid >> 6;
    for (int q = 0; q < 7; q++) {
        float val = bb[q];
        for (int o = 1; o < 64; o <<= 1) {
            const float other = __shfl_xor(val, o, 64);
            val = (q < 3) ? fminf(val, other) : fmaxf(val, other);
        }
        if (lane == 0) s_bb[wv][q] = val;
    }
    __syncthreads();
    if (tid < 7) {
        float val = s_bb[0][tid];
        for (int w = 1; w < TL_QWG / 64; w++) val = (tid < 3) ? fminf(val, s_bb[w][tid]) : fmaxf(val, s_bb[w][tid]);
        D.aabb[(long long)brick * 8 + tid] = val;
        if (tid == 6 && S.material_contact && val > 0.0f)
            atomicMax(D.hmax + (bi & (TL_HSLOTS - 1)) * TL_HSTRIDE, __float_as_int(val));
    }
}

// --------------------------------------------------------------- F update (MUSL)
// Per active brick and side key: the box's remapped velocities into LDS, then per
// particle F += dt sum_i v~_i (x) grad N_i; the
// rate is kept for viscosity and the plastic projection follows (MAT 1).
template <int MAT>
__global__ __launch_bounds__(TL_QWG) void k_q_F(SceneK S, SceneD D, int par)
{
    __shared__ uint32_t s_keys[TL_SCAP_MAX];
    __shared__ float4 s_vt[TL_QBOXP];
    const int bi = blockIdx.x, tid = threadIdx.x;
    const int brick = D.active[bi];
    const int bx = brick % S.cbx, by = (brick / S.cbx) % S.cby, bz = brick / (S.cbx * S.cby);
    const uint32_t* tab = q_table(S, D, par);
    const int rounds = q_rounds(D, bi);
    const QFirst first(D, bi, rounds);
    if (tid < TL_SCAP_MAX) s_keys[tid] = q_part_keys(S, D, bi)[tid]; // (of the P2G)
    __syncthreads();
    const long long N = S.N;
    const float dt = S.dt;
    for (int k = 0; k < TL_SCAP_MAX && s_keys[k] != TL_QEMPTY; k++) {
        const uint32_t key = s_keys[k];
        for (int bn = late(tid); bn < TL_QBOXN; bn += TL_QWG) { // absent slots read as zero
            const long long g = q_box_gid(S, bx, by, bz, bn);
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (g >= 0) {
                const float4 v0 = *(const float4*)(D.qrs + (size_t)g * 4); // (as in the G2P)
                const int s = q_find(S, tab, g, key);
                if (s == 0)
                    v = v0;
                else if (s > 0)
                    v = *(const float4*)(D.qrs + q_at(S, g, s) * 4);
            }
            s_vt[q_box_at(bn % TL_QBOX, (bn / TL_QBOX) % TL_QBOX, bn / 49)] = v;
        }
        __syncthreads();
        for (int r = 0; r < rounds; r++) {
            const QFirst q = r ? QFirst(D, bi, rounds, r) : first;
            const int p = q.p;
            if (p < 0 || slot_key(S, q.code) != key) continue;
            const float (&X)[3] = q.X;
            int c[3];
            const int h = late(tid) >> 6;
            q_cell(bx, by, bz, late(tid) & 63, c);
            QStencil Q;
            q_stencil(S, X, c, h, Q);
            float Lg[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            const int ox = Q.lo[0] - (bx * TL_B - 1), oy = Q.lo[1] - (by * TL_B - 1), oz = Q.lo[2] - (bz * TL_B - 1);
            auto gather = [&](auto guard) {
#pragma unroll
                for (int cz = 0; cz < 3; cz++)
#pragma unroll
                    for (int cy = 0; cy < 3; cy++) {
                        const int row = q_box_at(ox, oy, oz + cz) + cy * 14;
                        const float wyz = Q.w[1][cy] * Q.w[2][cz];
                        if (guard.value && wyz == 0.0f) continue;
                        float sg[3] = {0, 0, 0}, sw[3] = {0, 0, 0}; // sums of gx v and of wx v along the row
#pragma unroll
                        for (int cx = 0; cx < 3; cx++) {
                            if (guard.value && Q.w[0][cx] == 0.0f) continue;
                            const float4 n = s_vt[row + cx];
                            const float v[3] = {n.x, n.y, n.z};
#pragma unroll
                            for (int a = 0; a < 3; a++) {
                                sg[a] += Q.g[0][cx] * v[a];
                                sw[a] += Q.w[0][cx] * v[a];
                            }
                        }
#pragma unroll
                        for (int a = 0; a < 3; a++) {
                            Lg[3 * a + 0] += sg[a] * wyz;
                            Lg[3 * a + 1] += sw[a] * (Q.g[1][cy] * Q.w[2][cz]);
                            Lg[3 * a + 2] += sw[a] * (Q.w[1][cy] * Q.g[2][cz]);
                        }
                    }
            };
            if (__any(Q.zero()))
                gather(QGuard<true>{});
            else
                gather(QGuard<false>{});
            float H[9];
            bool fin = true;
#pragma unroll
            for (int a = 0; a < 9; a++) {
                H[a] = D.H[at9(N, p, a)] + dt * Lg[a];
                D.H[at9(N, p, a)] = H[a];
                fin = fin && isfinite(H[a]);
            }
            if (!fin) atomicOr(D.status, TL_ST_NONFINITE);
            if constexpr (MAT == 1) {
                if (S.visc > 0.0f)
#pragma unroll
                    for (int a = 0; a < 9; a++) D.Fdot[at9(N, p, a)] = Lg[a];
                if (S.ystress > 0.0f) {
                    float Gp[9], K[9];
#pragma unroll
                    for (int a = 0; a < 9; a++) Gp[a] = D.Gp[at9(N, p, a)];
#pragma unroll
                    for (int i = 0; i < 3; i++)
#pragma unroll
                        for (int j = 0; j < 3; j++) {
                            float kk = H[3 * i + j] + Gp[3 * i + j];
#pragma unroll
                            for (int l = 0; l < 3; l++) kk += H[3 * i + l] * Gp[3 * l + j];
                            K[3 * i + j] = kk;
                        }
                    float mu, lam;
                    lame(S, S.e_uniform ? 0.0f : D.E[p], mu, lam);
                    if (vm_project(mu, S.ystress, K, Gp))
#pragma unroll
                        for (int a = 0; a < 9; a++) D.Gp[at9(N, p, a)] = Gp[a];
                }
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ host launches
extern "C" {

// the transfers of one substep of a single scene with the quadratic stencil, in
// order, with the table of parity par; timing class per launch via the callback
hipError_t tl_launch_quad(const TlLaunch* L, int par, int stage)
{
    const SceneK& S = *L->S;
    const SceneD& D = *L->D;
    const int nb = D.n_active;
    const int nn = (int)(((long long)D.n_qnodes * 8 + TL_QNODE - 1) / TL_QNODE);
    if (nb == 0) return hipSuccess;
    switch (stage) {
    case 0:
        k_q_slots<<<nb, TL_QWG, 0, L->st>>>(S, D, par);
        break;
    case 1:
        if (L->general)
            k_q_p2g<1><<<nb, TL_QWG, 0, L->st>>>(S, D, par);
        else
            k_q_p2g<0><<<nb, TL_QWG, 0, L->st>>>(S, D, par);
        break;
    case 2:
        if (nn) k_q_grid<<<nn, TL_QNODE, 0, L->st>>>(S, D, par);
        break;
    case 3:
        k_q_g2p<<<nb, TL_QWG, 0, L->st>>>(S, D, par);
        break;
    case 4:
        if (nn) k_q_remap<<<nn, TL_QNODE, 0, L->st>>>(S, D, par);
        break;
    case 5:
        if (L->general)
            k_q_F<1><<<nb, TL_QWG, 0, L->st>>>(S, D, par);
        else
            k_q_F<0><<<nb, TL_QWG, 0, L->st>>>(S, D, par);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

} // extern "C"
