// gpr_kernels.hip -- gfx950 kernels of the Gen.ParRep hot path.
//
// Two stepping paths share every arithmetic routine, so they give bit-identical results:
//   plain      : per step, k_integrate (B A O A of Eq. 1's BAOAB discretisation) and k_forces (bonded
//                and pair forces, the closing B kick, pair-list rebuild when due); observables and
//                state tests as separate launches;
//   persistent : k_persist (k_persist_batch: several systems) advances each replica by one to 32
//                workgroups for a whole check period, its positions, parameters, velocities and
//                forces in LDS; k_persist_small does so for small replicas, one workgroup each, with
//                their bonded terms in LDS too and no pair lists.
// Gen.ParRep bookkeeping (Sec. 2.4.1 branching and Gelman-Rubin, Sec. 2.4.2 exit vote)
// runs in k_check / k_clone once per check.
#include "gpr_kernels.h"

namespace gpr {

// ------------------------------------------------------------------ small helpers
__device__ __forceinline__ float kick(float v, float F, float h, float im) { return v + (h * F) * im; }

// Sum over the wave, in every lane: pairs, quads, eights and rows of 16 by DPP moves, the four rows by
// scalar adds.  All lanes are active.  (Six shuffles through LDS took 0.3 us of a toy step.)
template <int CTRL>
__device__ __forceinline__ long long dpp_ll(long long v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xF, 0xF, true);
    return (long long)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ long long wave_sum_ll(long long v)
{
    v += dpp_ll<0xB1>(v);                                   // quad_perm [1, 0, 3, 2]
    v += dpp_ll<0x4E>(v);                                   // quad_perm [2, 3, 0, 1]
    v += dpp_ll<0x141>(v);                                  // row_half_mirror
    v += dpp_ll<0x140>(v);                                  // row_mirror
    long long s = 0;
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)v, 16 * row);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), 16 * row);
        s += (long long)(((unsigned long long)hi << 32) | lo);
    }
    return s;
}

// the P = 4 lanes of one atom are consecutive: (s0 + s1) + (s2 + s3) in a fixed order
__device__ __forceinline__ float quad_sum(float v)
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    return v;
}

struct PosLDS {
    const float4 *xs;
    __device__ float3 operator()(int a) const { const float4 p = xs[a]; return make_float3(p.x, p.y, p.z); }
};
struct PosGlob {
    const GPR_GLOBAL float *x;
    int np;
    __device__ float3 operator()(int a) const { return make_float3(x[a], x[np + a], x[2 * np + a]); }
};

__device__ __forceinline__ float3 neg3(float3 f) { return make_float3(-f.x, -f.y, -f.z); }

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni64(long long v)
{
    const int lo = uni((int)(unsigned)v), hi = uni((int)(v >> 32));
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// The value again, with its origin hidden: what is computed from it inside a loop stays there.  The
// step loops of the persistent kernels take their array addresses from such values, a few
// instructions per phase; hoisted out of the loop, as the compiler does with invariants, the
// addresses of all phases together exceed the registers, and every step reloads them from scratch.
__device__ __forceinline__ int fresh_s(int v) { v = uni(v); asm volatile("" : "+s"(v)); return v; }
__device__ __forceinline__ int fresh_v(int v) { asm volatile("" : "+v"(v)); return v; }

// ------------------------------------------------------------------ bonded terms of an atom range
// One unit of 64 terms of a kind (records w, p of the lane): adds the fixed-point forces on the
// atoms of the range to fa (LDS; component d of atom a at fa[(a - a0) sa + d sd]); EDGE: only on the
// atoms the range owns.  ENERGY: returns the lane's energy, counted by one range per term.
struct ForceLDS {
    long long *fa;
    int a0, sa, sd;
};
template <int KIND, bool EDGE, bool ENERGY, class Pos>
__device__ __forceinline__ long long bonded_terms(const uint2 w, const float4 p, const Pos &pos, const ForceLDS &F, const FixConsts &K)
{
    auto add = [&](unsigned field, float3 f) {
        if (!EDGE || (field & BONDED_ATOMS)) {
            long long *const t = F.fa + ((int)(field & (BONDED_ATOMS - 1)) - F.a0) * F.sa;
            lds_add(t, fix_f(K, f.x));
            lds_add(t + F.sd, fix_f(K, f.y));
            lds_add(t + 2 * F.sd, fix_f(K, f.z));
        }
    };
    auto at = [&](unsigned field) { return pos((int)(field & (BONDED_ATOMS - 1))); };
    if (!(w.y & 0x8000u)) return 0;
    const unsigned f0 = w.x, f1 = w.x >> 16, f2 = w.y, f3 = w.y >> 16;
    float u = 0.f;
    if (KIND == 0) {
        float3 fi;
        u = term_bond(at(f0), at(f1), make_float2(p.x, p.y), fi);
        add(f0, fi);
        add(f1, neg3(fi));
    } else if (KIND == 1) {
        float3 fi, fk;
        u = term_angle(at(f0), at(f1), at(f2), make_float2(p.x, p.y), fi, fk);
        add(f0, fi);
        add(f2, fk);
        add(f1, make_float3(-fi.x - fk.x, -fi.y - fk.y, -fi.z - fk.z));
    } else if (KIND == 2) {
        float3 fi, fj, fk, fl;
        u = term_torsion(at(f0), at(f1), at(f2), at(f3), p, fi, fj, fk, fl);
        add(f0, fi);
        add(f1, fj);
        add(f2, fk);
        add(f3, fl);
    } else if (KIND == 3) {
        const float3 x = at(f0);
        const float dx = x.x - p.x, dy = x.y - p.y, dz = x.z - p.z;
        add(f0, make_float3(-p.w * dx, -p.w * dy, -p.w * dz));
        if (ENERGY) u = 0.5f * p.w * (dx * dx + dy * dy + dz * dz);
    } else {
        float3 fi;
        u = term_pair14(at(f0), at(f1), p, fi);
        add(f0, fi);
        add(f1, neg3(fi));
    }
    return ENERGY && (f2 & 0x4000u) ? fix_f(K, u) : 0;
}

// Units [u0, u1) of the records bi, bp, taken in turn by waves wv = 0 .. nwv - 1 of the range's
// workgroup; each wave reads its next unit's records while it computes one, since what bounds the
// terms otherwise is the latency of reading them (the records come from the L2: the pair lists
// stream through the L1).
template <bool ENERGY, class Pos>
__device__ __forceinline__ long long bonded_units(const uint2 *bi, const float4 *bp, int u0, int u1, const Pos &pos,
                                                  const ForceLDS &F, int wv, int nwv, int lane)
{
    const FixConsts K = fix_consts();
    long long e = 0;
    int u = u0 + wv;
    uint2 w = make_uint2(0u, 0u);
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
    if (u < u1) {
        w = gld(gconst(bi) + (64 * u + lane));
        p = gld(gconst(bp) + (64 * u + lane));
    }
    while (u < u1) {
        const uint2 cw = w;
        const float4 cp = p;
        u += nwv;
        if (u < u1) {
            w = gld(gconst(bi) + (64 * u + lane));
            p = gld(gconst(bp) + (64 * u + lane));
        }
        const int kind = __builtin_amdgcn_readfirstlane((int)(((cw.x >> 14) & 3u) | ((cw.x >> 28) & 12u)));
        switch (kind) {
        case 0: e += bonded_terms<0, false, ENERGY>(cw, cp, pos, F, K); break;
        case 1: e += bonded_terms<1, false, ENERGY>(cw, cp, pos, F, K); break;
        case 2: e += bonded_terms<2, false, ENERGY>(cw, cp, pos, F, K); break;
        case 3: e += bonded_terms<3, false, ENERGY>(cw, cp, pos, F, K); break;
        case 4: e += bonded_terms<4, false, ENERGY>(cw, cp, pos, F, K); break;
        case BONDED_EDGE + 0: e += bonded_terms<0, true, ENERGY>(cw, cp, pos, F, K); break;
        case BONDED_EDGE + 1: e += bonded_terms<1, true, ENERGY>(cw, cp, pos, F, K); break;
        case BONDED_EDGE + 2: e += bonded_terms<2, true, ENERGY>(cw, cp, pos, F, K); break;
        case BONDED_EDGE + 3: e += bonded_terms<3, true, ENERGY>(cw, cp, pos, F, K); break;
        default: e += bonded_terms<4, true, ENERGY>(cw, cp, pos, F, K); break;
        }
    }
    return e;
}

// the double well of the toy system, U = (x^2 - 1)^2 + 2 y^2
__device__ __forceinline__ float toy_force(float x, float y, float &fx, float &fy)
{
    const float x2m1 = x * x - 1.0f;
    fx = -4.0f * x * x2m1;
    fy = -4.0f * y;
    return x2m1 * x2m1 + 2.0f * y * y;
}

// ------------------------------------------------------------------ pair search
// A value that every lane holds alike, as a scalar
__device__ __forceinline__ float uniform_f(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

// min / max over each row of 16 lanes and over each eight lanes, in every lane
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true)); }
constexpr int ROR8 = 0x128, ROR4 = 0x124, ROR2 = 0x122, ROR1 = 0x121, SWAP1 = 0xB1, SWAP2 = 0x4E, HALF_MIRROR = 0x141;
__device__ __forceinline__ float row_min(float v)
{
    v = fminf(v, dpp_f<ROR8>(v));
    v = fminf(v, dpp_f<ROR4>(v));
    v = fminf(v, dpp_f<ROR2>(v));
    return fminf(v, dpp_f<ROR1>(v));
}
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, dpp_f<ROR8>(v));
    v = fmaxf(v, dpp_f<ROR4>(v));
    v = fmaxf(v, dpp_f<ROR2>(v));
    return fmaxf(v, dpp_f<ROR1>(v));
}
__device__ __forceinline__ float oct_min(float v)
{
    v = fminf(v, dpp_f<SWAP1>(v));
    v = fminf(v, dpp_f<SWAP2>(v));
    return fminf(v, dpp_f<HALF_MIRROR>(v));
}
__device__ __forceinline__ float oct_max(float v)
{
    v = fmaxf(v, dpp_f<SWAP1>(v));
    v = fmaxf(v, dpp_f<SWAP2>(v));
    return fmaxf(v, dpp_f<HALF_MIRROR>(v));
}

// The point that the search's tiles take positions relative to: near the middle of the replica
__device__ __forceinline__ float3 search_centre(const GPR_LDS gv_f4 *xs, int n)
{
    const gv_f4 a = xs[0], b = xs[n / 3], c = xs[(2 * n) / 3], d = xs[n - 1];
    return make_float3(uniform_f(0.25f * (a.x + b.x + c.x + d.x)), uniform_f(0.25f * (a.y + b.y + c.y + d.y)),
                       uniform_f(0.25f * (a.z + b.z + c.z + d.z)));
}

constexpr float TILE_SHORT = 1.0f - 9.5367431640625e-7f;       // 1 - 2^-20 (see search_task)
constexpr float TILE_MAX2 = 4096.0f;                           // (64 nm)^2 (see search_task)

// Bounding boxes of blocks of BLK consecutive atoms (chain-local, so compact), eight lanes a block:
// the middle, and in one word the half extents in units of 1/128 nm, rounded up (a byte each; all
// three 255: too large to say) under the block's mask of light atoms, which is kept from what the
// word held (the caller set it once).  Each atom's |d|^2 - list2_j for the tiles (d from the centre
// c) takes the place of its sigma/2, which the caller restores after the search.  True when an atom is too far out
// for the tiles.
__device__ __forceinline__ bool block_boxes(const GPR_CONST Dev &S, const GPR_LDS gv_f4 *xs, GPR_LDS gv_f2 *pp, GPR_LDS gv_f4 *box,
                                            float3 c, int tid, int nthr)
{
    const int n = S.n, nblk = (n + BLK - 1) / BLK;
    const float list2_j = S.list2_j;
    bool out = false;
    for (int a = tid; a < BLK * nblk; a += nthr) {
        const int t = a / BLK, k = a % BLK;
        const unsigned light = __float_as_uint(box[t].w) >> 24;
        const gv_f4 x = xs[a];
        const bool real = a < n;
        const float dx = x.x - c.x, dy = x.y - c.y, dz = x.z - c.z;
        const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        pp[a].x = fmaf(d2, TILE_SHORT, ((light >> k) & 1u) ? -list2_j : 0.0f);
        out |= real && !(d2 < TILE_MAX2);
        const float big = 3.0e38f;
        const float lx = oct_min(real ? x.x : big), hx = oct_max(real ? x.x : -big);
        const float ly = oct_min(real ? x.y : big), hy = oct_max(real ? x.y : -big);
        const float lz = oct_min(real ? x.z : big), hz = oct_max(real ? x.z : -big);
        // (half the box, and what rounding may take from the distance to it: 2^-20 of a coordinate)
        auto units = [](float l, float h) {
            const float e = 0.5f * (h - l) + 9.5e-7f * fmaxf(fabsf(l), fabsf(h));
            return e < 1.97f ? (unsigned)(e * 128.0f) + 1u : 255u;      // (a NaN too)
        };
        const unsigned ux = units(lx, hx), uy = units(ly, hy), uz = units(lz, hz);
        const unsigned ext = (ux == 255u || uy == 255u || uz == 255u) ? 0xFFFFFFu : ux | (uy << 8) | (uz << 16);
        if (k == 0) {
            const gv_f4 b = {0.5f * (lx + hx), 0.5f * (ly + hy), 0.5f * (lz + hz), __uint_as_float(ext | (light << 24))};
            box[t] = b;
        }
    }
    return out;
}

// Entry 4 p + c of the table that packs a lane's kept candidates after the c entries of its pending
// group: of the four 16-bit values in (X, Y) those whose bit is set in p, in order, from slot c of
// eight; as the byte selectors of four v_perm_b32 (zeros in the other slots): the pending group's
// two words, then the two of the group after it
struct PickTable {
    unsigned w[64][4];
};
constexpr PickTable make_pick()
{
    PickTable t{};
    for (int e = 0; e < 64; ++e) {
        unsigned slot[8] = {0x0C0Cu, 0x0C0Cu, 0x0C0Cu, 0x0C0Cu, 0x0C0Cu, 0x0C0Cu, 0x0C0Cu, 0x0C0Cu};
        int m = e & 3;
        for (unsigned v = 0; v < 4; ++v)
            if ((e >> (2 + v)) & 1) slot[m++] = 2 * v | ((2 * v + 1) << 8);
        for (int k = 0; k < 4; ++k) t.w[e][k] = slot[2 * k] | (slot[2 * k + 1] << 16);
    }
    return t;
}
__device__ __constant__ const PickTable pick_table = make_pick();

// The list entries (8 j) of block b's atoms j of residue q mod 4: the first in the low half, the second in
// the high half.  Unsigned: from block 512 on the product passes 2^31, and the halves are meant to wrap.
__host__ __device__ constexpr unsigned block_entries(unsigned b, unsigned q) { return b * (8u * BLK * 0x10001u) + 0x200000u + q * 0x80008u; }
static_assert(block_entries(0, 3) == 0x00380018u && block_entries(511, 0) == 0x7FE07FC0u && block_entries(512, 1) == 0x80288008u &&
                  block_entries(767, 3) == 0xBFF8BFD8u && block_entries(1023, 3) == 0xFFF8FFD8u,
              "entries of the last blocks of any accepted size");

// Pair lists of the atoms [iw, iw + 16) below iend, by one wave; all 64 lanes call it together with
// the same arguments.  Lane 16 q + k owns sub-list (i, q) of atom i = iw + k: partners j = q (mod P),
// j != i, not excluded, r^2 < list2 of the two atoms' classes, in ascending order; entry e is the
// 16-bit word e % 4 of group e / 4, holding 8 j (the byte offset of j's LJ parameters in LDS, half
// that of its position); the last group is padded with the dummy atom n.  allpairs: no
// distance tests (vacuum, no cutoff).  After block_boxes, with its boxes and centre.
//
// Culling is wave-wide: each lane tests one block's box against the box of the wave's atoms, and
// the near blocks queue up in the wave's LDS scratch wblk (ascending).  Two blocks at a time are
// tested by one v_mfma_f32_16x16x4_f32: with d the positions relative to c, D = |d_j|^2 + |d_i|^2 -
// list2 - 2 d_i . d_j for 16 partners (rows) x 16 atoms (columns), the sum over K = 4 taking (d_x,
// d_y, d_z, |d_j|^2 - list2_j) of the partner against (-2 d_i, 1) of the atom, and a pair is listed when D < 0.
// Row 4 q + v holds atom 4 (v % 2) + q of block v / 2, so the four values a lane gets are its own
// candidates in order, one sign bit each: seven vector instructions for 256 pairs, where testing
// them one by one takes nine for 64.  A list may hold more pairs than needed but never fewer: the
// squares are taken 2^-20 short, which covers the rounding of D (each of its six terms is at most
// |d_i|^2 + |d_j|^2); with an atom more than 64 nm from c (`wide`), where that would admit pairs
// 0.008 nm^2 too far, the tiles take the distances directly.
// The kept candidates of a lane (at most four per tile) are packed and shifted into place by byte
// permutes whose selectors the lanes hold (entry `lane` of the table) and read from each other.
// Excluded partners within 32 atoms (and the atom itself) are dropped only in tiles that may hold
// some; farther ones are merged out against the atom's ascending list far_j.
// Bound by VALU issue: about 27 instructions per tile, 16 tiles a task on the 2,432-atom system; of a
// rebuild's 30 us there (four groups) the tasks take 22: the scattered stores of finished groups 7,
// the tiles 6, culling and a task's set-up 5, the exclusions 4.
// UNR tiles are read at a time (more registers, fewer exposed LDS latencies).
template <int UNR, bool PAD>
__device__ __forceinline__ int search_task(const GPR_CONST Dev &S, int r, int iw, int iend, const GPR_LDS gv_f4 *xs,
                                           const GPR_LDS gv_f2 *pp, const GPR_LDS gv_f4 *box, GPR_LDS int *wblk, float3 c,
                                           bool wide, bool allpairs)
{
    const int n = S.n, Kg = S.Kg, span = S.excl_span;
    const unsigned stride = (unsigned)S.np * P;
    const int lane = threadIdx.x & 63, q = lane >> 4, k16 = lane & 15;
    const int i = iw + k16;
    const bool valid = i < iend;
    const gv_u4 sel = *(const GPR_GLOBAL gv_u4 *)gconst(&pick_table.w[lane][0]);
    const gv_f4 pi = xs[valid ? i : n];
    // box of the wave's valid atoms (the same in every row of lanes)
    const float big = 3.0e38f;
    const float mnx = uniform_f(row_min(valid ? pi.x : big)), mxx = uniform_f(row_max(valid ? pi.x : -big));
    if (!(mnx <= mxx)) return 0;                                // no valid atom in this wave
    const float mny = uniform_f(row_min(valid ? pi.y : big)), mxy = uniform_f(row_max(valid ? pi.y : -big));
    const float mnz = uniform_f(row_min(valid ? pi.z : big)), mxz = uniform_f(row_max(valid ? pi.z : -big));
    const float bx = 0.5f * (mnx + mxx), by = 0.5f * (mny + mxy), bz = 0.5f * (mnz + mxz);
    const float hx = 0.5f * (mxx - mnx) * 1.00001f + 1e-6f * fabsf(bx);
    const float hy = 0.5f * (mxy - mny) * 1.00001f + 1e-6f * fabsf(by);
    const float hz = 0.5f * (mxz - mnz) * 1.00001f + 1e-6f * fabsf(bz);
    const float rl2 = S.rl * S.rl * 1.00001f;
    // atom i: exclusions, list radius, MFMA operand and accumulator start
    const unsigned long long ex = (valid ? gconst(S.excl)[i] : 0ull) | (1ull << 32);
    const bool ilight = (__float_as_uint(box[(valid ? i : iw) / BLK].w) >> (24 + (i & (BLK - 1)))) & 1u;
    const float list2 = allpairs ? 1.0e30f : (ilight ? S.list2_light : S.list2_heavy);
    const float dix = pi.x - c.x, diy = pi.y - c.y, diz = pi.z - c.z;
    const float ci = valid ? fmaf(fmaf(diz, diz, fmaf(diy, diy, dix * dix)), TILE_SHORT, -list2) : 1.0e30f;
    const float bop = q == 0 ? -2.0f * dix : (q == 1 ? -2.0f * diy : (q == 2 ? -2.0f * diz : 1.0f));
    // the operand this lane feeds: component q of the partner in row k16, atom jt of the tile's block jb
    const float cq = q == 0 ? c.x : (q == 1 ? c.y : (q == 2 ? c.z : 0.0f));
    const int jb = (k16 >> 1) & 1, jt = 4 * (k16 & 1) + (k16 >> 2);
    const GPR_LDS char *const opnd = q < 3 ? (const GPR_LDS char *)xs + 16 * jt + 4 * q : (const GPR_LDS char *)pp + 8 * jt;
    const int opsh = q < 3 ? 7 : 6;                             // log2 of a block's bytes there
    static_assert(BLK == 8, "operand addresses take a block as 8 x 16 or 8 x 8 bytes");
    int flo = 0, fhi = 0;
    const GPR_GLOBAL int *const fj = gconst(S.far_j);
    const bool has_far = S.has_far != 0;
    if (has_far && valid) { flo = gconst(S.far_start)[i]; fhi = gconst(S.far_start)[i + 1]; }
    const bool special = wide || has_far;
    // the replica's lists (a scalar base) and the byte offset of this lane's word in them: group g of
    // sub-list (i, q) is word g * np * P + i * P + q
    GPR_GLOBAL char *const Lr = (GPR_GLOBAL char *)gmut(S.nbl) + (size_t)r * Kg * stride * 8;
    const unsigned step = stride * 8, end = (unsigned)Kg * step;
    unsigned off = (unsigned)((valid ? i : 0) * P + q) * 8;
    const int nblk = (n + BLK - 1) / BLK;
    unsigned plo = 0u, phi = 0u;                                // the entries of the unfinished group
    unsigned cnt4 = 0u;                                         // four times the entries so far
    int nq = 0;                                                 // near blocks queued in wblk
    constexpr int CHUNK = WBLK - 8;                             // the rest of a batch waits in the queue
    static_assert(2 * UNR <= 8, "the queue holds a chunk and the rest of a batch");
    for (int cb = 0; cb < nblk; cb += CHUNK) {
        const int b = cb + lane;
        bool near = b < nblk && lane < CHUNK;
        if (near && !allpairs) {
            // distance between the two boxes, per axis
            const gv_f4 m = box[b];
            const unsigned w = __float_as_uint(m.w);
            const float dx = fmaxf(0.f, fabsf(m.x - bx) - fmaf((float)(w & 255u), 0.0078125f, hx));
            const float dy = fmaxf(0.f, fabsf(m.y - by) - fmaf((float)((w >> 8) & 255u), 0.0078125f, hy));
            const float dz = fmaxf(0.f, fabsf(m.z - bz) - fmaf((float)((w >> 16) & 255u), 0.0078125f, hz));
            near = fmaf(dz, dz, fmaf(dy, dy, dx * dx)) < rl2 || (w & 0xFFFFFFu) == 0xFFFFFFu;
        }
        const unsigned long long m = __ballot(near);
        __builtin_amdgcn_wave_barrier();
        if (near) wblk[nq + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = b;
        nq += __popcll(m);
        const bool last = cb + CHUNK >= nblk;
        if (last && lane < 2 * UNR && nq + lane < WBLK) wblk[nq + lane] = 0;    // slots read past the end, masked below
        __builtin_amdgcn_wave_barrier();
        int k0 = 0;
        while (nq - k0 >= 2 * UNR || (last && k0 < nq)) {
            int ent[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) ent[u] = wblk[k0 + 2 * u + jb];
            float val[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) val[u] = *(const GPR_LDS float *)(opnd + (ent[u] << opsh));
            __builtin_amdgcn_sched_barrier(0);                  // keep the reads ahead of the tests
            gv_f4 D[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const gv_f4 c4 = {ci, ci, ci, ci};
                D[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(val[u] - cq, bop, c4, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int left = nq - (k0 + 2 * u);             // blocks of the tile that are in the queue
                if (left <= 0) continue;
                const int b0 = __builtin_amdgcn_readlane(ent[u], 0), b1 = __builtin_amdgcn_readlane(ent[u], 2);
                const unsigned live = left == 1 ? 3u : 15u;
                // bit v: candidate v is within its list radius
                unsigned p = __float_as_uint(D[u][3]) >> 31;
                p = __builtin_amdgcn_alignbit(p, __float_as_uint(D[u][2]), 31);
                p = __builtin_amdgcn_alignbit(p, __float_as_uint(D[u][1]), 31);
                p = __builtin_amdgcn_alignbit(p, __float_as_uint(D[u][0]), 31);
                p &= live;
                const bool self = (b0 * BLK + BLK > iw - span && b0 * BLK < iw + 16 + span) ||
                                  (b1 * BLK + BLK > iw - span && b1 * BLK < iw + 16 + span);
                if (self || special) {
                    if (wide) {
                        p = 0u;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int bv = v < 2 ? b0 : b1, t = 4 * (v & 1) + q;
                            const gv_f4 xj = xs[bv * BLK + t];
                            const float dx = pi.x - xj.x, dy = pi.y - xj.y, dz = pi.z - xj.z;
                            const float lj = ((__float_as_uint(box[bv].w) >> (24 + t)) & 1u) ? S.list2_j : 0.f;
                            p |= (unsigned)(valid && fmaf(dz, dz, fmaf(dy, dy, dx * dx)) < list2 + lj) << v;
                        }
                        p &= live;
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int o = (v < 2 ? b0 : b1) * BLK + 4 * (v & 1) + q - i + 32;
                        const unsigned drop = (unsigned)((unsigned)o < 64u) & (unsigned)(ex >> (o & 63));
                        p &= ~((drop & 1u) << v);
                    }
                    if (has_far && __ballot(flo < fhi) != 0ull) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int j = (v < 2 ? b0 : b1) * BLK + 4 * (v & 1) + q;
                            if ((p >> v) & 1u) {
                                while (flo < fhi && fj[flo] < j) ++flo;
                                if (flo < fhi && fj[flo] == j) p &= ~(1u << v);
                            }
                        }
                    }
                }
                const int e4 = (int)((p << 4) | (cnt4 & 12u));
                const unsigned X = block_entries((unsigned)b0, (unsigned)q), Y = block_entries((unsigned)b1, (unsigned)q);
                const unsigned llo = plo | __builtin_amdgcn_perm(Y, X, (unsigned)__builtin_amdgcn_ds_bpermute(e4, (int)sel.x));
                const unsigned lhi = phi | __builtin_amdgcn_perm(Y, X, (unsigned)__builtin_amdgcn_ds_bpermute(e4, (int)sel.y));
                const unsigned olo = __builtin_amdgcn_perm(Y, X, (unsigned)__builtin_amdgcn_ds_bpermute(e4, (int)sel.z));
                const unsigned ohi = __builtin_amdgcn_perm(Y, X, (unsigned)__builtin_amdgcn_ds_bpermute(e4, (int)sel.w));
                const unsigned nc4 = cnt4 + 4u * (unsigned)__popc(p);
                const bool full = (nc4 ^ cnt4) > 15u;           // the pending group is complete
                if (full && off < end) {
                    const gv_u2 w = {llo, lhi};
                    *(GPR_GLOBAL gv_u2 *)(Lr + off) = w;
                }
                off += full ? step : 0u;
                plo = full ? olo : llo;
                phi = full ? ohi : lhi;
                cnt4 = nc4;
            }
            k0 += 2 * UNR;
        }
        if (!last) {
            // blocks short of a batch wait for the next chunk's
            __builtin_amdgcn_wave_barrier();
            const int rest = nq - k0;
            const int t = lane < rest ? wblk[k0 + lane] : 0;
            __builtin_amdgcn_wave_barrier();
            if (lane < rest) wblk[lane] = t;
            nq = rest;
        }
    }
    // a partial group is padded; PAD: the four sub-lists of an atom to the same number of groups
    // with the far-away atom n (exact zeros), so that one count (the largest, returned) serves the
    // atom's four lanes; the counts array keeps each sub-list's own count
    const int ng = min((int)((cnt4 + 15u) >> 4), Kg);
    const unsigned pad = (unsigned)n * 0x00080008u;
    if (valid && (cnt4 & 12u) != 0u && off < end) {
        const unsigned k = (cnt4 >> 2) & 3u;
        const gv_u2 w = {k == 1 ? plo | (pad << 16) : plo, k == 3 ? phi | (pad << 16) : pad};
        *(GPR_GLOBAL gv_u2 *)(Lr + off) = w;
        off += step;
    }
    int kq = ng;
    if (PAD) {
        kq = max(ng, __shfl_xor(ng, 16, 64));
        kq = max(kq, __shfl_xor(kq, 32, 64));
        if (valid)
            for (int w = ng; w < kq; ++w, off += step) {
                const gv_u2 pw = {pad, pad};
                *(GPR_GLOBAL gv_u2 *)(Lr + off) = pw;
            }
    }
    if (valid) {
        gmut(S.nbc)[(size_t)r * stride + (size_t)i * P + q] = (unsigned short)ng;
        if ((int)(cnt4 >> 2) > 4 * Kg) atomicOr(&S.err[ERR_LIST], 1);
    }
    return kq;
}

// ------------------------------------------------------------------ nonbonded partial sum of one lane
// Lennard-Jones + Coulomb (vacuum when krf = crf = 0 and rc2 = inf; reaction field
// otherwise) of one pair, accumulated into (fx, fy, fz) and, with energy, U/2 into e.
__device__ __forceinline__ void pair_term(const float4 pi, const float2 ppi, const float4 pj, const float2 ppj,
                                          float rc2, float krf2, float krf, float crf, bool energy,
                                          float &fx, float &fy, float &fz, float &e)
{
    const float dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
    const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    const float ri = __builtin_amdgcn_rsqf(r2);
    const float r2i = ri * ri;
    const float sg = ppi.x + ppj.x;
    const float s2 = (sg * sg) * r2i;
    const float s6 = (s2 * s2) * s2;
    const float e4 = ppi.y * ppj.y;
    const float qq = pi.w * pj.w;
    // -dU/dr / r = e4 r2i (12 s6^2 - 6 s6) + qq (ri r2i - 2 krf)
    const float lj = (e4 * r2i) * (s6 * fmaf(12.0f, s6, -6.0f));
    const float fs0 = fmaf(qq, fmaf(ri, r2i, -krf2), lj);
    const bool in = r2 < rc2;
    const float fs = in ? fs0 : 0.0f;
    fx = fmaf(fs, dx, fx);
    fy = fmaf(fs, dy, fy);
    fz = fmaf(fs, dz, fz);
    if (energy) {
        const float u = fmaf(e4 * s6, s6 - 1.0f, qq * (fmaf(krf, r2, ri) - crf));
        e = in ? fmaf(0.5f, u, e) : e;
    }
}

// The pair loop's parameters, as values (read once per step in a persistent launch)
struct NbConsts {
    const uint2 *nbl;
    const unsigned short *nbc;
    int np, Kg;
    float rc2, krf, crf;
};
__device__ __forceinline__ NbConsts nb_consts(const Dev &S)
{
    NbConsts k;
    k.nbl = S.nbl; k.nbc = S.nbc; k.np = S.np; k.Kg = S.Kg; k.rc2 = S.rc2; k.krf = S.krf; k.crf = S.crf;
    return k;
}

// Sum over one sub-list of ng words: word g at byte off + g step of its replica's lists.  Returns
// (F_x, F_y, F_z, sum U/2).  The next word is read one group ahead, without a branch, the offset
// stopping at the last word (which is then read again, from the cache: the row after it would be
// one more uncached read per sub-list).  Bound by VALU issue, 28 instructions per pair: with the
// read ahead kept in place and two address instructions per pair instead of four, the force phase
// of the persistent kernel (2,432 atoms x 64 replicas) went from 13.7 to 12.2 us.
template <bool ENERGY>
__device__ __forceinline__ float4 pair_sums(const GPR_GLOBAL char *lists, unsigned off, unsigned step, int ng, const float4 pi,
                                            const float2 ppi, const float4 *xs, const float2 *pp, float rc2, float krf2,
                                            float krf, float crf)
{
    float fx = 0.f, fy = 0.f, fz = 0.f, e = 0.f;
    if (ng > 0) {
        const unsigned last = off + (unsigned)(ng - 1) * step;
        // LDS addresses by hand: pb + entry (one instruction with its half-word select) is the partner's
        // parameters, twice that + xd its position
        const unsigned pb = (unsigned)fresh_v((int)(unsigned)(size_t)(const GPR_LDS char *)pp);
        const unsigned xd = (unsigned)fresh_s((int)((unsigned)(size_t)(const GPR_LDS char *)xs - 2 * (unsigned)(size_t)(const GPR_LDS char *)pp));
        auto x_at = [&](unsigned a) { const gv_f4 v = *(const GPR_LDS gv_f4 *)(size_t)(2 * a + xd); return make_float4(v.x, v.y, v.z, v.w); };
        auto p_at = [&](unsigned a) { const gv_f2 v = *(const GPR_LDS gv_f2 *)(size_t)a; return make_float2(v.x, v.y); };
        gv_u2 nxt = *(const GPR_GLOBAL gv_u2 *)(lists + off);
        for (int g = 0; g < ng; ++g) {
            const gv_u2 cur = nxt;
            off = min(off + step, last);
            nxt = *(const GPR_GLOBAL gv_u2 *)(lists + off);
            const unsigned o0 = (cur.x & 0xFFFFu) + pb, o1 = (cur.x >> 16) + pb, o2 = (cur.y & 0xFFFFu) + pb, o3 = (cur.y >> 16) + pb;
            const float4 x0 = x_at(o0), x1 = x_at(o1), x2 = x_at(o2), x3 = x_at(o3);
            const float2 p0 = p_at(o0), p1 = p_at(o1), p2 = p_at(o2), p3 = p_at(o3);
            pair_term(pi, ppi, x0, p0, rc2, krf2, krf, crf, ENERGY, fx, fy, fz, e);
            pair_term(pi, ppi, x1, p1, rc2, krf2, krf, crf, ENERGY, fx, fy, fz, e);
            pair_term(pi, ppi, x2, p2, rc2, krf2, krf, crf, ENERGY, fx, fy, fz, e);
            pair_term(pi, ppi, x3, p3, rc2, krf2, krf, crf, ENERGY, fx, fy, fz, e);
            // (used here, the read ahead cannot be moved to the top of the next pass)
            asm volatile("" : "+v"(nxt.x), "+v"(nxt.y));
        }
    }
    return make_float4(fx, fy, fz, e);
}

template <bool ENERGY>
__device__ __forceinline__ float4 nb_lane_t(const NbConsts &S, int r, int i, int q, const float4 *xs, const float2 *pp)
{
    const size_t stride = (size_t)S.np * P;
    const int ng = gconst(S.nbc)[(size_t)r * stride + (size_t)i * P + q];
    const GPR_GLOBAL char *lists = (const GPR_GLOBAL char *)gconst(S.nbl) + (size_t)r * S.Kg * stride * 8;
    return pair_sums<ENERGY>(lists, (unsigned)(i * P + q) * 8, (unsigned)stride * 8, ng, xs[i], pp[i], xs, pp, S.rc2, 2.0f * S.krf, S.krf, S.crf);
}

__device__ __forceinline__ float4 nb_lane(const NbConsts &S, int r, int i, int q, const float4 *xs, const float2 *pp,
                                          bool energy)
{
    return energy ? nb_lane_t<true>(S, r, i, q, xs, pp) : nb_lane_t<false>(S, r, i, q, xs, pp);
}

// ------------------------------------------------------------------ one B A O A for one atom
// The integrator's constants, as values: a persistent launch holds them in registers (read
// through the descriptor they would be loaded again after every fence of a step).
struct IntConsts {
    float h, c1;
    uint32_t key0, key1;
    int toy;
};
__device__ __forceinline__ IntConsts int_consts(const Dev &S)
{
    IntConsts k;
    k.h = S.h; k.c1 = S.c1; k.key0 = S.key0; k.key1 = S.key1; k.toy = S.kind == KIND_TOY;
    return k;
}

// the step with its Gaussians g given (drawn for (atom, step, replica) beforehand or by the caller)
__device__ __forceinline__ void integrate_baoa_g(const IntConsts &K, float3 &x, float3 &v, float3 F, float im, float sd,
                                                 float3 g)
{
    const float h = K.h, c1 = K.c1;
    v.x = kick(v.x, F.x, h, im);
    v.y = kick(v.y, F.y, h, im);
    v.z = kick(v.z, F.z, h, im);
    x.x = x.x + h * v.x;
    x.y = x.y + h * v.y;
    x.z = x.z + h * v.z;
    v.x = c1 * v.x + sd * g.x;
    v.y = c1 * v.y + sd * g.y;
    if (!K.toy) v.z = c1 * v.z + sd * g.z;
    x.x = x.x + h * v.x;
    x.y = x.y + h * v.y;
    x.z = x.z + h * v.z;
}

__device__ __forceinline__ float3 step_noise(const IntConsts &K, int a, int r, long long s)
{
    // (the round keys are computed where they are used: kept across the step they take 20 registers)
    const uint32_t key0 = (uint32_t)fresh_s((int)K.key0), key1 = (uint32_t)fresh_s((int)K.key1);
    return gauss3(philox_ctr((uint32_t)a, s, (uint32_t)r, STREAM_NOISE, key0, key1));
}

__device__ __forceinline__ void integrate_baoa_k(const IntConsts &K, int a, int r, long long s, float3 &x, float3 &v,
                                                 float3 F, float im, float sd)
{
    integrate_baoa_g(K, x, v, F, im, sd, step_noise(K, a, r, s));
}

__device__ __forceinline__ void integrate_baoa(const Dev &S, int a, int r, long long s, float3 &x, float3 &v,
                                               float3 F, float im, float sd)
{
    integrate_baoa_k(int_consts(S), a, r, s, x, v, F, im, sd);
}

__device__ __forceinline__ bool finite3(float3 a) { return isfinite(a.x) && isfinite(a.y) && isfinite(a.z); }

// ------------------------------------------------------------------ states and observables (FP64)
// Workgroup-collective.  Sums over atoms are taken in 2^-32 fixed point so that they do
// not depend on the launch shape.  red: LDS int64 scratch [MAX_OBS * 8 + 8].
// velocity component load; coh: device-coherent load of values another workgroup wrote
__device__ __forceinline__ float ldv(const float *p, bool coh)
{
    return coh ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

template <class Pos>
__device__ void group_sum_wg(const Dev &S, const Pos &xs, const float *vg, int off, int cnt, int what,
                             long long *dst, int tid, int nthr, bool coh = false)
{
    // what: 0 -> sum m x (3 slots), 1 -> sum |v|^2 (1 slot)
    for (int base = 0; base < cnt; base += nthr) {
        const int k = base + tid;
        long long s0 = 0, s1 = 0, s2 = 0;
        if (k < cnt) {
            const int a = S.groups[off + k];
            if (what == 0) {
                const double m = (double)S.mass[a];
                const float3 x = xs(a);
                s0 = fix_d(m * (double)x.x);
                s1 = fix_d(m * (double)x.y);
                s2 = fix_d(m * (double)x.z);
            } else {
                const double vx = ldv(vg + a, coh), vy = ldv(vg + S.np + a, coh), vz = ldv(vg + 2 * S.np + a, coh);
                s0 = fix_d(vx * vx + vy * vy + vz * vz);
            }
        }
        s0 = wave_sum_ll(s0);
        if (what == 0) { s1 = wave_sum_ll(s1); s2 = wave_sum_ll(s2); }
        if ((tid & 63) == 0) {
            lds_add(&dst[0], s0);
            if (what == 0) { lds_add(&dst[1], s1); lds_add(&dst[2], s2); }
        }
    }
}

template <class Pos>
__device__ __forceinline__ double3 xs_d(const Pos &xs, int a)
{
    const float3 x = xs(a);
    return make_double3((double)x.x, (double)x.y, (double)x.z);
}

template <class Pos>
__device__ int state_wg(const Dev &S, const Pos &xs, long long *red, int *sbuf, int tid, int nthr)
{
    const StateDesc &st = *S.st;
    if (st.kind == ST_SIGN_X) return xs(st.atoms[0]).x >= 0.0f ? 1 : 0;
    if (st.kind == ST_BOXES) {
        if (tid == 0) {
            const double phi = dihedral_d(xs_d(xs, st.atoms[0]), xs_d(xs, st.atoms[1]), xs_d(xs, st.atoms[2]), xs_d(xs, st.atoms[3]));
            const double psi = dihedral_d(xs_d(xs, st.atoms[4]), xs_d(xs, st.atoms[5]), xs_d(xs, st.atoms[6]), xs_d(xs, st.atoms[7]));
            int id = -1;
            for (int b = 0; b < st.nbox; ++b)
                if (st.box[b][0] < phi && phi <= st.box[b][1] && st.box[b][2] < psi && psi <= st.box[b][3]) { id = b; break; }
            *sbuf = id;
        }
        __syncthreads();
        const int id = *sbuf;
        __syncthreads();
        return id;
    }
    // centre of mass within a sphere
    if (tid < 3) red[tid] = 0;
    __syncthreads();
    group_sum_wg(S, xs, nullptr, st.g_off, st.g_n, 0, red, tid, nthr);
    __syncthreads();
    if (tid == 0) {
        const double cx = unfix_d(red[0]) / st.gm, cy = unfix_d(red[1]) / st.gm, cz = unfix_d(red[2]) / st.gm;
        const double dx = cx - st.center[0], dy = cy - st.center[1], dz = cz - st.center[2];
        *sbuf = sqrt(dx * dx + dy * dy + dz * dz) < st.radius ? 1 : 0;
    }
    __syncthreads();
    const int id = *sbuf;
    __syncthreads();
    return id;
}

// observable values into out[MAX_OBS] (LDS), valid after return
template <class Pos>
__device__ __noinline__ void observables_wg(const Dev &S, const Pos xs, const float *vg, double U, long long *red,
                               double *out, int tid, int nthr, bool coh = false)
{
    if (tid < MAX_OBS * 8) red[tid] = 0;
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < S.nobs; ++j) {
        const ObsDesc &o = S.obs[j];
        long long *dst = red + 8 * j;
        if (o.kind == OB_KIN) {
            for (int base = 0; base < S.n; base += nthr) {
                const int a = base + tid;
                long long s = 0;
                if (a < S.n) {
                    const double vx = ldv(vg + a, coh), vy = ldv(vg + S.np + a, coh), vz = ldv(vg + 2 * S.np + a, coh);
                    s = fix_d(0.5 * (double)S.mass[a] * (vx * vx + vy * vy + vz * vz));
                }
                s = wave_sum_ll(s);
                if ((tid & 63) == 0) lds_add(dst, s);
            }
        } else if (o.kind == OB_COMD) {
            group_sum_wg(S, xs, vg, o.ga_off, o.ga_n, 0, dst, tid, nthr);
            group_sum_wg(S, xs, vg, o.gb_off, o.gb_n, 0, dst + 3, tid, nthr);
        } else if (o.kind == OB_RMSV) {
            group_sum_wg(S, xs, vg, o.ga_off, o.ga_n, 1, dst, tid, nthr, coh);
        }
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll 1
        for (int j = 0; j < S.nobs; ++j) {
            const ObsDesc &o = S.obs[j];
            const long long *src = red + 8 * j;
            double val = 0.0;
            switch (o.kind) {
            case OB_COORD: {
                const float3 p = xs(o.atoms[0]);
                val = o.atoms[1] == 0 ? (double)p.x : (o.atoms[1] == 1 ? (double)p.y : (double)p.z);
                break;
            }
            case OB_POT: val = U; break;
            case OB_KIN: val = unfix_d(src[0]); break;
            case OB_DIH:
                val = dihedral_d(xs_d(xs, o.atoms[0]), xs_d(xs, o.atoms[1]), xs_d(xs, o.atoms[2]), xs_d(xs, o.atoms[3]));
                break;
            case OB_COMD: {
                const double ax = unfix_d(src[0]) / o.ma, ay = unfix_d(src[1]) / o.ma, az = unfix_d(src[2]) / o.ma;
                const double bx = unfix_d(src[3]) / o.mb, by = unfix_d(src[4]) / o.mb, bz = unfix_d(src[5]) / o.mb;
                val = sqrt((ax - bx) * (ax - bx) + (ay - by) * (ay - by) + (az - bz) * (az - bz));
                break;
            }
            case OB_RMSV: val = sqrt(unfix_d(src[0]) / (double)o.ga_n); break;
            default: break;
            }
            out[j] = val;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void accumulate_obs(const Dev &S, int r, const double *out)
{
    double *acc = S.acc + (size_t)r * MAX_OBS * 2;
    for (int j = 0; j < S.nobs; ++j) {
        const double xj = out[j] - S.shift[j];
        acc[2 * j] += xj;
        const double x2 = xj * xj;
        acc[2 * j + 1] += x2;
    }
}

// stage positions (x, y, z, q sqrt f) and (sigma/2, 2 sqrt eps) of replica r into LDS
__device__ __forceinline__ void stage_replica(const Dev &S, int r, float4 *xs, float2 *pp, int tid, int nthr)
{
    const GPR_GLOBAL float *xg = gconst(S.x) + (size_t)r * 3 * S.np;
    for (int a = tid; a < S.np; a += nthr) {
        const float4 pr = gld(gconst(S.prm) + a);
        if (a < S.n) xs[a] = make_float4(xg[a], xg[S.np + a], xg[2 * S.np + a], pr.z);
        else xs[a] = make_float4(FAR, FAR, FAR, 0.f);
        if (pp) pp[a] = make_float2(pr.x, pr.y);
    }
}

// ================================================================== plain path kernels
// Step and energy flag of a plain-path kernel: as given, or (codes DCLK_*) step k of a cycle
// that starts at the device clock (s, t) = (clock[0], clock[1]), with k passed in s; such a
// step samples when (t + k + 1) is a multiple of t_GR.
__device__ __forceinline__ void step_args(const Dev &S, long long &s, int &energy)
{
    if (energy < DCLK_SAMPLE) return;
    const long long k = s;
    const bool samp = energy == DCLK_SAMPLE && (S.clock[1] + k + 1) % S.t_gr == 0;
    s = S.clock[0] + k;
    energy = (samp && S.need_energy) ? 1 : 0;
}

__global__ void k_set_clock(const Dev *__restrict__ Sp, long long s, long long t)
{
    Sp->clock[0] = s;
    Sp->clock[1] = t;
}

__global__ void k_tick(const Dev *__restrict__ Sp, long long n)
{
    Sp->clock[0] += n;
    Sp->clock[1] += n;
}
// B A O A for every atom of replicas r_off + blockIdx.y; displacement guard; energy reset.
__global__ void __launch_bounds__(256) k_integrate(const Dev *__restrict__ Sp, long long s, int r_off, int energy)
{
    const Dev &S = *Sp;
    step_args(S, s, energy);
    const int r = r_off + blockIdx.y;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    int *guard = S.guard + (s & 1) * S.R + r;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (energy) S.E[r] = 0;
        if (S.need_build[r]) { atomicOr(guard, 1); S.need_build[r] = 0; }
    }
    if (a >= S.n) return;
    const size_t b = (size_t)r * 3 * S.np;
    const int np = S.np;
    GPR_GLOBAL float *X = gmut(S.x) + b, *V = gmut(S.v) + b;
    const GPR_GLOBAL float *XB = gconst(S.xb) + b;
    const GPR_GLOBAL long long *Fp = gconst(S.F) + b;
    float3 x = make_float3(X[a], X[np + a], X[2 * np + a]);
    float3 v = make_float3(V[a], V[np + a], V[2 * np + a]);
    const float3 F = make_float3(unfix_f(Fp[a]), unfix_f(Fp[np + a]), unfix_f(Fp[2 * np + a]));
    const float im = gld(gconst(S.prm) + a).w;
    integrate_baoa(S, a, r, s, x, v, F, im, gconst(S.sd)[a]);
    X[a] = x.x; X[np + a] = x.y; X[2 * np + a] = x.z;
    V[a] = v.x; V[np + a] = v.y; V[2 * np + a] = v.z;
    if (!finite3(x) || !finite3(v)) atomicOr(&S.err[ERR_UNSTABLE], 1);
    if (S.cutoff_on) {
        const float dx = x.x - XB[a], dy = x.y - XB[np + a], dz = x.z - XB[2 * np + a];
        if (!(dx * dx + dy * dy + dz * dz <= (im > S.im_light ? S.guard2_light : S.guard2_heavy))) atomicOr(guard, 1);
    }
}

// Forces of atoms [blockIdx.x * blockDim.x / P, ...) of replica r (256 atoms, P lanes each), then the
// closing B kick (apply_b).  The block stages the replica, rebuilds its atoms' pair lists first when
// due (period, displacement guard, force_build), and sums the bonded units of its atom range and
// their pairs in LDS fixed point, over the boxes and scratch of the rebuild.  Bound by the search
// when lists are rebuilt, else by the staging and the pairs.  Bonded terms in a kernel of their own
// waited for scattered positions from memory: 7.0 + 21.4 -> 22.5 us a step (19.1 with joint rebuilds; 5,200 atoms x 12
// replicas), 13.9 + 66.0 -> 70.6 us for 64 replicas of 2,432 atoms with a rebuild.  At most 64
// registers, so that two workgroups share a compute unit where their LDS fits, one staging or
// waiting while the other computes (89 us with one).
__global__ void __launch_bounds__(1024, 8) k_forces(const Dev *__restrict__ Sp, long long s, int r_off, int energy, int apply_b,
                                                   int force_build)
{
    step_args(*Sp, s, energy);
    const Dev &S = *Sp;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    float2 *pp = (float2 *)lds_raw;
    float4 *xs = (float4 *)(pp + S.np);
    float4 *box = xs + S.np;                               // boxes of the atom blocks
    int *wscr = (int *)(box + (S.n + BLK - 1) / BLK);      // [16][WBLK] build scratch per wave
    __shared__ long long e_acc;
    __shared__ int far_out;                                // (a word of its own: __syncthreads_or takes 256 bytes)
    const int r = r_off + blockIdx.y;
    const int tid = threadIdx.x, nthr = blockDim.x;
    stage_replica(S, r, xs, pp, tid, nthr);
    if (tid == 0) { e_acc = 0; far_out = 0; }
    for (int t = tid; t < (S.n + BLK - 1) / BLK; t += nthr) box[t].w = __uint_as_float((unsigned)gconst(S.cls)[t] << 24);
    // rebuild when forced, when flagged (displacement guard or a new configuration), or on the
    // steps s with s + 1 a multiple of period, the same steps for every replica: one launch
    // serves all replicas, so rebuilds that coincide cost one long launch instead of many.
    // The step of the last build is recorded by step parity (block 0 writes the next step's
    // slot while the other blocks read this step's) for the persistent path.
    bool rebuild = force_build != 0;
    if (!force_build) {
        long long lb = 0;
        if (S.cutoff_on) {
            lb = S.last_build[(s & 1) * S.R + r];
            const int *flags = S.guard + (s & 1) * S.R;
            rebuild = (s + 1) % S.period == 0 || flags[r] != 0;
            // A launch that fits the device at once lasts as long as its slowest block, so one replica
            // that rebuilds costs as much as all: then they all do, and their next guards fall due
            // together (12 replicas of 5,200 atoms: long launches on 20 % of the steps, not 36 %)
            if ((int)(gridDim.x * gridDim.y) <= S.cus)
                for (int q = tid & 63; q < (int)gridDim.y; q += 64) rebuild |= flags[r_off + q] != 0;
            rebuild = __any(rebuild);
        }
        if (blockIdx.x == 0 && tid == 0) {
            S.guard[((s + 1) & 1) * S.R + r] = 0;
            S.last_build[((s + 1) & 1) * S.R + r] = rebuild ? s : lb;
            if (rebuild) S.list_pad[r] = 0;
        }
    } else if (blockIdx.x == 0 && tid == 0) {
        S.last_build[r] = s;
        S.last_build[S.R + r] = s;
        S.list_pad[r] = 0;
    }
    __syncthreads();
    const int i = blockIdx.x * (nthr / P) + tid / P;
    const int q = tid % P;
    const size_t b = (size_t)r * 3 * S.np;
    if (rebuild) {
        const GPR_CONST Dev &C = *(const GPR_CONST Dev *)Sp;
        const GPR_LDS gv_f4 *xl = (const GPR_LDS gv_f4 *)xs;
        GPR_LDS gv_f2 *pl = (GPR_LDS gv_f2 *)pp;
        const float3 c = search_centre(xl, S.n);
        if (block_boxes(C, xl, pl, (GPR_LDS gv_f4 *)box, c, tid, nthr)) far_out = 1;
        __syncthreads();
        const bool wide = uni(far_out) != 0;
        const int wv = uni(tid >> 6);
        search_task<2, false>(C, r, blockIdx.x * (nthr / P) + 16 * wv, S.n, xl, pl, (const GPR_LDS gv_f4 *)box,
                              (GPR_LDS int *)wscr + wv * WBLK, c, wide, !S.cutoff_on);
        __syncthreads();
        for (int a = tid; a < BLK * ((S.n + BLK - 1) / BLK); a += nthr) pp[a].x = gld(gconst(S.prm) + a).x;
        if (i < S.n && q == 0) {
            S.xb[b + i] = xs[i].x; S.xb[b + S.np + i] = xs[i].y; S.xb[b + 2 * S.np + i] = xs[i].z;
        }
        __syncthreads();
    }
    long long eatom = 0;
    const int a0 = blockIdx.x * (nthr / P), l = tid / P, na = nthr / P;
    long long *const fa = (long long *)box;                // [na][3]
    for (int k = tid; k < 3 * na; k += nthr) fa[k] = 0;
    __syncthreads();
    if (S.kind == KIND_TOY) {
        if (tid == 0 && a0 == 0) {
            float fx, fy;
            const float u = toy_force(xs[0].x, xs[0].y, fx, fy);
            fa[0] = fix_f(fx);
            fa[1] = fix_f(fy);
            eatom = fix_f(u);
        }
    } else {
        // every wave its share of the bonded units, then its pairs
        const int wv = uni(tid >> 6), nwv = nthr >> 6, u0 = gconst(S.pl_first)[blockIdx.x], u1 = gconst(S.pl_first)[blockIdx.x + 1];
        const ForceLDS F{fa, a0, 3, 1};
        if (energy) eatom = bonded_units<true>(S.pl_bi, S.pl_bp, u0, u1, PosLDS{xs}, F, wv, nwv, tid & 63);
        else bonded_units<false>(S.pl_bi, S.pl_bp, u0, u1, PosLDS{xs}, F, wv, nwv, tid & 63);
        if (i < S.n) {
            float4 f = nb_lane(nb_consts(S), r, i, q, xs, pp, energy != 0);
            f.x = quad_sum(f.x);
            f.y = quad_sum(f.y);
            f.z = quad_sum(f.z);
            if (energy) f.w = quad_sum(f.w);
            if (q < 3) lds_add(&fa[3 * l + q], fix_f(q == 0 ? f.x : (q == 1 ? f.y : f.z)));
            else if (energy) eatom += fix_f(f.w);
        }
    }
    __syncthreads();
    for (int k = tid; k < 3 * na; k += nthr) {
        const int d = k / na, c = k - d * na, a = a0 + c;
        if (a >= S.n) continue;
        const long long Fi = fa[3 * c + d];
        const float f = unfix_f(Fi);
        gmut(S.F)[b + d * S.np + a] = Fi;
        if (bad_force(f)) atomicOr(&S.err[ERR_UNSTABLE], 1);
        if (apply_b) gmut(S.v)[b + d * S.np + a] = kick(gmut(S.v)[b + d * S.np + a], f, S.h, gld(gconst(S.prm) + a).w);
    }
    if (energy) {
        eatom = wave_sum_ll(eatom);
        if ((tid & 63) == 0 && eatom != 0) lds_add(&e_acc, eatom);
        __syncthreads();
        if (tid == 0 && e_acc != 0) atomicAdd((unsigned long long *)&S.E[r], (unsigned long long)e_acc);
    }
}

// observables of replicas r_off + blockIdx.x: accumulate (mode 0, workers), set the shift
// c_j from replica 0 (mode 1), or write the values to out[r][MAX_OBS] (mode 2)
__global__ void __launch_bounds__(1024) k_obs(const Dev *__restrict__ Sp, int r_off, int mode, double *out, int k)
{
    const Dev &S = *Sp;
    if (mode == 3 && (S.clock[1] + k + 1) % S.t_gr != 0) return;    // step k of a device-clock cycle: no sample
    extern __shared__ __align__(16) unsigned char lds_raw[];
    float4 *xs = (float4 *)lds_raw;
    __shared__ long long red[MAX_OBS * 8 + 8];
    __shared__ double vals[MAX_OBS];
    const int r = r_off + blockIdx.x;
    stage_replica(S, r, xs, nullptr, threadIdx.x, blockDim.x);
    __syncthreads();
    const float *vg = S.v + (size_t)r * 3 * S.np;
    observables_wg(S, PosLDS{xs}, vg, unfix_d(S.E[r]), red, vals, threadIdx.x, blockDim.x);
    if (threadIdx.x == 0) {
        if (mode == 0 || mode == 3) accumulate_obs(S, r, vals);
        else if (mode == 1) for (int j = 0; j < S.nobs; ++j) S.shift[j] = vals[j];
        else for (int j = 0; j < S.nobs; ++j) out[(size_t)r * MAX_OBS + j] = vals[j];
    }
}

// state ids of replicas r_off + blockIdx.x
__global__ void __launch_bounds__(256) k_state(const Dev *__restrict__ Sp, int r_off)
{
    const Dev &S = *Sp;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    float4 *xs = (float4 *)lds_raw;
    __shared__ long long red[8];
    __shared__ int sbuf;
    const int r = r_off + blockIdx.x;
    stage_replica(S, r, xs, nullptr, threadIdx.x, blockDim.x);
    __syncthreads();
    const int id = state_wg(S, PosLDS{xs}, red, &sbuf, threadIdx.x, blockDim.x);
    if (threadIdx.x == 0) S.state[r] = id;
}

// parameters of the n records of the bonded units, from those of the terms (src: 5 (sorted term) + kind, or -1)
__global__ void __launch_bounds__(256) k_unit_params(Topo T, const int *src, int n, float4 *bp)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const int t = src[c] / 5, kind = src[c] < 0 ? -1 : src[c] % 5;
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
    if (kind == 0 || kind == 1) {
        const float2 q = kind == 0 ? T.b_p[t] : T.a_p[t];
        p = make_float4(q.x, q.y, 0.f, 0.f);
    } else if (kind >= 0) {
        p = kind == 2 ? T.t_p[t] : kind == 3 ? T.r_p[t] : T.p_p[t];
    }
    bp[c] = p;
}

// ================================================================== force-field parameter gradient
// dU_r/dtheta for theta = (eps_i, sigma_i, q_i, torsion k_t), weighted by w[r] and summed over
// the replicas in 2^-32 fixed point (gacc).  With eps_ij = sqrt(eps_i eps_j), sigma_ij =
// (sigma_i + sigma_j)/2, s = sigma_ij / r and Coulomb kernel g(r):
//   dU/deps_i   = 1/(2 eps_i) sum_j 4 eps_ij (s^12 - s^6)
//   dU/dsigma_i = sum_j 1/2 4 eps_ij (12 s^12 - 6 s^6) / sigma_ij
//   dU/dq_i     = sqrt(f) sum_j (q_j sqrt(f)) g(r)
//   dU/dk_t     = 1 + cos(n phi - phi0)
// the constant factors 1/(2 eps_i) and sqrt(f) applied in k_grad_finish.  Pair sums run over
// the full pair lists (every partner of i in i's own sub-lists), so each atom's sums are
// complete without scattering to j; 1-4 pairs (scaled) and torsions come one term per thread.

// nonbonded pairs of replicas r_off + blockIdx.y at their current positions and pair lists
__global__ void __launch_bounds__(1024) k_grad_nb(const Dev *__restrict__ Sp, const double *w)
{
    const Dev &S = *Sp;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    float2 *pp = (float2 *)lds_raw;
    float4 *xs = (float4 *)(pp + S.np);
    const int r = blockIdx.y;
    const int tid = threadIdx.x, nthr = blockDim.x;
    stage_replica(S, r, xs, pp, tid, nthr);
    __syncthreads();
    const int i = blockIdx.x * (nthr / P) + tid / P;
    const int q = tid % P;
    float se = 0.f, ss = 0.f, sq = 0.f;
    if (i < S.n) {
        const size_t stride = (size_t)S.np * P;
        const GPR_GLOBAL uint2 *L = gconst(S.nbl) + (size_t)r * S.Kg * stride + (size_t)i * P + q;
        const int ng = gconst(S.nbc)[(size_t)r * stride + (size_t)i * P + q];
        const float4 pi = xs[i];
        const float2 ppi = pp[i];
        const float rc2 = S.rc2, krf = S.krf, crf = S.crf;
        for (int g = 0; g < ng; ++g) {
            const uint2 wv = gld(L + (size_t)g * stride);
            const int jj[4] = {(int)(wv.x & 0xFFFF) >> 3, (int)(wv.x >> 19), (int)(wv.y & 0xFFFF) >> 3, (int)(wv.y >> 19)};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 pj = xs[jj[k]];
                const float2 ppj = pp[jj[k]];
                const float dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
                const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                const float ri = __builtin_amdgcn_rsqf(r2);
                const float sg = ppi.x + ppj.x;
                const float t = sg * ri;
                const float s2 = t * t;
                const float s6 = s2 * s2 * s2, s12 = s6 * s6;
                const float e4 = ppi.y * ppj.y;
                const bool in = r2 < rc2;
                se += in ? e4 * (s12 - s6) : 0.0f;
                ss += in ? 0.5f * e4 * (12.0f * s12 - 6.0f * s6) * __builtin_amdgcn_rcpf(sg) : 0.0f;
                sq += in ? pj.w * (ri + krf * r2 - crf) : 0.0f;
            }
        }
    }
    se = quad_sum(se);
    ss = quad_sum(ss);
    sq = quad_sum(sq);
    if (i < S.n && q == 0) {
        const double wr = w[r];
        unsigned long long *G = (unsigned long long *)S.gacc;
        atomicAdd(G + i, (unsigned long long)fix_d(wr * se));
        atomicAdd(G + S.np + i, (unsigned long long)fix_d(wr * ss));
        atomicAdd(G + 2 * S.np + i, (unsigned long long)fix_d(wr * sq));
    }
}

// 1-4 pairs (no cutoff, vacuum Coulomb, scaled) and torsions of replica blockIdx.y
__global__ void __launch_bounds__(256) k_grad_terms(const Dev *__restrict__ Sp, const double *w)
{
    const Dev &S = *Sp;
    const Topo &T = S.tp;
    const int r = blockIdx.y;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const double wr = w[r];
    const PosGlob pos{gconst(S.x) + (size_t)r * 3 * S.np, S.np};
    unsigned long long *G = (unsigned long long *)S.gacc;
    if (t < T.n14) {
        const int2 ij = gld(gconst(T.p_ij) + t);
        const float4 a = gld(gconst(S.prm) + ij.x), b = gld(gconst(S.prm) + ij.y);
        const float3 xa = pos(ij.x), xb = pos(ij.y);
        const float dx = xa.x - xb.x, dy = xa.y - xb.y, dz = xa.z - xb.z;
        const float ri = __builtin_amdgcn_rsqf(dx * dx + dy * dy + dz * dz);
        const float sg = a.x + b.x, tt = sg * ri, s2 = tt * tt, s6 = s2 * s2 * s2, s12 = s6 * s6;
        const float e4 = a.y * b.y, sc = S.scale14;
        const double ulj = (double)(sc * e4 * (s12 - s6));
        const double dsg = (double)(sc * 0.5f * e4 * (12.0f * s12 - 6.0f * s6) * __builtin_amdgcn_rcpf(sg));
        atomicAdd(G + ij.x, (unsigned long long)fix_d(wr * ulj));
        atomicAdd(G + ij.y, (unsigned long long)fix_d(wr * ulj));
        atomicAdd(G + S.np + ij.x, (unsigned long long)fix_d(wr * dsg));
        atomicAdd(G + S.np + ij.y, (unsigned long long)fix_d(wr * dsg));
        atomicAdd(G + 2 * S.np + ij.x, (unsigned long long)fix_d(wr * (double)(sc * b.z * ri)));
        atomicAdd(G + 2 * S.np + ij.y, (unsigned long long)fix_d(wr * (double)(sc * a.z * ri)));
    }
    if (t < T.nt) {
        const int4 q = gld(gconst(T.t_ijkl) + t);
        const float ca = torsion_cos(pos(q.x), pos(q.y), pos(q.z), pos(q.w), gld(gconst(T.t_p) + t));
        atomicAdd(G + 3 * S.np + t, (unsigned long long)fix_d(wr * (double)(1.0f + ca)));
    }
}

__global__ void __launch_bounds__(256) k_grad_finish(const Dev *__restrict__ Sp, double *d_eps, double *d_sigma,
                                                     double *d_charge, double *d_tk)
{
    const Dev &S = *Sp;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const double sqrt_f = S.sqrt_f;
    if (a < S.n) {
        if (d_eps) d_eps[a] = unfix_d(S.gacc[a]) * S.inv2eps[a];
        if (d_sigma) d_sigma[a] = unfix_d(S.gacc[S.np + a]);
        if (d_charge) d_charge[a] = unfix_d(S.gacc[2 * S.np + a]) * sqrt_f;
        S.gacc[a] = S.gacc[S.np + a] = S.gacc[2 * S.np + a] = 0;      // for the next call
    }
    if (a < S.tp.nt) {
        if (d_tk) d_tk[S.tor_orig[a]] = unfix_d(S.gacc[3 * S.np + a]);
        S.gacc[3 * S.np + a] = 0;
    }
}

// dx[r] = w[r] dU_r/dx = -w[r] F_r, from the fixed-point forces
__global__ void __launch_bounds__(256) k_weighted_dx(const Dev *__restrict__ Sp, const double *w, float *dx)
{
    const Dev &S = *Sp;
    const int r = blockIdx.y;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a < S.n) {
        const double wr = w[r];
        for (int d = 0; d < 3; ++d)
            dx[((size_t)r * 3 + d) * S.n + a] = (float)(-wr * unfix_d(S.F[((size_t)r * 3 + d) * S.np + a]));
    }
}

// Positions [R][3][n] into the replicas' padded arrays, their energies cleared for the force kernels
__global__ void __launch_bounds__(256) k_load_x(const Dev *__restrict__ Sp, const float *x)
{
    const Dev &S = *Sp;
    const int r = blockIdx.y;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a == 0) S.E[r] = 0;
    if (a < S.n)
        for (int d = 0; d < 3; ++d) S.x[((size_t)r * 3 + d) * S.np + a] = x[((size_t)r * 3 + d) * S.n + a];
}

// Pieces of device memory into page-locked host memory: a read-back is one launch and one wait, where
// a copy per piece costs some 15 us each (a 300-atom replica's state 37 -> 18 us, call and all).
__global__ void __launch_bounds__(256) k_read(ReadList l, uint32_t *out)
{
    const unsigned t = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    for (int p = 0; p < 3; ++p) {
        for (unsigned w = t; w < l.words[p]; w += step) out[w] = l.src[p][w];
        out += l.words[p];
    }
}

// energies and forces of every replica out of the fixed-point accumulators, and the error flags
__global__ void __launch_bounds__(256) k_unfix_out(const Dev *__restrict__ Sp, double *energy, float *forces, int *err)
{
    const Dev &S = *Sp;
    const int r = blockIdx.y;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a < 4 && r == 0) err[a] = S.err[a];
    if (a == 0 && energy) energy[r] = unfix_d(S.E[r]);
    if (a < S.n && forces) {
        for (int d = 0; d < 3; ++d)
            forces[((size_t)r * 3 + d) * S.n + a] = (float)unfix_d(S.F[((size_t)r * 3 + d) * S.np + a]);
    }
}

// ================================================================== persistent path
// Phase timers, in a build with GPR_PHASE_PROBE defined (a measurement library built beside
// the product one; the product build has none of this).  Thread 0 of every workgroup reads
// the constant-rate clock at the ends of the phases of each step and adds the differences,
// per (replica, group), to gpr_phase_acc[(r * PHASE_MAX_G + g) * NPHASE + k]; the phases end
// at workgroup barriers the body has anyway, so thread 0's clock marks the group's progress.
// The timers add a few instructions per phase and change no result.
#ifdef GPR_PHASE_PROBE
__device__ unsigned long long gpr_phase_acc[PHASE_MAX_R * PHASE_MAX_G * NPHASE];
// (the last reading is kept in LDS too, so that no register is held across the phases)
#define PHASE_MARK(k)                                                       \
    do {                                                                    \
        if (tid == 0) {                                                     \
            const unsigned long long t_ = __builtin_amdgcn_s_memrealtime(); \
            ph_acc[(k)] += t_ - ph_acc[NPHASE];                             \
            ph_acc[NPHASE] = t_;                                            \
        }                                                                   \
    } while (0)
#define PHASE_COUNT(k) do { if (tid == 0) ph_acc[(k)] += 1; } while (0)
#else
#define PHASE_MARK(k) ((void)0)
#define PHASE_COUNT(k) ((void)0)
#endif

hipError_t phase_take(unsigned long long *out, int R, hipStream_t st)
{
#ifdef GPR_PHASE_PROBE
    if (R < 1 || R > PHASE_MAX_R) return hipErrorInvalidValue;
    const size_t bytes = sizeof(unsigned long long) * (size_t)R * PHASE_MAX_G * NPHASE;
    void *acc = nullptr;
    hipError_t e = hipGetSymbolAddress(&acc, HIP_SYMBOL(gpr_phase_acc));
    if (e == hipSuccess) e = hipMemcpyAsync(out, acc, bytes, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipMemsetAsync(acc, 0, bytes, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    return e;
#else
    (void)out; (void)R; (void)st;
    return hipErrorNotSupported;
#endif
}

// Barrier among the G workgroups of one replica: every thread waits for its own global
// stores to complete, then one thread adds to the replica's counter (device-scope relaxed
// atomic) and waits, with a bounded spin, for all G arrivals of this generation.  Data
// exchanged between the groups is written and read with device-scope relaxed atomics, so
// no cache writeback or invalidation is needed.  Returns false after a timeout.
__device__ __forceinline__ bool group_barrier(int *ctr, int target, int *err, int *sbuf)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int spins = 0, ok = 1;
        while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins > SPIN_MAX) {
                atomicOr(err + ERR_BARRIER, 1);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        *sbuf = ok;
    }
    __syncthreads();
    const bool ok = *sbuf != 0;
    __syncthreads();
    return ok;
}

__device__ __forceinline__ void st_coh(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// words of the position exchange: a coordinate under half a coordinate and a tag
__device__ __forceinline__ unsigned long long tagged(float x, unsigned upper) { return ((unsigned long long)upper << 32) | __float_as_uint(x); }
__device__ __forceinline__ unsigned step_tag(int step) { return 1u + (unsigned)step % 32767u; }
__device__ __forceinline__ void st_coh(GPR_GLOBAL unsigned long long *p, unsigned long long v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned long long ld_coh(const GPR_GLOBAL unsigned long long *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// G workgroups per replica advance nsteps BAOAB steps.  Group g of replica r owns the atoms
// [a0, a1) = [sp.bnd[g], sp.bnd[g + 1]) (ranges chosen on the host to even out the work); its LDS
// (persist_off) holds the positions (float4 with the scaled charge) and LJ parameters of every atom
// of the replica, and the velocities and fixed-point force accumulators of its own atoms (the
// accumulators carry the forces from one step to the next), block boxes and reduction scratch.  Per
// step: B A O A of own atoms -> (G > 1) positions exchanged through device-coherent words that say
// themselves which step they are of (a counter the groups wait on first is a trip to memory more: us
// per step with one / with tagged words, 300 atoms x 24 replicas 7.6 / 6.9, 2 replicas of 2,432 atoms
// on 8 groups 13.2 / 12.8, 64 on 4 groups 19.9 / 19.7) -> pair-list rebuild of own atoms when due -> bonded units touching own atoms (LDS atomics) and
// pair forces of own atoms (P lanes per atom) -> closing B; every t_GR steps (t counted from t0) the
// observables of workers are accumulated by group 0.  With state_end group 0 writes the state id.
// Workgroups map to replicas so that a replica's groups are meant to share an XCD (equal
// blockIdx mod 8) when the replica count allows; results do not depend on G, the block size or
// the placement.

// Pair-loop order of a group's nl atoms.  A task of the pair loop is 16 atoms on the 64 lanes
// of a wave and runs as long as its longest list, so the atoms go longest list first (key: the
// atom's longest sub-list, in words): tasks of similar lists, taken heaviest first.  perm has
// 16 * ceil(nl / 16) slots; those past nl hold 0xFFFF.  Forces do not depend on the order: an
// atom's four lanes stay together and sum its own sub-lists in their fixed order.
__device__ __forceinline__ void order_atoms(const GPR_LDS unsigned short *key, GPR_LDS unsigned short *perm, GPR_LDS int *hist,
                                            int nl, int tid, int nthr)
{
    const int nt = (nl + 15) >> 4;
    for (int k = tid; k < 16 * nt; k += nthr) perm[k] = 0xFFFF;
    for (int k = tid; k < 64; k += nthr) hist[k] = 0;
    __syncthreads();
    for (int l = tid; l < nl; l += nthr) lds_inc(&hist[63 - min((int)key[l], 63)]);
    __syncthreads();
    if (tid < 64) {                                        // exclusive prefix sum of the bins
        const int c = hist[tid];
        int x = c;
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (tid >= d) x += y;
        }
        hist[tid] = x - c;
    }
    __syncthreads();
    for (int l = tid; l < nl; l += nthr) perm[lds_inc(&hist[63 - min((int)key[l], 63)])] = (unsigned short)l;
    __syncthreads();
}

// The order of the search's tasks of 16 consecutive atoms, the costliest first by the lists of the
// last build (the summed longest sub-lists of a task's atoms)
__device__ __forceinline__ void order_tasks(const GPR_LDS unsigned short *key, GPR_LDS int *cost, GPR_LDS unsigned short *order,
                                            int nl, int tid, int nthr)
{
    const int ntk = (nl + 15) >> 4;
    for (int c = tid; c < ntk; c += nthr) {
        int sum = 0;
        for (int l = 16 * c; l < min(16 * c + 16, nl); ++l) sum += key[l];
        cost[c] = sum;
    }
    __syncthreads();
    for (int c = tid; c < ntk; c += nthr) {
        const int mine = cost[c];
        int rank = 0;
        for (int d = 0; d < ntk; ++d) rank += (cost[d] > mine) | (cost[d] == mine && d < c);
        order[rank] = (unsigned short)c;
    }
    __syncthreads();
}

// Rebuilds the pair lists of a group's atoms: the boxes of all blocks, then the search in tasks of
// 16 atoms, one wave each, taken by the waves from a counter as they come free.  The orders of the
// search's tasks and of the pair loop's atoms are kept from one rebuild to the next and renewed on
// every ORDER_PERIOD-th: list lengths change little in between, and renewing both costs 9 us (24 us
// for the rest of a rebuild on the 2,432-atom system with four groups).  They change no list and no
// force.  A function of its own: inlined, its registers cost the step loop spills on every step.
constexpr int ORDER_PERIOD = 8;
__device__ __noinline__ void persist_rebuild(const Dev *Sv, GPR_LDS unsigned char *raw, GPR_LDS int *counter, GPR_LDS int *torder,
                                             int lmax_, int a0_, int a1_, int r_, int renew_)
{
    const GPR_CONST Dev &S = *(const GPR_CONST Dev *)uni64((long long)Sv);
    const int lmax = uni(lmax_), a0 = uni(a0_), a1 = uni(a1_), r = uni(r_);
    const bool renew = uni(renew_) != 0;
    const int tid = threadIdx.x, BT = blockDim.x, n = S.n, np = S.np, nl = a1 - a0, ntk = (nl + 15) >> 4;
    const PersistOff o = persist_off(n, np, lmax);
    const GPR_LDS gv_f4 *const xs = (const GPR_LDS gv_f4 *)(raw + o.xs);
    GPR_LDS gv_f2 *const pp = (GPR_LDS gv_f2 *)raw;
    GPR_LDS gv_f4 *const box = (GPR_LDS gv_f4 *)(raw + o.box);
    GPR_LDS int *const wscr = (GPR_LDS int *)(raw + o.wscr);
    GPR_LDS unsigned short *const perm = (GPR_LDS unsigned short *)(raw + o.perm), *const keyl = (GPR_LDS unsigned short *)(raw + o.keyl);
    GPR_LDS unsigned short *const order = (GPR_LDS unsigned short *)torder;
    GPR_LDS float *const xbl = (GPR_LDS float *)(raw + o.xbl);
    if (tid == 0) *counter = 0;
    if (renew) order_tasks(keyl, wscr, order, nl, tid, BT);
    const float3 c = search_centre(xs, n);
    const bool wide = __syncthreads_or(block_boxes(S, xs, pp, box, c, tid, BT)) != 0;
    for (;;) {
        int t = 0;
        if ((tid & 63) == 0) t = lds_inc(counter);
        t = uni(t);
        if (t >= ntk) break;
        const int k = uni((int)order[t]);
        const int kq = search_task<4, true>(S, r, a0 + 16 * k, a1, xs, pp, box, wscr + (tid >> 6) * WBLK, c, wide, false);
        const int l = 16 * k + (tid & 63);
        if ((tid & 63) < 16 && l < nl) {
            const gv_f4 x = xs[a0 + l];
            xbl[l] = x.x; xbl[lmax + l] = x.y; xbl[2 * lmax + l] = x.z;
            keyl[l] = (unsigned short)kq;
        }
    }
    __syncthreads();
    for (int a = tid; a < BLK * ((n + BLK - 1) / BLK); a += BT) pp[a].x = gld(gconst(S.prm) + a).x;
    if (renew) order_atoms(keyl, perm, (GPR_LDS int *)(raw + o.red), nl, tid, BT);
    __syncthreads();
}

// Observables of a worker at the end of a sampled step, its closing B done: the groups' velocities
// and energy to group 0 of the replica, which accumulates them.  False after a barrier timeout.
__device__ __noinline__ bool persist_sample(const Dev *Sv, GPR_LDS unsigned char *rawl, GPR_LDS int *bufl, int lmax_, int a0_, int a1_,
                                            int r_, int g_, int G_, int target_, int energy_)
{
    const Dev &S = *(const Dev *)uni64((long long)Sv);
    unsigned char *const raw = (unsigned char *)rawl;
    const int lmax = uni(lmax_), a0 = uni(a0_), a1 = uni(a1_), r = uni(r_), g = uni(g_), G = uni(G_), target = uni(target_);
    const bool energy = uni(energy_) != 0;
    const int tid = threadIdx.x, BT = blockDim.x, n = S.n, np = S.np;
    const PersistOff o = persist_off(n, np, lmax);
    const PosLDS xs{(const float4 *)(raw + o.xs)};
    const float *vs = (const float *)(raw + o.vs);
    long long *red = (long long *)(raw + o.red), *eacc = red + MAX_OBS * 8;
    double *vals = (double *)(raw + o.vals);
    float *vg = S.v + (size_t)r * 3 * np;
    __syncthreads();
    if (G == 1) {
        for (int k = tid; k < 3 * np; k += BT) gmut(vg)[k] = k % np < n ? vs[(k / np) * lmax + k % np] : 0.f;
        __syncthreads();
        observables_wg(S, xs, vg, unfix_d(*eacc), red, vals, tid, BT);
        if (tid == 0) accumulate_obs(S, r, vals);
        return true;
    }
    for (int a = a0 + tid; a < a1; a += BT) {
        const int l = a - a0;
        st_coh(vg + a, vs[l]); st_coh(vg + np + a, vs[lmax + l]); st_coh(vg + 2 * np + a, vs[2 * lmax + l]);
    }
    if (tid == 0 && energy && *eacc != 0)
        __hip_atomic_fetch_add(S.esum + r, *eacc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!group_barrier(S.sync + (size_t)r * 64, target, S.err, (int *)bufl)) return false;
    if (g == 0) {
        // the sum of the groups' energies, by way of the accumulator.  The sum is cleared by the exchange that
        // reads it: its value is there, and so the clearing done, before this group's waves pass the
        // barrier and publish the next step's positions, which the other groups need to add to it again
        if (tid == 0) *eacc = __hip_atomic_exchange(S.esum + r, 0ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        observables_wg(S, xs, vg, unfix_d(*eacc), red, vals, tid, BT, true);
        if (tid == 0) accumulate_obs(S, r, vals);
    }
    return true;
}

// Waves of a workgroup that start with the bonded units (the others start the pair tasks; us per step
// with 8, 12 and 16: 2,432 atoms x 64 replicas 20.0, 20.2, 20.2; 1,200 x 192 35.9, 36.8, 36.8; 300 x 24
// 7.7, 7.5, 8.1)
constexpr int NBW = 8;
__device__ __forceinline__ void persist_replica(const Dev &S, int G, int lmax, int a0, int a1, int u0, int u1,
                                                const uint2 *bi, const float4 *bp, int noise_ahead, int r, int g,
                                                long long s0, int nsteps, int t0, int sample, int state_end)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int np = uni(S.np), n = uni(S.n);
    __shared__ int bbuf, hbuf, ptask, btask, torder[64];   // torder: [128] the search's task order, 16 bits each

    const int tid = threadIdx.x, BT = blockDim.x;
#ifdef GPR_PHASE_PROBE
    __shared__ unsigned long long ph_acc[NPHASE + 1];
    if (tid < NPHASE) ph_acc[tid] = 0;
#endif
    const size_t b = (size_t)r * 3 * np;
    GPR_GLOBAL int *const sync = gmut(((const GPR_CONST Dev *)&S)->sync) + (size_t)r * 64;
    // position exchange, one buffer per step parity, [2][2][np] 64-bit words: (x, half of y) and (z, the
    // other half) under a 16-bit tag, 2 (1 + step of this launch mod 32,767) + (the atom passed its
    // displacement margin).  A word is there when its tag is (the word it replaces has the tag of two
    // steps before, or none), so the groups need no barrier: a reader polls the words themselves.
    // A group writes step s + 1 over step s - 1 once it has every other group's step s, which each
    // of them wrote after reading step s - 1 (so every group owns atoms: the host lays out no other).
    GPR_GLOBAL unsigned long long *const xchg = gmut(((const GPR_CONST Dev *)&S)->xchg) + (size_t)r * 4 * np;
    int gen = 0;

#ifdef GPR_PHASE_PROBE
    if (tid == 0) ph_acc[NPHASE] = ph_acc[PH_START] = __builtin_amdgcn_s_memrealtime();
#endif
    // descriptor fields used every step, held in registers for the launch
    const GPR_CONST Dev &C = *(const GPR_CONST Dev *)&S;
    const IntConsts ik{C.h, C.c1, C.key0, C.key1, C.kind == KIND_TOY};
    const int nl = a1 - a0;
    {
        const PersistOff o = persist_off(n, np, lmax);
        long long *fa = (long long *)(lds_raw + o.fa);
        float *vs = (float *)(lds_raw + o.vs), *iml = (float *)(lds_raw + o.iml), *sdl = (float *)(lds_raw + o.sdl);
        float *xbl = (float *)(lds_raw + o.xbl), *gn = (float *)(lds_raw + o.gn);
        float4 *box = (float4 *)(lds_raw + o.box);
        stage_replica(S, r, (float4 *)(lds_raw + o.xs), (float2 *)lds_raw, tid, BT);
        const GPR_GLOBAL float *xbg = gconst(S.xb) + b, *vg = gconst(S.v) + b;
        const GPR_GLOBAL long long *Fg = gconst(S.F) + b;
        for (int k = tid; k < 3 * lmax; k += BT) {
            const int d = k / lmax, a = a0 + k % lmax;
            vs[k] = a < a1 ? vg[d * np + a] : 0.f;
            fa[3 * (k % lmax) + d] = a < a1 ? Fg[d * np + a] : 0;
            xbl[k] = a < a1 ? xbg[d * np + a] : 0.f;
        }
        for (int l = tid; l < lmax; l += BT) {
            const int a = a0 + l;
            iml[l] = a < a1 ? gld(gconst(S.prm) + a).w : 0.f;
            sdl[l] = a < a1 ? gconst(S.sd)[a] : 0.f;
            if (noise_ahead && a < a1) {
                const float3 z = step_noise(ik, a, r, s0);
                gn[l] = z.x; gn[lmax + l] = z.y; gn[2 * lmax + l] = z.z;
            }
        }
        for (int t = tid; t < (n + BLK - 1) / BLK; t += BT) box[t].w = __uint_as_float((unsigned)gconst(S.cls)[t] << 24);
    }
    // the pair loop below runs each atom's four sub-lists to one count, which needs lists
    // padded as this kernel's search writes them: lists from the plain path's search, or a
    // replica marked for a rebuild (a new configuration), are rebuilt at the first step;
    // padded lists from an earlier launch are kept, their counts and order recomputed
    const bool toy = C.kind == KIND_TOY;
    bool need = !toy && (S.need_build[r] != 0 || S.list_pad[r] == 0);
    int built = 0;                                          // rebuilds of this launch
    long long lastb = S.last_build[(s0 & 1) * S.R + r];     // step of the last pair-list build
    if (!toy && !need) {
        const PersistOff o = persist_off(n, np, lmax);
        GPR_LDS unsigned short *keyl = (GPR_LDS unsigned short *)(lds_raw + o.keyl);
        const size_t stride = (size_t)np * P;
        const GPR_GLOBAL unsigned short *cnt = gconst(S.nbc) + (size_t)r * stride;
        for (int l = tid; l < nl; l += BT) {
            const int i = a0 + l;
            int k = 0;
#pragma unroll
            for (int q = 0; q < P; ++q) k = max(k, (int)cnt[(size_t)i * P + q]);
            keyl[l] = (unsigned short)k;
        }
        __syncthreads();
        order_atoms(keyl, (GPR_LDS unsigned short *)(lds_raw + o.perm), (GPR_LDS int *)(lds_raw + o.red), nl, tid, BT);
    }
    if (tid == 0) { bbuf = 1; hbuf = 0; }
    bool alive = true;
    if (G > 1) {
        // no tag of an earlier launch is left when the first word is read
        for (int k = tid; k < 4 * nl; k += BT) {
            const int d = k / nl, l = k - d * nl;
            st_coh(xchg + d * np + a0 + l, 0ull);
        }
        alive = group_barrier((int *)sync, G * ++gen, (int *)gmut(C.err), &bbuf);
    }
    const int t_gr = C.t_gr, need_energy = C.need_energy, cutoff_on = C.cutoff_on, period = C.period;
    const float im_light = C.im_light, guard2_light = C.guard2_light, guard2_heavy = C.guard2_heavy;
    const float rc2 = C.rc2, krf = C.krf, krf2 = 2.0f * C.krf, crf = C.crf;
    GPR_GLOBAL int *const errp = gmut(C.err);
    // the replica's lists: word g of sub-list (i, q) is word g np P + i P + q
    const GPR_GLOBAL char *const lists = (const GPR_GLOBAL char *)gconst(C.nbl) + (size_t)r * C.Kg * np * P * 8;
    const unsigned lstep = (unsigned)np * P * 8;
    // the bonded units of the group's atoms go to its last (up to) NBW waves; the other waves
    // meanwhile start the pair tasks
    const int wv = uni(tid >> 6), nbw = min(BT >> 6, NBW), bw0 = (BT >> 6) - nbw;
    bool pend = false;                                      // the previous step's closing B is due
    __syncthreads();
    PHASE_MARK(PH_PROLOGUE);

    for (int step = 0; step < nsteps && alive; ++step) {
        const long long s = s0 + step;
        const bool samp = sample && r >= 1 && ((t0 + step + 1) % t_gr == 0);
        const bool energy = samp && need_energy;
        bool hit = false, bad = false;
        {
            const int lm = fresh_s(lmax);
            const PersistOff o = persist_off(fresh_s(n), fresh_s(np), lm);
            long long *fa = (long long *)(lds_raw + o.fa);
            float4 *xs = (float4 *)(lds_raw + o.xs);
            float *vs = (float *)(lds_raw + o.vs), *iml = (float *)(lds_raw + o.iml), *sdl = (float *)(lds_raw + o.sdl);
            const float *xbl = (const float *)(lds_raw + o.xbl), *gn = (const float *)(lds_raw + o.gn);
            GPR_GLOBAL unsigned long long *const xw = xchg + (step & 1) * 2 * np;
            for (int l = fresh_v(tid); l < nl; l = fresh_v(l + BT)) {
                const int a = a0 + l;
                float3 x = make_float3(xs[a].x, xs[a].y, xs[a].z);
                float3 v = make_float3(vs[l], vs[lm + l], vs[2 * lm + l]);
                const float3 F = make_float3(unfix_f(fa[3 * l]), unfix_f(fa[3 * l + 1]), unfix_f(fa[3 * l + 2]));
                fa[3 * l] = fa[3 * l + 1] = fa[3 * l + 2] = 0;    // (these forces are read here for the last time)
                const float im = iml[l];
                if (pend) {
                    // the previous step's closing B, deferred to here (same forces, same order)
                    v.x = kick(v.x, F.x, ik.h, im);
                    v.y = kick(v.y, F.y, ik.h, im);
                    v.z = kick(v.z, F.z, ik.h, im);
                    bad |= bad_force(F.x) || bad_force(F.y) || bad_force(F.z);
                }
                const float3 z = noise_ahead ? make_float3(gn[l], gn[lm + l], gn[2 * lm + l]) : step_noise(ik, a, r, s);
                integrate_baoa_g(ik, x, v, F, im, sdl[l], z);
                xs[a].x = x.x; xs[a].y = x.y; xs[a].z = x.z;
                vs[l] = v.x; vs[lm + l] = v.y; vs[2 * lm + l] = v.z;
                bad |= !(finite3(x) && finite3(v));
                bool out = false;
                if (cutoff_on) {
                    const float dx = x.x - xbl[l], dy = x.y - xbl[lm + l], dz = x.z - xbl[2 * lm + l];
                    out = !(dx * dx + dy * dy + dz * dz <= (im > im_light ? guard2_light : guard2_heavy));
                    hit |= out;
                }
                if (G > 1) {
                    const unsigned y = __float_as_uint(x.y), tag = 2u * step_tag(step) + (unsigned)out;
                    st_coh(xw + a, tagged(x.x, (tag << 16) | (y & 0xFFFFu)));
                    st_coh(xw + np + a, tagged(x.z, (tag << 16) | (y >> 16)));
                }
            }
            if (tid == 0) { *((long long *)(lds_raw + o.red) + MAX_OBS * 8) = 0; ptask = 0; atomicAnd(&hbuf, 1 << (step & 1)); }
        }
        if (bad) atomicOr((int *)&errp[ERR_UNSTABLE], 1);
        PHASE_MARK(PH_INTEGRATE);
        if (G > 1) {
            // while the words travel, draw the next step's Gaussians
            if (noise_ahead) {
                const int lm = fresh_s(lmax);
                float *gn = (float *)(lds_raw + persist_off(fresh_s(n), fresh_s(np), lm).gn);
                for (int l = fresh_v(tid); l < nl; l = fresh_v(l + BT)) {
                    const float3 z = step_noise(ik, a0 + l, r, s + 1);
                    gn[l] = z.x; gn[lm + l] = z.y; gn[2 * lm + l] = z.z;
                }
            }
            // then each thread polls its share of the other groups' atoms (bounded)
            const int nn = fresh_s(n), npp = fresh_s(np), others = nn - nl;
            float4 *xs = (float4 *)(lds_raw + persist_off(nn, npp, fresh_s(lmax)).xs);
            const GPR_GLOBAL unsigned long long *const xw = xchg + (step & 1) * 2 * npp;
            const unsigned tag = step_tag(step);
            constexpr int XU = 2;                           // (3 and 4 cost 1 to 2 %)
            int spins = 0;
            for (int k0 = fresh_v(tid); __any(k0 < others) && spins <= SPIN_MAX; k0 = fresh_v(k0 + XU * BT)) {
                unsigned long long w[XU][2];
                for (;;) {
                    int miss = -1;                          // a word that is not there yet
#pragma unroll
                    for (int u = 0; u < XU; ++u) {
                        const int k = min(k0 + u * BT, others - 1), a = k < a0 ? k : k + nl;
                        w[u][0] = ld_coh(xw + a);
                        w[u][1] = ld_coh(xw + npp + a);
                    }
#pragma unroll
                    for (int u = 0; u < XU; ++u) {
                        const int k = min(k0 + u * BT, others - 1), a = k < a0 ? k : k + nl;
                        if ((unsigned)(w[u][0] >> 49) != tag) miss = a;
                        if ((unsigned)(w[u][1] >> 49) != tag) miss = npp + a;
                    }
                    if (!__any(miss >= 0)) break;
                    // wait for one missing word per lane, then read all again
                    while (__any(miss >= 0) && ++spins <= SPIN_MAX) {
                        __builtin_amdgcn_s_sleep(1);
                        if (miss >= 0 && (unsigned)(ld_coh(xw + miss) >> 49) == tag) miss = -1;
                    }
                    if (spins > SPIN_MAX) {
                        atomicOr((int *)errp + ERR_BARRIER, 1);
                        bbuf = 0;
                        break;
                    }
                }
#pragma unroll
                for (int u = 0; u < XU; ++u) {
                    const int k = min(k0 + u * BT, others - 1), a = k < a0 ? k : k + nl;
                    const unsigned y = ((unsigned)(w[u][0] >> 32) & 0xFFFFu) | ((unsigned)(w[u][1] >> 32) << 16);
                    xs[a].x = __uint_as_float((unsigned)w[u][0]); xs[a].y = __uint_as_float(y);
                    xs[a].z = __uint_as_float((unsigned)w[u][1]);
                    hit |= ((w[u][0] >> 48) & 1) != 0;
                }
            }
        }
        // the step's hits in bit s % 2, cleared by the next step
        if (hit) atomicOr(&hbuf, 1 << (step & 1));
        __syncthreads();
        const bool any_hit = (hbuf >> (step & 1)) & 1;
        alive = bbuf != 0;
        if (!alive) break;
        PHASE_MARK(PH_EXCHANGE);
        // each replica is its own set of workgroups here, so its list is rebuilt when it is
        // period steps old (or flagged), independently of the other replicas
        if (need || (cutoff_on && (any_hit || s - lastb >= period))) {
            PHASE_COUNT(PH_NREBUILD);
            lastb = s;
            persist_rebuild(&S, (GPR_LDS unsigned char *)lds_raw, (GPR_LDS int *)&btask, (GPR_LDS int *)torder, lmax, a0, a1, r,
                            built % ORDER_PERIOD == 0);
            ++built;
            if (need && g == 0 && tid == 0) S.list_pad[r] = 1;
            need = false;
        }
        PHASE_MARK(PH_REBUILD);
        const int lm = fresh_s(lmax);
        const PersistOff o = persist_off(fresh_s(n), fresh_s(np), lm);
        long long *const fa = (long long *)(lds_raw + o.fa), *const eacc = (long long *)(lds_raw + o.red) + MAX_OBS * 8;
        const float4 *const xs = (const float4 *)(lds_raw + o.xs);
        const float2 *const pp = (const float2 *)lds_raw;
        if (toy) {
            if (tid == 0 && a0 == 0 && a1 > 0) {
                float fx, fy;
                const float u = toy_force(xs[0].x, xs[0].y, fx, fy);
                fa[0] = fix_f(fx);
                fa[1] = fix_f(fy);
                if (energy) *eacc = fix_f(u);
            }
        } else {
            const unsigned short *const perm = (const unsigned short *)(lds_raw + o.perm), *const keyl = (const unsigned short *)(lds_raw + o.keyl);
            float *const gn = (float *)(lds_raw + o.gn);
            const int lane = fresh_v(tid) & 63, q = lane & 3;
            // bonded units on the last waves, then the pair loop, whose tasks (16 atoms each,
            // longest lists first) the waves take from a shared counter as they come free
            if (wv >= bw0) {
                const ForceLDS F{fa, a0, 3, 1};
                if (energy) {
                    const long long e = bonded_units<true>(bi, bp, u0, u1, PosLDS{xs}, F, wv - bw0, nbw, lane);
                    if (e != 0) lds_add(eacc, e);
                } else {
                    bonded_units<false>(bi, bp, u0, u1, PosLDS{xs}, F, wv - bw0, nbw, lane);
                }
            }
            const int ntask = (nl + 15) >> 4, nnoise = G == 1 && noise_ahead ? (nl + 63) >> 6 : 0;
            for (;;) {
                int t = 0;
                if (lane == 0) t = lds_inc((GPR_LDS int *)&ptask);
                t = uni(t);
                if (t >= ntask) {
                    // after them, with no exchange to draw them in, the next step's Gaussians
                    if (t >= ntask + nnoise) break;
                    const int l = 64 * (t - ntask) + lane;
                    if (l < nl) {
                        const float3 z = step_noise(ik, a0 + l, r, s + 1);
                        gn[l] = z.x; gn[lm + l] = z.y; gn[2 * lm + l] = z.z;
                    }
                    continue;
                }
                const int l = perm[16 * t + (lane >> 2)];
                long long eatom = 0;
                if (l != 0xFFFF) {
                    const int i = a0 + l;
                    const unsigned off = (unsigned)(i * P + q) * 8;
                    float4 f = energy ? pair_sums<true>(lists, off, lstep, keyl[l], xs[i], pp[i], xs, pp, rc2, krf2, krf, crf)
                                      : pair_sums<false>(lists, off, lstep, keyl[l], xs[i], pp[i], xs, pp, rc2, krf2, krf, crf);
                    f.x = quad_sum(f.x);
                    f.y = quad_sum(f.y);
                    f.z = quad_sum(f.z);
                    // one lane of the atom per component, and one for the energy
                    if (q < 3) lds_add(&fa[3 * l + q], fix_f(q == 0 ? f.x : (q == 1 ? f.y : f.z)));
                    if (energy) {
                        f.w = quad_sum(f.w);
                        if (q == 3) eatom = fix_f(f.w);
                    }
                }
                if (energy) {
                    eatom = wave_sum_ll(eatom);
                    if (lane == 0 && eatom != 0) lds_add(eacc, eatom);
                }
            }
        }
        __syncthreads();
        PHASE_MARK(PH_FORCES);
        // the closing B: here when the step's velocities are read (a sample, the end of the
        // launch), else by the next step's integrator
        pend = !(samp || step + 1 == nsteps);
        if (!pend) {
            float *const vs = (float *)(lds_raw + o.vs);
            const float *const iml = (const float *)(lds_raw + o.iml);
            for (int l = fresh_v(tid); l < nl; l = fresh_v(l + BT)) {
                const float im = iml[l], h = ik.h;
                const float Fx = unfix_f(fa[3 * l]), Fy = unfix_f(fa[3 * l + 1]), Fz = unfix_f(fa[3 * l + 2]);
                vs[l] = kick(vs[l], Fx, h, im);
                vs[lm + l] = kick(vs[lm + l], Fy, h, im);
                vs[2 * lm + l] = kick(vs[2 * lm + l], Fz, h, im);
                if (bad_force(Fx) || bad_force(Fy) || bad_force(Fz)) atomicOr((int *)&errp[ERR_UNSTABLE], 1);
            }
            if (samp) {
                if (G > 1) ++gen;
                alive = persist_sample(&S, (GPR_LDS unsigned char *)lds_raw, (GPR_LDS int *)&bbuf, lmax, a0, a1, r, g, G, G * gen, energy);
            }
            __syncthreads();
        }
        PHASE_MARK(PH_TAIL);
        PHASE_COUNT(PH_NSTEP);
    }
    // write back this group's atoms
    const PersistOff o = persist_off(n, np, lmax);
    const float4 *const xs = (const float4 *)(lds_raw + o.xs);
    {
        const long long *fa = (const long long *)(lds_raw + o.fa);
        const float *vs = (const float *)(lds_raw + o.vs), *xbl = (const float *)(lds_raw + o.xbl);
        GPR_GLOBAL float *xg = gmut(S.x) + b, *vg = gmut(S.v) + b, *xbg = gmut(S.xb) + b;
        GPR_GLOBAL long long *Fg = gmut(S.F) + b;
        for (int l = tid; l < nl; l += BT) {
            const int a = a0 + l;
            xg[a] = xs[a].x; xg[np + a] = xs[a].y; xg[2 * np + a] = xs[a].z;
            for (int d = 0; d < 3; ++d) {
                vg[d * np + a] = vs[d * lmax + l];
                Fg[d * np + a] = fa[3 * l + d];
                xbg[d * np + a] = xbl[d * lmax + l];
            }
        }
    }
    if (g == 0 && tid == 0 && nsteps > 0) {
        S.need_build[r] = 0;
        S.last_build[((s0 + nsteps) & 1) * S.R + r] = lastb;
    }
    if (state_end && g == 0) {
        __syncthreads();
        const int id = state_wg(S, PosLDS{xs}, (long long *)(lds_raw + o.red), &hbuf, tid, BT);
        if (tid == 0) S.state[r] = id;
    }
    if (G > 1 && nsteps > 0) {
        // the replica's barrier line is left clear for the next launch by the last of its groups
        // to finish (each group counts itself out in slot 8 once none of its waves reads the
        // line again), so that no launch needs it cleared beforehand
        __syncthreads();
        if (tid == 0 && __hip_atomic_fetch_add(sync + 8, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1) {
            __hip_atomic_store(sync, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(sync + 8, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
#ifdef GPR_PHASE_PROBE
    PHASE_MARK(PH_EPILOGUE);
    if (tid == 0 && r < PHASE_MAX_R && g < PHASE_MAX_G) {
        unsigned long long *acc = gpr_phase_acc + ((size_t)r * PHASE_MAX_G + g) * NPHASE;
        for (int k = 0; k < PH_START; ++k) acc[k] += ph_acc[k];
        acc[PH_START] = ph_acc[PH_START];
        acc[PH_END] = __builtin_amdgcn_s_memrealtime();
    }
#endif
}

// The first step and local step of cycle it.cycle of a captured run; false after the check that
// ended the call
__device__ __forceinline__ bool cycle_start(const PersistItem &it, long long &s0, int &t0)
{
    if (it.cyc->halt_cycle < it.cycle) return false;
    const long long first = (long long)it.cycle * it.nsteps;
    s0 = it.cyc->s_start + first;
    t0 = (int)((it.cyc->t_start + first) % it.dev->t_gr);
    return true;
}

// A workgroup's place in a launch whose workgroups wait for one another: in the order in which they
// start, not by blockIdx.  Of the first `mapped` workgroups, those with equal blockIdx mod 8 keep that
// residue (they are of one XCD) and the order counts among them; the order of the others counts
// among all of those.  So when a launch gets only part of the device, beside another process's, the
// workgroups that do run make whole replicas but for one in each of these rows; the whole ones end
// and make room, where workgroups placed by blockIdx could all be waiting for others that have none.
// (The last to ask clears the counter for the next launch.)
__device__ __forceinline__ int start_place(int *ticket, int mapped)
{
    __shared__ int place;
    if (threadIdx.x == 0) {
        const int b = (int)blockIdx.x, c = b < mapped ? b % 8 : 8;
        int *const ctr = ticket + 32 * c;
        const int total = c < 8 ? mapped / 8 : (int)gridDim.x - mapped;
        const int t = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t == total - 1) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        place = c < 8 ? 8 * t + c : mapped + t;
    }
    __syncthreads();
    return uni(place);
}

// One system, one replica per set: replicas roff, roff + 1, ... (a system with more replicas
// than sets that fit at once takes several launches, each with the body inlined).
__global__ void __launch_bounds__(1024) k_persist(PersistItem it)
{
    int set, g;
    long long s0 = it.s0;
    int t0 = it.t0;
    if (it.cyc && !cycle_start(it, s0, t0)) return;
    // (with one workgroup per replica too, though it waits for none: a choice between the two here
    // cost the step loop 8 registers and 32 bytes of scratch, 5 to 11 % of a step)
    const int local = start_place(it.dev->ticket, it.xcd ? (int)gridDim.x : 0);
    if (!persist_place(it, local, set, g) || set + it.roff >= it.nrep) return;
    persist_replica(*it.dev, it.sp.G, it.sp.lmax, it.sp.bnd[g], it.sp.bnd[g + 1], it.sp.bu[g], it.sp.bu[g + 1], it.sp.bi,
                    it.sp.bp, it.noise_ahead, set + it.roff, g, s0, it.nsteps, t0, it.sample, it.state_end);
}

// ------------------------------------------------------------------ small systems
// A step of a small replica (one workgroup) is a chain of latencies, not work: on the general body
// it waits for list words and terms read from memory, runs the Philox rounds before every drift
// and passes six barriers.  Here everything a step reads is in LDS for the whole launch, the step
// has two barriers, and between them each wave takes units of independent work:
//   a block of 64 bonded terms of one kind; a pair task (16 atoms on 64 lanes, all partners in the
//   sub-list order of the pair lists: lane 4 (i - i0) + q runs over j = q, q + 4, ... with the
//   partners outside the list, the cutoff or the system adding an exact zero); the Gaussians of
//   the next step for 64 atoms.
// The arithmetic, its order and the fixed-point sums are the general body's, so are the bits.  The
// integrator takes a component per thread, which is a third of its chain (0.58 -> 0.42 of 1.6 us a
// step at 22 atoms); the rest is one wave's torsions or pairs, about 0.9 us of dependent arithmetic
// and LDS atomics whichever way they are split (four lanes a torsion came out the same).
// Pairs are not listed (up to SMALL_MAX atoms running over all of them costs less than reading a
// list), so the launch leaves a system with a cutoff marked for a list rebuild.
struct SmallLds {
    long long *fa;              // [2][3][n] force accumulators: one read, the other being summed
    long long *red;             // [8] scratch of the state test
    double *acc, *shift;        // [MAX_OBS][2], [MAX_OBS]
    float4 *xs;                 // [np]
    float2 *pp;                 // [np]
    unsigned long long *am;     // [64 ceil(n / 16)] bit k: partner 4 k + q of the lane's atom counts
    float4 *tp;                 // [nterm] parameters of the bonded terms
    uint2 *ti;                  // [nterm] their atoms, 16 bits each
    ObsDesc *ob;                // [MAX_OBS]
    float *vs, *im, *sd, *gn;   // [3][n], [n], [n], [3][n]: velocities, 1/m, noise amplitudes, Gaussians
};

__device__ __forceinline__ SmallLds small_lds_layout(unsigned char *raw, int n, int np, int nterm)
{
    SmallLds L;
    L.xs = (float4 *)raw;
    L.tp = L.xs + np;
    L.fa = (long long *)(L.tp + nterm);
    L.red = L.fa + 6 * n;
    L.acc = (double *)(L.red + 8);
    L.shift = L.acc + 2 * MAX_OBS;
    L.ob = (ObsDesc *)(L.shift + MAX_OBS);
    L.pp = (float2 *)(L.ob + MAX_OBS);
    L.am = (unsigned long long *)(L.pp + np);
    L.ti = (uint2 *)(L.am + 64 * ((n + 15) >> 4));
    L.vs = (float *)(L.ti + nterm);
    L.im = L.vs + 3 * n;
    L.sd = L.im + n;
    L.gn = L.sd + n;
    return L;
}

// Observable j of the replica by one wave (the value is valid in lane 0); the sums over atoms are
// the integer sums of observables_wg, in another order
__device__ double small_observable(const Dev &S, const ObsDesc &o, const SmallLds &L, double U, int lane)
{
    const int n = S.n;
    auto vel2 = [&](int a) {
        const double vx = L.vs[a], vy = L.vs[n + a], vz = L.vs[2 * n + a];
        return vx * vx + vy * vy + vz * vz;
    };
    auto com = [&](int off, int cnt, double m, double &cx, double &cy, double &cz) {
        long long s0 = 0, s1 = 0, s2 = 0;
        for (int k = lane; k < cnt; k += 64) {
            const int a = S.groups[off + k];
            const double ma = (double)S.mass[a];
            s0 += fix_d(ma * (double)L.xs[a].x);
            s1 += fix_d(ma * (double)L.xs[a].y);
            s2 += fix_d(ma * (double)L.xs[a].z);
        }
        cx = unfix_d(wave_sum_ll(s0)) / m;
        cy = unfix_d(wave_sum_ll(s1)) / m;
        cz = unfix_d(wave_sum_ll(s2)) / m;
    };
    switch (o.kind) {
    case OB_COORD: {
        const float4 p = L.xs[o.atoms[0]];
        return o.atoms[1] == 0 ? (double)p.x : (o.atoms[1] == 1 ? (double)p.y : (double)p.z);
    }
    case OB_POT: return U;
    case OB_KIN: {
        long long s = 0;
        for (int a = lane; a < n; a += 64) s += fix_d(0.5 * (double)S.mass[a] * vel2(a));
        return unfix_d(wave_sum_ll(s));
    }
    case OB_DIH: return dihedral_d(xs_d(PosLDS{L.xs}, o.atoms[0]), xs_d(PosLDS{L.xs}, o.atoms[1]), xs_d(PosLDS{L.xs}, o.atoms[2]),
                                   xs_d(PosLDS{L.xs}, o.atoms[3]));
    case OB_COMD: {
        double ax, ay, az, bx, by, bz;
        com(o.ga_off, o.ga_n, o.ma, ax, ay, az);
        com(o.gb_off, o.gb_n, o.mb, bx, by, bz);
        return sqrt((ax - bx) * (ax - bx) + (ay - by) * (ay - by) + (az - bz) * (az - bz));
    }
    case OB_RMSV: {
        long long s = 0;
        for (int k = lane; k < o.ga_n; k += 64) s += fix_d(vel2(S.groups[o.ga_off + k]));
        return sqrt(unfix_d(wave_sum_ll(s)) / (double)o.ga_n);
    }
    default: return 0.0;
    }
}

// The pairs of one lane with its nk partners xj[4 k], k = 0, 1, ... (staged far away past n), those
// not in the mask adding an exact zero
template <bool ENERGY>
__device__ __forceinline__ void small_pairs(const float4 pi, const float2 ppi, const float4 *xj, const float2 *pj,
                                            unsigned long long m, int nk, float rc2, float krf2, float krf, float crf,
                                            float &fx, float &fy, float &fz, float &e)
{
    auto pair = [&](int k, int bit) {
        const float lim = __uint_as_float(__float_as_uint(rc2) & (0u - (((unsigned)m >> bit) & 1u)));
        pair_term(pi, ppi, xj[4 * k], pj[4 * k], lim, krf2, krf, crf, ENERGY, fx, fy, fz, e);
    };
    int k = 0;
    for (; k + 4 <= nk; k += 4, m >>= 4) {
#pragma unroll
        for (int w = 0; w < 4; ++w) pair(k + w, w);
    }
    if (nk & 2) { pair(k, 0); pair(k + 1, 1); k += 2; m >>= 2; }
    if (nk & 1) pair(k, 0);
}

__device__ __forceinline__ void persist_small(const Dev &S, int r, long long s0, int nsteps, int t0, int sample,
                                              int state_end)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ int sbuf;
    __shared__ long long eacc[2];
    const int tid = threadIdx.x, BT = blockDim.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nwv = BT >> 6;
    const int n = S.n, np = S.np;
    const bool toy = S.kind == KIND_TOY;
    const Topo &T = S.tp;
    const int nt = T.nt, na = T.na, n14 = T.n14, nb = T.nb, nr = T.nr;
    const SmallLds L = small_lds_layout(lds_raw, n, np, nt + na + n14 + nb + nr);
#ifdef GPR_PHASE_PROBE
    __shared__ unsigned long long ph_acc[NPHASE + 1];
    if (tid < NPHASE) ph_acc[tid] = 0;
    if (tid == 0) ph_acc[NPHASE] = ph_acc[PH_START] = __builtin_amdgcn_s_memrealtime();
#endif
    const size_t b = (size_t)r * 3 * np;
    const IntConsts ik = int_consts(S);
    const float rc2 = S.rc2, krf = S.krf, krf2 = 2.0f * S.krf, crf = S.crf;
    const int t_gr = S.t_gr, need_energy = S.need_energy;
    int *const errp = S.err;
    const int npt = toy ? 0 : (n + 15) >> 4;

    // stage the replica and its terms
    stage_replica(S, r, L.xs, L.pp, tid, BT);
    for (int a = tid; a < n; a += BT) {
        const float3 g = step_noise(ik, a, r, s0);
        for (int d = 0; d < 3; ++d) {
            L.vs[d * n + a] = gconst(S.v)[b + d * np + a];
            L.fa[d * n + a] = gconst(S.F)[b + d * np + a];
            L.fa[(3 + d) * n + a] = 0;
        }
        L.im[a] = gld(gconst(S.prm) + a).w;
        L.sd[a] = gconst(S.sd)[a];
        L.gn[a] = g.x; L.gn[n + a] = g.y; L.gn[2 * n + a] = g.z;
    }
    auto pack = [](int i, int j, int k, int l) { return make_uint2((unsigned)i | ((unsigned)j << 16), (unsigned)k | ((unsigned)l << 16)); };
    for (int t = tid; t < nt; t += BT) {
        const int4 q = gld(gconst(T.t_ijkl) + t);
        L.ti[t] = pack(q.x, q.y, q.z, q.w);
        L.tp[t] = gld(gconst(T.t_p) + t);
    }
    for (int t = tid; t < na; t += BT) {
        const int4 q = gld(gconst(T.a_ijk) + t);
        const float2 p = gld(gconst(T.a_p) + t);
        L.ti[nt + t] = pack(q.x, q.y, q.z, 0);
        L.tp[nt + t] = make_float4(p.x, p.y, 0.f, 0.f);
    }
    for (int t = tid; t < n14; t += BT) {
        const int2 q = gld(gconst(T.p_ij) + t);
        L.ti[nt + na + t] = pack(q.x, q.y, 0, 0);
        L.tp[nt + na + t] = gld(gconst(T.p_p) + t);
    }
    for (int t = tid; t < nb; t += BT) {
        const int2 q = gld(gconst(T.b_ij) + t);
        const float2 p = gld(gconst(T.b_p) + t);
        L.ti[nt + na + n14 + t] = pack(q.x, q.y, 0, 0);
        L.tp[nt + na + n14 + t] = make_float4(p.x, p.y, 0.f, 0.f);
    }
    for (int t = tid; t < nr; t += BT) {
        L.ti[nt + na + n14 + nb + t] = pack(gconst(T.r_i)[t], 0, 0, 0);
        L.tp[nt + na + n14 + nb + t] = gld(gconst(T.r_p) + t);
    }
    // partners of lane (i, q): every j = 4 k + q < n but itself, the excluded and the 1-4 ones
    for (int c = tid; c < 64 * npt; c += BT) {
        const int i = c >> 2, q = c & 3;
        unsigned long long m = 0ull;
        if (i < n) {
            const unsigned long long ex = gconst(S.excl)[i] | (1ull << 32);
            for (int k = 0; 4 * k + q < n; ++k) {
                const int off = 4 * k + q - i + 32;
                const bool drop = (unsigned)off < 64u && ((ex >> off) & 1ull);
                m |= (unsigned long long)!drop << k;
            }
            if (S.has_far)
                for (int f = gconst(S.far_start)[i]; f < gconst(S.far_start)[i + 1]; ++f) {
                    const int j = gconst(S.far_j)[f];
                    if ((j & 3) == q) m &= ~(1ull << (j >> 2));
                }
        }
        L.am[c] = m;
    }
    if (tid < 2 * MAX_OBS) L.acc[tid] = S.acc[(size_t)r * 2 * MAX_OBS + tid];
    if (tid < MAX_OBS) {
        L.shift[tid] = S.shift[tid];
        L.ob[tid] = S.obs[tid];
    }
    if (tid < 2) eacc[tid] = 0;
    __syncthreads();
    PHASE_MARK(PH_PROLOGUE);

    // units of a step, the longest first: torsions, pair tasks, angles, noise, 1-4, bonds, restraints,
    // the toy potential
    const int u0 = (nt + 63) >> 6, u1 = u0 + npt, u2 = u1 + ((na + 63) >> 6), u3 = u2 + ((n + 63) >> 6), u4 = u3 + ((n14 + 63) >> 6), u5 = u4 + ((nb + 63) >> 6), u6 = u5 + ((nr + 63) >> 6), u7 = u6 + toy;
    bool pend = false;                                      // the previous step's closing B is due
    int cur = 0;                                            // accumulators holding the last forces
    for (int step = 0; step < nsteps; ++step) {
        const bool samp = sample && r >= 1 && ((t0 + step + 1) % t_gr == 0);
        const bool energy = samp && need_energy;
        // B A O A; the accumulators read here are cleared while the others are being summed
        long long *const f0 = L.fa + 3 * n * cur;
        bool bad = false;
        // (a component per thread: integrate_baoa_g's operations, none of which mixes them)
        for (int k = tid; k < 3 * n; k += BT) {
            const int d = (k >= n) + (k >= 2 * n), a = k - d * n;
            float *const xp = (float *)(L.xs + a) + d;
            float x = *xp, v = L.vs[k];
            const float F = unfix_f(f0[k]), im = L.im[a], h = ik.h;
            if (pend) {
                v = kick(v, F, h, im);
                bad |= bad_force(F);
            }
            v = kick(v, F, h, im);
            x = x + h * v;
            if (!(toy && d == 2)) v = ik.c1 * v + L.sd[a] * L.gn[k];
            x = x + h * v;
            *xp = x;
            L.vs[k] = v;
            bad |= !(isfinite(x) && isfinite(v));
        }
        if (bad) atomicOr(&errp[ERR_UNSTABLE], 1);
        cur ^= 1;
        long long *const fa = L.fa + 3 * n * cur;
        __syncthreads();
        PHASE_MARK(PH_INTEGRATE);
        auto add = [&](int a, float3 f) {
            lds_add(&fa[a], fix_f(f.x));
            lds_add(&fa[n + a], fix_f(f.y));
            lds_add(&fa[2 * n + a], fix_f(f.z));
        };
        const PosLDS pos{L.xs};
        long long e = 0;
        for (int u = wv; u < u7; u += nwv) {
            if (u >= u0 && u < u1) {
                const int i = 16 * (u - u0) + (lane >> 2), q = lane & 3;
                const float4 pi = L.xs[i];
                const float2 ppi = L.pp[i];
                const unsigned long long m = L.am[64 * (u - u0) + lane];
                float fx = 0.f, fy = 0.f, fz = 0.f, ep = 0.f;
                if (energy) small_pairs<true>(pi, ppi, L.xs + q, L.pp + q, m, (n + 3) >> 2, rc2, krf2, krf, crf, fx, fy, fz, ep);
                else small_pairs<false>(pi, ppi, L.xs + q, L.pp + q, m, (n + 3) >> 2, rc2, krf2, krf, crf, fx, fy, fz, ep);
                fx = quad_sum(fx);
                fy = quad_sum(fy);
                fz = quad_sum(fz);
                if (energy) ep = quad_sum(ep);
                // one lane of the atom per component
                if (i < n && q < 3) lds_add(&fa[q * n + i], fix_f(q == 0 ? fx : (q == 1 ? fy : fz)));
                if (energy && i < n && q == 3) e += fix_f(ep);
            } else if (u < u0) {
                const int t = 64 * u + lane;
                if (t < nt) {
                    const uint2 w = L.ti[t];
                    const int i = w.x & 0xFFFF, j = w.x >> 16, k = w.y & 0xFFFF, l = w.y >> 16;
                    float3 fi, fj, fk, fl;
                    const float ut = term_torsion(pos(i), pos(j), pos(k), pos(l), L.tp[t], fi, fj, fk, fl);
                    add(i, fi);
                    add(j, fj);
                    add(k, fk);
                    add(l, fl);
                    e += fix_f(ut);
                }
            } else if (u < u2) {
                const int t = 64 * (u - u1) + lane;
                if (t < na) {
                    const uint2 w = L.ti[nt + t];
                    const float4 p = L.tp[nt + t];
                    const int i = w.x & 0xFFFF, j = w.x >> 16, k = w.y & 0xFFFF;
                    float3 fi, fk;
                    const float ut = term_angle(pos(i), pos(j), pos(k), make_float2(p.x, p.y), fi, fk);
                    add(i, fi);
                    add(k, fk);
                    add(j, make_float3(-fi.x - fk.x, -fi.y - fk.y, -fi.z - fk.z));
                    e += fix_f(ut);
                }
            } else if (u < u3) {
                // the next step's Gaussians, and the clearing of the forces just used
                const int a = 64 * (u - u2) + lane;
                if (a < n) {
                    f0[a] = f0[n + a] = f0[2 * n + a] = 0;
                    const float3 g = step_noise(ik, a, r, s0 + step + 1);
                    L.gn[a] = g.x; L.gn[n + a] = g.y; L.gn[2 * n + a] = g.z;
                    if (a == 0) eacc[cur ^ 1] = 0;
                }
            } else if (u < u4) {
                const int t = 64 * (u - u3) + lane;
                if (t < n14) {
                    const uint2 w = L.ti[nt + na + t];
                    float3 fi;
                    const float ut = term_pair14(pos(w.x & 0xFFFF), pos(w.x >> 16), L.tp[nt + na + t], fi);
                    add(w.x & 0xFFFF, fi);
                    add(w.x >> 16, neg3(fi));
                    e += fix_f(ut);
                }
            } else if (u < u5) {
                const int t = 64 * (u - u4) + lane;
                if (t < nb) {
                    const uint2 w = L.ti[nt + na + n14 + t];
                    const float4 p = L.tp[nt + na + n14 + t];
                    float3 fi;
                    const float ut = term_bond(pos(w.x & 0xFFFF), pos(w.x >> 16), make_float2(p.x, p.y), fi);
                    add(w.x & 0xFFFF, fi);
                    add(w.x >> 16, neg3(fi));
                    e += fix_f(ut);
                }
            } else if (u < u6) {
                const int t = 64 * (u - u5) + lane;
                if (t < nr) {
                    const int i = L.ti[nt + na + n14 + nb + t].x;
                    const float4 p = L.tp[nt + na + n14 + nb + t];
                    const float3 x = pos(i);
                    const float dx = x.x - p.x, dy = x.y - p.y, dz = x.z - p.z;
                    add(i, make_float3(-p.w * dx, -p.w * dy, -p.w * dz));
                    e += fix_f(0.5f * p.w * (dx * dx + dy * dy + dz * dz));
                }
            } else if (lane == 0) {
                float3 f = make_float3(0.f, 0.f, 0.f);
                e += fix_f(toy_force(L.xs[0].x, L.xs[0].y, f.x, f.y));
                fa[0] = fix_f(f.x);
                fa[n] = fix_f(f.y);
            }
        }
        if (energy) {
            e = wave_sum_ll(e);
            if (lane == 0 && e != 0) lds_add(&eacc[cur], e);
        }
        __syncthreads();
        PHASE_MARK(PH_FORCES);
        // the closing B: here when the step's velocities are read, else by the next integrator
        pend = !(samp || step + 1 == nsteps);
        if (!pend) {
            for (int k = tid; k < 3 * n; k += BT) {
                const float F = unfix_f(fa[k]);
                L.vs[k] = kick(L.vs[k], F, ik.h, L.im[k - ((k >= n) + (k >= 2 * n)) * n]);
                if (bad_force(F)) atomicOr(&errp[ERR_UNSTABLE], 1);
            }
        }
        if (samp) {
            // one wave per observable, its sums kept in LDS
            __syncthreads();
            for (int j = wv; j < S.nobs; j += nwv) {
                const double val = small_observable(S, L.ob[j], L, unfix_d(eacc[cur]), lane);
                if (lane == 0) {
                    const double xj = val - L.shift[j];
                    L.acc[2 * j] += xj;
                    const double x2 = xj * xj;
                    L.acc[2 * j + 1] += x2;
                }
            }
            __syncthreads();
        }
        PHASE_MARK(PH_TAIL);
        PHASE_COUNT(PH_NSTEP);
    }
    __syncthreads();
    const long long *const fl = L.fa + 3 * n * cur;
    for (int a = tid; a < n; a += BT) {
        gmut(S.x)[b + a] = L.xs[a].x; gmut(S.x)[b + np + a] = L.xs[a].y; gmut(S.x)[b + 2 * np + a] = L.xs[a].z;
        for (int d = 0; d < 3; ++d) {
            gmut(S.v)[b + d * np + a] = L.vs[d * n + a];
            gmut(S.F)[b + d * np + a] = fl[d * n + a];
        }
    }
    if (sample && r >= 1 && tid < 2 * S.nobs) S.acc[(size_t)r * 2 * MAX_OBS + tid] = L.acc[tid];
    if (S.cutoff_on && tid == 0 && nsteps > 0) S.need_build[r] = 1;
    if (state_end) {
        const int id = state_wg(S, PosLDS{L.xs}, L.red, &sbuf, tid, BT);
        if (tid == 0) S.state[r] = id;
    }
#ifdef GPR_PHASE_PROBE
    PHASE_MARK(PH_EPILOGUE);
    if (tid == 0 && r < PHASE_MAX_R) {
        unsigned long long *acc = gpr_phase_acc + (size_t)r * PHASE_MAX_G * NPHASE;
        for (int k = 0; k < PH_START; ++k) acc[k] += ph_acc[k];
        acc[PH_START] = ph_acc[PH_START];
        acc[PH_END] = __builtin_amdgcn_s_memrealtime();
    }
#endif
}

// One workgroup per replica (sp.G = 1): replica roff + blockIdx.x
__global__ void __launch_bounds__(1024) k_persist_small(PersistItem it)
{
    const int r = (int)blockIdx.x + it.roff;
    if (r >= it.nrep) return;
    long long s0 = it.s0;
    int t0 = it.t0;
    if (it.cyc && !cycle_start(it, s0, t0)) return;
    persist_small(*it.dev, r, s0, it.nsteps, t0, it.sample, it.state_end);
}

// the per-replica body as a function of its own (one call per replica and launch), so that
// the loop around it in k_persist_batch does not add to the body's register pressure.  The
// arguments of a call arrive in vector registers; they are wave-uniform, and made so again,
// so that the values and branches that depend on them stay scalar.
__device__ __noinline__ void persist_replica_call(const Dev *dev, int G, int lmax, int a0, int a1, int u0, int u1,
                                                  const uint2 *bi, const float4 *bp, int noise_ahead, int r, int g,
                                                  long long s0, int nsteps, int t0, int sample, int state_end)
{
    const Dev *d = (const Dev *)uni64((long long)dev);
    persist_replica(*d, uni(G), uni(lmax), uni(a0), uni(a1), uni(u0), uni(u1), (const uint2 *)uni64((long long)bi),
                    (const float4 *)uni64((long long)bp), uni(noise_ahead), uni(r), uni(g), uni64(s0), uni(nsteps), uni(t0), uni(sample),
                    uni(state_end));
}

// Several systems, each item's sets taking its replicas r = set, set + nsets, ... in turn.
__global__ void __launch_bounds__(1024) k_persist_batch(PersistBatch pb)
{
    int k = 0;
    const int b = start_place(pb.it[0].dev->ticket, pb.mapped);
    while (k + 1 < pb.nitems && b >= pb.it[k + 1].boff) ++k;
    const PersistItem &it = pb.it[k];
    int set, g;
    if (!persist_place(it, b - it.boff, set, g)) return;
    for (int r = set; r < it.nrep; r += it.nsets) {
        persist_replica_call(it.dev, it.sp.G, it.sp.lmax, it.sp.bnd[g], it.sp.bnd[g + 1], it.sp.bu[g], it.sp.bu[g + 1],
                             it.sp.bi, it.sp.bp, it.noise_ahead, r, g, it.s0, it.nsteps, it.t0, it.sample, it.state_end);
        __syncthreads();
    }
}


// ================================================================== Gen.ParRep bookkeeping
// Sums over workers follow one canonical pairwise tree: the m terms padded with zeros to the
// next power of two p, each node the sum of its lower half and its upper half.  A wave
// evaluates it with lane l holding the c = max(1, p / 64) consecutive terms [l c, l c + c):
// their subtree inside the lane, then xor shuffles at partner distances 1, 2, 4, ... over the
// lanes that hold terms, which form exactly the upper levels of the tree (the two lanes of a
// pair add the same two values in either order, with identical bits).
constexpr int TREE_C = 16;                 // terms per lane summed in registers

// subtree of the c (a power of two) terms f(base .. base + c), those >= m being zero
template <class Fn>
__device__ __forceinline__ double lane_tree16(Fn f, int m, int base, int c)
{
    double e[TREE_C];
#pragma unroll
    for (int i = 0; i < TREE_C; ++i) e[i] = (i < c && base + i < m) ? f(base + i) : 0.0;
#pragma unroll
    for (int w = 1; w < TREE_C; w <<= 1)
#pragma unroll
        for (int i = 0; i + w < TREE_C; i += 2 * w)
            if (w < c) e[i] += e[i + w];
    return e[0];
}

template <class Fn>
__device__ double lane_tree(Fn f, int m, int base, int c)
{
    if (c <= TREE_C) return lane_tree16(f, m, base, c);
    // more terms than registers: subtrees of TREE_C terms merged in order by a binary counter
    // (a new subtree is added to the pending one of its own height, lower half first)
    double stk[12];
    int lvl[12], sp = 0;
    for (int b = 0; b < c; b += TREE_C) {
        double v = lane_tree16(f, m, base + b, TREE_C);
        int L = 0;
        while (sp > 0 && lvl[sp - 1] == L) { v = stk[--sp] + v; ++L; }
        stk[sp] = v; lvl[sp] = L; ++sp;
    }
    return stk[0];
}

// the whole wave: the tree over f(0 .. m), in every lane that holds terms
template <class Fn>
__device__ double wave_pairwise(Fn f, int m)
{
    int p = 1;
    while (p < m) p <<= 1;
    const int lanes = p > 64 ? 64 : p, c = p > 64 ? p / 64 : 1;
    const int lane = threadIdx.x & 63;
    double v = lane < lanes ? lane_tree(f, m, lane * c, c) : 0.0;
    for (int o = 1; o < lanes; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Gelman-Rubin R-hat (Eq. 3) of one observable over nw workers from the shifted sums S1, S2
// of n samples; the whole wave calls it, the value is valid in lane 0
template <class F1, class F2>
__device__ double rhat_wave(int nw, long long n, F1 s1, F2 s2)
{
    const double dn = (double)n, dw = (double)nw;
    const double m1 = wave_pairwise([&](int k) { return s1(k) / dn; }, nw) / dw;
    const double m2 = wave_pairwise([&](int k) { return s2(k) / dn; }, nw) / dw;
    const double den = wave_pairwise([&](int k) {
        const double ob = s1(k) / dn;
        const double a = s2(k) / dn;
        const double o2 = ob * ob;
        return a - o2;
    }, nw) / dw;
    const double m1sq = m1 * m1;
    const double num = m2 - m1sq;
    return den > 0.0 ? num / den : __longlong_as_double(0x7FF0000000000000LL);
}

// Survivors of a check (Sec. 2.4.1): the workers r >= 1 not exited, ascending, into surv[];
// returns their number.  Block-collective (blockDim a multiple of 64); wsum: LDS int[16].
template <class Ex>
__device__ int survivors_block(int R, Ex exited, int *surv, int *wsum)
{
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wv = tid >> 6, nwv = nthr >> 6;
    int run = 0;
    for (int base = 1; base < R; base += nthr) {
        const int r = base + tid;
        const bool f = r < R && !exited(r);
        const unsigned long long m = __ballot(f);
        const int pre = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        if (lane == 0) wsum[wv] = __popcll(m);
        __syncthreads();
        int off = run, tot = 0;
        for (int k = 0; k < nwv; ++k) {
            off += k < wv ? wsum[k] : 0;
            tot += wsum[k];
        }
        if (f) surv[off + pre] = r;
        run += tot;
        __syncthreads();
    }
    return run;
}

// Fleming-Viot donor of worker r at the check of global step s (Sec. 2.4.1): -1 for a
// survivor, S[(u |S|) >> 32] for an exited worker (u the first Philox word of (0, s, r,
// stream 2), S the ascending survivors, ns = |S|), -2 for every worker when no worker
// survived; replica 0 (the reference walker) is never branched: -1, or -2 with no survivor.
template <class Ex>
__device__ __forceinline__ int fv_donor(uint32_t k0, uint32_t k1, long long s, int r, Ex exited, const int *surv, int ns)
{
    if (ns == 0) return -2;
    if (r == 0 || !exited(r)) return -1;
    const uint4 w = philox_ctr(0u, s, (uint32_t)r, STREAM_BRANCH, k0, k1);
    const unsigned long long pick = ((unsigned long long)w.x * (unsigned long long)ns) >> 32;
    return surv[pick];
}

// Exit vote of Eq. 5 on first-exit check indices (0: no exit): M = the smallest positive
// fec, k = 1 + the smallest r with fec[r] = M, tau = (R (M - 1) + k) t_check; (0, 0, 0) when
// no replica exited.  Block-collective; the result is valid in thread 0.  red: LDS long long[32].
template <class Fec>
__device__ void vote_block(int R, Fec fec, long long t_check, long long *red, long long *M, int *k, long long *tau)
{
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wv = tid >> 6, nwv = nthr >> 6;
    // key = (fec, r) ordered lexicographically; no exit is the largest key
    long long bf = 0x7FFFFFFFFFFFFFFFLL;
    int br = 0x7FFFFFFF;
    for (int r = tid; r < R; r += nthr) {
        const long long f = fec(r);
        if (f > 0 && (f < bf || (f == bf && r < br))) { bf = f; br = r; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const long long of = __shfl_xor(bf, o, 64);
        const int orr = __shfl_xor(br, o, 64);
        if (of < bf || (of == bf && orr < br)) { bf = of; br = orr; }
    }
    if (lane == 0) { red[2 * wv] = bf; red[2 * wv + 1] = br; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < nwv; ++w) {
            const long long of = red[2 * w];
            const int orr = (int)red[2 * w + 1];
            if (of < bf || (of == bf && orr < br)) { bf = of; br = orr; }
        }
        if (bf == 0x7FFFFFFFFFFFFFFFLL) { *M = 0; *k = 0; *tau = 0; }
        else { *M = bf; *k = br + 1; *tau = ((long long)R * (bf - 1) + (br + 1)) * t_check; }
    }
    __syncthreads();
}

// Per-check bookkeeping and Fleming-Viot clone-on-kill in one launch; blocks of 256
// threads, grid (nx, ny).  Block (0, 0) writes the status: CHK_STATE reports replica 0's
// state; CHK_DEPHASE takes the reference-exit test, the branching plan (donor[], surv[])
// and R-hat over the workers with the sums they hold after this check's branching;
// CHK_PARALLEL records the replicas outside Omega at check `check_index` and takes the exit
// vote of Eq. 5 (M, k, tau; to_state of replica k - 1); CHK_ADVANCE records first exit
// checks in fec[] and computes, but does not act on, the plan and R-hat.  With CHK_DEPHASE
// the blocks of row y = r (ny = R) copy (x, v, F) of replica r's donor into replica r when
// r was killed (a slice of nx blocks each), mark r for a pair-list rebuild and copy the
// donor's observable sums (cleared when every worker is re-copied from the reference).
__global__ void __launch_bounds__(256) k_check(const Dev *__restrict__ Sp, int mode, long long s, int omega, int nrep,
                                               long long nsamp, long long check_index, long long t_check, Status *st,
                                               int *donor, int *surv, long long *fec, int fec_fresh, long long *fec_out,
                                               CycRec *cyc, int cycle)
{
    const Dev &S = *Sp;
    const int tid = threadIdx.x;
    const int r = blockIdx.y;
    __shared__ int wsum[16];
    __shared__ long long red[32];
    __shared__ int sh_ne;
    __shared__ double rh_l[MAX_OBS];
    const int *state = S.state;
    auto ex = [&](int q) { return state[q] != omega; };
    const bool head = blockIdx.x == 0 && r == 0;
    long long t_now = 0;                                   // cycle mode: steps of the call at this check
    if (cyc) {
        // cycle `cycle` of a captured run: its step, check index and status slot; nothing after
        // the check that ended the call
        if (cyc->halt_cycle < cycle) return;
        omega = cyc->omega;
        const long long after = (long long)(cycle + 1) * cyc->nsteps;
        s = cyc->s_start + after;
        check_index = cyc->M_start + cycle + 1;
        t_now = cyc->t_start + after;
        st += cycle;
        if (head) nsamp = cyc->nsamp + (t_now / S.t_gr - (t_now - cyc->nsteps) / S.t_gr);
    }
    if (mode == CHK_DEPHASE) {
        if (state[0] != omega) {
            // the reference walker left Omega: nothing is branched
            if (head && tid == 0) {
                st->mode = mode; st->ref_exited = 1; st->n_exited = 0; st->n_surv = 0; st->k = 0;
                st->M = 0; st->tau = 0; st->to_state = state[0];
                for (int e = 0; e < 4; ++e) st->err[e] = S.err[e];
                for (int j = 0; j < MAX_OBS; ++j) st->rhat[j] = __longlong_as_double(0x7FF0000000000000LL);
                if (cyc) { cyc->nsamp = nsamp; cyc->halt_cycle = cycle; }
            }
            return;
        }
        if (!head && (r == 0 || !ex(r))) return;          // survivors are never copied
    } else if (!head) {
        return;
    }
    // survivors (every block that needs a donor): into the global list from block (0, 0),
    // into LDS elsewhere
    extern __shared__ __align__(16) unsigned char lds_raw[];
    int *sl = head ? surv : (int *)lds_raw;
    const int ns = survivors_block(nrep, ex, sl, wsum);
    if (!head) {
        // an exited worker: copy its donor (the reference walker when no worker survived)
        __syncthreads();
        const int d = ns == 0 ? 0 : fv_donor(S.key0, S.key1, s, r, ex, sl, ns);
        const size_t bs = (size_t)d * 3 * S.np, bd = (size_t)r * 3 * S.np;
        for (int k = blockIdx.x * blockDim.x + tid; k < 3 * S.np; k += gridDim.x * blockDim.x) {
            S.x[bd + k] = S.x[bs + k];
            S.v[bd + k] = S.v[bs + k];
            S.F[bd + k] = S.F[bs + k];
        }
        if (blockIdx.x == 0 && tid == 0) S.need_build[r] = 1;
        if (blockIdx.x == 0 && tid < 2 * MAX_OBS)
            S.acc[(size_t)r * 2 * MAX_OBS + tid] = d == 0 ? 0.0 : S.acc[(size_t)d * 2 * MAX_OBS + tid];
        return;
    }
    // block (0, 0): the plan, the status and R-hat
    if (tid == 0) { sh_ne = 0; }
    __syncthreads();
    int ne = 0;
    for (int q = tid; q < nrep; q += blockDim.x) {
        const int dq = fv_donor(S.key0, S.key1, s, q, ex, sl, ns);
        if (mode == CHK_DEPHASE || mode == CHK_ADVANCE) donor[q] = dq;
        ne += q > 0 && ex(q);
        if (mode == CHK_ADVANCE) {
            // the check of the first exit: from none at a call's first check (fec_fresh)
            long long f = fec_fresh ? 0 : fec[q];
            if (f == 0 && ex(q)) f = check_index;
            fec[q] = f;
            if (fec_out) fec_out[q] = f;
        }
    }
    for (int o = 32; o > 0; o >>= 1) ne += __shfl_xor(ne, o, 64);
    if ((tid & 63) == 0 && ne) atomicAdd(&sh_ne, ne);
    long long vM = 0, vtau = 0;
    int vk = 0;
    if (mode == CHK_PARALLEL)
        vote_block(nrep, [&](int q) { return ex(q) ? check_index : 0ll; }, t_check, red, &vM, &vk, &vtau);
    __syncthreads();
    if (tid == 0) {
        st->mode = mode;
        st->ref_exited = 0;
        st->n_exited = (mode == CHK_DEPHASE || mode == CHK_ADVANCE) ? sh_ne : 0;
        st->n_surv = (mode == CHK_DEPHASE || mode == CHK_ADVANCE) ? ns : 0;
        st->k = vk;
        st->M = vM;
        st->tau = vtau;
        st->to_state = state[vk > 0 ? vk - 1 : 0];
        for (int e = 0; e < 4; ++e) st->err[e] = S.err[e];
    }
    if (mode == CHK_DEPHASE || mode == CHK_ADVANCE) {
        // one wave per observable; after this check's branching a killed worker holds its
        // donor's sums, and with no survivor every worker restarts (R-hat undefined)
        const int wv = tid >> 6, nwv = blockDim.x >> 6;
        for (int j = wv; j < MAX_OBS; j += nwv) {
            double rh = __longlong_as_double(0x7FF0000000000000LL);
            const bool skip = (mode == CHK_DEPHASE && ns == 0) || nsamp < 1 || j >= S.nobs;
            if (!skip) {
                auto src = [&](int k) {
                    const int q = k + 1;
                    return (mode == CHK_DEPHASE && donor[q] >= 0) ? donor[q] : q;
                };
                auto s1 = [&](int k) { return S.acc[((size_t)src(k) * MAX_OBS + j) * 2]; };
                auto s2 = [&](int k) { return S.acc[((size_t)src(k) * MAX_OBS + j) * 2 + 1]; };
                rh = rhat_wave(nrep - 1, nsamp, s1, s2);
            }
            if ((tid & 63) == 0) { st->rhat[j] = rh; rh_l[j] = rh; }
        }
    }
    if (cyc) {
        // the decision the host takes from the status, taken here so that the later cycles of
        // the run know whether to run: converged (Eq. 4 test, with the samples restarted when
        // every worker was re-copied) or a first exit in the parallel step
        __syncthreads();
        if (tid == 0) {
            bool halt = false;
            if (mode == CHK_DEPHASE) {
                const long long nafter = (ns == 0 && nrep > 1) ? 0 : nsamp;
                bool conv = t_now >= S.t_min && nafter >= 2;
                for (int j = 0; j < S.nobs && conv; ++j) conv = rh_l[j] < 1.0 + S.tol;
                cyc->nsamp = nafter;
                halt = conv;
            } else if (mode == CHK_PARALLEL) {
                halt = vk > 0;
            }
            if (halt) cyc->halt_cycle = cycle;
        }
    }
}

// Copies (x, v, F) of replica donor[r] into replica r for every r with donor[r] >= 0 and
// marks r for a pair-list rebuild; observable sums are copied too (acc_mode 1), or cleared
// when the donor is the reference walker (a fresh broadcast).
__global__ void __launch_bounds__(256) k_clone(const Dev *__restrict__ Sp, const int *donor, int acc_mode)
{
    const Dev &S = *Sp;
    const int r = blockIdx.y;
    const int d = donor[r];
    if (d < 0 || d == r) return;
    const size_t bs = (size_t)d * 3 * S.np, bd = (size_t)r * 3 * S.np;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < 3 * S.np; k += gridDim.x * blockDim.x) {
        S.x[bd + k] = S.x[bs + k];
        S.v[bd + k] = S.v[bs + k];
        S.F[bd + k] = S.F[bs + k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) S.need_build[r] = 1;
    if (acc_mode && blockIdx.x == 0 && threadIdx.x < 2 * MAX_OBS) {
        S.acc[(size_t)r * 2 * MAX_OBS + threadIdx.x] = d == 0 ? 0.0 : S.acc[(size_t)d * 2 * MAX_OBS + threadIdx.x];
    }
}

// Maxwell-Boltzmann velocities of replica 0 (stream 1, step 0)
__global__ void __launch_bounds__(256) k_init_vel(const Dev *__restrict__ Sp, float kT)
{
    const Dev &S = *Sp;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= S.n) return;
    const float3 g = gauss3(philox_ctr((uint32_t)a, 0, 0u, STREAM_INIT, S.key0, S.key1));
    const float sdev = sqrtf(kT * S.prm[a].w);
    S.v[a] = sdev * g.x;
    S.v[S.np + a] = sdev * g.y;
    S.v[2 * S.np + a] = S.kind == KIND_TOY ? 0.0f : sdev * g.z;
}

// ------------------------------------------------------------------ building blocks
__global__ void __launch_bounds__(256) k_noise_test(uint32_t k0, uint32_t k1, int replica, long long step, int stream,
                                                    int n, uint32_t *words, float *gauss)
{
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n) return;
    const uint4 w = philox_ctr((uint32_t)a, step, (uint32_t)replica, (uint32_t)stream, k0, k1);
    const float3 g = gauss3(w);
    words[4 * a] = w.x; words[4 * a + 1] = w.y; words[4 * a + 2] = w.z; words[4 * a + 3] = w.w;
    gauss[3 * a] = g.x; gauss[3 * a + 1] = g.y; gauss[3 * a + 2] = g.z;
}

// the branching plan of one check, by the routines k_check runs (one block of 256 threads)
__global__ void __launch_bounds__(256) k_fvplan_test(uint32_t k0, uint32_t k1, long long s, int R, const uint8_t *exited,
                                                     int *donor, int *surv)
{
    __shared__ int wsum[16];
    auto ex = [&](int r) { return exited[r] != 0; };
    const int ns = survivors_block(R, ex, surv, wsum);
    for (int r = threadIdx.x; r < R; r += blockDim.x) donor[r] = fv_donor(k0, k1, s, r, ex, surv, ns);
}

// R-hat of observable blockIdx.x, by the routine k_check runs (one wave per observable)
__global__ void __launch_bounds__(64) k_rhat_test(int nw, int nobs, long long n, const double *S1, const double *S2,
                                                  double *out)
{
    const int j = blockIdx.x;
    auto s1 = [&](int k) { return S1[(size_t)k * nobs + j]; };
    auto s2 = [&](int k) { return S2[(size_t)k * nobs + j]; };
    const double rh = rhat_wave(nw, n, s1, s2);
    if (threadIdx.x == 0) out[j] = rh;
}

// the exit vote of Eq. 5, by the routine k_check runs (one block of 256 threads)
__global__ void __launch_bounds__(256) k_vote_test(int R, const long long *fec, long long t_check, long long *out)
{
    __shared__ long long red[32];
    long long M, tau;
    int k;
    vote_block(R, [&](int r) { return fec[r]; }, t_check, red, &M, &k, &tau);
    if (threadIdx.x == 0) { out[0] = M; out[1] = k; out[2] = tau; }
}

} // namespace gpr
