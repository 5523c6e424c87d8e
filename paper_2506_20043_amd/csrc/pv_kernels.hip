// pv_kernels.hip -- gfx950 kernels of the docking hot path.
//
//  * grid maps ("Kernel 1" of the paper: one map per ligand atom type over
//    each pocket box, Methods "Accelerated Docking" and Supplementary
//    Algorithm 2, first step): FP32 VALU, lattice tiles of 16x4x4 points per
//    workgroup and 4x4x4 per wave, receptor atoms culled for both;
//  * pose evaluation (Eq. qvina_eq_1 forward kinematics, Eq. qvina_eq_3
//    score): one wave64 per pose, lanes over fragments for the frame tree,
//    over atoms for the trilinear gathers and over intra pairs, LDS force
//    accumulation and a wave scan that carries force and torque back to the
//    torsions;
//  * RILC-BFGS (Eqs. qvina_eq_6 .. qvina_eq_12) with the tangent-space
//    vectors spread one component per lane;
//  * Monte Carlo chains (Supplementary Algorithm 2, Eq. qvina_eq_13) in a
//    persistent launch whose waves pull (job, chain) items from a device
//    queue, with Philox4x64-10 draws.
//
// A chain, a pose and a minimisation are one wave of 64 lanes (a chain may have
// helper waves); the output stage, the maps and the surface points use workgroups
// of several.  Arithmetic is binary32, but for the maps' cutoff where binary32
// rounding could decide it (within_cutoff_f64).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "pv_internal.h"

namespace pv {

// Vina-form weights: gauss1, gauss2, repulsion, hydrophobic, hydrogen bond.
constexpr float kW1 = -0.0356f, kW2 = -0.00516f, kW3 = 0.840f, kW4 = -0.0351f, kW5 = -0.587f;
constexpr float kCut2 = 64.0f;
constexpr float kPi = 3.14159265358979323846f;

// ---------------------------------------------------------------- wave helpers
// Cross-lane sums use DPP row permutations inside each 16-lane row and
// readlane across rows: a few VALU cycles instead of LDS round trips, and
// every lane ends with bit-identical results (the control flow that depends
// on them stays uniform).
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp0(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

__device__ __forceinline__ float lane_f(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// lane `src4 / 4`'s value
__device__ __forceinline__ float from_lane(int src4, float v)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src4, __float_as_int(v)));
}

__device__ __forceinline__ int lane_i(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

// v plus lane 15 of the row before, in rows 1 and 3, then lane 31's in rows 2
// and 3; the other rows keep theirs.  One instruction each (the compiler makes
// three: it does not fold an addition into a permutation of some rows).  A
// permutation may read a register two wait states after it was written.
__device__ __forceinline__ float add_row_before(float v)
{
    asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf" : "+v"(v));
    return v;
}
__device__ __forceinline__ float add_rows_before(float v)
{
    asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf" : "+v"(v));
    return v;
}

// sum over the 64 lanes, identical in every lane
__device__ __forceinline__ float wsum(float v)
{
    v += dpp0<0xB1>(v);   // quad_perm(1,0,3,2): lane ^ 1
    v += dpp0<0x4E>(v);   // quad_perm(2,3,0,1): lane ^ 2
    v += dpp0<0x141>(v);  // row_half_mirror: the other quad of each 8 lanes
    v += dpp0<0x140>(v);  // row_mirror: the other half of each row
    // the rows' sums: (row 0 + row 1) + (row 2 + row 3) ends in lane 63
    return lane_f(add_rows_before(add_row_before(v)), 63);
}

// sum over lanes 0..n-1 of a b, where every lane from n up holds zero (n is
// wave-uniform): rows past the last non-zero one are not read.  A lane's own
// product is fused onto its neighbour's rounded one.
__device__ __forceinline__ float wdot_n(float a, float b, int n)
{
    float v = fmaf(a, b, dpp0<0xB1>(a * b));
    v += dpp0<0x4E>(v);
    v += dpp0<0x141>(v);
    v += dpp0<0x140>(v);
    if (n <= 16) return lane_f(v, 0);
    v = add_row_before(v);
    if (n <= 32) return lane_f(v, 31);
    return lane_f(add_rows_before(v), 63);
}

// integer sum over the 64 lanes, identical in every lane
__device__ __forceinline__ int64_t wsum_i64(int64_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// inclusive prefix sums of six values over the 64 lanes in lane order (side by
// side, so that their cross-row steps need no wait states between them)
__device__ __forceinline__ void wscan6(float v[6])
{
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] += dpp0<0x111>(v[c]);   // row_shr:1
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] += dpp0<0x112>(v[c]);   // row_shr:2
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] += dpp0<0x114>(v[c]);   // row_shr:4
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] += dpp0<0x118>(v[c]);   // row_shr:8
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_add_f32_dpp %5, %5, %5 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_add_f32_dpp %5, %5, %5 row_bcast:31 row_mask:0xc bank_mask:0xf"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]));
}

// the lane within the wave for the one-wave workgroups of the docking kernels
// (multi-wave kernels take threadIdx.x & (kWave - 1))
__device__ __forceinline__ int lane_id() { return threadIdx.x; }

// Synchronisation of a one-wave workgroup.  The LDS executes the requests of
// one wave in order, so ordering the compiler is enough: no wait for
// outstanding global loads (which may stay in flight across it).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}


// Orders LDS accesses between the waves of a workgroup; every wave that has not
// ended takes part.
__device__ __forceinline__ void team_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// ---------------------------------------------------------------- Philox4x64-10
__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) { k0 += W0; k1 += W1; }
        uint64_t h0 = __umul64hi(M0, c[0]), l0 = M0 * c[0];
        uint64_t h1 = __umul64hi(M1, c[2]), l1 = M1 * c[2];
        uint64_t n0 = h1 ^ c[1] ^ k0, n2 = h0 ^ c[3] ^ k1;
        c[0] = n0; c[1] = l1; c[2] = n2; c[3] = l0;
    }
}

__device__ __forceinline__ float u01(uint64_t w) { return (float)(uint32_t)(w >> 40) * 0x1p-24f; }

// counter = (block, step, chain, job), key = (seed, 0)
__device__ __forceinline__ uint64_t philox_word(uint64_t seed, int job, int chain, uint64_t step,
                                                uint64_t block, int word)
{
    uint64_t c[4] = {block, step, (uint64_t)chain, (uint64_t)job};
    philox4x64_10(c, seed, 0);
    return word == 0 ? c[0] : word == 1 ? c[1] : word == 2 ? c[2] : c[3];
}

// ---------------------------------------------------------------- small rotations
__device__ __forceinline__ void quat_mul(const float a[4], const float b[4], float o[4])
{
    float r0 = a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3];
    float r1 = a[0] * b[1] + a[1] * b[0] + a[2] * b[3] - a[3] * b[2];
    float r2 = a[0] * b[2] - a[1] * b[3] + a[2] * b[0] + a[3] * b[1];
    float r3 = a[0] * b[3] + a[1] * b[2] - a[2] * b[1] + a[3] * b[0];
    o[0] = r0; o[1] = r1; o[2] = r2; o[3] = r3;
}

__device__ __forceinline__ void rotvec_quat(float tx, float ty, float tz, float q[4])
{
    // (cos(a/2), sin(a/2)/a * theta); sin(a/2)/a -> 1/2 as a -> 0.  One
    // v_rsq gives both a = a^2 / a and 1 / a (hardware, ~1 ulp).
    const float a2 = tx * tx + ty * ty + tz * tz;
    const float inv = __builtin_amdgcn_rsqf(fmaxf(a2, 1e-30f));
    const float a = a2 * inv;
    float s, c;
    __sincosf(0.5f * a, &s, &c);
    const float k = a2 > 1e-30f ? s * inv : 0.5f;
    q[0] = c; q[1] = k * tx; q[2] = k * ty; q[3] = k * tz;
}

__device__ __forceinline__ void quat_normalize(float q[4])
{
    const float n = __builtin_amdgcn_rsqf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    q[0] *= n; q[1] *= n; q[2] *= n; q[3] *= n;
}

// ---------------------------------------------------------------- per-box grid view
struct BoxView {
    const float* maps;  // 8 maps of the box
    int nx, ny, nz;
    int64_t msz;
    float ox, oy, oz, h, inv_h, ex, ey, ez, kappa;
};

__device__ __forceinline__ BoxView box_view(const GridDev& g, int box)
{
    BoxView v;
    v.maps = g.maps + g.map_off[box];
    v.nx = g.dims[4 * box]; v.ny = g.dims[4 * box + 1]; v.nz = g.dims[4 * box + 2];
    v.msz = (int64_t)v.nx * v.ny * v.nz;
    const float* ge = g.geom + 8 * box;
    v.ox = ge[0]; v.oy = ge[1]; v.oz = ge[2]; v.h = ge[3]; v.inv_h = ge[4];
    v.ex = ge[5]; v.ey = ge[6]; v.ez = ge[7];
    v.kappa = g.kappa;
    return v;
}

// Values that are the same in every lane, moved to scalar registers: what a kernel
// loads after it has stored anything comes by vector loads (the compiler cannot
// tell that the tables did not change), so a box's and a ligand's numbers would
// hold some thirty vector registers for a chain's whole life.
__device__ __forceinline__ void to_scalar(int& v) { v = __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ void to_scalar(float& v)
{
    v = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
template <typename P>
__device__ __forceinline__ void to_scalar(const P*& p)
{
    const uint64_t v = (uint64_t)p;
    int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    to_scalar(lo);
    to_scalar(hi);
    p = (const P*)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}

__device__ __forceinline__ void to_scalar(BoxView& v)
{
    to_scalar(v.maps);
    to_scalar(v.nx); to_scalar(v.ny); to_scalar(v.nz);
    v.msz = (int64_t)v.nx * v.ny * v.nz;
    to_scalar(v.ox); to_scalar(v.oy); to_scalar(v.oz); to_scalar(v.h); to_scalar(v.inv_h);
    to_scalar(v.ex); to_scalar(v.ey); to_scalar(v.ez);
}

// One axis of the lookup: fractional coordinate clamped to [0, n-1], cell
// i0 = min(floor f, n-2), the out-of-box penalty and whether the axis is
// clamped (its interpolant gradient is then zero).
__device__ __forceinline__ void axis_setup(float x, float o, float inv_h, float ext, int n, float kappa,
                                           int& i0, float& u, float& pen, float& dpen, bool& clamped)
{
    // no branches: at most one side is out (ext >= 0), so the penalty is the
    // sum of both sides' excess; a NaN coordinate is on neither side and
    // keeps its NaN in f
    const float rel = x - o;
    const bool lo = x < o, hi = rel > ext;
    pen = kappa * (fmaxf(o - x, 0.f) + fmaxf(rel - ext, 0.f));
    dpen = lo ? -kappa : (hi ? kappa : 0.f);
    const float f = lo ? 0.f : (hi ? (float)(n - 1) : rel * inv_h);
    clamped = lo || hi;
    int c = (int)floorf(f);
    c = max(0, min(c, n - 2));  // also keeps a NaN coordinate inside the map
    i0 = c;
    u = f - (float)c;
}

// Trilinear lookup in two halves: tri_issue computes the cell and starts the
// 8 corner loads; tri_finish interpolates (value, gradient, penalty) once
// they are needed, so other work can hide the memory latency in between.
struct TriLoad {
    float m[8];
    float ux, uy, uz, pen, dx, dy, dz;
    bool cx, cy, cz;
};

__device__ __forceinline__ void tri_issue(const BoxView& B, int t, float x, float y, float z, TriLoad& L)
{
    int ix, iy, iz;
    float px, py, pz;
    axis_setup(x, B.ox, B.inv_h, B.ex, B.nx, B.kappa, ix, L.ux, px, L.dx, L.cx);
    axis_setup(y, B.oy, B.inv_h, B.ey, B.ny, B.kappa, iy, L.uy, py, L.dy, L.cy);
    axis_setup(z, B.oz, B.inv_h, B.ez, B.nz, B.kappa, iz, L.uz, pz, L.dz, L.cz);
    L.pen = px + py + pz;
    // a box's 8 maps hold fewer than 8 x 2^24 points (checked when the grids
    // are built), so the corner offsets are 32-bit byte offsets from the
    // maps' base, formed with 24-bit multiplies
    const uint32_t nx = (uint32_t)B.nx, ny = (uint32_t)B.ny;
    const uint32_t e = __umul24((uint32_t)t, (uint32_t)B.msz) + __umul24(__umul24((uint32_t)iz, ny) + (uint32_t)iy, nx) +
                       (uint32_t)ix;
    const uint32_t o0 = e << 2, oy = nx << 2, oz = __umul24(nx, ny) << 2;
    const char* mb = (const char*)B.maps;
    const float* r0 = (const float*)(mb + o0);
    const float* r1 = (const float*)(mb + (o0 + oy));
    const float* r2 = (const float*)(mb + (o0 + oz));
    const float* r3 = (const float*)(mb + (o0 + oz + oy));
    L.m[0] = r0[0]; L.m[1] = r0[1];
    L.m[2] = r1[0]; L.m[3] = r1[1];
    L.m[4] = r2[0]; L.m[5] = r2[1];
    L.m[6] = r3[0]; L.m[7] = r3[1];
}

__device__ __forceinline__ float tri_finish(const BoxView& B, const TriLoad& L, float& gx, float& gy, float& gz)
{
    const float m000 = L.m[0], m100 = L.m[1], m010 = L.m[2], m110 = L.m[3];
    const float m001 = L.m[4], m101 = L.m[5], m011 = L.m[6], m111 = L.m[7];
    const float ux = L.ux, uy = L.uy, uz = L.uz;
    float a00 = m000 + ux * (m100 - m000), a10 = m010 + ux * (m110 - m010);
    float a01 = m001 + ux * (m101 - m001), a11 = m011 + ux * (m111 - m011);
    float b0 = a00 + uy * (a10 - a00), b1 = a01 + uy * (a11 - a01);
    float v = b0 + uz * (b1 - b0);
    // derivatives of the interpolant in the cell
    float d00 = m100 - m000, d10 = m110 - m010, d01 = m101 - m001, d11 = m111 - m011;
    float e0 = d00 + uy * (d10 - d00), e1 = d01 + uy * (d11 - d01);
    float dvx = e0 + uz * (e1 - e0);
    float dvy = (a10 - a00) + uz * ((a11 - a01) - (a10 - a00));
    float dvz = b1 - b0;
    gx = (L.cx ? 0.f : dvx * B.inv_h) + L.dx;
    gy = (L.cy ? 0.f : dvy * B.inv_h) + L.dy;
    gz = (L.cz ? 0.f : dvz * B.inv_h) + L.dz;
    return v + L.pen;
}

// trilinear value + gradient of map `t` at x, plus the penalty
__device__ __forceinline__ float trilinear(const BoxView& B, int t, float x, float y, float z, float& gx,
                                           float& gy, float& gz)
{
    TriLoad L;
    tri_issue(B, t, x, y, z, L);
    return tri_finish(B, L, gx, gy, gz);
}

// ---------------------------------------------------------------- LDS carving
// A pose [t(3), q(4), psi(T)] has up to 39 entries and lives in a register,
// entry l in lane l: a chain alone on its SIMD spends a third of its time
// waiting, mostly for LDS, and every step of a pose through LDS (stored, copied
// between slots, read back entry by entry) was such a wait.  With the poses in
// registers, frames composed in place and the tail passes of the slot form: one
// ligand's dock (8 chains) 27.9 -> 25.4 ms, a screening slice 414 -> 402 ms, the
// local optimisation of 16,384 poses 3.31 -> 3.22 ms, and the searches the same
// bit for bit.
constexpr int kSlot = 40;

struct Lds {
    char* base;        // start of the wave's LDS
    uint32_t pos0;     // LDS byte address of pos
    float* frame;      // [kMaxFrag][12] frames (where a kernel keeps them)
    float4* pos;       // [ma + 1]; entry ma: a point far outside every box
    float4* frc;       // [max_atoms] dE/dx per atom, or NULL when nothing reads it back
    float* pre;        // [6][max_atoms]
    float4* map;       // with helper waves: [ma] map force per atom,
    uint32_t* count;   //   [helpers][64] the lanes' pairs inside the cutoff | an atom outside << 31,
    float* part;       //   [their chunks][64] the pairs' energies,
    float* e_map;      //   [1] the map energy,
    int* done;         //   [1] the chain has ended
    uint4* pairs;      // [max_pairs rounded up to kPairPass] pair records, slot layout (see stage_ligand)
    float* cp;         // [max_pairs rounded up to kWave] per-pair force coefficient, gather layout
    uint32_t* pw;      // [max_pairs rounded up to kWave] pair words, gather layout (see stage_ligand)
    float4* fs;        // [max_ell + 1] pair forces in slot rows of n | 1 atoms (slot-major), then one
                       // write-only slot for the padding records, slot layout
    int ma;
};

// LDS byte address of a pointer into LDS, and back.
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ uint32_t lds_addr(const void* p)
{
    return (uint32_t)(uintptr_t)(const lds_char*)p;
}
template <typename V>
__device__ __forceinline__ __attribute__((address_space(3))) V* lds_ptr(uint32_t a)
{
    return (__attribute__((address_space(3))) V*)(uintptr_t)a;
}

// Pairs per pass of the pair loop (lanes x pairs per lane); the LDS pair
// records are padded to a multiple of it.
constexpr int kPairUnroll = 4;
constexpr int kPairPass = kPairUnroll * kWave;

__host__ __device__ inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

// Atom entries of the per-wave atom arrays (a multiple of 4 keeps every
// region 16-byte aligned).
__host__ __device__ inline int lds_atoms(int max_atoms) { return round_up(max_atoms < 1 ? 1 : max_atoms, 4); }

// Two layouts of the intra-force tables.  Slots (ligands of at most 64
// atoms, one atom per lane): the pair list sits in LDS, packed with the slots
// each pair owns in its two atoms' rows, beside the per-slot pair forces, so
// an atom's intra force is a stream of independent LDS reads.  Gather: the
// pair words and the per-pair coefficients live in LDS and the atom -> pair
// table is read from global memory (a small footprint, for large ligands or
// launches that need many resident waves).
//
// Optional regions: the per-atom forces (read back only by the score
// kernel's coordinate gradient) and the fragment frames (needed when atoms
// take their frames from LDS: two atoms per lane, and the output stage's
// pose positions; with one atom per lane the frames travel by ds_bpermute,
// as the torsion derivatives do, and the area is only kept for its size, see
// kLdsSpare).
struct LdsNeeds {
    bool slots, frc, frames;
    bool pw;   // gather layout: the pair words in LDS too (one atom per lane), else read from global memory
    bool lean; // nothing but what the kernel uses (three waves per SIMD, see kLean)
};

// Bytes that no region uses.  They keep the sizes, and with them the choice
// between the two layouts (launch_shape), what they were when the poses were
// held here: the layouts sum forces in another order, so another choice would
// change the searches' last bits.
constexpr int kLdsSpare = 5 * kSlot * 4;

__host__ __device__ inline int lds_bytes(int max_atoms, int max_pairs, int max_ell, LdsNeeds nd)
{
    const int ma = lds_atoms(max_atoms);
    int b = (nd.lean ? 0 : kLdsSpare) + (ma + 1) * 16 + 6 * ma * 4;
    b += nd.frames ? kMaxFrag * 13 * 4 + 12 : nd.lean ? 0 : round_up(kMaxFrag, 4) * 4;
    if (nd.frc) b += ma * 16;
    if (nd.slots) b += round_up(max_pairs < 1 ? 1 : max_pairs, kPairPass) * 16 + (max_ell + 1) * 16;
    else b += (nd.pw ? 2 : 1) * round_up(max_pairs + 1, kWave) * 4;
    return b;
}

__device__ __forceinline__ Lds carve(char* base, int max_atoms, int max_pairs, int max_ell, LdsNeeds nd)
{
    Lds s;
    const int ma = lds_atoms(max_atoms);
    char* p = base;
    s.base = base;
    s.pos0 = 0;   // the kernels have no static LDS, so the dynamic LDS starts at address 0
    s.pos = (float4*)p; p += (ma + 1) * 16;
    s.pre = (float*)p; p += 6 * ma * 4;
    s.frc = nullptr;
    if (nd.frc) { s.frc = (float4*)p; p += ma * 16; }
    s.frame = (float*)p; p += nd.frames ? kMaxFrag * 13 * 4 + 12 : nd.lean ? 0 : round_up(kMaxFrag, 4) * 4;
    s.pairs = nullptr; s.fs = nullptr; s.cp = nullptr; s.pw = nullptr;
    if (nd.slots) {
        s.pairs = (uint4*)p; p += round_up(max_pairs < 1 ? 1 : max_pairs, kPairPass) * 16;
        s.fs = (float4*)p;
    } else {
        const int pp = round_up(max_pairs + 1, kWave);
        s.cp = (float*)p; p += pp * 4;
        if (nd.pw) s.pw = (uint32_t*)p;
    }
    s.ma = ma;
    return s;
}

// A chain is one wave's serial work, and a launch of few chains leaves most SIMDs
// idle while its longest runs on.  Such a launch gives every chain a team of W
// waves: its own and W - 1 helpers, which wait at a barrier for an evaluation's
// atom positions; the last one looks the maps up, and the chunks of 64 pairs are
// shared out.  Energies cross per pair and are added in the order of the list,
// so the searches stay the same bit for bit.  At most 168 VGPRs, so that a CU
// holds three teams of four or six of two.
//
// First of the nc chunks of wave w of a team (of wave W: nc): the map lookup is
// worth about three chunks (five pockets, 445 pairs, teams of two: own wave four
// of seven chunks 152 ms, five 142, six 145; one wave 165 ms).
template <int W>
__host__ __device__ inline int team_chunk(int nc, int w)
{
    if constexpr (W <= 1) return w * nc;
    else {
        const int last = nc > 3 * (W - 1) ? (nc - 3 * (W - 1)) / W : 0, rest = nc - last;
        return w == W ? nc : (rest * w + W - 2) / (W - 1);
    }
}

// The helpers' results in LDS, after the regions of carve.
template <int W>
__host__ __device__ inline int team_bytes(int max_atoms, int max_pairs)
{
    const int nc = (max_pairs + kWave - 1) / kWave;
    return lds_atoms(max_atoms) * 16 + (W - 1) * kWave * 4 + 16 + (nc - team_chunk<W>(nc, 1)) * kWave * 4;
}

template <int W>
__device__ __forceinline__ void carve_team(Lds& s, char* p, int max_atoms)
{
    s.map = (float4*)p; p += lds_atoms(max_atoms) * 16;
    s.count = (uint32_t*)p; p += (W - 1) * kWave * 4;
    s.done = (int*)p;
    s.e_map = (float*)p + 1;
    p += 16;
    s.part = (float*)p;
}

// The regions a kernel's LDS holds: per-atom forces for the score kernel's
// coordinate gradient; frames for two atoms per lane and the output stage;
// the pair words for one atom per lane on the gather layout (with two atoms
// per lane the pair lists are long and the words stay in global memory, so
// that LDS does not cut the resident waves).
constexpr int kKindOutput = 3;
__host__ __device__ inline LdsNeeds kernel_needs(int kind, int A, bool slots, bool lean = false)
{
    return LdsNeeds{slots, kind == kKindScore, A > 1 || kind == kKindOutput, !slots && A == 1, lean};
}

// Team size (template argument W) 0: one wave per chain, built for three waves per
// SIMD.  The gather form with one atom per lane holds about 230 VGPRs, two waves,
// and these keep the vector units 65% busy; with the map lookups ended before
// the pair loop, the uniform numbers in scalar registers and the rest spilled (20
// to 40 registers, in the code around the evaluations) it fits 168.  16,384 poses
// of local optimisation 3.14 -> 2.59 ms; screens of 8-40 atoms 494 -> 406 ms, of
// 30-50 atoms 392 -> 326 ms.  Used where a launch has more waves than two per
// SIMD and the LDS holds twelve per CU: with nine (ligands of up to 64 atoms) a
// screen took 5% longer, and with the pair words left in global memory to make
// room for twelve 20% (the optimisation 2.80 ms).
constexpr int kLean = 0;

// Least value over all surface distances of a pair's energy, by class (the
// Vina terms above: plain at d = 0.003, hydrophobic at d = 0.003, hydrogen
// bond at d = -0.466), rounded down in the fourth digit.
constexpr float kPairMin0 = -0.03615f, kPairMin1 = -0.07125f, kPairMin2 = -0.22356f;

float least_pair_energy(uint32_t cls) { return cls == 0 ? kPairMin0 : (cls == 1 ? kPairMin1 : kPairMin2); }

// ---------------------------------------------------------------- staged ligand
// Topology lives in registers: atoms blocked A per lane (atom = lane*A + a),
// fragments one per lane, and for lane 6+k the fragment of torsion k.
template <int A, bool SL>
struct Topo {
    int n, nf, nt, np, rounds, lig, ell_w, fs_stride;
    float rot_scale;
    float4 ref[A];
    int psi_src;      // 4 x the lane of this fragment lane's torsion angle in the pose
    int f_child, f_a0, f_end;
    uint32_t link0, link1;   // 4 x the lane of the ancestor a fragment lane composes with in each
                             // pointer-doubling round (itself: none), a byte per round: rounds 0..3, 4..5
    float ax, ay, az; // unit axis of the fragment's torsion
    float cx, cy, cz; // a point of that axis (the child atom's reference position); the root: its anchor
    int dof_src;      // 4 x the fragment lane of this tangent lane's torsion
    int np0, np1;     // pairs below np0 are plain, below np1 hydrophobic, the rest hydrogen bonds
    float lb;   // a lower bound of the intra energy: the sum over the pairs of their class's least pair energy
    const uint32_t* gpairs;   // pair list and atom -> pair table in global
    const uint32_t* gell;     // memory (read from there when A > 1)
};

template <int A, bool SL>
__device__ __forceinline__ void to_scalar(Topo<A, SL>& T)
{
    to_scalar(T.n); to_scalar(T.nf); to_scalar(T.nt); to_scalar(T.np); to_scalar(T.rounds); to_scalar(T.ell_w);
    T.fs_stride = T.n | 1;
    to_scalar(T.rot_scale); to_scalar(T.lb); to_scalar(T.np0); to_scalar(T.np1);
    to_scalar(T.gpairs); to_scalar(T.gell);
}

template <int A, bool SL>
__device__ void stage_ligand(Topo<A, SL>& T, const LigDev& L, int lig, const Lds& S, bool fill = true)
{
    const int l = lane_id();
    const DevLig d = L.ligs[lig];
    T.lig = lig;
    T.n = d.n_atoms; T.nf = d.n_frag; T.nt = d.n_tors; T.np = d.n_pairs; T.rounds = d.rounds;
    T.ell_w = d.ell_w;
    // slot rows of an odd number of float4 (one per atom): the row reads of
    // the gather are contiguous, and the slots of one atom fall in different
    // LDS banks
    T.fs_stride = T.n | 1;
    T.rot_scale = d.rot_amp_scale;
#pragma unroll
    for (int a = 0; a < A; ++a) {
        int i = l * A + a;
        T.ref[a] = i < T.n ? L.atoms[d.atom_base + i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    int parent = -1;
    T.psi_src = 0; T.f_child = 0; T.f_a0 = 0; T.f_end = 0;
    T.ax = T.ay = T.az = T.cx = T.cy = T.cz = 0.f;
    if (l < T.nf) {
        const DevFrag F = L.frags[d.frag_base + l];
        parent = F.parent;
        T.psi_src = 4 * (7 + max(F.tors, 0)); T.f_child = F.child_atom; T.f_a0 = F.a0; T.f_end = F.sub_end;
        T.ax = F.axis[0]; T.ay = F.axis[1]; T.az = F.axis[2];
        T.cx = l == 0 ? d.anchor[0] : F.xc[0];
        T.cy = l == 0 ? d.anchor[1] : F.xc[1];
        T.cz = l == 0 ? d.anchor[2] : F.xc[2];
    }
    T.dof_src = (l >= 6 && l < 6 + T.nt) ? 4 * (int)L.tors_frag[d.tors_base + l - 6] : 0;
    {
        // the links do not depend on the pose: jumped once here (a lane
        // with an ancestor takes that ancestor's link after each round)
        static_assert(kMaxFrag <= 63, "a link holds 4 x a fragment lane in a byte");
        int anc = (l >= 1 && l < T.nf) ? parent : -1;
        T.link0 = T.link1 = 0;
        for (int r = 0; r < T.rounds; ++r) {
            const uint32_t src = (uint32_t)(4 * (anc >= 0 ? anc : l)) << (8 * (r & 3));
            if (r < 4) T.link0 |= src;
            else T.link1 |= src;
            const int panc = __builtin_amdgcn_ds_bpermute((anc >= 0 ? anc : l) << 2, anc);
            if (anc >= 0) anc = panc;
        }
    }
    T.gpairs = L.pairs + d.pair_base;
    T.gell = L.ell + d.ell_base;
    T.np0 = d.n_plain; T.np1 = d.n_hyd; T.lb = d.intra_lb;
    if (!fill) return;
    if (l == 0) S.pos[S.ma] = make_float4(1e18f, 1e18f, 1e18f, 0.f);
    if (SL) {
        // Pair record, everything the pair loop needs without decoding:
        //   x: LDS byte addresses of both positions (i | j << 16; S.pos opens
        //      the LDS, so both fit)
        //   y, z: LDS byte addresses of the pair's force slots in the rows of
        //         i and of j (slot * row stride + atom)
        //   w: the radius sum 3.4 + 0.1 rk (bits)
        // Records past the last pair fill the final pass: their first atom is
        // the far point, so they fall outside the cutoff, and both their
        // slots are the write-only one past the rows.
        const uint32_t* ps = L.pslot + d.pair_base;
        const uint32_t ns = (uint32_t)T.fs_stride;
        const int nfs = T.ell_w * T.fs_stride;
        const uint32_t fs0 = lds_addr(S.fs), pos0 = S.pos0;
        const int npad = round_up(T.np < 1 ? 1 : T.np, kPairPass);
        for (int p = l; p < npad; p += kWave) {
            uint4 r;
            if (p < T.np) {
                const uint32_t pk = T.gpairs[p], sl = ps[p];
                const uint32_t i = pk & 0xff, j = (pk >> 8) & 0xff;
                r.x = (pos0 + (i << 4)) | (pos0 + (j << 4)) << 16;
                r.y = fs0 + (((sl & 0xffff) * ns + i) << 4);
                r.z = fs0 + (((sl >> 16) * ns + j) << 4);
                r.w = __float_as_uint(fmaf((float)((pk >> 16) & 7u), 0.1f, 3.4f));
            } else {
                r.x = (pos0 + ((uint32_t)S.ma << 4)) | pos0 << 16;
                r.y = r.z = fs0 + ((uint32_t)nfs << 4);
                r.w = __float_as_uint(3.4f);
            }
            S.pairs[p] = r;
        }
        for (int k = l; k < nfs; k += kWave) S.fs[k] = make_float4(0.f, 0.f, 0.f, 0.f);   // padding stays zero
    } else {
        // one atom per lane: pair words up to a whole pass of 64 in LDS; the padding pairs join the far
        // point to atom 0, so they fall outside the cutoff and store c = 0
        // (which also serves the atom -> pair table's padding entries, p = np).
        // A word holds 16 i | 16 j << 12 (byte offsets in S.pos) | the
        // radius-sum code << 24, so that each part is one instruction away.
        if (A == 1) {
            // eight loads per lane in flight before their stores
            const int npad = round_up(T.np + 1, kWave);
            for (int p0 = l; p0 < npad; p0 += 8 * kWave) {
                uint32_t w[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int p = p0 + q * kWave;
                    w[q] = p < T.np ? T.gpairs[p] : (uint32_t)S.ma;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (p0 + q * kWave < npad)
                        S.pw[p0 + q * kWave] = (w[q] & 0xffu) << 4 | (w[q] & 0xff00u) << 8 | (w[q] & 0xff0000u) << 8;
            }
        }
        if (l == 0) S.cp[T.np] = 0.f;   // not written by the pair loop when np is a multiple of 64
    }
    wave_sync();
}

// ---------------------------------------------------------------- evaluation
struct Eval {
    float e, e_inter, e_intra;
    float g;          // this lane's tangent component (lane < 6 + T)
    int pairs_in;     // this lane's intra pairs inside the cutoff
    bool outside;     // some atom lies outside the box (its lookup was clamped)
    bool bounded;     // a trial decided by its map energy and the intra bound (no pair loop)
};

// Frame of every fragment: x = R X + b on reference coordinates.  Lane f
// starts from its local map (the root's pose map, or the rotation by psi
// about its torsion axis) and composes with its ancestors by pointer
// doubling; after `rounds` rounds every frame is world-absolute.
// y_first: the order in which the dock kernels of at most kShortM history pairs
// sum a line-search trial's frame offsets; every other evaluation starts from
// the x terms.  The searches are chaotic, so the last bits matter: each
// evaluation keeps the order it has always had, written out here because the
// compiler's own choice of fused products changes with the code around it.
template <int A, bool SL>
__device__ __forceinline__ void frames(const Topo<A, SL>& T, float pose, bool y_first, float R[9], float b[3])
{
    const int l = lane_id();
    // Local map of every fragment lane, one formula for the root and the
    // torsions: R = I + [s]x + w w^T - |w|^2 I, b = p - R a.
    //   root:     unit q = (qw, v): s = 2 qw v, w = sqrt(2) v; p = t, a = anchor
    //   torsion:  angle psi about unit axis u through c: with h = psi / 2,
    //             s = 2 sin h cos h u, w = sqrt(2) sin h u; p = a = c
    const float psi = from_lane(T.psi_src, pose);
    const float t0 = lane_f(pose, 0), t1 = lane_f(pose, 1), t2 = lane_f(pose, 2);
    const float qw = lane_f(pose, 3), qx = lane_f(pose, 4), qy = lane_f(pose, 5), qz = lane_f(pose, 6);
    const float qi = __builtin_amdgcn_rsqf(fmaf(qz, qz, fmaf(qy, qy, fmaf(qw, qw, qx * qx))));
    const bool root = l == 0;
    float sh, ch;
    __sincosf(0.5f * psi, &sh, &ch);
    const float ux = root ? qx * qi : T.ax, uy = root ? qy * qi : T.ay, uz = root ? qz * qi : T.az;
    const float k1 = root ? 2.f * qw * qi : 2.f * sh * ch;
    const float k2 = root ? 1.41421356f : 1.41421356f * sh;
    const float sx = k1 * ux, sy = k1 * uy, sz = k1 * uz;
    const float wx = k2 * ux, wy = k2 * uy, wz = k2 * uz;
    const float c0 = 1.f - fmaf(wz, wz, fmaf(wx, wx, wy * wy));
    R[0] = fmaf(wx, wx, c0);  R[1] = fmaf(wx, wy, -sz); R[2] = fmaf(wx, wz, sy);
    R[3] = fmaf(wx, wy, sz);  R[4] = fmaf(wy, wy, c0);  R[5] = fmaf(wy, wz, -sx);
    R[6] = fmaf(wx, wz, -sy); R[7] = fmaf(wy, wz, sx);  R[8] = fmaf(wz, wz, c0);
    const float px = root ? t0 : T.cx, py = root ? t1 : T.cy, pz = root ? t2 : T.cz;
    b[0] = px - fmaf(R[2], T.cz, fmaf(R[1], T.cy, R[0] * T.cx));
    // (x, y) or (y, x): the first product is rounded, the second fused onto it
    const float f1 = y_first ? R[4] : R[3], f2 = y_first ? R[7] : R[6], fc = y_first ? T.cy : T.cx;
    const float g1 = y_first ? R[3] : R[4], g2 = y_first ? R[6] : R[7], gc = y_first ? T.cx : T.cy;
    b[1] = py - fmaf(R[5], T.cz, fmaf(g1, gc, f1 * fc));
    b[2] = pz - fmaf(R[8], T.cz, fmaf(g2, gc, f2 * fc));
    // pointer doubling across lanes: every round each fragment fetches the
    // partial frame of its ancestor of that round (links jumped at staging)
    // straight from that lane's registers (ds_bpermute, all lanes taking
    // part), then composes, column by column in place; a lane without an
    // ancestor fetches its own values and keeps its frame
    uint32_t link = T.link0;
    for (int r = 0; r < T.rounds; ++r) {
        if (r == 4) link = T.link1;
        const int src = (int)(link & 0xffu);
        link >>= 8;
        float P[9], pb[3];
#pragma unroll
        for (int k = 0; k < 9; ++k) P[k] = from_lane(src, R[k]);
#pragma unroll
        for (int k = 0; k < 3; ++k) pb[k] = from_lane(src, b[k]);
        if (src != 4 * l) {
            auto turn = [&](float& x, float& y, float& z) {
                const float u = fmaf(P[0], x, P[1] * y), v = fmaf(P[3], x, P[4] * y), w = fmaf(P[6], x, P[7] * y);
                x = fmaf(P[2], z, u);
                y = fmaf(P[5], z, v);
                z = fmaf(P[8], z, w);
            };
            turn(R[0], R[3], R[6]);
            turn(R[1], R[4], R[7]);
            turn(R[2], R[5], R[8]);
            turn(b[0], b[1], b[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) b[k] += pb[k];
        }
    }
}

typedef float f3v __attribute__((ext_vector_type(3)));
constexpr float kLog2e = 1.4426950408889634f;

// One pass of U pairs per lane starting at pair c0 (the first lane's; uniform);
// adds this lane's energy to e and its pairs inside the cutoff to cnt.
template <int A, bool SL, int U>
__device__ __forceinline__ void pair_pass(const Topo<A, SL>& T, const Lds& S, int c0, float& e, int& cnt,
                                          const uint32_t* words = nullptr, float* part = nullptr)
{
    const int p0 = c0 + lane_id();
    // position addresses; slot addresses; radius sum bits (slots) or the
    // radius-sum code (gather)
    uint32_t ai[U], aj[U], ya[U], za[U], rc[U];
    bool v[U];
    float4 xi[U], xj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int p = p0 + u * kWave;
        if (SL) {
            const uint4 w = S.pairs[p];
            ai[u] = w.x & 0xffffu; aj[u] = w.x >> 16;
            ya[u] = w.y; za[u] = w.z; rc[u] = w.w;
            v[u] = true;
        } else {
            // LDS pair words are padded to whole passes of 64 with far-point
            // pairs; with two atoms per lane the caller brings the words
            // from global memory (a lane past the end holds pair 0 and
            // discards it)
            if (A == 1) {
                const uint32_t g = S.pw[p];
                v[u] = true;
                ai[u] = S.pos0 + (g & 0xff0u); aj[u] = S.pos0 + ((g >> 12) & 0xfffu);
                rc[u] = g >> 24;
            } else {
                const uint32_t g = words[u];
                v[u] = p < T.np;
                ai[u] = S.pos0 + ((g & 0xffu) << 4); aj[u] = S.pos0 + ((g >> 4) & 0xff0u);
                rc[u] = (g >> 16) & 0xffu;
            }
            ya[u] = za[u] = 0u;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        xi[u] = *(const float4*)lds_ptr<const float4>(ai[u]);
        xj[u] = *(const float4*)lds_ptr<const float4>(aj[u]);
    }
    float dx[U], dy[U], dz[U], d[U], en[U], de[U], rinv[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        dx[u] = xi[u].x - xj[u].x; dy[u] = xi[u].y - xj[u].y; dz[u] = xi[u].z - xj[u].z;
        const float r2 = dx[u] * dx[u] + dy[u] * dy[u] + dz[u] * dz[u];
        in[u] = v[u] && r2 < kCut2;
        // one v_rsq_f32: r = r2 / sqrt(r2) and c = de / r = de * rsq; a
        // zero distance gets a tiny finite r and its zero direction
        // zeroes the force
        const float r2c = fmaxf(r2, 1e-12f);
        rinv[u] = __builtin_amdgcn_rsqf(r2c);
        const float rs = SL ? __uint_as_float(rc[u]) : fmaf((float)rc[u], 0.1f, 3.4f);
        const float dd = r2c * rinv[u] - rs;
        d[u] = dd;
        // exp(-(d/0.5)^2) and exp(-((d-3)/2)^2), the second exponent
        // expanded around d^2 so both share it: c (d-3)^2 = c d^2 - 6c d + 9c
        const float d2 = dd * dd;
        const float g1 = __builtin_amdgcn_exp2f(d2 * (-4.f * kLog2e));
        constexpr float c2 = -0.25f * kLog2e;
        const float g2 = __builtin_amdgcn_exp2f(fmaf(d2, c2, fmaf(dd, -6.f * c2, 9.f * c2)));
        const float dn = fminf(dd, 0.f);                                             // repulsion d^2, d < 0
        en[u] = fmaf(kW1, g1, fmaf(kW2, g2, kW3 * (dn * dn)));
        constexpr float k2 = -0.5f * kW2;                                            // d/dd of the second: k2 (d-3)
        de[u] = fmaf(g1, dd * (-8.f * kW1), fmaf(g2, fmaf(dd, k2, -3.f * k2), dn * (2.f * kW3)));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        // class 1 (both hydrophobic) adds the hydrophobic term, class 2
        // (donor with acceptor) the hydrogen-bond term; the classes follow
        // one another in the pair list
        if (c0 + (u + 1) * kWave > T.np0 && c0 + u * kWave < T.np) {
            const int p = p0 + u * kWave;
            const float wy = p >= T.np0 && p < T.np1 ? kW4 : 0.f, wz = p >= T.np1 ? kW5 : 0.f;
            const float dd = d[u];
            const float hv = fminf(fmaxf(1.5f - dd, 0.f), 1.f);            // 1 below 0.5, 0 above 1.5
            const float bv = fminf(fmaxf(dd * -(1.f / 0.7f), 0.f), 1.f);   // 1 below -0.7, 0 above 0
            en[u] = fmaf(wy, hv, fmaf(wz, bv, en[u]));
            const float hs = (dd >= 0.5f && dd < 1.5f) ? -wy : 0.f;
            const float bs = (dd >= -0.7f && dd < 0.f) ? wz * -(1.f / 0.7f) : 0.f;
            de[u] += hs + bs;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (part) part[u * kWave + lane_id()] = in[u] ? en[u] : 0.f;
        else e += in[u] ? en[u] : 0.f;
        cnt += in[u] ? 1 : 0;
        const float c = in[u] ? de[u] * rinv[u] : 0.f;
        if (SL) {
            // 12-byte writes (ds_write_b96) into the 16-byte slots; the
            // gather reads x, y, z
            const float fx = c * dx[u], fy = c * dy[u], fz = c * dz[u];
            *(f3v*)lds_ptr<f3v>(ya[u]) = f3v{fx, fy, fz};
            *(f3v*)lds_ptr<f3v>(za[u]) = f3v{-fx, -fy, -fz};
        } else if (v[u]) {
            S.cp[p0 + u * kWave] = c;
        }
    }
}

// Intra pairs, lanes over pairs: whole passes of kPairUnroll pairs per lane
// (every load of a pass issued before any of its arithmetic, so the LDS
// latency is paid once per pass), then, on the gather layout with one atom
// per lane, whole passes of two pairs per lane and passes of one over the
// rest, so at most 63 padding pairs are evaluated.
// Per pair, with d the surface distance and inside 8 A: the gauss,
// repulsion, hydrophobic and hydrogen-bond terms of the Vina form and the
// force coefficient c = (dphi/dr) / r.  Pairs are grouped by interaction
// class, so a whole 64-pair chunk usually has no hydrophobic or
// hydrogen-bond weight and skips those terms on a wave-uniform branch.  With
// the slot layout each pair writes +f / -f into its slots of the two atoms'
// rows (records padded to whole passes, no per-lane guard); otherwise it
// stores c for the table gather.  No atomics either way.  Returns this
// lane's energy; adds this lane's pairs inside the cutoff to cnt.
template <int A, bool SL>
__device__ __forceinline__ float pair_loop(const Topo<A, SL>& T, const Lds& S, int& cnt)
{
    const int np = T.np;
    float e = 0.f;
    int c0 = 0;
    if (A > 1) {
        // two atoms per lane (ligands of 65 to 128 atoms, long pair lists):
        // whole passes only; the pair words come from global memory, each
        // pass's loaded during the pass before (a lane past the end reads
        // pair 0, np >= 1 here, and discards it)
        const int l = lane_id();
        uint32_t w[kPairUnroll], nw[kPairUnroll];
        if (np > 0) {
#pragma unroll
            for (int u = 0; u < kPairUnroll; ++u) {
                const int p = l + u * kWave;
                w[u] = T.gpairs[p < np ? p : 0];
            }
        }
        for (; c0 < np; c0 += kPairPass) {
#pragma unroll
            for (int u = 0; u < kPairUnroll; ++u) {
                const int p = c0 + l + kPairPass + u * kWave;
                nw[u] = T.gpairs[p < np ? p : 0];
            }
            pair_pass<A, SL, kPairUnroll>(T, S, c0, e, cnt, w);
#pragma unroll
            for (int u = 0; u < kPairUnroll; ++u) w[u] = nw[u];
        }
        return e;
    }
    // the slot form, a few waves per SIMD, pays more for another pass's
    // latency than for one chunk of padding: three chunks take a whole pass
    const int whole = SL ? kPairPass - kWave : kPairPass;
    for (; c0 + whole <= np || (SL && c0 + 2 * kWave < np); c0 += kPairPass) pair_pass<A, SL, kPairUnroll>(T, S, c0, e, cnt);
    for (; c0 + 2 * kWave <= np || (SL && c0 + kWave < np); c0 += 2 * kWave) pair_pass<A, SL, 2>(T, S, c0, e, cnt);
    for (; c0 < np; c0 += kWave) pair_pass<A, SL, 1>(T, S, c0, e, cnt);
    return e;
}

// The chunks [k, end) of 64 pairs; their energies go to part where it is given.
template <int A, bool SL>
__device__ __forceinline__ void pair_chunks(const Topo<A, SL>& T, const Lds& S, int k, int end, float& e, int& cnt,
                                            float* part)
{
    const int first = k;
    auto to = [&] { return part ? part + (k - first) * kWave : nullptr; };
    for (; k + kPairUnroll <= end; k += kPairUnroll) pair_pass<A, SL, kPairUnroll>(T, S, k * kWave, e, cnt, nullptr, to());
    if (k + 2 <= end) {
        pair_pass<A, SL, 2>(T, S, k * kWave, e, cnt, nullptr, to());
        k += 2;
    }
    if (k < end) pair_pass<A, SL, 1>(T, S, k * kWave, e, cnt, nullptr, to());
}

// row loads of the global atom -> pair table issued together by the gather:
// the table sits in L2, so a row walked one load at a time pays one L2
// round trip per four entries.  The loads are issued by four: past the row
// they read the next rows (past the last one the table's padding, kEllPad
// entries), which are not summed.
constexpr int kGatherChunk = 8;
static_assert(4 * kGatherChunk <= kEllPad, "the padding covers a chunk");

// dE/dx_i of the intra term.  LDS tables: the sum of atom i's row of pair
// forces (independent reads, rows padded to a multiple of four with zeros).
// Global tables: sum over the pairs holding atom i of c_p (x_i - x_j); an
// entry holds p's byte offset in S.cp in its low half and j's in S.pos in its high half.
template <int A, bool SL>
__device__ __forceinline__ void gather_pair_forces(const Topo<A, SL>& T, const Lds& S, int i, float4 xi, float& gx,
                                                   float& gy, float& gz)
{
    if (SL) {
        // sixteen, eight and four independent reads in flight per group (rows are
        // padded to a multiple of four); without the groups of sixteen the
        // five-pocket dock took 1% longer
        const float4* row = S.fs + i;
        const int ns = T.fs_stride;
        int k = 0;
        for (; k + 16 <= T.ell_w; k += 16) {
            float4 f[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) f[u] = row[(k + u) * ns];
#pragma unroll
            for (int u = 0; u < 16; ++u) { gx += f[u].x; gy += f[u].y; gz += f[u].z; }
        }
        for (; k + 8 <= T.ell_w; k += 8) {
            float4 f[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) f[u] = row[(k + u) * ns];
#pragma unroll
            for (int u = 0; u < 8; ++u) { gx += f[u].x; gy += f[u].y; gz += f[u].z; }
        }
        if (k < T.ell_w) {
            float4 f[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) f[u] = row[(k + u) * ns];
#pragma unroll
            for (int u = 0; u < 4; ++u) { gx += f[u].x; gy += f[u].y; gz += f[u].z; }
        }
        return;
    }
    // the atom's row is contiguous ([n][ell_w], ell_w a multiple of four): one
    // 16-byte load per four entries, a chunk's issued before any is used, so a
    // row of at most 4 * kGatherChunk entries pays one load latency.  Issued by
    // four with one base address and no test per load: the screening slice
    // 357 -> 351 ms, a batch score of 8-80 atoms 39.6 -> 36.0 us (all eight
    // without a test read too much: 375 ms).
    const char* row = (const char*)T.gell + (uint32_t)(i * T.ell_w * 4);
    for (int k0 = 0; k0 < T.ell_w; k0 += 4 * kGatherChunk) {
        uint4 e4[kGatherChunk];
#pragma unroll
        for (int q = 0; q < kGatherChunk; ++q)
            if (q < 4 || T.ell_w - k0 > 16) e4[q] = *(const uint4*)(row + (uint32_t)(k0 * 4) + 16 * q);
#pragma unroll
        for (int q = 0; q < kGatherChunk; ++q) {
            if (k0 + 4 * q >= T.ell_w) break;
            const uint32_t e[4] = {e4[q].x, e4[q].y, e4[q].z, e4[q].w};
            float c[4];
            float4 xj[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = *(const float*)((const char*)S.cp + (e[u] & 0xffff));
                xj[u] = *(const float4*)((const char*)S.pos + (e[u] >> 16));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                gx = fmaf(c[u], xi.x - xj[u].x, gx);
                gy = fmaf(c[u], xi.y - xj[u].y, gy);
                gz = fmaf(c[u], xi.z - xj[u].z, gz);
            }
        }
    }
}

// World position of one atom from its reference record (x, y, z, type |
// fragment << 8) and its fragment's frame in LDS.
__device__ __forceinline__ float4 atom_position(float4 ref, const Lds& S)
{
    const int f = __float_as_uint(ref.w) >> 8;
    const float4* fr = (const float4*)(S.frame + 12 * f);
    const float4 r0 = fr[0], r1 = fr[1], r2 = fr[2];
    const float x = r0.x * ref.x + r0.y * ref.y + r0.z * ref.z + r2.y;
    const float y = r0.w * ref.x + r1.x * ref.y + r1.y * ref.z + r2.z;
    const float z = r1.z * ref.x + r1.w * ref.y + r2.x * ref.z + r2.w;
    return make_float4(x, y, z, 0.f);
}

// Score and tangent gradient of the pose (entry l in lane l).  Leaves
// atom positions in S.pos and dE/dx in S.frc.  When the energy exceeds
// e_limit (a line-search trial that fails the sufficient-decrease test,
// whose gradient nobody reads) it returns after the energy, with g = 0 and
// S.frc not written.  use_bound lets such a trial try the intra lower bound
// before its pair loop.
template <int A, bool SL, int W = 1>
__device__ Eval evaluate(const Topo<A, SL>& T, const BoxView& B, const Lds& S, float pose,
                         float e_limit = __builtin_inff(), bool use_bound = true, bool y_first = false)
{
    const int l = lane_id();
    Eval out;
    float R[9], b[3];
    frames(T, pose, y_first, R, b);
    // the world axis of this fragment lane's torsion, the one use of the
    // frame after the atom positions (so R and b need not stay live)
    const float awx = R[0] * T.ax + R[1] * T.ay + R[2] * T.az;
    const float awy = R[3] * T.ax + R[4] * T.ay + R[5] * T.az;
    const float awz = R[6] * T.ax + R[7] * T.ay + R[8] * T.az;
    if (A > 1) {
        if (l < T.nf) {
            float* fr = S.frame + 12 * l;
#pragma unroll
            for (int k = 0; k < 9; ++k) fr[k] = R[k];
            fr[9] = b[0]; fr[10] = b[1]; fr[11] = b[2];
        }
        wave_sync();
    }
    float e_in = 0.f;
    float4 X4[A];
    float G[A][3];
    TriLoad TL[A];
    if (A == 1) {
        // one atom per lane: its fragment's frame straight from that lane
        const int src = (int)(__float_as_uint(T.ref[0].w) >> 8) << 2;
        float P[9], pb[3];
#pragma unroll
        for (int k = 0; k < 9; ++k) P[k] = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(R[k])));
#pragma unroll
        for (int k = 0; k < 3; ++k) pb[k] = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(b[k])));
        const float4 rf = T.ref[0];
        X4[0] = make_float4(P[0] * rf.x + P[1] * rf.y + P[2] * rf.z + pb[0],
                            P[3] * rf.x + P[4] * rf.y + P[5] * rf.z + pb[1],
                            P[6] * rf.x + P[7] * rf.y + P[8] * rf.z + pb[2], 0.f);
        G[0][0] = G[0][1] = G[0][2] = 0.f;
        if (l < T.n) {
            S.pos[l] = X4[0];
            if (W == 1) tri_issue(B, __float_as_uint(rf.w) & 0xff, X4[0].x, X4[0].y, X4[0].z, TL[0]);
        } else {
            X4[0] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    } else {
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = l * A + a;
            X4[a] = make_float4(0.f, 0.f, 0.f, 0.f);
            G[a][0] = G[a][1] = G[a][2] = 0.f;
            if (i < T.n) {
                X4[a] = atom_position(T.ref[a], S);
                S.pos[i] = X4[a];
            }
        }
    }
    wave_sync();
    // A line-search trial whose map energy plus the intra lower bound is
    // already above its sufficient-decrease bound is rejected by the full
    // energy too: it stops before the pair loop (a margin covers rounding).
    // The slot form runs few waves per SIMD, where ending the map loads before
    // the pair loop costs more latency than the skipped trials save: it
    // always runs both.
    const bool bound = !SL && use_bound && e_limit < 3.0e38f;   // wave-uniform
    bool outl = false, map_done = false;
    if (W == kLean || bound) {
        if (A > 1 || W == kLean) {
#pragma unroll
            for (int a = 0; a < A; ++a)
                if (l * A + a < T.n)
                    tri_issue(B, __float_as_uint(T.ref[a].w) & 0xff, X4[a].x, X4[a].y, X4[a].z, TL[a]);
        }
#pragma unroll
        for (int a = 0; a < A; ++a)
            if (l * A + a < T.n) {
                e_in += tri_finish(B, TL[a], G[a][0], G[a][1], G[a][2]);
                outl = outl || TL[a].cx || TL[a].cy || TL[a].cz;
            }
        out.e_inter = wsum(e_in);
        map_done = true;
        if (bound && out.e_inter + T.lb > e_limit + 1e-3f + 1e-4f * (fabsf(out.e_inter) + fabsf(T.lb))) {
            out.e_intra = T.lb;
            out.e = out.e_inter + T.lb;
            out.pairs_in = 0;
            out.outside = __ballot(outl) != 0;
            out.bounded = true;
            out.g = 0.f;
            wave_sync();
            return out;
        }
        // the map forces wait in the scan area (unused until the scans), so
        // no registers are held across the pair loop
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = l * A + a;
            if (i < T.n) { S.pre[i] = G[a][0]; S.pre[S.ma + i] = G[a][1]; S.pre[2 * S.ma + i] = G[a][2]; }
        }
    }
    int cnt = 0;
    float e_ia = 0.f;
    if (W > 1) {
        const int nc = (T.np + kWave - 1) / kWave, own = team_chunk<W>(nc, 1);
        team_sync();
        pair_chunks(T, S, 0, own, e_ia, cnt, nullptr);
        team_sync();
        // four energies in flight
        const float* part = S.part + l;
        int k = own;
        for (; k + 4 <= nc; k += 4, part += 4 * kWave) {
            const float p0 = part[0], p1 = part[kWave], p2 = part[2 * kWave], p3 = part[3 * kWave];
            e_ia += p0; e_ia += p1; e_ia += p2; e_ia += p3;
        }
        if (k < nc) {
            const float p0 = part[0], p1 = part[k + 1 < nc ? kWave : 0], p2 = part[k + 2 < nc ? 2 * kWave : 0];
            e_ia += p0;
            if (k + 1 < nc) e_ia += p1;
            if (k + 2 < nc) e_ia += p2;
        }
#pragma unroll
        for (int h = 0; h < W - 1; ++h) {
            const uint32_t c = S.count[h * kWave + l];
            cnt += (int)(c & 0x7fffffffu);
            outl = c >> 31;
        }
        if (l < T.n) {
            const float4 m = S.map[l];
            G[0][0] = m.x; G[0][1] = m.y; G[0][2] = m.z;
        }
        out.e_inter = lane_f(*S.e_map, 0);
    } else {
        e_ia = pair_loop(T, S, cnt);   // hides the map loads (one atom per lane)
    }
    // the energy sums start here, so their cross-lane steps overlap the
    // force gather and the scans below
    out.e_intra = wsum(e_ia);
    wave_sync();
    if (W <= 1 && !map_done) {
        if (A > 1) {
            // two atoms per lane: the map loads start only now, since holding
            // both lookups across the pair loop would cost a resident wave
#pragma unroll
            for (int a = 0; a < A; ++a)
                if (l * A + a < T.n)
                    tri_issue(B, __float_as_uint(T.ref[a].w) & 0xff, X4[a].x, X4[a].y, X4[a].z, TL[a]);
        }
#pragma unroll
        for (int a = 0; a < A; ++a)
            if (l * A + a < T.n) {
                e_in += tri_finish(B, TL[a], G[a][0], G[a][1], G[a][2]);
                outl = outl || TL[a].cx || TL[a].cy || TL[a].cz;
            }
        out.e_inter = wsum(e_in);
    } else if (W <= 1) {
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = l * A + a;
            if (i < T.n) { G[a][0] = S.pre[i]; G[a][1] = S.pre[S.ma + i]; G[a][2] = S.pre[2 * S.ma + i]; }
        }
    }
    out.outside = __ballot(outl) != 0;
    out.bounded = false;
    out.e = out.e_inter + out.e_intra;
    out.pairs_in = cnt;
    if (out.e > e_limit) {    // wave-uniform
        out.g = 0.f;
        wave_sync();
        return out;
    }
#pragma unroll
    for (int a = 0; a < A; ++a)
        if (l * A + a < T.n) gather_pair_forces(T, S, l * A + a, X4[a], G[a][0], G[a][1], G[a][2]);
    // per-atom force (inter + intra) and torque about t, blocked scan over atoms
    const float tx = lane_f(pose, 0), ty = lane_f(pose, 1), tz = lane_f(pose, 2);
    float v[A][6];
    float run[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int i = l * A + a;
        float rx = 0, ry = 0, rz = 0;
        if (i < T.n) {
            if (S.frc) S.frc[i] = make_float4(G[a][0], G[a][1], G[a][2], 0.f);
            rx = X4[a].x - tx; ry = X4[a].y - ty; rz = X4[a].z - tz;
        }
        const float m[6] = {G[a][0], G[a][1], G[a][2], fmaf(ry, G[a][2], -(rz * G[a][1])),
                            fmaf(rz, G[a][0], -(rx * G[a][2])), fmaf(rx, G[a][1], -(ry * G[a][0]))};
#pragma unroll
        for (int c = 0; c < 6; ++c) run[c] = a == 0 ? m[c] : run[c] + m[c];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[a][c] = run[c];
    }
    float incl[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) incl[c] = run[c];
    wscan6(incl);
    // atom i's prefix: lane i's inclusive scan (one atom per lane), else the
    // lane's exclusive scan plus its running sum up to the atom
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        if (A == 1) {
            if (l < T.n) S.pre[c * S.ma + l] = incl[c];
        } else {
            const float excl = incl[c] - run[c];
#pragma unroll
            for (int a = 0; a < A; ++a) {
                const int i = l * A + a;
                if (i < T.n) S.pre[c * S.ma + i] = excl + v[a][c];
            }
        }
    }
    wave_sync();
    // torsion derivative: world axis . sum over the moved atoms of (x - x_c) x G
    const float total = S.pre[(l < 6 ? l : 0) * S.ma + T.n - 1];
    float dpsi = 0.f;
    if (l >= 1 && l < T.nf) {
        const int e = T.f_end - 1, s0 = T.f_a0 - 1;
        float Sg[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) Sg[c] = S.pre[c * S.ma + e] - S.pre[c * S.ma + s0];
        const float4 pc = S.pos[T.f_child];
        const float cx = pc.x - tx, cy = pc.y - ty, cz = pc.z - tz;
        const float mx = Sg[3] - (cy * Sg[2] - cz * Sg[1]);
        const float my = Sg[4] - (cz * Sg[0] - cx * Sg[2]);
        const float mz = Sg[5] - (cx * Sg[1] - cy * Sg[0]);
        dpsi = awx * mx + awy * my + awz * mz;
    }
    const float own = __int_as_float(__builtin_amdgcn_ds_bpermute(T.dof_src, __float_as_int(dpsi)));
    out.g = l < 6 ? total : l < 6 + T.nt ? own : 0.f;
    wave_sync();
    return out;
}

// Wave w > 0 of a chain's team: until the chain ends, its chunks of pairs of each
// evaluation and, the last wave, the map lookups.
template <int W, int A, bool SL>
__device__ void help(const Topo<A, SL>& T, const BoxView& B, const Lds& S, int w)
{
    const int l = lane_id();
    const int type = __float_as_uint(T.ref[0].w) & 0xff;
    __builtin_amdgcn_s_setprio(2);   // the chain waits for it
    const bool maps = w == W - 1 && l < T.n;
    const int nc = (T.np + kWave - 1) / kWave, first = team_chunk<W>(nc, w), end = team_chunk<W>(nc, w + 1);
    float* part = S.part + (first - team_chunk<W>(nc, 1)) * kWave;
    while (true) {
        team_sync();   // the positions are in place, or the chain has ended
        if (__builtin_amdgcn_readfirstlane(*S.done)) break;
        TriLoad L;
        if (maps) {
            const float4 p = S.pos[l];
            tri_issue(B, type, p.x, p.y, p.z, L);
        }
        int cnt = 0;
        float e = 0.f;
        pair_chunks(T, S, first, end, e, cnt, part);
        uint32_t outl = 0;
        if (w == W - 1) {
            float em = 0.f;
            if (maps) {
                float4 m;
                em += tri_finish(B, L, m.x, m.y, m.z);
                m.w = 0.f;
                S.map[l] = m;
                outl = L.cx || L.cy || L.cz;
            }
            em = wsum(em);
            if (l == 0) *S.e_map = em;
        }
        S.count[(w - 1) * kWave + l] = (uint32_t)cnt | outl << 31;
        team_sync();
    }
}

// Score on given coordinates already in S.pos: forces in S.frc (with grads).
template <int A, bool SL>
__device__ Eval evaluate_xyz(const Topo<A, SL>& T, const BoxView& B, const Lds& S, bool grads)
{
    const int l = lane_id();
    Eval out;
    float e_in = 0.f;
    int cnt = 0;
    const float e_ia = pair_loop(T, S, cnt);
    wave_sync();
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int i = l * A + a;
        if (i < T.n) {
            const int ty = __float_as_uint(T.ref[a].w) & 0xff;
            const float4 p = S.pos[i];
            float gx, gy, gz;
            e_in += trilinear(B, ty, p.x, p.y, p.z, gx, gy, gz);
            if (grads) {
                gather_pair_forces(T, S, i, p, gx, gy, gz);
                if (S.frc) S.frc[i] = make_float4(gx, gy, gz, 0.f);
            }
        }
    }
    wave_sync();
    out.g = 0.f;
    out.outside = false;
    out.bounded = false;
    out.e_inter = wsum(e_in);
    out.e_intra = wsum(e_ia);
    out.e = out.e_inter + out.e_intra;
    out.pairs_in = cnt;
    return out;
}

// ---------------------------------------------------------------- pose registers
// the value one lane below / above (whole-wave shifts)
__device__ __forceinline__ float lane_below(float v) { return dpp0<0x138>(v); }   // wave_shr:1
__device__ __forceinline__ float lane_above(float v) { return dpp0<0x130>(v); }   // wave_shl:1

// pose entries 3..6 replaced by the quaternion q
__device__ __forceinline__ float with_quat(float v, const float q[4])
{
    const int l = lane_id();
    v = l == 6 ? q[3] : v;
    v = l == 5 ? q[2] : v;
    v = l == 4 ? q[1] : v;
    return l == 3 ? q[0] : v;
}

// x (+) lam d : t + lam d_t, exp(lam d_theta) q, psi + lam d_psi.  d is the
// lane-distributed tangent vector.
__device__ __forceinline__ float retract(float x, float d, float lam)
{
    const int l = lane_id();
    const float th0 = lane_f(d, 3) * lam, th1 = lane_f(d, 4) * lam, th2 = lane_f(d, 5) * lam;
    float dq[4], q[4] = {lane_f(x, 3), lane_f(x, 4), lane_f(x, 5), lane_f(x, 6)}, nq[4];
    rotvec_quat(th0, th1, th2, dq);
    quat_mul(dq, q, nq);
    quat_normalize(nq);
    // pose entries 0..2 move by tangent lanes 0..2, entry k >= 7 (a torsion)
    // by tangent lane k - 1
    const float below = lane_below(d);
    return with_quat(fmaf(lam, l < 3 ? d : below, x), nq);
}

// ---------------------------------------------------------------- RILC-BFGS
constexpr int kMaxM = 8;     // the most history pairs a search may keep (bfgs_m)
constexpr int kShortM = 5;   // the dock kernel is also built for at most this many (the default m): the history
                             // lives in registers, and room for 8 pairs cost the shift and copies of 3 more

struct BfgsOut {
    float x;          // this lane's pose entry at the result
    float f;
    float g;          // this lane's tangent gradient component at the result
    int evals;
    int grads;        // evaluations that computed the gradient
    int bounded;      // evaluations decided by the intra lower bound (no pair loop)
    int64_t pairs;    // this lane's share of the intra pairs inside the cutoff
    bool skipped;     // the consistency check ended the run after its first evaluation
    bool outside0;    // the start pose has an atom outside the box
};

// The neighbour of a mutated pose for the first-order consistency check:
// the current pose x, its energy and this lane's tangent
// gradient component, and the tangent coordinates [p_lo, p_hi) the
// mutation moved.
struct CheckIn {
    float x, f, g;
    int p_lo, p_hi;
};

__device__ __forceinline__ float fsgn(float v) { return (float)((v > 0.f) - (v < 0.f)); }

// Eqs. qvina_eq_4 and qvina_eq_5 for the pose x (energy fx, this
// lane's gradient gx) against its neighbour: true (optimise) when in some
// tested coordinate the derivative changes sign between the two poses or
// disagrees with the secant slope.  Tangent differences: translation, the
// rotation vector of q_x conj(q_cur) (only its sign is used), torsions
// wrapped to (-pi, pi].
__device__ __forceinline__ bool consistency_passes(float x, float fx, float gx, const CheckIn& ck)
{
    const int l = lane_id();
    const float y = ck.x, xa = lane_above(x), ya = lane_above(y);
    float dl = 0.f;
    if (l < 3) {
        dl = x - y;
    } else if (l < 6) {
        const float qx[4] = {lane_f(x, 3), lane_f(x, 4), lane_f(x, 5), lane_f(x, 6)};
        const float cy[4] = {lane_f(y, 3), -lane_f(y, 4), -lane_f(y, 5), -lane_f(y, 6)};
        float qd[4];
        quat_mul(qx, cy, qd);
        const float v = l == 3 ? qd[1] : (l == 4 ? qd[2] : qd[3]);
        dl = qd[0] < 0.f ? -v : v;
    } else if (l + 1 < kSlot) {
        const float kPi = 3.14159265358979f, k2Pi = 6.28318530717959f;
        float d = xa - ya;
        d -= k2Pi * floorf((d + kPi) * (1.f / k2Pi));
        dl = d == -kPi ? kPi : d;
    }
    const bool in = l >= ck.p_lo && l < ck.p_hi;
    const float sx = fsgn(gx);
    const bool hold = sx * fsgn(ck.g) <= 0.f || sx * fsgn(fx - ck.f) * fsgn(dl) <= 0.f;
    return __ballot(in && hold) != 0;
}

// Minimises from the pose x (entry l in lane l); the result is out.x.  The
// start's evaluation and the line search's are two copies of the evaluation
// code; the line search is a loop of its own, so that the state of the outer
// iteration (the history above all) stays in its registers across the trials.
template <int A, bool SL, int MM = kMaxM, int W = 1>
__device__ BfgsOut bfgs(const Topo<A, SL>& T, const BoxView& B, const Lds& S, const SearchParams& P, int max_iter,
                        float x, bool check = false, CheckIn ck = CheckIn{0.f, 0.f, 0.f, 0, 0})
{
    static_assert(MM >= 1 && MM <= kMaxM, "history capacity");
    const int l = lane_id();
    const int nd = 6 + T.nt;
    const bool act = l < nd;
    BfgsOut out;
    const Eval e0 = evaluate<A, SL, W>(T, B, S, x);
    float f = e0.e, g = act ? e0.g : 0.f;
    out.evals = out.grads = 1;
    out.bounded = 0;
    out.pairs = e0.pairs_in;
    out.outside0 = e0.outside;
    out.skipped = check && !consistency_passes(x, f, g, ck);
    float Sh[MM], Yh[MM], rh[MM];
#pragma unroll
    for (int h = 0; h < MM; ++h) { Sh[h] = 0.f; Yh[h] = 0.f; rh[h] = 0.f; }
    int hn = 0;
    const int m = P.m;
    float sy_new = 0.f, yy_new = 1.f;   // s.y and y.y of the newest stored pair (the H0 scale)
    for (int it = 0; it < max_iter && !out.skipped; ++it) {
        const float gn = __builtin_amdgcn_sqrtf(wdot_n(g, g, nd));
        if (gn <= P.eps_g) break;                 // Eq. qvina_eq_12
        // two-loop recursion: d = -H g (d = -g with no pairs, Eq. qvina_eq_6)
        float q = g, al[MM];
#pragma unroll
        for (int h = MM - 1; h >= 0; --h) {
            al[h] = 0.f;
            if (h < hn) {
                al[h] = rh[h] * wdot_n(Sh[h], q, nd);
                q = fmaf(-Yh[h], al[h], q);
            }
        }
        if (hn > 0) q *= sy_new * __builtin_amdgcn_rcpf(yy_new);
#pragma unroll
        for (int h = 0; h < MM; ++h) {
            if (h < hn) {
                const float bb = rh[h] * wdot_n(Yh[h], q, nd);
                q = fmaf(Sh[h], al[h] - bb, q);
            }
        }
        const float d = -q;
        const float gd = wdot_n(g, d, nd);
        if (!(gd < 0.f)) break;                   // not a descent direction
        // Lewis-Overton search (Eqs. qvina_eq_7 and qvina_eq_8): lam between
        // lo, the largest step at or below the sufficient-decrease bound, and
        // beta, the least above it
        float lo = 0.f, lam = 1.f, beta = 0.f, fn = 0.f, gnw = 0.f, xn = x, lam_ok = 0.f;
        bool beta_inf = true;
        for (int tr = 0;; ) {
            const float xt = retract(x, d, lam);
            // a trial above the sufficient-decrease bound needs no gradient.  The
            // intra bound decides an iteration's first trial (the full step) less
            // often than the later ones, and with one atom per lane trying it costs
            // the corner loads their cover by the pair loop: that form tries it
            // once a trial of the iteration has failed, and while no history pair
            // is stored, when the full step is the unscaled gradient step
            const float armijo = fmaf(P.rho * lam, gd, f);
            const Eval ev = evaluate<A, SL, W>(T, B, S, xt, armijo,
                                               !(P.flags & kDockNoIntraBound) && (A > 1 || tr > 0 || hn == 0), MM <= kShortM);
            const float ft = ev.e, gt = act ? ev.g : 0.f;
            const bool above = ft > armijo;
            ++out.evals;
            out.grads += above ? 0 : 1;
            out.bounded += ev.bounded ? 1 : 0;
            out.pairs += ev.pairs_in;
            bool accepted = false;
            if (above) {
                beta = lam; beta_inf = false;
            } else {
                // kept as the fallback too, should the trials run out
                accepted = !(wdot_n(gt, d, nd) < P.sigma * gd);
                lo = lam_ok = lam;
                fn = ft; gnw = gt; xn = xt;
            }
            if (accepted || ++tr >= P.ls_max) break;
            lam = beta_inf ? 2.f * lam : 0.5f * (lo + beta);
        }
        if (!(lam_ok > 0.f)) break;
        // s = lam d, y = g+ - g; cautious update (Eqs. qvina_eq_10, qvina_eq_11)
        const float sv = lam_ok * d, yv = gnw - g;
        const float ys = wdot_n(yv, sv, nd), ss = wdot_n(sv, sv, nd), yy = wdot_n(yv, yv, nd);
        if (ys * __builtin_amdgcn_rcpf(ss) > P.eps_c * gn) {
            sy_new = ys;
            yy_new = yy;
            if (hn == m) {
#pragma unroll
                for (int h = 0; h < MM - 1; ++h) { Sh[h] = Sh[h + 1]; Yh[h] = Yh[h + 1]; rh[h] = rh[h + 1]; }
                --hn;
            }
#pragma unroll
            for (int h = 0; h < MM; ++h)
                if (h == hn) { Sh[h] = sv; Yh[h] = yv; rh[h] = __builtin_amdgcn_rcpf(ys); }
            ++hn;
        }
        x = xn;   // Eq. qvina_eq_9
        f = fn;
        g = gnw;
    }
    out.x = x;
    out.f = f;
    out.g = g;
    return out;
}

// ---------------------------------------------------------------- Monte Carlo
struct ChainOut {
    float best_x;                  // this lane's entry of the best pose
    float best_e;
    int64_t evals, grads, bounded, pairs;   // pairs: this lane's share
    int status;                    // PV_JOB_BUDGET | PV_JOB_OUTSIDE bits
};

constexpr int kStatusBudget = 2, kStatusOutside = 4;   // the PV_JOB_* bits of the ABI

template <int A, bool SL>
__device__ float init_pose(const Topo<A, SL>& T, const BoxView& B, uint64_t seed, int job, int chain)
{
    const int l = lane_id();
    // lane l draws uniform l (block l/4, word l%4) of step 0
    const float u = u01(philox_word(seed, job, chain, 0, (uint64_t)(l >> 2), l & 3));
    const float u3 = lane_f(u, 3), u4 = lane_f(u, 4), u5 = lane_f(u, 5);
    const float s1 = sqrtf(1.f - u3), s2 = sqrtf(u3);
    float sa, ca, sb, cb;
    sincosf(2.f * kPi * u4, &sa, &ca);
    sincosf(2.f * kPi * u5, &sb, &cb);
    // entry k >= 7 takes uniform k - 1
    const float w = lane_below(u);
    float x = l >= 7 && l < 7 + T.nt ? -kPi + 2.f * kPi * w : 0.f;
    if (l == 0) x = B.ox + u * B.ex;
    if (l == 1) x = B.oy + u * B.ey;
    if (l == 2) x = B.oz + u * B.ez;
    const float q[4] = {s2 * cb, s1 * sa, s1 * ca, s2 * sb};
    return with_quat(x, q);
}

// The pose x with one POT entity mutated (Eq. qvina_eq_2) from the 8 words w
// of the step.
template <int A, bool SL>
__device__ float mutate(const Topo<A, SL>& T, float x, const SearchParams& P, const uint64_t w[8])
{
    const int l = lane_id();
    const uint64_t n_ent = (uint64_t)(2 + T.nt);
    const int ent = (int)(((w[0] >> 32) * n_ent) >> 32);
    const float u1 = u01(w[1]), u2 = u01(w[2]), u3 = u01(w[3]), u4 = u01(w[4]);
    const float ur = u01(w[5]), ua = u01(w[6]);
    const float r12 = sqrtf(-2.f * logf(1.f - u1)), r34 = sqrtf(-2.f * logf(1.f - u3));
    float s2, c2, s4, c4;
    sincosf(2.f * kPi * u2, &s2, &c2);
    sincosf(2.f * kPi * u4, &s4, &c4);
    const float vx = r12 * c2, vy = r12 * s2, vz = r34 * c4;
    const float vn2 = vx * vx + vy * vy + vz * vz;
    float dx = 0.f, dy = 0.f, dz = 1.f;
    if (vn2 > 0.f) { const float inv = 1.f / sqrtf(vn2); dx = vx * inv; dy = vy * inv; dz = vz * inv; }
    const float rad = cbrtf(ur);
    if (ent == 0) {
        const float a = P.pos_amp * rad;
        const float mv = l == 0 ? dx : (l == 1 ? dy : dz);
        if (l < 3) x += a * mv;
    } else if (ent == 1) {
        const float amp = P.rot_amp * T.rot_scale * rad;
        float dq[4], q[4] = {lane_f(x, 3), lane_f(x, 4), lane_f(x, 5), lane_f(x, 6)}, nq[4];
        rotvec_quat(amp * dx, amp * dy, amp * dz, dq);
        quat_mul(dq, q, nq);
        quat_normalize(nq);
        x = with_quat(x, nq);
    } else {
        if (l == 7 + (ent - 2)) x = -kPi + 2.f * kPi * ua;
    }
    return x;
}

// Wave priority from the chain's predicted remaining work: its evaluations
// per step so far times the steps left, per step of the whole run.  Waves
// that share a SIMD (or a CU's LDS and memory pipes) then serve the chain
// with the most work left first, which shortens a launch that ends with its
// longest chain.  Arbitration only: the results do not change.
__device__ __forceinline__ void chain_priority(int64_t evals, int s, int steps)
{
    const float q = (float)evals * (float)(steps - s) / ((float)s * (float)steps);
    if (q >= 24.f) __builtin_amdgcn_s_setprio(3);
    else if (q >= 16.f) __builtin_amdgcn_s_setprio(2);
    else if (q >= 8.f) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

template <int A, bool SL, int MM = kMaxM, int W = 1>
__device__ ChainOut mc_chain(const Topo<A, SL>& T, const BoxView& B, const Lds& S, const SearchParams& P, int job,
                             int chain)
{
    const int l = lane_id();
    ChainOut out;
    out.evals = 0;
    out.grads = 0;
    out.bounded = 0;
    out.pairs = 0;
    out.status = 0;
    float x = init_pose(T, B, P.seed, job, chain), best = x;
    float e_cur = 0.f, e_best = 0.f, um = 0.f;
    CheckIn ck;            // the current pose, also the consistency check's neighbour
    ck.x = x;
    ck.g = 0.f;
    ck.p_lo = ck.p_hi = 0;
    // 0 initial pose, 1 step optimisation, 2 refinement, 3 the closing
    // look at the best pose (one uncounted evaluation: is it inside the box?)
    int s = 0, mode = 0;
    while (true) {
        const int iters = mode == 0 || mode == 3 ? 0 : (mode == 1 ? P.max_iter : P.refine_max_iter);
        ck.f = e_cur;
        const BfgsOut bo = bfgs<A, SL, MM, W>(T, B, S, P, iters, x, mode == 1 && P.consistency, ck);
        if (mode == 3) {
            if (bo.outside0) out.status |= kStatusOutside;
            break;
        }
        out.evals += bo.evals;
        out.grads += bo.grads;
        out.bounded += bo.bounded;
        out.pairs += bo.pairs;
        bool next = true;
        if (mode == 0) {
            e_cur = e_best = bo.f;
            ck.g = bo.g;
            ck.x = best = bo.x;
        } else if (mode == 1) {
            if (!bo.skipped) {
                const float e_o = bo.f;
                if (e_o < e_cur || um < __expf((e_cur - e_o) / P.temperature)) {   // Eq. qvina_eq_13
                    ck.x = bo.x;
                    e_cur = e_o;
                    ck.g = bo.g;
                }
                if (e_o < e_best) { mode = 2; next = false; x = bo.x; }
            }
        } else {
            ck.x = best = bo.x;
            e_best = bo.f;
            e_cur = bo.f;
            ck.g = bo.g;
        }
        if (!next) continue;
        const bool spent = P.max_evals > 0 && out.evals >= P.max_evals;
        if (spent) out.status |= kStatusBudget;
        if (s >= P.steps || spent) {
            x = best;
            mode = 3;
            continue;
        }
        // the 8 draws of step s + 1: lanes 0-3 compute block 0, lanes 4-7 block 1
        const uint64_t mine = philox_word(P.seed, job, chain, (uint64_t)s + 1, (uint64_t)((l >> 2) & 1), l & 3);
        uint64_t w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t lo = (uint32_t)lane_i((int)(uint32_t)mine, k);
            const uint32_t hi = (uint32_t)lane_i((int)(uint32_t)(mine >> 32), k);
            w[k] = ((uint64_t)hi << 32) | lo;
        }
        um = u01(w[7]);
        // tangent coordinates the mutation moves (its entity draw, as in mutate)
        const int ent = (int)(((w[0] >> 32) * (uint64_t)(2 + T.nt)) >> 32);
        ck.p_lo = ent == 0 ? 0 : (ent == 1 ? 3 : 4 + ent);
        ck.p_hi = ent <= 1 ? ck.p_lo + 3 : ck.p_lo + 1;
        x = mutate(T, ck.x, P, w);
        ++s;
        mode = 1;
        chain_priority(out.evals, s, P.steps);
    }
    __builtin_amdgcn_s_setprio(0);
    out.best_x = best;
    out.best_e = e_best;
    return out;
}

// ---------------------------------------------------------------- kernels

// Two waves per SIMD for the slot form and the two-atom form: without the
// hint they take AGPRs above 256 VGPRs and fall to one wave (with it the slot
// form holds 244 VGPRs, the two-atom form 256 with 8 spilled).  The one-atom
// gather form fits two waves by itself and is faster without the hint.  With
// helper waves (W > 1) three waves per SIMD, see team_chunk.
template <int A, bool SL, int MM, int W = 1>
__global__ __launch_bounds__(64 * (W > 1 ? W : 1))
__attribute__((amdgpu_waves_per_eu(W != 1 ? 3 : SL || A > 1 ? 2 : 1))) void dock_kernel(DockArgs a)
{
    extern __shared__ __align__(16) char smem[];
    const LdsNeeds nd = kernel_needs(kKindDock, A, SL, W == kLean);
    Lds S = carve(smem, a.l.max_atoms, a.l.max_pairs, a.l.max_ell, nd);
    if (W > 1) carve_team<W>(S, smem + lds_bytes(a.l.max_atoms, a.l.max_pairs, a.l.max_ell, nd), a.l.max_atoms);
    const int l = lane_id();
    Topo<A, SL> T;
    T.lig = -1;
    const int chains = a.sp.chains;
    const bool persistent = W <= 1 && a.persistent;   // with helpers every chain has its workgroup
    int64_t item = persistent ? -1 : (int64_t)blockIdx.x;
    while (true) {
        if (persistent) {
            uint32_t v = 0;
            if (l == 0) v = atomicAdd(a.queue, 1u);
            item = (int64_t)(uint32_t)lane_i((int)v, 0);
        }
        if (item >= a.n_items) break;
        const int gj = (int)(item / chains);
        const int job = a.job_map ? a.job_map[gj] : a.job_begin + gj;
        const int chain = (int)(item % chains);
        const int2 jb = a.jobs[job];
        const int wave = W > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.y) : 0;
        if (jb.x != T.lig) stage_ligand(T, a.l, jb.x, S, wave == 0);
        BoxView B = box_view(a.g, jb.y);
        if (W == kLean) {
            to_scalar(T);
            to_scalar(B);
        }
        if (W > 1) {
            if (wave == 0 && l == 0) *S.done = 0;
            team_sync();
            if (wave > 0) {
                help<W>(T, B, S, wave);
                break;
            }
        }
        uint64_t t0 = 0;
        if (a.sp.flags & 1u) t0 = wall_clock64();
        ChainOut co = mc_chain<A, SL, MM, W>(T, B, S, a.sp, job, chain);
        if (W > 1) {
            if (l == 0) *S.done = 1;
            team_sync();
        }
        const int64_t pairs = wsum_i64(co.pairs);
        const int64_t ci = (int64_t)job * chains + chain;
        if (a.chain_best_dof && l < a.dof_stride)
            a.chain_best_dof[ci * a.dof_stride + l] = l < 7 + T.nt ? co.best_x : 0.f;
        if (l == 0) {
            if (a.chain_best_e) a.chain_best_e[ci] = co.best_e;
            if (a.chain_evals) a.chain_evals[ci] = co.evals;
            if (a.chain_pairs) a.chain_pairs[ci] = pairs;
            if (a.chain_grads) a.chain_grads[ci] = co.grads;
            if (a.chain_bounded) a.chain_bounded[ci] = co.bounded;
            a.chain_status[ci] = co.status;
            if (a.sp.flags & 1u) {
                const uint64_t t1 = wall_clock64();
                atomicMin((unsigned long long*)&a.job_t_start[job], (unsigned long long)t0);
                atomicMax((unsigned long long*)&a.job_t_end[job], (unsigned long long)t1);
            }
        }
        wave_sync();
        if (!persistent) break;
    }
}

// zeroes both size classes' queue counters
__global__ void reset_queue_kernel(uint32_t* q) { if (threadIdx.x < 2) q[threadIdx.x] = 0u; }

// Measurement aid, the VALU FP32 issue rate: every thread runs 16 independent
// multiply-add chains for `iters` rounds with no memory traffic and stores
// their sum once, so the launch is bound by FMA issue alone.
__global__ __launch_bounds__(256) void fma_peak_kernel(float* out, int iters)
{
    const int gid = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    const float a = 0.999999f, b = 1e-7f * (float)(threadIdx.x & 7u);
    float x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = (float)(gid + k) * 1e-6f;
#pragma unroll 4
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = fmaf(x[k], a, b);
    }
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += x[k];
    out[gid] = sum;
}

__global__ void reset_times_kernel(uint64_t* t0, uint64_t* t1, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) { t0[i] = ~0ull; t1[i] = 0ull; }
}

// Per job: the best chain (lowest energy, ties to the lower chain, a number
// before NaN), the evaluation total and the status bits: not finite, some
// chain stopped at its budget, the best chain's pose outside the box.
__global__ void job_reduce_kernel(const float* cbe, const int64_t* cev, const int32_t* cst, int n_jobs, int chains,
                                  float* jbe, int32_t* jbc, int64_t* jev, int32_t* jst)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_jobs) return;
    int bc = 0;
    float be = cbe[(int64_t)j * chains];
    int64_t ev = cev ? cev[(int64_t)j * chains] : 0;
    int budget = cst[(int64_t)j * chains] & kStatusBudget;
    for (int c = 1; c < chains; ++c) {
        const float e = cbe[(int64_t)j * chains + c];
        if (e < be || (be != be && e == e)) { be = e; bc = c; }
        if (cev) ev += cev[(int64_t)j * chains + c];
        budget |= cst[(int64_t)j * chains + c] & kStatusBudget;
    }
    if (jbe) jbe[j] = be;
    if (jbc) jbc[j] = bc;
    if (jev) jev[j] = ev;
    if (jst) jst[j] = (isfinite(be) ? 0 : 1) | budget | (cst[(int64_t)j * chains + bc] & kStatusOutside);
}

// The one-atom gather form fits three waves per SIMD in 168 VGPRs (4 of them
// spilled to scratch; three waves measured 10% faster than two); the other
// forms need more.
template <int A, bool SL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(A == 1 && !SL ? 3 : 1))) void score_kernel(ScoreArgs a)
{
    extern __shared__ __align__(16) char smem[];
    const Lds S = carve(smem, a.l.max_atoms, a.l.max_pairs, a.l.max_ell, kernel_needs(kKindScore, A, SL));
    const int l = lane_id();
    Topo<A, SL> T;
    T.lig = -1;
    const float nanv = __int_as_float(0x7fc00000);
    // a contiguous run of poses per workgroup (runs of one ligand stage it
    // once), the runs' lengths differing by at most one so no wave idles
    const int p_begin = (int)(((int64_t)blockIdx.x * a.n_poses) / (int64_t)gridDim.x);
    const int p_end = (int)(((int64_t)(blockIdx.x + 1) * a.n_poses) / (int64_t)gridDim.x);
    // the next pose's indices and pose vector are loaded while this one is
    // evaluated (lane l holds pose entry l)
    const bool dof_in = !a.from_xyz, grads = a.grad_dof || a.grad_xyz;
    int n_lig = 0, n_box = 0;
    float n_dof = 0.f;
    if (p_begin < p_end) {
        n_lig = a.lig_of_pose[p_begin];
        n_box = a.box_of_pose[p_begin];
        if (dof_in && l < a.dof_stride) n_dof = a.dof[(int64_t)p_begin * a.dof_stride + l];
    }
    for (int pose = p_begin; pose < p_end; ++pose) {
        const int lig = n_lig, box = n_box;
        const float dof_l = n_dof;
        if (pose + 1 < p_end) {
            n_lig = a.lig_of_pose[pose + 1];
            n_box = a.box_of_pose[pose + 1];
            if (dof_in && l < a.dof_stride) n_dof = a.dof[(int64_t)(pose + 1) * a.dof_stride + l];
        }
        if (lig < 0 || lig >= a.l.n_lig || box < 0 || box >= a.g.n_boxes) {
            if (l == 0 && a.energy) a.energy[pose] = nanv;
            if (l < 2 && a.e_parts) a.e_parts[2 * (int64_t)pose + l] = nanv;
            if (a.grad_dof && l < a.dof_stride) a.grad_dof[(int64_t)pose * a.dof_stride + l] = nanv;
            for (int k = l; k < 3 * a.xyz_stride; k += kWave) {
                if (a.xyz_out && !a.from_xyz) a.xyz_out[(int64_t)pose * a.xyz_stride * 3 + k] = nanv;
                if (a.grad_xyz) a.grad_xyz[(int64_t)pose * a.xyz_stride * 3 + k] = nanv;
            }
            continue;
        }
        if (lig != T.lig) stage_ligand(T, a.l, lig, S);
        const BoxView B = box_view(a.g, box);
        const float scale = a.grad_energy ? a.grad_energy[pose] : 1.f;
        const int16_t* perm = a.l.perm + a.l.ligs[lig].atom_base;
        Eval ev;
        if (!a.from_xyz) {
            // without a gradient output the evaluation ends with the energy,
            // as a rejected line-search trial's does
            ev = evaluate(T, B, S, dof_l, grads ? __builtin_inff() : -__builtin_inff(), false);
        } else {
            for (int i = l; i < T.n; i += kWave) {
                const float* src = a.dof + ((int64_t)pose * a.xyz_stride + perm[i]) * 3;
                S.pos[i] = make_float4(src[0], src[1], src[2], 0.f);
            }
            wave_sync();
            ev = evaluate_xyz(T, B, S, grads);
        }
        if (l == 0 && a.energy) a.energy[pose] = ev.e;
        if (a.e_parts && l < 2) a.e_parts[2 * (int64_t)pose + l] = l == 0 ? ev.e_inter : ev.e_intra;
        if (a.grad_dof && !a.from_xyz) {
            // dE/dt, dE/d(raw q) = 2 ((0, torque) (x) q)/|p|, dE/dpsi
            const float tq0 = lane_f(ev.g, 3), tq1 = lane_f(ev.g, 4), tq2 = lane_f(ev.g, 5);
            const float dpsi = __shfl(ev.g, l - 1 < 0 ? 0 : (l - 1 > 63 ? 63 : l - 1));
            float p[4] = {lane_f(dof_l, 3), lane_f(dof_l, 4), lane_f(dof_l, 5), lane_f(dof_l, 6)};
            const float pn = sqrtf(p[0] * p[0] + p[1] * p[1] + p[2] * p[2] + p[3] * p[3]);
            float qh[4] = {p[0] / pn, p[1] / pn, p[2] / pn, p[3] / pn};
            float t4[4] = {0.f, tq0, tq1, tq2}, gq[4];
            quat_mul(t4, qh, gq);
            float v = 0.f;
            if (l < 3) v = ev.g;
            if (l == 3) v = 2.f * gq[0] / pn;
            if (l == 4) v = 2.f * gq[1] / pn;
            if (l == 5) v = 2.f * gq[2] / pn;
            if (l == 6) v = 2.f * gq[3] / pn;
            if (l >= 7 && l < 7 + T.nt) v = dpsi;
            if (l < a.dof_stride) a.grad_dof[(int64_t)pose * a.dof_stride + l] = l < 7 + T.nt ? v * scale : 0.f;
        }
        if (a.xyz_out || a.grad_xyz) {
            // rows past the ligand's atoms (a batch of mixed sizes) are zero
            for (int k = 3 * T.n + l; k < 3 * a.xyz_stride; k += kWave) {
                if (a.xyz_out && !a.from_xyz) a.xyz_out[(int64_t)pose * a.xyz_stride * 3 + k] = 0.f;
                if (a.grad_xyz) a.grad_xyz[(int64_t)pose * a.xyz_stride * 3 + k] = 0.f;
            }
            for (int i = l; i < T.n; i += kWave) {
                const int64_t o = ((int64_t)pose * a.xyz_stride + perm[i]) * 3;
                if (a.xyz_out) {
                    const float4 p = S.pos[i];
                    a.xyz_out[o] = p.x; a.xyz_out[o + 1] = p.y; a.xyz_out[o + 2] = p.z;
                }
                if (a.grad_xyz) {
                    const float4 f = S.frc[i];
                    a.grad_xyz[o] = f.x * scale; a.grad_xyz[o + 1] = f.y * scale; a.grad_xyz[o + 2] = f.z * scale;
                }
            }
        }
        wave_sync();
    }
}

// The backward of a score whose gradient the forward computed: each row times
// its pose's upstream factor, a value per thread and round.  Values past the ligand's
// own (7 + torsions of a pose vector, 3 per atom of coordinates) are 0, or NaN
// where the pose's ligand or box does not exist, and stay so whatever the
// factor.  16,384 poses of 17 values take 3 us; evaluating them again took 63.
__global__ __launch_bounds__(256) void scale_grad_kernel(LigDev L, int64_t n, int row, const int32_t* lig_of_pose,
                                                         bool of_xyz, const float* grad, const float* scale, float* out)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int pose = (int)(i / row), k = (int)(i % row), lig = lig_of_pose[pose];
        const float v = grad[i];
        int own = 0;
        if (lig >= 0 && lig < L.n_lig) own = of_xyz ? 3 * L.ligs[lig].n_atoms : 7 + L.ligs[lig].n_tors;
        out[i] = k < own ? v * scale[pose] : v;
    }
}

// a launch may not have 2^32 threads in a dimension: from 2^31 values on a thread takes several
constexpr int64_t kScaleBlocks = (int64_t)1 << 23;

hipError_t launch_scale_grad(const LigDev& l, int64_t n, int row, const int32_t* lig_of_pose, bool of_xyz,
                             const float* grad, const float* scale, float* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, kScaleBlocks);
    hipLaunchKernelGGL(scale_grad_kernel, dim3((unsigned)blocks), dim3(256), 0, s, l, n, row, lig_of_pose, of_xyz, grad,
                       scale, out);
    return hipGetLastError();
}

template <int A, bool SL, int W = 1>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(W == kLean ? 3 : SL || A > 1 ? 2 : 1))) void local_opt_kernel(OptArgs a)
{
    extern __shared__ __align__(16) char smem[];
    const Lds S = carve(smem, a.l.max_atoms, a.l.max_pairs, a.l.max_ell, kernel_needs(kKindOpt, A, SL, W == kLean));
    const int l = lane_id();
    Topo<A, SL> T;
    T.lig = -1;
    for (int pose = blockIdx.x; pose < a.n_poses; pose += gridDim.x) {
        const int lig = a.lig_of_pose[pose], box = a.box_of_pose[pose];
        if (lig < 0 || lig >= a.l.n_lig || box < 0 || box >= a.g.n_boxes) {
            if (l == 0 && a.energy) a.energy[pose] = __int_as_float(0x7fc00000);
            continue;
        }
        if (lig != T.lig) stage_ligand(T, a.l, lig, S);
        BoxView B = box_view(a.g, box);
        if (W == kLean) {
            to_scalar(T);
            to_scalar(B);
        }
        float v = l < 7 + T.nt ? a.dof_in[(int64_t)pose * a.dof_stride + l] : 0.f;
        // normalise the quaternion once so the run starts from a unit q
        float q0 = lane_f(v, 3), q1 = lane_f(v, 4), q2 = lane_f(v, 5), q3 = lane_f(v, 6);
        const float qn = rsqrtf(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
        if (l >= 3 && l < 7) v *= qn;
        const BfgsOut bo = bfgs<A, SL, kMaxM, W>(T, B, S, a.sp, a.sp.max_iter, v);
        if (l < a.dof_stride) a.dof_out[(int64_t)pose * a.dof_stride + l] = l < 7 + T.nt ? bo.x : 0.f;
        if (l == 0) {
            if (a.energy) a.energy[pose] = bo.f;
            if (a.n_evals) a.n_evals[pose] = bo.evals;
        }
        wave_sync();
    }
}

// ---------------------------------------------------------------- output stage
// Atom positions of the pose (entry l in lane l) into S.pos.
template <int A, bool SL>
__device__ void pose_positions(const Topo<A, SL>& T, const Lds& S, float pose)
{
    const int l = lane_id();
    float R[9], b[3];
    frames(T, pose, false, R, b);
    if (l < T.nf) {
        float* fr = S.frame + 12 * l;
#pragma unroll
        for (int k = 0; k < 9; ++k) fr[k] = R[k];
        fr[9] = b[0]; fr[10] = b[1]; fr[11] = b[2];
    }
    wave_sync();
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int i = l * A + a;
        if (i < T.n) S.pos[i] = atom_position(T.ref[a], S);
    }
    wave_sync();
}

// Order of the output stage: a before b for a smaller energy, any number
// before NaN, then the lower index.
__device__ __forceinline__ bool precedes(float ea, int ia, float eb, int ib)
{
    const bool na = ea != ea, nb = eb != eb;
    if (na != nb) return nb;
    if (!na && ea != eb) return ea < eb;
    return ia < ib;
}

// Sum over atoms of |S.pos - other|^2 (identical in every lane).
template <int A, bool SL>
__device__ __forceinline__ float sq_dev(const Topo<A, SL>& T, const Lds& S, const float4* other)
{
    const int l = lane_id();
    float s = 0.f;
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int i = l * A + a;
        if (i < T.n) {
            const float4 p = S.pos[i], q = other[i];
            const float dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
            s += dx * dx + dy * dy + dz * dz;
        }
    }
    return wsum(s);
}

// One workgroup per job (Methods, end of "Accelerated Docking with QuickVina
// 2-GPU 2.1"; last steps of Supplementary Algorithm 2): the chains' best
// poses in ascending energy; greedy r.m.s.d. clustering keeps a pose unless
// it lies within rmsd_cut of a kept one, up to `modes`; each kept pose is
// refined by BFGS and rescored (E, and the affinity e_inter / (1 + w T));
// the refined poses are sorted again, filtered by r.m.s.d. the same way and
// written out.  r.m.s.d. < cut is tested as sum |dx|^2 < cut^2 N.
//
// Bound by the latency of one wave's chain of evaluations, so a job's work is
// spread over up to kOutWaves waves (threadIdx.y), each with its own LDS
// tables: they take the clustering's poses a batch at a time (each wave its
// pose against the kept ones and against the batch's earlier ones, then the
// batch is decided in order from the recorded conflicts), the refinements and
// the rows of the final filter's conflict table.  Every comparison and every
// refinement is the one a single wave makes, so the results do not depend on
// the number of waves (output_waves).  One wave -> this: 5 jobs x 256 chains, 20 modes 718 ->
// 141 us; 256 jobs of 65-80 atoms x 16 chains 1,294 -> 359 us.
constexpr int kOutWaves = 8;

template <int A>
__global__ __launch_bounds__(kWave * kOutWaves) void output_kernel(OutputArgs a)
{
    extern __shared__ __align__(16) char smem[];
    const int W = (int)blockDim.y, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int one = lds_bytes(a.l.max_atoms, a.l.max_pairs, a.l.max_ell, kernel_needs(kKindOutput, A, false));
    Lds S = carve(smem + wv * one, a.l.max_atoms, a.l.max_pairs, a.l.max_ell, kernel_needs(kKindOutput, A, false));
    S.pos0 = lds_addr(S.pos);
    char* ext = smem + W * one;
    const int ma = S.ma, M = a.modes, C = a.chains;
    int* order = (int*)ext;     ext += round_up(C, 4) * 4;
    float4* rep = (float4*)ext; ext += M * ma * 16;
    float* rdof = (float*)ext;  ext += M * kSlot * 4;
    float* re = (float*)ext;    ext += round_up(M, 4) * 4;
    float* ra = (float*)ext;    ext += round_up(M, 4) * 4;
    int* kc = (int*)ext;        ext += round_up(M, 4) * 4;
    int* fo = (int*)ext;        ext += round_up(M, 4) * 4;
    // conflict masks of the final filter; before it, the next pose to refine
    uint32_t* conf = (uint32_t*)ext;
    // conflict masks of a clustering batch, in the first wave's scan area (no evaluation runs meanwhile)
    uint32_t* flags = (uint32_t*)(smem + ((char*)S.pre - S.base));
    static_assert(kOutWaves <= 6 * 4, "the scan area holds 6 x 4 words at least");
    constexpr uint32_t kStands = 0x80000000u;   // a pose of the batch that no kept pose excludes
    const int l = lane_id(), tid = wv * kWave + l, nthr = W * kWave;
    const int job = blockIdx.x;
    Topo<A, false> T;
    T.lig = -1;
    const int2 jb = a.jobs[job];
    stage_ligand(T, a.l, jb.x, S);
    const BoxView B = box_view(a.g, jb.y);
    const float* ce = a.chain_e + (int64_t)job * C;
    const float cut2n = a.rmsd_cut * a.rmsd_cut * (float)T.n;
    // 1. chains in ascending energy (rank of each chain by counting)
    for (int c = tid; c < C; c += nthr) {
        const float ec = ce[c];
        int rank = 0;
#pragma unroll 8
        for (int c2 = 0; c2 < C; ++c2) rank += precedes(ce[c2], c2, ec, c) ? 1 : 0;
        order[rank] = c;
    }
    if (tid == 0) conf[0] = 0;
    __syncthreads();
    // 2. greedy clustering in that order, W poses at a time
    int nk = 0;
    for (int r0 = 0; r0 < C && nk < M; r0 += W) {
        const int r = r0 + wv;
        bool stands = r < C;
        if (stands) {
            const float* src = a.chain_dof + ((int64_t)job * C + order[r]) * a.in_stride;
            pose_positions(T, S, l < 7 + T.nt ? src[l] : 0.f);
            for (int q = 0; q < nk && stands; ++q) stands = !(sq_dev(T, S, rep + q * ma) < cut2n);
        }
        __syncthreads();   // every wave's positions are in place
        uint32_t f = stands ? kStands : 0u;
        for (int w = 0; w < wv && stands; ++w)
            if (sq_dev(T, S, (const float4*)(smem + w * one + ((char*)S.pos - S.base))) < cut2n) f |= 1u << w;
        if (l == 0) flags[wv] = f;
        __syncthreads();
        uint32_t kept = 0;
        for (int w = 0; w < W && nk < M; ++w) {
            const uint32_t fw = flags[w];
            if (!(fw & kStands) || (fw & kept)) continue;
            kept |= 1u << w;
            if (w == wv) {
#pragma unroll
                for (int aa = 0; aa < A; ++aa) {
                    const int i = l * A + aa;
                    if (i < T.n) rep[nk * ma + i] = S.pos[i];
                }
                if (l == 0) kc[nk] = order[r];
            }
            ++nk;
        }
        __syncthreads();   // the batch's flags and positions are read, its kept poses stored
    }
    // 3. refine and rescore every kept pose, each wave the next one when it is free
    while (true) {
        uint32_t v0 = 0;
        if (l == 0) v0 = atomicAdd(&conf[0], 1u);
        const int q = lane_i((int)v0, 0);
        if (q >= nk) break;
        const float* src = a.chain_dof + ((int64_t)job * C + kc[q]) * a.in_stride;
        float v = l < 7 + T.nt ? src[l] : 0.f;
        if (a.refine_max_iter > 0) v = bfgs(T, B, S, a.sp, a.refine_max_iter, v).x;
        // a unit quaternion, then the rescoring evaluation
        if (l >= 7 + T.nt) v = 0.f;
        const float q0 = lane_f(v, 3), q1 = lane_f(v, 4), q2 = lane_f(v, 5), q3 = lane_f(v, 6);
        const float qn = 1.f / sqrtf(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
        if (l >= 3 && l < 7) v *= qn;
        const Eval ev = evaluate(T, B, S, v);
#pragma unroll
        for (int aa = 0; aa < A; ++aa) {
            const int i = l * A + aa;
            if (i < T.n) rep[q * ma + i] = S.pos[i];
        }
        if (l < kSlot) rdof[q * kSlot + l] = v;
        if (l == 0) {
            re[q] = ev.e;
            ra[q] = ev.e_inter / (1.f + a.affinity_w * (float)T.nt);
        }
        wave_sync();
    }
    __syncthreads();
    // 4. final sort of the refined poses, r.m.s.d. filter, output
    if (tid < nk) {
        int rank = 0;
        for (int q2 = 0; q2 < nk; ++q2) rank += precedes(re[q2], q2, re[tid], tid) ? 1 : 0;
        fo[rank] = tid;
    }
    __syncthreads();
    for (int r = wv; r < nk; r += W) {
#pragma unroll
        for (int aa = 0; aa < A; ++aa) {
            const int i = l * A + aa;
            if (i < T.n) S.pos[i] = rep[fo[r] * ma + i];
        }
        wave_sync();
        uint32_t m = 0;
        for (int s2 = 0; s2 < r; ++s2)
            if (sq_dev(T, S, rep + fo[s2] * ma) < cut2n) m |= 1u << s2;
        if (l == 0) conf[r] = m;
        wave_sync();
    }
    __syncthreads();
    const int64_t o0 = (int64_t)job * M;
    int no = 0;
    uint32_t kept = 0;
    for (int r = 0; r < nk; ++r) {
        if (conf[r] & kept) continue;
        kept |= 1u << r;
        if (no % W == wv) {
            const int q = fo[r];
            if (l == 0) {
                a.mode_chain[o0 + no] = kc[q];
                a.mode_e[o0 + no] = re[q];
                if (a.mode_affinity) a.mode_affinity[o0 + no] = ra[q];
            }
            if (a.mode_dof && l < a.out_stride)
                a.mode_dof[(o0 + no) * a.out_stride + l] = l < 7 + T.nt ? rdof[q * kSlot + l] : 0.f;
        }
        ++no;
    }
    const float nanv = __int_as_float(0x7fc00000);
    for (int o = no + tid; o < M; o += nthr) {
        a.mode_chain[o0 + o] = -1;
        a.mode_e[o0 + o] = nanv;
        if (a.mode_affinity) a.mode_affinity[o0 + o] = nanv;
    }
    if (a.mode_dof)
        for (int o = no + wv; o < M; o += W)
            if (l < a.out_stride) a.mode_dof[(o0 + o) * a.out_stride + l] = 0.f;
    if (tid == 0) a.n_modes[job] = no;
}

// ---------------------------------------------------------------- grid maps
// One workgroup of four waves per 16x4x4 tile of one box, a wave per 4x4x4
// points: a cube of 1.1 A edges at the usual spacing, so that the points of a
// wave lie at nearly one distance of a receptor atom.
// The receptor atoms near the box are streamed in chunks of 256; those within
// reach of the tile are appended in the atoms' order (a ballot per wave, the
// waves' counts in wave order) to a list in LDS.  Each wave then tests the
// list 64 atoms at a time against its own cube and walks the bits of the
// ballot.  Every point so sums its terms in the atoms' order on every build
// and the maps are reproducible bit for bit.
//
// Bound by VALU issue (the VALU is busy throughout; 68 instructions per wave
// and atom, 110 atoms per wave where 79 reach an average point).  A term of a
// far atom needs one exponential per ligand radius (the second gaussian
// alone), a near one two and the linear terms, so a wave branches on whether
// any of its points is near.  16 pockets of 20-30 A (4.5e6 points, 8,000
// atoms): 1,900 us with waves of 16x4x1 points that computed every term of
// every atom, 955 us now; 32 boxes of 15-30 A (7.4e6 points): 3,190 -> 1,690.
// Tiles of 8x4x4 take 17% longer, 16x8x4 2%, 16x8x8 54%; 8x8x8 2% less on
// many boxes and 5% more on one.
constexpr int kGridThreads = kTileX * kTileY * kTileZ;
constexpr int kGridList = 2 * kGridThreads;             // LDS list entries
constexpr int kGridRun = 4;                             // consecutive tiles one XCD takes (see below)

// The 8 A cutoff of a map term as r < 8 on binary64 values: the lattice
// point origin + h i, the differences, squares and sum each rounded on its
// own (no contraction).  s < 64 decides as the correctly rounded sqrt(s) < 8
// does: the largest binary64 s below 64 has a root that rounds below 8.  Used
// for the few (point, atom) pairs whose binary32 squared distance lies within
// 0.01 A^2 of 64, where binary32 rounding could decide the other way.
__device__ __forceinline__ bool within_cutoff_f64(int i, int j, int k, float ox, float oy, float oz, float h,
                                                  float ax, float ay, float az)
{
#pragma clang fp contract(off)
    const double gx = (double)ox + (double)h * (double)i;
    const double gy = (double)oy + (double)h * (double)j;
    const double gz = (double)oz + (double)h * (double)k;
    const double dx = gx - (double)ax, dy = gy - (double)ay, dz = gz - (double)az;
    const double s = dx * dx + dy * dy + dz * dz;
    return s < 64.0;
}

// The 8 maps' sums at one point, by ligand type (named registers: an array
// here is copied whole where the branches below meet).
struct MapSums {
    float ch, cp, np, nd, na, oa, oda, sp;
};

// Adds one receptor atom's terms at distance r of this lane's point.  rt (the
// atom's XS type) is wave-uniform; rs: its radius plus the ligand radii C, N,
// O and S.
// From d = 2.25 A on (kGridFar) a term is its second gaussian alone, bit for
// bit: the first one's share, 0.0356 exp(-4 d^2), is below a quarter of a unit
// in the last place of 0.00516 exp(-(d-3)^2/4) there (4 d^2 - (d-3)^2/4 > 20.1),
// and the other terms are zero.
constexpr float kGridFar = 2.25f;

__device__ __forceinline__ void add_map_terms(float r, int rt, float4 rs, MapSums& m)
{
#pragma clang fp contract(off)
    constexpr float kE = 1.4426950408889634f;   // log2 e
    const float dc = r - rs.x, dn = r - rs.y, dx = r - rs.z, ds = r - rs.w;
    auto gauss2 = [](float d) {
#pragma clang fp contract(off)
        const float t = d - 3.f;
        return kW2 * __builtin_amdgcn_exp2f(t * t * (-0.25f * kE));
    };
    float bc = gauss2(dc), bn = gauss2(dn), bo = gauss2(dx), bs = gauss2(ds);
    if (__ballot(ds < kGridFar) == 0) {   // the S radius has the smallest d
        m.ch += bc;
        m.cp += bc;
        m.np += bn;
        m.nd += bn;
        m.na += bn;
        m.oa += bo;
        m.oda += bo;
        m.sp += bs;
        // an opaque use of the sums: without it the compiler merges these
        // additions with the near path's and moves every register there
        asm volatile("" : "+v"(m.ch), "+v"(m.cp), "+v"(m.np), "+v"(m.nd), "+v"(m.na), "+v"(m.oa), "+v"(m.oda), "+v"(m.sp));
        return;
    }
    auto gauss1 = [](float d, float b) {
#pragma clang fp contract(off)
        return __builtin_fmaf(__builtin_amdgcn_exp2f(d * d * (-4.f * kE)), kW1, b);
    };
    bc = gauss1(dc, bc); bn = gauss1(dn, bn); bo = gauss1(dx, bo); bs = gauss1(ds, bs);
    if (__ballot(ds < 0.f)) {
        auto repel = [](float d, float b) {
#pragma clang fp contract(off)
            const float v = __builtin_fmaf(kW3 * d, d, b);
            return d < 0.f ? v : b;
        };
        bc = repel(dc, bc); bn = repel(dn, bn); bo = repel(dx, bo); bs = repel(ds, bs);
    }
    float vch = bc, vnd = bn, vna = bn, voa = bo, voda = bo;
    if (rt == 0 && __ballot(dc < 1.5f)) {   // both hydrophobic
        const float v = kW4 * (1.5f - dc);
        const float w = dc < 1.5f ? v : 0.f;
        vch += dc < 0.5f ? kW4 : w;
    }
    const bool don = rt == 3 || rt == 6, acc = rt == 4 || rt == 5 || rt == 6;
    if ((don || acc) && __ballot(dn < 0.f)) {   // hydrogen bonds; the N radius has the smaller d
        auto hbond = [](float d) {
#pragma clang fp contract(off)
            const float v = kW5 * (d * -(1.f / 0.7f));
            const float w = d < 0.f ? v : 0.f;
            return d < -0.7f ? kW5 : w;
        };
        const float hn = bn + hbond(dn), ho = bo + hbond(dx);
        vnd = acc ? hn : bn;
        vna = don ? hn : bn;
        voa = don ? ho : bo;
        voda = ho;
    }
    m.ch += vch;
    m.cp += bc;
    m.np += bn;
    m.nd += vnd;
    m.na += vna;
    m.oa += voa;
    m.oda += voda;
    m.sp += bs;
}

// squared distance from an atom to the box [lo, hi]
__device__ __forceinline__ float box_dist2(const float4& at, const float lo[3], const float hi[3])
{
    const float dx = fmaxf(fmaxf(lo[0] - at.x, at.x - hi[0]), 0.f);
    const float dy = fmaxf(fmaxf(lo[1] - at.y, at.y - hi[1]), 0.f);
    const float dz = fmaxf(fmaxf(lo[2] - at.z, at.z - hi[2]), 0.f);
    return dx * dx + dy * dy + dz * dz;
}

__global__ __launch_bounds__(kGridThreads) void gridmap_kernel(GridBuildArgs a)
{
    constexpr int kWaves = kGridThreads / kWave;
    __shared__ float4 list[kGridList], rsum[kGridList];   // atom records; their radii plus each ligand radius
    __shared__ int wave_n[2][kWaves];
    const int l = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // Workgroups go round robin to the 8 XCDs: each XCD takes runs of kGridRun
    // consecutive tiles, so that tiles that share map lines write them through
    // one L2.
    const int q = blockIdx.x >> 3;
    const int tile = a.first_tile + (q / kGridRun) * (8 * kGridRun) + (blockIdx.x & 7) * kGridRun + q % kGridRun;
    if (tile >= a.tile_off[a.n_boxes]) return;
    // which box: the boxes whose first tile is at or before this one
    int box = -1;
    for (int b0 = 0; b0 < a.n_boxes; b0 += kWave)
        box += __popcll(__ballot(b0 + l < a.n_boxes && a.tile_off[b0 + l] <= tile));
    const int nx = a.dims[4 * box], ny = a.dims[4 * box + 1], nz = a.dims[4 * box + 2];
    const float ox = a.geom[8 * box], oy = a.geom[8 * box + 1], oz = a.geom[8 * box + 2], h = a.geom[8 * box + 3];
    const int tx = (nx + kTileX - 1) / kTileX, ty = (ny + kTileY - 1) / kTileY;
    const int t = tile - a.tile_off[box];
    const int x0 = t % tx * kTileX, y0 = (t / tx) % ty * kTileY, z0 = t / (tx * ty) * kTileZ;
    // this lane's point; points past the lattice repeat its last one and are not stored
    constexpr int kWx = kTileX / 4, kWy = kTileY / 4;
    const int cx = 4 * (wv % kWx), cy = 4 * (wv / kWx % kWy), cz = 4 * (wv / (kWx * kWy));   // the wave's cube in the tile
    const int wx = x0 + cx, wy = y0 + cy, wz = z0 + cz;
    const bool idle = wx >= nx || wy >= ny || wz >= nz;
    const int i = min(wx + (l & 3), nx - 1), j = min(wy + ((l >> 2) & 3), ny - 1), k = min(wz + (l >> 4), nz - 1);
    const float gx = fmaf((float)i, h, ox), gy = fmaf((float)j, h, oy), gz = fmaf((float)k, h, oz);
    // bounding boxes of the tile's and of the wave's points
    const float tlo[3] = {fmaf((float)x0, h, ox), fmaf((float)y0, h, oy), fmaf((float)z0, h, oz)};
    const float thi[3] = {fmaf((float)(min(x0 + kTileX, nx) - 1), h, ox), fmaf((float)(min(y0 + kTileY, ny) - 1), h, oy),
                          fmaf((float)(min(z0 + kTileZ, nz) - 1), h, oz)};
    const float wlo[3] = {fmaf((float)wx, h, ox), fmaf((float)wy, h, oy), fmaf((float)wz, h, oz)};
    const float whi[3] = {fmaf((float)(min(wx + 4, nx) - 1), h, ox), fmaf((float)(min(wy + 4, ny) - 1), h, oy),
                          fmaf((float)(min(wz + 4, nz) - 1), h, oz)};
    const float reach2 = 8.01f * 8.01f;
    MapSums acc = {0, 0, 0, 0, 0, 0, 0, 0};
    const int abeg = a.atom_off[box], aend = a.atom_off[box + 1];
    int n = 0, flip = 0;
    float4 next = abeg + (int)threadIdx.x < aend ? a.atoms[abeg + threadIdx.x] : make_float4(0.f, 0.f, 0.f, 0.f);
    for (int base = abeg; base < aend; base += kGridThreads) {
        const float4 at = next;
        const int an = base + kGridThreads + (int)threadIdx.x;
        if (an < aend) next = a.atoms[an];
        const bool keep = base + (int)threadIdx.x < aend && box_dist2(at, tlo, thi) < reach2;
        const uint64_t m = __ballot(keep);
        if (l == 0) wave_n[flip][wv] = __popcll(m);
        __syncthreads();
        int off = n;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int c = wave_n[flip][w];
            off += w < wv ? c : 0;
            n += c;
        }
        // the next chunk writes the other counts, so those readers may lag
        flip ^= 1;
        if (keep) {
            off += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const int rt = __float_as_int(at.w) & 0xff;
            const float Rr = rt <= 1 ? 1.9f : rt <= 4 ? 1.8f : rt <= 6 ? 1.7f : 2.0f;
            list[off] = at;
            rsum[off] = make_float4(1.9f + Rr, 1.8f + Rr, 1.7f + Rr, 2.0f + Rr);
        }
        if (n + kGridThreads <= kGridList && base + kGridThreads < aend) continue;   // room for one more chunk
        __syncthreads();
        for (int c0 = 0; c0 < n && !idle; c0 += kWave) {
            uint64_t near = __ballot(c0 + l < n && box_dist2(list[min(c0 + l, n - 1)], wlo, whi) < reach2);
            if (!near) continue;
            // the next atom's record is read while this one is worked on
            int q = c0 + __builtin_ctzll(near);
            float4 nc = list[q], ns = rsum[q];
            while (near) {
                const float4 c = nc, rs = ns;
                near &= near - 1;
                q = near ? c0 + __builtin_ctzll(near) : c0;
                nc = list[q];
                ns = rsum[q];
                const float dx = gx - c.x, dy = gy - c.y, dz = gz - c.z;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                bool in = r2 < kCut2 - 0.01f;
                // from kCut2 - 0.01 to below kCut2 + 0.01, as one unsigned range (r2 >= 0)
                const uint32_t lo = __float_as_uint(kCut2 - 0.01f), hi = __float_as_uint(kCut2 + 0.01f);
                if (__float_as_uint(r2) - lo < hi - lo)
                    in = r2 <= kCut2 - 0.01f || within_cutoff_f64(i, j, k, ox, oy, oz, h, c.x, c.y, c.z);
                const int rt = __builtin_amdgcn_readfirstlane(__float_as_int(c.w)) & 0xff;
                if (in) add_map_terms(__builtin_amdgcn_sqrtf(r2), rt, rs, acc);
            }
        }
        n = 0;
        __syncthreads();
    }
    // through LDS, so that the stores go out in rows of 16 points
    float* stage = (float*)list;
    static_assert(sizeof(list) >= 8 * kGridThreads * sizeof(float), "the list area holds the tile's maps");
    const float sums[8] = {acc.ch, acc.cp, acc.np, acc.nd, acc.na, acc.oa, acc.oda, acc.sp};
#pragma unroll
    for (int m = 0; m < 8; ++m)
        stage[m * kGridThreads + ((cz + (l >> 4)) * kTileY + cy + ((l >> 2) & 3)) * kTileX + cx + (l & 3)] = sums[m];
    __syncthreads();
    const int si = x0 + (int)threadIdx.x % kTileX, sj = y0 + ((int)threadIdx.x / kTileX) % kTileY,
              sk = z0 + (int)threadIdx.x / (kTileX * kTileY);
    if (si < nx && sj < ny && sk < nz) {
        const int64_t msz = (int64_t)nx * ny * nz;
        float* out = a.maps + a.map_off[box] + ((int64_t)sk * ny + sj) * nx + si;
#pragma unroll
        for (int m = 0; m < 8; ++m) out[m * msz] = stage[m * kGridThreads + threadIdx.x];
    }
}

// ---------------------------------------------------------------- surface points
// The step before the path (Methods, "Pocket prediction with P2Rank"):
// solvent-accessible surface points of the receptor and their Eq.
// prank_eq_1 features.  Atom records are float4 (x, y, z, type bits) with
// the expanded radius r = X-Score radius + probe computed in binary32.
constexpr int kSasThreads = 256;
constexpr int kSasWaves = kSasThreads / kWave;
constexpr int kSasList = 320;    // neighbours collected per atom before they are tested (above 4 waves' worth)

__device__ __forceinline__ float sas_radius(int t, float probe)
{
    const float R = t <= 1 ? 1.9f : (t <= 4 ? 1.8f : (t <= 6 ? 1.7f : 2.0f));
    return R + probe;
}

// candidate c = x_a + r_a u
__device__ __forceinline__ float3 sas_candidate(const float4& xa, float ra, const float* u)
{
    return make_float3(__builtin_fmaf(ra, u[0], xa.x), __builtin_fmaf(ra, u[1], xa.y), __builtin_fmaf(ra, u[2], xa.z));
}

// Which candidates c = x_a + r_a u_k lie strictly inside no other atom's
// expanded sphere, two atoms per wave.  Lanes run over the receptor and
// collect, per atom, those whose sphere can reach a candidate (the candidates
// lie within r_a max|u| of x_a; slack covers the rounding of their
// coordinates); the candidates then meet these alone, both atoms' side by side
// in the wave's halves when there are at most 32 directions, else 64
// directions of one atom at a time.  Bound by VALU issue: 13 instructions per
// atom and 64 atoms looked at, so the cost grows with n_rec^2 / 64 rather than
// n_rec^2 n_dirs.  8,000 atoms x 30 directions: 807 us when every candidate
// met every atom, 56 us now (36 us of them VALU issue); with the receptor
// staged in LDS tiles, one atom per wave, 85-102 us.
// Few atoms with many directions fill the chip with pieces of `per` chunks of 64
// directions (blockIdx.y), each of which collects the neighbours again: a wave
// that takes all of an atom's chunks is a serial chain of up to 128 tests of the
// list.  Writes the kept directions as bit masks (ceil(n_dirs / 64) words per
// atom) and their number by atom and piece.
constexpr int kSasAtoms = 2;

__global__ __launch_bounds__(kSasThreads) void sas_keep_kernel(const float4* atoms, int n_rec, const float* dirs,
                                                               int n_dirs, float probe, float umax, float slack,
                                                               int per, uint64_t* keep, int32_t* count)
{
    __shared__ float4 lists[kSasWaves][kSasAtoms][kSasList];
    const int l = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    float4(*list)[kSasList] = lists[wv];
    const int a0 = (int)(blockIdx.x * kSasWaves + wv) * kSasAtoms;
    if (a0 >= n_rec) return;
    float4 xa[kSasAtoms];
    float ra[kSasAtoms], reach2[kSasAtoms][4];   // squared reach by the neighbour's radius class
    int n[kSasAtoms];
    uint64_t buried[kSasAtoms];   // bit c: this lane's direction of chunk c
#pragma unroll
    for (int p = 0; p < kSasAtoms; ++p) {
        xa[p] = atoms[min(a0 + p, n_rec - 1)];
        ra[p] = sas_radius(__float_as_uint(xa[p].w) & 0xff, probe);
        n[p] = 0;
        buried[p] = 0;
        const int first[4] = {0, 2, 5, 7};   // a type of each class
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float thr = fmaf(ra[p], umax, slack) + sas_radius(first[e], probe);
            // a square that could overflow becomes NaN, which takes every atom
            reach2[p][e] = thr > 1e18f ? __builtin_nanf("") : thr * thr * 1.0001f;
        }
    }
    const bool packed = n_dirs <= kWave / 2;
    const int chunks = (n_dirs + kWave - 1) / kWave;   // at most 64 (PV_MAX_SAS_DIRS)
    const int c0 = (int)blockIdx.y * per, nc = min(per, chunks - c0);   // this piece's, at least one
    auto test = [&]() {
        wave_sync();
        for (int pass = 0; pass < (packed ? 1 : kSasAtoms * nc); ++pass) {
            const int p = packed ? l / (kWave / 2) : pass / nc, c = packed ? 0 : c0 + pass % nc;
            const int k = packed ? l % (kWave / 2) : c * kWave + l;
            const float4 xp = p ? xa[1] : xa[0];
            const float3 x = sas_candidate(xp, p ? ra[1] : ra[0], dirs + 3 * min(k, n_dirs - 1));
            const int np = p ? n[1] : n[0], nj = packed ? max(n[0], n[1]) : np;
            bool in = false;
#pragma unroll 4
            for (int j = 0; j < nj; ++j) {
                const float4 b = list[p][j];
                const float ex = x.x - b.x, ey = x.y - b.y, ez = x.z - b.z;
                in |= __builtin_fmaf(ex, ex, __builtin_fmaf(ey, ey, ez * ez)) < b.w && j < np;
            }
            if (p == 0) buried[0] |= (uint64_t)in << c;
            else buried[1] |= (uint64_t)in << c;
        }
        n[0] = n[1] = 0;
        wave_sync();
    };
    for (int base = 0; base < n_rec; base += 4 * kWave) {
        float4 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = base + u * kWave + l;
            t[u] = b < n_rec ? atoms[b] : make_float4(__builtin_inff(), 0.f, 0.f, 0.f);   // past the end: far
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = base + u * kWave + l, ty = __float_as_uint(t[u].w) & 0xff;
#pragma unroll
            for (int p = 0; p < kSasAtoms; ++p) {
                const float dx = xa[p].x - t[u].x, dy = xa[p].y - t[u].y, dz = xa[p].z - t[u].z;
                const float thr2 = ty <= 1 ? reach2[p][0] : ty <= 4 ? reach2[p][1] : ty <= 6 ? reach2[p][2] : reach2[p][3];
                const bool near = !(dx * dx + dy * dy + dz * dz >= thr2);
                const uint64_t m = __ballot(near);
                if (!m) continue;
                if (near) {
                    const float rb = sas_radius(ty, probe);
                    list[p][n[p] + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                        make_float4(t[u].x, t[u].y, t[u].z, b == a0 + p ? -1.f : rb * rb);   // itself buries nothing
                }
                n[p] += __popcll(m);
            }
        }
        // test the lists when the next four loads could overflow them, and at the end
        if (max(n[0], n[1]) > kSasList - 4 * kWave || base + 4 * kWave >= n_rec) test();
    }
#pragma unroll
    for (int p = 0; p < kSasAtoms; ++p) {
        if (a0 + p >= n_rec) break;
        int total = 0;
        for (int c = c0; c < c0 + nc; ++c) {
            uint64_t m;
            if (packed)
                m = (__ballot(!(buried[p] & 1)) >> (p * (kWave / 2))) & ((1ull << n_dirs) - 1);
            else
                m = __ballot(c * kWave + l < n_dirs && !((buried[p] >> c) & 1));
            if (l == 0) keep[(int64_t)(a0 + p) * chunks + c] = m;
            total += __popcll(m);
        }
        if (l == 0) count[(int64_t)(a0 + p) * gridDim.y + blockIdx.y] = total;
    }
}

// Exclusive sum of the n counts in place; the total goes to count[n].
// One workgroup, a run of consecutive counts per thread.
__global__ __launch_bounds__(1024) void sas_scan_kernel(int32_t* count, int n)
{
    __shared__ int wave_n[1024 / kWave];
    const int t = threadIdx.x, per = (n + 1023) / 1024;
    const int b = min(t * per, n), e = min(b + per, n);
    int sum = 0;
#pragma unroll 8
    for (int i = b; i < e; ++i) sum += count[i];
    int incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if ((t & (kWave - 1)) >= o) incl += v;
    }
    if ((t & (kWave - 1)) == kWave - 1) wave_n[t / kWave] = incl;
    __syncthreads();
    int off = incl - sum, all = 0;
    for (int w = 0; w < 1024 / kWave; ++w) {
        off += w < t / kWave ? wave_n[w] : 0;
        all += wave_n[w];
    }
#pragma unroll 8
    for (int i = b; i < e; ++i) {
        const int c = count[i];
        count[i] = off;
        off += c;
    }
    if (t == 0) count[n] = all;
}

// The kept candidates in (atom, direction) order, one wave per atom and piece.
__global__ __launch_bounds__(kSasThreads) void sas_scatter_kernel(const float4* atoms, int n_rec, const float* dirs,
                                                                  int n_dirs, float probe, int pieces, int per,
                                                                  const uint64_t* keep, const int32_t* offset,
                                                                  float4* pts)
{
    const int l = threadIdx.x & (kWave - 1), w = blockIdx.x * kSasWaves + threadIdx.x / kWave;
    if (w >= n_rec * pieces) return;
    const int a = w / pieces, c0 = w % pieces * per;
    const float4 xa = atoms[a];
    const float ra = sas_radius(__float_as_uint(xa.w) & 0xff, probe);
    const int chunks = (n_dirs + kWave - 1) / kWave;
    int off = offset[w];
    for (int c = c0; c < min(c0 + per, chunks); ++c) {
        const uint64_t m = keep[(int64_t)a * chunks + c];
        if ((m >> l) & 1) {
            const float3 x = sas_candidate(xa, ra, dirs + 3 * (c * kWave + l));
            pts[off + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                make_float4(x.x, x.y, x.z, __int_as_float(a));
        }
        off += __popcll(m);
    }
}

// Point records (x, y, z, atom bits) into separate arrays (either may be NULL).
__global__ __launch_bounds__(kSasThreads) void sas_split_kernel(const float4* pts, int n_pts, float* xyz, int32_t* atom)
{
    const int p = blockIdx.x * kSasThreads + threadIdx.x;
    if (p >= n_pts) return;
    const float4 v = pts[p];
    if (xyz) { xyz[3 * (int64_t)p] = v.x; xyz[3 * (int64_t)p + 1] = v.y; xyz[3 * (int64_t)p + 2] = v.z; }
    if (atom) atom[p] = __float_as_int(v.w);
}

// Eq. prank_eq_1 per point: channels 0..7 the one-hot XS type, 8..10 the
// hydrophobic, donor and acceptor flags, each summing max(0, 1 - d/6) over
// atoms with d^2 < 36; channel 11 counts the atoms with d^2 < 100 (the
// protrusion).  One wave per kSasPoints points, lanes over atoms, four loads
// in flight; the weights are summed only where some lane has an atom within
// 6 A, the flags are sums of their types' channels.  Bound by VALU issue (ten
// instructions per point and 64 atoms).  6,439 points x 8,000 atoms: 765 us
// with one point per thread, which filled 26 of the 256 CUs, 39 us now.
constexpr int kSasPoints = 2;

__global__ __launch_bounds__(kSasThreads) void sas_features_kernel(const float4* atoms, int n_rec, const float4* pts,
                                                                   int n_pts, float* feat)
{
    const int l = threadIdx.x & (kWave - 1);
    const int p0 = (int)__builtin_amdgcn_readfirstlane(blockIdx.x * kSasWaves + threadIdx.x / kWave) * kSasPoints;
    if (p0 >= n_pts) return;
    float4 c[kSasPoints];
    float f[kSasPoints][8];
    int near[kSasPoints];
#pragma unroll
    for (int p = 0; p < kSasPoints; ++p) {
        c[p] = pts[min(p0 + p, n_pts - 1)];
        near[p] = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) f[p][k] = 0.f;
    }
    for (int base = 0; base < n_rec; base += 4 * kWave) {
        float4 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = base + u * kWave + l;
            t[u] = b < n_rec ? atoms[b] : make_float4(__builtin_inff(), 0.f, 0.f, 0.f);   // past the end: far
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int p = 0; p < kSasPoints; ++p) {
                const float dx = c[p].x - t[u].x, dy = c[p].y - t[u].y, dz = c[p].z - t[u].z;
                const float d2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
                near[p] += __popcll(__ballot(d2 < 100.f));
                if (__ballot(d2 < 36.f)) {
                    const float w = d2 < 36.f ? 1.f - __builtin_amdgcn_sqrtf(d2) * (1.f / 6.f) : 0.f;
                    const int ty = __float_as_uint(t[u].w) & 0xff;
#pragma unroll
                    for (int k = 0; k < 8; ++k) f[p][k] += ty == k ? w : 0.f;
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < kSasPoints; ++p) {
#pragma unroll
        for (int k = 0; k < 8; ++k) f[p][k] = wsum(f[p][k]);
        if (p0 + p < n_pts && l < 12) {
            float v = l == 8 ? f[p][0] : l == 9 ? f[p][3] + f[p][6] : l == 10 ? f[p][4] + f[p][5] + f[p][6] : (float)near[p];
#pragma unroll
            for (int k = 0; k < 8; ++k) v = l == k ? f[p][k] : v;
            feat[(int64_t)(p0 + p) * 12 + l] = v;
        }
    }
}

// ---------------------------------------------------------------- allocation-free scratch
// The allocation-free dock entry point keeps its scratch (kNoAllocBytes,
// laid out by noalloc_layout) in this array.  Each GPU the library runs on
// holds its own copy until the process ends.  Host code never passes the
// array's name to a kernel: it takes the device address that
// hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

hipError_t noalloc_scratch(void** out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    *out = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

// Stable split of the jobs into the two size classes, in chunks of 1024:
// a ballot per wave ranks the members of each class inside the wave, and
// the waves' counts, added in wave order, place them after the earlier
// chunks.  Also zeroes the classes' queue counters.
__global__ __launch_bounds__(1024) void class_map_kernel(const int2* jobs, int n_jobs, const DevLig* ligs,
                                                         int n_small, int32_t* map, uint32_t* queues)
{
    __shared__ int wn0[16], wn1[16];
    const int t = threadIdx.x, w = t / kWave;
    if (t < 2) queues[t] = 0u;
    int base0 = 0, base1 = n_small;
    for (int c = 0; c < n_jobs; c += 1024) {
        const int j = c + t;
        const bool valid = j < n_jobs;
        const bool big = valid && ligs[jobs[j].x].n_atoms > 64;
        const bool small = valid && !big;
        const uint64_t ms = __ballot(small), mb = __ballot(big);
        if ((t & (kWave - 1)) == 0) { wn0[w] = __popcll(ms); wn1[w] = __popcll(mb); }
        __syncthreads();
        int off0 = 0, off1 = 0, tot0 = 0, tot1 = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int a = wn0[q], b = wn1[q];
            off0 += q < w ? a : 0;
            off1 += q < w ? b : 0;
            tot0 += a;
            tot1 += b;
        }
        const int r0 = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(ms >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ms, 0u));
        const int r1 = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mb >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mb, 0u));
        if (small) map[base0 + off0 + r0] = j;
        if (big) map[base1 + off1 + r1] = j;
        base0 += tot0;
        base1 += tot1;
        __syncthreads();   // every wave has read wn0 / wn1 before the next chunk writes them
    }
}

hipError_t launch_class_map(const int2* jobs, int32_t n_jobs, const DevLig* ligs, int32_t n_small, int32_t* map,
                            uint32_t* queues, hipStream_t s)
{
    hipLaunchKernelGGL(class_map_kernel, dim3(1), dim3(1024), 0, s, jobs, n_jobs, ligs, n_small, map, queues);
    return hipGetLastError();
}

// ---------------------------------------------------------------- launchers
hipError_t launch_build_grids(const GridBuildArgs& a, int64_t n_tiles, hipStream_t s)
{
    if (n_tiles <= 0) return hipSuccess;
    const int64_t runs = 8 * kGridRun;   // whole runs for every XCD; workgroups past the last tile return
    // a launch may not have 2^32 threads in a dimension: at most 2^20 workgroups each (whole runs, 8.6 GB of maps)
    constexpr int64_t kMost = (int64_t)1 << 20;
    GridBuildArgs b = a;
    for (int64_t first = 0; first < n_tiles; first += kMost) {
        const int64_t grid = (std::min<int64_t>(n_tiles - first, kMost) + runs - 1) / runs * runs;
        b.first_tile = (int32_t)first;
        hipLaunchKernelGGL(gridmap_kernel, dim3((unsigned)grid), dim3(kGridThreads), 0, s, b);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename K>
static int occupancy(K kernel, int lds, int threads = kWave)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds) != hipSuccess) {
        (void)hipGetLastError();   // answered by 0: the launch that follows must not report it
        return 0;
    }
    return n;
}

template <int A, bool SL>
static int kind_occupancy(int kind, int lds)
{
    if (kind == kKindDock) {   // the fewer of the history capacities' resident blocks
        return std::min(occupancy(dock_kernel<A, SL, kShortM>, lds), occupancy(dock_kernel<A, SL, kMaxM>, lds));
    }
    if (kind == kKindScore) return occupancy(score_kernel<A, SL>, lds);
    return occupancy(local_opt_kernel<A, SL>, lds);
}

static int lean_lds(int kind, const LigDev& l)
{
    return lds_bytes(l.max_atoms, l.max_pairs, l.max_ell, kernel_needs(kind, 1, false, true));
}

// The gather form's shape: of the lean kernels where three of their waves fit a SIMD.
static LaunchShape gather_shape(int kind, const LigDev& l, int lds, int occ)
{
    LaunchShape s = {1, lds, occ, false, occ};
    if (kind == kKindScore) return s;
    const int ll = lean_lds(kind, l);
    const int lean = kind == kKindOpt ? occupancy(local_opt_kernel<1, false, kLean>, ll)
                                      : std::min(occupancy(dock_kernel<1, false, kShortM, kLean>, ll),
                                                 occupancy(dock_kernel<1, false, kMaxM, kLean>, ll));
    s.lean = lean >= 12;
    if (s.lean) s.per_cu = lean;
    return s;
}

// Slots are faster per evaluation but take 16 B per pair end in LDS; they
// are used while the CUs can still hold as many of the launch's waves as the
// gather layout would at two waves per SIMD (a persistent launch over few chains, or small
// ligands), else the gather layout keeps the occupancy.
hipError_t launch_shape(int kind, const LigDev& l, int64_t items, int n_cu, LaunchShape* out)
{
    const int64_t cus = n_cu > 0 ? n_cu : 1;
    if (l.max_atoms > 64) {
        const int lds = lds_bytes(l.max_atoms, l.max_pairs, l.max_ell, kernel_needs(kind, 2, false));
        *out = {2, lds, kind_occupancy<2, false>(kind, lds), false, 0};
        return out->per_cu > 0 ? hipSuccess : hipErrorInvalidConfiguration;
    }
    const int lds_s = lds_bytes(l.max_atoms, l.max_pairs, l.max_ell, kernel_needs(kind, 1, true));
    const int lds_g = lds_bytes(l.max_atoms, l.max_pairs, l.max_ell, kernel_needs(kind, 1, false));
    const int occ_s = kind_occupancy<1, true>(kind, lds_s);
    const int occ_g = kind_occupancy<1, false>(kind, lds_g);
    const int64_t need = std::min<int64_t>(items > 0 ? items : 1, (int64_t)occ_g * cus);
    if (occ_s > 0 && (int64_t)occ_s * cus >= need)
        *out = {0, lds_s, occ_s, false, 0};
    else
        *out = gather_shape(kind, l, lds_g, occ_g);
    return out->per_cu > 0 ? hipSuccess : hipErrorInvalidConfiguration;
}

hipError_t launch_shape_variant(int kind, const LigDev& l, int variant, LaunchShape* out)
{
    *out = {variant, 0, 0, false, 0};
    if (variant < 0 || variant > 2 || (variant < 2 && l.max_atoms > 64)) return hipErrorInvalidValue;
    const int lds = lds_bytes(l.max_atoms, l.max_pairs, l.max_ell, kernel_needs(kind, variant == 2 ? 2 : 1, variant == 0));
    int occ;
    if (variant == 0) occ = kind_occupancy<1, true>(kind, lds);
    else if (variant == 1) occ = kind_occupancy<1, false>(kind, lds);
    else occ = kind_occupancy<2, false>(kind, lds);
    *out = {variant, lds, occ, false, 0};
    if (variant == 1 && occ > 0) *out = gather_shape(kind, l, lds, occ);
    return occ > 0 ? hipSuccess : hipErrorInvalidConfiguration;
}

hipError_t launch_score(const ScoreArgs& a, bool ragged, int n_cu, hipStream_t s)
{
    if (a.n_poses <= 0) return hipSuccess;
    LaunchShape sh;
    hipError_t e;
    if ((e = launch_shape(kKindScore, a.l, a.n_poses, n_cu, &sh)) != hipSuccess) return e;
    // One wave per slot the CUs can hold, each with a contiguous run of poses,
    // where the ligands are alike.  Where their sizes differ (pairs on average
    // below three quarters of the largest's) a run of large ligands would end
    // long after the others: up to 6 waves per slot, shorter runs, and a slot
    // takes the next run when it is free.  96 ligands of 8-80 atoms: 3,001 poses
    // 43 -> 40 us, 10,000 97 -> 88 us, 30,000 sorted by ligand 320 -> 225 us; but
    // 64 ligands of 40 atoms: 4,000 poses 22 -> 24 us, 16,384 61 -> 67 us.
    const int64_t cap = (int64_t)sh.per_cu * (n_cu > 0 ? n_cu : 1) * (ragged ? 6 : 1);
    const int grid = (int)(a.n_poses < cap ? a.n_poses : cap);
    if (sh.variant == 0)
        hipLaunchKernelGGL((score_kernel<1, true>), dim3(grid), dim3(64), sh.lds, s, a);
    else if (sh.variant == 1)
        hipLaunchKernelGGL((score_kernel<1, false>), dim3(grid), dim3(64), sh.lds, s, a);
    else
        hipLaunchKernelGGL((score_kernel<2, false>), dim3(grid), dim3(64), sh.lds, s, a);
    return hipGetLastError();
}

// Whether a launch's chains can have teams of W waves: all of them resident at
// once, and beside them as many equal launches of other streams as without teams,
// up to `side`, the four that a process's hardware queues run side by side (on the
// null stream, which callers of one stream use, itself alone).  Launches that
// no longer fit together run one after the other (chains of 60 steps, teams where
// one launch fits / one wave each / this rule):
//     20 atoms, 320 chains, three streams 16.0 / 12.4 / 10.9 ms; 500, two 15.7 / 12.2 / 10.9
//     20 atoms, 750 chains, two streams 19.7 / 12.8 / 10.6 ms; 35 atoms, 240, four 14.4 / - / 10.5
// One launch alone on such a stream pays where the smaller team is slower: 35 atoms,
// 320 chains 8.9 / 11.8 / 9.7 ms.
template <int MM, int W>
static bool team_fits(const LigDev& l, int64_t items, const LaunchShape& sh, int side, int n_cu)
{
    items *= std::min<int64_t>(side, std::max<int64_t>(1, (int64_t)sh.per_cu * n_cu / items));
    const int lds = sh.lds + team_bytes<W>(l.max_atoms, l.max_pairs);
    return (int64_t)occupancy(dock_kernel<1, true, MM, W>, lds, W * kWave) * n_cu >= items;
}

template <int MM, int W>
static void launch_slots(const DockArgs& a, const LaunchShape& sh, unsigned grid, hipStream_t s)
{
    const int lds = sh.lds + (W > 1 ? team_bytes<W>(a.l.max_atoms, a.l.max_pairs) : 0);
    hipLaunchKernelGGL((dock_kernel<1, true, MM, W>), dim3(grid), dim3(kWave, W), lds, s, a);
}

// Slot launches: teams where every chain is resident at once with its helpers (team_fits),
// with more than one chunk of pairs (fewer take no longer than the waits for the
// helpers: 16 atoms, 61 pairs, 1,024 chains 11.2 ms alone, 11.6 in teams of two),
// and with no other class's launch beside it.  Teams of four before teams of two,
// chains of 60 steps alone / of two / of four:
//     20 atoms, 122 pairs     8 chains 10.3 / 9.8 / 9.9 ms     256: 11.4 / 10.9 / 11.1
//     35 atoms, 445 pairs     8 chains 5.93 / 5.15 / 4.51      256: 9.32 / 8.08 / 7.22
//     64 atoms, 1,717 pairs   8 chains 7.88 / 6.14 / 4.66      256: 9.91 / 7.80 / 5.97
//     35 atoms, 1,024 chains 9.87 / 8.50 (no room for teams of four)
template <int MM>
static int team_waves(const LigDev& l, int64_t items, const LaunchShape& sh, unsigned grid, int side, int n_cu)
{
    if (!side || grid < items || l.max_pairs <= kWave) return 1;
    return team_fits<MM, 4>(l, items, sh, side, n_cu) ? 4 : team_fits<MM, 2>(l, items, sh, side, n_cu) ? 2 : 1;
}

int dock_waves(const LigDev& l, int m, int64_t items, const LaunchShape& sh, int32_t workgroups, int side, int n_cu)
{
    if (sh.variant != 0) return 1;
    return m <= kShortM ? team_waves<kShortM>(l, items, sh, (unsigned)workgroups, side, n_cu)
                        : team_waves<kMaxM>(l, items, sh, (unsigned)workgroups, side, n_cu);
}

template <int MM>
static void launch_slot_dock(const DockArgs& a, const LaunchShape& sh, unsigned grid, int side, int n_cu, hipStream_t s)
{
    const int waves = team_waves<MM>(a.l, a.n_items, sh, grid, side, n_cu);
    if (waves == 4) launch_slots<MM, 4>(a, sh, grid, s);
    else if (waves == 2) launch_slots<MM, 2>(a, sh, grid, s);
    else launch_slots<MM, 1>(a, sh, grid, s);
}

hipError_t launch_dock(const DockArgs& a, const LaunchShape& sh, int32_t workgroups, int side, int n_cu, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    const unsigned grid = a.persistent ? (unsigned)workgroups : (unsigned)a.n_items;
    const bool short_m = a.sp.m <= kShortM;
    if (sh.variant == 0) {
        if (short_m) launch_slot_dock<kShortM>(a, sh, grid, side, n_cu, s);
        else launch_slot_dock<kMaxM>(a, sh, grid, side, n_cu, s);
    } else if (sh.variant == 1 && sh.lean && grid > (int64_t)sh.full_cu * n_cu) {
        const int lds = lean_lds(kKindDock, a.l);
        if (short_m) hipLaunchKernelGGL((dock_kernel<1, false, kShortM, kLean>), dim3(grid), dim3(64), lds, s, a);
        else hipLaunchKernelGGL((dock_kernel<1, false, kMaxM, kLean>), dim3(grid), dim3(64), lds, s, a);
    } else if (sh.variant == 1) {
        if (short_m) hipLaunchKernelGGL((dock_kernel<1, false, kShortM>), dim3(grid), dim3(64), sh.lds, s, a);
        else hipLaunchKernelGGL((dock_kernel<1, false, kMaxM>), dim3(grid), dim3(64), sh.lds, s, a);
    } else {
        if (short_m) hipLaunchKernelGGL((dock_kernel<2, false, kShortM>), dim3(grid), dim3(64), sh.lds, s, a);
        else hipLaunchKernelGGL((dock_kernel<2, false, kMaxM>), dim3(grid), dim3(64), sh.lds, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_fma_peak(float* out, int n, int iters, hipStream_t s)
{
    hipLaunchKernelGGL(fma_peak_kernel, dim3((unsigned)(n / 256)), dim3(256), 0, s, out, iters);
    return hipGetLastError();
}

hipError_t launch_reset_queue(uint32_t* q, hipStream_t s)
{
    hipLaunchKernelGGL(reset_queue_kernel, dim3(1), dim3(64), 0, s, q);
    return hipGetLastError();
}

hipError_t launch_reset_times(uint64_t* t0, uint64_t* t1, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(reset_times_kernel, dim3((n + 255) / 256), dim3(256), 0, s, t0, t1, n);
    return hipGetLastError();
}

hipError_t launch_job_reduce(const float* cbe, const int64_t* cev, const int32_t* cst, int32_t n_jobs,
                             int32_t chains, float* jbe, int32_t* jbc, int64_t* jev, int32_t* jst, hipStream_t s)
{
    if (n_jobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(job_reduce_kernel, dim3((n_jobs + 255) / 256), dim3(256), 0, s, cbe, cev, cst, n_jobs, chains,
                       jbe, jbc, jev, jst);
    return hipGetLastError();
}

hipError_t launch_local_opt(const OptArgs& a, int n_cu, hipStream_t s)
{
    if (a.n_poses <= 0) return hipSuccess;
    LaunchShape sh;
    hipError_t e;
    if ((e = launch_shape(kKindOpt, a.l, a.n_poses, n_cu, &sh)) != hipSuccess) return e;
    const int grid = a.n_poses < 65536 ? a.n_poses : 65536;
    if (sh.variant == 0)
        hipLaunchKernelGGL((local_opt_kernel<1, true>), dim3(grid), dim3(64), sh.lds, s, a);
    else if (sh.variant == 1 && sh.lean && a.n_poses > (int64_t)sh.full_cu * n_cu)
        hipLaunchKernelGGL((local_opt_kernel<1, false, kLean>), dim3(grid), dim3(64), lean_lds(kKindOpt, a.l), s, a);
    else if (sh.variant == 1)
        hipLaunchKernelGGL((local_opt_kernel<1, false>), dim3(grid), dim3(64), sh.lds, s, a);
    else
        hipLaunchKernelGGL((local_opt_kernel<2, false>), dim3(grid), dim3(64), sh.lds, s, a);
    return hipGetLastError();
}

// Waves per job: the fewest rounds of refinements, times the rounds of workgroups
// that the CUs take to get through the jobs (a CU holds eight waves, two per SIMD,
// or as many workgroups as its LDS; a started round counts as three quarters of a
// whole one at least, since the jobs' lengths differ).  In rounds of refinements, a
// workgroup's serial parts count as 0.6 and the clustering of a chain as 0.02, shared
// by the waves; of numbers within 6% the most waves.  Few jobs so get all eight
// waves for the latency, and many jobs as many as keep every wave at work: jobs of
// 64-atom ligands x 32 chains of random poses, one / two / four / eight waves each:
//     120 x 20 modes 10.8 / 5.8 / 3.0 / 2.2 ms      1,000 x 20 modes 22.2 / 12.7 / 12.0 / 8.4 ms
//     1,500 x 5 modes 3.5 / 3.8 / 6.6 / 4.2 ms      6,000 x 3 modes 7.9 / 9.4 / 8.1 / 14.6 ms
// Four for every job count above the CUs took up to 1.9 times as long as one wave;
// by this rule no set of 8 to 128 atoms x 120 to 6,000 jobs x 3 to 20 modes, on
// random and on docked poses, takes above 3% longer than with one wave, and all of
// them on average 2% longer than with their best number.
static int output_waves(const OutputArgs& a, int n_cu, int lds_per_block)
{
    double cost[kOutWaves + 1], least = 0.0;
    int top = 0;
    for (int w = 1; w <= kOutWaves; ++w) {
        const int lds = output_lds_bytes(a.l, a.chains, a.modes, w);
        if (w > 1 && lds > lds_per_block) break;
        const int held = std::max(1, std::min(kOutWaves / w, lds_per_block / lds)) * std::max(n_cu, 1);
        const double x = (double)a.n_jobs / held, rounds = x > 1.0 ? 0.75 * std::ceil(x) + 0.25 * x : 1.0 + 0.05 * x;
        cost[w] = rounds * ((std::min(a.modes, a.chains) + w - 1) / w + 0.6 + 0.02 * a.chains / w);
        if (w == 1 || cost[w] < least) least = cost[w];
        top = w;
    }
    while (cost[top] > 1.06 * least) --top;
    return top;
}

hipError_t launch_output(const OutputArgs& a, int n_cu, int lds_per_block, hipStream_t s)
{
    if (a.n_jobs <= 0) return hipSuccess;
    const int waves = output_waves(a, n_cu, lds_per_block);
    const int lds = output_lds_bytes(a.l, a.chains, a.modes, waves);
    if (a.l.max_atoms <= 64)
        hipLaunchKernelGGL((output_kernel<1>), dim3(a.n_jobs), dim3(kWave, waves), lds, s, a);
    else
        hipLaunchKernelGGL((output_kernel<2>), dim3(a.n_jobs), dim3(kWave, waves), lds, s, a);
    return hipGetLastError();
}

int output_lds_bytes(const LigDev& l, int chains, int modes, int waves)
{
    const int ma = lds_atoms(l.max_atoms);
    return waves * lds_bytes(l.max_atoms, l.max_pairs, l.max_ell, kernel_needs(kKindOutput, l.max_atoms > 64 ? 2 : 1, false)) +
           round_up(chains, 4) * 4 + modes * ma * 16 + modes * kSlot * 4 + 5 * round_up(modes, 4) * 4;
}

// Pieces of a whole number of chunks until the keep kernel has eight waves per CU:
// 20 atoms x 4,096 directions 286 -> 103 us for the call, 500 x 4,096 606 -> 171.
int sas_pieces(int n_rec, int n_dirs, int n_cu)
{
    const int chunks = (n_dirs + kWave - 1) / kWave, waves = n_rec / kSasAtoms + 1;
    const int want = std::min(chunks, (8 * std::max(n_cu, 1) + waves - 1) / waves);
    const int per = (chunks + want - 1) / want;
    return (chunks + per - 1) / per;   // none of them empty
}

static int sas_per(int n_dirs, int pieces)
{
    return ((n_dirs + kWave - 1) / kWave + pieces - 1) / pieces;
}

hipError_t launch_sas_keep(const float4* atoms, int n_rec, const float* dirs, int n_dirs, float probe, float umax,
                           float slack, int pieces, uint64_t* keep, int32_t* count, hipStream_t s)
{
    if (n_rec > 0) {
        hipLaunchKernelGGL(sas_keep_kernel, dim3((n_rec + kSasWaves * kSasAtoms - 1) / (kSasWaves * kSasAtoms), pieces),
                           dim3(kSasThreads), 0, s, atoms, n_rec, dirs, n_dirs, probe, umax, slack,
                           sas_per(n_dirs, pieces), keep, count);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(sas_scan_kernel, dim3(1), dim3(1024), 0, s, count, n_rec * pieces);
    return hipGetLastError();
}

hipError_t launch_sas_scatter(const float4* atoms, int n_rec, const float* dirs, int n_dirs, float probe, int pieces,
                              const uint64_t* keep, const int32_t* offset, float4* pts, hipStream_t s)
{
    if (n_rec <= 0) return hipSuccess;
    hipLaunchKernelGGL(sas_scatter_kernel, dim3((n_rec * pieces + kSasWaves - 1) / kSasWaves), dim3(kSasThreads), 0, s,
                       atoms, n_rec, dirs, n_dirs, probe, pieces, sas_per(n_dirs, pieces), keep, offset, pts);
    return hipGetLastError();
}

hipError_t launch_sas_split(const float4* pts, int n_pts, float* xyz, int32_t* atom, hipStream_t s)
{
    if (n_pts <= 0 || (!xyz && !atom)) return hipSuccess;
    hipLaunchKernelGGL(sas_split_kernel, dim3((n_pts + kSasThreads - 1) / kSasThreads), dim3(kSasThreads), 0, s, pts,
                       n_pts, xyz, atom);
    return hipGetLastError();
}

hipError_t launch_sas_features(const float4* atoms, int n_rec, const float4* pts, int n_pts, float* feat,
                               hipStream_t s)
{
    if (n_pts <= 0) return hipSuccess;
    const int per = kSasWaves * kSasPoints;
    hipLaunchKernelGGL(sas_features_kernel, dim3((n_pts + per - 1) / per), dim3(kSasThreads), 0, s, atoms, n_rec, pts,
                       n_pts, feat);
    return hipGetLastError();
}

}  // namespace pv
