// HIP kernels for gfx950 of the three-dimensional (D3Q19) binary Shan-Chen capillary: the 3-D
// extension the paper names as future work (Conclusions), with the step of Sec. 2 written for
// D3Q19: equilibrium w_i n (1 + 3 c.u + 9/2 (c.u)^2 - 3/2 u.u) with w = 1/3, 1/18 (axis),
// 1/36 (edge); bulk force -G psi_k sum_i w_i psi_kbar(x + c_i) c_i (psi = n, 0 on solids); wall
// force -G_kw n_k sum_i w_i s(x + c_i) c_i; common velocity U and shifted equilibrium; BGK;
// pull streaming with half-way bounce-back.  The z-projection of these weights is D2Q9 with rest
// fraction 4/9, so z-independent states follow the 2-D model.
//
// The fused step (k3_fused) walks y-slices of x-z tiles with the densities in an LDS ring; the
// two-kernel variant (k3_density, k3_collide) writes a density field and reads it back.
// Storage: FP32, f[k][i][z][y][pitch], x fastest, pitch = nx rounded up to 64.
#include "scf3d_internal.h"

#include <algorithm>

// Every multiply-add is written out (no implicit contraction), as in the 2-D kernels.
#pragma clang fp contract(off)

namespace scf3 {
namespace {

constexpr int kThreads = 256;

// D3Q19 velocities: rest, six axis links, twelve edge links.
constexpr __constant__ int kCX[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
constexpr __constant__ int kCY[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
constexpr __constant__ int kCZ[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
constexpr __constant__ int kOpp[19] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};

// Interaction weights of the links (rest excluded): 1/18 (axis), 1/36 (edge).
constexpr float kWA = 1.0f / 18.0f;
constexpr float kWE = 1.0f / 36.0f;
// 3 w_i for the odd part of the equilibrium: 1/6 (axis) and 1/12 (edge), with 1/6 carried as
// two terms (a single rounded constant would bias the equilibrium momentum at every step).
constexpr float kSixthHi = 1.0f / 6.0f;
constexpr float kSixthLo = (float)(1.0 / 6.0 - (double)kSixthHi);

__device__ __forceinline__ float sixth(float v) { return __builtin_fmaf(v, kSixthHi, v * kSixthLo); }

__device__ __forceinline__ int wrapc(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// v + d on the periodic axis of n nodes, d in {-1, 0, 1}.
__device__ __forceinline__ int wrap_step(int v, int d, int n) {
    return d > 0 ? (v == n - 1 ? 0 : v + 1) : d < 0 ? (v == 0 ? n - 1 : v - 1) : v;
}

__device__ __forceinline__ bool in_x(const Chan3& c, int x) { return (unsigned)(x - c.x0) < (unsigned)(c.x1 - c.x0); }

// Row (y, z) is solid over the capillary; a row whose neighbours may be.
__device__ __forceinline__ bool wall_row(const Chan3& c, int y, int z) {
    return (c.walls_y && (y == 0 || y == c.ny - 1)) || (c.walls_z && (z == 0 || z == c.nz - 1));
}
__device__ __forceinline__ bool near_wall_row(const Chan3& c, int y, int z) {
    return (c.walls_y && (y <= 1 || y >= c.ny - 2)) || (c.walls_z && (z <= 1 || z >= c.nz - 2));
}

__device__ __forceinline__ bool solid(const Chan3& c, int x, int y, int z) { return wall_row(c, y, z) && in_x(c, x); }

// Directions (bits) whose component along an axis (0 x, 1 y, 2 z) is d.
constexpr uint32_t dirs_along(int axis, int d) {
    constexpr int C[3][19] = {{0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0},
                              {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1},
                              {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1}};
    uint32_t m = 0;
    for (int i = 0; i < 19; ++i) m |= C[axis][i] == d ? 1u << i : 0u;
    return m;
}

// Solid-neighbourhood code of node (x, y, z): bit i is set when x + c_i is solid (bit 0: the node
// itself).  Population i streams in from x - c_i and bounces back when bit opp(i) is set.
__device__ __forceinline__ uint32_t solid_code(const Chan3& c, int x, int y, int z) {
    if (!near_wall_row(c, y, z)) return 0u;
    uint32_t mx = 0, mw = 0;
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
        const int xn = wrap_step(x, d, c.nx), yn = wrap_step(y, d, c.ny), zn = wrap_step(z, d, c.nz);
        mx |= in_x(c, xn) ? dirs_along(0, d) : 0u;
        mw |= c.walls_y && (yn == 0 || yn == c.ny - 1) ? dirs_along(1, d) : 0u;
        mw |= c.walls_z && (zn == 0 || zn == c.nz - 1) ? dirs_along(2, d) : 0u;
    }
    return mx & mw;
}

__device__ __forceinline__ int64_t idx(const Chan3& c, int x, int y, int z) {
    return ((int64_t)z * c.ny + y) * c.pitch + x;
}

// Buffer-descriptor access: one descriptor per component of a buffer (19 planes) of at most 4 GiB,
// unsigned 32-bit byte offsets.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const float* base, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)(uint32_t)bytes, 0x00020000);
}
__device__ __forceinline__ float bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ unsigned row_bytes(const Chan3& c, int y, int z) {
    return ((unsigned)z * (unsigned)c.ny + (unsigned)y) * (unsigned)c.pitch * 4u;
}

// The populations of a buffer, by descriptors.
struct Pops {
    __amdgpu_buffer_rsrc_t A, B;
    unsigned Pb;   // plane bytes
    __device__ __forceinline__ Pops(const Chan3& c, const float* ws, int b) {
        const float* g = ws + c.off + (int64_t)b * 38 * c.plane;
        const int64_t bytes = (int64_t)19 * c.plane * 4;
        A = make_rsrc(g, bytes);
        B = make_rsrc(g + 19 * c.plane, bytes);
        Pb = (unsigned)(c.plane * 4);
    }
};

// Populations f_i(x, t) of both components streaming into (x, y, z), whose solid code is `code`.
// UNIFORM: y and z are the same in every lane of the wave, so the row offsets are scalar.
template <bool UNIFORM>
__device__ __forceinline__ void pull(const Pops& g, const Chan3& c, int x, int y, int z, uint32_t code, float f[38]) {
    const unsigned xo[3] = {(unsigned)wrap_step(x, -1, c.nx) * 4u, (unsigned)x * 4u, (unsigned)wrap_step(x, 1, c.nx) * 4u};
    const unsigned own = row_bytes(c, y, z) + xo[1];
    if (__any(code != 0u)) {
#pragma unroll
        for (int i = 0; i < 19; ++i) {
            // bounce-back lanes read their own node's opposite direction: the plane goes into the
            // per-lane offset
            const unsigned row = row_bytes(c, wrap_step(y, -kCY[i], c.ny), wrap_step(z, -kCZ[i], c.nz)) + (unsigned)i * g.Pb;
            const unsigned o = i > 0 && ((code >> kOpp[i]) & 1u) ? own + (unsigned)kOpp[i] * g.Pb : xo[1 - kCX[i]] + row;
            f[i] = bload(g.A, o, 0u);
            f[19 + i] = bload(g.B, o, 0u);
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const unsigned row = row_bytes(c, wrap_step(y, -kCY[i], c.ny), wrap_step(z, -kCZ[i], c.nz)) + (unsigned)i * g.Pb;
        const unsigned xs = xo[1 - kCX[i]];
        f[i] = UNIFORM ? bload(g.A, xs, row) : bload(g.A, xs + row, 0u);
        f[19 + i] = UNIFORM ? bload(g.B, xs, row) : bload(g.B, xs + row, 0u);
    }
}

// The same by 64-bit addresses, for components above 4 GiB.
__device__ __forceinline__ void pull_wide(const float* __restrict__ g, const Chan3& c, int x, int y, int z, uint32_t code,
                                          float f[38]) {
    const int64_t own = idx(c, x, y, z);
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const bool back = i > 0 && ((code >> kOpp[i]) & 1u);
        const int64_t at = back ? kOpp[i] * c.plane + own
                                : i * c.plane + idx(c, wrap_step(x, -kCX[i], c.nx), wrap_step(y, -kCY[i], c.ny),
                                                    wrap_step(z, -kCZ[i], c.nz));
        f[i] = g[at];
        f[19 + i] = g[19 * c.plane + at];
    }
}

template <bool UNIFORM, bool WIDE>
__device__ __forceinline__ void pull_from(const Chan3& c, const float* ws, int b, int x, int y, int z, uint32_t code,
                                          float f[38]) {
    if (WIDE) pull_wide(ws + c.off + (int64_t)b * 38 * c.plane, c, x, y, z, code, f);
    else pull<UNIFORM>(Pops(c, ws, b), c, x, y, z, code, f);
}

__device__ __forceinline__ float sum19(const float* f) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 19; ++i) s += f[i];
    return s;
}

// The two-kernel step works on rows: a wave's 64 nodes lie on one row (y, z), so row addresses,
// periodic wraps in y and z and the rows' wall tests are scalar.  Blocks of four waves cover 256
// nodes of a row, or several rows where a row has fewer.  With EIGHTHS XCD k (blocks b = k mod 8) takes
// the k-th contiguous eighth of the rows, so that the densities of the rows around a row, which nine rows
// read, come from one L2; see by_eighths.
struct Row {
    int x, y, z;
    bool in;
};

template <bool EIGHTHS>
__device__ __forceinline__ Row row_of(const Chan3& c) {
    const int wpr = min((c.nx + 63) / 64, kThreads / 64), per_block = kThreads / 64 / wpr;   // waves a row, rows a block
    const int segs = (c.nx + kThreads - 1) / kThreads;
    const int nb = gridDim.x, blk = blockIdx.x, xcd = blk & 7, per = nb >> 3, rem = nb & 7;
    const int b = EIGHTHS ? xcd * per + min(xcd, rem) + (blk >> 3) : blk;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t row = (uint32_t)(b / segs) * per_block + wave / wpr, rows = (uint32_t)c.ny * (uint32_t)c.nz;   // < 2^32
    Row r;
    r.x = (b % segs) * kThreads + (wave % wpr) * 64 + (threadIdx.x & 63);
    r.in = wave < wpr * per_block && row < rows && r.x < c.nx;
    r.z = __builtin_amdgcn_readfirstlane((int)(row / (uint32_t)c.ny));
    r.y = __builtin_amdgcn_readfirstlane((int)(row - (uint32_t)r.z * (uint32_t)c.ny));
    return r;
}

__device__ __forceinline__ int64_t row_at(const Chan3& c, int y, int z) { return ((int64_t)z * c.ny + y) * c.pitch; }

template <bool WIDE, bool EIGHTHS>
__global__ void __launch_bounds__(kThreads)
k3_density(const Chan3 c, float* __restrict__ ws, int src) {
    const Row r = row_of<EIGHTHS>(c);
    if (!r.in) return;
    const uint32_t code = solid_code(c, r.x, r.y, r.z);
    float* __restrict__ dn = ws + c.off + 76 * c.plane + row_at(c, r.y, r.z);
    float f[38];
    pull_from<true, WIDE>(c, ws, src, r.x, r.y, r.z, code, f);
    dn[r.x] = code & 1u ? 0.0f : sum19(f);
    dn[c.plane + r.x] = code & 1u ? 0.0f : sum19(f + 19);
}

// c_i . u and the accumulation of v c_i, without the terms of zero components: the sums of the
// others come in the same order, so finite values are the same bit for bit.
__device__ __forceinline__ float signed_of(int c, float v) { return c > 0 ? v : -v; }

__device__ __forceinline__ float along(int i, float ux, float uy, float uz) {
    float s = 0.0f;
    bool any = false;
    if (kCX[i]) { s = signed_of(kCX[i], ux); any = true; }
    if (kCY[i]) { s = any ? s + signed_of(kCY[i], uy) : signed_of(kCY[i], uy); any = true; }
    if (kCZ[i]) s = any ? s + signed_of(kCZ[i], uz) : signed_of(kCZ[i], uz);
    return s;
}

__device__ __forceinline__ void add_along(int i, float v, float s[3]) {
    if (kCX[i]) s[0] += signed_of(kCX[i], v);
    if (kCY[i]) s[1] += signed_of(kCY[i], v);
    if (kCZ[i]) s[2] += signed_of(kCZ[i], v);
}

// Deviation-form BGK of one component: D_i = (w_i n - f_i) + n w_i (3 c.u + 9/2 (c.u)^2 - 3/2 u.u)
// for i > 0, D_0 = -sum D_i; out(q, f*) takes f*_i = f_i + omega D_i.
template <class Out>
__device__ __forceinline__ void relax(const float* f, float n, float ux, float uy, float uz, float om, const Out& out,
                                      int qbase) {
    const float usq = __builtin_fmaf(ux, ux, __builtin_fmaf(uy, uy, uz * uz));
    float sumD = 0.0f;
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        const float cu = along(i, ux, uy, uz);
        const bool axis = i < 7;
        const float w = axis ? kWA : kWE;
        const float odd = axis ? sixth(cu) : 0.5f * sixth(cu);            // 3 w_i c.u
        const float even = w * __builtin_fmaf(4.5f * cu, cu, -1.5f * usq);  // w_i (9/2 cu^2 - 3/2 u^2)
        const float D = __builtin_fmaf(n, odd + even, w * n - f[i]);
        sumD += D;
        out(qbase + i, __builtin_fmaf(om, D, f[i]));
        if (i % 3 == 0) __builtin_amdgcn_sched_barrier(0);
    }
    out(qbase, __builtin_fmaf(om, -sumD, f[0]));
}

// Forces, common velocity and collision of a node with pulled populations f and densities nA, nB;
// out(q, v) takes population q (B's from 19), neighbour(i, a, b) gives the densities at x + c_i.  The
// scheduling barriers keep the neighbour loads and the two relaxations from being spread over each
// other: the walk holds two slices of populations, and its registers decide how many blocks a CU
// takes.
template <class Out, class N>
__device__ __forceinline__ void collide(const Chan3& c, const float* f, float nA, float nB, uint32_t code, const Out& out,
                                        N neighbour) {
    float jA[3] = {0.0f, 0.0f, 0.0f}, jB[3] = {0.0f, 0.0f, 0.0f};
    float sA[3] = {0.0f, 0.0f, 0.0f}, sB[3] = {0.0f, 0.0f, 0.0f}, sw[3] = {0.0f, 0.0f, 0.0f};
    if (__any(code != 0u)) {
#pragma unroll
        for (int i = 1; i < 19; ++i) add_along(i, (code >> i) & 1u ? (i < 7 ? kWA : kWE) : 0.0f, sw);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        add_along(i, f[i], jA);
        add_along(i, f[19 + i], jB);
        const float w = i < 7 ? kWA : kWE;
        float a, b;
        neighbour(i, a, b);
        add_along(i, w * a, sA);
        add_along(i, w * b, sB);
        if (i % 6 == 0) __builtin_amdgcn_sched_barrier(0);
    }
    // accelerations a_k = F_k / n_k
    float aA[3], aB[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        aA[q] = __builtin_fmaf(-c.G, sB[q], -(c.gw[0] * sw[q]));
        aB[q] = __builtin_fmaf(-c.G, sA[q], -(c.gw[1] * sw[q]));
    }
    const float inv = 1.0f / __builtin_fmaf(c.wm[0], nA, c.wm[1] * nB);
    float U[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) U[q] = __builtin_fmaf(c.wm[0], jA[q], c.wm[1] * jB[q]) * inv;
    relax(f, nA, __builtin_fmaf(c.tm[0], aA[0], U[0]), __builtin_fmaf(c.tm[0], aA[1], U[1]),
          __builtin_fmaf(c.tm[0], aA[2], U[2]), c.omega[0], out, 0);
    __builtin_amdgcn_sched_barrier(0);
    relax(f + 19, nB, __builtin_fmaf(c.tm[1], aB[0], U[0]), __builtin_fmaf(c.tm[1], aB[1], U[1]),
          __builtin_fmaf(c.tm[1], aB[2], U[2]), c.omega[1], out, 19);
}

template <bool WIDE, bool NT, bool EIGHTHS>
__global__ void __launch_bounds__(kThreads)
k3_collide(const Chan3 c, float* __restrict__ ws, int src) {
    const Row r = row_of<EIGHTHS>(c);
    if (!r.in) return;
    const int x = r.x, y = r.y, z = r.z;
    const uint32_t code = solid_code(c, x, y, z);
    if (code & 1u) return;
    const int xs[3] = {wrap_step(x, -1, c.nx), x, wrap_step(x, 1, c.nx)};
    float f[38], a[19], b[19];
    pull_from<true, WIDE>(c, ws, src, x, y, z, code, f);
    // all neighbour densities with the populations: small boxes have one wave per SIMD, which waited
    // for them in three more turns
    const float* __restrict__ field = ws + c.off + 76 * c.plane;
    const __amdgpu_buffer_rsrc_t fr = make_rsrc(field, (int64_t)2 * c.plane * 4);
    const unsigned Pb = (unsigned)(c.plane * 4);
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        const int yn = wrap_step(y, kCY[i], c.ny), zn = wrap_step(z, kCZ[i], c.nz), xn = xs[1 + kCX[i]];
        if (WIDE) {
            const float* n = field + row_at(c, yn, zn);
            a[i] = n[xn];
            b[i] = n[c.plane + xn];
        } else {
            const unsigned at = __builtin_amdgcn_readfirstlane(row_bytes(c, yn, zn));
            a[i] = bload(fr, (unsigned)xn * 4u, at);
            b[i] = bload(fr, (unsigned)xn * 4u, at + Pb);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const float nA = sum19(f), nB = sum19(f + 19);
    float* __restrict__ d = ws + c.off + (int64_t)(src ^ 1) * 38 * c.plane + row_at(c, y, z);
    const Pops to(c, ws, src ^ 1);
    const unsigned row = __builtin_amdgcn_readfirstlane(row_bytes(c, y, z));
    collide(c, f, nA, nB, code,
            [&](int q, float v) {
                if (WIDE)
                    __builtin_nontemporal_store(v, d + q * c.plane + x);
                else
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), q < 19 ? to.A : to.B, x * 4,
                                                          (int)(row + (unsigned)(q % 19) * Pb), NT ? 2 : 0);
            },
            [&](int i, float& p, float& q) {
                p = a[i];
                q = b[i];
            });
}

// ---------------------------------------------------------------------------------------------
// Fused 3-D step (the walk).  A block of BX x BZ threads (BX a multiple of 64) owns the columns x in
// [xb, xb + BX), z in [zb, zb + BZ) and walks rows y upward through [yb, ye).  Iteration `it` pulls
// one y-slice of the tile plus its one-node halo ring in x and z, writes the slice's densities into
// a 4-slot LDS ring, and after one barrier collides the previous slice, whose populations were kept
// in registers: all 18 neighbour densities of a node come from three ring slots.  The first and
// last slices pulled are density-only halos.  A slot written at iteration it+1 was last read by the
// collision of iteration it-1, finished by every thread before the barrier of iteration it.
//
// A wave's 64 nodes lie on one row (y, z), so the row offsets of a pull, its periodic wraps and the
// wall tests of its rows are scalar; per lane there are three byte offsets (x - 1, x, x + 1).  The
// ring's z rows are pulled by waves 0 .. 2 BX / 64 - 1, its x columns and corners by the next wave.
// What it waits for are the lines that reach L2 from beyond it: the node's own 304 bytes, the z rows and
// x columns of the ring, 352 bytes per node at 5.1 TB/s with the 23 rows per tile that 512 x 182 x 182
// takes (501 at 5.6 on the former 64 x 4 tiles).  Two slices of populations take 76 registers; the rest
// fits into 128 but for one (64 x 8: three), which lets 16 waves share a CU (157 registers and three
// blocks of 64 x 4 before: 1.52 ms per step of 512 x 182 x 182, 11.2 GLUPS; now 1.17 ms, 14.5).
// ---------------------------------------------------------------------------------------------
// A value the compiler may not reason about: keeps what is derived from it inside the loop, where
// recomputing it costs a few instructions and holding it a register for the whole walk.
__device__ __forceinline__ int here_s(int v) {
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ int here_v(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Densities of a node pulled for its densities only (0 on solid nodes).
template <bool UNIFORM>
__device__ __forceinline__ void halo_node(const Pops& g, const Chan3& c, int x, int y, int z, float& nA, float& nB) {
    const uint32_t code = solid_code(c, x, y, z);
    float h[38];
    pull<UNIFORM>(g, c, x, y, z, code, h);
    nA = code & 1u ? 0.0f : sum19(h);
    nB = code & 1u ? 0.0f : sum19(h + 19);
}

template <int BX, int BZ, bool NT>
__global__ void __launch_bounds__(BX * BZ) __attribute__((amdgpu_waves_per_eu(4)))
k3_fused(const Chan3 c, float* __restrict__ ws, int src, int cy) {
    constexpr int SX = BX + 2, SZ = BZ + 2, WX = BX / 64, NX = 2 * SZ;   // NX: x columns and corners
    static_assert(BX % 64 == 0 && NX <= 64 && BZ * WX > 2 * WX, "one wave for the columns after the z rows");
    __shared__ float sn[2][4][SZ][SX];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tz = wave / WX, tx = (wave % WX) * 64 + lane;
    // Workgroups are dispatched to the eight XCDs in turn (block b to XCD b mod 8), each XCD with
    // its own L2.  Give XCD k the k-th contiguous eighth of the tiles (x fastest, then z, then
    // the row chunk), so that the tiles whose halos overlap share one L2.
    const int gx = (c.nx + BX - 1) / BX, gz = (c.nz + BZ - 1) / BZ;
    const int ntiles = gridDim.x;
    const int blk = blockIdx.x, xcd = blk & 7, per = ntiles >> 3, rem = ntiles & 7;
    const int t = xcd * per + min(xcd, rem) + (blk >> 3);
    const int xb = (t % gx) * BX, zb = ((t / gx) % gz) * BZ;
    const int yb = (t / gx / gz) * cy, ye = min(yb + cy, c.ny);
    // Tile columns past the edge of the box hold the periodic images of nodes (as many times over
    // as needed when the box is narrower than the tile), so the LDS neighbours of every active
    // column are the true periodic neighbours; only active threads collide and store.
    const bool act = xb + tx < c.nx && zb + tz < c.nz;
    const int x0 = (xb + tx) % c.nx, z0 = (zb + tz) % c.nz;
    // this wave's part of the halo ring: a stretch of a z row (UNIFORM), the x columns, or none
    const int part = wave < 2 * WX ? 0 : wave == 2 * WX ? 1 : 2;
    const int hz = part == 0 ? (wave < WX ? 0 : SZ - 1) : lane < SZ ? lane : lane - SZ;
    const int hx = part == 0 ? tx + 1 : lane < SZ ? 0 : SX - 1;
    const Pops g(c, ws, src), d(c, ws, src ^ 1);
    float q[38];
#pragma unroll
    for (int i = 0; i < 38; ++i) q[i] = 0.0f;
    float qA = 0.0f, qB = 0.0f;
    uint32_t qcode = 0;
    int y = wrapc(yb - 1, c.ny);
    const int niter = ye - yb + 2;
    for (int it = 0; it < niter; ++it) {
        const int slot = it & 3;
        // the halo ring first, so that its registers are free again before the slice's own pull
        if (part < 2 && (part == 0 || lane < NX)) {
            const int xh = (xb - 1 + here_v(hx) + c.nx) % c.nx;
            float hA, hB;
            if (part == 0) halo_node<true>(g, c, xh, y, (zb - 1 + here_s(hz) + c.nz) % c.nz, hA, hB);
            else halo_node<false>(g, c, xh, y, (zb - 1 + here_v(hz) + c.nz) % c.nz, hA, hB);
            sn[0][slot][hz][hx] = hA;
            sn[1][slot][hz][hx] = hB;
        }
        const int x = here_v(x0), z = here_s(z0);
        float p[38];
        float nA = 0.0f, nB = 0.0f;
        const uint32_t code = solid_code(c, x, y, z);
        pull<true>(g, c, x, y, z, code, p);
        if (!(code & 1u)) {
            nA = sum19(p);
            nB = sum19(p + 19);
        }
        sn[0][slot][tz + 1][tx + 1] = nA;
        sn[1][slot][tz + 1][tx + 1] = nB;
        __syncthreads();
        const int yc = here_s(y == 0 ? c.ny - 1 : y - 1);   // the slice pulled one iteration ago
        if (it >= 2 && act && !(qcode & 1u)) {
            const float* lA[3];
            const float* lB[3];   // this node in slices yc - 1, yc, yc + 1
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                lA[k] = &sn[0][(it + 2 + k) & 3][tz + 1][tx + 1];
                lB[k] = &sn[1][(it + 2 + k) & 3][tz + 1][tx + 1];
            }
            const unsigned row = row_bytes(c, yc, z);
            collide(c, q, qA, qB, qcode,
                    [&](int k, float v) {
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), k < 19 ? d.A : d.B, x * 4,
                                                              (int)(row + (unsigned)(k < 19 ? k : k - 19) * d.Pb), NT ? 2 : 0);
                    },
                    [&](int i, float& a, float& b) {
                        a = lA[kCY[i] + 1][kCZ[i] * SX + kCX[i]];
                        b = lB[kCY[i] + 1][kCZ[i] * SX + kCX[i]];
                    });
        }
#pragma unroll
        for (int i = 0; i < 38; ++i) q[i] = p[i];
        qA = nA;
        qB = nB;
        qcode = code;
        y = y == c.ny - 1 ? 0 : y + 1;
    }
}

// Initial state: the resident buffer holds the populations whose pull is the rest equilibrium
// w_i n0(x): g_i(x) = w_i n0(x + c_i) if x + c_i is fluid, else w_i n0(x).  The FP64 host
// fields (nz*ny*nx each) are staged in population buffer 1.
__global__ void __launch_bounds__(kThreads)
k3_init(const Chan3* __restrict__ cp, float* __restrict__ ws) {
    const Chan3 c = *cp;
    const int x = blockIdx.x * kThreads + threadIdx.x, y = blockIdx.y, z = blockIdx.z;
    if (x >= c.nx) return;
    const double* __restrict__ rho = reinterpret_cast<const double*>(ws + c.off + 38 * c.plane);
    float* __restrict__ g = ws + c.off;
    const int64_t cells = (int64_t)c.nx * c.ny * c.nz;
    const bool sol = solid(c, x, y, z);
    const int64_t at = idx(c, x, y, z);
    for (int k = 0; k < 2; ++k) {
        const double* rk = rho + k * cells;
        const double n0 = rk[((int64_t)z * c.ny + y) * c.nx + x] * (double)c.inv_m[k];
        for (int i = 0; i < 19; ++i) {
            const float w = i == 0 ? 1.0f / 3.0f : (i < 7 ? kWA : kWE);
            const int xn = wrapc(x + kCX[i], c.nx), yn = wrapc(y + kCY[i], c.ny), zn = wrapc(z + kCZ[i], c.nz);
            double nn = n0;
            if (!solid(c, xn, yn, zn)) nn = rk[((int64_t)zn * c.ny + yn) * c.nx + xn] * (double)c.inv_m[k];
            g[(k * 19 + i) * c.plane + at] = sol ? 0.0f : w * (float)nn;
        }
    }
}

// Pulled populations f(t) of every node into buffer 1 - src.
__global__ void __launch_bounds__(kThreads)
k3_pull_out(const Chan3* __restrict__ cp, float* __restrict__ ws, int src) {
    const Chan3 c = *cp;
    const int x = blockIdx.x * kThreads + threadIdx.x, y = blockIdx.y, z = blockIdx.z;
    if (x >= c.nx) return;
    const float* __restrict__ g = ws + c.off + (int64_t)src * 38 * c.plane;
    float* __restrict__ o = ws + c.off + (int64_t)(src ^ 1) * 38 * c.plane;
    float f[38];
    const bool sol = solid(c, x, y, z);
    if (!sol) pull_wide(g, c, x, y, z, solid_code(c, x, y, z), f);
    const int64_t at = idx(c, x, y, z);
#pragma unroll
    for (int i = 0; i < 38; ++i) o[i * c.plane + at] = sol ? 0.0f : f[i];
}

// Observables from the density field (k3_density first): FP64 mass per (y, z) row and a health
// flag, then one block sums the rows in order and finds the centre-line front.  Block reductions
// run in a fixed order: a butterfly over each wave's 64 lanes, then the wave results through LDS.
constexpr int kWaves = kThreads / 64;
// One block sums every row's partials and searches the centre line, a serial chain of loads per
// thread: 1024 threads (512 x 182 x 182: 15 us for 39 with 256), one barrier for all reductions.
constexpr int kFinalThreads = 1024, kFinalWaves = kFinalThreads / 64;

template <typename T>
__device__ __forceinline__ T wsum(T v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ int wmin(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
    return v;
}

__global__ void __launch_bounds__(kThreads)
k3_obs_rows(const Chan3* __restrict__ cp, const float* __restrict__ ws, Part3* __restrict__ parts) {
    __shared__ double sd[2][kWaves];
    __shared__ int si[kWaves];
    const Chan3 c = *cp;
    const int y = blockIdx.x, z = blockIdx.y;
    const float* __restrict__ nAf = ws + c.off + 76 * c.plane;
    const float* __restrict__ nBf = nAf + c.plane;
    double mA = 0.0, mB = 0.0;
    int bad = 0;
    for (int x = threadIdx.x; x < c.nx; x += kThreads) {
        if (solid(c, x, y, z)) continue;
        const float a = nAf[idx(c, x, y, z)], b = nBf[idx(c, x, y, z)];
        mA += (double)a;
        mB += (double)b;
        if (!(a >= -1e-3f) || !(b >= -1e-3f) || !isfinite(a) || !isfinite(b)) bad = 1;
    }
    mA = wsum(mA);
    mB = wsum(mB);
    bad = wsum(bad);
    if ((threadIdx.x & 63) == 0) {
        sd[0][threadIdx.x >> 6] = mA;
        sd[1][threadIdx.x >> 6] = mB;
        si[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWaves; ++w) {
            mA += sd[0][w];
            mB += sd[1][w];
            bad += si[w];
        }
        Part3 p;
        p.mass[0] = mA;
        p.mass[1] = mB;
        p.bad = bad;
        p.pad = 0;
        parts[(int64_t)z * c.ny + y] = p;
    }
}

__global__ void __launch_bounds__(kFinalThreads)
k3_obs_final(const Chan3* __restrict__ cp, const float* __restrict__ ws, const Part3* __restrict__ parts,
             Obs3* __restrict__ out) {
    __shared__ double sd[2][kFinalWaves];
    __shared__ int si[2][kFinalWaves];
    const Chan3 c = *cp;
    const int tid = threadIdx.x;
    const float* __restrict__ nAf = ws + c.off + 76 * c.plane;
    const float* __restrict__ nBf = nAf + c.plane;
    double mA = 0.0, mB = 0.0;
    int bad = 0;
    for (int r = tid; r < c.ny * c.nz; r += kFinalThreads) {
        mA += parts[r].mass[0];
        mB += parts[r].mass[1];
        bad |= parts[r].bad;
    }
    // centre line: the (up to) four lines nearest (y, z) = ((ny-1)/2, (nz-1)/2)
    const int ys[2] = {(c.ny - 1) / 2, c.ny / 2}, zs[2] = {(c.nz - 1) / 2, c.nz / 2};
    auto phi = [&](int x) -> double {
        double v = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b)
                v += 0.25 * ((double)nAf[idx(c, x, ys[a], zs[b])] - (double)nBf[idx(c, x, ys[a], zs[b])]);
        return v;
    };
    const int big = 0x7fffffff;
    int xz = big;
    const int xs0 = c.x0 / 2;
    for (int x = xs0 + tid; x + 1 < c.nx; x += kFinalThreads)
        if (phi(x) >= 0.0 && phi(x + 1) < 0.0) xz = min(xz, x);
    mA = wsum(mA);
    mB = wsum(mB);
    bad = wsum(bad);
    xz = wmin(xz);
    if ((tid & 63) == 0) {
        sd[0][tid >> 6] = mA;
        sd[1][tid >> 6] = mB;
        si[0][tid >> 6] = bad;
        si[1][tid >> 6] = xz;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kFinalWaves; ++w) {
            mA += sd[0][w];
            mB += sd[1][w];
            bad += si[0][w];
            xz = min(xz, si[1][w]);
        }
        Obs3 o;
        o.t = 0;
        o.mass[0] = mA;
        o.mass[1] = mB;
        if (xz == big) {
            o.z = __builtin_nan("");
        } else {
            const double a = phi(xz), b = phi(xz + 1);
            o.z = (double)xz + a / (a - b) - (double)c.x0;
        }
        o.flags = (phi(xs0) < 0.0 ? 1 : 0) | (bad ? 2 : 0);
        o.reserved = 0;
        *out = o;
    }
}

// The density field without padding into `out` (n_A, then n_B): FP64 as the caller's arrays have it, or
// FP32 for half the way to the host.
template <class T>
__global__ void __launch_bounds__(kThreads)
k3_density_out(Chan3 c, const float* __restrict__ ws, T* __restrict__ out) {
    const int64_t row = (int64_t)blockIdx.y * c.ny + blockIdx.x, cells = (int64_t)c.nx * c.ny * c.nz;
    const float* __restrict__ n = ws + c.off + 76 * c.plane + row * c.pitch;
    T* o = out + row * c.nx;
    for (int x = threadIdx.x; x < c.nx; x += kThreads) {
        o[x] = n[x];
        o[cells + x] = n[c.plane + x];
    }
}

// Blocks of the row kernels (row_of).
int row_blocks(const Chan3& c) {
    const int wpr = std::min((c.nx + 63) / 64, kThreads / 64), per_block = kThreads / 64 / wpr;
    const int64_t rows = (int64_t)c.ny * c.nz, segs = (c.nx + kThreads - 1) / kThreads;
    return (int)((rows + per_block - 1) / per_block * segs);
}

dim3 grid_of(const Chan3& c) { return dim3((c.nx + kThreads - 1) / kThreads, c.ny, c.nz); }

// Both buffers' nodes beyond the 256 MB last-level cache: the stores of a step then go past L2,
// which keeps the walk's halos (512 x 182 x 182: 1.39 ms per step for 1.49), and cost boxes that
// fit what the next step would have found (200 x 60 x 60: 72 us for 65).
bool streams(const Chan3& c) { return (int64_t)304 * c.nx * c.ny * c.nz > ((int64_t)256 << 20); }

bool wide(const Chan3& c) { return !fused_fits(c.plane); }

// Rows by XCD eighths (row_of), or all XCDs side by side: then the z planes around a row are still in the
// last-level cache that the XCDs share, where eighths keep eight sets of planes there (us per step,
// eighths and side by side: 96 x 24 x 24 11.0 and 12.9, 256 x 128 x 64 187 and 193, 300 x 120 x 90 384 and
// 399, 500 x 60 x 182 519 and 503, 512 x 182 x 182 1593 and 1528, 512 x 340 x 340 5640 and 5440).
// Boxes of 64-bit addresses count as past the line.
bool by_eighths(const Chan3& c) { return (int64_t)c.nx * c.ny * c.nz < 4000000; }

void density(const Chan3& h, float* ws, int src, hipStream_t s) {
    const dim3 grid(row_blocks(h)), block(kThreads);
    if (wide(h)) hipLaunchKernelGGL((k3_density<true, false>), grid, block, 0, s, h, ws, src);
    else if (by_eighths(h)) hipLaunchKernelGGL((k3_density<false, true>), grid, block, 0, s, h, ws, src);
    else hipLaunchKernelGGL((k3_density<false, false>), grid, block, 0, s, h, ws, src);
}

int64_t walk_tiles(const Chan3& c, int bx, int bz, int cy) {
    return (int64_t)((c.nx + bx - 1) / bx) * ((c.nz + bz - 1) / bz) * ((c.ny + cy - 1) / cy);
}

template <int BX, int BZ>
hipError_t launch_walk(const Chan3& h, float* ws, int src, int cy, hipStream_t s) {
    const int64_t n = walk_tiles(h, BX, BZ, cy);
    if (n > INT32_MAX) return hipErrorInvalidConfiguration;
    if (streams(h)) hipLaunchKernelGGL((k3_fused<BX, BZ, true>), dim3((unsigned)n), dim3(BX * BZ), 0, s, h, ws, src, cy);
    else hipLaunchKernelGGL((k3_fused<BX, BZ, false>), dim3((unsigned)n), dim3(BX * BZ), 0, s, h, ws, src, cy);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_init(const Chan3& h, const Chan3* c, float* ws, hipStream_t s) {
    hipLaunchKernelGGL(k3_init, grid_of(h), dim3(kThreads), 0, s, c, ws);
    return hipGetLastError();
}

hipError_t launch_step(const Chan3& h, float* ws, int src, hipStream_t s) {
    density(h, ws, src, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(row_blocks(h)), block(kThreads);
    if (wide(h)) hipLaunchKernelGGL((k3_collide<true, true, false>), grid, block, 0, s, h, ws, src);
    else if (!by_eighths(h)) hipLaunchKernelGGL((k3_collide<false, true, false>), grid, block, 0, s, h, ws, src);
    else if (streams(h)) hipLaunchKernelGGL((k3_collide<false, true, true>), grid, block, 0, s, h, ws, src);
    else hipLaunchKernelGGL((k3_collide<false, false, true>), grid, block, 0, s, h, ws, src);
    return hipGetLastError();
}

// The walk's tiles.  Registers allow 16 waves per CU: one block of 256 x 4, or two of 128 x 4 or
// 64 x 8.  Wider tiles have fewer x-halo columns, which cost a cache line for each population of
// one node (256 x 4 with 23 rows: 1.18 ms per step of 512 x 182 x 182, 128 x 4 1.22, 64 x 8 1.26),
// unless the box leaves their columns idle.
namespace {
struct Walk {
    int bx, bz, per_cu;
    double speed;
};
constexpr Walk kWalks[3] = {{256, 4, 1, 1.0}, {128, 4, 2, 0.97}, {64, 8, 2, 0.94}};

// Row iterations of a launch (of 1024 nodes per CU each), weighted by the shape's speed: whole
// rounds of blocks, two density-only slices per tile.
double walk_cost(const Chan3& c, const Walk& w, int cy, int cus) {
    const int64_t slots = (int64_t)std::max(cus, 1) * w.per_cu;
    return (double)((walk_tiles(c, w.bx, w.bz, cy) + slots - 1) / slots) * (cy + 2) / w.speed;
}
}  // namespace

hipError_t launch_step_fused(const Chan3& h, float* ws, int src, int cy, int cus, hipStream_t s) {
    cy = cy < 1 ? 1 : (cy > h.ny ? h.ny : cy);
    int best = 0;
    for (int k = 1; k < 3; ++k)
        if (walk_cost(h, kWalks[k], cy, cus) < walk_cost(h, kWalks[best], cy, cus)) best = k;
    // so few tiles that a CU gets one of 128 x 4 at most: these have half the threads, and an iteration of
    // one alone is shorter (300 x 120 x 90 in 60 rows 444 us for 575 with 256 x 4, 40 x 100 x 30 in 4 rows 33
    // for 50, 512 x 8 x 8 in single rows 17 for 22)
    if (walk_tiles(h, 128, 4, cy) <= cus) best = 1;
    switch (best) {
        case 0: return launch_walk<256, 4>(h, ws, src, cy, s);
        case 1: return launch_walk<128, 4>(h, ws, src, cy, s);
        default: return launch_walk<64, 8>(h, ws, src, cy, s);
    }
}

// A walk's iteration takes about 16 us at full CUs and the two kernels 95 ps per node (LLC-resident
// boxes 80): 96 x 24 x 24 11.7 us per step with two kernels, 27 with the walk at its best; 256 x 128
// x 64 188 and 203; 300 x 120 x 90 384 and 273; 512 x 182 x 182 1528 and 1168.  Returns the rows per
// tile, 0 for the two kernels.
int best_schedule(const Chan3& h, int cus) {
    if (wide(h)) return 0;
    double best = 95e-6 * h.nx * (double)h.ny * h.nz;
    int rows = 0;
    for (int k = 1; k <= h.ny; ++k) {
        const int cy = (h.ny + k - 1) / k;
        if (cy < 4) break;
        for (const Walk& w : kWalks) {
            const double t = 16.0 * walk_cost(h, w, cy, cus);
            if (t < best) {
                best = t;
                rows = cy;
            }
        }
    }
    return rows;
}

hipError_t launch_observe(const Chan3& h, const Chan3* c, float* ws, int src, Part3* parts, Obs3* out,
                          hipStream_t s) {
    density(h, ws, src, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k3_obs_rows, dim3(h.ny, h.nz), dim3(kThreads), 0, s, c, ws, parts);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k3_obs_final, dim3(1), dim3(kFinalThreads), 0, s, c, ws, parts, out);
    return hipGetLastError();
}

hipError_t launch_density_out(const Chan3& h, const float* ws, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k3_density_out<double>, dim3(h.ny, h.nz), dim3(kThreads), 0, s, h, ws, out);
    return hipGetLastError();
}

hipError_t launch_density_out(const Chan3& h, const float* ws, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k3_density_out<float>, dim3(h.ny, h.nz), dim3(kThreads), 0, s, h, ws, out);
    return hipGetLastError();
}

hipError_t launch_pull_out(const Chan3& h, const Chan3* c, float* ws, int src, hipStream_t s) {
    hipLaunchKernelGGL(k3_pull_out, grid_of(h), dim3(kThreads), 0, s, c, ws, src);
    return hipGetLastError();
}

}  // namespace scf3
