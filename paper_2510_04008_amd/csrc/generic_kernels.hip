// Generic RACE Attention passes: any (L, P <= 8, d <= 256, d % 8 == 0; P = 8: d <= 152), fp32 or bf16 tensors, all arithmetic in fp32
// (the contractions on the fp32 matrix instructions, v_mfma_f32_16x16x4_f32).  This family serves the fp32 element type
// and every bf16 shape the bf16 MFMA family has no instantiation for.
//
// Decomposition.  The sequence is cut into tiles of C = 16 RT tokens and segments of one or more tiles; a workgroup of
// four wavefronts owns one segment.  Per tile, Algorithm 2 in its chunked form:
//     O_i = [ Phi_Q(i) S  +  sum_{j <= i in the tile} (Phi_Q(i) . Phi_K(j)) V_j ] / (the same with V = 1)
// with S the statistics [B | A] of all earlier tiles, so nothing inside a tile is sequential and a short sequence is one
// round of small independent workgroups.  The L R bucket rows are taken as one flat axis in blocks of 64 (whole tables,
// or a share of one table for R > 64); an output accumulates over the blocks in registers, so no per-table partial
// result ever goes to memory.
//
// What bounds it: at the sizes it serves (small layers) the number of dependent launches and the latency of one
// workgroup, hence three launches forward (totals with the hashing, scan, output), three backward (totals, scan, all
// three gradients), tiles of 16 tokens until they fill the chip, and all loads of a tile requested together.  Measured
// forward + backward (B = H = 1, N = 1024, d = 64, L = P = 4, fp32, not causal): 337 us with a token-at-a-time kernel per
// table, 41 with the loads of a tile under conditions, one trip to memory after the other, 34 now (B = 2, H = 4, N = 2003, causal:
// 96 -> 79; bf16, B = 2, H = 8, N = 1024, d = 32: 76 -> 62; fp32, B = 2, H = 4, N = 3501, d = 128, L = 6, P = 5: 477 -> 360).
//
// Matrix operand layouts (lane = 16 q + n): A: row n, k = q; B: column n, k = q; C/D: column n, rows 4 q + v in register v.
// Four consecutive k-steps take k = 4 q + v, v = 0..3, so that an operand whose k axis runs along a row of LDS is one
// 16-byte read, and a D tile [rows][columns] is itself the B operand (k = its rows) of a following product.
// LDS row strides are 4 (mod 8) words: 16-byte row reads of 16 rows and 4-byte reads of 4 x 16 consecutive words both
// touch every bank once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"

namespace race {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kThreads = 256;
constexpr int KB = 64;          // bucket rows per block
constexpr int PHS = KB + 4;     // row stride of an assignment tile
constexpr int CSS = 33;         // row stride of the hashed rows of a block (at most 32 hyperplanes: R <= 2 gives 32 tables)
constexpr int DZS = 36;         // row stride of the dz tiles

struct bf16_t { uint16_t bits; };

// The thread's number, hidden from the optimiser: addresses and conditions that derive from it are worked out where they are
// used.  (Hoisted out of the loops over tiles and blocks they took 200 scalar and 100 vector registers of the gradient kernel.)
__device__ __forceinline__ int thread_id()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t & (kThreads - 1);
}
// the same for a value that is the same in all lanes
__device__ __forceinline__ int uniform(int x)
{
    asm volatile("" : "+s"(x));
    return x;
}
// this wavefront's number, as the uniform value that it is
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

__device__ __forceinline__ float load1(const float *p) { return *p; }
__device__ __forceinline__ float load1(const bf16_t *p) { return __uint_as_float(static_cast<uint32_t>(p->bits) << 16); }
// four consecutive elements of a caller's tensor, which need be aligned to its elements only (a view into a larger buffer);
// the wide loads stay one instruction: global memory takes them at any address
typedef f32x4 __attribute__((aligned(4))) f32x4_of_elements;
typedef __attribute__((ext_vector_type(2), aligned(2))) uint32_t u32x2_of_elements;
__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4_of_elements *>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t *p)
{
    const u32x2_of_elements w = *reinterpret_cast<const u32x2_of_elements *>(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                 __uint_as_float(w.y & 0xffff0000u)};
}
__device__ __forceinline__ void store1(float *p, float v) { *p = v; }
__device__ __forceinline__ void store1(bf16_t *p, float v)
{
    uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) > 0x7f800000u) { p->bits = 0x7fc0; return; }      // NaN
    b += 0x7fffu + ((b >> 16) & 1u);                                        // nearest even
    p->bits = static_cast<uint16_t>(b >> 16);
}
__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// fp64 form: same operand layout, D: column n, rows q + 4 v
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 lds4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }

struct GArgs {
    int H, BH, L, P, R, d, dp, LP, LR;  // dp: d rounded up to 16
    int TB;                             // tables per block of 64 bucket rows (1 if a table spans blocks)
    int bpt;                            // blocks per table (1 unless R > 64)
    int nblk, PB;                       // blocks, hyperplanes per block
    int nseg, tps, causal, unit;
    int64_t N;
    float beta;
    size_t ST;                          // floats per saved state: B [LR][d], A [LR], padded
    const float *W;                     // (H, L P, d)
    float *Cq, *Ck, *Zq, *Zk;           // (BH, N, L P): hashed rows (see code()) and projections
    float *nrm;                         // (2, BH, N): 1 / max(|x|, floor) of the rows of Q and K (unit-norm option)
    float *carry;                       // (BH, nseg, ST): running statistics inside a segment of several tiles (the second set of
                                        // states: scratch of the forward pass and of dQ's; dK's and dV's carries its own on in place)
};

// The same arguments with their sizes hidden from the optimiser (see thread_id()): a loop body that starts with this works out
// its conditions itself.
__device__ __forceinline__ GArgs fresh(GArgs a)
{
    a.d = uniform(a.d); a.dp = uniform(a.dp); a.L = uniform(a.L); a.P = uniform(a.P); a.R = uniform(a.R); a.LP = uniform(a.LP);
    a.LR = uniform(a.LR); a.TB = uniform(a.TB); a.bpt = uniform(a.bpt); a.PB = uniform(a.PB); a.causal = uniform(a.causal);
    a.unit = uniform(a.unit);
    return a;
}

// first table and hyperplane of a block; tables of the block that exist
__device__ __forceinline__ int block_table(const GArgs &a, int b) { return a.bpt > 1 ? b / a.bpt : b * a.TB; }
__device__ __forceinline__ int block_rtiles(const GArgs &a, int b)
{
    const int left = a.LR - b * KB;
    return left >= KB ? 4 : (left + 15) >> 4;
}

// Unit-norm option: rows shorter than the floor are divided by the floor (a zero row stays zero).
constexpr float kUnitFloor = 1e-12f;

// The hashed form of a projection: +-small, small = sigmoid(-2 beta |tanh z|) the mass of the bit's minor side, the sign
// bit set where z < 0 (the major side is -1).  beta = +infinity gives +-0, the hard hash (at z = 0 the NaN of -inf * 0
// is dropped by fmaxf and the bit counts as set).
// The exponent 2 beta |tanh z| is large exactly where tanh is close to one, and a rounded fp32 product would be off by its
// last place (5e-7 at beta = 8, in every saturated bit alike): tanh there is 1 - 2 w with w = e2 / (1 + e2), e2 = exp(-2 |z|),
// and what the rounding of 1 - 2 w and of the product leaves over goes into the exponential as a factor.
__device__ __forceinline__ float code(float z, float beta)
{
    const float az = fabsf(z), e2 = expf(-2.0f * az), w = e2 / (1.0f + e2), b2 = -2.0f * beta;
    float hi = 1.0f - 2.0f * w, lo = (1.0f - hi) - 2.0f * w;
    if (az < 0.55f) { hi = tanhf(az); lo = 0.f; }
    const float p = b2 * hi, r = p > -1e4f ? fmaf(b2, lo, fmaf(b2, hi, -p)) : 0.f;
    float e = expf(fmaxf(p, -1e30f));
    e = fmaf(e, r, e);
    const float small = e / (1.0f + e);
    return z >= 0.f ? small : -small;
}
__device__ __forceinline__ float mass_of(float c, int bit)      // mass on the +1 (bit = 1) or -1 side
{
    const bool minor1 = (__float_as_uint(c) >> 31) != 0;        // the minor side is +1
    return (minor1 == (bit != 0)) ? fabsf(c) : 1.0f - fabsf(c);
}

// Loads of a tile.  All of them are unconditional, at addresses clamped into the tensors, and go to registers first (fetch_*)
// and to LDS later (put_*): what a tile needs is requested together and costs one trip to memory.  (A load under a condition
// is a branch, and the compiler waits for the loads before it: the passes spent three to five such trips of about a
// microsecond one after the other, 3.5 us before the first product of the gradients.)
// 16 / RT threads share a row of the tile; thread `sub` of them takes columns 4 (sub + k 16 / RT) ..
template <int RT>
struct RowThread {
    static constexpr int TPR = kThreads / (16 * RT);
    int row, sub;
    __device__ RowThread()
    {
        const int t = thread_id();
        row = t / TPR;
        sub = t % TPR;
    }
    __device__ int column(int k) const { return 4 * (sub + k * TPR); }
};
template <int RT, int NCT>
struct RowRegs { f32x4 v[RT * NCT]; };
template <typename T, int RT, int NCT>
__device__ __forceinline__ void fetch_rows(const GArgs &a, const T *X, size_t row0, int nv, RowRegs<RT, NCT> &r)
{
    const RowThread<RT> t;
    const T *src = X + (row0 + (t.row < nv ? t.row : nv - 1)) * a.d;
#pragma unroll
    for (int k = 0; k < RT * NCT; ++k) r.v[k] = load4(src + (t.column(k) < a.d ? t.column(k) : 0));
}
// ... into xs [C][XS]; rows >= nv and columns >= d are zeros
template <int RT, int NCT>
__device__ __forceinline__ void put_rows(const GArgs &a, const RowRegs<RT, NCT> &r, int nv, float *xs, int XS)
{
    const RowThread<RT> t;
#pragma unroll
    for (int k = 0; k < RT * NCT; ++k) {
        const int c = t.column(k);
        if (c < a.dp) *reinterpret_cast<f32x4 *>(xs + t.row * XS + c) = (t.row < nv && c < a.d) ? r.v[k] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// Read-out cotangents g = dO / e (e = L Den) into gs and ge[row] = -(g . O): the cotangents of the un-averaged numerator
// and normaliser of Algorithm 1, step 7.
template <int RT, int NCT>
struct CotRegs {
    RowRegs<RT, NCT> g, o;
    float den;
};
template <typename T, int RT, int NCT>
__device__ __forceinline__ void fetch_cotangents(const GArgs &a, const T *dO, const T *O, const float *den, size_t row0, int nv, CotRegs<RT, NCT> &r)
{
    const RowThread<RT> t;
    r.den = den[row0 + (t.row < nv ? t.row : nv - 1)];
    fetch_rows<T, RT, NCT>(a, O, row0, nv, r.o);
    fetch_rows<T, RT, NCT>(a, dO, row0, nv, r.g);
}
template <int RT, int NCT>
__device__ __forceinline__ void put_cotangents(const GArgs &a, const CotRegs<RT, NCT> &r, int nv, float *gs, int XS, float *ge)
{
    const RowThread<RT> t;
    // (Den = 0: the forward pass leaves O = 0 there, a constant; so does an underflow of every bucket mass the query sees)
    const float e = t.row < nv ? r.den * static_cast<float>(a.L) : 0.f, inv = e != 0.f ? 1.0f / e : 0.f;
    float dot = 0.f;
#pragma unroll
    for (int k = 0; k < RT * NCT; ++k) {
        const int c = t.column(k);
        f32x4 g = {0.f, 0.f, 0.f, 0.f};
        if (t.row < nv && c < a.d) {
            const f32x4 o = r.o.v[k];
            g = r.g.v[k] * inv;
            dot = fmaf(g.x, o.x, fmaf(g.y, o.y, fmaf(g.z, o.z, fmaf(g.w, o.w, dot))));
        }
        if (c < a.dp) *reinterpret_cast<f32x4 *>(gs + t.row * XS + c) = g;
    }
#pragma unroll
    for (int m = 1; m < RowThread<RT>::TPR; m <<= 1) dot += __shfl_xor(dot, m, 64);
    if (t.sub == 0) ge[t.row] = -dot;
}

// Hashed rows (or projections) of block b from the workspace, into cs [C][CSS].  One row per 32 (or 8) consecutive threads: the
// hyperplanes of a block are contiguous.
template <int RT>
struct CodeRegs { float v[2 * RT]; };
struct CodeThread {
    int t, pl0, np, sh;
    __device__ CodeThread(const GArgs &a, int b) : t(thread_id()), pl0(block_table(a, b) * a.P), np(a.LP - pl0 < a.PB ? a.LP - pl0 : a.PB), sh(a.PB > 8 ? 5 : 3) {}
    __device__ int row(int k) const { return (t + k * kThreads) >> sh; }
    __device__ int plane() const { return t & ((1 << sh) - 1); }
};
template <int RT>
__device__ __forceinline__ void fetch_codes(const GArgs &a, const float *Cx, size_t row0, int nv, int b, CodeRegs<RT> &r)
{
    const CodeThread t(a, b);
    const float *src = Cx + row0 * a.LP + t.pl0 + (t.plane() < t.np ? t.plane() : 0);
#pragma unroll
    for (int k = 0; k < 2 * RT; ++k) r.v[k] = src[static_cast<size_t>(t.row(k) < nv ? t.row(k) : nv - 1) * a.LP];
}
template <int RT>
__device__ __forceinline__ void put_codes(const GArgs &a, const CodeRegs<RT> &r, int nv, int b, float *cs)
{
    const CodeThread t(a, b);
#pragma unroll
    for (int k = 0; k < 2 * RT; ++k)
        if (t.plane() < t.np && t.row(k) < nv) cs[t.row(k) * CSS + t.plane()] = r.v[k];
}

// Assignments of block b as fp32 rows ph [C][PHS] from the hashed rows: phi_r = prod_t mass_t(bit t of r); eight corners
// per thread.  Rows >= nv and bucket rows of tables that do not exist are zeros.
template <int RT>
__device__ __forceinline__ void build_phi(const GArgs &a, int b, const float *cs, int nv, float *ph)
{
    const int tb0 = block_table(a, b);
    for (int g = thread_id(); g < 16 * RT * (KB / 8); g += kThreads) {
        const int tok = g >> 3, k0 = (g & 7) * 8, lr = b * KB + k0;
        float f[8];
        if (a.P >= 3) {
            const int table = lr >> a.P, r0 = lr & (a.R - 1);
            float hi = (tok < nv && table < a.L) ? 1.f : 0.f;
            if (hi != 0.f) {
                const float *c = cs + tok * CSS + (table - tb0) * a.P;
                for (int t = 3; t < a.P; ++t) hi *= mass_of(c[t], (r0 >> t) & 1);
                const float q0 = mass_of(c[0], 0), p0 = mass_of(c[0], 1), q1 = mass_of(c[1], 0), p1 = mass_of(c[1], 1);
                const float h0 = hi * mass_of(c[2], 0), h1 = hi * mass_of(c[2], 1);
                const float l[4] = {q0 * q1, p0 * q1, q0 * p1, p0 * p1};
#pragma unroll
                for (int e = 0; e < 4; ++e) { f[e] = h0 * l[e]; f[4 + e] = h1 * l[e]; }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = 0.f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int table = (lr + e) >> a.P, r = (lr + e) & (a.R - 1);
                f[e] = 0.f;
                if (tok < nv && table < a.L) {
                    const float *c = cs + tok * CSS + (table - tb0) * a.P;
                    f[e] = mass_of(c[0], r & 1);
                    if (a.P == 2) f[e] *= mass_of(c[1], r >> 1);
                }
            }
        }
        *reinterpret_cast<f32x4 *>(ph + tok * PHS + k0) = f32x4{f[0], f[1], f[2], f[3]};
        *reinterpret_cast<f32x4 *>(ph + tok * PHS + k0 + 4) = f32x4{f[4], f[5], f[6], f[7]};
    }
}

// acc[rt][ci] += ph^T . ys over the tile's tokens: 16 x 16 tiles of the statistics, rows = the block's bucket rows, columns
// = column tiles w, w + 4, ... of this wavefront.
template <int RT, int NCT>
__device__ __forceinline__ void accumulate(const GArgs &a, const float *ph, const float *ys, int XS, int nrt, f32x4 (&acc)[4][NCT])
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, w = wave_id();
#pragma unroll
    for (int jt = 0; jt < RT; ++jt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = 16 * jt + 4 * q + v;
            float y[NCT];
#pragma unroll
            for (int ci = 0; ci < NCT; ++ci) {
                const int c = 16 * (w + 4 * ci);
                y[ci] = c < a.dp ? ys[j * XS + c + n] : 0.f;
            }
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) {
                if (rt >= nrt) break;
                const float p = ph[j * PHS + 16 * rt + n];
#pragma unroll
                for (int ci = 0; ci < NCT; ++ci) acc[rt][ci] = mfma(p, y[ci], acc[rt][ci]);
            }
        }
    }
}
template <int NCT>
__device__ __forceinline__ void store_state(const GArgs &a, float *S, int b, int nrt, const f32x4 (&acc)[4][NCT])
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, w = wave_id();
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
        if (rt >= nrt) break;
#pragma unroll
        for (int ci = 0; ci < NCT; ++ci) {
            const int c = 16 * (w + 4 * ci) + n;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = b * KB + 16 * rt + 4 * q + v;
                if (c < a.d && r < a.LR) S[static_cast<size_t>(r) * a.d + c] = acc[rt][ci][v];
            }
        }
    }
}
// The block's statistics as tiles in the C/D layout (= B operands of a product over bucket rows).  Rows and columns that do not
// exist repeat the last ones: their assignments are zeros and their results go nowhere, but a zero does not silence an infinity,
// so clear_rows() has to come before a product over bucket rows (row tiles beyond nrt take no part in any).
template <int NCT>
__device__ __forceinline__ void load_state(const GArgs &a, const float *S, int b, f32x4 (&acc)[4][NCT])
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, w = wave_id(), last = a.LR - 1 - b * KB;
    const float *Sb = S + static_cast<size_t>(b) * KB * a.d;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
        for (int ci = 0; ci < NCT; ++ci) {
            const int c = 16 * (w + 4 * ci) + n;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc[rt][ci][v] = Sb[static_cast<uint32_t>(min(16 * rt + 4 * q + v, last) * a.d + min(c, a.d - 1))];
        }
    }
}
template <int NCT>
__device__ __forceinline__ void clear_rows(const GArgs &a, int b, f32x4 (&acc)[4][NCT])
{
    if ((a.LR & 15) == 0) return;                       // (only tables of fewer than 16 corners leave part of a row tile)
    const int q = (thread_id() & 63) >> 4;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool in = b * KB + 16 * rt + 4 * q + v < a.LR;
#pragma unroll
            for (int ci = 0; ci < NCT; ++ci) acc[rt][ci][v] = in ? acc[rt][ci][v] : 0.f;
        }
    }
}
// out[ti][ci] += ph . S for the block: rows = tokens
template <int RT, int NCT>
__device__ __forceinline__ void read_out(const float *ph, int nrt, const f32x4 (&S)[4][NCT], f32x4 (&out)[RT][NCT])
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
        if (rt >= nrt) break;
#pragma unroll
        for (int ti = 0; ti < RT; ++ti) {
            const f32x4 p = lds4(ph + (16 * ti + n) * PHS + 16 * rt + 4 * q);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int ci = 0; ci < NCT; ++ci) out[ti][ci] = mfma(p[v], S[rt][ci][v], out[ti][ci]);
            }
        }
    }
}
// out[ti][ci] += M . ys (TR: M^T . ys) for an in-tile matrix M [C][MS]: tokens x tokens times tokens x columns.  M is zero above
// its diagonal, and a row of ys must reach its own token and those behind it (TR: in front of it) only, also where it holds an
// infinity or a NaN, which a zero does not silence: 16 x 16 tiles above the diagonal are left out, and on the diagonal such
// entries stay out of the matrix product and are added one by one.
template <int RT, int NCT, bool TR>
__device__ __forceinline__ void apply_tile(const GArgs &a, const float *M, int MS, const float *ys, int XS, f32x4 (&out)[RT][NCT])
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, w = wave_id();
    bool finite = true;
#pragma unroll
    for (int jt = 0; jt < RT; ++jt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = 16 * jt + 4 * q + v;
            float y[NCT], yf[NCT];
#pragma unroll
            for (int ci = 0; ci < NCT; ++ci) {
                const int c = 16 * (w + 4 * ci);
                y[ci] = c < a.dp ? ys[j * XS + c + n] : 0.f;
                const bool f = __builtin_isfinite(y[ci]);
                yf[ci] = f ? y[ci] : 0.f;
                finite &= f;
            }
#pragma unroll
            for (int ti = 0; ti < RT; ++ti) {
                if (TR ? ti > jt : ti < jt) continue;
                const float m = TR ? M[j * MS + 16 * ti + n] : M[(16 * ti + n) * MS + j];
#pragma unroll
                for (int ci = 0; ci < NCT; ++ci) out[ti][ci] = mfma(m, ti == jt ? yf[ci] : y[ci], out[ti][ci]);
            }
        }
    }
    if (__all(finite)) return;
#pragma unroll 1
    for (int j = 0; j < 16; ++j) {
#pragma unroll
        for (int ti = 0; ti < RT; ++ti) {
#pragma unroll
            for (int ci = 0; ci < NCT; ++ci) {
                const int c = 16 * (w + 4 * ci);
                const float y = c < a.dp ? ys[(16 * ti + j) * XS + c + n] : 0.f;
                if (__builtin_isfinite(y)) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 4 * q + v;
                    const float m = TR ? M[(16 * ti + j) * MS + 16 * ti + i] : M[(16 * ti + i) * MS + 16 * ti + j];
                    if (TR ? j >= i : j <= i) out[ti][ci][v] = fmaf(m, y, out[ti][ci][v]);
                }
            }
        }
    }
}

// In-tile kernel values Phi_Q(i) . Phi_K(j), accumulated over the blocks: one 16 x 16 tile (i, j) per wavefront for
// C = 32; for C = 16 every wavefront takes 16 of the block's bucket rows and the four partial tiles are added at the end.
template <int RT>
__device__ __forceinline__ void tile_kernel(const float *phq, const float *phk, int nrt, f32x4 &kk)
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, w = wave_id();
    const int ti = RT == 2 ? w >> 1 : 0, tj = RT == 2 ? w & 1 : 0;
    if (ti < tj) return;                              // wholly above the diagonal
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
        if (rt >= nrt || (RT == 1 && rt != w)) continue;
        const f32x4 x = lds4(phq + (16 * ti + n) * PHS + 16 * rt + 4 * q);
        const f32x4 y = lds4(phk + (16 * tj + n) * PHS + 16 * rt + 4 * q);
#pragma unroll
        for (int v = 0; v < 4; ++v) kk = mfma(x[v], y[v], kk);
    }
}
// The finished kernel values, masked to j <= i, into KK [C][C + 4]; part: LDS for the partial tiles of C = 16 (4 x 256 floats).
// Ends with a barrier.
template <int RT>
__device__ __forceinline__ void store_tile_kernel(const f32x4 &kk, float *KK, float *part)
{
    constexpr int MS = 16 * RT + 4;
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, w = wave_id();
    if (RT == 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[w * 256 + (4 * q + v) * 16 + n] = kk[v];
        __syncthreads();
        const int i = threadIdx.x >> 4, j = threadIdx.x & 15;
        const float s = (part[threadIdx.x] + part[256 + threadIdx.x]) + (part[512 + threadIdx.x] + part[768 + threadIdx.x]);
        KK[i * MS + j] = j <= i ? s : 0.f;
    } else {
        const int ti = w >> 1, tj = w & 1;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * ti + 4 * q + v, j = 16 * tj + n;
            KK[i * MS + j] = j <= i ? kk[v] : 0.f;
        }
    }
    __syncthreads();
}

// 1 / max(|x|, floor) of the row of the tile in xs that this thread shares with its neighbours, 16 / RT threads per row
// (unit-norm option)
template <int RT>
__device__ __forceinline__ float row_scale(const GArgs &a, const float *xs, int XS)
{
    constexpr int TPR = kThreads / (16 * RT);
    const int row = threadIdx.x / TPR, sub = threadIdx.x % TPR;
    float ss = 0.f;
    for (int c = sub; c < a.d; c += TPR) { const float x = xs[row * XS + c]; ss = fmaf(x, x, ss); }
#pragma unroll
    for (int m = 1; m < TPR; m <<= 1) ss += __shfl_xor(ss, m, 64);
    return 1.0f / fmaxf(sqrtf(ss), kUnitFloor);
}
// Hashed rows of a tile on np <= 32 hyperplanes (W: the first one's row) into cs [C][CSS]; those of its first nst rows and the
// projections also to Cx and Zx (token row0 and hyperplane pl0 on).  z = X W^T: 16 tokens x 16 hyperplanes are a tile, and the
// waves share tiles and the contraction over d: its k-steps go round four partial sums, a wavefront forms one, two or all of
// them, and they are added in pairs, the same for every split.  Accumulated in fp64 (products of fp32 are exact there): a bit's mass
// multiplies an error of z by 2 beta, and the projection is a small share of the work.  Then one (token, hyperplane) per
// thread.  (A tile per wavefront left three of four idle at L = P = 4 and gave the busy one four evaluations a lane.)
// zp: LDS, 4 x 256 doubles.  Two barriers: before the partial sums are read, and none behind (cs is not visible yet).
template <int NCT>
struct PlaneRegs {                              // this lane's share of its hyperplane's row, k-steps of its wavefront's parts
    // (With more than 64 columns the first part only; the others are requested one part ahead, under the 8 matrix instructions and more of
    // the part in front.  All of them at once, next to the rows and the statistics, cost a workgroup per CU and spilled 22 to
    // 32 registers at 256 columns: fp32, L = P = 4, B H = 32, N = 4096, 114 us for the totals at d = 128 and 220 at 256; 97 and 176 now.)
    static constexpr int HELD = NCT > 1 ? 1 : 4;
    f32x4 v[HELD * NCT];
};
struct HashSplit {
    int tiles, parts, tile, part0;              // tiles of a pass over the hyperplanes; partial sums of this wavefront: part0 ..
    template <int RT>
    __device__ static HashSplit of(int np)
    {
        HashSplit h;
        const int w = wave_id();
        h.tiles = RT * ((np + 15) >> 4);        // 1, 2 or 4
        h.parts = h.tiles;
        h.tile = w & (h.tiles - 1);
        h.part0 = (w / h.tiles) * h.parts;
        return h;
    }
};
// COUNT parts of them from p0 on, as far as there are such
template <int RT, int NCT, int COUNT>
__device__ __forceinline__ void fetch_parts(const GArgs &a, const float *W, int np, const HashSplit &h, int p0, f32x4 (&v)[COUNT * NCT])
{
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4, pl = 16 * (h.tile / RT) + n;
    const float *wr = W + static_cast<size_t>(pl < np ? pl : 0) * a.d;
#pragma unroll
    for (int p = 0; p < COUNT; ++p) {
#pragma unroll
        for (int j = 0; j < NCT; ++j) {
            const int c = 16 * (4 * j + h.part0 + p0 + p) + 4 * q;
            if (p0 + p < h.parts) v[p * NCT + j] = *reinterpret_cast<const f32x4 *>(wr + (c < a.d ? c : 0));
        }
    }
}
template <int RT, int NCT>
__device__ __forceinline__ void fetch_planes(const GArgs &a, const float *W, int np, PlaneRegs<NCT> &r)
{
    fetch_parts<RT, NCT, PlaneRegs<NCT>::HELD>(a, W, np, HashSplit::of<RT>(np), 0, r.v);
}
template <int RT, int NCT>
__device__ __forceinline__ void hash_block(const GArgs &a, const PlaneRegs<NCT> &wr, const float *W, int np, const float *xs, int XS, const float *inv, double *zp,
                                           float *cs, float *Cx, float *Zx, size_t row0, int pl0, int nst)
{
    const HashSplit h = HashSplit::of<RT>(np);
    const int lane = thread_id() & 63, n = lane & 15, q = lane >> 4;
    const float *xrow = xs + (16 * (h.tile % RT) + n) * XS + 4 * q;
    f64x4 sum = {0., 0., 0., 0.}, pair = sum;
    constexpr bool kAhead = PlaneRegs<NCT>::HELD == 1;
    f32x4 next[NCT];
    if (kAhead) {
#pragma unroll
        for (int j = 0; j < NCT; ++j) next[j] = wr.v[j];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (p >= h.parts) break;
        f64x4 z0 = {0., 0., 0., 0.}, z1 = z0;
        f32x4 part[NCT];
        if constexpr (kAhead) {
#pragma unroll
            for (int j = 0; j < NCT; ++j) part[j] = next[j];
            fetch_parts<RT, NCT, 1>(a, W, np, h, p + 1, next);
        }
#pragma unroll
        for (int j = 0; j < NCT; ++j) {
            const int c0 = 16 * (4 * j + h.part0 + p);
            if (c0 >= a.dp) break;
            const f32x4 x = lds4(xrow + c0), y = kAhead ? part[j] : wr.v[kAhead ? 0 : p * NCT + j];          // (columns beyond d are zeros in xs)
            z0 = mfma64(x[0], y[0], z0);
            z1 = mfma64(x[1], y[1], z1);
            z0 = mfma64(x[2], y[2], z0);
            z1 = mfma64(x[3], y[3], z1);
        }
        if (p & 1) sum = sum + (pair + (z0 + z1));
        else pair = z0 + z1;
    }
    if (h.parts == 1) sum = pair;
#pragma unroll
    for (int v = 0; v < 4; ++v) zp[wave_id() * 256 + (q + 4 * v) * 16 + n] = sum[v];
    __syncthreads();
    for (int t = 0; t < h.tiles; ++t) {
        const int tok = 16 * (t % RT) + (threadIdx.x >> 4), pl = 16 * (t / RT) + (threadIdx.x & 15);
        const double *z4 = zp + t * 256 + threadIdx.x;
        const double zd = h.tiles == 1 ? (z4[0] + z4[256]) + (z4[512] + z4[768]) : (h.tiles == 2 ? z4[0] + z4[512] : z4[0]);
        float zz = static_cast<float>(zd);
        if (a.unit) zz *= inv[tok];
        const float c = code(zz, a.beta);
        if (pl < np) {
            cs[tok * CSS + pl] = c;
            if (tok < nst) {
                Cx[(row0 + tok) * a.LP + pl0 + pl] = c;
                Zx[(row0 + tok) * a.LP + pl0 + pl] = zz;
            }
        }
    }
}

// ================================================================ totals
// blockIdx = (segment, block, batch*head).  SIDE 0: block < nblk: hashes the keys of the segment on the block's
// hyperplanes (Algorithm 1, steps 2-4; hashed rows and projections go to the workspace) and accumulates the block's
// statistics of (phi_K, [V | 1]) (step 5); block >= nblk: only hashes the queries on block - nblk's hyperplanes.
// SIDE 1: the statistics of (phi_Q, [g | g_e]) of the backward pass from the hashed queries.
template <int RT>
struct TotalsLds {
    // (the assignments' place also takes the partial projections, 4 x 256 doubles)
    static constexpr int PH = 16 * RT * PHS > 2048 ? 16 * RT * PHS : 2048;
    float *ys, *xs, *ph, *cs, *ge, *inv;
    static size_t floats(int dp, int side) { return static_cast<size_t>(16 * RT) * ((side == 0 ? 2 : 1) * (dp + 4) + CSS + 2) + PH + 16; }
    __device__ TotalsLds(float *p, int dp, int side)
    {
        constexpr int C = 16 * RT;
        ys = p; p += C * (dp + 4);
        xs = p; if (side == 0) p += C * (dp + 4);
        ph = p; p += PH;
        ge = p; p += C;
        inv = p; p += C;
        cs = p;
    }
};

// (Three workgroups per CU where 168 registers do: 192 columns, B H = 8, N = 2048, L = 6, P = 5: 75 us for the totals with two, at 180
// registers, 66 with three.  256 columns would spill 74: 89 us with two, 112 with three.  64 columns take 115 by themselves.)
template <typename T, int RT, int NCT, int SIDE>
__global__ __launch_bounds__(kThreads, RT * NCT <= 4 && NCT < 4 && NCT > 1 ? 3 : 2) void generic_totals(GArgs a, const T *Xq, const T *Xk, const T *Y, const T *O,
                                                              const float *den, float *state)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    constexpr int C = 16 * RT, TPR = kThreads / C;
    TotalsLds<RT> s(lds, a.dp, SIDE);
    const int XS = a.dp + 4;
    const int seg = blockIdx.x, bh = blockIdx.z, tid = threadIdx.x;
    const bool query = SIDE == 0 && static_cast<int>(blockIdx.y) >= a.nblk;
    const int b = query ? blockIdx.y - a.nblk : blockIdx.y;
    const bool writes = a.bpt == 1 || b % a.bpt == 0;       // hashed rows: the first block of a table
    if (query && !writes) return;
    const int nrt = block_rtiles(a, b), tb0 = block_table(a, b), pl0 = tb0 * a.P;
    const int np = a.LP - pl0 < a.PB ? a.LP - pl0 : a.PB;
    const float *W = a.W + (static_cast<size_t>(bh % a.H) * a.LP + pl0) * a.d;
    f32x4 acc[4][NCT];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
        for (int ci = 0; ci < NCT; ++ci) acc[rt][ci] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float mass = 0.f;                                       // threads 0..63: extra column of bucket row tid
    PlaneRegs<NCT> wr;
    if (SIDE == 0) fetch_planes<RT, NCT>(a, W, np, wr);
    const int64_t seg0 = static_cast<int64_t>(seg) * a.tps * C;
    for (int it = 0; it < a.tps; ++it) {
        const int64_t t0 = seg0 + it * C;
        if (t0 >= a.N) break;
        const int nv = a.N - t0 < C ? static_cast<int>(a.N - t0) : C;
        const size_t row0 = static_cast<size_t>(bh) * a.N + t0;
        if (SIDE == 0) {
            RowRegs<RT, NCT> x, y;
            fetch_rows<T, RT, NCT>(a, query ? Xq : Xk, row0, nv, x);
            if (!query) fetch_rows<T, RT, NCT>(a, Y, row0, nv, y);
            if (it > 0) __syncthreads();                    // the previous tile's readers are done
            put_rows<RT, NCT>(a, x, nv, s.xs, XS);
            if (!query) put_rows<RT, NCT>(a, y, nv, s.ys, XS);
            __syncthreads();
            if (a.unit) {
                const float inv = row_scale<RT>(a, s.xs, XS);
                if (tid % TPR == 0) {
                    const int row = tid / TPR;
                    s.inv[row] = inv;
                    if (b == 0 && row < nv) a.nrm[(query ? 0 : static_cast<size_t>(a.BH) * a.N) + row0 + row] = inv;
                }
            }
            hash_block<RT, NCT>(a, wr, W, np, s.xs, XS, s.inv, reinterpret_cast<double *>(s.ph), s.cs, query ? a.Cq : a.Ck, query ? a.Zq : a.Zk, row0,
                                pl0, writes ? nv : 0);
            if (query) continue;
        } else {
            CodeRegs<RT> c;
            CotRegs<RT, NCT> g;
            fetch_codes<RT>(a, a.Cq, row0, nv, b, c);
            fetch_cotangents<T, RT, NCT>(a, Y, O, den, row0, nv, g);
            if (it > 0) __syncthreads();
            put_codes<RT>(a, c, nv, b, s.cs);
            put_cotangents<RT, NCT>(a, g, nv, s.ys, XS, s.ge);
        }
        __syncthreads();
        build_phi<RT>(a, b, s.cs, nv, s.ph);
        __syncthreads();
        accumulate<RT, NCT>(a, s.ph, s.ys, XS, nrt, acc);
        if (tid < KB) {
#pragma unroll 8
            for (int j = 0; j < C; ++j) mass = fmaf(s.ph[j * PHS + tid], SIDE == 0 ? 1.f : s.ge[j], mass);
        }
    }
    if (query) return;
    float *S = state + (static_cast<size_t>(bh) * a.nseg + seg) * a.ST;
    store_state<NCT>(a, S, b, nrt, acc);
    if (tid < KB && b * KB + tid < a.LR) S[static_cast<size_t>(a.LR) * a.d + b * KB + tid] = mass;
}

// ================================================================ forward
template <int RT>
struct FwdLds {
    float *vs, *phq, *phk, *kk, *part, *csq, *csk, *am, *den;
    static size_t floats(int dp) { return static_cast<size_t>(16 * RT) * (dp + 4 + 2 * PHS + 16 * RT + 4 + 2 * CSS + 1) + KB + (RT == 1 ? 1024 : 0) + 16; }
    __device__ FwdLds(float *p, int dp)
    {
        constexpr int C = 16 * RT;
        vs = p; p += C * (dp + 4);
        phq = p; p += C * PHS;
        phk = p; p += C * PHS;
        kk = p; p += C * (C + 4);
        part = p; p += RT == 1 ? 1024 : 0;
        am = p; p += KB;
        den = p; p += C;
        csq = p; p += C * CSS;
        csk = p;
    }
};

template <typename T, int RT, int NCT>
__global__ __launch_bounds__(kThreads, 2) void generic_forward(GArgs args, const T *V, const float *state, T *Out, float *den_out)
{
    const GArgs &a = args;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    constexpr int C = 16 * RT, MS = C + 4, TPR = kThreads / C;
    FwdLds<RT> s(lds, a.dp);
    const int XS = a.dp + 4;
    const int seg = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x, w = wave_id(), lane = tid & 63, n = lane & 15, q = lane >> 4;
    const float *S0 = state + (static_cast<size_t>(bh) * a.nseg + (a.causal ? seg : 0)) * a.ST;
    float *Sc = a.carry + (static_cast<size_t>(bh) * a.nseg + seg) * a.ST;
    const int64_t seg0 = static_cast<int64_t>(seg) * a.tps * C;
    const int tok_r = tid / TPR, sub = tid % TPR;                // row and share of the normaliser sums
    for (int it = 0; it < args.tps; ++it) {
        const GArgs a = fresh(args);
        const int64_t t0 = seg0 + it * C;
        if (t0 >= a.N) break;
        const int nv = a.N - t0 < C ? static_cast<int>(a.N - t0) : C;
        const size_t row0 = static_cast<size_t>(bh) * a.N + t0;
        const bool more = a.causal && it + 1 < a.tps && t0 + C < a.N;      // a later tile of the segment reads the statistics
        const float *S = (a.causal && it > 0) ? Sc : S0;
        f32x4 out[RT][NCT], kk = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ti = 0; ti < RT; ++ti) {
#pragma unroll
            for (int ci = 0; ci < NCT; ++ci) out[ti][ci] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        float dn = 0.f;
        // the first block's operands and the rows of V are requested together, a following block's next to the products of the one
        // in front of it
        f32x4 sb[4][NCT];
        CodeRegs<RT> cq, ck;
        float am;
        auto fetch_block = [&](int b) __attribute__((always_inline)) {
            fetch_codes<RT>(a, a.Cq, row0, nv, b, cq);
            if (a.causal) fetch_codes<RT>(a, a.Ck, row0, nv, b, ck);
            const bool mrow = tid < KB && b * KB + tid < a.LR;
            const float x = S[static_cast<size_t>(a.LR) * a.d + (mrow ? b * KB + tid : 0)];
            am = mrow ? x : 0.f;
        };
        RowRegs<RT, NCT> vr;
        fetch_block(0);
        if (a.causal) fetch_rows<T, RT, NCT>(a, V, row0, nv, vr);
        load_state<NCT>(a, S, 0, sb);
        if (it > 0) __syncthreads();
        if (a.causal) put_rows<RT, NCT>(a, vr, nv, s.vs, XS);
        for (int b = 0; b < args.nblk; ++b) {
            const GArgs a = fresh(args);
            const int nrt = block_rtiles(a, b);
            const float am_b = am;
            put_codes<RT>(a, cq, nv, b, s.csq);
            if (a.causal) put_codes<RT>(a, ck, nv, b, s.csk);
            if (tid < KB) s.am[tid] = am;
            if (b + 1 < a.nblk) fetch_block(b + 1);
            __syncthreads();
            build_phi<RT>(a, b, s.csq, nv, s.phq);
            if (a.causal) build_phi<RT>(a, b, s.csk, nv, s.phk);
            __syncthreads();
            clear_rows<NCT>(a, b, sb);
            read_out<RT, NCT>(s.phq, nrt, sb, out);
#pragma unroll
            for (int k = 0; k < KB / TPR; ++k) dn = fmaf(s.phq[tok_r * PHS + sub + k * TPR], s.am[sub + k * TPR], dn);
            if (a.causal) tile_kernel<RT>(s.phq, s.phk, nrt, kk);
            if (more) {
                accumulate<RT, NCT>(a, s.phk, s.vs, XS, nrt, sb);
                store_state<NCT>(a, Sc, b, nrt, sb);
                if (tid < KB && b * KB + tid < a.LR) {
                    float m = am_b;
                    for (int j = 0; j < C; ++j) m += s.phk[j * PHS + tid];
                    Sc[static_cast<size_t>(a.LR) * a.d + b * KB + tid] = m;
                }
            }
            if (b + 1 < a.nblk) load_state<NCT>(a, S, b + 1, sb);
            __syncthreads();
        }
        if (a.causal) {
            store_tile_kernel<RT>(kk, s.kk, s.part);
#pragma unroll
            for (int k = 0; k < C / TPR; ++k) dn += s.kk[tok_r * MS + sub + k * TPR];
            apply_tile<RT, NCT, false>(a, s.kk, MS, s.vs, XS, out);
        }
#pragma unroll
        for (int m = 1; m < TPR; m <<= 1) dn += __shfl_xor(dn, m, 64);
        if (sub == 0) {
            s.den[tok_r] = dn;
            if (tok_r < nv) den_out[row0 + tok_r] = dn / static_cast<float>(a.L);
        }
        __syncthreads();
#pragma unroll
        for (int ti = 0; ti < RT; ++ti) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int tok = 16 * ti + 4 * q + v;
                const float e = s.den[tok], inv = e > 0.f ? 1.0f / e : 0.f;    // e = 0: only the hard hash, empty buckets
#pragma unroll
                for (int ci = 0; ci < NCT; ++ci) {
                    const int c = 16 * (w + 4 * ci) + n;
                    if (tok < nv && c < a.d) store1(Out + (row0 + tok) * a.d + c, out[ti][ci][v] * inv);
                }
            }
        }
    }
}

// ================================================================ gradients
// All three gradients of a tile: with S the statistics before the tile and dS = (dB | dA) the cotangent statistics behind
// it, T[i][j] = V_j . g_i + g_e(i) and K[i][j] = phi_Q(i) . phi_K(j), both masked to j <= i,
//     dphi_Q(i) = S [g_i | g_e(i)] + sum_j T[i][j] phi_K(j)        dphi_K(j) = dS [V_j | 1] + sum_i T[i][j] phi_Q(i)
//     dV_j = phi_K(j) dB + sum_i K[i][j] g_i
// (not causal: only the first terms, with the totals), then the chain rule through the corner softmax, tanh and W.  With
// w_r = phi_r dphi_r, m = sum_r w_r and G_t = sum of w_r over the corners on bit t's minor side, the cotangent of tanh z_t
// is +-2 beta (small_t (m - G_t) - big_t G_t): no cancellation where a bit is saturated.
// Segments of one tile take both sides in one launch; longer causal segments carry dS right to left and S left to right, one
// launch each, in this order (sides: bit 0 = dQ, bit 1 = dK and dV): dS is carried where it stands, and S where dS has been.
template <int RT>
struct GradLds {
    float *gs, *vs, *phq, *phk, *tt, *kk, *csq, *csk, *zsq, *zsk, *dz, *am, *dam, *ge, *rec, *rad, *part;
    static size_t floats(int dp)
    {
        return static_cast<size_t>(16 * RT) * (2 * (dp + 4) + 2 * PHS + 2 * (16 * RT + 4) + 4 * CSS + 2 * DZS + 1 + 18 + 2) + 2 * KB +
               (RT == 1 ? 1024 : 0) + 16;
    }
    __device__ GradLds(float *p, int dp)
    {
        constexpr int C = 16 * RT;
        gs = p; p += C * (dp + 4);
        vs = p; p += C * (dp + 4);
        phq = p; p += C * PHS;
        phk = p; p += C * PHS;
        tt = p; p += C * (C + 4);
        kk = p; p += C * (C + 4);
        dz = p; p += 2 * C * DZS;
        part = p; p += RT == 1 ? 1024 : 0;
        am = p; p += KB;
        dam = p; p += KB;
        ge = p; p += C;
        rec = p; p += 2 * C * 9;        // (side, token): m and G_t of a table that spans several blocks
        rad = p; p += 2 * C;
        csq = p; p += C * CSS;
        csk = p; p += C * CSS;
        zsq = p; p += C * CSS;
        zsk = p;
    }
};

// CARRY: causal segments of several tiles.
// (One workgroup per CU where the accumulators need more than 256 registers; LDS allows no more there either.  Three where 168
// registers do: four, with 21 spilled, measured the same.)
template <typename T, int RT, int NCT, bool CARRY>
__global__ __launch_bounds__(kThreads, RT * NCT > 2 ? 1 : (RT * NCT == 2 ? 2 : 3)) void generic_grads(GArgs args, int sides, const T *Q, const T *K, const T *V, const T *O,
                                                             const float *den, const T *dO, const float *stateS, const float *stateD,
                                                             T *dQ, T *dK, T *dV, float *dbeta_part)
{
    const GArgs &a = args;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    constexpr int C = 16 * RT, MS = C + 4, NCH = 2 * RT;
    constexpr bool PRE = RT * NCT <= 2;                      // registers for the rows of the statistics a block ahead
    GradLds<RT> s(lds, a.dp);
    const int XS = a.dp + 4;
    const int seg = blockIdx.x, bh = blockIdx.y, w = wave_id();
    const bool do_q = CARRY ? (sides & 1) != 0 : true, do_kv = CARRY ? (sides & 2) != 0 : true;
    const size_t slot = (static_cast<size_t>(bh) * a.nseg + (a.causal ? seg : 0)) * a.ST;
    float *Sc = a.carry + (static_cast<size_t>(bh) * a.nseg + seg) * a.ST;
    const float *W = a.W + static_cast<size_t>(bh % a.H) * a.LP * a.d;
    const int64_t seg0 = static_cast<int64_t>(seg) * a.tps * C;
    const int64_t left = a.N - seg0;
    const int ntiles = left >= static_cast<int64_t>(a.tps) * C ? a.tps : static_cast<int>((left + C - 1) / C);
    // dphi chains of this wavefront: one side, C = 32: one token tile and all row tiles; C = 16: two row tiles
    const int cside = w >> 1, ct = RT == 2 ? w & 1 : 0, cr0 = RT == 2 ? 0 : 2 * (w & 1);
    const bool cdo = cside == 0 ? do_q : do_kv;
    float dbeta_acc = 0.f;
    for (int i = threadIdx.x; i < 2 * C * DZS; i += kThreads) s.dz[i] = 0.f;          // padding hyperplanes stay zero
    for (int it = 0; it < ntiles; ++it) {
        const GArgs a = fresh(args);
        const int tid = thread_id(), n = tid & 15, q = (tid & 63) >> 4;
        const int tile = (!CARRY || do_q) ? it : ntiles - 1 - it;
        const int64_t t0 = seg0 + static_cast<int64_t>(tile) * C;
        const int nv = a.N - t0 < C ? static_cast<int>(a.N - t0) : C;
        const size_t row0 = static_cast<size_t>(bh) * a.N + t0;
        const bool more = CARRY && it + 1 < ntiles;
        const float *S = (CARRY && it > 0 && do_q) ? Sc : stateS + slot;
        const float *D = (CARRY && it > 0 && do_kv) ? Sc : stateD + slot;
        f32x4 aq[RT][NCT], ak[RT][NCT], av[RT][NCT], kk = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ti = 0; ti < RT; ++ti) {
#pragma unroll
            for (int ci = 0; ci < NCT; ++ci) aq[ti][ci] = ak[ti][ci] = av[ti][ci] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        float radial = 0.f;                                     // threads (side, token) < 2 C: sum of z . dz (unit-norm option)
        // the first block's operands and the tile's rows are requested together, a following block's as soon as the registers are free
        CodeRegs<RT> cq, ck, zq, zk;
        f32x4 db[4][NCT], st[PRE ? 4 * NCT : 1][NCH];
        float am, dam;
        auto fetch_block = [&](int b) __attribute__((always_inline)) {
            fetch_codes<RT>(a, a.Cq, row0, nv, b, cq);
            fetch_codes<RT>(a, a.Ck, row0, nv, b, ck);
            const bool mrow = tid < KB && b * KB + tid < a.LR;
            const size_t at = static_cast<size_t>(a.LR) * a.d + (mrow ? b * KB + tid : 0);
            const float x = S[at], y = D[at];
            am = mrow ? x : 0.f;
            dam = mrow ? y : 0.f;
            fetch_codes<RT>(a, a.Zq, row0, nv, b, zq);
            fetch_codes<RT>(a, a.Zk, row0, nv, b, zk);
        };
        // rows of the statistics for dphi (contraction over columns) of this wavefront's side: k-step j, row tile cr0 + i
        // (rows that do not exist repeat the last one: their share of dphi is not used; columns beyond d are cleared where they are used)
        const float *St = cside == 0 ? S : D;
        auto state_row = [&](int b, int j, int i) __attribute__((always_inline)) {
            const int r = min(16 * (cr0 + i) + n, a.LR - 1 - b * KB), c = min(16 * j + 4 * q, a.d - 4);
            return *reinterpret_cast<const f32x4 *>(St + static_cast<size_t>(b) * KB * a.d + static_cast<uint32_t>(r * a.d + c));
        };
        auto fetch_state_rows = [&](int b) __attribute__((always_inline)) {
            if constexpr (PRE) {
#pragma unroll
                for (int j = 0; j < 4 * NCT; ++j) {
#pragma unroll
                    for (int i = 0; i < NCH; ++i) st[j][i] = state_row(b, j, i);
                }
            }
        };
        {
            CotRegs<RT, NCT> g;
            RowRegs<RT, NCT> v;
            fetch_cotangents<T, RT, NCT>(a, dO, O, den, row0, nv, g);
            fetch_rows<T, RT, NCT>(a, V, row0, nv, v);
            fetch_block(0);
            fetch_state_rows(0);
            if (do_kv) load_state<NCT>(a, D, 0, db);
            __syncthreads();
            put_cotangents<RT, NCT>(a, g, nv, s.gs, XS, s.ge);
            put_rows<RT, NCT>(a, v, nv, s.vs, XS);
        }
        __syncthreads();
        if (a.causal) {
            // T: C = 32: one 16 x 16 tile per wavefront; C = 16: wavefront 0
            const int ti = RT == 2 ? w >> 1 : 0, tj = RT == 2 ? w & 1 : 0;
            if (RT == 2 || w == 0) {
                f32x4 t = {0.f, 0.f, 0.f, 0.f}, t1 = t;
                if (ti >= tj) {
                    for (int c = 4 * q; c < a.dp; c += 16) {
                        const f32x4 x = lds4(s.gs + (16 * ti + n) * XS + c), y = lds4(s.vs + (16 * tj + n) * XS + c);
                        t = mfma(x[0], y[0], t);
                        t1 = mfma(x[1], y[1], t1);
                        t = mfma(x[2], y[2], t);
                        t1 = mfma(x[3], y[3], t1);
                    }
                    t = t + t1;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + 4 * q + v, j = 16 * tj + n;
                    s.tt[i * MS + j] = j <= i ? t[v] + s.ge[i] : 0.f;
                }
            }
        }
        for (int b = 0; b < a.nblk; ++b) {
            const GArgs a = fresh(args);
            const int tid = thread_id(), n = tid & 15, q = (tid & 63) >> 4;
            const int nrt = block_rtiles(a, b), tb0 = block_table(a, b), pl0 = tb0 * a.P;
            const bool first = a.bpt == 1 || b % a.bpt == 0, last = a.bpt == 1 || b % a.bpt == a.bpt - 1;
            const size_t aoff = static_cast<size_t>(a.LR) * a.d + b * KB;
            const bool mrow = tid < KB && b * KB + tid < a.LR;
            const float am_b = am, dam_b = dam;
            put_codes<RT>(a, cq, nv, b, s.csq);
            put_codes<RT>(a, ck, nv, b, s.csk);
            put_codes<RT>(a, zq, nv, b, s.zsq);
            put_codes<RT>(a, zk, nv, b, s.zsk);
            if (tid < KB) { s.am[tid] = am; s.dam[tid] = dam; }
            if (b + 1 < a.nblk) fetch_block(b + 1);
            __syncthreads();
            build_phi<RT>(a, b, s.csq, nv, s.phq);
            build_phi<RT>(a, b, s.csk, nv, s.phk);
            __syncthreads();
            // ---- dphi, transposed (rows = bucket rows, columns = tokens), then w = phi dphi
            f32x4 dp[NCH];
#pragma unroll
            for (int i = 0; i < NCH; ++i) dp[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (cdo) {
                const float *ys = cside == 0 ? s.gs : s.vs;
#pragma unroll
                for (int j = 0; j < 4 * NCT; ++j) {
                    if (16 * j >= a.dp) break;
                    const f32x4 y = lds4(ys + (16 * ct + n) * XS + 16 * j + 4 * q);
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
                        f32x4 x;
                        if constexpr (PRE) x = st[j][i];
                        else x = state_row(b, j, i);
                        if (16 * j + 16 > a.d) x = 16 * j + 4 * q < a.d ? x : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int v = 0; v < 4; ++v) dp[i] = mfma(x[v], y[v], dp[i]);
                    }
                }
                if (b + 1 < a.nblk) fetch_state_rows(b + 1);
                if (a.causal) {
                    const float *po = cside == 0 ? s.phk : s.phq;
#pragma unroll
                    for (int jt = 0; jt < RT; ++jt) {
                        // above-diagonal token tiles hold zeros: dQ needs j <= i, dK needs i >= j
                        if (RT == 2 && (cside == 0 ? jt > ct : jt < ct)) continue;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int j = 16 * jt + 4 * q + v;
                            const float t = cside == 0 ? s.tt[(16 * ct + n) * MS + j] : s.tt[j * MS + 16 * ct + n];
#pragma unroll
                            for (int i = 0; i < NCH; ++i) dp[i] = mfma(po[j * PHS + 16 * (cr0 + i) + n], t, dp[i]);
                        }
                    }
                }
                const float e = cside == 0 ? s.ge[16 * ct + n] : 1.f;
                const float *am4 = cside == 0 ? s.am : s.dam;
                const float *ps = (cside == 0 ? s.phq : s.phk) + (16 * ct + n) * PHS;
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
                    const int r = 16 * (cr0 + i) + 4 * q;
                    dp[i] = (dp[i] + lds4(am4 + r) * e) * lds4(ps + r);
                }
            }
            if (do_kv) {
                clear_rows<NCT>(a, b, db);
                read_out<RT, NCT>(s.phk, nrt, db, av);
                if (a.causal) tile_kernel<RT>(s.phq, s.phk, nrt, kk);
            }
            if (more) {                                         // the statistics behind this tile, for the next one
                f32x4 sb[4][NCT];
                if (do_q) load_state<NCT>(a, S, b, sb);
                else {
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
                        for (int ci = 0; ci < NCT; ++ci) sb[rt][ci] = db[rt][ci];
                    }
                }
                accumulate<RT, NCT>(a, do_q ? s.phk : s.phq, do_q ? s.vs : s.gs, XS, nrt, sb);
                __syncthreads();                                // S and the carry may be the same memory: all of it has been read
                store_state<NCT>(a, Sc, b, nrt, sb);
                if (mrow) {
                    float m = do_q ? am_b : dam_b;
                    for (int j = 0; j < C; ++j) m += do_q ? s.phk[j * PHS + tid] : s.phq[j * PHS + tid] * s.ge[j];
                    Sc[aoff + tid] = m;
                }
            }
            if (do_kv && b + 1 < a.nblk) load_state<NCT>(a, D, b + 1, db);
            __syncthreads();
            if (cdo) {
                float *ps = (cside == 0 ? s.phq : s.phk) + (16 * ct + n) * PHS;
#pragma unroll
                for (int i = 0; i < NCH; ++i) *reinterpret_cast<f32x4 *>(ps + 16 * (cr0 + i) + 4 * q) = dp[i];
            }
            if (a.bpt > 1 && first)
                for (int i = tid; i < 2 * C * 9; i += kThreads) s.rec[i] = 0.f;
            __syncthreads();
            // ---- back through the corner softmax: an item is (side, table, token, share of CP corners); the shares of a
            //      token's table are neighbouring lanes
            {
                const int items = 2 * a.TB * C * (((a.R < KB ? a.R : KB) + 8 * RT - 1) / (8 * RT));
                for (int ix = thread_id(); ix < items; ix += kThreads) {
                    const int P = uniform(a.P), R = 1 << P, Rb = R < KB ? R : KB, CP = Rb < 8 * RT ? Rb : 8 * RT;
                    const int lcp = __builtin_ctz(CP), lns = __builtin_ctz(Rb) - lcp, NS = 1 << lns;
                    const int sub = ix & (NS - 1), tok = (ix >> lns) & (C - 1), st = (ix >> lns) / C;
                    const int side = st & 1, tl = st >> 1, table = tb0 + tl;
                    if (side == 0 ? !do_q : !do_kv) continue;
                    const float *wv = (side == 0 ? s.phq : s.phk) + tok * PHS + tl * Rb + sub * CP;
                    const float *cs = (side == 0 ? s.csq : s.csk) + tok * CSS + tl * P;
                    float *dzr = s.dz + (side * C + tok) * DZS + tl * P;
                    const bool real = table < a.L && tok < nv;
                    float v[8 * RT], g[8], m = 0.f;
#pragma unroll
                    for (int i = 0; i < 8 * RT; ++i) v[i] = (real && i < CP) ? wv[i] : 0.f;
                    // bits inside the share: sum of the minor side, then fold
                    int len = 8 * RT;
#pragma unroll
                    for (int t = 0; t < 3 + (RT == 2); ++t) {
                        const bool minor1 = t < P && real && (__float_as_uint(cs[t]) >> 31) != 0;
                        float sum = 0.f;
#pragma unroll
                        for (int i = 0; i < 4 * RT; ++i) {
                            if (i >= (len >> 1)) break;
                            sum += minor1 ? v[2 * i + 1] : v[2 * i];
                            v[i] = v[2 * i] + v[2 * i + 1];
                        }
                        g[t] = sum;
                        len >>= 1;
                    }
                    m = v[0];
                    // bits above the share: the whole share is on one side
                    const int r0 = (sub * CP) | (a.bpt > 1 ? (b % a.bpt) * KB : 0);
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        if (t < lcp || t >= P) { if (t >= lcp) g[t] = 0.f; continue; }
                        const bool minor1 = real && (__float_as_uint(cs[t]) >> 31) != 0;
                        g[t] = (minor1 == (((r0 >> t) & 1) != 0)) ? m : 0.f;
                    }
                    for (int o = 1; o < NS; o <<= 1) {
                        m += __shfl_xor(m, o, 64);
#pragma unroll
                        for (int t = 0; t < 8; ++t) g[t] += __shfl_xor(g[t], o, 64);
                    }
                    // finish: the shares take hyperplanes in turn (a table over several blocks: the first share, in its last block)
                    int t0 = sub, step = NS;
                    if (a.bpt > 1) {
                        if (sub != 0) continue;
                        float *rec = s.rec + (side * C + tok) * 9;
                        rec[8] += m;
                        m = rec[8];
#pragma unroll
                        for (int t = 0; t < 8; ++t) { rec[t] += g[t]; g[t] = rec[t]; }
                        if (!last) continue;
                        step = 1;
                    }
                    const float *zr = (side == 0 ? s.zsq : s.zsk) + tok * CSS + tl * P;
                    for (int t = t0; t < P; t += step) {
                        float dz = 0.f, gt = g[0];
#pragma unroll
                        for (int k = 1; k < 8; ++k) gt = t == k ? g[k] : gt;
                        if (real) {
                            const float c = cs[t], z = zr[t], small = fabsf(c), big = 1.0f - small;
                            const float e2 = expf(-2.0f * fabsf(z)), s2 = 4.0f * e2 / ((1.0f + e2) * (1.0f + e2));   // 1 - tanh^2 z
                            const float half = small * (m - gt) - big * gt;
                            const float du = (__float_as_uint(c) >> 31) ? -2.0f * half : 2.0f * half;
                            dz = a.beta * du * s2;
                            if (dbeta_part) dbeta_acc = fmaf(du, tanhf(z), dbeta_acc);
                        }
                        dzr[t] = dz;
                    }
                }
            }
            __syncthreads();
            // ---- dX += dz . W over the block's hyperplanes
            if (last) {
                const int np = a.LP - pl0 < a.PB ? a.LP - pl0 : a.PB;
                for (int p0 = 0; p0 < np; p0 += 16) {
                    f32x4 wb[NCT];
#pragma unroll
                    for (int ci = 0; ci < NCT; ++ci) {
                        const int c = 16 * (w + 4 * ci) + n;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int pl = p0 + 4 * q + v;
                            wb[ci][v] = (pl < np && c < a.d) ? W[static_cast<size_t>(pl0 + pl) * a.d + c] : 0.f;
                        }
                    }
#pragma unroll
                    for (int ti = 0; ti < RT; ++ti) {
                        const f32x4 xq = lds4(s.dz + (16 * ti + n) * DZS + p0 + 4 * q), xk = lds4(s.dz + (C + 16 * ti + n) * DZS + p0 + 4 * q);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
#pragma unroll
                            for (int ci = 0; ci < NCT; ++ci) {
                                if (do_q) aq[ti][ci] = mfma(xq[v], wb[ci][v], aq[ti][ci]);
                                if (do_kv) ak[ti][ci] = mfma(xk[v], wb[ci][v], ak[ti][ci]);
                            }
                        }
                    }
                }
                if (a.unit && tid < 2 * C && (tid % C) < nv) {
                    const float *zr = (tid < C ? s.zsq : s.zsk) + (tid % C) * CSS;
                    for (int p = 0; p < np; ++p) radial = fmaf(zr[p], s.dz[tid * DZS + p], radial);
                }
            }
            // (the next block rewrites the hashed rows behind this barrier-free stretch only after everybody has left the finish
            // step, phi and w after its own barriers, and dz after three more; the projections are still read above)
            if (a.unit && b + 1 < a.nblk) __syncthreads();
        }
        if (do_kv && a.causal) {
            store_tile_kernel<RT>(kk, s.kk, s.part);
            apply_tile<RT, NCT, true>(a, s.kk, MS, s.gs, XS, av);
        }
        if (a.unit) {
            if (tid < 2 * C) s.rad[tid] = radial;
            __syncthreads();
        }
#pragma unroll
        for (int ti = 0; ti < RT; ++ti) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int tok = 16 * ti + 4 * q + v;
                if (tok >= nv) continue;
                float iq = 1.f, ik = 1.f, rq = 0.f, rk = 0.f;
                if (a.unit) {
                    // dx = (g - xhat (xhat . g)) / |x| with g = W^T dz and xhat . g = z . dz
                    iq = a.nrm[row0 + tok];
                    ik = a.nrm[static_cast<size_t>(a.BH) * a.N + row0 + tok];
                    rq = s.rad[tok] * iq * iq;
                    rk = s.rad[C + tok] * ik * ik;
                }
#pragma unroll
                for (int ci = 0; ci < NCT; ++ci) {
                    const int c = 16 * (w + 4 * ci) + n;
                    if (c >= a.d) continue;
                    const size_t at = (row0 + tok) * a.d + c;
                    if (do_q) store1(dQ + at, a.unit ? iq * aq[ti][ci][v] - rq * load1(Q + at) : aq[ti][ci][v]);
                    if (do_kv) {
                        store1(dK + at, a.unit ? ik * ak[ti][ci][v] - rk * load1(K + at) : ak[ti][ci][v]);
                        store1(dV + at, av[ti][ci][v]);
                    }
                }
            }
        }
    }
    // ---- partial cotangent of beta, (2, BH, nseg): slot 0 holds dQ's side (or both), slot 1 dK's
    if (!dbeta_part) return;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dbeta_acc += __shfl_xor(dbeta_acc, m, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s.dz[w] = dbeta_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float t = (s.dz[0] + s.dz[1]) + (s.dz[2] + s.dz[3]);
        if (do_q) dbeta_part[static_cast<size_t>(bh) * a.nseg + seg] = t;
        if (do_kv) dbeta_part[(static_cast<size_t>(a.BH) + bh) * a.nseg + seg] = do_q ? 0.f : t;
    }
}

// Debug tap: hard codes and assignments of 16 rows of X on the hyperplanes of one block, as the passes form them.
// blockIdx = (tile, block, batch*head); the first block of a table writes its codes.
template <typename T>
__global__ __launch_bounds__(kThreads) void generic_hash_tap(GArgs a, const T *X, uint8_t *codes, float *phi)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    TotalsLds<1> s(lds, a.dp, 1);           // (the rows of X take the place of the cotangents)
    const int XS = a.dp + 4, bh = blockIdx.z, b = blockIdx.y, tid = threadIdx.x;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * 16;
    const int nv = a.N - t0 < 16 ? static_cast<int>(a.N - t0) : 16;
    const size_t row0 = static_cast<size_t>(bh) * a.N + t0;
    const int tb0 = block_table(a, b), pl0 = tb0 * a.P, np = a.LP - pl0 < a.PB ? a.LP - pl0 : a.PB;
    RowRegs<1, 4> x;
    PlaneRegs<4> wr;
    fetch_rows<T, 1, 4>(a, X, row0, nv, x);
    const float *W = a.W + (static_cast<size_t>(bh % a.H) * a.LP + pl0) * a.d;
    fetch_planes<1, 4>(a, W, np, wr);
    put_rows<1, 4>(a, x, nv, s.ys, XS);
    __syncthreads();
    if (a.unit) {
        const float inv = row_scale<1>(a, s.ys, XS);
        if (tid % 16 == 0) s.inv[tid / 16] = inv;
    }
    hash_block<1, 4>(a, wr, W, np, s.ys, XS, s.inv, reinterpret_cast<double *>(s.ph), s.cs, nullptr, nullptr, 0, 0, 0);
    __syncthreads();
    if (a.bpt == 1 || b % a.bpt == 0) {
        for (int i = tid; i < 16 * a.TB; i += kThreads) {
            const int tok = i / a.TB, table = tb0 + i % a.TB;
            if (tok >= nv || table >= a.L) continue;
            unsigned c = 0;
            for (int t = 0; t < a.P; ++t) c |= (1u - (__float_as_uint(s.cs[tok * CSS + (table - tb0) * a.P + t]) >> 31)) << t;
            codes[(row0 + tok) * a.L + table] = static_cast<uint8_t>(c);
        }
    }
    if (!phi) return;
    build_phi<1>(a, b, s.cs, nv, s.ph);
    __syncthreads();
    for (int i = tid; i < 16 * KB; i += kThreads) {
        const int tok = i / KB, r = b * KB + i % KB;
        if (tok < nv && r < a.LR) phi[(row0 + tok) * a.LR + r] = s.ph[tok * PHS + i % KB];
    }
}

// Sum of the per-segment totals, written as A[row * a_stride] and Bsum[row * b_stride + column], row = (bh, l, r).
__global__ void generic_bucket_tap(GArgs a, const float *state, float *A, float *Bsum, int a_stride, int b_stride)
{
    const size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
    const size_t per = static_cast<size_t>(a.LR) * (a.d + 1);
    if (i >= per * a.BH) return;
    const size_t bh = i / per, e = i - bh * per;
    float run = 0.f;
    for (int s = 0; s < a.nseg; ++s) run += state[(bh * a.nseg + s) * a.ST + e];
    if (e < static_cast<size_t>(a.LR) * a.d) {
        const size_t r = e / a.d;
        Bsum[(bh * a.LR + r) * b_stride + (e - r * a.d)] = run;
    } else {
        A[(bh * a.LR + (e - static_cast<size_t>(a.LR) * a.d)) * a_stride] = run;
    }
}

// In-place scan over the segments of one batch*head, four floats per thread; the blockDim.y groups of a workgroup take
// consecutive runs of segments.  mode: see ScanMode; `open`: the open forms.
// (Bound by memory: every state is read once and written once when a group's run fits registers.  One thread per element
// walking all segments alone is bound by its chain of loads instead: 30 us against 6 at 64 segments of 4160 floats.)
constexpr int kScanRun = 8;
__global__ __launch_bounds__(1024) void scan_states_kernel(float *state, int nseg, int n4, size_t stride, int mode, int open)
{
    __shared__ f32x4 tot[16][64];
    const int G = blockDim.y, g = threadIdx.y, x = threadIdx.x, e = blockIdx.x * 64 + x;
    const int per = (nseg + G - 1) / G, i0 = g * per, i1 = i0 + per < nseg ? i0 + per : nseg, i1r = i1 - (open && i1 == nseg ? 1 : 0);
    const int first = open ? 1 : 0;                        // the first state that is written
    const bool on = e < n4;
    f32x4 *base = reinterpret_cast<f32x4 *>(state + static_cast<size_t>(blockIdx.y) * nseg * stride) + e;
    const size_t st4 = stride / 4;
    auto at = [&](int i) { return base + static_cast<size_t>(mode == 1 ? nseg - 1 - i : i) * st4; };
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 v[kScanRun], sum = zero;
    if (per <= kScanRun) {
#pragma unroll
        for (int k = 0; k < kScanRun; ++k) v[k] = (on && k < per && i0 + k < i1r) ? *at(i0 + k) : zero;
#pragma unroll
        for (int k = 0; k < kScanRun; ++k) sum += v[k];
    } else if (on) {
        for (int i = i0; i < i1; i += kScanRun) {
#pragma unroll
            for (int k = 0; k < kScanRun; ++k) v[k] = i + k < i1r ? *at(i + k) : zero;
#pragma unroll
            for (int k = 0; k < kScanRun; ++k) sum += v[k];
        }
    }
    tot[g][x] = sum;
    __syncthreads();
    f32x4 run = zero;
    for (int k = 0; k < (mode == 2 ? G : g); ++k) run += tot[k][x];
    if (!on) return;
    if (mode == 2) {
        if (g == 0) *base = run;
        return;
    }
    if (per <= kScanRun) {
#pragma unroll
        for (int k = 0; k < kScanRun; ++k) {
            if (k < per && i0 + k < i1 && i0 + k >= first) *at(i0 + k) = run;
            run += v[k];
        }
    } else {
        for (int i = i0; i < i1; i += kScanRun) {
#pragma unroll
            for (int k = 0; k < kScanRun; ++k) v[k] = i + k < i1r ? *at(i + k) : zero;
#pragma unroll
            for (int k = 0; k < kScanRun; ++k) {
                if (i + k < i1 && i + k >= first) *at(i + k) = run;
                run += v[k];
            }
        }
    }
}

// ================================================================ host side
#define RACE_TRY(expr)                                   \
    do {                                                 \
        hipError_t e_ = (expr);                          \
        if (e_ != hipSuccess) return e_;                 \
    } while (0)

GArgs make_args(const Plan &p, char *ws)
{
    GArgs a;
    a.H = p.H; a.BH = p.BH; a.L = p.L; a.P = p.P; a.R = p.R; a.d = p.d; a.dp = (p.d + 15) & ~15;
    a.LP = p.LP; a.LR = p.LR;
    a.TB = p.R >= KB ? 1 : KB / p.R;
    a.bpt = p.R > KB ? p.R / KB : 1;
    a.nblk = (p.LR + KB - 1) / KB;
    a.PB = a.TB * p.P;
    a.nseg = p.nseg; a.tps = static_cast<int>(p.seg_len / (16 * p.rt)); a.causal = p.causal; a.unit = p.unit_qk;
    a.N = p.N; a.beta = p.beta;
    a.ST = generic_state_floats(p);
    a.W = reinterpret_cast<const float *>(ws + p.off_W);
    const size_t rows = static_cast<size_t>(p.BH) * p.N;
    a.Cq = reinterpret_cast<float *>(ws + p.off_massQ);
    a.Ck = reinterpret_cast<float *>(ws + p.off_massK);
    a.Zq = a.Cq + rows * p.LP;
    a.Zk = a.Ck + rows * p.LP;
    a.nrm = reinterpret_cast<float *>(ws + p.off_part);
    a.carry = reinterpret_cast<float *>(ws + p.off_stateB);
    return a;
}

// Calls f(row tiles per tile, column tiles per wavefront) with the plan's values as compile-time constants.
template <int N> using Int = std::integral_constant<int, N>;
template <int RT, typename F>
hipError_t dispatch_columns(const GArgs &a, F f)
{
    switch ((a.dp + 63) / 64) {
    case 1: return f(Int<RT>{}, Int<1>{});
    case 2: return f(Int<RT>{}, Int<2>{});
    case 3: return f(Int<RT>{}, Int<3>{});
    default: return f(Int<RT>{}, Int<4>{});
    }
}
template <typename F>
hipError_t dispatch(const Plan &p, const GArgs &a, F f)
{
    return p.rt == 1 ? dispatch_columns<1>(a, f) : dispatch_columns<2>(a, f);
}

// Statistics of (phi_K, [V | 1]) per segment and the hashed rows of K (and of Q, if given).
template <typename T>
hipError_t totals_kv(const Plan &p, const GArgs &a, const T *Q, const T *K, const T *V, float *state, hipStream_t st)
{
    ProfileScope prof("simple_totals_kv", st);
    const dim3 grid(p.nseg, a.nblk * (Q ? 2 : 1), p.BH);
    return dispatch(p, a, [&](auto rt, auto nct) {
        constexpr int RT = decltype(rt)::value, NCT = decltype(nct)::value;
        const size_t lds = TotalsLds<RT>::floats(a.dp, 0) * sizeof(float);
        RACE_TRY(allow_lds(generic_totals<T, RT, NCT, 0>, lds));
        hipLaunchKernelGGL((generic_totals<T, RT, NCT, 0>), grid, dim3(kThreads), lds, st, a, Q, K, V,
                           static_cast<const T *>(nullptr), static_cast<const float *>(nullptr), state);
        return hipGetLastError();
    });
}

template <typename T>
hipError_t fwd_impl(const Plan &p, const T *Q, const T *K, const T *V, T *O, float *den, char *ws, hipStream_t st)
{
    const GArgs a = make_args(p, ws);
    float *state = reinterpret_cast<float *>(ws + p.off_stateA);
    RACE_TRY(totals_kv<T>(p, a, Q, K, V, state, st));
    RACE_TRY(scan_states("simple_scan", state, p.nseg, p.BH, a.ST, p.causal ? kScanPrefix : kScanTotal, st));
    ProfileScope prof("simple_fwd_replay", st);
    return dispatch(p, a, [&](auto rt, auto nct) {
        constexpr int RT = decltype(rt)::value, NCT = decltype(nct)::value;
        const size_t lds = FwdLds<RT>::floats(a.dp) * sizeof(float);
        RACE_TRY(allow_lds(generic_forward<T, RT, NCT>, lds));
        hipLaunchKernelGGL((generic_forward<T, RT, NCT>), dim3(p.nseg, p.BH), dim3(kThreads), lds, st, a, V,
                           static_cast<const float *>(state), O, den);
        return hipGetLastError();
    });
}

template <typename T>
hipError_t bwd_impl(const Plan &p, const T *Q, const T *K, const T *V, const T *O, const float *den, const T *dO,
                    T *dQ, T *dK, T *dV, float *dbeta, char *ws, hipStream_t st)
{
    const GArgs a = make_args(p, ws);
    float *stateS = reinterpret_cast<float *>(ws + p.off_stateA), *stateD = reinterpret_cast<float *>(ws + p.off_stateB);
    float *dbeta_part = reinterpret_cast<float *>(ws + p.off_dbeta);
    if (!p.fwd_state_kept) {
        RACE_TRY(totals_kv<T>(p, a, Q, K, V, stateS, st));
        RACE_TRY(scan_states("simple_scan", stateS, p.nseg, p.BH, a.ST, p.causal ? kScanPrefix : kScanTotal, st));
    }
    {
        ProfileScope prof("simple_totals_qg", st);
        RACE_TRY(dispatch(p, a, [&](auto rt, auto nct) {
            constexpr int RT = decltype(rt)::value, NCT = decltype(nct)::value;
            const size_t lds = TotalsLds<RT>::floats(a.dp, 1) * sizeof(float);
            RACE_TRY(allow_lds(generic_totals<T, RT, NCT, 1>, lds));
            hipLaunchKernelGGL((generic_totals<T, RT, NCT, 1>), dim3(p.nseg, a.nblk, p.BH), dim3(kThreads), lds, st, a,
                               static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), dO, O, den, stateD);
            return hipGetLastError();
        }));
    }
    RACE_TRY(scan_states("simple_scan", stateD, p.nseg, p.BH, a.ST, p.causal ? kScanSuffix : kScanTotal, st));
    const auto launch = [&](auto carry, int sides) {
        ProfileScope prof("simple_grads", st);
        return dispatch(p, a, [&](auto rt, auto nct) {
            constexpr int RT = decltype(rt)::value, NCT = decltype(nct)::value;
            constexpr bool CARRY = decltype(carry)::value;
            const size_t lds = GradLds<RT>::floats(a.dp) * sizeof(float);
            RACE_TRY(allow_lds(generic_grads<T, RT, NCT, CARRY>, lds));
            hipLaunchKernelGGL((generic_grads<T, RT, NCT, CARRY>), dim3(p.nseg, p.BH), dim3(kThreads), lds, st, a, sides, Q, K, V, O, den, dO,
                               static_cast<const float *>(stateS), static_cast<const float *>(stateD), dQ, dK, dV, dbeta ? dbeta_part : nullptr);
            return hipGetLastError();
        });
    };
    if (generic_carries(p)) {
        RACE_TRY(launch(std::true_type{}, 2));
        RACE_TRY(launch(std::true_type{}, 1));
    } else {
        RACE_TRY(launch(std::false_type{}, 3));
    }
    if (dbeta) RACE_TRY(reduce_dbeta(p, dbeta_part, dbeta, st));
    return hipSuccess;
}

template <typename T>
hipError_t buckets_impl(const Plan &p, const T *K, const T *V, float *A, float *Bsum, int a_stride, int b_stride, char *ws, hipStream_t st)
{
    const GArgs a = make_args(p, ws);
    float *state = reinterpret_cast<float *>(ws + p.off_stateA);
    RACE_TRY(totals_kv<T>(p, a, nullptr, K, V, state, st));
    const size_t total = static_cast<size_t>(p.BH) * p.LR * (p.d + 1);
    hipLaunchKernelGGL(generic_bucket_tap, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, st, a, state, A, Bsum,
                       a_stride, b_stride);
    return hipGetLastError();
}

template <typename T>
hipError_t hash_impl(const Plan &p, const T *X, uint8_t *codes, float *phi, char *ws, hipStream_t st)
{
    const GArgs a = make_args(p, ws);
    const size_t lds = TotalsLds<1>::floats(a.dp, 1) * sizeof(float);
    RACE_TRY(allow_lds(generic_hash_tap<T>, lds));
    hipLaunchKernelGGL((generic_hash_tap<T>), dim3(static_cast<unsigned>((p.N + 15) / 16), a.nblk, p.BH), dim3(kThreads), lds, st, a, X, codes, phi);
    return hipGetLastError();
}

}  // namespace

hipError_t scan_states(const char *name, float *state, int nseg, int BH, size_t stride, int mode, hipStream_t st)
{
    // (one segment: its total is where it belongs, and an open scan would neither read nor write a state)
    if (nseg == 1 && (mode == kScanTotal || mode == kScanPrefixOpen || mode == kScanSuffixOpen)) return hipSuccess;
    ProfileScope prof(name, st);
    int groups = 1;
    while (groups < 16 && groups * kScanRun < nseg) groups *= 2;
    const int n4 = static_cast<int>(stride / 4);
    hipLaunchKernelGGL(scan_states_kernel, dim3((n4 + 63) / 64, BH), dim3(64, groups), 0, st, state, nseg, n4, stride, mode & 3, mode >> 2);
    return hipGetLastError();
}

size_t generic_state_floats(const Plan &p) { return (static_cast<size_t>(p.LR) * (p.d + 1) + 63) & ~static_cast<size_t>(63); }

bool generic_carries(const Plan &p) { return p.causal && p.seg_len > 16 * p.rt; }

// Tile and segment length.  Tiles of 16 tokens while they make less than four workgroups per CU, else 32 (half the reads
// of the statistics per token).  Segments are single tiles unless that makes more than 2048 workgroups, where longer
// segments save states (memory, the scan's traffic) and the chip stays full; a caller's chunk is rounded up to tiles, and no
// segment is longer than the sequence (tiles per segment are an int in the kernels).
// A wide hash's state is large (d = 128, L = 32, P = 8: 4.2 MB per segment and head), so the two sets of states are bounded: by
// kFreeStateBytes or, where that is more, by what keeps the workspace at the size of one fp32 row per token and table three times
// (what the size limit counts) plus the states of 2048 tables twice.
// Against a state per tile, fp32, d = 128, P = 8, forward + backward, causal (not causal): B H = 8, N = 8192, L = 32: workspace
// 17.6 -> 2.4 GB, 43.2 -> 56.4 ms (33.6 -> 25.9); B H = 4, N = 4096, L = 8: 2.2 -> 1.1 GB, 3.8 -> 2.7 ms (2.6 -> 2.2); B H = 1,
// N = 16384, L = 64: 17.5 -> 1.9 GB, 28 -> 64 ms (18 -> 28).  The shapes of up to 512 bucket rows of 128 columns stay below
// the bound at every length (2048 states: 1.08 GB).
constexpr double kFreeStateBytes = 1.25 * (1 << 30);
static double most_state_bytes(const Plan &p)
{
    const double rows = static_cast<double>(p.BH) * static_cast<double>(p.N > 0 ? p.N : 1), column = sizeof(float) * (p.d + 1.0);
    const double hashed = 4.0 * sizeof(float) * p.LP * rows;           // masses and projections of Q and K
    return std::max(kFreeStateBytes, 3.0 * column * p.L * rows + 2.0 * 2048 * p.R * column - hashed);
}
void generic_geometry(int64_t chunk, Plan *p)
{
    const int64_t n = p->N > 0 ? p->N : 1;
    p->rt = (static_cast<int64_t>(p->BH) * ((n + 15) / 16) <= 1024) ? 1 : 2;
    int64_t C = 16 * p->rt, all = (n + C - 1) / C;
    int64_t tiles = 1;
    if (chunk > 0) tiles = std::min((chunk - 1) / C + 1, all);
    else {
        if (p->BH * all > 2048) tiles = (p->BH * all + 2047) / 2048;
        const double per_segment = 2.0 * sizeof(float) * p->BH * generic_state_floats(*p);
        const double most = std::floor(std::max(most_state_bytes(*p) / per_segment, 1.0));
        if (static_cast<double>((all + tiles - 1) / tiles) > most) {
            if (p->rt == 1) { p->rt = 2; C = 32; all = (n + 31) / 32; }       // first of all, larger tiles
            const int64_t least = std::max<int64_t>(1, static_cast<int64_t>(std::ceil(static_cast<double>(all) / most)));
            // of the lengths up to twice the least (64 more), the one whose workgroups make the fewest rounds of tiles over 256 CUs
            const auto rounds = [&](int64_t t) { return (p->BH * ((all + t - 1) / t) + 255) / 256 * t; };
            tiles = least;
            for (int64_t t = least + 1; t <= std::min(least + std::min<int64_t>(least, 64), all); ++t) tiles = rounds(t) < rounds(tiles) ? t : tiles;
        }
    }
    p->seg_len = tiles * C;
}

hipError_t simple_fwd(const Plan &p, const void *Q, const void *K, const void *V, void *O, float *den, char *ws, hipStream_t st)
{
    if (p.dtype == RACE_F32)
        return fwd_impl<float>(p, (const float *)Q, (const float *)K, (const float *)V, (float *)O, den, ws, st);
    return fwd_impl<bf16_t>(p, (const bf16_t *)Q, (const bf16_t *)K, (const bf16_t *)V, (bf16_t *)O, den, ws, st);
}

hipError_t simple_bwd(const Plan &p, const void *Q, const void *K, const void *V, const void *O, const float *den,
                      const void *dO, void *dQ, void *dK, void *dV, float *dbeta, char *ws, hipStream_t st)
{
    if (p.dtype == RACE_F32)
        return bwd_impl<float>(p, (const float *)Q, (const float *)K, (const float *)V, (const float *)O, den,
                               (const float *)dO, (float *)dQ, (float *)dK, (float *)dV, dbeta, ws, st);
    return bwd_impl<bf16_t>(p, (const bf16_t *)Q, (const bf16_t *)K, (const bf16_t *)V, (const bf16_t *)O, den,
                            (const bf16_t *)dO, (bf16_t *)dQ, (bf16_t *)dK, (bf16_t *)dV, dbeta, ws, st);
}

hipError_t simple_hash(const Plan &p, const void *X, uint8_t *codes, float *phi, char *ws, hipStream_t st)
{
    if (p.dtype == RACE_F32) return hash_impl<float>(p, (const float *)X, codes, phi, ws, st);
    return hash_impl<bf16_t>(p, (const bf16_t *)X, codes, phi, ws, st);
}

hipError_t simple_buckets(const Plan &p, const void *K, const void *V, float *A, float *Bsum, int a_stride, int b_stride,
                          char *ws, hipStream_t st)
{
    if (p.dtype == RACE_F32) return buckets_impl<float>(p, (const float *)K, (const float *)V, A, Bsum, a_stride, b_stride, ws, st);
    return buckets_impl<bf16_t>(p, (const bf16_t *)K, (const bf16_t *)V, A, Bsum, a_stride, b_stride, ws, st);
}

}  // namespace race
