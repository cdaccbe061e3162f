// Building blocks of the bf16 MFMA kernel family (gfx950): compile-time shapes, LDS tile layouts,
// operand loads, the projection + soft-assignment "production" step.
//
// Execution shape.  One workgroup of eight wavefronts (two per SIMD, 256 registers each) owns one
// (batch*head, segment) and walks its tokens in tiles of 32.  The bucket statistics of all L tables,
// [L*R][d] fp32 (B of Algorithm 1, step 5; A is kept beside it), never leave the register file: every
// wavefront holds an eighth of them as 32x32 MFMA accumulator tiles (stream kernels: a quarter of the
// bucket rows x half of the columns; grad kernel: an eighth of the bucket rows x all columns, transposed).
// Per tile the workgroup
//   1. turns the hashed rows of the tile's queries and keys (bit_code()) into soft assignments phi (vector ALU), written
//      as bf16 tiles to LDS;
//   2. contracts them with the register-resident statistics and with each other (MFMA).
// Two barriers per tile: whatever goes to LDS for a tile is written in the first half (next to the output of the previous
// tile), whatever reads it runs in the second.
// MFMA 32x32x16 bf16 register layouts used throughout (lane = 32*h + n):
//   A operand: row n of A, columns 8h..8h+7 of the 16-wide k-step;   B operand: column n of B, rows 8h..8h+7;
//   C/D      : column n, rows 8*(v/4) + 4h + v%4 for register v = 0..15.
// An accumulator tile is fed back as a B operand without touching LDS: registers 8s..8s+7 of the
// tile, packed to bf16, are the B operand of k-step s if k-slot (h, e) is taken to mean row
// 16s + 8*(e/4) + 4h + e%4.  The other operand must use the same k order; assignment tiles, which are contracted
// against such operands, keep their bucket rows "pair-interleaved" in LDS (il()): inside every
// group of 16 the two middle blocks of 4 are swapped, so that the 8 a lane needs
// are one aligned 16-byte read.
// LDS bank arithmetic as measured on gfx950 (64 banks of 4 bytes, 256 bytes per clock for reads: 16-byte
// accesses go 16 lanes at a time, 8-byte ones 32 lanes): rows read 16 bytes per lane want a row stride of
// 4 mod 64 words; tiles read through the transposing 8-byte loads (per 16 lanes 4 rows x 32 bytes, the
// next 16 lanes 32 bytes further) want 16 mod 32 words, or rows at spread_row() under 4 mod 64.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace race {
namespace mfma {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef uint16_t bf16raw;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kRowGroups = 4;  // most row groups a workgroup's statistics are split into (stream kernels)
constexpr int kTile = 32;      // tokens per tile

// PAD_: the instantiation also serves problems with fewer tables and hyperplanes than its shape (see Soft).
template <int D_, int P_, int L_, bool PAD_ = false>
struct Cfg {
    static constexpr int D = D_, P = P_, L = L_;
    static constexpr bool PAD = PAD_;
    static constexpr int R = 1 << P, LR = L * R;
    static constexpr int PP = P > 4 ? 8 : 4;            // hyperplanes per table, padded; row l * PP + t of the packed W is
                                                        // hyperplane t of table l
    static constexpr int NG = (L * PP + 31) / 32;       // groups of 32 packed rows
    static constexpr int LPP = NG * 32;                 // packed rows (padding rows are zero)
    static constexpr int PT = (L * PP + 15) / 16;       // 16-row tiles of them that hold hyperplanes
    // stream kernels: wavefront w owns bucket-row group w % RG and column group w / RG (four row groups x two
    // column groups, or two x four when there are only 64 bucket rows)
    static constexpr int RG = LR / 32 >= kRowGroups ? kRowGroups : LR / 32;
    static constexpr int CG = kWaves / RG;
    static constexpr int LRW = LR / RG;                 // bucket rows of one row group
    static constexpr int MT = LRW / 32;                 // 32-row tiles of bucket rows per row group
    static constexpr int NT = D / 32;                   // 32-column tiles of the head dimension
    static constexpr int NTW = NT / CG;                 // column tiles per wavefront
    static constexpr int DW = D / CG;                   // columns per wavefront
    static constexpr int MA = (MT + CG - 1) / CG;       // row tiles whose extra column a wavefront carries
    static_assert(MT == 1 || MT % CG == 0, "row tiles over the column groups");
    // wavefronts per SIMD the stream and totals kernels are compiled for: shapes with at most two accumulator
    // tiles of statistics and one column tile per wavefront fit 128 registers and leave room for a second workgroup
    // on the CU, whose phases interleave with the first one's (measured: with two column tiles the kernels spill
    // at 128 registers and lose more than the second workgroup gains)
    static constexpr int STREAM_WAVES_PER_SIMD = (MT * NTW <= 2 && NTW == 1) ? 4 : 2;
    static constexpr int PLO = P < 3 ? P : 3, PHI = P - PLO;
    static constexpr int CPR = D / 8;                   // 16-byte chunks per row
    // LDS row strides, in bf16 elements (rows stay 16-byte aligned; the pad staggers banks)
    static constexpr int XS = D + 8;                    // [token][d] tiles and W rows, read by rows
    static constexpr int YS = D + 32;                   // [token][d] tiles read through transposing loads
    static constexpr int PS = LR + 8;                   // [token][L*R] assignment tiles, rows at spread_row() of the token
    static constexpr int PST = LR + 16;                 // ... rows in order, read through the 16-row transposing loads (16-byte row
                                                        // writes and transposing reads both 2-way at most)
    static constexpr int STATE = LR * (D + 1);          // floats per saved state: B [LR][D] then A [LR]
    // hashed form of a row (see bit_code()): one float per (table, hyperplane).  In memory a tile of 32 tokens is
    // [table][32 tokens][4 hyperplanes], for P = 6 followed per table by [32 tokens][2 hyperplanes], so that a half
    // wavefront whose lanes are the tile's tokens reads and writes a table's hyperplanes as contiguous pieces: every pass
    // loads them straight into the lanes that rebuild the assignments, without a stop in LDS.
    static constexpr int LP = L * P;
    static constexpr int HT = kTile * P;                // floats of one table of a tile
    static_assert(P == 4 || P == 6, "hashed rows are quads, or a quad and a pair");
    static_assert(L == 4 || L % 8 == 0, "tables over the eight half wavefronts of a side");
    static_assert(RG >= 1 && LR % (32 * RG) == 0 && NT % CG == 0 && NTW >= 1, "bucket rows and columns over the wavefronts");
    static_assert(D % 64 == 0 && P >= 4, "shape (assignments are written for pairs of high-bit indices)");
    static_assert(PT <= 4, "tiles of packed rows over the wavefronts that project them");
};

// Scheduling fence: keeps the instruction scheduler from hoisting the loads and conversions of later
// loop iterations (and with them dozens of live registers) above this point.
#define RACE_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// Lets this wavefront issue before the other one of its SIMD (wavefronts w and w + 4), which wins by its age otherwise.  In the
// second half of a tile the two run the same code: with the younger one ahead in the first part and the older one from
// there on, one's matrix products meet the other's vector work and both reach the barrier together.  (By age alone the older
// wavefront was done 1300 of 4800-5500 cycles early and the younger one ran out the rest alone, at half the issue rate.  Training
// steps of 4.2 million rows of 128 columns, L = 8, P = 6: 44.26 -> 43.02 ms; 160 000 rows of 64 columns: 366 -> 359 us.)
__device__ __forceinline__ void lead(bool on)
{
    if (on) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// Waits for this wavefront's loads.  Loads and stores share a counter and count in order: where loaded rows are used behind
// stores that may or may not be issued (output rows past the end), the compiler has to wait for the stores as well, a
// trip to memory.  With this in front of the stores nothing is left to wait for behind them.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }        // vmcnt(0), the other counters as they are

// Hides the value of an index from the optimiser inside a loop body, so that the dozens of addresses
// derived from it (index + constant) are folded into instruction offsets instead of being hoisted out of
// the loop as separate loop-invariant registers (which then spill).  `step` is the loop's counter: a value that depends on it
// cannot leave the loop.  (Not as a volatile statement: no load or store is moved across one of those, which left every LDS read
// where it was written, its latency in front of its use.)
__device__ __forceinline__ int opaque(int x, int step)
{
    asm("" : "+v"(x) : "s"(step));
    return x;
}
// The same for a uniform value: what is added to it is added again in every pass of the loop (one instruction), not kept in a
// register of its own per sum.
__device__ __forceinline__ int opaque_uniform(int x, int step)
{
    asm("" : "+s"(x) : "s"(step));
    return x;
}

// The soft assignment's run-time parameters.  A compiled shape <d, P, L> also serves smaller problems
// (tables L_real <= L, hyperplanes P_real <= P): tables beyond L_real get zero assignments, and a hyperplane
// beyond P_real is a bit whose mass sits entirely on its +1 side, so that the 2^P_real real corners are the
// corners of the compiled hypercube with all padding bits set.
struct Soft {
    float beta;
    int L, P;
};

// kernel arguments common to the family
struct KArgs {
    int H, nseg;
    int scanned;           // totals: their segments are scanned (not added up), which leaves the last one's unread
    int hash_tokens;       // tokens per workgroup of the hashing kernel
    int64_t N, seg_len;
    float beta, inv_tables;
    int L_real, P_real;    // the problem's tables and hyperplanes (<= the compiled shape's)
    __host__ __device__ Soft soft() const { return Soft{beta, L_real, P_real}; }
    const bf16raw *Wp;     // (H, LPP, D) bf16, rows table by table (see Cfg::PP)
    float *state;          // (BH, nseg, STATE) fp32
    float *Mq, *Mk;        // (BH, ceil(N / 32), 32 * L * P) fp32: the hashed rows of Q and K, tile by tile (see Cfg::HT)
    float *ge;             // (BH, N) fp32: extra column of the read-out cotangents (backward only)
    int want_dbeta;
    float *dbeta_part;     // (2, BH, workgroups per head-batch) fp32: partial cotangents of beta (backward only)
};

// ---------------------------------------------------------------- small helpers
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}
// 16 x 16 x 32 product: A row / B column lane % 16, k-slots 8 (lane / 16) ..; D column lane % 16, rows 4 (lane / 16) + v.
__device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ u32x4 lds128(const bf16raw *p) { return *reinterpret_cast<const u32x4 *>(p); }
// accumulator registers 8s..8s+7 as a bf16 B (or A) operand
__device__ __forceinline__ u32x4 acc_operand(const f32x16 &t, int s)
{
    return s == 0 ? u32x4{pack2(t[0], t[1]), pack2(t[2], t[3]), pack2(t[4], t[5]), pack2(t[6], t[7])}
                  : u32x4{pack2(t[8], t[9]), pack2(t[10], t[11]), pack2(t[12], t[13]), pack2(t[14], t[15])};
}
// fp32 value as a bf16 pair (hi, lo) with hi + lo = x to 16 mantissa bits
__device__ __forceinline__ void split_bf16(float x, float &hi, float &lo)
{
    hi = bf_lo(pack2(x, 0.f));
    lo = x - hi;
}
// a.lo * b.lo + a.hi * b.hi + c on words of two bf16 (v_dot2c_f32_bf16: exact products, fp32 sums)
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
constexpr uint32_t kOnePair = 0x3F803F80u;     // (1.0, 1.0)
// row of accumulator register v for lane half h
__device__ __forceinline__ int acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }
// pair-interleaved position of bucket row c: bits 2 and 3 of the index swapped
__device__ __forceinline__ constexpr int il(int c) { return (c & ~12) | ((c & 4) << 1) | ((c & 8) >> 1); }

// ---------------------------------------------------------------- transposing operand reads
// MFMA operand whose k index runs along the ROWS of a row-major LDS tile M[k][n] (stride in elements):
// lane (n, h) gets column n0 + n, rows k0a..k0a+3 then k0b..k0b+3.  Built from two ds_read_b64_tr_b16:
// within a block of 16 lanes, lane i supplies the address of a 4-element row chunk and receives element
// i%4 of the chunks of lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12; with chunk (row i/4, columns 4(i%4)..) per
// lane that is column i of four consecutive rows.
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef s16x4 __attribute__((address_space(3))) lds_s16x4;
// IL: the tile's columns are pair-interleaved (the chunk of logical columns 4c.. sits at 4 * swap(c)).
// SPREAD: its rows are at spread_row(): the four rows of a block lie four apart, 16 banks under a stride of 4 mod 64 words, which
// suits reads by rows and transposing reads alike (64 KB read by transposing loads: 256 cycles; with the rows in order 1024 under
// that stride, 512 under 8 mod 64 words).
__device__ __forceinline__ constexpr int spread_row(int r) { return (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3); }
template <bool IL = false, bool SPREAD = false>
__device__ __forceinline__ u32x4 lds_tr8(const bf16raw *M, int stride, int k0a, int k0b, int n0, int ln)
{
    const int sub = ln & 15;
    const int chunk = IL ? (((sub & 1) << 1) | ((sub >> 1) & 1)) : (sub & 3);
    const bf16raw *p = M + (SPREAD ? 4 : 1) * (sub >> 2) * stride + n0 + 16 * (ln >> 4) + 4 * chunk;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + (SPREAD ? spread_row(k0a) : k0a) * stride));
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + (SPREAD ? spread_row(k0b) : k0b) * stride));
    const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
    return u32x4{ua.x, ua.y, ub.x, ub.y};
}
// k-slots in plain order (rows k0 + 8h + 0..7) or in accumulator order (pairs with acc_operand); k0: a multiple of 16
template <bool IL = false, bool SPREAD = false>
__device__ __forceinline__ u32x4 lds_tr_plain(const bf16raw *M, int stride, int k0, int n0, int ln, int h)
{
    if (SPREAD) return lds_tr8<IL, true>(M + (k0 + 2 * h) * stride, stride, 0, 4, n0, ln);
    return lds_tr8<IL>(M, stride, k0 + 8 * h, k0 + 8 * h + 4, n0, ln);
}
template <bool IL = false, bool SPREAD = false>
__device__ __forceinline__ u32x4 lds_tr_acc(const bf16raw *M, int stride, int k0, int n0, int ln, int h)
{
    if (SPREAD) return lds_tr8<IL, true>(M + (k0 + h) * stride, stride, 0, 8, n0, ln);
    return lds_tr8<IL>(M, stride, k0 + 4 * h, k0 + 8 + 4 * h, n0, ln);
}

// Operands of 16 x 16 x 32 products along the ROWS of a tile: lane (n = lane % 16, q = lane / 16) gets column n of the 16
// columns whose blocks of four start at the given chunk positions, rows ka .. ka+3 then kb .. kb+3.  chunk: position of the
// lane's block (lane % 4) of the row that it addresses (lane % 16 / 4).
__device__ __forceinline__ u32x4 lds_tr16(const bf16raw *M, int stride, int ka, int kb, int chunk, int lane)
{
    const bf16raw *p = M + ((lane & 15) >> 2) * stride + chunk;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + ka * stride));
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + kb * stride));
    const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
    return u32x4{ua.x, ua.y, ub.x, ub.y};
}

// Sum over the two halves of the wavefront / over the four rows of 16 lanes, in every lane (register swaps, no LDS).
__device__ __forceinline__ float sum_halves(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_rows(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return sum_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Two sums over the halves at once: the lower half of the lanes gets the sum of x0, the upper one that of x1.
__device__ __forceinline__ float sum_halves2(float x0, float x1)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Four sums over the rows of 16 lanes at once: row i of lanes gets the sum of x_i.
__device__ __forceinline__ float sum_rows4(float x0, float x1, float x2, float x3)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x2), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x1), __float_as_uint(x3), false, false);
    const float x02 = __uint_as_float(a[0]) + __uint_as_float(a[1]), x13 = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x02), __float_as_uint(x13), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ---------------------------------------------------------------- the extra column of the statistics (bucket masses)
// Sums of assignments over the tokens of a k-step, with weights, on the matrix cores: the same registers that are the
// assignments' operand of the 32 x 32 x 16 update (lane = 32 h + n: bucket row n, tokens 8 h ..) are, read as the B operand of a
// 16 x 16 x 32 product, column n % 16 with k-slots 8 (n / 16 + 2 h) .., i.e. both halves of the bucket rows in one column.  An A
// operand whose rows 4 q + 0 .. 2 hold the weights in slots 8 q .. and zeros in the others keeps them apart: D register v of lane
// 32 h + n is the sum over tokens 8 h .. of bucket row n with weight part v.  With rows 0 .. 2 holding them in slots 0 .. 7 and
// 16 .. 23 and rows 4 .. 6 in the others the halves of the tokens are added up too, lane n < 32 gets the sum (`whole`).  fp32
// weights enter as three bf16 parts (truncated, 8 bits each: exact from about 2^-110 up, below which the last bits of the third part
// are lost), weights of one as a single part.  (One 16-cycle matrix
// instruction in place of 16 vector ones; both totals kernels spent 128 of their 320-450 vector instructions a step on these sums.)
constexpr int kParts = 4;                       // rows of a [kParts][tokens] bf16 array of weight parts; the last one is zeros
__device__ __forceinline__ bf16raw weight_part(float x, int i)
{
    const float a = bf_hi(__float_as_uint(x)), r = __builtin_isfinite(x) ? x - a : 0.f, b = bf_hi(__float_as_uint(r)), c = r - b;
    const float part = i == 0 ? a : (i == 1 ? b : c);
    return static_cast<bf16raw>(i < kParts - 1 ? __float_as_uint(part) >> 16 : 0u);
}
// This lane's element of a [kParts][tokens] array for a k-step at its first token, and the operand of weights of one.
// Form 32: against operands of 32 bucket rows; form 16: against B operands of 16 x 16 x 32 products (16 bucket rows, 32 tokens).
template <bool WHOLE>
__device__ __forceinline__ int parts_offset32(int tokens, int lane)
{
    const int i = lane & 15, q = lane >> 4;
    return ((i >> 2) == (WHOLE ? q & 1 : q) ? i & 3 : kParts - 1) * tokens + 8 * (q >> 1);
}
__device__ __forceinline__ int parts_offset16(int tokens, int lane)
{
    const int i = lane & 15, q = lane >> 4;
    return (i < kParts - 1 ? i : kParts - 1) * tokens + 8 * q;
}
template <bool WHOLE>
__device__ __forceinline__ u32x4 ones32(int lane)
{
    const int q = lane >> 4;
    const uint32_t one = (lane & 15) == 4 * (WHOLE ? q & 1 : q) ? kOnePair : 0u;
    return u32x4{one, one, one, one};
}
__device__ __forceinline__ u32x4 ones16(int lane)
{
    const uint32_t one = (lane & 15) == 0 ? kOnePair : 0u;
    return u32x4{one, one, one, one};
}
// A product starts from zero and the vector ALU adds what it returns to the running sum.  (The matrix cores do not round to
// nearest when they add to a large accumulator: with the running sum there the masses of 524288 tokens in one segment were
// 3.1e-6 to 4.7e-6 too small and 4.8e-6 to 6.0e-6 off by root mean square; so 1.6e-6 to 2.1e-6, as with sums in the vector ALU alone, which
// the halves of the tokens keep apart as well.  One register between products instead of four.)
template <bool PARTS>
__device__ __forceinline__ float column_sum(u32x4 weights, u32x4 phi)
{
    const f32x4 x = mma16(weights, phi, f32x4{0.f, 0.f, 0.f, 0.f});
    return PARTS ? (x[2] + x[1]) + x[0] : x[0];
}

// ---------------------------------------------------------------- global -> registers -> LDS tiles
// A tile of ROWS rows is ROWS*CPR chunks of 16 bytes; thread t owns chunks t, t + 512, ...  Loads are
// issued ahead of use (fetch) and written to LDS later (store), so that HBM latency overlaps arithmetic.
template <class C, int ROWS>
struct RowChunks {
    static constexpr int N = (ROWS * C::CPR + kThreads - 1) / kThreads;
    static constexpr bool EVEN = ROWS * C::CPR % kThreads == 0;        // every thread's chunks are inside the tile
    u32x4 v[N];
};

// Every lane loads, unconditionally: rows past the end of the tile (nvalid >= 1 rows are real) re-read the last real row.
// Such rows stay in the tiles as they are: their assignments are zeros, so they reach neither statistics nor other
// tokens, and their own results are not stored.  (A load under a condition, into registers cleared first, makes the
// compiler wait for every load in flight before the clearing moves: the loads of a tile would complete one by one.)
// The address is a uniform base plus a 32-bit byte offset per lane, which lets the loads take their base from scalar
// registers.
template <class C, int ROWS>
__device__ __forceinline__ void fetch_rows(const bf16raw *X, int64_t t0, int nvalid, RowChunks<C, ROWS> &r)
{
    const char *base = reinterpret_cast<const char *>(X + t0 * C::D);
#pragma unroll
    for (int k = 0; k < RowChunks<C, ROWS>::N; ++k) {
        const int c = threadIdx.x + k * kThreads, row = c / C::CPR, ch = c % C::CPR;
        const int rr = row < nvalid ? row : nvalid - 1;
        r.v[k] = *reinterpret_cast<const u32x4 *>(base + static_cast<uint32_t>((rr * C::D + ch * 8) * 2));
    }
}

// Column order of a row-major tile: as they are; or, in groups of 32, the eight features {4q .. 4q+3, 16 + 4q .. 16 + 4q+3} that a lane
// of a 16 x 16 x 32 product holds in two accumulator tiles as neighbours (position 8 q + 4 (c / 16) + c % 4; a 16-byte chunk's two
// blocks of 4 land 8 positions apart).
enum Order { kPlain = 0, kPairs32 = 1 };

// A 32-row tile, every thread's chunk (columns 8 ch .. 8 ch + 7 of its row) at the byte offset `at` from the tile (its place under STRIDE,
// worked out once per kernel).
template <class C, int STRIDE, int ORDER>
__device__ __forceinline__ int chunk_offset(int tid)
{
    const int row = tid / C::CPR, ch = tid % C::CPR;
    return (row * STRIDE + (ORDER == kPlain ? 8 * ch : 32 * (ch >> 2) + 16 * (ch & 1) + 4 * ((ch >> 1) & 1))) * 2;
}
template <class C, int ORDER>
__device__ __forceinline__ void store_tile(const RowChunks<C, kTile> &r, unsigned char *at)
{
    static_assert(RowChunks<C, kTile>::N == 1, "one chunk per thread at most");
    if (!RowChunks<C, kTile>::EVEN && threadIdx.x >= kTile * C::CPR) return;
    const u32x4 v = r.v[0];
    if (ORDER == kPlain) {
        *reinterpret_cast<u32x4 *>(at) = v;
    } else {
        *reinterpret_cast<u32x2 *>(at) = u32x2{v.x, v.y};
        *reinterpret_cast<u32x2 *>(at + 16) = u32x2{v.z, v.w};
    }
}

// Rows, chunk by chunk, into a tile of row stride STRIDE, columns as they are.
template <class C, int ROWS, int STRIDE = C::XS>
__device__ __forceinline__ void store_rows(const RowChunks<C, ROWS> &r, bf16raw *dst, int step)
{
    const uint32_t tid = opaque(static_cast<int>(threadIdx.x), step) & (kThreads - 1);      // keeps the tile addresses out of long-lived registers
#pragma unroll
    for (int k = 0; k < RowChunks<C, ROWS>::N; ++k) {
        const uint32_t c = tid + k * kThreads, row = c / C::CPR, ch = c % C::CPR;
        if (RowChunks<C, ROWS>::EVEN || row < ROWS) *reinterpret_cast<u32x4 *>(dst + static_cast<int>(row) * STRIDE + static_cast<int>(ch) * 8) = r.v[k];
    }
}

// Unit-norm option (the setting |Q_i| = |K_j| = 1 of Theorem 1's proof): scale[row] = 1 / max(|x_row|, 1e-12) for the
// rows held in r, from the fp32 sum of squares of the stored elements.  (Rows past the end of a tile hold a copy of
// the last real row.)
template <class C, int ROWS>
__device__ __forceinline__ void store_row_scales(const RowChunks<C, ROWS> &r, float *scale, int step)
{
    const int tid = opaque(static_cast<int>(threadIdx.x), step);
#pragma unroll
    for (int k = 0; k < RowChunks<C, ROWS>::N; ++k) {
        const int c = tid + k * kThreads, row = c / C::CPR, ch = c % C::CPR;
        const uint32_t xw[4] = {r.v[k].x, r.v[k].y, r.v[k].z, r.v[k].w};
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) ss = dot2(xw[e], xw[e], ss);
        // the CPR threads of one row are consecutive lanes
#pragma unroll
        for (int m = C::CPR / 2; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
        if (ch == 0 && row < ROWS) scale[row] = __builtin_amdgcn_rsqf(fmaxf(ss, 1e-24f));
    }
}

// Read-out cotangent rows: gn = dO / e (e = L * Den) as bf16 rows, ge[row] = -(gn . O) as fp32 (= -(dO . O) / e).
template <class C, int ROWS>
struct CotChunks {
    RowChunks<C, ROWS> g, o;
    float den[RowChunks<C, ROWS>::N];
};

template <class C, int ROWS>
__device__ __forceinline__ void fetch_cotangent(const bf16raw *dO, const bf16raw *O, const float *den, int64_t t0,
                                                int nvalid, CotChunks<C, ROWS> &r)
{
    fetch_rows<C, ROWS>(dO, t0, nvalid, r.g);
    fetch_rows<C, ROWS>(O, t0, nvalid, r.o);
    const char *dbase = reinterpret_cast<const char *>(den + t0);
#pragma unroll
    for (int k = 0; k < RowChunks<C, ROWS>::N; ++k) {
        const int row = (threadIdx.x + k * kThreads) / C::CPR;
        const int rr = row < nvalid ? row : nvalid - 1;
        r.den[k] = *reinterpret_cast<const float *>(dbase + static_cast<uint32_t>(rr * 4));
    }
}

// Forms the cotangent rows of a tile, into LDS (dst, ge_parts) and into memory (Gout, ge_out: rows from t0 on), where the later
// passes read them back as plain rows.  ge_parts: [kParts][ROWS], see weight_part().
template <class C, int ROWS, int STRIDE>
__device__ __forceinline__ void store_cotangent(const CotChunks<C, ROWS> &r, bf16raw *dst, bf16raw *ge_parts, int L_real, int nvalid,
                                                bf16raw *Gout, float *ge_out, int64_t t0, int step)
{
    const int tid = opaque(static_cast<int>(threadIdx.x), step);
    char *gbase = reinterpret_cast<char *>(Gout + t0 * C::D);
#pragma unroll
    for (int k = 0; k < RowChunks<C, ROWS>::N; ++k) {
        const int c = tid + k * kThreads, row = c / C::CPR, ch = c % C::CPR;
        const float inv = r.den[k] > 0.f ? __builtin_amdgcn_rcpf(r.den[k] * static_cast<float>(L_real)) : 0.f;
        const uint32_t gw[4] = {r.g.v[k].x, r.g.v[k].y, r.g.v[k].z, r.g.v[k].w};
        const uint32_t ow[4] = {r.o.v[k].x, r.o.v[k].y, r.o.v[k].z, r.o.v[k].w};
        uint32_t out[4];
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            out[e] = pack2(bf_lo(gw[e]) * inv, bf_hi(gw[e]) * inv);
            // the extra column is formed from the rounded cotangents the matrix products will see: for a row of the
            // statistics made of few keys, V_j . gn + ge = (V_j - O_i) . gn then cancels as it does in exact arithmetic
            dot = dot2(out[e], ow[e], dot);
        }
        const u32x4 v = {out[0], out[1], out[2], out[3]};
        if (row < ROWS) *reinterpret_cast<u32x4 *>(dst + row * STRIDE + ch * 8) = v;
        if (row < nvalid) *reinterpret_cast<u32x4 *>(gbase + static_cast<uint32_t>((row * C::D + ch * 8) * 2)) = v;
        // the CPR threads of one row are consecutive lanes
#pragma unroll
        for (int m = C::CPR / 2; m >= 1; m >>= 1) dot += __shfl_xor(dot, m, 64);
        if (ch < kParts && row < ROWS) ge_parts[ch * ROWS + row] = weight_part(-dot, ch);
        if (ch == 0 && row < nvalid) ge_out[t0 + row] = -dot;
    }
}

// ---------------------------------------------------------------- projection + soft assignment
// The hashed form of one projection: c = +small or -small, where small = sigmoid(-2 beta |tanh z|) is the mass of the
// bit's minor side and the sign bit tells which side that is (clear: z >= 0, the major side is +1).  One float per
// (token, table, hyperplane) is all that the soft assignment of Algorithm 1, step 4 depends on: every pass after the
// first rebuilds phi from it instead of projecting and exponentiating again.  beta = +infinity gives +-0 (the hard
// hash); a padding hyperplane is +0 (all mass on the +1 side).
__device__ __forceinline__ float bit_code(float zt, float beta)
{
    const float e2 = __expf(-2.0f * fabsf(zt));
    const float ua = (1.0f - e2) * __builtin_amdgcn_rcpf(1.0f + e2);             // |tanh z|
    const float e = __expf(fmaxf(-2.0f * beta * ua, -1e30f));                    // (-inf * 0 = NaN at z = 0: fmaxf returns -1e30)
    const float small = e * __builtin_amdgcn_rcpf(1.0f + e);
    return zt >= 0.f ? small : -small;
}
// masses on the +1 side (p) and the -1 side (q) from the hashed form
__device__ __forceinline__ void code_masses(float c, float &p, float &q)
{
    const float small = fabsf(c), big = 1.0f - small;
    const bool pos = (__float_as_uint(c) >> 31) == 0;
    p = pos ? big : small;
    q = pos ? small : big;
}

// the mass on one side (bit != 0: +1), and the product of the two
__device__ __forceinline__ float side_mass(float c, int bit)
{
    const float small = fabsf(c);
    return ((__float_as_uint(c) >> 31) != 0) == (bit != 0) ? small : 1.0f - small;
}
__device__ __forceinline__ float minor_major(float c) { return fabsf(c) * (1.0f - fabsf(c)); }

// Hashed rows of NTAB tables for one token per lane.
template <class C, int NTAB>
struct Codes {
    float c[NTAB][C::P];
};
// Mt: uniform; lane_off: table_offset() of the lane's table and token, worked out once per kernel
template <class C>
__device__ __forceinline__ uint32_t table_offset(int table, int ln) { return static_cast<uint32_t>(table * C::HT + 4 * ln) * 4u; }
template <class C>
__device__ __forceinline__ void load_table_codes(const float *Mt, uint32_t lane_off, int ln, float *c)
{
    const char *src = reinterpret_cast<const char *>(Mt);
    const float4 a = *reinterpret_cast<const float4 *>(src + lane_off);
    c[0] = a.x; c[1] = a.y; c[2] = a.z; c[3] = a.w;
    if (C::P == 6) {
        const float2 b = *reinterpret_cast<const float2 *>(src + 16 * kTile + (lane_off - 8u * ln));
        c[4] = b.x; c[5] = b.y;
    }
}

// Production: SLOTS half wavefronts share the tables of a tile of 32 tokens (lane = token).  Half wavefront `slot` takes
// tables NTAB slot .. NTAB slot + NTAB - 1; with fewer tables than slots, two share a table (the lower and upper half of its
// 16-byte pieces) and the rest are idle.
template <class C, int SLOTS>
struct Share {
    static constexpr int NTAB = C::L >= SLOTS ? C::L / SLOTS : 1;
    static constexpr int PARTS = C::L >= SLOTS ? 1 : 2;
    static_assert(C::L >= SLOTS ? C::L % SLOTS == 0 : SLOTS % C::L == 0, "tables over half wavefronts");
    __device__ static __forceinline__ int table(int slot, int i) { return PARTS == 1 ? slot * NTAB + i : slot % C::L; }
    __device__ static __forceinline__ int part(int slot) { return PARTS == 1 ? 0 : slot / C::L; }       // >= PARTS: idle
    typedef Codes<C, NTAB> Regs;
    // Mt: the tile's hashed rows; lane_off: table_offset() of table(slot, 0)
    __device__ static __forceinline__ void load(const float *Mt, uint32_t lane_off, int ln, Regs &r)
    {
#pragma unroll
        for (int i = 0; i < NTAB; ++i) load_table_codes<C>(Mt + i * C::HT, lane_off, ln, r.c[i]);
    }
};

// Hashed rows formed where they are used: the tables of a wavefront's two half wavefronts (slots 2 a and 2 a + 1 of Share) are at most
// 16 packed rows of W, projected as two 16 x 16 tiles of 16 tokens whose rows 4 q + v are, for q = 2 h + i, quad i of the hyperplanes
// (P = 6) or table i (P = 4) of half wavefront h.  Swapping rows of 16 lanes between the two tiles then leaves every lane with all
// projections of its token and tables.  W stays in registers, the rows come from an LDS tile [tokens][XS].
template <class C, int SLOTS>
struct Hasher {
    using Sh = Share<C, SLOTS>;
    u32x4 w[C::D / 32];
    __device__ __forceinline__ void load(const bf16raw *Wp, int a, int lane)
    {
        const int m = lane & 15, q = m >> 2, hh = q >> 1, i = q & 1;
        const int row = C::PP == 8 ? Sh::table(2 * a + hh, 0) * 8 + 4 * i + (m & 3) : Sh::table(2 * a + hh, i < Sh::NTAB ? i : 0) * 4 + (m & 3);
#pragma unroll
        for (int s = 0; s < C::D / 32; ++s) w[s] = *reinterpret_cast<const u32x4 *>(Wp + row * C::D + 32 * s + 8 * (lane >> 4));
    }
    // the tile's rows as operands; row_of: where a token's row begins
    struct Rows { u32x4 x[2][C::D / 32]; };
    template <class RowOf>
    __device__ __forceinline__ static void fetch(RowOf row_of, int lane, Rows &r)
    {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16raw *row = row_of(16 * t + (lane & 15)) + 8 * (lane >> 4);
#pragma unroll
            for (int s = 0; s < C::D / 32; ++s) r.x[t][s] = *reinterpret_cast<const u32x4 *>(row + 32 * s);
        }
    }
    // x: an LDS tile [tokens][XS]; M: where the tile's hashed rows go (null: nowhere)
    template <bool UNIT>
    __device__ __forceinline__ void run(const bf16raw *x, int slot, int lane, const Soft &sf, float *M, typename Sh::Regs &r) const
    {
        Rows rows;
        fetch([&](int token) __attribute__((always_inline)) { return x + token * C::XS; }, lane, rows);
        run_rows<UNIT>(rows, slot, lane, sf, M, r);
    }
    template <bool UNIT>
    __device__ __forceinline__ void run_rows(const Rows &rows, int slot, int lane, const Soft &sf, float *M, typename Sh::Regs &r) const
    {
        const int ln = lane & 31;
        f32x4 z[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const u32x4 (&xv)[C::D / 32] = rows.x[t];
            z[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < C::D / 32; ++s) z[t] = mma16(w[s], xv[s], z[t]);
            if (UNIT) {
                // 1 / max(|x|, 1e-12), from the fp32 sum of squares of the stored elements
                float ss = 0.f;
#pragma unroll
                for (int s = 0; s < C::D / 32; ++s) ss = dot2(xv[s].x, xv[s].x, dot2(xv[s].y, xv[s].y, dot2(xv[s].z, xv[s].z, dot2(xv[s].w, xv[s].w, ss))));
                z[t] = z[t] * __builtin_amdgcn_rsqf(fmaxf(sum_rows(ss), 1e-24f));
            }
        }
        float zz[2][4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(z[0][v]), __float_as_uint(z[1][v]), false, false);
            zz[0][v] = __uint_as_float(s[0]);
            zz[1][v] = __uint_as_float(s[1]);
        }
#pragma unroll
        for (int i = 0; i < Sh::NTAB; ++i) {
            const int table = Sh::table(slot, i);
#pragma unroll
            for (int t = 0; t < C::P; ++t) {
                const float code = bit_code(C::PP == 8 ? zz[t / 4][t % 4] : zz[i][t], sf.beta);      // (worked out in any case: no branch)
                r.c[i][t] = !C::PAD || (table < sf.L && t < sf.P) ? code : 0.f;
            }
            if (!M || Sh::part(slot) > 0) continue;
            float *dst = M + table * C::HT;
            *reinterpret_cast<float4 *>(dst + 4 * ln) = float4{r.c[i][0], r.c[i][1], r.c[i][2], r.c[i][3]};
            if (C::P == 6) *reinterpret_cast<float2 *>(dst + 4 * kTile + 2 * ln) = float2{r.c[i][4], r.c[i][5]};
        }
    }
};

// Writes the half wavefront's share of the assignments of the lane's token as bf16 into row `row` of ph [token][L*R] (row
// stride STRIDE): phi[a * 8 + b] = hi[a] * lo[b] (the corner softmax is a product of per-bit two-point distributions; a: bits
// 3.., b: bits 0..2), corners pair-interleaved: the 16 corners of high-bit indices (a, a+1), a even, are stored as
// [a: b 0..3 | a+1: b 0..3 | a: b 4..7 | a+1: b 4..7].
// valid == false writes zeros (a token past the end of the sequence must not reach the statistics).
// MASS: returns sum_r phi[r] * mass[r] over what was written (bucket masses in the same pair-interleaved order): the read-out of the
// bucket masses A by this token, i.e. its share of the normaliser.  (As a test of the pointer every use of it was a branch.)
template <class C, int SLOTS, int STRIDE, bool MASS = false>
__device__ __forceinline__ float produce(const typename Share<C, SLOTS>::Regs &codes, int slot, int row, const Soft &sf, bool valid,
                                         bf16raw *ph, int step, const float *mass = nullptr)
{
    using Sh = Share<C, SLOTS>;
    static_assert(C::PLO == 3 && C::PHI >= 1, "eight low corners per high-bit index, indices in pairs");
    constexpr int NA = 1 << C::PHI;
    // two shares of a table: halves of the high-bit indices if there are two pairs of them, else of the low corners
    constexpr bool kSplitA = Sh::PARTS == 2 && C::PHI >= 2;
    const int part = Sh::part(slot);
    float dn[4] = {0.f, 0.f, 0.f, 0.f};
    if (part >= Sh::PARTS) return 0.f;
#pragma unroll
    for (int i = 0; i < Sh::NTAB; ++i) {
        const int table = Sh::table(slot, i);
        const bool live = valid && (!C::PAD || table < sf.L);     // (a padding table: zero assignments)
        const int tbase = opaque(table * C::R, step);                   // one base register, constants folded into offsets
        bf16raw *prow = ph + opaque(row * STRIDE, step);
        float p[C::P], q[C::P], lo[8], hi[NA];
#pragma unroll
        for (int t = 0; t < C::P; ++t) code_masses(codes.c[i][t], p[t], q[t]);
        lo[0] = q[0] * q[1]; lo[1] = p[0] * q[1]; lo[2] = q[0] * p[1]; lo[3] = p[0] * p[1];
#pragma unroll
        for (int b = 0; b < 4; ++b) { lo[4 + b] = lo[b] * p[2]; lo[b] = lo[b] * q[2]; }
        // with a split over the high-bit indices the top bit is this share's
        constexpr int kTop = kSplitA ? C::P - 1 : C::P;
        hi[0] = !live ? 0.f : (kSplitA ? (part ? p[C::P - 1] : q[C::P - 1]) : 1.f);
#pragma unroll
        for (int t = 3; t < kTop; ++t) {
#pragma unroll
            for (int b = 0; b < (1 << (t - 3)); ++b) {
                hi[b + (1 << (t - 3))] = hi[b] * p[t];
                hi[b] = hi[b] * q[t];
            }
        }
        constexpr int kA = kSplitA ? NA / 2 : NA;
        const int abase = kSplitA ? part * (NA / 2) * 8 : 0;
        // (the masses of a pair are requested one pair ahead: read where they are used, their latency was a third of the
        // production's time)
        float4 next[4];
        auto load_masses = [&](int a) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) next[i] = *reinterpret_cast<const float4 *>(mass + tbase + abase + a * 8 + 4 * i);
        };
        if (MASS) load_masses(0);
#pragma unroll
        for (int a = 0; a < kA; a += 2) {
            const float ha[2] = {hi[a], hi[a + 1]};
            float4 mq[4];
            if (MASS) {
#pragma unroll
                for (int i = 0; i < 4; ++i) mq[i] = next[i];
                if (a + 2 < kA) load_masses(a + 2);
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (Sh::PARTS == 2 && !kSplitA && half != part) continue;
                const int pos = tbase + abase + a * 8 + 8 * half;
                const float4 m0 = mq[2 * half], m1 = mq[2 * half + 1];
                float f[8];
#pragma unroll
                for (int b = 0; b < 4; ++b) { f[b] = ha[0] * lo[4 * half + b]; f[4 + b] = ha[1] * lo[4 * half + b]; }
                if (MASS) {
                    dn[0] = fmaf(f[0], m0.x, dn[0]); dn[1] = fmaf(f[1], m0.y, dn[1]); dn[2] = fmaf(f[2], m0.z, dn[2]); dn[3] = fmaf(f[3], m0.w, dn[3]);
                    dn[0] = fmaf(f[4], m1.x, dn[0]); dn[1] = fmaf(f[5], m1.y, dn[1]); dn[2] = fmaf(f[6], m1.z, dn[2]); dn[3] = fmaf(f[7], m1.w, dn[3]);
                }
                *reinterpret_cast<u32x4 *>(prow + pos) =
                    u32x4{pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7])};
            }
            if (MASS) asm volatile("" : "+v"(dn[0]), "+v"(dn[1]), "+v"(dn[2]), "+v"(dn[3]));    // (else the sums wait, with all products and masses, for the last pair)
            RACE_SCHED_FENCE();
        }
    }
    return (dn[0] + dn[1]) + (dn[2] + dn[3]);
}

// One table's assignments of 32 tokens by the wavefront that uses them (lane = token ln, half h of the corners: bit 2 is h), into
// its own columns of ph.
template <class C, int STRIDE>      // (rows at spread_row())
__device__ __forceinline__ void produce_table(const float (&c)[C::P], int table, int ln, int h, const Soft &sf, bool valid, bf16raw *ph, int step)
{
    static_assert(C::PLO == 3 && C::PHI >= 1, "eight low corners per high-bit index, indices in pairs");
    constexpr int NA = 1 << C::PHI;
    const bool live = valid && (!C::PAD || table < sf.L);
    float p[C::P], q[C::P], lo[4], hi[NA];
#pragma unroll
    for (int t = 0; t < C::P; ++t) code_masses(c[t], p[t], q[t]);
    const float m2 = h ? p[2] : q[2];
    lo[0] = q[0] * q[1] * m2; lo[1] = p[0] * q[1] * m2; lo[2] = q[0] * p[1] * m2; lo[3] = p[0] * p[1] * m2;
    hi[0] = live ? 1.f : 0.f;
#pragma unroll
    for (int t = 3; t < C::P; ++t) {
#pragma unroll
        for (int b = 0; b < (1 << (t - 3)); ++b) {
            hi[b + (1 << (t - 3))] = hi[b] * p[t];
            hi[b] = hi[b] * q[t];
        }
    }
    bf16raw *dst = ph + opaque(spread_row(ln) * STRIDE + table * C::R + 8 * h, step);
#pragma unroll
    for (int a = 0; a < NA; a += 2) {
        float f[8];
#pragma unroll
        for (int b = 0; b < 4; ++b) { f[b] = hi[a] * lo[b]; f[4 + b] = hi[a + 1] * lo[b]; }
        *reinterpret_cast<u32x4 *>(dst + 8 * a) = u32x4{pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7])};
    }
}

// Stores whose lanes are dropped by the address check where they lie past `bytes` (a store under a condition is a branch, behind
// which the compiler no longer knows how many of the loads issued before it are in flight, and waits for too many).
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t store_buffer(void *base, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000); }
__device__ __forceinline__ void buffer_store128(buffer_t b, int offset, u32x4 v) { __builtin_amdgcn_raw_buffer_store_b128(v, b, offset, 0, 0); }

}  // namespace mfma
}  // namespace race
