// bf16 MFMA kernel family for RACE Attention on gfx950 (see mfma_common.h for the execution shape).
//
// Kernels
//   hashed rows      projection and per-bit soft-hash masses of every row of Q and K, once per call: one float per token, table and
//                    hyperplane that every later pass rebuilds phi from.  Formed by hash_kernel or, by a rule on the sizes
//                    (hashing_pays()), in the passes of the forward: the totals form K's, the replay Q's (Hasher).
//   totals_kernel    statistics of every segment from a zero start, of (phi_K, [V | 1]) (Algorithm 1, step 5) or, for the
//                    backward pass, of (phi_Q, read-out cotangents); an exclusive prefix (forward) or suffix (backward)
//                    scan over segments (scan_states) turns them into segment-start states.
//   stream_kernel    one pass over a segment carrying statistics [L*R][d] in accumulator registers
//                    as tiles (bucket rows x head columns).  Modes:
//                      kForward   Algorithm 2's loop / Algorithm 1's read-out: O and Den
//                      kGradV     the mirrored pass, right to left: dV
//   grad_kernel      (mfma_grad.h) the passes that contract over the head dimension: dQ and dK.
#include <hip/hip_runtime.h>

#include "internal.h"
#include <algorithm>
#include <cstring>

#include "mfma_common.h"
#include "mfma_grad.h"

namespace race {
namespace mfma {

enum Mode { kForward, kGradV };

// state element (bucket row r, column c) in the saved layout: B [LR][D] row-major, then A [LR]
template <class C>
__device__ __forceinline__ int state_b(int r, int c) { return r * C::D + c; }
template <class C>
__device__ __forceinline__ int state_a(int r) { return C::LR * C::D + r; }

// ================================================================ hash_kernel
// Algorithm 1, steps 2-4 up to the per-bit masses, for every row of a tensor (blockIdx.z: of one or the other): one float per (table,
// hyperplane), see bit_code().  For calls whose passes do not hash for themselves: see hashing_pays(), and race_attn_bwd, whose
// pass over Q would be the forward's.  The same arithmetic as theirs (Hasher), the rows straight from memory: no LDS, no barrier.
// Bound by the latency of one tile where there are few, by memory where there are many.  (Q and K of two sequences of 2000 tokens, (128, 8,
// 6), all shares of a tile in one wavefront: 6.3 us, each in its own 4.8; of eight of 5000, (128, 8, 4), in shares of the passes' eight half
// wavefronts 12.3, of four 9.8.)
constexpr int kHashThreads = 256;
constexpr int kHashTokens = 512;        // most tokens per workgroup (amortises the load of W)
// Half wavefronts that share a tile's tables here, so that a wavefront's 16 rows of an MFMA tile are 16 packed rows of W (in the passes,
// which share eight ways, (4, 8) and (4, 4) fill half of them).
template <class C> constexpr int hash_slots() { return C::P == 6 ? C::L : C::L / 2; }
template <class C> constexpr int hash_shares() { return hash_slots<C>() / 2; }

// This wavefront's SHARES shares, from `share` on, of tiles first, first + stride, ... < end of one (batch, head) (X, M: its first
// row's; Wp: its head's), the next tile's rows requested before a tile's arithmetic.
template <class C, bool UNIT, int SHARES>
__device__ __forceinline__ void hash_tiles(const KArgs &a, const bf16raw *X, const bf16raw *Wp, float *M, int share, int64_t first, int64_t end,
                                           int stride, int lane)
{
    using Hash = Hasher<C, hash_slots<C>()>;
    Hash hasher[SHARES];
#pragma unroll
    for (int i = 0; i < SHARES; ++i) hasher[i].load(Wp, share + i, lane);
    auto fetch = [&](int64_t tile, typename Hash::Rows &rows) __attribute__((always_inline)) {
        // (rows past the end repeat the last one: finite values in the padding of the last tile)
        Hash::fetch([&](int token) __attribute__((always_inline)) {
            const int64_t t = tile * kTile + token;
            return X + (t < a.N ? t : a.N - 1) * C::D;
        }, lane, rows);
    };
    typename Hash::Rows rows;
    if (first < end) fetch(first, rows);
    for (int64_t tile = first; tile < end; tile += stride) {
        const typename Hash::Rows now = rows;
        if (tile + stride < end) fetch(tile + stride, rows);
#pragma unroll
        for (int i = 0; i < SHARES; ++i) {
            typename Hash::Sh::Regs codes;
            hasher[i].template run_rows<UNIT>(now, 2 * (share + i) + (lane >> 5), lane, a.soft(), M + tile * (kTile * C::LP), codes);
        }
    }
}

template <class C, bool UNIT, int SHARES>
__global__ __launch_bounds__(kHashThreads) void hash_kernel(KArgs a, const bf16raw *X, float *M, const bf16raw *X1, float *M1)
{
    if (blockIdx.z) { X = X1; M = M1; }
    const int bh = blockIdx.y;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t all_tiles = (a.N + kTile - 1) / kTile;
    const int64_t t_first = static_cast<int64_t>(blockIdx.x) * (a.hash_tokens / kTile);
    const int64_t t_end = (t_first + a.hash_tokens / kTile < all_tiles) ? t_first + a.hash_tokens / kTile : all_tiles;
    constexpr int kParties = hash_shares<C>() / SHARES;         // wavefronts on a tile
    hash_tiles<C, UNIT, SHARES>(a, X + static_cast<size_t>(bh) * a.N * C::D, a.Wp + static_cast<size_t>(bh % a.H) * C::LPP * C::D,
                                M + static_cast<size_t>(bh) * all_tiles * kTile * C::LP, SHARES * (w % kParties), t_first + w / kParties, t_end,
                                kHashThreads / 64 / kParties, lane);
}

// ================================================================ totals_kernel
// Statistics of one segment from a zero start, 64 tokens per step (each half of the workgroup builds the assignments of
// 32 tokens).  QG == 0: (phi_K, [V | 1]), Algorithm 1 step 5.  QG == 1: (phi_Q, [dO/e | -(dO.O)/e]),
// the statistics the key side of the backward pass reads.
template <class C>
struct TotalsLds {
    static constexpr int TT = 64;
    static constexpr int y = 0;                                         // [64][YS] accumulated rows
    static constexpr int ph = y + TT * C::YS * 2;                       // [64][PS] assignments
    static constexpr int ge = ph + TT * C::PS * 2;                     // [kParts][64] bf16
    static constexpr int x = ge + kParts * TT * 2;                      // [64][XS] rows of K (HASH)
    static constexpr int total = x, total_hash = x + TT * C::XS * 2;
    static_assert(total_hash <= 160 * 1024, "LDS budget");
};

// The wavefronts of a row group share its row tiles' extra column: the one of column group cg takes the MA tiles that come first in
// its own order, which starts at tile cg MA.  (Ownership by the tile's number was a branch around every tile's sum: the loads of the
// products of one tile waited behind those of the one before it.  A single tile is the first one's.)
// First bucket row of the mt-th tile in that order:
template <class C>
__device__ __forceinline__ int tile_row(int r_own, int mt, int cg) { return r_own + 32 * ((mt / C::MA + cg) % C::CG * C::MA % C::MT + mt % C::MA); }

// HASH (QG == 0): hashes the rows of K (X) itself and leaves the hashed rows in memory (M; null: nobody reads them): the pass over K that
// hashed it before, and the pass over its hashed rows here, are one.  Next to the products' latencies the projection and the
// exponentials cost less than their own kernel at the memory's rate (see hashing_pays()), also at (128, 4, 16) and (64, 6, 8), where they
// take the second workgroup's place on a CU (160 to 164 registers, 118 to 122 without; held to 128 the first spills, the second's LDS is
// past 80 KB with the rows of K).  B H = 64, N = 8192, causal, us, kernel for Q and K, totals, replay: 108 + 59 + 191, in the passes 100 + 235;
// (64, 6, 8) 67 + 64 + 209, 91 + 215.  Else M are the hashed rows of K or, QG == 1, of Q.  QG == 1 also leaves the
// cotangent rows it forms in memory, rows in Gout (the caller's buffer for dK, which nothing else uses before dK is
// written, tile behind tile of its own reading) and the extra column in a.ge: the passes behind it then read 260 bytes a token instead of dO,
// O and Den, and do not form the rows again (35 of 750 vector instructions a tile and wavefront).
template <class C, int QG, bool HASH, bool UNIT>
__global__ __launch_bounds__(kThreads, (C::MT * C::NTW <= 2 ? 4 : 2))      // (two workgroups on a CU where their registers fit it)
void totals_kernel(KArgs a, float *M, const bf16raw *X, const bf16raw *Y, const bf16raw *Oin, const float *den_in, bf16raw *Gout)
{
    using S = TotalsLds<C>;
    constexpr int TT = S::TT;
    extern __shared__ __attribute__((aligned(256))) unsigned char lds[];
    bf16raw *ys = reinterpret_cast<bf16raw *>(lds + S::y);
    bf16raw *ph = reinterpret_cast<bf16raw *>(lds + S::ph);
    bf16raw *ge_lds = reinterpret_cast<bf16raw *>(lds + S::ge);
    bf16raw *xs = reinterpret_cast<bf16raw *>(lds + S::x);

    const int seg = blockIdx.x, bh = blockIdx.y;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, h = lane >> 5;
    const int rg = w % C::RG, cg = w / C::RG;
    const int r_own = rg * C::LRW, c_own = cg * C::DW;
    const size_t base = static_cast<size_t>(bh) * a.N * C::D;
    if (M) M += static_cast<size_t>(bh) * ((a.N + kTile - 1) / kTile) * (kTile * C::LP);
    Y += base;
    if (HASH) X += base;
    float *ge_out = a.ge + static_cast<size_t>(bh) * a.N;
    if (QG) { Oin += base; Gout += base; den_in += static_cast<size_t>(bh) * a.N; }
    float *st = a.state + (static_cast<size_t>(bh) * a.nseg + seg) * C::STATE;
    // causal: the totals of the last segment (backward: of the first) are in no other segment's start state
    // (the last segment's rows of K are hashed all the same, and nothing else is done for it: a forward call of B H = 80, N = 4000, three
    // segments, (128, 8, 6), 271 us when it ran the whole loop, 265; N = 1500, B H = 128, two, 173 and 166)
    const bool unread = a.scanned && seg == (QG ? 0 : a.nseg - 1);
    if (!QG && unread) {
        if (HASH) {
            constexpr int kShares = hash_shares<C>();
            const int64_t t0 = static_cast<int64_t>(seg) * a.seg_len, t1 = t0 + a.seg_len < a.N ? t0 + a.seg_len : a.N;
            hash_tiles<C, UNIT, 1>(a, X, a.Wp + static_cast<size_t>(bh % a.H) * C::LPP * C::D, M, w % kShares, t0 / kTile + w / kShares,
                                   (t1 + kTile - 1) / kTile, kWaves / kShares, lane);
        }
        return;
    }

    f32x16 Sacc[C::MT][C::NTW];
    float macc[C::MA];                 // extra column of the first row tiles: lane n <-> row, per-half partial sums
#pragma unroll
    for (int i = 0; i < C::MA; ++i) macc[i] = 0.f;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
#pragma unroll
        for (int nt = 0; nt < C::NTW; ++nt) Sacc[mt][nt] = f32x16{0};
    }
    const int64_t t_begin = seg * a.seg_len;
    const int64_t t_end = (t_begin + a.seg_len < a.N) ? t_begin + a.seg_len : a.N;
    const int nsteps = static_cast<int>((t_end - t_begin + TT - 1) / TT);
    auto step_nv = [&](int64_t t0) { return (t_end - t0 < TT) ? static_cast<int>(t_end - t0) : TT; };

    // this wavefront's tokens of a step (its half) and its lanes' share of the tables
    const int half = w / 4, slot = 2 * (w % 4) + h, row = half * kTile + ln;
    const uint32_t lane_off = table_offset<C>(Share<C, 8>::table(slot, 0), ln);
    const bf16raw *ge_lane = ge_lds + parts_offset32<false>(TT, lane);
    typename Share<C, 8>::Regs pre_m;
    RowChunks<C, TT> pre_y, pre_x;
    CotChunks<C, TT> pre_c;
    auto fetch = [&](int it) {
        const int64_t t0 = t_begin + static_cast<int64_t>(it) * TT;
        const int nv = step_nv(t0);
        // (the second half of the last step may lie past the end: it reads the first half's tile, and its tokens are not valid)
        const int64_t tile = t0 / kTile + (half && nv > kTile ? 1 : 0);
        if (!HASH) Share<C, 8>::load(M + tile * (kTile * C::LP), lane_off, ln, pre_m);
        if (QG) fetch_cotangent<C, TT>(Y, Oin, den_in, t0, nv, pre_c);
        else fetch_rows<C, TT>(Y, t0, nv, pre_y);
    };
    // rows of K: requested two steps ahead, in LDS one step ahead
    auto fetch_x = [&](int it) {
        const int64_t t0 = t_begin + static_cast<int64_t>(it < nsteps ? it : nsteps - 1) * TT;
        fetch_rows<C, TT>(X, t0, step_nv(t0), pre_x);
    };
    Hasher<C, 8> hasher;
    if (nsteps > 0) {
        if (HASH) {
            fetch_x(0);
            hasher.load(a.Wp + static_cast<size_t>(bh % a.H) * C::LPP * C::D, w % 4, lane);
        }
        fetch(0);
        if (HASH) {
            store_rows<C, TT, C::XS>(pre_x, xs, 0);
            fetch_x(1);
            __syncthreads();
        }
    }

    for (int it = 0; it < nsteps; ++it) {
        const int64_t t0 = t_begin + static_cast<int64_t>(it) * TT;
        const int nvalid = step_nv(t0);
        if constexpr (HASH) {
            const bool exists = half * kTile < nvalid;
            hasher.template run<UNIT>(xs + half * kTile * C::XS, slot, lane, a.soft(), exists && M ? M + (t0 / kTile + half) * (kTile * C::LP) : nullptr, pre_m);
        }
        produce<C, 8, C::PS>(pre_m, slot, half * kTile + spread_row(ln), a.soft(), row < nvalid, ph, it);
        if (QG) {
            wait_loads();
            store_cotangent<C, TT, C::YS>(pre_c, ys, ge_lds, a.L_real, nvalid, Gout, ge_out, t0, it);
        } else {
            store_rows<C, TT, C::YS>(pre_y, ys, it);
        }
        if (it + 1 < nsteps) fetch(it + 1);
        __syncthreads();
        // (two workgroups on a CU leave 128 registers, which (128, 4, 8) would pass with the rows of W kept)
        if (HASH && C::D == 128 && C::MT * C::NTW == 2) hasher.load(a.Wp + static_cast<size_t>(bh % a.H) * C::LPP * C::D, w % 4, opaque(lane, it));
#pragma unroll
        for (int s = 0; s < TT / 16; ++s) {
            u32x4 by[C::NTW];
#pragma unroll
            for (int nt = 0; nt < C::NTW; ++nt) by[nt] = lds_tr_plain(ys, C::YS, 16 * s, c_own + 32 * nt, ln, h);
            const u32x4 gw = QG ? lds128(ge_lane + 16 * s) : ones32<false>(lane);
#pragma unroll
            for (int mt = 0; mt < C::MT; ++mt) {
                const u32x4 ap = lds_tr_plain<true, true>(ph, C::PS, 16 * s, tile_row<C>(r_own, mt, cg), ln, h);
                if (mt < C::MA && (C::MT > 1 || cg == 0)) macc[mt] += column_sum<QG != 0>(gw, ap);      // the extra column (bucket mass, or its cotangent)
#pragma unroll
                for (int nt = 0; nt < C::NTW; ++nt) Sacc[mt][nt] = mma(ap, by[nt], Sacc[mt][nt]);
            }
        }
        if (HASH) {
            store_rows<C, TT, C::XS>(pre_x, xs, it);
            fetch_x(it + 2);
        }
        __syncthreads();
    }
    if (unread) return;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
#pragma unroll
        for (int nt = 0; nt < C::NTW; ++nt) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                st[state_b<C>(tile_row<C>(r_own, mt, cg) + acc_row(v, h), c_own + 32 * nt + ln)] = Sacc[mt][nt][v];
        }
        if (mt < C::MA) {
            const float tot = sum_halves(macc[mt]);
            if (h == 0 && (C::MT > 1 || cg == 0)) st[state_a<C>(tile_row<C>(r_own, mt, cg) + ln)] = tot;
        }
    }
}

// ================================================================ stream_kernel
// One pass over a segment carrying the statistics as tiles S[bucket row][head column].
//   kForward: Algorithm 2's loop body (Algorithm 1's read-out when not causal): O and Den.
//   kGradV  : the mirrored pass, right to left, over the cotangent statistics: dV.
// "reader" = tensor whose assignments read the statistics (Q forward, K for dV), "writer" = tensor
// whose assignments feed them (K forward, Q for dV), Y = rows accumulated (V forward, the
// cotangent rows for dV).
template <class C, bool NC>
struct StreamLds {
    // half wavefronts that share the production of a side: half of the workgroup.  (All of it where there is no writer's side: 182
    // instead of 169 us for the forward pass at B H = 64, N = 16384, (64, 4, 16).)
    static constexpr int SLOTS = 8;
    static constexpr int y = 0;                                         // [32][YS] bf16: accumulated rows
    static constexpr int mass = y + (NC ? 0 : kTile * C::YS * 2);       // [LR] fp32: bucket masses A before this tile, pair-interleaved
    static constexpr int dnp = mass + C::LR * 4;                        // [2][SLOTS / 2][32] fp32: mass read-outs per reader wavefront,
                                                                        // two buffers used by alternate tiles
    static constexpr int phr = (dnp + SLOTS * kTile * 4 + 255) & ~255;  // [32][PS] reader assignments
    static constexpr int phw = phr + kTile * C::PS * 2;                 // [32][PS] writer assignments
    // reduction over the bucket-row groups, in bytes of its own: a tile's sums are formed next to the production of the
    // following tile
    static constexpr int RS = C::D + 4;                                 // fp32 row stride: D numerators, 1 normaliser part
    static constexpr int red = (phw + (NC ? 0 : kTile * C::PS * 2) + 255) & ~255;  // [RG][32][RS] fp32
    static constexpr int total = red + C::RG * kTile * RS * 4;
    static constexpr int x = total, total_hash = x + kTile * C::XS * 2;  // [32][XS] rows of Q (HASH)
    static_assert(total_hash <= 160 * 1024 && (C::STREAM_WAVES_PER_SIMD < 4 || total_hash <= 80 * 1024), "LDS budget");
};

// NC: not causal (the in-tile term and the update are compiled out).
// Mr, Mw: the hashed rows of the reader and the writer tensor.  HASH (kForward): hashes the reader's rows itself (X: Q) and leaves them
// in Mr, see hashing_pays().
template <class C, int MODE, bool NC, bool HASH, bool UNIT>
__global__ __launch_bounds__(kThreads, C::STREAM_WAVES_PER_SIMD)
void stream_kernel(KArgs a, float *Mr, const float *Mw, const bf16raw *X, const bf16raw *Y, bf16raw *Out, float *den_out)
{
    using S = StreamLds<C, NC>;
    using Sh = Share<C, S::SLOTS>;
    extern __shared__ __attribute__((aligned(256))) unsigned char lds[];
    bf16raw *ytile = reinterpret_cast<bf16raw *>(lds + S::y);
    float *mass = reinterpret_cast<float *>(lds + S::mass);
    float *dnp = reinterpret_cast<float *>(lds + S::dnp);
    bf16raw *phr = reinterpret_cast<bf16raw *>(lds + S::phr);
    bf16raw *phw = reinterpret_cast<bf16raw *>(lds + S::phw);
    float *red = reinterpret_cast<float *>(lds + S::red);
    bf16raw *xs = reinterpret_cast<bf16raw *>(lds + S::x);

    constexpr bool kReverse = (MODE == kGradV);
    // Without the in-tile term half of the wavefronts have nothing to produce.  They finish the output under the others' production
    // either way; where the producing ones come to it last, the tile waits for them.  With the output first and no lead in the
    // second half dV takes 100.2 instead of 118.7 us at B H = 16, N = 65536, (d, L, P) = (128, 4, 4), 97.4 instead of 106.4 at B H = 8,
    // (128, 16, 4), 91.7 instead of 97.3 at (64, 8, 6), 102.1 and 102.8 at B H = 64, N = 16384, (64, 16, 4); the forward pass of 128
    // columns 107.9 instead of 111.7, 117.4 instead of 124.6 (86.1 and 85.5 at B H = 16, N = 16384, (128, 8, 6)).  The forward pass of 64
    // columns, whose output is half as long, has it last: 125.3 instead of 133.5 us at (64, 16, 4).
    constexpr bool kOutputFirst = NC && (MODE == kGradV || C::D == 128);
    const int seg = blockIdx.x, bh = blockIdx.y;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, h = lane >> 5;
    const int rg = w % C::RG, cg = w / C::RG;
    const int r_own = rg * C::LRW, c_own = cg * C::DW;
    constexpr bool intra = !NC;

    const size_t base = static_cast<size_t>(bh) * a.N * C::D;
    const size_t mbase = static_cast<size_t>(bh) * ((a.N + kTile - 1) / kTile) * (kTile * C::LP);
    Mr += mbase; Mw += mbase;
    Y += base; Out += base;
    if (HASH) X += base;
    if (MODE == kForward) den_out += static_cast<size_t>(bh) * a.N;
    // statistics at the start of the segment (not causal: the totals, which the scan leaves in the first segment's place)
    const float *st = a.state + (static_cast<size_t>(bh) * a.nseg + (NC ? 0 : seg)) * C::STATE;

    f32x16 Sacc[C::MT][C::NTW];
    float macc[C::MA];                 // bucket masses of the first row tiles: lane n <-> row, per-half partial sums
#pragma unroll
    for (int i = 0; i < C::MA; ++i) macc[i] = 0.f;
    // (causal: nothing precedes the first segment, right to left the last one, and the scan writes no state for it)
    const bool from_zero = !NC && seg == (kReverse ? a.nseg - 1 : 0);
    if (from_zero) {
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
#pragma unroll
            for (int nt = 0; nt < C::NTW; ++nt) Sacc[mt][nt] = f32x16{0};
        }
    } else {
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
#pragma unroll
            for (int nt = 0; nt < C::NTW; ++nt) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    Sacc[mt][nt][v] = st[state_b<C>(tile_row<C>(r_own, mt, cg) + acc_row(v, h), c_own + 32 * nt + ln)];
            }
        }
    }
    if (MODE == kForward) {
        // (behind the loads of the statistics, all of which are in flight together)
#pragma unroll
        for (int i = 0; i < C::MA; ++i)
            if (!from_zero) macc[i] = st[state_a<C>(tile_row<C>(r_own, i, cg) + ln)];
#pragma unroll
        for (int i = 0; i < C::MA; ++i) {
            macc[i] = h == 0 ? macc[i] : 0.f;
            if (h == 0) mass[tile_row<C>(r_own, i, cg) + il(ln)] = macc[i];
        }
    }

    const int64_t t_begin = seg * a.seg_len;
    const int64_t t_end = (t_begin + a.seg_len < a.N) ? t_begin + a.seg_len : a.N;
    const int ntiles = static_cast<int>((t_end - t_begin + kTile - 1) / kTile);
    auto tile_t0 = [&](int it) { return t_begin + static_cast<int64_t>(kReverse ? ntiles - 1 - it : it) * kTile; };
    auto tile_nv = [&](int64_t t0) { return (t_end - t0 < kTile) ? static_cast<int>(t_end - t0) : kTile; };

    // production: wavefronts 0-3 build the reader's assignments, 4-7 the writer's; a lane's token is ln, its tables by slot
    constexpr int kHalf = S::SLOTS / 2;
    const int side = w / kHalf, slot = 2 * (w % kHalf) + h;
    const uint32_t lane_off = table_offset<C>(Sh::table(slot, 0), ln);
    // loads run one tile ahead of the arithmetic
    typename Sh::Regs pre_m;
    RowChunks<C, kTile> pre_y;
    auto fetch = [&](int it) {
        const int64_t t0 = tile_t0(it);
        if (HASH ? side == 1 && intra : side == 0 || intra) Sh::load((side == 0 ? Mr : Mw) + t0 * C::LP, lane_off, ln, pre_m);
        if (intra) fetch_rows<C, kTile>(Y, t0, tile_nv(t0), pre_y);
    };
    // the reader's rows, in LDS at the end of the tile before theirs: requested behind its read-out, or, where a tile is that and little
    // more (not causal: 210 instead of 169 us at B H = 64, N = 16384, (64, 4, 16)), a tile earlier
    RowChunks<C, kTile> pre_x;
    auto fetch_x = [&](int it) {
        const int64_t t0 = tile_t0(it < ntiles ? it : ntiles - 1);
        fetch_rows<C, kTile>(X, t0, tile_nv(t0), pre_x);
    };
    // (the rows of W stay in registers; at (64, 4, 16), causal, whose 128 are full, they are read again for every tile)
    constexpr bool kReloadW = HASH && !NC && C::STREAM_WAVES_PER_SIMD == 4 && C::LR == 256;
    Hasher<C, S::SLOTS> hasher;
    const bf16raw *Wp = a.Wp + static_cast<size_t>(bh % a.H) * C::LPP * C::D;
    if (ntiles > 0) {
        if (HASH) {
            fetch_x(0);
            hasher.load(Wp, w % kHalf, lane);
        }
        fetch(0);
        if (HASH) {
            store_rows<C, kTile>(pre_x, xs, 0);
            if (NC) fetch_x(1);
        }
    }

    // (NC: half of the work, and registers to keep the addresses in that the causal passes rebuild in every tile: 37.2 -> 36.3 us for
    // the forward pass and 30.4 -> 29.7 for dV at 32 workgroups of 32 tiles, (128, 4, 4))
    auto step = [&](int it) { return NC ? 0 : it; };
    // ---- epilogue of one tile: thread = (token, pieces of 4 columns: 4i.. and, for d = 128, 64 + 4i..; consecutive
    //      threads read consecutive 16-byte pieces of the partials): sum, normalise, store
    auto epilogue = [&](int it) __attribute__((always_inline)) {
        const int64_t t0 = tile_t0(it);
        const int nvalid = tile_nv(t0);
        const float *dnr = dnp + (it & 1) * (kHalf * kTile);
        {
        constexpr int NP = C::D / 64;                // pieces of 4 columns per thread
        const int to = opaque(tid, step(it)), tok = to >> 4, c0 = (to & 15) * 4;      // (addresses rebuilt per tile, not kept in registers)
        float acc[NP][4];
#pragma unroll
        for (int c = 0; c < NP; ++c) acc[c][0] = acc[c][1] = acc[c][2] = acc[c][3] = 0.f;
        float e = 0.f;
#pragma unroll
        for (int gg = 0; gg < kHalf; ++gg) {          // row groups (at most four) and the reader wavefronts
            const float *src = red + (gg * kTile + tok) * S::RS;
            if (gg < C::RG) {
#pragma unroll
                for (int c = 0; c < NP; ++c) {
                    const float4 p4 = *reinterpret_cast<const float4 *>(src + c0 + 64 * c);
                    acc[c][0] += p4.x; acc[c][1] += p4.y; acc[c][2] += p4.z; acc[c][3] += p4.w;
                }
            }
            if (MODE == kForward) {
                const float dpart = dnr[gg * 32 + tok];
                e += gg < C::RG ? src[C::D] + dpart : dpart;
            }
        }
        if (tok < nvalid) {
            const float scale = (MODE == kForward) ? (e > 0.f ? __builtin_amdgcn_rcpf(e) : 0.f) : 1.0f;   // e = 0: hard hash, empty buckets
            char *dst = reinterpret_cast<char *>(Out + t0 * C::D);
#pragma unroll
            for (int c = 0; c < NP; ++c)
                *reinterpret_cast<u32x2 *>(dst + static_cast<uint32_t>((tok * C::D + c0 + 64 * c) * 2)) =
                    u32x2{pack2(acc[c][0] * scale, acc[c][1] * scale), pack2(acc[c][2] * scale, acc[c][3] * scale)};
            if (MODE == kForward && (to & 15) == 0) (den_out + t0)[static_cast<uint32_t>(tok)] = e * a.inv_tables;
        }
    }
    };
    __syncthreads();        // the bucket masses and the first tile's reader rows are in place
    for (int it = 0; it < ntiles; ++it) {
        const int nvalid = tile_nv(tile_t0(it));
        // ---- first half: this tile's rows and assignments -> LDS, then the previous tile's output (its stores are issued when
        //      nothing loaded is waited for any more; in front of the production every tile waited for them to complete)
        if (kOutputFirst && it > 0) epilogue(it - 1);
        if (intra) store_rows<C, kTile, C::YS>(pre_y, ytile, it);
        if (side == 0) {
            if constexpr (HASH) hasher.template run<UNIT>(xs, slot, lane, a.soft(), Mr + tile_t0(it) * C::LP, pre_m);
            const float dnl = produce<C, S::SLOTS, C::PS, MODE == kForward>(pre_m, slot, spread_row(ln), a.soft(), true, phr, step(it), mass);
            if (MODE == kForward) {
                // this wavefront's tables' share of the normaliser
                const float both = sum_halves(dnl);
                if (h == 0) dnp[(it & 1) * (kHalf * kTile) + w * kTile + opaque(ln, step(it))] = both;
            }
        } else if (intra) {
            produce<C, S::SLOTS, C::PS>(pre_m, slot, spread_row(ln), a.soft(), ln < nvalid, phw, step(it));
        }
        if (!kOutputFirst && it > 0) epilogue(it - 1);
        __syncthreads();

        if (!kOutputFirst && w >= 4) lead(true);
        // ---- contraction with the register-resident statistics (own bucket rows x own columns)
        f32x16 out[C::NTW];     // read-out, transposed: lane = reader token, register v = column acc_row(v, h) of the tile
        f32x16 sct = {0};       // in-tile kernel values, transposed: row = writer token, lane = reader token
        float rowsum = 0.f;     // in-tile part of the normaliser, reader token = ln
#pragma unroll
        for (int nt = 0; nt < C::NTW; ++nt) out[nt] = f32x16{0};
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int rr = tile_row<C>(r_own, mt, cg) + 16 * s + 8 * h;      // pair-interleaved corners: one 16-byte read
                const u32x4 ar = lds128(phr + spread_row(ln) * C::PS + rr);
#pragma unroll
                for (int nt = 0; nt < C::NTW; ++nt) out[nt] = mma(acc_operand(Sacc[mt][nt], s), ar, out[nt]);
                if (intra) {
                    const u32x4 aw = lds128(phw + spread_row(ln) * C::PS + rr);
                    sct = mma(aw, ar, sct);
                }
                RACE_SCHED_FENCE();
            }
        }
        if (!kOutputFirst && w >= 4) lead(false);
        if (HASH && !NC) fetch_x(it + 1);
        if (kReloadW) hasher.load(Wp, w % kHalf, opaque(lane, it));
        if (intra) {
            // mask (writer token j = row, reader token i = lane), row sums, and (mask o kernel) . Y
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int j = acc_row(v, h);
                const bool keep = kReverse ? (j >= ln) : (j <= ln);
                sct[v] = keep ? sct[v] : 0.f;
                rowsum += sct[v];
            }
            rowsum += __shfl_xor(rowsum, 32, 64);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const u32x4 ak = acc_operand(sct, s);
#pragma unroll
                for (int nt = 0; nt < C::NTW; ++nt)
                    out[nt] = mma(lds_tr_acc(ytile, C::YS, 16 * s, c_own + 32 * nt, ln, h), ak, out[nt]);
            }
        }
        // the next tile's loads fly during the reduction and the update (few registers are live there)
        if (it + 1 < ntiles) fetch(it + 1);

        // ---- reduction over the bucket-row groups: partial read-outs through LDS, 16 bytes per store
        //      (a lane holds four consecutive columns of its token in registers 4k .. 4k+3), under the products of the update
        const int rbase = opaque((rg * kTile + ln) * S::RS + c_own + 4 * h, step(it));
#pragma unroll
        for (int nt = 0; nt < C::NTW; ++nt) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<float4 *>(red + rbase + 32 * nt + 8 * k) =
                    float4{out[nt][4 * k], out[nt][4 * k + 1], out[nt][4 * k + 2], out[nt][4 * k + 3]};
        }
        // in-tile part of the normaliser: row sums of the masked kernel values (partial over this row group)
        if (MODE == kForward && cg == 0 && h == 0) red[(rg * kTile + ln) * S::RS + C::D] = rowsum;
        if (intra) {
            // ---- statistics += phi_writer^T . Y  (the read-out above used the old statistics)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                u32x4 by[C::NTW];
#pragma unroll
                for (int nt = 0; nt < C::NTW; ++nt) by[nt] = lds_tr_plain(ytile, C::YS, 16 * s, c_own + 32 * nt, ln, h);
#pragma unroll
                for (int mt = 0; mt < C::MT; ++mt) {
                    const u32x4 ap = lds_tr_plain<true, true>(phw, C::PS, 16 * s, tile_row<C>(r_own, mt, cg), ln, h);
                    if (MODE == kForward && mt < C::MA && (C::MT > 1 || cg == 0)) macc[mt] += column_sum<false>(ones32<false>(opaque(lane, it)), ap);
#pragma unroll
                    for (int nt = 0; nt < C::NTW; ++nt) Sacc[mt][nt] = mma(ap, by[nt], Sacc[mt][nt]);
                    RACE_SCHED_FENCE();
                }
            }
        }
        if (MODE == kForward && intra) {
            // masses after this tile, for the next tile's read-out
#pragma unroll
            for (int mt = 0; mt < C::MA; ++mt) {
                const float tot = sum_halves(macc[mt]);
                if (h == 0 && (C::MT > 1 || cg == 0)) mass[tile_row<C>(r_own, mt, cg) + il(ln)] = tot;
            }
        }
        if (HASH) {
            store_rows<C, kTile>(pre_x, xs, it);
            if (NC) fetch_x(it + 2);
        }
        __syncthreads();
    }
    if (ntiles > 0) epilogue(ntiles - 1);
}

// Totals over all segments of the problem's own buckets, written as A[row * a_stride] and
// Bsum[row * b_stride + c] with row = (bh * L_real + l) * R_real + r.  Real corner r of a real table sits at
// the compiled corner with all padding bits set.  `groups` (a power of two, at most eight) threads share an element's segments and
// add them up in runs of eight, whose loads are requested together; more than 64 segments take several runs a thread.  (Bound by memory; one thread per element adding up 63 segments alone is bound by its chain of
// loads: 22.7 us at B H = 4, 264 KB a state.  Where there is one segment, as with many heads, a second thread has nothing to add.
// State of a prompt, one thread an element -> this: 4 x 30011 tokens 74.9 -> 67.6 us, 256 x 4096 320 -> 309 us.)
constexpr int kTapThreads = 512, kTapRun = 8, kTapMaxGroups = kTapThreads / 64;
inline int tap_groups(int nseg)
{
    int g = 1;
    while (g < kTapMaxGroups && g * kTapRun < nseg) g *= 2;
    return g;
}
template <class C>
__global__ __launch_bounds__(kTapThreads) void bucket_tap_kernel(const float *state, int nseg, int groups, int L_real, int P_real, float *A, float *Bsum,
                                  int a_stride, int b_stride)
{
    const int R_real = 1 << P_real, pad = (C::R - 1) & ~(R_real - 1);
    const uint32_t per = static_cast<uint32_t>(L_real) * R_real * (C::D + 1), elements = kTapThreads / groups;
    __shared__ float part[kTapThreads];
    const uint32_t x = threadIdx.x & (elements - 1);
    const int g = threadIdx.x / elements, run_len = (nseg + groups - 1) / groups;
    const size_t bh = blockIdx.y;
    const uint32_t at = blockIdx.x * elements + x;
    const uint32_t e = at < per ? at : per - 1;
    const uint32_t row = e / (C::D + 1), c = e % (C::D + 1), l = row / R_real, r = row % R_real;
    const uint32_t src = l * C::R + (r | pad);
    const uint32_t off = c < C::D ? src * C::D + c : C::LR * C::D + src;
    float run = 0.f;
    const float *base = state + bh * nseg * C::STATE + off;
    const int s1 = (g + 1) * run_len < nseg ? (g + 1) * run_len : nseg;
    if (nseg == 1) run = *base;
    else {
        for (int s = g * run_len; s < s1; s += kTapRun) {
            float v[kTapRun];
#pragma unroll
            for (int k = 0; k < kTapRun; ++k) v[k] = base[static_cast<size_t>(s + k < s1 ? s + k : s) * C::STATE];
#pragma unroll
            for (int k = 0; k < kTapRun; ++k) run += s + k < s1 ? v[k] : 0.f;
        }
    }
    if (groups > 1) {
        part[threadIdx.x] = run;
        __syncthreads();
    }
    if (g != 0 || at >= per) return;
    for (int k = 1; k < groups; ++k) run += part[k * elements + x];
    const size_t dst = (bh * L_real + l) * R_real + r;
    if (c < C::D) Bsum[dst * b_stride + c] = run;
    else A[dst * a_stride] = run;
}

// Debug tap: hard codes and phi from the passes' own hashing and production.
template <class C, bool UNIT>
__global__ __launch_bounds__(kThreads) void hash_tap_kernel(KArgs a, const bf16raw *X, uint8_t *codes, float *phi)
{
    extern __shared__ __attribute__((aligned(256))) unsigned char lds[];
    bf16raw *ph = reinterpret_cast<bf16raw *>(lds);                             // [32][PS]
    const int bh = blockIdx.y;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, h = lane >> 5;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int nvalid = (a.N - t0 < kTile) ? static_cast<int>(a.N - t0) : kTile;
    const Soft sf = a.soft();
    if (w < 4) {
        const int slot = 2 * w + h;
        X += (static_cast<size_t>(bh) * a.N + t0) * C::D;
        Hasher<C, 8> hasher;
        hasher.load(a.Wp + static_cast<size_t>(bh % a.H) * C::LPP * C::D, w, lane);
        typename Share<C, 8>::Regs r;
        typename Hasher<C, 8>::Rows rows;
        Hasher<C, 8>::fetch([&](int token) { return X + (token < nvalid ? token : nvalid - 1) * C::D; }, lane, rows);
        hasher.template run_rows<UNIT>(rows, slot, lane, sf, nullptr, r);
#pragma unroll
        for (int i = 0; i < Share<C, 8>::NTAB; ++i) {
            const int table = Share<C, 8>::table(slot, i);
            unsigned code = 0;
#pragma unroll
            for (int t = 0; t < C::P; ++t) code |= (t < a.P_real && (__float_as_uint(r.c[i][t]) >> 31) == 0 ? 1u : 0u) << t;      // (clear sign: z >= 0)
            if (Share<C, 8>::part(slot) == 0 && table < a.L_real && ln < nvalid)
                codes[(static_cast<size_t>(bh) * a.N + t0 + ln) * a.L_real + table] = static_cast<uint8_t>(code);
        }
        produce<C, 8, C::PS>(r, slot, ln, sf, true, ph, 0);
    }
    __syncthreads();
    if (phi) {
        // the problem's own corners: real corner r of a real table is the compiled corner with all padding bits set
        const int R_real = 1 << a.P_real, LR_real = a.L_real * R_real, pad = (C::R - 1) & ~(R_real - 1);
        for (int i = tid; i < nvalid * LR_real; i += kThreads) {
            const int row = i / LR_real, lr = i % LR_real, src = (lr / R_real) * C::R + ((lr % R_real) | pad);
            phi[(static_cast<size_t>(bh) * a.N + t0 + row) * LR_real + lr] =
                __uint_as_float(static_cast<uint32_t>(ph[row * C::PS + il(src)]) << 16);
        }
    }
}

// Attainable matrix rate: four independent accumulators per wavefront, operands from registers only.
// NV > 0: every matrix instruction is followed by NV independent vector multiplies on registers of the same
// wavefront (eight dependency chains), the mix of a kernel that builds its operands with the vector ALU.
template <int NV>
__global__ __launch_bounds__(256) void calibration_mfma_kernel(int iters, float *sink)
{
    const uint32_t seed = 0x3F803F80u ^ (threadIdx.x & 1);          // bf16 values near one
    u32x4 a = {seed, seed, seed, seed}, b = {seed, seed, seed, seed};
    f32x16 c[4] = {f32x16{0}, f32x16{0}, f32x16{0}, f32x16{0}};
    float v[8];
    const float m = 1.0f + 1e-7f * static_cast<float>(threadIdx.x & 3);
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = 1.0f + static_cast<float>(r);
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[k] = mma(a, b, c[k]);
            // (as instructions: plain C multiplies by a loop-invariant factor would be folded into one per chain)
#pragma unroll
            for (int r = 0; r < NV; ++r) asm volatile("v_mul_f32 %0, %0, %1" : "+v"(v[r % 8]) : "v"(m));
        }
    }
    const f32x16 cs = (c[0] + c[1]) + (c[2] + c[3]);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) s += cs[e];
#pragma unroll
    for (int r = 0; r < 8; ++r) s += v[r];
    sink[static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x] = s;
}

}  // namespace mfma

// ================================================================================ host side
namespace {

using namespace mfma;

#define RACE_TRY(expr)                                   \
    do {                                                 \
        hipError_t e_ = (expr);                          \
        if (e_ != hipSuccess) return e_;                 \
    } while (0)

template <class C>
KArgs make_kargs(const Plan &p, char *ws)
{
    KArgs a;
    a.H = p.H; a.nseg = p.nseg; a.N = p.N; a.seg_len = p.seg_len; a.beta = p.beta;
    a.L_real = p.L; a.P_real = p.P;
    a.inv_tables = 1.0f / static_cast<float>(p.L);
    a.Wp = reinterpret_cast<const bf16raw *>(ws + p.off_W);
    a.state = reinterpret_cast<float *>(ws + p.off_stateA);
    a.Mq = reinterpret_cast<float *>(ws + p.off_massQ);
    a.Mk = reinterpret_cast<float *>(ws + p.off_massK);
    a.dbeta_part = reinterpret_cast<float *>(ws + p.off_dbeta);
    a.ge = reinterpret_cast<float *>(ws + p.off_ge);
    a.want_dbeta = 0;
    a.hash_tokens = 0;
    a.scanned = 0;
    return a;
}

// Whether anything reads the key and value totals of the forward pass: the only segment of a causal sequence starts from zeros.  (A step of
// two heads of 302 tokens, (128, 4, 4), without them and the two scans: 94.7 -> 89.9 us.)
bool wants_totals(const Plan &p) { return !p.causal || p.nseg > 1; }

// Whether the passes that read rows hash them as well.  That is work next to the latencies of a tile: 1.1 us a tile over both passes.  A
// kernel of its own spreads any problem over the chip; it takes its launch, launch_us, and the memory's time, (4 d + 8 L P) bytes a token
// and head: 1.1 us for a tile each of as many workgroups as 145 000 over those bytes, 142 to 227.  Kernel minus passes, forward calls in a
// graph, us, (128, 8, 6), causal, at 16, 64, 128, 192, 256 workgroups: 2 tiles +0.6 +0.8 +4.1 +4.1 +6.2; 4 tiles -0.9 +0.2 +4.7 +4.0 +4.7; 8
// tiles -3.3 +0.8 +4.3 +4.5 +7.2; 32 tiles -16 -10 -3 +10 +17; (64, 16, 4) of 32 tiles -22 -18 -12 -4 -1, (128, 4, 4) -20 -15 -9 -4 +3.
// (128, 8, 4) fits a CU twice where it does not hash and once where it does: its passes' time goes by rounds of 256 workgroups.  (Not
// causal, 32 tiles, 288 and 512 workgroups: 154 and 214 us with the kernel, 186 and 208 in the passes.)
bool hashing_pays(const Plan &p, double launch_us)
{
    const int64_t tiles = (std::min(p.seg_len, p.N) + kTile - 1) / kTile, groups = static_cast<int64_t>(p.BH) * p.nseg;
    const int64_t rounds = p.LRc == 128 ? (groups + 255) / 256 : 1;
    const double tile_us = 1.1 * static_cast<double>(tiles), row_bytes = 4.0 * p.d + 8.0 * p.Lc * p.Pc;
    return tile_us * static_cast<double>(rounds) <= launch_us + tile_us * static_cast<double>(groups) * row_bytes / 145e3;
}

// The forward pass (its totals K's rows, its replay Q's), and the totals of the taps and of a decoding state.
bool hash_in_passes(const Plan &p) { return hashing_pays(p, 3.5); }

// Hashed rows of X, and of X1 if there is one.
template <class C>
hipError_t launch_hash(const Plan &p, KArgs a, const void *X, float *M, const void *X1, float *M1, hipStream_t st)
{
    constexpr int kShares = hash_shares<C>();
    const int64_t rows = static_cast<int64_t>(p.BH) * (X1 ? 2 : 1);
    // too few tiles for the chip: a wavefront per share of a tile, else one per tile, with fewer tokens per workgroup, down to a tile per
    // wavefront, until there are four workgroups per CU
    const bool split = rows * ((p.N + kTile - 1) / kTile) <= 1024;
    auto kern = p.unit_qk ? hash_kernel<C, true, kShares> : hash_kernel<C, false, kShares>;
    if (split) kern = p.unit_qk ? hash_kernel<C, true, 1> : hash_kernel<C, false, 1>;
    a.hash_tokens = split ? kTile * kHashThreads / 64 / kShares : kHashTokens;
    while (!split && a.hash_tokens > kTile * kHashThreads / 64 && rows * ((p.N + a.hash_tokens - 1) / a.hash_tokens) < 1024) a.hash_tokens /= 2;
    ProfileScope prof("hash_rows", st);
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((p.N + a.hash_tokens - 1) / a.hash_tokens), p.BH, X1 ? 2 : 1), dim3(kHashThreads), 0, st, a,
                       static_cast<const bf16raw *>(X), M, static_cast<const bf16raw *>(X1), M1);
    return hipGetLastError();
}

// X: rows of K to be hashed into M (or null: M are the hashed rows; and M null: nobody reads them)
template <class C, int QG>
hipError_t launch_totals(const Plan &p, KArgs a, float *M, const void *X, const void *Y, const void *O, const float *den_in, void *Gout,
                         hipStream_t st)
{
    auto kern = totals_kernel<C, QG, false, false>;
    if (!QG && X) kern = p.unit_qk ? totals_kernel<C, QG, QG == 0, QG == 0> : totals_kernel<C, QG, QG == 0, false>;
    const int lds = X ? TotalsLds<C>::total_hash : TotalsLds<C>::total;
    RACE_TRY(allow_lds(kern, lds));
    ProfileScope prof(QG ? "stream_totals_qg" : "stream_totals_kv", st);
    hipLaunchKernelGGL(kern, dim3(p.nseg, p.BH), dim3(kThreads), lds, st, a, M, static_cast<const bf16raw *>(X),
                       static_cast<const bf16raw *>(Y), static_cast<const bf16raw *>(O), den_in, static_cast<bf16raw *>(Gout));
    return hipGetLastError();
}

// X: rows of Q to be hashed into Mr (or null: Mr are the hashed rows)
template <class C, int MODE, bool NC>
hipError_t launch_stream_nc(const Plan &p, KArgs a, float *Mr, const float *Mw, const void *X, const void *Y, void *Out, float *den_out,
                            hipStream_t st)
{
    static const char *const names[] = {"stream_forward", "stream_grad_v"};
    constexpr bool kFwd = MODE == kForward;
    auto kern = stream_kernel<C, MODE, NC, false, false>;
    if (kFwd && X) kern = p.unit_qk ? stream_kernel<C, MODE, NC, kFwd, kFwd> : stream_kernel<C, MODE, NC, kFwd, false>;
    const int lds = X ? StreamLds<C, NC>::total_hash : StreamLds<C, NC>::total;
    RACE_TRY(allow_lds(kern, lds));
    ProfileScope prof(names[MODE], st);
    hipLaunchKernelGGL(kern, dim3(p.nseg, p.BH), dim3(kThreads), lds, st, a, Mr, Mw, static_cast<const bf16raw *>(X),
                       static_cast<const bf16raw *>(Y), static_cast<bf16raw *>(Out), den_out);
    return hipGetLastError();
}
template <class C, int MODE>
hipError_t launch_stream(const Plan &p, KArgs a, float *Mr, const float *Mw, const void *X, const void *Y, void *Out, float *den_out,
                         hipStream_t st)
{
    return p.causal ? launch_stream_nc<C, MODE, false>(p, a, Mr, Mw, X, Y, Out, den_out, st)
                    : launch_stream_nc<C, MODE, true>(p, a, Mr, Mw, X, Y, Out, den_out, st);
}

template <class C>
hipError_t fwd_t(const Plan &p, const void *Q, const void *K, const void *V, void *O, float *den, char *ws, hipStream_t st)
{
    KArgs a = make_kargs<C>(p, ws);
    a.scanned = p.causal;
    // (no totals, no pass over K to hash it in: a step of B H = 512, N = 500, (128, 8, 6), takes 653 us with one that also sums, 630
    // with one that only hashes, 612 with the kernel)
    const bool in_passes = wants_totals(p) && hash_in_passes(p);
    if (!in_passes) RACE_TRY((launch_hash<C>(p, a, Q, a.Mq, K, a.Mk, st)));
    if (wants_totals(p)) RACE_TRY((launch_totals<C, 0>(p, a, a.Mk, in_passes ? K : nullptr, V, nullptr, nullptr, nullptr, st)));
    RACE_TRY(scan_states("segment_scan", a.state, p.nseg, p.BH, C::STATE, p.causal ? kScanPrefixOpen : kScanTotal, st));
    RACE_TRY((launch_stream<C, kForward>(p, a, a.Mq, a.Mk, in_passes ? Q : nullptr, V, O, den, st)));
    return hipSuccess;
}

// dphi and the chain rule through the soft assignment and W (grad_kernel).
template <class C, int SIDE>
hipError_t launch_grad(const Plan &p, KArgs a, const void *X, const void *V, const void *G, void *dX, hipStream_t st)
{
    auto kern = p.causal ? (p.unit_qk ? grad_kernel<C, SIDE, true, true> : grad_kernel<C, SIDE, false, true>)
                         : (p.unit_qk ? grad_kernel<C, SIDE, true, false> : grad_kernel<C, SIDE, false, false>);
    int lds = p.causal ? (p.unit_qk ? GradLds<C, true, true>::total : GradLds<C, false, true>::total)
                       : (p.unit_qk ? GradLds<C, true, false>::total : GradLds<C, false, false>::total);
    if (a.want_dbeta) lds += GradLds<C, false, false>::th_bytes;
    RACE_TRY(allow_lds(kern, lds));
    ProfileScope prof(SIDE == 0 ? "grad_q" : "grad_k", st);
    hipLaunchKernelGGL(kern, dim3(p.nseg, p.BH), dim3(kThreads), lds, st, a, static_cast<const bf16raw *>(X),
                       static_cast<const bf16raw *>(V), static_cast<const bf16raw *>(G), static_cast<bf16raw *>(dX));
    return hipGetLastError();
}

template <class C>
hipError_t bwd_t(const Plan &p, const void *Q, const void *K, const void *V, const void *O, const float *den,
                 const void *dO, void *dQ, void *dK, void *dV, float *dbeta, char *ws, hipStream_t st)
{
    KArgs a = make_kargs<C>(p, ws);
    a.scanned = p.causal;
    KArgs b = a;
    b.state = reinterpret_cast<float *>(ws + p.off_stateB);
    // the hashed rows of Q and K and the statistics of (phi_K, [V | 1]) at segment starts (the forward leaves exactly
    // these behind: its scan is in place and its streaming pass only reads them); then the statistics of
    // (phi_Q, read-out cotangents) at segment ends
    if (!p.fwd_state_kept) {
        // (no pass over Q comes that could hash it, and the kernel for it is launched in any case: K's rows leave it where the memory's
        // time alone is more than a pass's work)
        const bool in_passes = wants_totals(p) && hashing_pays(p, 0.0);
        RACE_TRY((launch_hash<C>(p, a, Q, a.Mq, in_passes ? nullptr : K, a.Mk, st)));
        if (wants_totals(p)) RACE_TRY((launch_totals<C, 0>(p, a, a.Mk, in_passes ? K : nullptr, V, nullptr, nullptr, nullptr, st)));
        RACE_TRY(scan_states("segment_scan", a.state, p.nseg, p.BH, C::STATE, p.causal ? kScanPrefixOpen : kScanTotal, st));
    }
    a.want_dbeta = b.want_dbeta = dbeta != nullptr;
    // dK's buffer holds the cotangent rows until dK itself is written
    RACE_TRY((launch_totals<C, 1>(p, b, a.Mq, nullptr, dO, O, den, dK, st)));
    RACE_TRY(scan_states("segment_scan", b.state, p.nseg, p.BH, C::STATE, p.causal ? kScanSuffixOpen : kScanTotal, st));
    RACE_TRY((launch_stream<C, kGradV>(p, b, a.Mk, a.Mq, nullptr, dK, dV, nullptr, st)));
    RACE_TRY((launch_grad<C, 0>(p, a, Q, V, dK, dQ, st)));
    RACE_TRY((launch_grad<C, 1>(p, b, K, V, dK, dK, st)));
    if (dbeta) RACE_TRY(reduce_dbeta(p, a.dbeta_part, dbeta, st));
    return hipSuccess;
}

template <class C>
hipError_t buckets_t(const Plan &p, const void *K, const void *V, float *A, float *Bsum, int a_stride, int b_stride,
                     char *ws, hipStream_t st)
{
    KArgs a = make_kargs<C>(p, ws);
    const bool in_passes = hash_in_passes(p);
    if (!in_passes) RACE_TRY((launch_hash<C>(p, a, K, a.Mk, nullptr, nullptr, st)));
    RACE_TRY((launch_totals<C, 0>(p, a, in_passes ? nullptr : a.Mk, in_passes ? K : nullptr, V, nullptr, nullptr, nullptr, st)));
    const int per = p.LR * (C::D + 1), groups = tap_groups(p.nseg), elements = kTapThreads / groups;
    hipLaunchKernelGGL(bucket_tap_kernel<C>, dim3((per + elements - 1) / elements, p.BH), dim3(kTapThreads), 0, st, a.state,
                       p.nseg, groups, p.L, p.P, A, Bsum, a_stride, b_stride);
    return hipGetLastError();
}

template <class C>
hipError_t hash_t(const Plan &p, const void *X, uint8_t *codes, float *phi, char *ws, hipStream_t st)
{
    KArgs a = make_kargs<C>(p, ws);
    const size_t lds = static_cast<size_t>(kTile) * C::PS * 2;
    auto kern = p.unit_qk ? hash_tap_kernel<C, true> : hash_tap_kernel<C, false>;
    RACE_TRY(allow_lds(kern, lds));
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((p.N + kTile - 1) / kTile), p.BH), dim3(kThreads), lds, st, a,
                       static_cast<const bf16raw *>(X), codes, phi);
    return hipGetLastError();
}

uint16_t host_bf16(float x)
{
    uint32_t b;
    std::memcpy(&b, &x, 4);
    b += 0x7fffu + ((b >> 16) & 1u);
    return static_cast<uint16_t>(b >> 16);
}

// W (H, L*P, D) -> Wp (H, LPP, D): row l * PP + t is hyperplane t of table l; rows of padding (and of tables and hyperplanes
// the problem does not have) are zero.
template <class C>
void pack_t(const Plan &p, const float *W, void *image)
{
    uint16_t *wp = static_cast<uint16_t *>(image);
    for (int hd = 0; hd < p.H; ++hd) {
        for (int row = 0; row < C::LPP; ++row) {
            const int table = row / C::PP, t = row % C::PP;
            for (int c = 0; c < C::D; ++c) {
                float v = 0.f;
                if (table < p.L && t < p.P) v = W[(static_cast<size_t>(hd) * p.LP + table * p.P + t) * C::D + c];
                wp[(static_cast<size_t>(hd) * C::LPP + row) * C::D + c] = host_bf16(v);
            }
        }
    }
}

// Dispatch over the compiled shapes.
#define RACE_SHAPES(X) RACE_MFMA_SHAPES(X)

}  // namespace

hipError_t calibration_mfma(int workgroups, int iters, int vector_ops, float *sink, hipStream_t st)
{
    switch (vector_ops) {
    case 0: hipLaunchKernelGGL(mfma::calibration_mfma_kernel<0>, dim3(workgroups), dim3(256), 0, st, iters, sink); break;
    case 4: hipLaunchKernelGGL(mfma::calibration_mfma_kernel<4>, dim3(workgroups), dim3(256), 0, st, iters, sink); break;
    case 8: hipLaunchKernelGGL(mfma::calibration_mfma_kernel<8>, dim3(workgroups), dim3(256), 0, st, iters, sink); break;
    case 16: hipLaunchKernelGGL(mfma::calibration_mfma_kernel<16>, dim3(workgroups), dim3(256), 0, st, iters, sink); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

bool mfma_pick(int d, int L, int P, int *Lc, int *Pc, int *pad)
{
    int best = 0;
#define X(DD, PP_, LL, PD)                                                                              \
    if (PD == 0 && d == DD && P == PP_ && L == LL) {                                                    \
        *Lc = LL; *Pc = PP_; *pad = 0;                                                                  \
        return true;                                                                                    \
    }
    RACE_SHAPES(X)
#undef X
#define X(DD, PP_, LL, PD)                                                                              \
    if (PD == 1 && d == DD && P <= PP_ && L <= LL && (best == 0 || LL * (1 << PP_) < best)) {           \
        best = LL * (1 << PP_);                                                                         \
        *Lc = LL; *Pc = PP_; *pad = 1;                                                                  \
    }
    RACE_SHAPES(X)
#undef X
    return best != 0;
}

size_t mfma_hashed_bytes(const Plan &p)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) \
        return static_cast<size_t>(p.BH) * static_cast<size_t>((p.N + kTile - 1) / kTile * kTile) * Cfg<DD, PP_, LL, PD != 0>::LP * sizeof(float);
    RACE_SHAPES(X)
#undef X
    return 0;
}

int mfma_workgroups_per_cu(const Plan &p)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return Cfg<DD, PP_, LL, PD != 0>::STREAM_WAVES_PER_SIMD / 2;
    RACE_SHAPES(X)
#undef X
    return 1;
}

size_t mfma_projection_bytes(const Plan &p)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return static_cast<size_t>(p.H) * Cfg<DD, PP_, LL, PD != 0>::LPP * DD * 2;
    RACE_SHAPES(X)
#undef X
    return 0;
}

void mfma_pack_projection(const Plan &p, const float *W, void *image)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return pack_t<Cfg<DD, PP_, LL, PD != 0>>(p, W, image);
    RACE_SHAPES(X)
#undef X
}

hipError_t mfma_fwd(const Plan &p, const void *Q, const void *K, const void *V, void *O, float *den, char *ws, hipStream_t st)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return fwd_t<Cfg<DD, PP_, LL, PD != 0>>(p, Q, K, V, O, den, ws, st);
    RACE_SHAPES(X)
#undef X
    return hipErrorNotSupported;
}

int mfma_dbeta_parts(const Plan &p)
{
    return p.nseg;
}

hipError_t mfma_bwd(const Plan &p, const void *Q, const void *K, const void *V, const void *O, const float *den,
                    const void *dO, void *dQ, void *dK, void *dV, float *dbeta, char *ws, hipStream_t st)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return bwd_t<Cfg<DD, PP_, LL, PD != 0>>(p, Q, K, V, O, den, dO, dQ, dK, dV, dbeta, ws, st);
    RACE_SHAPES(X)
#undef X
    return hipErrorNotSupported;
}

hipError_t mfma_hash(const Plan &p, const void *X_, uint8_t *codes, float *phi, char *ws, hipStream_t st)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return hash_t<Cfg<DD, PP_, LL, PD != 0>>(p, X_, codes, phi, ws, st);
    RACE_SHAPES(X)
#undef X
    return hipErrorNotSupported;
}

hipError_t mfma_buckets(const Plan &p, const void *K, const void *V, float *A, float *Bsum, int a_stride, int b_stride,
                        char *ws, hipStream_t st)
{
#define X(DD, PP_, LL, PD) if (p.d == DD && p.Pc == PP_ && p.Lc == LL && p.pad == PD) return buckets_t<Cfg<DD, PP_, LL, PD != 0>>(p, K, V, A, Bsum, a_stride, b_stride, ws, st);
    RACE_SHAPES(X)
#undef X
    return hipErrorNotSupported;
}

}  // namespace race
