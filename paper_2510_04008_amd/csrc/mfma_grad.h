// grad_kernel: the two backward passes that contract the bucket statistics over the head dimension.
// Register budget: with eight wavefronts of 256 registers a wavefront can carry up to 64 bucket rows x 128
// columns of fp32 statistics (128 registers) next to its working set, i.e. 512 bucket rows per workgroup.
// The workgroup then also forms dX = dz . W for its tile.  (Shapes with more bucket rows than that are not compiled.)
//
//   SIDE 0 (dQ), left to right, statistics S = (B | A) of (phi_K, [V | 1]) before/with token i:
//       dphi_Q(i)[r] = S[r,:] . [dO_i/e_i | -(dO_i.O_i)/e_i]
//   SIDE 1 (dK), right to left, statistics dS = (dB | dA) of (phi_Q, read-out cotangents) of tokens >= j:
//       dphi_K(j)[r] = dS[r,:] . [V_j | 1]
// followed in both cases by the chain rule through the corner softmax, tanh and W:  dx = W^T dz.
// "reader" is the tensor whose gradient is produced, "writer" the tensor that feeds the statistics.  The assignments of
// both are rebuilt from their hashed rows; the chain rule through tanh needs tanh z and its derivative as
// well, for which the reader's rows are projected here, a 16 x 16 tile per wavefront.
//
// The statistics are held transposed, tiles S^T[head column][bucket row], so that a tile's accumulator
// registers are the B operand of the contraction over columns (lane = bucket row).  The in-tile part
// uses T^T[b][a] = Yw_b . Yr_a (+ the product of the two extra columns), masked to b <= a (b >= a
// right to left), which goes to LDS as the A operand of  T . phi_writer.
//
// Two barriers per tile.  First half: what the tile needs before its dphi (the derivative of tanh, the writer's assignments, the
// in-tile term) and dX of the tile before it; second half: dphi, the corner softmax backwards, dz, and the rows of the following
// tile -> LDS (two buffers).  R = 64: a wavefront builds the assignments of its own table, which nothing else reads, so the update of
// the statistics belongs to the first half of the following tile, whose vector work runs next to its products.  Loads and stores
// are unconditional, a tile that does not exist repeating the last one's: behind a branch the compiler no longer knows how
// many are in flight and waits for the newest, which at the production cost every tile a trip to memory.
// (Both gradients of 4.2 million rows of 128 columns, L = 8, P = 6: 4.42 ms with the production on four wavefronts, the update in the
// second half and W read through transposing loads; now 4.10.  The clock gives part of it back: 7880 -> 7060 cycles a tile, 1.87 ->
// 1.81 GHz on the same box.)
#pragma once
#include "mfma_common.h"

namespace race {
namespace mfma {

// Two forms of the second half.  R = 64 (P = 6): a wavefront owns the 64 bucket rows of one table as 32 x 32 tiles.  R = 16
// (P = 4): 16 x 16 tiles, one table per tile of bucket rows: eight tables or more are shared out over the wavefronts, four
// go to two wavefronts each, which take half of the tile's tokens each (and both keep the table's statistics).  Both
// gradients of 4.2 million rows of 128 columns at L = P = 4 take 2.16 ms; with 32 x 32 tiles, which kept two of the eight
// wavefronts busy in the second half, 3.05 ms.
template <class C>
struct GradCfg {
    static constexpr bool T16 = C::R == 16;
    static_assert(T16 || C::R == 64, "one or four 16-row tiles per table");
    // R = 64
    static constexpr int MTG = 2;                                       // 32-row tiles of bucket rows per wavefront (128 registers of
                                                                        // statistics per lane is what fits next to the working set)
    static constexpr int RW = T16 ? 16 : 32 * MTG;                      // bucket rows of a table
    static_assert(T16 || C::L == kWaves, "one table per wavefront");
    // R = 16
    static constexpr int TPW = C::L >= kWaves ? C::L / kWaves : 1;      // tables per wavefront
    static constexpr int TS = C::L >= kWaves ? 1 : kWaves / C::L;       // wavefronts that share a table's tokens
    static_assert(TS <= 2 && (T16 || TPW == 1), "tables over wavefronts");
    static constexpr int SREGS = T16 ? TPW * C::D / 4 : MTG * C::NT * 16;        // registers of statistics
    // W transposed next to W: dX's operands are reads by rows.  (Transposing reads of W, under its stride for reads by rows, take
    // four times as long.  R = 16: two workgroups on a CU need the room.)
    static constexpr bool WT = !T16;
    static constexpr int YORDER = T16 ? kPairs32 : kPlain;
    // First half of a tile, by role.  Production (R = 16): `SLOTS` half wavefronts from wavefront 0 on; projection of the reader's rows:
    // 2 PT 16 x 16 tiles; in-tile term: three 16 x 16 tiles; dX of the previous tile: 2 NT pieces.
    static constexpr int SLOTS = C::L >= 16 ? 16 : 8;
    static constexpr int proj_wave(int i, bool causal)
    {
        if (!causal || C::PT == 4) return i % kWaves;
        return i == 0 ? 0 : 3 + i;
    }
    static constexpr int tt_wave(int i) { return T16 ? (C::L >= 16 ? 5 + i : 1 + i) : i; }
    static constexpr int dx_wave(int i, bool causal) { return T16 && causal && C::L >= 16 ? i : kWaves - 1 - i; }
    static_assert(2 * C::NT <= kWaves, "one piece of dX per wavefront at most");
};

// UNIT: the unit-norm option's extras (row scales, projections, parts of z . dz, a second buffer of the reader's rows, which
// dX of a tile still reads when the next tile's rows are stored).
// INTRA: the causal variant, whose tiles also feed the statistics: the writer's rows, assignments and the in-tile term.
template <class C, bool UNIT, bool INTRA>
struct GradLds {
    using G = GradCfg<C>;
    static constexpr int XB = UNIT ? 2 : 1;                             // buffers of the reader's rows and of the scales
    static constexpr int wp = 0;                                        // [LPP][XS] bf16
    static constexpr int DZS = C::LPP + 8;                              // bf16 row stride of the dz tile
    static constexpr int WTS = C::LPP + 8;                              // bf16 row stride of W transposed
    static constexpr int wt = wp + C::LPP * C::XS * 2;                  // [D][WTS] bf16: W transposed, column c at wt_row(c)
    static constexpr int dz = wt + (G::WT ? C::D * WTS * 2 : 0);        // [32][DZS] bf16
    static constexpr int sr = dz + kTile * DZS * 2;                     // [2][32] fp32 extra column of reader-Y
    static constexpr int sw = sr + 2 * kTile * 4;                       // [2][32] fp32 extra column of writer-Y
    static constexpr int swp = sw + 2 * kTile * 4;                      // [2][kParts][32] bf16: parts of sw (key side)
    static constexpr int nrm = swp + 2 * kParts * kTile * 2;                      // [XB][32] fp32: 1 / |x| of the reader's rows
    static constexpr int rad = nrm + (UNIT ? XB * kTile * 4 : 0);       // [kWaves][32] fp32: per-wavefront parts of z . dz per token
    static constexpr int QUADS = C::L * C::PP / 4;
    static constexpr int s2 = (rad + (UNIT ? kWaves * kTile * 4 : 0) + 15) & ~15;     // [QUADS][32] float4: 1 - tanh^2 z of four hyperplanes
    static constexpr int zz = s2 + QUADS * kTile * 16;                  // [QUADS][32] float4: z
    static constexpr int yr = zz + (UNIT ? QUADS * kTile * 16 : 0);     // [2][32][XS] reader-Y rows, columns in YORDER
    static constexpr int yr_bytes = kTile * C::XS * 2;
    static constexpr int xr = yr + 2 * yr_bytes;                        // [XB][32][XS] reader rows
    static constexpr int xr_bytes = kTile * C::XS * 2;
    static constexpr int ttop = xr + XB * xr_bytes;                     // [2][64] x 16 B: masked in-tile term as MFMA operands
    static constexpr int yw = ttop + (INTRA ? 2 * 64 * 16 : 0);         // [2][32][YS] writer-Y rows, columns in YORDER
    static constexpr int yw_bytes = kTile * C::YS * 2;
    static constexpr int phw = yw + (INTRA ? 2 * yw_bytes : 0);         // [32][PS or PST] writer assignments
    static constexpr int mass = phw + (INTRA ? kTile * (G::T16 ? C::PST : C::PS) * 2 : 0); // R = 16: [kWaves][TPW * 16] fp32: extra column of each wavefront's rows
    static constexpr int total = mass + (G::T16 ? kWaves * G::TPW * 16 * 4 : 0);
    // where the cotangent of beta is wanted:
    static constexpr int th = total;                                    // [QUADS][32] float4: tanh z
    static constexpr int th_bytes = QUADS * kTile * 16;
    static_assert(yr % 16 == 0 && th % 16 == 0 && total + th_bytes <= 160 * 1024, "LDS budget");
};

// Wavefronts per SIMD the gradient kernel is compiled for: four (128 registers, two workgroups per CU, whose phases
// interleave) where the statistics do not change, 32 registers hold a wavefront's share of them and the tiles fit 80 KB.
// The causal variants are compiled for two.  Those of (128, 4, 4) fit a CU twice all the same, at 123 to 128 registers (at 129, dK with the
// unit-norm option, B H = 64, N = 4096: 92 us instead of 74); (128, 4, 8) takes 136 to 143 and (64, 4, 16) 140 to 149.  (Kernels that
// wanted 139 spilled when they were held to 128 and took 1.6 times as long.)
template <class C, bool UNIT, bool INTRA>
constexpr int grad_waves_per_simd()
{
    return (!INTRA && GradCfg<C>::SREGS <= 32 && GradLds<C, UNIT, INTRA>::total <= 80 * 1024) ? 4 : 2;
}

// Row of W transposed that holds column c: in every 32 columns the first 16 rows are the first halves of the eights, the others
// the second ones (the order in which dX's tiles take them).
__device__ __forceinline__ constexpr int wt_row(int c) { return (c & ~31) | ((c & 4) << 2) | ((c >> 1) & 12) | (c & 3); }

template <class C, int SIDE, bool UNIT, bool INTRA>
__global__ __launch_bounds__(kThreads, (grad_waves_per_simd<C, UNIT, INTRA>()))
void grad_kernel(KArgs a, const bf16raw *Xr, const bf16raw *V, const bf16raw *G_, bf16raw *dX)
{
    using S = GradLds<C, UNIT, INTRA>;
    using G = GradCfg<C>;
    extern __shared__ __attribute__((aligned(256))) unsigned char lds[];
    bf16raw *wp = reinterpret_cast<bf16raw *>(lds + S::wp);
    bf16raw *wt = reinterpret_cast<bf16raw *>(lds + S::wt);
    bf16raw *dz = reinterpret_cast<bf16raw *>(lds + S::dz);
    float *rad = reinterpret_cast<float *>(lds + S::rad);
    f32x4 *s2t = reinterpret_cast<f32x4 *>(lds + S::s2);
    f32x4 *tht = reinterpret_cast<f32x4 *>(lds + S::th);
    f32x4 *zzt = reinterpret_cast<f32x4 *>(lds + S::zz);
    bf16raw *phw = reinterpret_cast<bf16raw *>(lds + S::phw);
    u32x4 *ttop = reinterpret_cast<u32x4 *>(lds + S::ttop);
    auto buf_yr = [&](int it) { return reinterpret_cast<bf16raw *>(lds + S::yr + (it & 1) * S::yr_bytes); };
    auto buf_yw = [&](int it) { return reinterpret_cast<bf16raw *>(lds + S::yw + (it & 1) * S::yw_bytes); };
    auto buf_sr = [&](int it) { return reinterpret_cast<float *>(lds + S::sr) + (it & 1) * kTile; };
    auto buf_sw = [&](int it) { return reinterpret_cast<float *>(lds + S::sw) + (it & 1) * kTile; };
    auto buf_swp = [&](int it) { return reinterpret_cast<bf16raw *>(lds + S::swp) + (it & 1) * kParts * kTile; };
    auto buf_xr = [&](int it) { return reinterpret_cast<bf16raw *>(lds + S::xr + (UNIT ? it & 1 : 0) * S::xr_bytes); };
    auto buf_nrm = [&](int it) { return reinterpret_cast<float *>(lds + S::nrm) + (UNIT ? it & 1 : 0) * kTile; };

    constexpr bool kReverse = (SIDE == 1);
    const int seg = blockIdx.x, bh = blockIdx.y, head = bh % a.H;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, h = lane >> 5;
    const int n16 = lane & 15, q16 = lane >> 4;
    // this wavefront's first table (R = 16, fewer tables than wavefronts: wavefronts w and w + 4 share one)
    const int tl0 = G::TS == 2 ? (w & 3) : w * G::TPW;
    const int r_own = tl0 * C::R;                    // ... and its bucket rows
    constexpr bool intra = INTRA;

    const size_t base = static_cast<size_t>(bh) * a.N * C::D;
    Xr += base; V += base; dX += base;
    const bf16raw *Gr = G_ + base;                   // cotangent rows and their extra column (may be dX's own memory: read two tiles ahead)
    const float *ge = a.ge + static_cast<size_t>(bh) * a.N;
    const size_t mbase = static_cast<size_t>(bh) * ((a.N + kTile - 1) / kTile) * (kTile * C::LP);
    const float *Mw = (SIDE == 0 ? a.Mk : a.Mq) + mbase, *Mr = (SIDE == 0 ? a.Mq : a.Mk) + mbase;
    const float *st = a.state + (static_cast<size_t>(bh) * a.nseg + (INTRA ? seg : 0)) * C::STATE;     // (not causal: the totals)

    {
        const bf16raw *src = a.Wp + static_cast<size_t>(head) * C::LPP * C::D;
        for (int c = tid; c < C::LPP * C::CPR; c += kThreads) {
            const int row = c / C::CPR, ch = c % C::CPR;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(src + row * C::D + ch * 8);
            *reinterpret_cast<u32x4 *>(wp + row * C::XS + ch * 8) = v;
            const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < (G::WT ? 8 : 0); ++e) wt[wt_row(8 * ch + e) * S::WTS + row] = static_cast<bf16raw>(vw[e / 2] >> (16 * (e & 1)));
        }
    }
    if (C::L * C::PP < C::LPP) {
        // projection slots that belong to no table are never written below: they must be zeros for dX = dz . W
        for (int i = tid; i < kTile * S::DZS; i += kThreads) dz[i] = 0;
    }
    // the off-diagonal 16 x 16 tile of the in-tile term that the mask clears is never written below
    if (intra && tid < 128) ttop[tid] = u32x4{0u, 0u, 0u, 0u};
    // statistics at the start of the segment, transposed tiles: columns x bucket rows
    f32x16 ST[G::MTG][C::NT];                        // R = 64: 32 x 32 tiles [row tile][column tile]
    f32x4 SU[G::TPW][C::D / 16];                     // R = 16: 16 x 16 tiles [table][column tile]
    float macc[G::T16 ? G::TPW : G::MTG];            // extra column (A or dA): lane n < 32 <-> row r_own + 32 mr + n (n < 16 <-> r_own + 16 i + n)
    float *mass = reinterpret_cast<float *>(lds + S::mass) + w * G::TPW * 16;
    // (causal: nothing precedes the first segment, right to left the last one, and the scan writes no state for it)
    const bool from_zero = INTRA && seg == (kReverse ? a.nseg - 1 : 0);
    if (from_zero) {
#pragma unroll
        for (int i = 0; i < (G::T16 ? G::TPW : G::MTG); ++i) macc[i] = 0.f;
        if constexpr (G::T16) {
#pragma unroll
            for (int i = 0; i < G::TPW; ++i) {
#pragma unroll
                for (int ct = 0; ct < C::D / 16; ++ct) SU[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (q16 == 0) mass[16 * i + n16] = 0.f;
            }
        } else {
#pragma unroll
            for (int mr = 0; mr < G::MTG; ++mr) {
#pragma unroll
                for (int mtc = 0; mtc < C::NT; ++mtc) ST[mr][mtc] = f32x16{0};
            }
        }
    } else if constexpr (G::T16) {
#pragma unroll
        for (int i = 0; i < G::TPW; ++i) {
#pragma unroll
            for (int ct = 0; ct < C::D / 16; ++ct)
                SU[i][ct] = *reinterpret_cast<const f32x4 *>(st + (r_own + 16 * i + n16) * C::D + 16 * ct + 4 * q16);
            macc[i] = q16 == 0 ? st[C::LR * C::D + r_own + 16 * i + n16] : 0.f;
            if (q16 == 0) mass[16 * i + n16] = macc[i];
        }
    } else {
#pragma unroll
        for (int mr = 0; mr < G::MTG; ++mr) {
#pragma unroll
            for (int mtc = 0; mtc < C::NT; ++mtc) {
#pragma unroll
                for (int v = 0; v < 16; ++v) ST[mr][mtc][v] = st[(r_own + 32 * mr + ln) * C::D + 32 * mtc + 16 * (v / 8) + 8 * h + v % 8];
            }
            macc[mr] = h == 0 ? st[C::LR * C::D + r_own + 32 * mr + ln] : 0.f;
        }
    }

    const int64_t t_begin = seg * a.seg_len;
    const int64_t t_end = (t_begin + a.seg_len < a.N) ? t_begin + a.seg_len : a.N;
    const int ntiles = static_cast<int>((t_end - t_begin + kTile - 1) / kTile);
    auto tile_t0 = [&](int it) { return t_begin + static_cast<int64_t>(kReverse ? ntiles - 1 - it : it) * kTile; };
    // the loads of a tile that does not exist repeat the last one's (and are not used): see store_buffer()
    const int64_t t_last = t_begin + static_cast<int64_t>(ntiles - 1) * kTile;
    auto existing_t0 = [&](int it) { const int64_t t = tile_t0(it); return kReverse ? (t > t_begin ? t : t_begin) : (t < t_last ? t : t_last); };
    auto tile_nv = [&](int64_t t0) { return (t_end - t0 < kTile) ? static_cast<int>(t_end - t0) : kTile; };

    // LDS addresses are a lane's offset under a stride plus a uniform one, added where it is used.  The lane's offsets are worked out
    // here, or, where they would push two workgroups' registers past a CU's (R = 16, causal) or spill (the unit-norm option beside 128
    // registers of statistics), again in every tile.  R = 16, not causal, has registers to spare and few instructions a tile: there
    // the uniform parts are the instructions' own offsets.  (dQ at 32 workgroups of up to 32 tiles, (128, 4, 4): 59.7 -> 55.8 us; a step
    // of B H = 64, N = 16384, (64, 4, 16): 1031 -> 1016 us.)
    constexpr bool kRebuild = (G::T16 && INTRA) || (UNIT && G::SREGS == 128);
    constexpr bool kFold = G::T16 && !INTRA;
    int step = 0;       // (the loop counter of these sums)
    auto at = [&](int uniform, int lane_offset) __attribute__((always_inline)) { return lds + ((kFold ? uniform : opaque_uniform(uniform, step)) + lane_offset); };
    const int at16x_ = (n16 * C::XS + 8 * q16) * 2, at16d_ = (n16 * S::DZS + 8 * q16) * 2;      // 16-row operands
    const int at_x_ = chunk_offset<C, C::XS, kPlain>(tid), at_yr_ = chunk_offset<C, C::XS, G::YORDER>(tid), at_yw_ = chunk_offset<C, C::YS, G::YORDER>(tid);
    auto rebuilt_lane = [&]() __attribute__((always_inline)) { return opaque(lane, step); };
    auto at16 = [&](int stride, int kept) __attribute__((always_inline)) {
        if (!kRebuild) return kept;
        const int lo = rebuilt_lane();
        return ((lo & 15) * stride + 8 * (lo >> 4)) * 2;
    };
    static_assert(S::DZS == S::WTS, "one offset for both operands of dX");
    auto operand = [&](const unsigned char *p, int bytes) __attribute__((always_inline)) { return *reinterpret_cast<const u32x4 *>(p + bytes); };
    // rows: requested two tiles ahead, written to LDS one tile ahead (the reader's in the second half of a tile, behind its
    // projection; the others there as well for R = 64, in the first half for R = 16)
    RowChunks<C, kTile> pre_r, pre_v, pre_g;
    float pre_ge = 0.f;
    auto fetch_y = [&](int it) __attribute__((always_inline)) {
        const int64_t t0 = existing_t0(it);
        const int nv = tile_nv(t0);
        if (SIDE == 1 || intra) fetch_rows<C, kTile>(V, t0, nv, pre_v);
        if (SIDE == 0 || intra) {
            fetch_rows<C, kTile>(Gr, t0, nv, pre_g);
            pre_ge = (ge + t0)[static_cast<uint32_t>(ln < nv ? ln : nv - 1)];
        }
    };
    auto fetch_x = [&](int it) __attribute__((always_inline)) {
        const int64_t t0 = existing_t0(it);
        fetch_rows<C, kTile>(Xr, t0, tile_nv(t0), pre_r);
    };
    auto stage_y = [&](int it) __attribute__((always_inline)) {
        store_tile<C, G::YORDER>(SIDE == 0 ? pre_g : pre_v, at(S::yr + (it & 1) * S::yr_bytes, kRebuild ? chunk_offset<C, C::XS, G::YORDER>(opaque(tid, step)) : at_yr_));
        if (intra) store_tile<C, G::YORDER>(SIDE == 0 ? pre_v : pre_g, at(S::yw + (it & 1) * S::yw_bytes, kRebuild ? chunk_offset<C, C::YS, G::YORDER>(opaque(tid, step)) : at_yw_));
        if (tid < kTile) {
            buf_sr(it)[tid] = SIDE == 0 ? pre_ge : 1.f;
            buf_sw(it)[tid] = SIDE == 0 ? 1.f : pre_ge;
        }
        if (SIDE == 1 && intra && tid < kParts * kTile) buf_swp(it)[tid] = weight_part(pre_ge, tid / kTile);
    };
    auto stage_x = [&](int it) __attribute__((always_inline)) {
        store_tile<C, kPlain>(pre_r, at(S::xr + (UNIT ? it & 1 : 0) * S::xr_bytes, kRebuild ? chunk_offset<C, C::XS, kPlain>(opaque(tid, step)) : at_x_));
        if (UNIT) store_row_scales<C, kTile>(pre_r, buf_nrm(it), step);
    };
    // the writer's assignments.  R = 64: every wavefront builds those of its own table, which nothing else reads; R = 16: the first
    // wavefronts build all of them
    using Sh = Share<C, G::SLOTS>;
    const int slot = 2 * (w & (G::SLOTS / 2 - 1)) + h;
    const bool produces = intra && (!G::T16 || w < G::SLOTS / 2);
    typename Sh::Regs pre_w;
    float own_w[C::P];
    const uint32_t woff = table_offset<C>(G::T16 ? Sh::table(slot, 0) : tl0, ln);
    auto fetch_w = [&](int it) __attribute__((always_inline)) {
        if (!produces) return;
        if constexpr (G::T16) Sh::load(Mw + existing_t0(it) * C::LP, woff, ln, pre_w);
        else load_table_codes<C>(Mw + existing_t0(it) * C::LP, woff, ln, own_w);
    };
    // the reader's hashed rows: R = 64: token ln of the wavefront's table; R = 16: tokens n16 (and 16 + n16) of its tables
    const int th0 = G::TS == 2 ? w >> 2 : 0;
    const uint32_t roff = table_offset<C>(tl0, G::T16 ? 16 * th0 + n16 : ln);
    // this wavefront's roles in the first half (compile-time tables, looked up once)
    int my_dx = -1, my_tt = -1, my_proj[2] = {-1, -1};
#pragma unroll
    for (int i = 0; i < 2 * C::NT; ++i) my_dx = w == G::dx_wave(i, INTRA) ? i : my_dx;
#pragma unroll
    for (int i = 0; i < 3; ++i) my_tt = w == G::tt_wave(i) ? i : my_tt;
#pragma unroll
    for (int i = 0; i < 2 * C::PT; ++i) {
        if (w == G::proj_wave(i, INTRA)) {
            if (my_proj[0] < 0) my_proj[0] = i;
            else my_proj[1] = i;
        }
    }
    if (ntiles > 0) {
        fetch_x(0);
        fetch_y(0);
        fetch_w(0);
        stage_x(0);
        stage_y(0);
        fetch_x(1);
        fetch_y(1);
        __syncthreads();
    }

    // ---- dX = dz . W for one tile (the chain rule through W), one step late, next to the production of the following tile.  Piece
    //      i is 16 tokens x 32 columns, as two transposed 16 x 16 tiles whose rows are columns 8 q + 0 .. 3 and 8 q + 4 .. 7: lane
    //      (n, q) holds eight consecutive columns of token n and stores them as one 16-byte piece, without a stop in LDS.
    //      (As 32 x 32 tiles on four wavefronts, staged in LDS on their way out, this chain of dependent steps took 1700 of the
    //      3750 cycles of the first half; here every wavefront has a quarter of that.)
    struct DxOperands { u32x4 d[C::LPP / 32], wa[C::LPP / 32], wb[C::LPP / 32]; };
    auto dx_load = [&](int i, DxOperands &o) __attribute__((always_inline)) {
        const unsigned char *d = at(S::dz + 16 * (i & 1) * S::DZS * 2, at16(S::DZS, at16d_));
        if constexpr (G::WT) {
            const unsigned char *wc = at(S::wt + 32 * (i >> 1) * S::WTS * 2, at16(S::DZS, at16d_));
#pragma unroll
            for (int s = 0; s < C::LPP / 32; ++s) {
                o.d[s] = operand(d, 64 * s);
                o.wa[s] = operand(wc, 64 * s);
                o.wb[s] = operand(wc, 16 * S::WTS * 2 + 64 * s);
            }
        } else {
            const int lo = rebuilt_lane(), chunk = 32 * (i >> 1) + 8 * (lo & 3);
#pragma unroll
            for (int s = 0; s < C::LPP / 32; ++s) {
                const int k = 32 * s + 8 * (lo >> 4);
                o.d[s] = operand(d, 64 * s);
                o.wa[s] = lds_tr16(wp, C::XS, k, k + 4, chunk, lo);
                o.wb[s] = lds_tr16(wp, C::XS, k, k + 4, chunk + 4, lo);
            }
        }
    };
    auto dx_mma = [&](const DxOperands &o, f32x4 &x0, f32x4 &x1) __attribute__((always_inline)) {
        x0 = x1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < C::LPP / 32; ++s) {
            x0 = mma16(o.wa[s], o.d[s], x0);
            x1 = mma16(o.wb[s], o.d[s], x1);
        }
    };
    auto dx_store = [&](int i, int it, f32x4 x0, f32x4 x1) __attribute__((always_inline)) {
        const int64_t t0 = tile_t0(it);
        const int c0 = 32 * (i >> 1);
        if (UNIT) {
            const int lo = opaque(lane, step), n = lo & 15, q = lo >> 4, tok = 16 * (i & 1) + n;
            float cp = 0.f;                              // (z . dz) / |x|^2 of the token, parts in wavefront order
#pragma unroll
            for (int w8 = 0; w8 < kWaves / G::TS; ++w8) cp += rad[((G::TS == 2 ? 4 * (tok >> 4) : 0) + w8) * kTile + tok];
            cp *= buf_nrm(it)[tok];
            const u32x4 xv = lds128(buf_xr(it) + tok * C::XS + c0 + 8 * q);
            x0[0] = fmaf(-cp, bf_lo(xv.x), x0[0]); x0[1] = fmaf(-cp, bf_hi(xv.x), x0[1]);
            x0[2] = fmaf(-cp, bf_lo(xv.y), x0[2]); x0[3] = fmaf(-cp, bf_hi(xv.y), x0[3]);
            x1[0] = fmaf(-cp, bf_lo(xv.z), x1[0]); x1[1] = fmaf(-cp, bf_hi(xv.z), x1[1]);
            x1[2] = fmaf(-cp, bf_lo(xv.w), x1[2]); x1[3] = fmaf(-cp, bf_hi(xv.w), x1[3]);
        }
        buffer_store128(store_buffer(dX + t0 * C::D, tile_nv(t0) * C::D * 2), opaque_uniform((16 * (i & 1) * C::D + c0) * 2, step) + at16(C::D, (n16 * C::D + 8 * q16) * 2),
                        u32x4{pack2(x0[0], x0[1]), pack2(x0[2], x0[3]), pack2(x1[0], x1[1]), pack2(x1[2], x1[3])});
    };
    // ---- projections of the reader's rows, 16 packed hyperplanes x 16 tokens (tile i of 2 PT), and what the chain rule through
    //      tanh needs of them: tanh z and 1 - tanh^2 z
    constexpr bool kAllProject = 2 * C::PT == kWaves;       // one tile per wavefront, no roles
    auto project = [&](int i, int it) __attribute__((always_inline)) {
        const unsigned char *wrow = at(S::wp + 16 * (i >> 1) * C::XS * 2, at16(C::XS, at16x_));
        const unsigned char *xrow = at(S::xr + (UNIT ? it & 1 : 0) * S::xr_bytes + 16 * (i & 1) * C::XS * 2, at16(C::XS, at16x_));
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < C::D / 32; ++s) z = mma16(operand(wrow, 64 * s), operand(xrow, 64 * s), z);
        return z;
    };
    auto finish_projection = [&](int i, int it, f32x4 z) __attribute__((always_inline)) {
        int n = n16, q = q16;
        if constexpr (INTRA && UNIT && SIDE == 1 && G::TS == 2) {       // (129 registers with this address kept: see grad_waves_per_simd())
            const int lo = rebuilt_lane();
            n = lo & 15;
            q = lo >> 4;
        }
        const int quad = 4 * (i >> 1) + q, slot16 = opaque_uniform((4 * (i >> 1) * kTile + 16 * (i & 1)) * 16, step) + (q * kTile + n) * 16;
        if (UNIT) z = z * buf_nrm(it)[16 * (i & 1) + n];
        f32x4 sv, uv;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float e2 = __expf(-2.0f * fabsf(z[v])), inv = __builtin_amdgcn_rcpf(1.0f + e2), ua = (1.0f - e2) * inv;
            sv[v] = 4.0f * e2 * inv * inv;
            uv[v] = z[v] >= 0.f ? ua : -ua;
        }
        if (C::L * C::PP % 16 == 0 || quad < S::QUADS) {
            *reinterpret_cast<f32x4 *>(lds + S::s2 + slot16) = sv;
            if (a.want_dbeta) *reinterpret_cast<f32x4 *>(lds + S::th + slot16) = uv;
            if (UNIT) *reinterpret_cast<f32x4 *>(lds + S::zz + slot16) = z;
        }
    };

    if (G::T16 && w >= 4) lead(true);       // (R = 16: all along; handing the lead back half way through the tables is slower)
    float dbeta_acc = 0.f;    // this lane's share of the cotangent of beta: sum of 2 p_t q_t E_t tanh z_t
    // ================ first half of tile `it`: all that it needs before its dphi, and dX of the tile before it
    // (the reader's hashed rows of this wavefront's tables: used in the second half)
    constexpr int kTh = G::T16 && G::TS == 1 ? 2 : 1;      // R = 16: halves of the tile's tokens
    float rc[G::TPW * kTh][C::P];
    // A tile's first half follows the second half of the tile before it in the loop's body.  (The causal kernels of (128, 8, 4) have it in
    // order: dQ and dK at B H = 64, N = 4096, 83.2 and 85.8 against 81.7 and 83.2 us.  (128, 4, 4) needs 130 registers that way and has the
    // CU for itself; (64, 16, 4) with the unit-norm option takes 2 to 3 % more, (128, 16, 4) 2 %.)
    constexpr bool kRotate = !G::T16 || !INTRA || G::TS == 2 || G::TPW > 1;
    auto first_half = [&](int it, bool first) __attribute__((always_inline)) {
        const int64_t t0 = existing_t0(it);
        const int nvalid = tile_nv(t0);
#pragma unroll
        for (int i = 0; i < G::TPW * kTh; ++i)
            load_table_codes<C>(Mr + t0 * C::LP + (i / kTh) * C::HT + (i % kTh) * 64, roff, ln, rc[i]);      // (16 tokens are 64 floats)
        f32x4 z_own = {0.f, 0.f, 0.f, 0.f};
        // (R = 64, a piece of dX for every wavefront: its products run under the production)
        constexpr bool kAllDx = 2 * C::NT == kWaves && !G::T16;
        DxOperands dxo;
        f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
        if (kAllDx && !first) dx_load(my_dx, dxo);
        if (kAllProject) z_own = project(w, it);             // (under the production)
        if (kAllDx && !first) dx_mma(dxo, x0, x1);
        if (G::T16) {
            stage_y(it + 1);
            fetch_y(it + 2);
        }
        if (!kAllDx && !first && my_dx >= 0) {
            dx_load(my_dx, dxo);
            dx_mma(dxo, x0, x1);
            dx_store(my_dx, it - 1, x0, x1);
        }
        if (produces) {
            if constexpr (G::T16) produce<C, G::SLOTS, C::PST>(pre_w, slot, ln, a.soft(), ln < nvalid, phw, step);
            else produce_table<C, C::PS>(own_w, tl0, ln, h, a.soft(), ln < nvalid, phw, step);
        }
        if (kAllDx && !first) dx_store(my_dx, it - 1, x0, x1);
        fetch_w(it + 1);
        if (kAllProject) {
            finish_projection(w, it, z_own);
        } else {
#pragma unroll
            for (int pi = 0; pi < 2; ++pi) {
                if (my_proj[pi] < 0) break;
                finish_projection(my_proj[pi], it, project(my_proj[pi], it));
            }
        }
        if (intra && my_tt >= 0) {
            // T^T[b][a] = Yw_b . Yr_a + sw_b sr_a, one of the three 16 x 16 tiles (b, a) that the mask leaves: the two on the
            // diagonal and one off it; both row tiles keep their columns in the same order, which is all a contraction needs
            const int lo = opaque(lane, step), n = lo & 15, q = lo >> 4;
            const int bt = my_tt < 2 ? my_tt : (kReverse ? 1 : 0), rt = my_tt < 2 ? my_tt : 1 - bt;
            const bf16raw *brow = buf_yw(it) + (16 * bt + n) * C::YS + 8 * q;
            const unsigned char *arow = at(S::yr + (it & 1) * S::yr_bytes + 16 * rt * C::XS * 2, at16(C::XS, at16x_));
            f32x4 tt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < C::D / 32; ++s) tt = mma16(lds128(brow + 32 * s), operand(arow, 64 * s), tt);
            const int ai = 16 * rt + n;
            const float sra = buf_sr(it)[ai];
            const f32x4 swb = *reinterpret_cast<const f32x4 *>(buf_sw(it) + 16 * bt + 4 * q);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = 16 * bt + 4 * q + v;
                tt[v] = (kReverse ? b >= ai : b <= ai) ? fmaf(swb[v], sra, tt[v]) : 0.f;
            }
            // R = 64: rows 4 q .. of k-step bt belong to lane half q % 2, words 2 (q / 2) .. of its operand;
            // R = 16: k-slots 4 .. 7 of a lane are its rows of the second tile
            uint32_t *dst = G::T16 ? reinterpret_cast<uint32_t *>(ttop + 64 * rt + lo) + 2 * bt
                                   : reinterpret_cast<uint32_t *>(ttop + 64 * bt + 32 * (q & 1) + ai) + 2 * (q >> 1);
            *reinterpret_cast<u32x2 *>(dst) = u32x2{pack2(tt[0], tt[1]), pack2(tt[2], tt[3])};
        }
    };
    if constexpr (kRotate) {
        if (ntiles > 0) first_half(0, true);
    }
    for (int it = 0; it < ntiles; ++it) {
        step = it;
        if constexpr (!kRotate) first_half(it, it == 0);
        const int64_t t0 = tile_t0(it);
        const int nvalid = tile_nv(t0);
        __syncthreads();

        // ================ second half
        if (!G::T16 && w >= 4) lead(true);
        const bf16raw *yr = buf_yr(it), *yw = buf_yw(it);
        if constexpr (G::T16) {
            // ---- R = 16.  Per table and half of the tokens, lane (n16, q16): cotangents of corners 4 q16 + v of token 16 th + n16.
            // The sums over corners and the finish are those of the other form, below: bits 0, 1 of the corner are the
            // register, bits 2, 3 the row of lanes; lane row q16 finishes hyperplane q16.
            const int tr_ph = 4 * (((lane & 1) << 1) | ((lane >> 1) & 1));         // a table's corners: blocks 0, 2, 1, 3
            float radial[kTh];
#pragma unroll
            for (int t = 0; t < kTh; ++t) radial[t] = 0.f;
#pragma unroll
            for (int i = 0; i < G::TPW; ++i) {
                u32x4 sop[C::D / 32];
#pragma unroll
                for (int j = 0; j < C::D / 32; ++j)
                    sop[j] = u32x4{pack2(SU[i][2 * j][0], SU[i][2 * j][1]), pack2(SU[i][2 * j][2], SU[i][2 * j][3]),
                                   pack2(SU[i][2 * j + 1][0], SU[i][2 * j + 1][1]), pack2(SU[i][2 * j + 1][2], SU[i][2 * j + 1][3])};
                u32x4 pa;
                if (intra) pa = lds_tr16(phw + r_own + 16 * i, C::PST, 4 * q16, 16 + 4 * q16, tr_ph, lane);
                const f32x4 am = *reinterpret_cast<const f32x4 *>(mass + 16 * i + 4 * q16);
#pragma unroll
                for (int th = 0; th < kTh; ++th) {
                    const int tok = 16 * (th0 + th) + n16;
                    const float *c = rc[i * kTh + th];
                    f32x4 dP = am * buf_sr(it)[tok];
                    if (intra) dP = mma16(pa, ttop[64 * (th0 + th) + lane], dP);
                    const bf16raw *yrow = yr + tok * C::XS + 8 * q16;
#pragma unroll
                    for (int j = 0; j < C::D / 32; ++j) dP = mma16(sop[j], lds128(yrow + 32 * j), dP);
                    float p0, q0, p1, q1;
                    code_masses(c[0], p0, q0);
                    code_masses(c[1], p1, q1);
                    const float m2 = side_mass(c[2], q16 & 1), m3 = side_mass(c[3], q16 >> 1);
                    // expectations over bit 0, then differences and expectation over bits 0 and 1
                    const float f0 = fmaf(p0, dP[1], q0 * dP[0]), f1 = fmaf(p0, dP[3], q0 * dP[2]);
                    const float e0 = fmaf(p1, dP[3] - dP[2], q1 * (dP[1] - dP[0])), e1 = f1 - f0, m = fmaf(p1, f1, q1 * f0);
                    const float F = m2 * m3, E = sum_rows4(F * e0, F * e1, m3 * ((q16 & 1) ? m : -m), m2 * ((q16 & 2) ? m : -m));
                    // (values, not elements: a selection between array elements is taken for an index and sends the array to memory)
                    const float c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
                    const float ce = (q16 & 2) ? ((q16 & 1) ? +c3 : +c2) : ((q16 & 1) ? +c1 : +c0);
                    const float du = 2.f * minor_major(ce) * E;
                    const int at = ((tl0 + i) * kTile + tok) * 4 + q16;
                    float dzv = a.beta * du * reinterpret_cast<const float *>(s2t)[at];
                    if (UNIT) dzv *= buf_nrm(it)[tok];
                    const uint32_t dzw = pack2(dzv, 0.f);
                    dz[tok * S::DZS + 4 * (tl0 + i) + q16] = static_cast<bf16raw>(dzw);
                    if (a.want_dbeta && tok < nvalid) dbeta_acc = fmaf(du, reinterpret_cast<const float *>(tht)[at], dbeta_acc);
                    if (UNIT) radial[th] = fmaf(reinterpret_cast<const float *>(zzt)[at], bf_lo(dzw), radial[th]);
                }
                if (intra) {
                    // ---- statistics += Yw^T . phi_writer
                    const u32x4 pb = lds_tr16(phw + r_own + 16 * i, C::PST, 8 * q16, 8 * q16 + 4, tr_ph, lane);
                    macc[i] += column_sum<SIDE == 1>(SIDE == 1 ? lds128(buf_swp(it) + parts_offset16(kTile, opaque(lane, step))) : ones16(opaque(lane, step)), pb);
#pragma unroll
                    for (int ct = 0; ct < C::D / 16; ++ct)
                        SU[i][ct] = mma16(lds_tr16(yw, C::YS, 8 * q16, 8 * q16 + 4, 32 * (ct >> 1) + 8 * (lane & 3) + 4 * (ct & 1), lane), pb, SU[i][ct]);
                    if (q16 == 0) mass[16 * i + n16] = macc[i];
                }
            }
            if (UNIT) {
#pragma unroll
                for (int th = 0; th < kTh; ++th) {
                    const float x = sum_rows(radial[th]);
                    if (q16 == 0) rad[w * kTile + 16 * (th0 + th) + n16] = x;
                }
            }
        } else {
            // extra columns as bf16 (hi, lo) pairs: three products hi*hi + hi*lo + lo*hi keep 16 mantissa bits
            float sr_hi = 1.f, sr_lo = 0.f;                  // (key side: [V | 1])
            if (SIDE == 0) split_bf16(buf_sr(it)[ln], sr_hi, sr_lo);
            const u32x4 sr_a = (h == 0) ? u32x4{pack2(sr_hi, sr_hi), pack2(sr_lo, 0.f), 0u, 0u} : u32x4{0u, 0u, 0u, 0u};

            // ---- per 32-row tile of this wavefront: cotangent of the reader's assignments, transposed (lane = token,
            //      register v = bucket row r_own + 32 mr + acc_row(v, h)), then straight back through the corner
            //      softmax (Algorithm 1, step 4) in those registers.  phi_c is the product over the bits of p_t (bit set) or
            //      q_t (Section 3.3: the corner softmax factorises), so sum_c phi_c dphi_c is linear in every p_t, and with
            //      E_t the difference of its two sides, the expectation of dphi over the other bits with bit t set minus
            //      that with bit t clear, the cotangent of u_t = tanh z_t is 2 beta p_t q_t E_t: p_t q_t = small (1 - small)
            //      is exact to rounding also where a bit is saturated (small ~ 1e-7 at beta = 8), which the cotangent of
            //      beta needs.  Register v of lane half h is corner 32 mr + 8 (v / 4) + 4 h + v % 4: bits 0, 1 are v % 4, bit 2
            //      is h, bits 3, 4 are v / 4, bit 5 is mr.  The 32 corners of a lane are contracted once over bits 3 - 5
            //      (into lows[4]) and once over bits 0, 1 and then bit 5 (into highs[4]), and the E_t are differences of those.  (Sums over the minor side of each bit: 170 vector instructions a tile instead of 120.)
            float p[C::P], q[C::P];
#pragma unroll
            for (int t = 0; t < C::P; ++t) code_masses(rc[0][t], p[t], q[t]);
            const float wl[4] = {q[0] * q[1], p[0] * q[1], q[0] * p[1], p[0] * p[1]};
            const float wm[4] = {q[3] * q[4], p[3] * q[4], q[3] * p[4], p[3] * p[4]};
            float lows[4], highs[4], e5 = 0.f;      // (bit 5 is contracted, and its difference taken, as the tiles come)
#pragma unroll
            for (int mr = 0; mr < G::MTG; ++mr) {
                f32x16 dP;
                if (mr == 1 && w >= 4) lead(false);
                {
                    // extra column first: sr_a * (A or dA)[r] with the masses before this tile
                    float m_hi, m_lo;
                    split_bf16(macc[mr], m_hi, m_lo);
                    const u32x4 mb = (h == 0) ? u32x4{pack2(m_hi, m_lo), pack2(m_hi, 0.f), 0u, 0u} : u32x4{0u, 0u, 0u, 0u};
                    dP = mma(mb, sr_a, f32x16{0});
                }
                if (intra) {
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        dP = mma(lds_tr_acc<true, true>(phw, C::PS, 16 * s, r_own + 32 * mr, ln, h), ttop[64 * s + lane], dP);
                }
                {
                    const int yo = ln * C::XS + 8 * h;
#pragma unroll
                    for (int mtc = 0; mtc < C::NT; ++mtc) {
#pragma unroll
                        for (int s = 0; s < 2; ++s) {
                            const int cc = 32 * mtc + 16 * s;
                            dP = mma(acc_operand(ST[mr][mtc], s), lds128(yr + yo + cc), dP);
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float wh = wm[k] * (mr ? p[C::P - 1] : q[C::P - 1]);
                    float x = wl[0] * dP[4 * k];
#pragma unroll
                    for (int v = 1; v < 4; ++v) x = fmaf(wl[v], dP[4 * k + v], x);
                    highs[k] = mr ? fmaf(p[C::P - 1], x, highs[k]) : q[C::P - 1] * x;
                    e5 = fmaf(mr ? wm[k] : -wm[k], x, e5);
#pragma unroll
                    for (int v = 0; v < 4; ++v) lows[v] = (mr || k) ? fmaf(wh, dP[4 * k + v], lows[v]) : wh * dP[v];
                }
            }
            // E_t of this lane half, the mass of its value of bit 2 included (for bit 2 itself: the signed half)
            float E[8];
            {
                const float F = h ? p[2] : q[2];
                E[0] = F * fmaf(p[1], lows[3] - lows[2], q[1] * (lows[1] - lows[0]));
                E[1] = F * fmaf(p[0], lows[3] - lows[1], q[0] * (lows[2] - lows[0]));
                const float g0 = fmaf(p[3], highs[1], q[3] * highs[0]), g1 = fmaf(p[3], highs[3], q[3] * highs[2]), m = fmaf(p[4], g1, q[4] * g0);
                E[2] = h ? m : -m;
                E[3] = F * fmaf(p[4], highs[3] - highs[2], q[4] * (highs[1] - highs[0]));
                E[4] = F * (g1 - g0);
                E[5] = F * e5;
                E[6] = E[7] = 0.f;
            }
            // ---- finish per (token, table): du_t = 2 beta p_t q_t E_t,  dz_t = du_t (1 - tanh^2 z_t);
            //      the two lane halves hold the two values of bit 2: add them up; lane half h' gets the quad 4h' .. 4h'+3
            // unit-norm option: dz is the cotangent of W xhat, so the reader's row gets dx = (g - xhat (xhat . g)) / |x| with
            // g = W^T dz and xhat . g = z . dz; dz is scaled by 1 / |x| here and this lane's share of z . dz is summed from the
            // bf16 values the matrix product below will see (which keeps dx orthogonal to x to fp32 accuracy)
            float radial = 0.f;
            {
                const float rs = UNIT ? buf_nrm(it)[ln] : 1.f;
                {
                    const int quad = (C::PP / 4) * tl0 + h, at = quad * kTile + ln;
                    const f32x4 s2 = s2t[at];
                    f32x4 uu = {0.f, 0.f, 0.f, 0.f};
                    if (a.want_dbeta) uu = tht[at];
                    float dzv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // slots beyond the table's hyperplanes: all mass on one side, du = 0
                        const float pq = h ? (4 + e < C::P ? p[4 + e < C::P ? 4 + e : 0] * q[4 + e < C::P ? 4 + e : 0] : 0.f) : p[e] * q[e];
                        const float du = 2.f * pq * sum_halves2(E[e], E[4 + e]);       // cotangent of u_t up to the factor beta
                        dzv[e] = a.beta * du * s2[e] * rs;
                        if (a.want_dbeta && ln < nvalid) dbeta_acc = fmaf(du, uu[e], dbeta_acc);   // (not the copies past the end)
                    }
                    const u32x2 dzw = {pack2(dzv[0], dzv[1]), pack2(dzv[2], dzv[3])};
                    *reinterpret_cast<u32x2 *>(dz + ln * S::DZS + 4 * quad) = dzw;
                    if (UNIT) {
                        const f32x4 z4 = zzt[at];
                        radial = fmaf(z4[0], bf_lo(dzw.x), radial);
                        radial = fmaf(z4[1], bf_hi(dzw.x), radial);
                        radial = fmaf(z4[2], bf_lo(dzw.y), radial);
                        radial = fmaf(z4[3], bf_hi(dzw.y), radial);
                    }
                }
            }
            if (UNIT) {
                radial = sum_halves(radial);
                if (h == 0) rad[w * kTile + ln] = radial;
            }
        }
        if (!G::T16) {          // (not before every wavefront has updated its statistics with the rows that lie there)
            stage_y(it + 1);
            fetch_y(it + 2);
        }
        stage_x(it + 1);
        fetch_x(it + 2);
        __syncthreads();        // dz is visible; this tile's assignments, in-tile term and tanh are dead from here on
        if (kRotate && G::T16 && it + 1 == ntiles) break;
        if constexpr (!G::T16) {
            // ---- statistics += Yw^T . phi_writer
            if (intra) {
                const int lo = opaque(lane, step), swp_off = parts_offset32<true>(kTile, lo);
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const u32x4 gw = SIDE == 1 ? lds128(buf_swp(it) + swp_off + 16 * s) : ones32<true>(lo);   // (SIDE 0: [V | 1])
                    u32x4 ay[C::NT];
#pragma unroll
                    for (int mtc = 0; mtc < C::NT; ++mtc) ay[mtc] = lds_tr_plain<true>(yw, C::YS, 16 * s, 32 * mtc, ln, h);
#pragma unroll
                    for (int mr = 0; mr < G::MTG; ++mr) {
                        const u32x4 bp = lds_tr_plain<true, true>(phw, C::PS, 16 * s, r_own + 32 * mr, ln, h);
                        macc[mr] += column_sum<SIDE == 1>(gw, bp);
#pragma unroll
                        for (int mtc = 0; mtc < C::NT; ++mtc) ST[mr][mtc] = mma(ay[mtc], bp, ST[mr][mtc]);
                    }
                }
            }
        }
        if constexpr (kRotate) first_half(it + 1, false);
    }
    // (R = 64 comes past the end of the last tile and forms its dX there: with the loop left in the middle the statistics of the long
    // sequences are spilled, and both gradients take 4 % more)
    if (G::T16 && ntiles > 0 && my_dx >= 0) {
        DxOperands dxo;
        f32x4 x0, x1;
        dx_load(my_dx, dxo);
        dx_mma(dxo, x0, x1);
        dx_store(my_dx, ntiles - 1, x0, x1);
    }
    // ---- cotangent of beta: lanes -> wavefront (shuffles) -> workgroup (LDS, wavefront order) -> one workspace slot
    if (a.want_dbeta) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) dbeta_acc += __shfl_xor(dbeta_acc, m, 64);
        __syncthreads();
        float *sums = reinterpret_cast<float *>(lds + S::sr);
        if (lane == 0) sums[w] = dbeta_acc;
        __syncthreads();
        if (tid == 0) {
            float s = 0.f;
            for (int i = 0; i < kWaves; ++i) s += sums[i];
            const int wgs = gridDim.x;                  // workgroups per (side, batch*head)
            a.dbeta_part[(static_cast<size_t>(SIDE) * gridDim.y + bh) * wgs + seg] = s;
        }
    }
}

}  // namespace mfma
}  // namespace race
