// Fused tiled Newton–Schulz kernels for gfx950 (MI355X).
//
// One launch evaluates Phi_K (Sec. 2.2, eqs. ns_iteration / ns_quintic /
// phi_k_def) on every tile of a chunk of the batched tile set (Sec. 4.1,
// eq. tiled_ns; Sec. 4.4.2, cross-layer batching). Each tile is read from HBM
// once, kept on chip (registers + LDS) for all K steps, and written once.
//
// Data layout on chip. A tile is a grid of 32x32 blocks (NB = T/32 per side).
// A wave owns RB consecutive block rows ("row blocks") of its tile and keeps
// them as fp32 v_mfma 32x32 accumulators. In that accumulator layout lane l
// holds, for block column q, the 16 values
//     row  = l % 32,
//     cols = 8g + 4(l/32) + e        (g, e = 0..3; register 4g+e),
// i.e. a piece of one row ("row piece"). Because A = X X^T and A^2 = A A^T
// contract over columns, a row piece is already a valid MFMA operand for
// both Gram-type products, and with the operands in the order
// (other rows, own rows) the MFMA result is again a row piece of the output
// (A is symmetric). No transpose is needed for those two products.
//
// The third product, B X, contracts X over rows. Its MFMA operand is a
// "column piece" of X (one column, rows in the same 8g+4h+e pattern); every
// step writes X once more to LDS in that layout, after a 4x4 transpose
// inside each lane quad done with DPP (no LDS traffic for the transpose).
//
// Epilogues. With 16-bit operands they live in the accumulators: the A^2
// accumulator starts from (b/c)·A and is scaled by c, giving B = bA + cA^2
// from fp32 A; the product accumulator starts from a·X (fp32 master copy),
// giving aX + BX. With fp32 operands every accumulator starts at zero (four
// chains each) and B = fma(c, A^2, bA), X = fma(a, X, BX) are formed once at
// the end, which keeps large partial sums out of the fp32 rounding walk.
// Operands are rounded once (fp16 or bf16, round to nearest even) or stay fp32.
//
// fp32 tiles of 64 and 128 evaluate only the upper blocks of the symmetric A and
// B (40 and 36 of 48 block products; steps64, steps128 below): 24 matrices of 4M
// entries, T = 128, K = 8 5131 -> 3893 us, T = 64, K = 5 1843 -> 1383 us: 159 and
// 140 TFLOP/s counted as if every product were done (the fp32 MFMA peak is 157).
//
// LDS holds, per tile, one operand matrix of row pieces ("xr", only when a
// tile is split over several waves; it carries X and then A) and one of
// column pieces ("xc"), both as 16-byte-per-lane slots in lane order so
// every LDS read and most writes are conflict-free 128-bit accesses.
#include "ns_device.h"

#include <atomic>
#include <type_traits>

namespace himuon {
namespace {

using namespace dev;

constexpr int kThreads = 256;  // four waves per workgroup

// T: tile size; RB: 32-row blocks per wave. A tile is spread over
// WT = T/(32 RB) waves, and a workgroup of four waves runs 4/WT tiles.
// OPT: the optimizer step of Alg. 1 rides on the tile I/O (KernelArgs): the
// gather loads G and M, stores M <- beta M + G and takes the lookahead
// G + beta M (Nesterov) or M, formed from the stored M, as the tile; the
// write-back loads W and stores (1 - lr lambda) W - lr tau U.
template <int T, int RB, Storage ST, Operand OP, bool OPT = false>
__global__ void __launch_bounds__(kThreads) ns_tiled_kernel(const KernelArgs args)
{
    constexpr int NB = T / 32;
    constexpr int WT = NB / RB;
    static_assert(NB % RB == 0 && WT >= 1 && WT <= 4, "tile split");
    constexpr int TPW = 4 / WT;
    constexpr int S = OperandTraits<OP>::kSlots;
    constexpr int NC = OperandTraits<OP>::kChains;
    constexpr int MAT = NB * NB * S * 64;  // 16-byte slots in one operand matrix
    constexpr bool SHARED_ROWS = WT > 1;
    // fp32 tiles of more than one block evaluate the upper blocks of the
    // symmetric A and B only (steps64, steps128)
    constexpr bool SYM = OP == Operand::F32 && NB > 1;
    static_assert(!SYM || (NB == 2 && WT == 1) || (NB == 4 && WT == 4), "fp32 splits");
    constexpr int BLK = S * 64;  // 16-byte slots of one 32x32 block
    // block exchange: one block per 64-tile, two per wave of a 128-tile (whose
    // 32 KB also lend the reductions of the normalisation their few bytes)
    constexpr int EX = !SYM ? 1 : (SHARED_ROWS ? 8 * BLK : TPW * BLK);

    __shared__ u32x4 s_xr[SHARED_ROWS ? TPW * MAT : 1];
    __shared__ u32x4 s_xc[TPW * MAT];
    __shared__ u32x4 s_ex[EX];
    __shared__ float s_own_red[SYM && SHARED_ROWS ? 1 : 8];
    float (*const s_red)[4] = reinterpret_cast<float (*)[4]>(SYM && SHARED_ROWS ? reinterpret_cast<float*>(s_ex) : s_own_red);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tslot = wave / WT;
    const int p0 = (wave % WT) * RB;  // first owned row block
    const int li = lane & 31, lh = lane >> 5;
    u32x4* const xr = s_xr + (SHARED_ROWS ? tslot * MAT : 0);
    u32x4* const xc = s_xc + tslot * MAT;

    const int64_t n_tiles = args.tile_end - args.tile_begin;
    const int64_t n_groups = (n_tiles + TPW - 1) / TPW;

    int mhint = 0;  // owner of the wave's previous valid tile
    for (int64_t grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
        const int64_t local = grp * TPW + tslot;
        const bool valid = local < n_tiles;
        if constexpr (!SHARED_ROWS || TPW == 1) {
            if (!valid) continue;  // no workgroup barrier depends on this wave
        }
        const int64_t tile = args.tile_begin + (valid ? local : 0);

        // matrix owning the tile: last descriptor with tile_begin <= tile.
        // A wave's valid tiles only grow, so the search starts from the
        // previous owner; an idle wave (the chunk's first tile) searches all.
        const ConstDesc* const descs = desc_table(args);
        int lo;
        if (valid) {
            mhint = find_matrix_from(args, tile, mhint);
            lo = mhint;
        } else {
            int l = 0, hi = args.n_mats - 1;
            while (l < hi) {
                const int mid = (l + hi + 1) >> 1;
                if (descs[mid].tile_begin <= tile) l = mid;
                else hi = mid - 1;
            }
            lo = __builtin_amdgcn_readfirstlane(l);
        }
        const ConstDesc& d = descs[lo];
        // (32-bit: tile ids of one call fit in 32 bits, checked on the host)
        const uint32_t lt = (uint32_t)(tile - d.tile_begin);
        const uint32_t tc = (uint32_t)d.tiles_c;
        const uint32_t tr = lt / tc;
        const int64_t row0 = (int64_t)tr * T, col0 = (int64_t)(lt - tr * tc) * T;
        const bool full = row0 + T <= d.rows && col0 + T <= d.cols;
        const bool vin = full && (d.flags & MAT_VEC_IN);
        const bool vout = full && (d.flags & MAT_VEC_OUT);
        const int64_t rows_eff = valid ? d.rows : 0;  // an idle wave reads zeros

        void* mom = nullptr;
        float tau = 0.f;
        if constexpr (OPT) {
            const ConstOpt& O = opt_table(args)[lo];
            mom = O.mom;
            tau = O.tau;
        }

        // ---- gather the tile (zero padded) into fp32 row pieces
        f32x16 X[RB][NB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int64_t gr = row0 + 32 * (p0 + rb) + li;
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int64_t gc = col0 + 32 * q + 8 * g + 4 * lh;
                    const f32x4 v = load4<ST>(d.in, gr, gc, d.ld_in, rows_eff, d.cols, vin);
                    float x4[4] = {v[0], v[1], v[2], v[3]};
                    if constexpr (OPT) {
                        // (the momentum shares the gradient's layout; padding stays zero)
                        const f32x4 m = load4<ST>(mom, gr, gc, d.ld_in, rows_eff, d.cols, vin);
                        const f32x4 mn = stored4<ST>(f32x4{args.beta * m[0] + x4[0], args.beta * m[1] + x4[1],
                                                           args.beta * m[2] + x4[2], args.beta * m[3] + x4[3]});
                        if (valid) store4<ST>(mom, gr, gc, d.ld_in, d.rows, d.cols, vin, mn);
                        const float nb = args.nesterov ? args.beta : 0.f;
                        const float keep = args.nesterov ? 1.f : 0.f;
                        const float mb = args.nesterov ? 0.f : 1.f;
#pragma unroll
                        for (int e = 0; e < 4; ++e) x4[e] = keep * x4[e] + nb * mn[e] + mb * mn[e];
                    }
                    X[rb][q][4 * g + 0] = x4[0];
                    X[rb][q][4 * g + 1] = x4[1];
                    X[rb][q][4 * g + 2] = x4[2];
                    X[rb][q][4 * g + 3] = x4[3];
                }
        }

        // ---- X_0 = S / ||S||_F, after an exact power-of-two pre-scale so the
        //      fp32 sum of squares neither overflows nor underflows
        float mx = 0.f;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, fabsf(X[rb][q][v]));
        mx = wave_max(mx);
        if constexpr (SHARED_ROWS) {
            if (lane == 0) s_red[0][wave] = mx;
            __syncthreads();
            mx = s_red[0][tslot * WT];
#pragma unroll
            for (int w = 1; w < WT; ++w) mx = fmaxf(mx, s_red[0][tslot * WT + w]);
        }
        int ex = 0;
        (void)frexpf(mx, &ex);
        const float s1 = ldexpf(1.f, -(ex / 2)), s2 = ldexpf(1.f, -(ex - ex / 2));
        float ss = 0.f;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float y = X[rb][q][v] * s1 * s2;
                    X[rb][q][v] = y;
                    ss = fmaf(y, y, ss);
                }
        ss = wave_sum(ss);
        if constexpr (SHARED_ROWS) {
            if (lane == 0) s_red[1][wave] = ss;
            __syncthreads();
            ss = s_red[1][tslot * WT];
#pragma unroll
            for (int w = 1; w < WT; ++w) ss += s_red[1][tslot * WT + w];
        }
        // 16-bit operands round the tile anyway: X_0 = S / ||S||_F. fp32
        // operands: the exact power-of-two normalisation (exact_norm), the
        // rest of ||S||_F in the step's coefficients and the output factor.
        float inv = ss > 0.f ? 1.f / sqrtf(ss) : 0.f;  // Phi_K(0) = 0
        ExactNorm en{};
        if constexpr (OP == Operand::F32) {
            en = exact_norm(ss, args.b, args.c);
            inv = en.scale;
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int q = 0; q < NB; ++q) X[rb][q] *= inv;

        // ---- K Newton–Schulz steps, all on chip
        const int t4 = li & 3, quad = li >> 2;
        const int xg = quad >> 1, xh = quad & 1;  // row group of this quad in a block

        // fp32 steps on the upper blocks. What bounds them is the fp32 MFMA (64
        // cycles each) and, on the same units, the vector ALU: a v_add between two
        // of these MFMAs adds its 4 cycles in full and a change from one to the
        // other 13 more (measured; fp16 MFMAs hide such work, fp32 ones do not).
        // So blocks are evaluated one at a time, each product a run of MFMAs
        // alone, and the vector work is kept to the sums and polynomials: no
        // copies out of accumulation registers, and transposes go through
        // LDS by 4-byte writes instead of lane exchanges.
#define HM_INL __attribute__((always_inline))
        // A block's column pieces: rows 4q .. 4q + 3 of column c in the 16-byte
        // chunk 32 q + (c ^ q), so that neither the 4-byte writes (32 rows of one
        // column) nor the 16-byte reads (32 columns of one q) meet in a bank.
        int twr[4], trd[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            twr[e] = 128 * (li >> 2) + 4 * ((4 * lh + e) ^ (li >> 2)) + (li & 3);
            trd[e] = 32 * (2 * e + lh) + (li ^ (2 * e + lh));
        }
        auto put_t = [&](const f32x16& v, u32x4* dst) HM_INL {
            float* const d = reinterpret_cast<float*>(dst);
#pragma unroll
            for (int r = 0; r < 16; ++r) d[twr[r & 3] + 32 * (r >> 2)] = v[r];
        };
        auto get = [&](const u32x4* src, f32x16& v) HM_INL {
#pragma unroll
            for (int sl = 0; sl < 4; ++sl) {
                const u32x4 w = src[trd[sl]];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * sl + e] = __uint_as_float(w[e]);
            }
        };
        // acc = sum over g < NG of opa(g) x opb(g), LDS operands two groups ahead
        auto product = [&](auto ng, auto&& opa, auto&& opb, f32x16 (&acc)[NC]) HM_INL {
            constexpr int NG = decltype(ng)::value;
#pragma unroll
            for (int ch = 0; ch < NC; ++ch) acc[ch] = f32x16{};
            u32x4 nxt[2] = {opa(0), opa(1)};
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const u32x4 cur = nxt[g & 1];
                if (g + 2 < NG) nxt[g & 1] = opa(g + 2);
                mma<OP>(cur, opb(g), acc);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto sum4 = [](const f32x16 (&acc)[NC], int r) HM_INL -> float {
            if constexpr (NC == 4) return (acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r]);
            else return acc[0][r];
        };
        auto sum = [&](const f32x16 (&acc)[NC], f32x16& v) HM_INL {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = sum4(acc, r);
        };
        // b' A + c' Q, Q the sum of the chains (b' A for c = 0)
        auto poly = [&](const f32x16& g, const f32x16 (&acc)[NC], f32x16& v) HM_INL {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = poly2(en, g[r], sum4(acc, r));
        };
        auto linear = [&](const f32x16& g, f32x16& v) HM_INL {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = fmaf(en.bh, g[r], en.bl * g[r]);
        };
        auto update = [&](f32x16& x, const f32x16 (&acc)[NC]) HM_INL {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = fmaf(args.a, x[r], sum4(acc, r));
        };

        // 64-tile, one wave: block (1, 0) of A and of B is the transpose of (0, 1)
        auto steps64 = [&](auto quintic) HM_INL {
          if constexpr (SYM && NB == 2) {
            constexpr bool QUINTIC = decltype(quintic)::value;  // c != 0
            u32x4* const ex = s_ex + tslot * BLK;
            constexpr std::integral_constant<int, 8> ng{};
            auto op = [&](const f32x16 (&R)[2]) HM_INL { return [&](int g) HM_INL { return make_slot<OP>(R[g >> 2], g & 3); }; };
            auto xcol = [&](int N) HM_INL { return [&, N](int g) HM_INL { return xc[((g >> 2) * 2 + N) * BLK + trd[g & 3]]; }; };
            for (int k = 0; k < args.K; ++k) {
                f32x16 G[2][2], B[2][2], acc[NC];
#pragma unroll
                for (int b = 0; b < 4; ++b) put_t(X[b >> 1][b & 1], xc + b * BLK);
                product(ng, op(X[1]), op(X[0]), acc);
                sum(acc, G[0][1]);
                put_t(G[0][1], ex);
                product(ng, op(X[0]), op(X[0]), acc);
                sum(acc, G[0][0]);
                get(ex, G[1][0]);
                product(ng, op(X[1]), op(X[1]), acc);
                sum(acc, G[1][1]);
                if constexpr (QUINTIC) {
                    product(ng, op(G[1]), op(G[0]), acc);
                    poly(G[0][1], acc, B[0][1]);
                    put_t(B[0][1], ex);
                    product(ng, op(G[0]), op(G[0]), acc);
                    poly(G[0][0], acc, B[0][0]);
                    product(ng, op(G[1]), op(G[1]), acc);
                    poly(G[1][1], acc, B[1][1]);
                    get(ex, B[1][0]);
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b) linear(G[b >> 1][b & 1], B[b >> 1][b & 1]);
                }
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    product(ng, xcol(b & 1), op(B[b >> 1]), acc);
                    update(X[b >> 1][b & 1], acc);
                }
            }
          }
        };

        // 128-tile, four waves of one block row each. Wave p evaluates blocks
        // (p, p), (p, p + 1) and half the k range of (p, p + 2) (indices mod 4; the
        // other half of that block comes, transposed, from wave p + 2), which
        // is every block pair once and the same work for every wave. Block
        // (p, p + 3) is the transpose of wave p - 1's (p - 1, p). k blocks run in
        // an order that ends with the wave's own (the diagonal block of B is the
        // largest: entering the chains last it rounds the fewest partial sums).
        auto steps128 = [&](auto quintic) HM_INL {
          if constexpr (SYM && NB == 4) {
            constexpr bool QUINTIC = decltype(quintic)::value;  // c != 0
            constexpr std::integral_constant<int, 16> n16{};
            constexpr std::integral_constant<int, 8> n8{};
            const int p = p0, p1 = (p + 1) & 3, p2 = (p + 2) & 3;
            // the k block (offset from p) of group g: 2, 3, 1, 0, or the half's 1, 0
            auto off16 = [](int g) HM_INL { return (g >> 2) < 2 ? 2 + (g >> 2) : 3 - (g >> 2); };
            auto off8 = [](int g) HM_INL { return 1 - (g >> 2); };
            auto row16 = [&](int J) HM_INL { return [&, J](int g) HM_INL { return xr[((J * 4 + ((p + off16(g)) & 3)) * S + (g & 3)) * 64 + lane]; }; };
            auto row8 = [&](int J) HM_INL { return [&, J](int g) HM_INL { return xr[((J * 4 + ((p + off8(g)) & 3)) * S + (g & 3)) * 64 + lane]; }; };
            auto op16 = [&](const f32x16 (&R)[4]) HM_INL { return [&](int g) HM_INL { return make_slot<OP>(R[off16(g)], g & 3); }; };
            auto op8 = [&](const f32x16 (&R)[4]) HM_INL { return [&](int g) HM_INL { return make_slot<OP>(R[off8(g)], g & 3); }; };
            auto xcol = [&](int j) HM_INL {
                return [&, j](int g) HM_INL { return xc[(((p + off16(g)) & 3) * 4 + ((p + j) & 3)) * BLK + trd[g & 3]]; };
            };
            auto publish = [&](const f32x16 (&R)[4]) HM_INL {  // the wave's block row as operand slots
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int sl = 0; sl < S; ++sl) xr[((p * 4 + ((p + j) & 3)) * S + sl) * 64 + lane] = make_slot<OP>(R[j], sl);
            };
            // s_ex: blocks 0..3 for wave p + 1 ((p, p + 1) transposed, its R[3]), 4..7 for
            // wave p + 2 (this wave's half of (p, p + 2), transposed)
            auto offer = [&](const f32x16& r1, const f32x16& r2) HM_INL {
                put_t(r1, s_ex + p1 * BLK);
                put_t(r2, s_ex + (4 + p2) * BLK);
                __syncthreads();
            };
            auto take = [&](f32x16 (&R)[4]) HM_INL {
                f32x16 h;
                get(s_ex + p * BLK, R[3]);
                get(s_ex + (4 + p) * BLK, h);
                R[2] += h;
            };
            // the block rows in rotated order: R[j] is block (p, p + j) (selected,
            // not indexed: an index would send the tile to scratch)
            f32x16 Xr[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                Xr[j] = X[0][j];
                if (p == 1) Xr[j] = X[0][(j + 1) % 4];
                if (p == 2) Xr[j] = X[0][(j + 2) % 4];
                if (p == 3) Xr[j] = X[0][(j + 3) % 4];
            }
            for (int k = 0; k < args.K; ++k) {
                f32x16 G[4], B[4], acc[NC];
                publish(Xr);
#pragma unroll
                for (int j = 0; j < 4; ++j) put_t(Xr[j], xc + (p * 4 + ((p + j) & 3)) * BLK);
                product(n16, op16(Xr), op16(Xr), acc);  // (the stores above land meanwhile)
                sum(acc, G[0]);
                __syncthreads();
                product(n16, row16(p1), op16(Xr), acc);
                sum(acc, G[1]);
                product(n8, row8(p2), op8(Xr), acc);
                sum(acc, G[2]);
                offer(G[1], G[2]);  // (its barrier: every wave is done reading X from xr)
                take(G);
                if constexpr (QUINTIC) {
                    publish(G);
                    product(n16, op16(G), op16(G), acc);
                    poly(G[0], acc, B[0]);
                    __syncthreads();
                    product(n16, row16(p1), op16(G), acc);
                    poly(G[1], acc, B[1]);
                    product(n8, row8(p2), op8(G), acc);
                    sum(acc, B[2]);
                    offer(B[1], B[2]);
                    take(B);
#pragma unroll
                    for (int r = 0; r < 16; ++r) B[2][r] = poly2(en, G[2][r], B[2][r]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) linear(G[j], B[j]);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    product(n16, xcol(j), op16(B), acc);
                    update(Xr[j], acc);
                }
                __syncthreads();  // xr, xc and the exchange blocks are rewritten next step
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                X[0][j] = Xr[j];
                if (p == 1) X[0][j] = Xr[(j + 3) % 4];
                if (p == 2) X[0][j] = Xr[(j + 2) % 4];
                if (p == 3) X[0][j] = Xr[(j + 1) % 4];
            }
          }
        };
#undef HM_INL
        constexpr std::true_type with_c{};
        constexpr std::false_type without_c{};
        if constexpr (SYM && NB == 2) {
            if (args.c != 0.f) steps64(with_c);
            else steps64(without_c);
        } else if constexpr (SYM) {
            if (args.c != 0.f) steps128(with_c);
            else steps128(without_c);
        } else {
        for (int k = 0; k < args.K; ++k) {
            u32x4 Xop[RB][NB][S];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int q = 0; q < NB; ++q)
#pragma unroll
                    for (int s = 0; s < S; ++s) Xop[rb][q][s] = make_slot<OP>(X[rb][q], s);

            if constexpr (SHARED_ROWS) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int q = 0; q < NB; ++q)
#pragma unroll
                        for (int s = 0; s < S; ++s) xr[(((p0 + rb) * NB + q) * S + s) * 64 + lane] = Xop[rb][q][s];
            }
            // column pieces of X for the B X product
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int Q = p0 + rb;
#pragma unroll
                for (int N = 0; N < NB; ++N)
#pragma unroll
                    for (int gp = 0; gp < 4; ++gp) {
                        const int lane_dst = xh * 32 + 8 * gp + 4 * lh + t4;
                        if constexpr (OP == Operand::F32) {
                            const f32x4 c = {X[rb][N][4 * gp + 0], X[rb][N][4 * gp + 1], X[rb][N][4 * gp + 2],
                                             X[rb][N][4 * gp + 3]};
                            const f32x4 o = quad_transpose32(c, t4);
                            xc[((Q * NB + N) * S + xg) * 64 + lane_dst] = __builtin_bit_cast(u32x4, o);
                        } else {
                            const u32x4& w = Xop[rb][N][gp >> 1];
                            const u32x2 o = quad_transpose16(w[(gp & 1) * 2], w[(gp & 1) * 2 + 1], t4);
                            u32x2* dst = reinterpret_cast<u32x2*>(&xc[((Q * NB + N) * S + (xg >> 1)) * 64 + lane_dst]);
                            dst[xg & 1] = o;
                        }
                    }
            }
            if constexpr (SHARED_ROWS) __syncthreads();

            // A = X X^T as row pieces of the owned rows
            f32x16 G[RB][NB];
            {
                f32x16 Gc[RB][NB][NC];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int J = 0; J < NB; ++J)
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch) Gc[rb][J][ch] = f32x16{};
#pragma unroll
                for (int J = 0; J < NB; ++J)
#pragma unroll
                    for (int q = 0; q < NB; ++q)
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            u32x4 opa;
                            if constexpr (SHARED_ROWS) opa = xr[((J * NB + q) * S + s) * 64 + lane];
                            else opa = Xop[J][q][s];
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma<OP>(opa, Xop[rb][q][s], Gc[rb][J]);
                        }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int J = 0; J < NB; ++J) G[rb][J] = chain_sum<NC>(Gc[rb][J]);
            }

            // B = bA + cA^2. 16-bit operands: accumulated in place as
            // c((b/c)A + A A^T). fp32 operands: A^2 in zero-started chains,
            // then one fused b*A + c*A^2 from the fp32 A (no large partial sums).
            if (args.c != 0.f) {
                u32x4 Aop[RB][NB][S];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int J = 0; J < NB; ++J) {
#pragma unroll
                        for (int s = 0; s < S; ++s) Aop[rb][J][s] = make_slot<OP>(G[rb][J], s);
                        if constexpr (OP != Operand::F32) G[rb][J] *= args.b_over_c;
                    }
                if constexpr (SHARED_ROWS) {
                    __syncthreads();  // every wave is done reading X from xr
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int J = 0; J < NB; ++J)
#pragma unroll
                            for (int s = 0; s < S; ++s) xr[(((p0 + rb) * NB + J) * S + s) * 64 + lane] = Aop[rb][J][s];
                    __syncthreads();
                }
                f32x16 Gc[RB][NB][NC];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int J = 0; J < NB; ++J) {
                        if constexpr (OP == Operand::F32) Gc[rb][J][0] = f32x16{};
                        else Gc[rb][J][0] = G[rb][J];
#pragma unroll
                        for (int ch = 1; ch < NC; ++ch) Gc[rb][J][ch] = f32x16{};
                    }
#pragma unroll
                for (int J = 0; J < NB; ++J)
#pragma unroll
                    for (int q = 0; q < NB; ++q)
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            u32x4 opa;
                            if constexpr (SHARED_ROWS) opa = xr[((J * NB + q) * S + s) * 64 + lane];
                            else opa = Aop[J][q][s];
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma<OP>(opa, Aop[rb][q][s], Gc[rb][J]);
                        }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int J = 0; J < NB; ++J) {
                        const f32x16 sq = chain_sum<NC>(Gc[rb][J]);
                        if constexpr (OP == Operand::F32) {
#pragma unroll
                            for (int v = 0; v < 16; ++v) G[rb][J][v] = poly2(en, G[rb][J][v], sq[v]);
                        } else {
                            G[rb][J] = sq * args.c;
                        }
                    }
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int J = 0; J < NB; ++J) {
                        if constexpr (OP == Operand::F32) {
#pragma unroll
                            for (int v = 0; v < 16; ++v) G[rb][J][v] = fmaf(en.bh, G[rb][J][v], en.bl * G[rb][J][v]);
                        } else {
                            G[rb][J] *= args.b;
                        }
                    }
            }

            // X <- aX + B X
            u32x4 Bop[RB][NB][S];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int Q = 0; Q < NB; ++Q)
#pragma unroll
                    for (int s = 0; s < S; ++s) Bop[rb][Q][s] = make_slot<OP>(G[rb][Q], s);
            {
                f32x16 Pc[RB][NB][NC];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int N = 0; N < NB; ++N) {
                        if constexpr (OP == Operand::F32) Pc[rb][N][0] = f32x16{};
                        else Pc[rb][N][0] = X[rb][N] * args.a;
#pragma unroll
                        for (int ch = 1; ch < NC; ++ch) Pc[rb][N][ch] = f32x16{};
                    }
#pragma unroll
                for (int N = 0; N < NB; ++N)
#pragma unroll
                    for (int Q = 0; Q < NB; ++Q)
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            const u32x4 opa = xc[((Q * NB + N) * S + s) * 64 + lane];
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma<OP>(opa, Bop[rb][Q][s], Pc[rb][N]);
                        }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int N = 0; N < NB; ++N) {
                        const f32x16 bx = chain_sum<NC>(Pc[rb][N]);
                        if constexpr (OP == Operand::F32) {
#pragma unroll
                            for (int v = 0; v < 16; ++v) X[rb][N][v] = fmaf(args.a, X[rb][N][v], bx[v]);
                        } else {
                            X[rb][N] = bx;
                        }
                    }
            }
            if constexpr (SHARED_ROWS) __syncthreads();  // xr / xc are rewritten next step
        }

        }

        // ---- write back the unpadded part
        if constexpr (OP == Operand::F32) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int q = 0; q < NB; ++q) X[rb][q] *= en.out;
        }
        if (valid) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int64_t gr = row0 + 32 * (p0 + rb) + li;
#pragma unroll
                for (int q = 0; q < NB; ++q)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int64_t gc = col0 + 32 * q + 8 * g + 4 * lh;
                        f32x4 v = {X[rb][q][4 * g + 0], X[rb][q][4 * g + 1], X[rb][q][4 * g + 2],
                                   X[rb][q][4 * g + 3]};
                        if constexpr (OPT) {
                            // U as the storage type holds it, then the update of the loaded W
                            const f32x4 u = stored4<ST>(v);
                            const f32x4 w = load4<ST>(d.out, gr, gc, d.ld_out, d.rows, d.cols, vout);
                            const float step = args.lr * tau;
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = args.decay * w[e] - step * u[e];
                        }
                        store4<ST>(d.out, gr, gc, d.ld_out, d.rows, d.cols, vout, v);
                    }
            }
        }
    }
}

// fp32 32-tiles, one workgroup of four waves per tile, for calls that leave most
// of the chip idle. A 32-tile's step is a serial chain in one wave: 48 fp32 MFMAs
// of 64 cycles and the sums between them. The four accumulator chains of a
// product (one per element e of an operand slot) are independent: here
// wave w runs chain w, which reads only its elements 4s + w of the row pieces, and
// holds only those. The partial sums go through LDS, each wave taking the
// registers of its own elements from all four chains, so every sum has the terms
// and the order of the one-wave kernel and the result its bits.
// A 256 x 256 matrix (64 tiles), K = 5: 10.1 us a call, 14.1 with one wave per tile.
__global__ void __launch_bounds__(kThreads) ns_tiled_f32_split32_kernel(const KernelArgs args)
{
    __shared__ f32x4 s_ex[2][4][4][64];  // [exchange parity][chain][element][lane]
    __shared__ float s_x[32 * 33];       // X by rows
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int64_t tile = args.tile_begin + blockIdx.x;
    const ConstDesc& d = desc_table(args)[find_matrix_from(args, tile, 0)];
    const uint32_t lt = (uint32_t)(tile - d.tile_begin);
    const uint32_t tc = (uint32_t)d.tiles_c;
    const uint32_t tr = lt / tc;
    const int64_t row0 = (int64_t)tr * 32, col0 = (int64_t)(lt - tr * tc) * 32;
    const bool vin = row0 + 32 <= d.rows && col0 + 32 <= d.cols && (d.flags & MAT_VEC_IN);

    // every wave reads the tile and normalises it as the one-wave kernel does
    f32x16 X;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4 v = load4<Storage::F32>(d.in, row0 + li, col0 + 8 * g + 4 * lh, d.ld_in, d.rows, d.cols, vin);
#pragma unroll
        for (int e = 0; e < 4; ++e) X[4 * g + e] = v[e];
    }
    float mx = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, fabsf(X[v]));
    mx = wave_max(mx);
    int ex = 0;
    (void)frexpf(mx, &ex);
    const float s1 = ldexpf(1.f, -(ex / 2)), s2 = ldexpf(1.f, -(ex - ex / 2));
    float ss = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float y = X[v] * s1 * s2;
        X[v] = y;
        ss = fmaf(y, y, ss);
    }
    ss = wave_sum(ss);
    const ExactNorm en = exact_norm(ss, args.b, args.c);
    X *= en.scale;
    auto mine = [&](const f32x16& v, int s) -> float {
        return w == 0 ? v[4 * s] : (w == 1 ? v[4 * s + 1] : (w == 2 ? v[4 * s + 2] : v[4 * s + 3]));
    };
    float x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = mine(X, s);

    // the wave's elements of the sum of the four chains
    auto reduce = [&](const f32x16& acc, int parity, float (&v)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s_ex[parity][w][e][lane] = f32x4{acc[e], acc[4 + e], acc[8 + e], acc[12 + e]};
        __syncthreads();
        const f32x4 c0 = s_ex[parity][0][w][lane], c1 = s_ex[parity][1][w][lane];
        const f32x4 c2 = s_ex[parity][2][w][lane], c3 = s_ex[parity][3][w][lane];
        const f32x4 t = (c0 + c1) + (c2 + c3);
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = t[s];
    };
    auto chain = [&](const float (&a)[4], const float (&b)[4]) -> f32x16 {
        f32x16 acc = {};
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], b[s], acc, 0, 0, 0);
        return acc;
    };
    int parity = 0;  // (an exchange buffer is rewritten two barriers after it was read)
    for (int k = 0; k < args.K; ++k) {
        // (read again behind the barrier of the first exchange; last read before
        // the barrier of the previous step's last one)
#pragma unroll
        for (int s = 0; s < 4; ++s) s_x[li * 33 + 8 * s + 4 * lh + w] = x[s];
        float g[4], b[4], xc[4];
        reduce(chain(x, x), parity, g);
        parity ^= 1;
#pragma unroll
        for (int s = 0; s < 4; ++s) xc[s] = s_x[(8 * s + 4 * lh + w) * 33 + li];
        if (args.c != 0.f) {
            float q[4];
            reduce(chain(g, g), parity, q);
            parity ^= 1;
#pragma unroll
            for (int s = 0; s < 4; ++s) b[s] = poly2(en, g[s], q[s]);
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) b[s] = fmaf(en.bh, g[s], en.bl * g[s]);
        }
        float bx[4];
        reduce(chain(xc, b), parity, bx);
        parity ^= 1;
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = fmaf(args.a, x[s], bx[s]);
    }
    __syncthreads();  // (K = 0, in place: every wave has read the tile)
    float* const out = static_cast<float*>(d.out) + (row0 + li) * d.ld_out + col0 + 4 * lh + w;
    if (row0 + li < d.rows) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (col0 + 8 * s + 4 * lh + w < d.cols) out[8 * s] = x[s] * en.out;
    }
}

// ----------------------------------------------------------------- launch

constexpr int kMaxDevices = 64;

template <int T, int RB, Storage ST, Operand OP, bool OPT>
hipError_t launch_one(const KernelArgs& args, hipStream_t stream)
{
    constexpr int WT = (T / 32) / RB;
    constexpr int TPW = 4 / WT;
    static std::atomic<int> resident[kMaxDevices];  // workgroups that fit at once, per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    int cap = resident[dev].load(std::memory_order_relaxed);
    if (cap == 0) {
        int per_cu = 0, cus = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, ns_tiled_kernel<T, RB, ST, OP, OPT>, kThreads, 0);
        if (e != hipSuccess) return e;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        cap = (per_cu < 1 ? 1 : per_cu) * (cus < 1 ? 1 : cus);
        resident[dev].store(cap, std::memory_order_relaxed);
    }
    const int64_t n = args.tile_end - args.tile_begin;
    if (n <= 0) return hipSuccess;
    const int64_t groups = (n + TPW - 1) / TPW;
    const int grid = (int)(groups < cap ? groups : cap);
    hipLaunchKernelGGL((ns_tiled_kernel<T, RB, ST, OP, OPT>), dim3(grid), dim3(kThreads), 0, stream, args);
    return hipGetLastError();
}

// us a call, K = 5, split / one wave: 256 tiles 10.3 / 14, 512 11.5 / 14.2, 768
// 15.2 / 14.3, 1024 17.9 / 14.9: two tiles per CU hide each other's exchanges, from
// three on the one-wave tiles use the four SIMDs better.
constexpr int64_t kSplit32Tiles = 512;

// Kernel choice per tile size: rows of a T <= 64 tile stay in one wave (no
// workgroup barriers); a T = 128 tile is split over four waves.
template <Storage ST, Operand OP>
hipError_t launch_T(int T, const KernelArgs& args, hipStream_t stream)
{
    if (args.step) {
        switch (T) {
        case 32: return launch_one<32, 1, ST, OP, true>(args, stream);
        case 64: return launch_one<64, 2, ST, OP, true>(args, stream);
        case 128: return launch_one<128, 1, ST, OP, true>(args, stream);
        default: return hipErrorInvalidValue;
        }
    }
    if constexpr (OP == Operand::F32) {
        const int64_t n = args.tile_end - args.tile_begin;
        if (T == 32 && n > 0 && n <= kSplit32Tiles) {
            hipLaunchKernelGGL(ns_tiled_f32_split32_kernel, dim3((unsigned)n), dim3(kThreads), 0, stream, args);
            return hipGetLastError();
        }
    }
    switch (T) {
    case 32: return launch_one<32, 1, ST, OP, false>(args, stream);
    case 64: return launch_one<64, 2, ST, OP, false>(args, stream);
    case 128: return launch_one<128, 1, ST, OP, false>(args, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool has_kernel(int T, Storage st, Operand op)
{
    if (T == 256) return st == Storage::BF16 && op == Operand::F16;  // fp16-operand kernel only
    const bool t_ok = T == 32 || T == 64 || T == 128;
    if (!t_ok) return false;
    if (st == Storage::F32) return op == Operand::F32;
    return op == Operand::F16 || op == Operand::BF16;
}

hipError_t launch_ns_tiled(int T, Storage st, Operand op, const KernelArgs& args, hipStream_t stream)
{
    if (!has_kernel(T, st, op)) return hipErrorInvalidValue;
    if (st == Storage::F32) return launch_T<Storage::F32, Operand::F32>(T, args, stream);
    if (op == Operand::F16) return launch_ns_tiled_f16(T, args, stream);
    return launch_T<Storage::BF16, Operand::BF16>(T, args, stream);
}

}  // namespace himuon
