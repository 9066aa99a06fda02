// The three products of a Newton-Schulz step (eq. ns_iteration) on iterates
// too large for one CU, as MFMA kernels for gfx950 (16-bit operands):
//     GRAM    A  = X X^T                            (m x m, symmetric)
//     POLY    B  = alpha A A + beta A               (m x m, symmetric)
//     APPLY   X' = B X + a X                        (m x n)
// on a batch of m x n iterates (m, n multiples of 64, zero padded; in panels of
// 32 columns, each m rows of 64 contiguous bytes), fp32 accumulation, every
// result rounded once to the operand type, but for the diagonal d_i = a + B_ii:
// POLY stores it in fp32 beside a B whose diagonal is zero, and APPLY adds d_i X_i
// from the slice of X whose k are its own output rows. So neither the coefficient nor a diagonal entry
// is rounded to 16 bits (a coefficient's rounding perturbs every row alike in every
// step). Emulated, error against fp64 at K = 5, fp16 operands, with a X added in
// fp32 / a I rounded into the diagonal / as here: default coefficients on 512 x 512
// Gauss 1.34e-3 / 1.24e-3 / 0.98e-3, orthonormal rows of 15 shapes (geometric mean)
// 1.29e-3 / 1.32e-3 / 1.00e-3; (1.5, -0.5, -0.0625) on 1024 x 3000 0.52e-3 / 0.87e-3
// / 0.52e-3.
//
// GRAM and POLY compute the tiles on and above the diagonal only and store each
// of them twice, the second time transposed through LDS: 5/8 of the products at
// m = 512 with 128-tiles, 1/2 for large m. A library product computes both.
// POLY's addend beta A needs no pass over A either: the A tile of an output
// tile is one of the k slices that its product reads anyway, and is taken from
// LDS when it comes by.
//
// A workgroup owns a BM x BN tile; k advances in slices of 32 (one panel),
// staged by LDS DMA (global_load_lds_dwordx4) into a ring of NS buffers, one
// barrier per slice; in panels a slice of a tile is contiguous. The operand
// rows are permuted in 16-byte chunks by the lane's choice of source address, so
// that every ds_read_b128 of 32 rows is free of bank conflicts; the X slices of
// APPLY (k along rows) are read through ds_read_b64_tr_b16.
//
// What bounds it (one MI355X, us a launch, medians of a kernel trace; the tuned
// batched library products in brackets): m, n = 2048, 6144, three problems: GRAM 87
// (119), POLY 36 (55), APPLY 143 (153), 1.08 PFLOP/s, near what a large library
// product sustains at the board's power. 128 problems of 512 x 512: 37 (44), 39 (52),
// 48 (52): each launch moves 128 to 192 MB, at about 4 TB/s. Eight problems of
// 512 x 512: 6.4 (13), 6.7 (11), 8.1 (14): latency of one tile. Spreading the DMA and
// the LDS reads over the products, with waits that the compiler knows of, took GRAM
// at 2048 x 6144 from 93 to 84 and APPLY (then without addend) from 163 to 130; a
// ring of five or of two 64-deep slices, row-major iterates or 256-tiles changed
// nothing by 3%.
#include "elementwise8.h"
#include "ns_device.h"

#include <type_traits>

namespace himuon {
namespace {

using namespace dev;

constexpr int kBK = 32;  // k slice; columns of a panel

struct BlkArgs {
    const uint16_t* a;   // GRAM: X; POLY, APPLY: the m x m left operand
    const uint16_t* x;   // APPLY: X
    uint16_t* out;
    float* d;            // d_i = a + B_ii, m per problem: POLY writes, APPLY reads
    int64_t sa, sx, so;  // elements between problems
    int32_t m, n;        // iterate shape
    int32_t ti, tj;      // tiles per problem along i and j
    int32_t tpp;         // tiles per problem that are computed
    int32_t total;       // tiles of the launch
    float alpha, ratio;  // POLY: B = alpha (A A + ratio A)
    float diag;          // POLY: a
    // APPLY as the last step: results go to the caller's matrices (scaled by
    // inv_scale, rounded to bf16) or, with the optimizer step, into its weights
    const GemmProb* probs;
    float inv_scale;
    OptArgs opt;
};

// where APPLY's results go: the next iterate, the output matrices, the weights
enum class Dest : int { ITERATE, OUT, WEIGHTS };

HM_DEV uint32_t lds_offset(const void* p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint8_t*)(p);
}

// 64 lanes x 16 bytes from base + voff to LDS bytes dst .. dst + 1023, lane order.
// (An asm statement without outputs: the compiler would otherwise order every
// LDS read behind all DMA in flight. The waits are dma_wait_barrier's.)
HM_DEV void dma16(uint32_t dst, uint32_t voff, uint64_t base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(base)
                 : "m0", "memory");
}

// The same with 4 bytes a lane: LDS bytes dst .. dst + 255.
HM_DEV void dma4(uint32_t dst, uint32_t voff, uint64_t base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(dst), "v"(voff), "s"(base)
                 : "m0", "memory");
}

// Waits until at most N of this wave's DMA are in flight and its LDS reads
// have returned, then for the other waves. (Builtins, so that the compiler
// knows that earlier LDS reads need no further wait.)
template <int N> HM_DEV void dma_wait_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 7 << 4);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Value e of four operand values as fp32.
template <Operand OP> HM_DEV float widen(const u32x2& w, int e)
{
    const uint16_t h = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
    if constexpr (OP == Operand::F16) return (float)__builtin_bit_cast(_Float16, h);
    else return __uint_as_float((uint32_t)h << 16);
}

enum class Product : int { GRAM, POLY, APPLY };

template <Product P, Dest D, Operand OP, int BM, int BN, int WGM, int WGN, int NS, int MINW>
__global__ void __launch_bounds__(64 * WGM * WGN, MINW) block_gemm(const BlkArgs p)
{
    constexpr int W = WGM * WGN;            // waves
    constexpr int RB = BM / 32 / WGM;       // 32-row blocks per wave
    constexpr int CB = BN / 32 / WGN;       // 32-column blocks per wave
    constexpr bool SYM = P != Product::APPLY;
    static_assert(!SYM || BM == BN, "square tiles");
    constexpr int ABYTES = BM * kBK * 2, BBYTES = BN * kBK * 2;
    constexpr int STAGE = ABYTES + BBYTES;
    constexpr int AI = ABYTES / 1024 / W, BI = BBYTES / 1024 / W;  // DMA instructions per wave and slice
    constexpr int NI = AI + BI;
    static_assert(AI * 1024 * W == ABYTES && BI * 1024 * W == BBYTES, "whole DMA instructions");
    static_assert(STAGE * NS >= BM * BN * 2, "the output tile fits the ring");
    // (APPLY: the tile's d behind the ring)
    __shared__ __attribute__((aligned(1024))) uint8_t lds[STAGE * NS + (P == Product::APPLY ? BM * 4 : 0)];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int wi = (wave / WGN) * RB * 32, wj = (wave % WGN) * CB * 32;  // the wave's part of the tile

    // Workgroups go to the eight XCDs in turn; each XCD gets a contiguous run
    // of tiles, so that the tiles of a problem share one L2.
    int t;
    {
        const int b = blockIdx.x, x = b & 7, per = p.total >> 3, rem = p.total & 7;
        t = x * per + min(x, rem) + (b >> 3);
    }
    const int prob = t / p.tpp;
    int r = t - prob * p.tpp, ti = 0, tj = 0;
    if constexpr (SYM) {  // row-major over ti <= tj
        while (r >= p.ti - ti) r -= p.ti - ti, ++ti;
        tj = ti + r;
    } else {  // bands of four tile rows, column by column
        const int band = r / (4 * p.tj), h = min(4, p.ti - 4 * band);
        r -= band * 4 * p.tj;
        tj = r / h;
        ti = 4 * band + (r - tj * h);
    }
    const int i0 = ti * BM, j0 = tj * BN;
    const int kdim = P == Product::GRAM ? p.n : p.m;   // contraction length; row length of `a`
    const int nk = kdim / kBK;
    const uint16_t* const a = p.a + prob * p.sa;

    // DMA sources. Instruction q of a wave fills operand rows 16 (q W + wave) ..
    // + 15, lane l row l / 4 and the 16-byte chunk that sits at position l % 4
    // of the row, (l % 4) ^ ((row >> 2) & 3). Rows past the matrix read its last
    // row (their results are not stored).
    uint32_t va[AI], vb[BI];
    const int64_t panel = (int64_t)p.m * kBK;
    const uint16_t* a_base = a + (int64_t)i0 * kBK;
    const uint16_t* b_base;
#pragma unroll
    for (int q = 0; q < AI; ++q) {
        const int row = 16 * (q * W + wave) + (lane >> 2);
        va[q] = (uint32_t)min(row, p.m - 1 - i0) * (kBK * 2u) + 16u * ((lane & 3) ^ ((row >> 2) & 3));
    }
    int64_t b_step;
    if constexpr (SYM) {
        b_base = a + (int64_t)j0 * kBK;
        b_step = panel;
#pragma unroll
        for (int q = 0; q < BI; ++q) {
            const int row = 16 * (q * W + wave) + (lane >> 2);
            vb[q] = (uint32_t)min(row, p.m - 1 - j0) * (kBK * 2u) + 16u * ((lane & 3) ^ ((row >> 2) & 3));
        }
    } else {
        // X slice: 32 rows (k) of BN columns, panel by panel, chunks permuted like A's
        b_base = p.x + prob * p.sx + (int64_t)(j0 / kBK) * panel;
        b_step = kBK * kBK;
#pragma unroll
        for (int q = 0; q < BI; ++q) {
            const int u = q * W + wave;  // half a panel's slice
            const int pan = min(u >> 1, p.n / kBK - 1 - j0 / kBK);
            vb[q] = (uint32_t)pan * (uint32_t)(panel * 2) + 1024u * (u & 1) + 64u * (lane >> 2) +
                    16u * ((lane & 3) ^ (lane >> 4));
        }
    }
    const uint32_t lds0 = lds_offset(lds);
    auto uniform = [](const void* q) -> uint64_t {
        const uint64_t v = (uint64_t)(uintptr_t)q;
        return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
    };
    // DMA instruction q of the next slice, into ring buffer `buf`
    auto issue1 = [&](int buf, int q) {
        const uint32_t d = __builtin_amdgcn_readfirstlane(lds0 + buf * STAGE + wave * 1024);
        if (q < AI) dma16(d + q * W * 1024, va[q < AI ? q : 0], uniform(a_base));
        else dma16(d + ABYTES + (q - AI) * W * 1024, vb[q < AI ? 0 : q - AI], uniform(b_base));
    };
    auto advance = [&]() {
        a_base += panel;
        b_base += b_step;
    };

    f32x16 acc[RB][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = f32x16{};

    // lane offsets of the operand reads
    const int rsw = (li >> 2) & 3;
    int ra[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) ra[s] = li * 64 + 16 * ((2 * s + lh) ^ rsw);
    // APPLY: transposing reads, k half x (rows 4x ..), whose chunks are permuted by 2 (g16 / 2) + x
    const int g16 = lane >> 4;
    int rx[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
        rx[x] = (8 * (g16 >> 1) + 4 * x + ((lane & 15) >> 2)) * 64 +
                16 * ((2 * (g16 & 1) + ((lane & 3) >> 1)) ^ (2 * (g16 >> 1) + x)) + 8 * (lane & 1);

    // Operand fragments of 16 k are read one step ahead of their products; the
    // first step of a slice is read during the last of the one before, behind
    // the barrier that also frees the older slice's buffer. One LDS read (or
    // two transposing ones) goes out before each product, and the DMA of the
    // slice that refills that buffer is spread over the products too: issued
    // together it fills the memory pipe's queue and holds the wave.
    u32x4 fa[2][RB], fb[2][CB];
    constexpr int READS = RB + CB, PROD = RB * CB;
    auto load1 = [&](const uint8_t* ta, int s, int h, int r) {
        const uint8_t* const tb = ta + ABYTES;
        if (r < RB) {
            const int i = r < RB ? r : 0;
            fa[h][i] = *reinterpret_cast<const u32x4*>(ta + (wi + 32 * i) * 64 + ra[s]);
        } else {
            const int j = r < RB ? 0 : r - RB;
            if constexpr (SYM) {
                fb[h][j] = *reinterpret_cast<const u32x4*>(tb + (wj + 32 * j) * 64 + ra[s]);
            } else {
                const uint8_t* const tx = tb + (wj / 32 + j) * 2048 + 1024 * s;
                const u32x2 lo = tr_read(tx + rx[0]);
                const u32x2 hi = tr_read(tx + rx[1]);
                fb[h][j] = u32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        }
    };
    constexpr int RPP = (READS + PROD - 1) / PROD;                           // reads per product
    constexpr int DPP = (NI + PROD - 1) / PROD, DEV = PROD / ((NI + DPP - 1) / DPP);  // DPP DMA every DEV products
    // the products of fragment set h beside the reads of step s of slice `ta`
    // into the other set (read) and the DMA into buffer `dst` (refill)
    auto phase = [&](int h, const uint8_t* ta, int s, auto read, auto refill, int dst) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < PROD; ++e) {
            if constexpr (decltype(read)::value) {
#pragma unroll
                for (int r = e * RPP; r < (e + 1) * RPP; ++r)
                    if (r < READS) load1(ta, s, h ^ 1, r);
            }
            acc[e / CB][e % CB] = mma1<OP>(fb[h][e % CB], fa[h][e / CB], acc[e / CB][e % CB]);
            if constexpr (decltype(refill)::value) {
                if (e % DEV == DEV - 1) {
#pragma unroll
                    for (int q = e / DEV * DPP; q < (e / DEV + 1) * DPP; ++q)
                        if (q < NI) issue1(dst, q);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (decltype(refill)::value) advance();
    };
    // v += f M for a 32 x 32 block M whose rows of 64 bytes lie at `tm`, chunks
    // permuted like the operands'
    auto add_block = [&](const uint8_t* tm, float f, f32x16& v) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const u32x2 w = *reinterpret_cast<const u32x2*>(tm + li * 64 + 16 * (g ^ rsw) + 8 * lh);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * g + e] = fmaf(f, widen<OP>(w, e), v[4 * g + e]);
        }
    };
    // POLY: the slice whose k are the wave's output columns holds its part of A
    auto addend = [&](const uint8_t* ta, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            if ((j0 + wj) / kBK + j == k) {
#pragma unroll
                for (int i = 0; i < RB; ++i) add_block(ta + (wi + 32 * i) * 64, p.ratio, acc[i][j]);
            }
        }
    };

    if constexpr (P == Product::APPLY) {  // (ahead of the slices: whoever waits for slice 0 waits for it too)
        if (wave < BM / 64)
            dma4(__builtin_amdgcn_readfirstlane(lds0 + STAGE * NS + wave * 256),
                 4u * (uint32_t)min(64 * wave + lane, p.m - 1 - i0), uniform(p.d + (int64_t)prob * p.m + i0));
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s < nk) {
#pragma unroll
            for (int q = 0; q < NI; ++q) issue1(s, q);
            advance();
        }
    }
    if (nk >= NS) dma_wait_barrier<(NS - 1) * NI>();
    else dma_wait_barrier<0>();
#pragma unroll
    for (int r = 0; r < READS; ++r) load1(lds, 0, 0, r);
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    int buf = 0, k = 0;
    auto slice = [&](auto more, auto refill) __attribute__((always_inline)) {
        const uint8_t* const ta = lds + buf * STAGE;
        const int nbuf = buf + 1 == NS ? 0 : buf + 1;
        phase(0, ta, 1, yes, no, 0);
        if constexpr (P == Product::POLY) addend(ta, k);
        if constexpr (decltype(more)::value) {
            // slice k + 1 has landed; every wave has read slice k
            dma_wait_barrier<decltype(refill)::value ? (NS - 2) * NI : 0>();
        }
        phase(1, lds + nbuf * STAGE, 0, more, refill, buf);
        buf = nbuf;
    };
    auto run_to = [&](int end) __attribute__((always_inline)) {
        for (const int e = min(end, nk - NS); k < e; ++k) slice(yes, yes);
        for (const int e = min(end, nk - 1); k < e; ++k) slice(yes, no);
        if (k < end) {
            slice(no, no);
            ++k;
        }
    };
    if constexpr (P == Product::APPLY) {
        // The slices whose k are the wave's output rows hold its part of X. The loops
        // stop ahead of each of them instead of asking in every slice (APPLY on eight
        // problems of 512 x 512 7.9 us asking, 7.7 so, 7.0 without the addend; on three of
        // 2048 x 6144 142 and 139 so and without it).
        const int r0 = (i0 + wi) / kBK;
#pragma unroll 1
        for (int b = 0; b <= RB; ++b) {
            run_to(b < RB ? min(r0 + b, nk) : nk);
#pragma unroll
            for (int i = 0; i < RB; ++i)
                if (b == i) {
                    const float d = *reinterpret_cast<const float*>(lds + STAGE * NS + (wi + 32 * i + li) * 4);
#pragma unroll
                    for (int j = 0; j < CB; ++j)
                        add_block(lds + buf * STAGE + ABYTES + (wj / 32 + j) * 2048, d, acc[i][j]);
                }
        }
    } else {
        run_to(nk);
    }

    // results in the operand type into LDS: rows of BN, 16-byte chunk c of row r at c ^ (r & 7)
    dma_wait_barrier<0>();
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            if constexpr (P == Product::POLY) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] *= p.alpha;
                if (i0 == j0 && wi + 32 * i == wj + 32 * j) {
                    const int row = i0 + wi + 32 * i + li;
                    float d = 0.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const bool on = 8 * (v >> 2) + 4 * lh + (v & 3) == li;
                        d = on ? acc[i][j][v] : d;
                        acc[i][j][v] = on ? 0.f : acc[i][j][v];
                    }
                    if (((li >> 2) & 1) == lh && row < p.m) p.d[(int64_t)prob * p.m + row] = d + p.diag;
                }
            }
            const int row = wi + 32 * i + li;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = (wj + 32 * j) / 8 + g;
                *reinterpret_cast<u32x2*>(lds + row * (BN * 2) + 16 * (c ^ (row & 7)) + 8 * lh) =
                    u32x2{pack2<OP>(acc[i][j][4 * g], acc[i][j][4 * g + 1]),
                          pack2<OP>(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3])};
            }
        }
    // the lane's eight rows ib + 8 (lane / 16) .. of column jb + lane % 16
    auto transposed8 = [&](int jb, int ib) -> u32x4 {
        u32x2 h[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int row = ib + 8 * g16 + 4 * x + ((lane & 15) >> 2);
            const int c8 = jb / 4 + (lane & 3);
            h[x] = tr_read(lds + row * (BN * 2) + 16 * ((c8 >> 1) ^ (row & 7)) + 8 * (c8 & 1));
        }
        return u32x4{h[0][0], h[0][1], h[1][0], h[1][1]};
    };
    if constexpr (D != Dest::ITERATE) {
        // Eight consecutive elements of a row of the problem's block at a time,
        // inside the block only. The values are those that the next iterate would
        // hold, so the result does not depend on who scatters it. The weights are
        // asked for before the tile is exchanged. On 128 problems of 512 x 512 the
        // launch takes 89 us (49 into the iterate, and 34 for a scatter pass); on
        // three of 2048 x 6144 174 (138 and 71).
        const GemmProb Q = p.probs[prob];  // (a copy: through a reference every store reloads its fields)
        constexpr int E = BM * BN / 8 / (64 * W);  // chunks per thread
        constexpr int CPR = BN / 8;
        const bool trans = Q.trans != 0;
        auto place = [&](int e, int& r, int& c) {
            if (!trans) {
                const int x = (int)threadIdx.x + 64 * W * e;
                r = i0 + x / CPR;
                c = j0 + 8 * (x % CPR);
            } else {
                const int u = wave + W * e;
                r = j0 + 16 * (u / (BM / 32)) + (lane & 15);
                c = i0 + 32 * (u % (BM / 32)) + 8 * g16;
            }
        };
        auto whole = [&](int r, int c) { return r < Q.h && c + 8 <= Q.w && (Q.vec & GEMM_VEC_OUT) != 0; };
        u32x4 old[D == Dest::WEIGHTS ? E : 1];
        if constexpr (D == Dest::WEIGHTS) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                int r, c;
                place(e, r, c);
                old[e] = u32x4{};
                if (whole(r, c))
                    old[e] = *(const gbl_u32x4*)(static_cast<const uint16_t*>(Q.out) + (Q.row0 + r) * Q.ld_out + Q.col0 + c);
            }
        }
        __syncthreads();
        const float step = D == Dest::WEIGHTS ? p.opt.lr * Q.tau : 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            int r, c;
            place(e, r, c);
            u32x4 w;
            if (!trans) {
                const int row = r - i0, ch = (c - j0) / 8;
                w = *reinterpret_cast<const u32x4*>(lds + row * (BN * 2) + 16 * (ch ^ (row & 7)));
            } else {
                w = transposed8(r - j0 - (lane & 15), c - i0 - 8 * g16);
            }
            if (r >= Q.h || c >= Q.w) continue;
            float u[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const uint16_t h = (uint16_t)(w[x >> 1] >> (16 * (x & 1)));
                if constexpr (OP == Operand::F16) u[x] = (float)__builtin_bit_cast(_Float16, h) * p.inv_scale;
                else u[x] = __uint_as_float((uint32_t)h << 16) * p.inv_scale;
            }
            const bool vec = whole(r, c);
            const int nv = min(8, Q.w - c);
            const int64_t idx = (Q.row0 + r) * Q.ld_out + Q.col0 + c;
            if constexpr (D == Dest::WEIGHTS) {
                float v[8];
                if (vec) {
#pragma unroll
                    for (int x = 0; x < 8; ++x)
                        v[x] = __uint_as_float((x & 1) ? (old[e][x >> 1] & 0xffff0000u) : (old[e][x >> 1] << 16));
                } else {
                    load8<GemmStore::BF16>(Q.out, idx, nv, false, v);
                }
#pragma unroll
                for (int x = 0; x < 8; ++x) u[x] = p.opt.decay * v[x] - step * u[x];
            }
            store8<GemmStore::BF16>(Q.out, idx, nv, vec, u);
        }
        return;
    }
    __syncthreads();
    const int ncols = SYM ? p.m : p.n;
    uint16_t* const out = p.out + prob * p.so;
    constexpr int CPR = BN / 8;
#pragma unroll 4
    for (int e = threadIdx.x; e < BM * CPR; e += 64 * W) {  // panel by panel
        const int row = (e / 4) % BM, c = e % 4 + 4 * (e / (4 * BM));
        const u32x4 v = *reinterpret_cast<const u32x4*>(lds + row * (BN * 2) + 16 * (c ^ (row & 7)));
        if (i0 + row < p.m && j0 + 8 * c < ncols && (!SYM || ti != tj || row / 32 <= c / 4))
            *reinterpret_cast<u32x4*>(out + (j0 / kBK + c / 4) * panel + (i0 + row) * kBK + 8 * (c % 4)) = v;
    }
    if constexpr (SYM) {
        // the transposed tile (of a diagonal tile, the 32-blocks above its
        // diagonal: what lies below it in memory is their mirror image, whatever
        // the tile size): a wave moves 16 columns x 32 rows at a time, 16 whole
        // output rows of a panel
        constexpr int UNITS = (BN / 16) * (BM / 32);
#pragma unroll 4
        for (int u = wave; u < UNITS; u += W) {
            const int jb = 16 * (u / (BM / 32)), ib = 32 * (u % (BM / 32));
            if (ti == tj && jb / 32 <= ib / 32) continue;
            const u32x4 v = transposed8(jb, ib);
            const int orow = j0 + jb + (lane & 15), ocol = i0 + ib + 8 * g16;
            if (orow < p.m && ocol < p.m)
                *reinterpret_cast<u32x4*>(out + (ocol / kBK) * panel + orow * kBK + ocol % kBK) = v;
        }
    }
}

template <Product P, Dest D, Operand OP, int BM, int BN, int WGM, int WGN, int NS, int MINW>
hipError_t launch_cfg(BlkArgs p, int batch, hipStream_t stream)
{
    p.ti = (p.m + BM - 1) / BM;
    p.tj = P == Product::APPLY ? (p.n + BN - 1) / BN : p.ti;
    p.tpp = P == Product::APPLY ? p.ti * p.tj : p.ti * (p.ti + 1) / 2;
    const int64_t total = (int64_t)p.tpp * batch;
    if (total <= 0 || total > INT32_MAX) return hipErrorInvalidValue;
    p.total = (int)total;
    hipLaunchKernelGGL((block_gemm<P, D, OP, BM, BN, WGM, WGN, NS, MINW>), dim3((unsigned)total), dim3(64 * WGM * WGN), 0,
                       stream, p);
    return hipGetLastError();
}

int64_t tiles_of(Product P, int m, int n, int batch, int bi, int bj)
{
    const int64_t ti = (m + bi - 1) / bi, tj = (n + bj - 1) / bj;
    return batch * (P == Product::APPLY ? ti * tj : ti * (ti + 1) / 2);
}

// The largest tile that still gives the 256 CUs enough workgroups. Measured
// (us, one MI355X; 128-tiles against 64-tiles, by the number of 128-tiles):
// GRAM 80: 7.0 / 5.6, 144: 11.0 / 14.7, 272: 28 / 39, 1280: 37 / 50; APPLY
// 64: 10.2 / 7.8, 128: 6.4 / 6.8, 256: 7.3 / 10.8, 2048: 47 / 81: the line is
// at 128 tiles. 128 x 256 tiles of APPLY against 128-tiles, 256 and more of
// them: m = 512 50 / 47, m = 2048 138 / 143 and 118 / 127, m = 4096 112 / 122:
// they pay where k is long. 256 x 256 tiles won nowhere by more than 3%.
template <Product P, Dest D, Operand OP> hipError_t launch_product(const BlkArgs& p, int batch, hipStream_t stream)
{
    if constexpr (P == Product::APPLY) {
        if (p.m >= 1024 && tiles_of(P, p.m, p.n, batch, 128, 256) >= 256)
            return launch_cfg<P, D, OP, 128, 256, 2, 2, 3, 2>(p, batch, stream);
    }
    // (a ring of three, 48 KB, lets three workgroups share a CU; against a ring of
    // four and two of them, steps at T = 512: 8 x 2048^2 644 us / 679, 8 x 4096^2
    // 2718 / 2799, both repeated on the same gradients)
    if (tiles_of(P, p.m, p.n, batch, 128, 128) >= 128) return launch_cfg<P, D, OP, 128, 128, 2, 2, 3, 3>(p, batch, stream);
    return launch_cfg<P, D, OP, 64, 64, 2, 2, 8, 2>(p, batch, stream);
}

template <Product P, Dest D = Dest::ITERATE> hipError_t launch_op(GemmOperand op, const BlkArgs& p, int batch, hipStream_t stream)
{
    if (op == GemmOperand::F16) return launch_product<P, D, Operand::F16>(p, batch, stream);
    if (op == GemmOperand::BF16) return launch_product<P, D, Operand::BF16>(p, batch, stream);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_block_step(GemmOperand op, int m, int n, int batch, float alpha, float beta, float diag,
                             const void* x, void* A, void* B, float* d, void* x_out, const GemmProb* probs, float inv_scale,
                             const OptArgs* opt, hipStream_t stream)
{
    if (m < 64 || n < 64 || m % 64 || n % 64) return hipErrorInvalidValue;
    const int64_t mn = (int64_t)m * n, mm = (int64_t)m * m;
    BlkArgs p{};
    p.m = m;
    p.n = n;
    p.a = static_cast<const uint16_t*>(x);
    p.sa = mn;
    p.out = static_cast<uint16_t*>(A);
    p.so = mm;
    hipError_t e = launch_op<Product::GRAM>(op, p, batch, stream);
    if (e != hipSuccess) return e;
    p.a = static_cast<const uint16_t*>(A);
    p.sa = mm;
    p.out = static_cast<uint16_t*>(B);
    p.alpha = alpha;
    p.ratio = beta / alpha;
    p.diag = diag;
    p.d = d;
    e = launch_op<Product::POLY>(op, p, batch, stream);
    if (e != hipSuccess) return e;
    p.a = static_cast<const uint16_t*>(B);
    p.x = static_cast<const uint16_t*>(x);
    p.sx = mn;
    p.out = static_cast<uint16_t*>(x_out);
    p.so = mn;
    if (!probs) return launch_op<Product::APPLY>(op, p, batch, stream);
    p.probs = probs;
    p.inv_scale = inv_scale;
    if (!opt) return launch_op<Product::APPLY, Dest::OUT>(op, p, batch, stream);
    p.opt = *opt;
    return launch_op<Product::APPLY, Dest::WEIGHTS>(op, p, batch, stream);
}

}  // namespace himuon
