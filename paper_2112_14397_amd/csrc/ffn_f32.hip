// Expert FFNs of a float32 layer (EvoMoE Eq. ffn per expert over its ragged row range, and its backward) on the bf16 matrix
// cores, at float32 accuracy:
//
//   NT  C[r,n] = sum_k A[arow(r),k] * W_g[n,k]          forward GEMMs (A rows optionally gathered by token)
//   NN  C[r,n] = sum_k A[r,k]       * W_g[k,n]          dH = dO W2,  dXp = dH W1
//   TN  C_g[m,n] = sum_{r in g} L[r,m] * R[rrow(r),n]   weight gradients (contraction over the ragged rows)
//
// Every float32 value is taken apart into three bf16 values whose sum it is (of very small ones almost: below), and a product
// a * b into the six largest of the nine products of their terms: bf16 MFMAs run at sixteen times the rate of float32 ones, so
// six of them take 0.38 of the time.  Left out are mid * lo and lo * mid, up to 2^-23 of the product each (the first term is cut off,
// so the second is up to 2^-7 of the value, the third 2^-16), and lo * lo.  A single product is therefore less exact than in
// float32, a sum more, as below; contractions of up to 16 k's take mid * lo and lo * mid too.  Relative rms error by the number
// of products (N(0,1) operands; float32 chains of eight / six products / eight): 1 2.5e-8 / 3.4e-8 / 2.5e-8, 2 3.1e-8 / 3.4e-8 /
// 2.6e-8, 3 3.6e-8 / 3.5e-8 / 2.6e-8, 16 6.0e-8 / 3.8e-8 / 3.1e-8, 17 6.4e-8 / 4.6e-8 / 4.0e-8.  The products are exact and each
// of four partial sums per output has one rounding per 16 k's (the small products have a sum of their own), where float32 MFMAs
// round for every k: relative rms error against float64 at 5632 pairs, d = 256, E = 8, F = 1024 (float32 MFMAs / here; smaller
// at every size measured, 64 to 2048 k's): H 1.5e-7 / 7.2e-8, O 2.9e-7 / 1.0e-7, dH 1.6e-7 / 8.2e-8, dXp 2.9e-7 / 1.1e-7, dW
// 2.4e-7 / 9.7e-8.  With one sum for all six products the contractions of 64 k's had larger errors than float32 MFMAs (H 9.5e-8
// against 8.8e-8).
//
// Range: the terms of values below 2^-110 (7.7e-34) reach below the smallest bf16 subnormal, 2^-133, which the matrix cores do take:
// each such value is off by up to 2^-134, that is by 2^-24 of itself at 2^-110 and by 2^-8 at the smallest normal float32 value
// (relative rms error of H with all x between 2^-112 and 2^-111, -116 and -115, -122 and -121: 1.1e-7, 1.4e-6, 9.3e-5; float32
// MFMAs 8.5e-8).  In a sum with larger products that is nothing; where whole tensors are that small, scale the loss.  Between there and
// the largest float32 value everything is as above, infinities and NaNs give what float32 products give.
//
// What bounds it: a 64x64 tile's slab of 64 k's takes 768 clocks of the matrix pipes, about as many of the VALU for taking the
// operands apart, and 32 KB from the L2; two blocks per CU overlap these in part.  The operands go to the LDS as they are, by
// asynchronous loads, one slab ahead.  A wave has 16 of a slab's k's for the whole tile: what it takes apart no other wave
// needs.  (The terms in the LDS, each taken apart by one thread: six bytes per value instead of four, two barriers per slab
// and the loads through registers: 244 us instead of 217 for the step below.)  us, float32 MFMAs / here, GEMM1, GEMM2, dH,
// dXp, both dW, whole training step: 5632 pairs, d = 256, E = 8, F = 1024: 40 / 35, 40 / 29, 45 / 36, 41 / 32, 68 / 50, 269 /
// 219; 8700 pairs, d = 512, E = 16, F = 2048: 208 / 160, 203 / 133, 233 / 167, 218 / 146, 418 / 312, 1302 / 983.
// The bias gradients' column sums are further tiles behind dXp's and behind the weight gradients': colsum_tile().
//
// Tiles: 64x64, and 32x32 for launches that would leave most of the chip idle; cheapest() says which and why.  Both add the
// products of one output in the same order, so that results do not depend on the pair count announced, nor on how many rows
// a call has.
#include "ffn_internal.h"

namespace evomoe {

namespace {

enum { L_NT = 0, L_NN = 1, L_TN = 2 };
enum { E_HA = 0, E_BIAS = 1, E_ACTGRAD = 2, E_NONE = 3, E_WGRAD = 4 };

struct F32Args {
    const float* A;  int lda;           // NT/NN: A rows [*,K];  TN: L [P,M]
    const float* B;  int ldb;           // NT: W_g [N,K];  NN: W_g [K,N];  TN: R [*,N]
    int64_t b_group_stride;             // NT/NN: elements between two experts' weight matrices
    const int32_t* rows;                // NT: gather of A rows; TN: gather of R rows (or null)
    int M, N, K;                        // M: TN only.  K: NT/NN only
    const float* bias;                  // [E,N] or null
    const float* Hin;                   // E_ACTGRAD: pre-activations [P,N]
    float* out1;                        // C (H for E_HA)
    float* out2;                        // E_HA: act(H)
};

struct F32Pair { F32Args p[2]; };       // TN: two problems in one launch; NT/NN use the first

// Where a tile lies: expert, first row (NT/NN) or contraction range (TN).
// NT/NN row tiles are numbered expert by expert; lane e knows expert e's share, so the search is one scan over the
// lanes and one ballot, without LDS.
struct Offsets {
    int begin, count;                   // of the lane's expert
    int t_end, t_begin;                 // its row tiles [t_begin, t_end)
};
// Column sums of dO and dH over every expert's rows (the bias gradients).  The dXp launch leaves part[split][expert][column]
// of both matrices, the weight-gradient launch adds the splits in order.
// An expert of n rows is cut into ceil(n / 64) ranges, kSumSplit at most: a block's loads for one of 64 rows go out together.
// Sums inside the weight-gradient tiles, whose left operand the matrices are, cost no extra pass, but there every row of an
// expert passes through one block: a backward with the bias gradients alone took 220 us at d = 64, E = 1, F = 256, 16384
// pairs (now 41, without them 34), and chains of 4096 additions had eight times the error (1.1e-6 relative rms; now 1.3e-7).
constexpr int kSumSplit = kF32ColsumSplit, kSumCols = 128;
struct F32Sums {
    const float* m[2];                  // dO [P,N0], dH [P,N1]
    int N[2], blocks[2];                // columns; column blocks (0: not wanted)
    float* part[2];                     // [kSumSplit][E][N]
    float* db[2];                       // [E,N]
};
__device__ __forceinline__ int sum_splits(int rows) { return max(1, min(kSumSplit, (rows + 63) / 64)); }

// Tile b of the first pass: (split, expert, column block).
__device__ __forceinline__ void colsum_tile(const F32Sums& q, int b, const Offsets& off, int E, float* red) {
    const int nb = q.blocks[0] + q.blocks[1];
    const int g = b / nb % E, split = b / nb / E, i = b % nb >= q.blocks[0];
    const int begin = __builtin_amdgcn_readlane(off.begin, g), count = __builtin_amdgcn_readlane(off.count, g);
    const int splits = sum_splits(count);
    if (split >= splits) return;                                  // block-uniform
    const int N = q.N[i], n0 = (b % nb - (i ? q.blocks[0] : 0)) * kSumCols;
    const int CL = min(kSumCols, N) / 4, RL = min(32, 256 / CL);  // column lanes (16 bytes each), row lanes
    const int cl = threadIdx.x % CL, rl = threadIdx.x / CL, n = n0 + cl * 4;
    const int per = (count + splits - 1) / splits, rb = begin + split * per, re = min(begin + count, rb + per);
    const bool on = rl < RL && n < N;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    if (on) {
        const float* src = q.m[i] + n;
        for (int r = rb + rl; r < re; r += 8 * RL) {
            f32x4 v[8], t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4*>(src + (int64_t)min(r + u * RL, re - 1) * N);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (r + u * RL < re) t += v[u];
            sum += t;
        }
        *reinterpret_cast<f32x4*>(red + (rl * CL + cl) * 4) = sum;
    }
    __syncthreads();
    if (rl == 0 && n < N) {
        sum = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int l = 0; l < RL; ++l) sum += *reinterpret_cast<const f32x4*>(red + (l * CL + cl) * 4);
        *reinterpret_cast<f32x4*>(q.part[i] + ((int64_t)split * E + g) * N + n) = sum;
    }
    __syncthreads();
}
// Second pass: column i of both matrices' E * N.
__device__ __forceinline__ void colsum_final(const F32Sums& q, int64_t i, const int32_t* expert_offsets, int E, int64_t P_cap,
                                             int accumulate) {
    const int64_t n0 = q.blocks[0] ? (int64_t)E * q.N[0] : 0;
    const int k = i >= n0;
    const int64_t j = k ? i - n0 : i, stride = (int64_t)E * q.N[k];
    const int g = (int)(j / q.N[k]);
    const int splits = sum_splits(clamp_pairs(expert_offsets[g + 1], P_cap) - clamp_pairs(expert_offsets[g], P_cap));
    float v[kSumSplit], s = 0.f;
    const float old = accumulate ? q.db[k][j] : 0.f;
#pragma unroll
    for (int u = 0; u < kSumSplit; ++u) v[u] = q.part[k][(int64_t)min(u, splits - 1) * stride + j];
#pragma unroll
    for (int u = 0; u < kSumSplit; ++u)
        if (u < splits) s += v[u];
    q.db[k][j] = accumulate ? old + s : s;
}

template <int BM> __device__ __forceinline__ Offsets scan_offsets(const int32_t* expert_offsets, int E, int64_t P_cap, int lane) {
    Offsets o;
    o.begin = lane < E ? clamp_pairs(expert_offsets[lane], P_cap) : 0;
    o.count = lane < E ? clamp_pairs(expert_offsets[lane + 1], P_cap) - o.begin : 0;
    const int nt = (o.count + BM - 1) / BM;
    int incl = nt;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const int v = __shfl_up(incl, s, 64);
        if (lane >= s) incl += v;
    }
    o.t_end = incl;
    o.t_begin = incl - nt;
    return o;
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
// The three bf16 terms of eight float32 values: hi (cut off, so that no finite value becomes infinite) + mid (rounded) + lo
// (what is left, eight bits at most) is the value itself, from 2^-110 on (above).  An infinity or a NaN gives NaN terms behind itself,
// a NaN with a payload in its low half only (a signalling one) an infinity as its first.
__device__ __forceinline__ void split8(const float* v, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
    u32x4 h, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b0 = __float_as_uint(v[2 * i]), b1 = __float_as_uint(v[2 * i + 1]);
        const float r0 = v[2 * i] - __uint_as_float(b0 & 0xffff0000u), r1 = v[2 * i + 1] - __uint_as_float(b1 & 0xffff0000u);
        h[i] = __builtin_amdgcn_perm(b1, b0, 0x07060302);
        asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(m[i]) : "v"(r0), "v"(r1));      // (seen through, it would be made twice)
        l[i] = pack_bf16x2(r0 - lo_bf16(m[i]), r1 - hi_bf16(m[i]));
    }
    hi = __builtin_bit_cast(bf16x8, h);
    mid = __builtin_bit_cast(bf16x8, m);
    lo = __builtin_bit_cast(bf16x8, l);
}

// 16 bytes per lane, global -> LDS: lane l's data lands at lds + 16 l.  Inline assembly, so that the compiler does not guard
// every LDS read of the other stage with a wait for it; the kernel waits itself.
__device__ __forceinline__ void load_to_lds(const float* from, const unsigned char* lds_wave_base) {
    const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)lds_wave_base;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(from), "s"(at) : "m0", "memory");
}
// For every wave of the block: its loads have landed, and it is done with the LDS it was reading.  The wait is the builtin: the
// compiler, which counts its own loads, would wait again later, for the next slab's too, if it did not know of it.
__device__ __forceinline__ void all_landed() {
    __builtin_amdgcn_s_waitcnt(0x0070);     // vmcnt(0) lgkmcnt(0)
    asm volatile("s_barrier" ::: "memory");
}

// Weight gradients: an expert of at most so many rows is not worked in 64x64 tiles that go through the LDS, where the start and the end
// of a tile are most of its time with the two blocks that fit a CU, but by single waves (below), where that makes work for half of
// the waves.  us, float32 MFMAs / tiles / here: E = 64, d = 196, F = 880, 33 pairs 41 / 67 / 31; d = 280, F = 768, 1231 pairs 54 / 79 /
// 44, 2500 70 / 77 / 57 (5000, experts of 78 rows, 93 / 104 / 105); E = 16, d = 512, F = 2048, 200 pairs 58 / 79 / 37; E = 16, d = 256,
// F = 512, 60 pairs 14 / 19 / 12, 600 17 / 18 / 17; E = 4, d = 456, F = 1096, 64 pairs 19 / 20 / 22; E = 1, d = 512, F = 2048, 10 pairs 10 /
// 12 / 12.  E = 16, d = 228, F = 464, where a third of the experts have so few of 1021 pairs, 16 / 17 / 20.  With a line at 64 rows the
// experts of 78 rows took 109.
constexpr int kFewRows = 48;
// Blocks per CU, for the registers, the LDS and the grid.
template <int B> constexpr int blocks_per_cu() { return B == 64 ? 2 : 4; }

template <int LAYOUT, int EPI, int BM, int BN>
__global__ __launch_bounds__(256, (blocks_per_cu<BM>())) void grouped_gemm_f32(
    F32Pair q, int tiles0, int tiles_all, F32Sums sums, const int32_t* __restrict__ expert_offsets, int E, int64_t P_cap,
    int act, int accumulate)
{
    constexpr int B = BM, BK = 64;                      // wave w takes the 16 k's from 16 w on of every slab, for the whole tile
    static_assert(BM == BN && (B == 32 || B == 64), "tile");
    constexpr bool A_KC = LAYOUT != L_TN, B_KC = LAYOUT == L_NT;
    constexpr int TM = B / 32;                          // 32x32 pieces along a side of the tile
    constexpr int OPERAND = B * BK * 4, STAGE = 2 * OPERAND;
    constexpr int NI = OPERAND / 4096;                  // 1 KB load instructions per wave, operand and slab
    // An operand whose contraction index is contiguous in memory lies as [row][64 k], its 16-byte chunk c at c ^ (row & 15):
    // sixteen rows that read the same chunk cover all 64 banks.  One whose contraction index is the row index lies as
    // [k][columns]; 32 lanes read 32 columns of a row, or 64 in pairs: then piece i of the tile has the columns 2 l + i.
    constexpr bool A_PAIR = !A_KC && TM == 2, B_PAIR = !B_KC && TM == 2;
    __shared__ __align__(16) unsigned char smem[2 * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kg = lane >> 5;

    const Offsets off = scan_offsets<BM>(expert_offsets, E, P_cap, lane);
    const int row_tiles = __builtin_amdgcn_readlane(off.t_end, 63);

    // Consecutive tiles share operand panels, and blocks are dealt round-robin to the 8 XCDs: each XCD walks one
    // contiguous eighth of the tiles, so that its L2 sees the panels and no XCD gets a round more than another.
    // TN: the tiles are those of the experts with more than kFewRows rows; lane e knows expert e's place among them, or among the others
    const int wanted0 = tiles0 / E, wanted1 = tiles_all / E - wanted0;      // TN: an expert's tiles of either problem
    const int units0 = wanted0 ? ((q.p[0].M + 31) / 32) * ((q.p[0].N + BN - 1) / BN) : 0,      // TN: what few rows are worked in
              units1 = wanted1 ? ((q.p[1].M + 31) / 32) * ((q.p[1].N + BN - 1) / BN) : 0;
    uint64_t few = LAYOUT == L_TN && TM == 2 ? __ballot(lane < E && off.count <= kFewRows) : 0;
    if (__popcll(few) * (units0 + units1) < 2 * (int)gridDim.x) few = 0;
    const bool mine_few = few >> lane & 1;
    const uint64_t many = __ballot(lane < E && !mine_few);
    const int place = __popcll((mine_few ? few : many) & (((uint64_t)1 << lane) - 1));
    if (LAYOUT == L_TN) tiles0 = wanted0 * __popcll(many);
    const int total = LAYOUT == L_TN ? tiles0 + wanted1 * __popcll(many) : row_tiles * ((q.p[0].N + BN - 1) / BN);
    int tile = blockIdx.x, tile_end = total, step = gridDim.x;
    if ((gridDim.x & 7) == 0) {
        const int x = blockIdx.x & 7;
        tile = (int)((int64_t)total * x / 8) + (blockIdx.x >> 3);
        tile_end = (int)((int64_t)total * (x + 1) / 8);
        step = gridDim.x >> 3;
    }
    struct Tile { int second, g, row0, rows, m0, n0, kbeg, kend; };
    auto locate = [&](int tile) {
        Tile t{};
        t.second = LAYOUT == L_TN && tile >= tiles0;
        const F32Args& p = q.p[t.second];
        const int nct = (p.N + BN - 1) / BN;
        if (LAYOUT == L_TN) {
            const int i = t.second ? tile - tiles0 : tile, nmt = (p.M + BM - 1) / BM;
            const int nth = i / (nmt * nct), rem = i - nth * nmt * nct;
            t.g = __ffsll((unsigned long long)__ballot(lane < E && !mine_few && place == nth)) - 1;
            t.m0 = rem / nct * BM;
            t.n0 = rem % nct * BN;
            t.kbeg = __builtin_amdgcn_readlane(off.begin, t.g);
            t.kend = t.kbeg + __builtin_amdgcn_readlane(off.count, t.g);
        } else {
            const int rt = tile / nct;
            t.n0 = (tile - rt * nct) * BN;
            t.g = __ffsll((unsigned long long)__ballot(rt >= off.t_begin && rt < off.t_end)) - 1;
            const int in = (rt - __builtin_amdgcn_readlane(off.t_begin, t.g)) * BM;
            t.row0 = __builtin_amdgcn_readlane(off.begin, t.g) + in;
            t.rows = min(BM, __builtin_amdgcn_readlane(off.count, t.g) - in);
            t.kend = p.K;
        }
        return t;
    };
    // This lane's part in load instruction number wave + 4 i of an operand.  k-contiguous: row 4 (wave + 4 i) + lane / 16, chunk
    // lane % 16 (holding the one that the swizzle puts there: it does not depend on i).  k-strided: k-row
    // (wave + 4 i) * KPI + lane / CPR, chunk lane % CPR.
    constexpr int CPR = B / 4, KPI = 64 / CPR;
    const int kc_row = wave * 4 + lane / 16, kc_k = ((lane % 16) ^ (kc_row & 15)) * 4;
    const int ks_row = wave * KPI + lane / CPR, ks_col = lane % CPR * 4;
    const float* pa[A_KC ? NI : 1];
    const float* pb[B_KC ? NI : 1];
    int lda = 0, ldb = 0;                               // of the tile that is being fetched, kept in registers: a TN launch
    const int32_t* rows = nullptr;                      // would read its problem's from memory for every slab
    int bidx[NI];                                       // TN with gathered R rows: the next slab's row numbers
    // Rows and columns outside the tile are clamped onto valid ones (their products are never stored), k's outside the
    // contraction range too; those are zeroed in both operands (0 times an infinity in the clamped element of the
    // other would be NaN).
    auto fetch_rows = [&](const Tile& t, int k0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) bidx[i] = rows[min(k0 + ks_row + i * 4 * KPI, t.kend - 1)];
    };
    auto aim = [&](const Tile& t) {
        const F32Args& p = q.p[t.second];
        lda = p.lda; ldb = p.ldb; rows = p.rows;
        asm volatile("" : "+s"(lda), "+s"(ldb), "+s"(rows));
        const float* Bg = LAYOUT == L_TN ? p.B : p.B + (int64_t)t.g * p.b_group_stride;
        if (A_KC) {
            int r[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) r[i] = t.row0 + min(kc_row + 16 * i, t.rows - 1);
            if (rows)
#pragma unroll
                for (int i = 0; i < NI; ++i) r[i] = rows[r[i]];
#pragma unroll
            for (int i = 0; i < NI; ++i) pa[A_KC ? i : 0] = p.A + (int64_t)r[i] * lda;
        } else {
            pa[0] = p.A + min(t.m0 + ks_col, p.M - 4);
        }
        if (B_KC) {
#pragma unroll
            for (int i = 0; i < NI; ++i) pb[B_KC ? i : 0] = Bg + (int64_t)min(t.n0 + kc_row + 16 * i, p.N - 1) * ldb;
        } else {
            pb[0] = Bg + min(t.n0 + ks_col, p.N - 4);
        }
        if (LAYOUT == L_TN && rows && t.kbeg < t.kend) fetch_rows(t, t.kbeg);
    };
    auto issue = [&](const Tile& t, int k0, int stage) {
        unsigned char* sa = smem + stage * STAGE + wave * 1024;
        unsigned char* sb = sa + OPERAND;
        const int kc = min(k0 + kc_k, t.kend - 4);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int ks = min(k0 + ks_row + i * 4 * KPI, t.kend - 1);
            load_to_lds(A_KC ? pa[A_KC ? i : 0] + kc : pa[0] + (int64_t)ks * lda, sa + i * 4096);
        }
        const bool gathered = LAYOUT == L_TN && rows;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int ks = gathered ? bidx[i] : min(k0 + ks_row + i * 4 * KPI, t.kend - 1);
            load_to_lds(B_KC ? pb[B_KC ? i : 0] + kc : pb[0] + (int64_t)ks * ldb, sb + i * 4096);
        }
        if (gathered && k0 + BK < t.kend) fetch_rows(t, k0 + BK);
    };

    // both operands beyond the end of the contraction (`left` k's into the slab): each lane clears what it has loaded
    auto zero_tail = [&](int stage, int left) {
        unsigned char* sa = smem + stage * STAGE + wave * 1024 + lane * 16;
        unsigned char* sb = sa + OPERAND;
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int i = 0; i < NI; ++i) {
            const bool out = ks_row + i * 4 * KPI >= left;
            if (A_KC ? kc_k >= left : out) *reinterpret_cast<f32x4*>(sa + i * 4096) = z;
            if (B_KC ? kc_k >= left : out) *reinterpret_cast<f32x4*>(sb + i * 4096) = z;
        }
    };

    // Behind an infinite or NaN operand the smaller products are NaN; the large ones have what float32 products would give, unless the
    // operand is a NaN that looks like an infinity in its first term.
    // (Asked of the small sum: the sum of both overflows where a float32 sum does.)
    auto both = [](float large, float small) {
        return fabsf(small) <= 3.402823466e38f ? large + small : large;
    };
    // So an infinite output is one only if there is no NaN among its operands: element (row, column) of C of expert g, k's
    // [kbeg, kend).  (Made canonical before they are taken apart, all operands would pay for it, with 3 % of a training step.)
    auto nan_among = [&](const F32Args& p, int g, int row, int column, int kbeg, int kend) {
        const float* Bg = LAYOUT == L_TN ? p.B : p.B + (int64_t)g * p.b_group_stride;
        const int64_t arow = LAYOUT == L_TN ? 0 : p.rows ? p.rows[row] : row;
        bool nan = false;
#pragma unroll 1
        for (int k = kbeg; k < kend; ++k) {
            const int64_t brow = LAYOUT == L_TN && p.rows ? p.rows[k] : k;
            const float a = LAYOUT == L_TN ? p.A[(int64_t)k * p.lda + row] : p.A[arow * p.lda + k],
                        b = B_KC ? Bg[(int64_t)column * p.ldb + k] : Bg[brow * p.ldb + column];
            nan |= a != a || b != b;
        }
        return nan;
    };
    auto infinite = [](float v) { return fabsf(v) == __builtin_inff(); };
    int first = 0;                                      // stage of the tile's first slab
    auto start = [&](const Tile& t) {
        aim(t);
        if (t.kbeg < t.kend) issue(t, t.kbeg, first);
    };
    Tile next{};
    if (tile < tile_end) {
        next = locate(tile);
        start(next);
    }
    for (; tile < tile_end; tile += step) {
        const Tile t = next;
        const F32Args& p = q.p[t.second];
        const int kbeg = t.kbeg, kend = t.kend, nslab = (kend - kbeg + BK - 1) / BK;
        const bool more = tile + step < tile_end;
        if (more) next = locate(tile + step);

        f32x16 acc[TM][TM], small[TM][TM];              // hi * hi; the five smaller products
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = small[i][j][r] = 0.f;

        auto read = [&](const float* operand, bool k_contiguous, int i, float (&out)[TM][8]) {
            float* v = out[i];
            if (k_contiguous) {
                const float* row = operand + (i * 32 + l32) * BK;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 c = *reinterpret_cast<const f32x4*>(row + ((wave * 4 + kg * 2 + h) ^ (l32 & 15)) * 4);
                    v[4 * h] = c.x; v[4 * h + 1] = c.y; v[4 * h + 2] = c.z; v[4 * h + 3] = c.w;
                }
            } else if (TM == 1) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = operand[(wave * 16 + kg * 8 + e) * B + l32];
            } else if (i == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const f32x2 c = *reinterpret_cast<const f32x2*>(operand + (wave * 16 + kg * 8 + e) * B + 2 * l32);
                    out[0][e] = c.x;
                    out[TM - 1][e] = c.y;
                }
            }
        };
        for (int s = 0; s < nslab; ++s) {
            all_landed();                               // slab s is there, and everyone is done with the other stage
            const int stage = first ^ (s & 1), k0 = kbeg + s * BK;
            if (s + 1 < nslab) issue(t, k0 + BK, stage ^ 1);
            if (k0 + BK > kend) {                       // block-uniform: the contraction ends inside this slab
                zero_tail(stage, kend - k0);
                __syncthreads();
            }
            const float* sa = reinterpret_cast<const float*>(smem + stage * STAGE);
            const float* sb = sa + OPERAND / 4;
            const int kw = k0 + wave * 16;              // this wave's 16 k's
            if (kw < kend) {
                // raw fragments: eight k's of a row (column) per lane
                float va[TM][8], vb[TM][8];
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    read(sa, A_KC, i, va);
                    read(sb, B_KC, i, vb);
                }
                bf16x8 fa[3][TM], fb[3][TM];
                auto products = [&](int i, int j) {
#pragma unroll
                    for (int u = 0; u < 6; ++u) {
                        constexpr int TA[6] = {0, 0, 1, 1, 0, 2}, TB[6] = {0, 1, 0, 1, 2, 0};
                        f32x16& c = u == 0 ? acc[i][j] : small[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[TA[u]][i], fb[TB[u]][j], c, 0, 0, 0);
                    }
                };
                // the next fragment is split under the products of the ones before it: eight VALU slots per MFMA
                auto spread = [&]() {
#pragma unroll
                    for (int u = 0; u < 6; ++u) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                split8(va[0], fa[0][0], fa[1][0], fa[2][0]);
                split8(vb[0], fb[0][0], fb[1][0], fb[2][0]);
                __builtin_amdgcn_sched_barrier(0);
                products(0, 0);
                if (TM == 2) {
                    split8(va[TM - 1], fa[0][TM - 1], fa[1][TM - 1], fa[2][TM - 1]);
                    spread();
                    products(TM - 1, 0);
                    split8(vb[TM - 1], fb[0][TM - 1], fb[1][TM - 1], fb[2][TM - 1]);
                    spread();
                    products(0, TM - 1);
                    products(TM - 1, TM - 1);
                }
            }
        }
        if (kend - kbeg <= 16 && wave == 0 && nslab) {
            // mid * lo and lo * mid, from the only slab's operands, read and taken apart again, so that the loop keeps nothing for it
            const float* sa = reinterpret_cast<const float*>(smem + first * STAGE);
            const float* sb = sa + OPERAND / 4;
            float va[TM][8], vb[TM][8];
            bf16x8 fa[3][TM], fb[3][TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                read(sa, A_KC, i, va);
                read(sb, B_KC, i, vb);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                split8(va[i], fa[0][i], fa[1][i], fa[2][i]);
                split8(vb[i], fb[0][i], fb[1][i], fb[2][i]);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    small[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1][i], fb[2][j], small[i][j], 0, 0, 0);
                    small[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[2][i], fb[1][j], small[i][j], 0, 0, 0);
                }
        }
        first ^= nslab & 1;
        if (more) start(next);                          // the next tile's first slab is fetched under this tile's epilogue

        // ---------------- epilogue: the four waves' partial tiles, added in wave order, 32 rows at a time ----------------
        const int lim_r = LAYOUT == L_TN ? p.M - t.m0 : t.rows;         // rows of the tile that exist
        const int64_t origin = LAYOUT == L_TN ? ((int64_t)t.g * p.M + t.m0) * p.N : (int64_t)t.row0 * p.N;
        const float* reads = EPI == E_ACTGRAD ? p.Hin + origin : EPI == E_WGRAD && accumulate ? p.out1 + origin : nullptr;
        float* red = reinterpret_cast<float*>(smem + (first ^ 1) * STAGE);      // the stage that the next tile does not start in
        auto row_of = [](int i, int r) { return A_PAIR ? 2 * r + i : i * 32 + r; };     // of row r of pass i
        constexpr int NO = B / 32;                      // vectors of four outputs per thread and pass
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    red[(wave * 32 + 8 * (r >> 2) + 4 * kg + (r & 3)) * B + (B_PAIR ? 2 * l32 + j : j * 32 + l32)] =
                        both(acc[i][j][r], small[i][j][r]);
            f32x4 old[NO], bias[NO];
#pragma unroll
            for (int u = 0; u < NO; ++u) {
                const int o = tid + 256 * u, tr = min(row_of(i, o / (B / 4)), lim_r - 1), n = min(t.n0 + o % (B / 4) * 4, p.N - 4);
                old[u] = bias[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (reads) old[u] = *reinterpret_cast<const f32x4*>(reads + (int64_t)tr * p.N + n);
                if ((EPI == E_HA || EPI == E_BIAS) && p.bias) bias[u] = *reinterpret_cast<const f32x4*>(p.bias + (int64_t)t.g * p.N + n);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NO; ++u) {
                const int o = tid + 256 * u, tr = row_of(i, o / (B / 4)), n = t.n0 + o % (B / 4) * 4;
                if (tr >= lim_r || n >= p.N) continue;
                f32x4 v = {0.f, 0.f, 0.f, 0.f}, a;
#pragma unroll
                for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const f32x4*>(red + (w * 32 + o / (B / 4)) * B + o % (B / 4) * 4);
                if (infinite(fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))))) {
#pragma unroll 1
                    for (int e = 0; e < 4; ++e)
                        if (infinite(v[e]) && nan_among(p, t.g, LAYOUT == L_TN ? t.m0 + tr : t.row0 + tr, n + e, kbeg, kend))
                            v[e] = __builtin_nanf("");
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (EPI == E_HA || EPI == E_BIAS) v[e] += bias[u][e];
                    if (EPI == E_ACTGRAD) v[e] *= act_grad(old[u][e], act);
                    if (EPI == E_WGRAD && accumulate) v[e] += old[u][e];
                    a[e] = EPI == E_HA ? act_fwd(v[e], act) : 0.f;
                }
                *reinterpret_cast<f32x4*>(p.out1 + origin + (int64_t)tr * p.N + n) = v;
                if (EPI == E_HA) *reinterpret_cast<f32x4*>(p.out2 + origin + (int64_t)tr * p.N + n) = a;
            }
        }
    }
    if constexpr (LAYOUT == L_TN && TM == 2) {
        // Experts with few rows: a wave takes 32 rows by 64 columns of a gradient by itself, its operands straight from memory.  The same
        // products in the same order as in a tile, whose waves have 16 k's each and whose sums are added in their order.
        const int experts = __popcll(few), all = experts * (units0 + units1);
        const int block = (gridDim.x & 7) == 0 ? (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
        for (int u = block * 4 + wave; u < all; u += gridDim.x * 4) {
            const int second = u >= experts * units0, i = second ? u - experts * units0 : u, per = second ? units1 : units0;
            const F32Args& p = q.p[second];
            const int nth = i / per, rem = i - nth * per, nn = (p.N + BN - 1) / BN;
            const int g = __ffsll((unsigned long long)__ballot(mine_few && place == nth)) - 1;
            const int kbeg = __builtin_amdgcn_readlane(off.begin, g), count = __builtin_amdgcn_readlane(off.count, g);
            const int m0 = rem / nn * 32, n0 = rem % nn * BN;
            const float* A = p.A + (int64_t)kbeg * p.lda + min(m0 + l32, p.M - 1);
            const float* R[TM];
#pragma unroll
            for (int j = 0; j < TM; ++j) R[j] = p.B + min(n0 + j * 32 + l32, p.N - 1);
            f32x16 sum[TM];
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[j][r] = 0.f;
#pragma unroll 1
            for (int k = 0; k < count; k += 16) {
                const int k0 = k + kg * 8;              // this lane's eight k's
                int row[8];
                float va[8], vb[TM][8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    row[e] = kbeg + min(k0 + e, count - 1);
                    if (p.rows) row[e] = p.rows[row[e]];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) va[e] = A[min(k0 + e, count - 1) * p.lda];
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int j = 0; j < TM; ++j) vb[j][e] = R[j][(int64_t)row[e] * p.ldb];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (k0 + e >= count) {
                        va[e] = 0.f;
#pragma unroll
                        for (int j = 0; j < TM; ++j) vb[j][e] = 0.f;
                    }
                bf16x8 fa[3], fb[3];
                split8(va, fa[0], fa[1], fa[2]);
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    split8(vb[j], fb[0], fb[1], fb[2]);
                    f32x16 large, small;
#pragma unroll
                    for (int r = 0; r < 16; ++r) large[r] = small[r] = 0.f;
                    constexpr int TA[8] = {0, 0, 1, 1, 0, 2, 1, 2}, TB[8] = {0, 1, 0, 1, 2, 0, 2, 1};
#pragma unroll
                    for (int u = 0; u < 6; ++u) {
                        f32x16& c = u == 0 ? large : small;
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[TA[u]], fb[TB[u]], c, 0, 0, 0);
                    }
                    if (count <= 16) {
#pragma unroll
                        for (int u = 6; u < 8; ++u) small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[TA[u]], fb[TB[u]], small, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum[j][r] += both(large[r], small[r]);
                }
            }
            float largest = 0.f;
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) largest = fmaxf(largest, fabsf(sum[j][r]));
            float* out = p.out1 + ((int64_t)g * p.M + m0) * p.N + n0 + l32;
            auto row_at = [&](int r) { return 8 * (r >> 2) + 4 * kg + (r & 3); };
            if (accumulate) {           // the old gradient, at clamped addresses, before the first store
                float old[TM][16];
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        old[j][r] = out[(int64_t)min(row_at(r), p.M - 1 - m0) * p.N + min(j * 32, p.N - 1 - n0 - l32)];
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum[j][r] += old[j][r];
            }
            auto store = [&](bool whole) {
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (whole || (m0 + row_at(r) < p.M && n0 + j * 32 + l32 < p.N))
                            out[(int64_t)row_at(r) * p.N + j * 32] = sum[j][r];
            };
            if (m0 + 32 <= p.M && n0 + BN <= p.N) store(true); else store(false);
            if (infinite(largest)) {
#pragma unroll 1
                for (int r = 0; r < 16 * TM; ++r) {
                    const int m = row_at(r & 15), n = r / 16 * 32;
                    float* at = out + (int64_t)m * p.N + n;
                    if (m0 + m < p.M && n0 + n + l32 < p.N && infinite(*at) && nan_among(p, g, m0 + m, n0 + n + l32, kbeg, kbeg + count))
                        *at = __builtin_nanf("");
                }
            }
        }
    }
    // the column sums, dealt from the last block on: those have a tile less, or none
    if (EPI == E_NONE) {
        const int tiles = kSumSplit * E * (sums.blocks[0] + sums.blocks[1]);
        if (tiles) __syncthreads();
        for (int b = gridDim.x - 1 - blockIdx.x; b < tiles; b += gridDim.x) colsum_tile(sums, b, off, E, reinterpret_cast<float*>(smem));
    }
    if (LAYOUT == L_TN) {
        const int64_t n = (int64_t)E * ((sums.blocks[0] ? sums.N[0] : 0) + (sums.blocks[1] ? sums.N[1] : 0));
        for (int64_t i = (int64_t)(gridDim.x - 1 - blockIdx.x) * 256 + tid; i < n; i += (int64_t)gridDim.x * 256)
            colsum_final(sums, i, expert_offsets, E, P_cap, accumulate);
    }
}

// Which tile.  A launch takes about (tiles each CU gets) x (work of a tile); 32x32 tiles pad and quantise less, but take twice
// as many operands apart and fetch twice as much: 1.4 times as long per output, 1.25 where the contraction is short (its
// start and end then count) and for the weight gradients.  Measured (us, 64x64 / 32x32) at d = 256, E = 8, F = 1024: 5632
// pairs GEMM1 37 / 41, GEMM2 30 / 33, dXp 33 / 36, both dW 51 / 72; 1340 pairs GEMM1 19 / 17, GEMM2 21 / 15, dW 24 / 28;
// d = 512, E = 16, F = 2048, 11000 pairs GEMM1 181 / 236, dW 351 / 499; d = 64, E = 4, F = 256, 650 pairs GEMM2 11 / 7;
// d = 64, E = 1, F = 256, 4096 pairs dW 69 / 40.
enum class Size { T64, T32 };
int64_t tiles_of(int64_t row_tiles, int n, int b) { return row_tiles * ((n + b - 1) / b); }
Size cheapest(const Ctx& c, int64_t t64, int64_t t32, double per_output) {
    auto rounds = [&](int64_t tiles) { return (double)((tiles + c.num_cu - 1) / c.num_cu); };
    return rounds(t32) * (32 * 32 * per_output) < rounds(t64) * (64 * 64) ? Size::T32 : Size::T64;
}

template <int LAYOUT, int EPI, int B>
hipError_t launch(const Ctx& c, const evomoe_shape& s, const F32Args& a, int64_t t0, const F32Args& b, int64_t t1,
                  const F32Sums& sums, int64_t sum_tiles, const int32_t* expert_offsets, int accumulate) {
    const int64_t cap = (int64_t)c.num_cu * blocks_per_cu<B>(), want = (t0 + t1 + sum_tiles + 7) / 8 * 8;
    hipLaunchKernelGGL((grouped_gemm_f32<LAYOUT, EPI, B, B>), dim3((unsigned)(want < cap ? want : cap)), dim3(256), 0,
                       c.stream, F32Pair{{a, b}}, (int)t0, (int)(t0 + t1), sums, expert_offsets, s.E, s.P_cap, s.act,
                       accumulate);
    return hipGetLastError();
}

// NT / NN: one problem over the row tiles of all experts
Size rows_tile(const Ctx& c, const evomoe_shape& s, int n, int k) {
    const int64_t P = c.pair_hint > 0 && c.pair_hint < s.P_cap ? c.pair_hint : s.P_cap;
    auto expected = [&](int b) { return tiles_of((P + b - 1) / b + s.E / 2, n, b); };
    return cheapest(c, expected(64), expected(32), k < 512 ? 1.25 : 1.4);
}
template <int LAYOUT, int EPI>
hipError_t launch_rows(const Ctx& c, const evomoe_shape& s, const F32Args& a, const int32_t* expert_offsets,
                       const F32Sums& sums = F32Sums{}) {
    auto worst = [&](int b) { return tiles_of((s.P_cap + b - 1) / b + s.E, a.N, b); };
    const int64_t st = (int64_t)kSumSplit * s.E * (sums.blocks[0] + sums.blocks[1]);
    if (rows_tile(c, s, a.N, a.K) == Size::T64)
        return launch<LAYOUT, EPI, 64>(c, s, a, worst(64), a, 0, sums, st, expert_offsets, 0);
    return launch<LAYOUT, EPI, 32>(c, s, a, worst(32), a, 0, sums, st, expert_offsets, 0);
}
// TN: the tiles of one of the two problems; both count for the choice, whichever is wanted
int64_t wgrad_tiles(const evomoe_shape& s, int b) { return (int64_t)s.E * ((s.d + b - 1) / b) * ((s.F + b - 1) / b); }
Size wgrad_tile(const Ctx& c, const evomoe_shape& s) { return cheapest(c, 2 * wgrad_tiles(s, 64), 2 * wgrad_tiles(s, 32), 1.25); }

}  // namespace

FfnTile f32_ffn_tile(const Ctx& c, const evomoe_shape& s, int kernel) {
    Size t;
    switch (kernel) {
        case EVOMOE_K_FFN_GEMM1: case EVOMOE_K_FFN_BWD_DH: t = rows_tile(c, s, s.F, s.d); break;
        case EVOMOE_K_FFN_GEMM2: case EVOMOE_K_FFN_BWD_DX: t = rows_tile(c, s, s.d, s.F); break;
        case EVOMOE_K_FFN_BWD_DW2: t = wgrad_tile(c, s); break;
        default: return {};
    }
    return t == Size::T64 ? FfnTile{64, 64, 4} : FfnTile{32, 32, 4};
}

hipError_t f32_ffn_fwd(const Ctx& c, const evomoe_shape& s, const void* x, const int32_t* pair_token,
                       const int32_t* expert_offsets, const void* W1, const float* b1, const void* W2,
                       const float* b2, void* H, void* A, void* O) {
    hipError_t err;
    {   // H = X W1^T + b1, A = act(H)
        ProfScope ps(c, EVOMOE_K_FFN_GEMM1);
        F32Args a{};
        a.A = (const float*)x; a.lda = s.d; a.rows = pair_token;
        a.B = (const float*)W1; a.ldb = s.d; a.b_group_stride = (int64_t)s.F * s.d;
        a.N = s.F; a.K = s.d; a.bias = b1; a.out1 = (float*)H; a.out2 = (float*)A;
        err = launch_rows<L_NT, E_HA>(c, s, a, expert_offsets);
    }
    if (err != hipSuccess || !O) return err;      // O == nullptr: recomputation of H and A only
    // O = A W2^T + b2
    ProfScope ps(c, EVOMOE_K_FFN_GEMM2);
    F32Args a{};
    a.A = (const float*)A; a.lda = s.F;
    a.B = (const float*)W2; a.ldb = s.F; a.b_group_stride = (int64_t)s.d * s.F;
    a.N = s.d; a.K = s.F; a.bias = b2; a.out1 = (float*)O;
    return launch_rows<L_NT, E_BIAS>(c, s, a, expert_offsets);
}

hipError_t f32_ffn_bwd(const Ctx& c, const evomoe_shape& s, const void* dO, const void* H, const void* A,
                       const void* x, const int32_t* pair_token, const int32_t* expert_offsets, const void* W1,
                       const void* W2, void* dW1, float* db1, void* dW2, float* db2, void* dXp, int accumulate,
                       void* dH) {
    hipError_t err;
    {   // dH = (dO W2) * act'(H)
        ProfScope ps(c, EVOMOE_K_FFN_BWD_DH);
        F32Args a{};
        a.A = (const float*)dO; a.lda = s.d; a.B = (const float*)W2; a.ldb = s.F;
        a.b_group_stride = (int64_t)s.d * s.F; a.N = s.F; a.K = s.d; a.Hin = (const float*)H; a.out1 = (float*)dH;
        err = launch_rows<L_NN, E_ACTGRAD>(c, s, a, expert_offsets);
        if (err != hipSuccess) return err;
    }
    // db2 = column sums of dO, db1 = column sums of dH
    F32Sums sums{};
    float* part = reinterpret_cast<float*>(static_cast<char*>(dH) + dh_bytes(s));
    sums.m[0] = (const float*)dO; sums.N[0] = s.d; sums.db[0] = db2; sums.part[0] = part;
    sums.m[1] = (const float*)dH; sums.N[1] = s.F; sums.db[1] = db1; sums.part[1] = part + (size_t)kSumSplit * s.E * s.d;
    for (int i = 0; i < 2; ++i) sums.blocks[i] = sums.db[i] ? (sums.N[i] + kSumCols - 1) / kSumCols : 0;
    {   // dXp = dH W1
        ProfScope ps(c, EVOMOE_K_FFN_BWD_DX);
        F32Args a{};
        a.A = (const float*)dH; a.lda = s.F; a.B = (const float*)W1; a.ldb = s.d;
        a.b_group_stride = (int64_t)s.F * s.d; a.N = s.d; a.K = s.F; a.out1 = (float*)dXp;
        err = launch_rows<L_NN, E_NONE>(c, s, a, expert_offsets, sums);
        if (err != hipSuccess) return err;
    }
    // dW2_g = dO_g^T A_g [d,F], dW1_g = dH_g^T X_g [F,d]: one launch over both problems' tiles
    F32Args w[2]{};
    int n = 0;
    auto add = [&](const void* L, int M, const void* R, int N, const int32_t* rows, void* dW) {
        if (!dW) return;
        F32Args& a = w[n++];
        a.A = (const float*)L; a.lda = M; a.M = M; a.B = (const float*)R; a.ldb = N; a.N = N; a.rows = rows;
        a.out1 = (float*)dW;
    };
    add(dO, s.d, A, s.F, nullptr, dW2);
    add(dH, s.F, x, s.d, pair_token, dW1);
    const int64_t st = ((int64_t)s.E * ((db2 ? s.d : 0) + (db1 ? s.F : 0)) + 255) / 256;
    if (n == 0 && st == 0) return hipSuccess;
    ProfScope ps(c, dW2 ? EVOMOE_K_FFN_BWD_DW2 : dW1 ? EVOMOE_K_FFN_BWD_DW1 : EVOMOE_K_FFN_BWD_DB);
    auto run = [&](auto launcher, int b) {
        return launcher(c, s, w[0], n > 0 ? wgrad_tiles(s, b) : 0, w[1], n > 1 ? wgrad_tiles(s, b) : 0, sums, st, expert_offsets,
                        accumulate);
    };
    return wgrad_tile(c, s) == Size::T64 ? run(launch<L_TN, E_WGRAD, 64>, 64) : run(launch<L_TN, E_WGRAD, 32>, 32);
}

}  // namespace evomoe
