// Expert FFNs of a float32 layer (EvoMoE Eq. ffn per expert over its ragged row range, and its backward) on the
// float32 matrix cores.  One grouped-GEMM kernel, v_mfma_f32_32x32x2_f32 (products and sums are float32 throughout):
//
//   NT  C[r,n] = sum_k A[arow(r),k] * W_g[n,k]          forward GEMMs (A rows optionally gathered by token)
//   NN  C[r,n] = sum_k A[r,k]       * W_g[k,n]          dH = dO W2,  dXp = dH W1
//   TN  C_g[m,n] = sum_{r in g} L[r,m] * R[rrow(r),n]   weight gradients (contraction over the ragged rows)
//
// What bounds it: the float32 matrix rate (256 flop per clock and CU, a sixteenth of bf16's), so neither LDS nor L2
// needs more than plain double buffering: global -> registers -> LDS one slab ahead, several blocks per CU.  GEMM1 of
// 11160 pairs, d = 512, F = 2048: 102 TFLOP/s; a 4096^3 library product reaches 137 on the same card, the float32-FMA
// kernels that stood here before 25.  The bias gradients' column sums are further tiles behind dXp's and behind the weight
// gradients': colsum_tile().
// A lane's four k's of one fragment come from one 16-byte LDS read where k is contiguous and from four 4-byte reads
// where it is the row index; both operands use the same k order, so the order inside a slab is free.
//
// Tiles: 64x64 (four waves, 2 x 2), and 32x32 with the slab's k's split over the four waves for launches that would
// leave most of the chip idle; cheapest() says which and why.  Both add the products of one output in the same order, so
// that results do not depend on the pair count announced, nor on how many rows a call has.
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

// Blocks per CU, for the registers and for the grid: four (128 registers) fill the stalls that one's loads and barriers
// leave; 64x64 tiles of dH, whose act'(H) epilogue spills there, and of GEMM2 take three.  us at d = 512, F = 2048, 11160 /
// 8126 / 30000 pairs, and d = 256, F = 1024, 5626: dH with four 266 / - / - / 56, with three and a grid for four 291 / 215 /
// 758 / 51, with three 268 / 198 / 700 / 51; GEMM2 with four 236 / 167 / 570 / 44, with three 229 / 166 / 557 / 44; dXp and
// the weight gradients are 2-5 % slower with three.  (All before the fragments were read ahead: NP below.)
template <int EPI, int B> constexpr int blocks_per_cu() { return B == 64 && (EPI == E_ACTGRAD || EPI == E_BIAS) ? 3 : 4; }
template <int LAYOUT, int EPI, int BM, int BN>
__global__ __launch_bounds__(256, (blocks_per_cu<EPI, BM>())) void grouped_gemm_f32(
    F32Pair q, int tiles0, int tiles_all, F32Sums sums, const int32_t* __restrict__ expert_offsets, int E, int64_t P_cap,
    int act, int accumulate)
{
    constexpr bool SPLIT = BM == 32;                    // 32x32: the four waves share one tile, a quarter of the k's each
    constexpr int BK = SPLIT ? 64 : 32;
    static_assert(BM == BN && (BM == 32 || BM == 64), "tile");
    constexpr bool A_KC = LAYOUT != L_TN, B_KC = LAYOUT == L_NT;
    // LDS rows: [row][BK + 4] (16 lanes' 16-byte reads of one k chunk then cover all 64 banks) or [k][cols + 8]
    // (the two k groups of a 4-byte read lie 32 banks apart)
    constexpr int A_LD = A_KC ? BK + 4 : BM + 8, B_LD = B_KC ? BK + 4 : BN + 8;
    constexpr int A_SZ = A_KC ? BM * A_LD : BK * A_LD, B_SZ = B_KC ? BN * B_LD : BK * B_LD;
    constexpr int A_V = BM * BK / 1024, B_V = BN * BK / 1024;              // 16-byte vectors per thread and slab
    // Groups of 8 k's are dealt round-robin to four partial sums, which are added in order at the end.  In the 32x32 tile
    // each wave has one of them, in the 64x64 tile every wave has all four for its quarter of the tile: the order of the
    // additions, and with it every bit of the result, is the same in both.  (One sum per output in the 64x64 tile, as long as
    // the whole contraction, took 1 % less for the GEMMs and 2-4 % for dXp, and gave other bits than the 32x32 tile.)
    constexpr int NP = SPLIT ? 1 : 4, NG = BK / 32;                        // partial sums per wave, groups of each per slab
    // A group's fragments are read under the MFMAs of the group before, which the scheduler keeps to where registers allow:
    // 64x64 tiles of GEMM1, GEMM2 and dH at d = 512, F = 2048, 30000 pairs 608, 561 and 700 -> 592, 543 and 686 us, dXp's
    // 590 -> 618 if it is held to it, the weight gradients' 1205 -> 1266, and 150 -> 155 in 32x32 tiles if they read ahead.
    constexpr bool AHEAD = LAYOUT != L_TN, PIN = AHEAD && !SPLIT && EPI != E_NONE;
    __shared__ float smem[2 * (A_SZ + B_SZ)];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kg = lane >> 5;
    const int wm = SPLIT ? 0 : (wave >> 1) * (BM / 2), wn = SPLIT ? 0 : (wave & 1) * (BN / 2);
    const int wk = SPLIT ? wave * 8 : 0;

    const Offsets off = scan_offsets<BM>(expert_offsets, E, P_cap, lane);
    const int row_tiles = __builtin_amdgcn_readlane(off.t_end, 63);

    // Consecutive tiles share operand panels, and blocks are dealt round-robin to the 8 XCDs: each XCD walks one
    // contiguous eighth of the tiles, so that its L2 sees the panels and no XCD gets a round more than another.
    const int total = LAYOUT == L_TN ? tiles_all : row_tiles * ((q.p[0].N + BN - 1) / BN);
    int tile = blockIdx.x, tile_end = total, step = gridDim.x;
    if ((gridDim.x & 7) == 0) {
        const int x = blockIdx.x & 7;
        tile = (int)((int64_t)total * x / 8) + (blockIdx.x >> 3);
        tile_end = (int)((int64_t)total * (x + 1) / 8);
        step = gridDim.x >> 3;
    }
    for (; tile < tile_end; tile += step) {
        const bool second = LAYOUT == L_TN && tile >= tiles0;
        const F32Args& p = q.p[second];
        const int nct = (p.N + BN - 1) / BN;
        int g, row0 = 0, rows = 0, m0 = 0, n0, kbeg = 0, kend;
        if (LAYOUT == L_TN) {
            const int t = second ? tile - tiles0 : tile, nmt = (p.M + BM - 1) / BM;
            g = t / (nmt * nct);
            const int rem = t - g * nmt * nct;
            m0 = rem / nct * BM;
            n0 = rem % nct * BN;
            kbeg = __builtin_amdgcn_readlane(off.begin, g);
            kend = kbeg + __builtin_amdgcn_readlane(off.count, g);
        } else {
            const int rt = tile / nct;
            n0 = (tile - rt * nct) * BN;
            g = __ffsll((unsigned long long)__ballot(rt >= off.t_begin && rt < off.t_end)) - 1;
            const int in = (rt - __builtin_amdgcn_readlane(off.t_begin, g)) * BM;
            row0 = __builtin_amdgcn_readlane(off.begin, g) + in;
            rows = min(BM, __builtin_amdgcn_readlane(off.count, g) - in);
            kend = p.K;
        }
        const float* Bg = LAYOUT == L_TN ? p.B : p.B + (int64_t)g * p.b_group_stride;
        const int nslab = (kend - kbeg + BK - 1) / BK;

        // This thread's share of a slab: vector v of an operand is number tid + 256 v of the slab's 16-byte pieces.
        // Rows and columns outside the tile are clamped onto valid ones (their products are never stored), k's outside
        // the contraction range too; both operands are zero there (0 times an infinity in the clamped element of the other
        // would be NaN).  No load sits in a branch, so a slab's loads go out together.
        const float* arow[A_V];
        const float* brow[B_V];
        int bidx[B_V];                                          // TN with gathered R rows: the next slab's row numbers
        const bool gathered = LAYOUT == L_TN && p.rows;
#pragma unroll
        for (int v = 0; v < A_V; ++v) {
            const int i = tid + 256 * v;
            if (A_KC) {
                const int r = row0 + min(i / (BK / 4), rows - 1);
                arow[v] = p.A + (int64_t)(p.rows ? p.rows[r] : r) * p.lda;
            } else {
                arow[v] = p.A + min(m0 + (i % (BM / 4)) * 4, p.M - 4);
            }
        }
#pragma unroll
        for (int v = 0; v < B_V; ++v) {
            const int i = tid + 256 * v;
            if (B_KC) brow[v] = Bg + (int64_t)min(n0 + i / (BK / 4), p.N - 1) * p.ldb;
            else brow[v] = Bg + min(n0 + (i % (BN / 4)) * 4, p.N - 4);
        }
        f32x4 ra[A_V], rb[B_V];
        auto fetch_rows = [&](int k0) {
#pragma unroll
            for (int v = 0; v < B_V; ++v) bidx[v] = p.rows[min(k0 + (tid + 256 * v) / (BN / 4), kend - 1)];
        };
        auto fetch = [&](int k0) {
#pragma unroll
            for (int v = 0; v < A_V; ++v) {
                const int i = tid + 256 * v;
                if (A_KC) ra[v] = *reinterpret_cast<const f32x4*>(arow[v] + min(k0 + (i % (BK / 4)) * 4, kend - 4));
                else ra[v] = *reinterpret_cast<const f32x4*>(arow[v] + (int64_t)min(k0 + i / (BM / 4), kend - 1) * p.lda);
            }
#pragma unroll
            for (int v = 0; v < B_V; ++v) {
                const int i = tid + 256 * v;
                if (B_KC) {
                    rb[v] = *reinterpret_cast<const f32x4*>(brow[v] + min(k0 + (i % (BK / 4)) * 4, kend - 4));
                } else {
                    const int k = gathered ? bidx[v] : min(k0 + i / (BN / 4), kend - 1);
                    rb[v] = *reinterpret_cast<const f32x4*>(brow[v] + (int64_t)k * p.ldb);
                }
            }
            if (gathered && k0 + BK < kend) fetch_rows(k0 + BK);
            if (k0 + BK > kend) {                               // block-uniform: the last, partial slab
#pragma unroll
                for (int v = 0; v < A_V; ++v) {
                    const int i = tid + 256 * v;
                    if (k0 + (A_KC ? (i % (BK / 4)) * 4 : i / (BM / 4)) >= kend) ra[v] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int v = 0; v < B_V; ++v) {
                    const int i = tid + 256 * v;
                    if (k0 + (B_KC ? (i % (BK / 4)) * 4 : i / (BN / 4)) >= kend) rb[v] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        };
        auto place = [&](float* sa, float* sb) {
#pragma unroll
            for (int v = 0; v < A_V; ++v) {
                const int i = tid + 256 * v;
                *reinterpret_cast<f32x4*>(A_KC ? sa + i / (BK / 4) * A_LD + (i % (BK / 4)) * 4
                                               : sa + i / (BM / 4) * A_LD + (i % (BM / 4)) * 4) = ra[v];
            }
#pragma unroll
            for (int v = 0; v < B_V; ++v) {
                const int i = tid + 256 * v;
                *reinterpret_cast<f32x4*>(B_KC ? sb + i / (BK / 4) * B_LD + (i % (BK / 4)) * 4
                                               : sb + i / (BN / 4) * B_LD + (i % (BN / 4)) * 4) = rb[v];
            }
        };
        f32x16 acc[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;

        if (nslab > 0) {
            if (gathered) fetch_rows(kbeg);
            fetch(kbeg);
            place(smem, smem + A_SZ);
        }
        __syncthreads();
        for (int s = 0; s < nslab; ++s) {
            const float* sa = smem + (s & 1) * (A_SZ + B_SZ);
            const float* sb = sa + A_SZ;
            if (s + 1 < nslab) fetch(kbeg + (s + 1) * BK);
            f32x4 fa[2], fb[2];
            auto frags = [&](int gk) {
                const int k = wk + gk * (SPLIT ? 32 : 8) + kg * 4, m = wm + l32, n = wn + l32;
                f32x4 &a = fa[gk & 1], &b = fb[gk & 1];
                if (A_KC) a = *reinterpret_cast<const f32x4*>(sa + m * A_LD + k);
                else a = f32x4{sa[k * A_LD + m], sa[(k + 1) * A_LD + m], sa[(k + 2) * A_LD + m], sa[(k + 3) * A_LD + m]};
                if (B_KC) b = *reinterpret_cast<const f32x4*>(sb + n * B_LD + k);
                else b = f32x4{sb[k * B_LD + n], sb[(k + 1) * B_LD + n], sb[(k + 2) * B_LD + n], sb[(k + 3) * B_LD + n]};
            };
            if (AHEAD) frags(0);
#pragma unroll
            for (int gk = 0; gk < NG * NP; ++gk) {
                if (!AHEAD) frags(gk);
                else if (gk + 1 < NG * NP) frags(gk + 1);
                if (PIN) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    acc[gk % NP] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[gk & 1][u], fb[gk & 1][u], acc[gk % NP], 0, 0, 0);
                if (PIN) __builtin_amdgcn_sched_barrier(0);
            }
            if (s + 1 < nslab) {
                float* na = smem + ((s + 1) & 1) * (A_SZ + B_SZ);
                place(na, na + A_SZ);
            }
            __syncthreads();
        }

        // ---------------- epilogue ----------------
        // What the epilogue reads (bias, H, the old gradient) is loaded, at clamped addresses, before its first store.
        // Its lane constants come from an opaque copy of the lane number: they are not carried through the main loop.
        int lane_e = tid & 63;
        asm volatile("" : "+v"(lane_e));
        const int l32e = lane_e & 31, rowe = wm + 4 * (lane_e >> 5);
        const int lim_r = LAYOUT == L_TN ? p.M - m0 : rows;             // rows of the tile that exist
        const int64_t origin = LAYOUT == L_TN ? ((int64_t)g * p.M + m0) * p.N : (int64_t)row0 * p.N;
        const float* reads = EPI == E_ACTGRAD ? p.Hin + origin : EPI == E_WGRAD && accumulate ? p.out1 + origin : nullptr;
        auto offset_of = [&](int tr, int n) { return (uint32_t)(min(tr, lim_r - 1) * p.N + min(n, p.N - 1)); };
        auto bias_of = [&](int n) {
            return (EPI == E_HA || EPI == E_BIAS) && p.bias ? p.bias[(int64_t)g * p.N + min(n, p.N - 1)] : 0.f;
        };
        auto finish = [&](int tr, int n, float v, float bias, float old) {
            if (EPI == E_HA || EPI == E_BIAS) v += bias;
            if (EPI == E_ACTGRAD) v *= act_grad(old, act);
            if (EPI == E_WGRAD && accumulate) v += old;
            const float a = EPI == E_HA ? act_fwd(v, act) : 0.f;
            const uint32_t o = offset_of(tr, n);
            if (tr < lim_r && n < p.N) {
                p.out1[origin + o] = v;
                if (EPI == E_HA) p.out2[origin + o] = a;
            }
        };
        if (SPLIT) {
            // the four waves' partial tiles, added in wave order
            constexpr int LD = 36;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                smem[(wave * 32 + 8 * (r >> 2) + 4 * kg + (r & 3)) * LD + l32] = acc[0][r];
            const float bias = bias_of(n0 + l32);
            float old[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) old[u] = reads ? reads[offset_of((tid >> 5) + 8 * u, n0 + l32)] : 0.f;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int tr = (tid >> 5) + 8 * u;
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) v += smem[(w * 32 + tr) * LD + l32];
                finish(tr, n0 + l32, v, bias, old[u]);
            }
            __syncthreads();
        } else {
            const int n = n0 + wn + l32e;
            float sum[16], old[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sum[r] = 0.f;
#pragma unroll
                for (int q = 0; q < NP; ++q) sum[r] += acc[q][r];
            }
            const float bias = bias_of(n);
#pragma unroll
            for (int r = 0; r < 16; ++r) old[r] = reads ? reads[offset_of(rowe + 8 * (r >> 2) + (r & 3), n)] : 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) finish(rowe + 8 * (r >> 2) + (r & 3), n, sum[r], bias, old[r]);
        }
    }
    // the column sums, dealt from the last block on: those have a tile less, or none
    if (EPI == E_NONE) {
        const int tiles = kSumSplit * E * (sums.blocks[0] + sums.blocks[1]);
        if (tiles) __syncthreads();
        for (int b = gridDim.x - 1 - blockIdx.x; b < tiles; b += gridDim.x) colsum_tile(sums, b, off, E, smem);
    }
    if (LAYOUT == L_TN) {
        const int64_t n = (int64_t)E * ((sums.blocks[0] ? sums.N[0] : 0) + (sums.blocks[1] ? sums.N[1] : 0));
        for (int64_t i = (int64_t)(gridDim.x - 1 - blockIdx.x) * 256 + tid; i < n; i += (int64_t)gridDim.x * 256)
            colsum_final(sums, i, expert_offsets, E, P_cap, accumulate);
    }
}

// Which tile.  A launch takes about (tiles each CU gets) x (work of a tile); 32x32 tiles pad and quantise less but take
// about 1.25 times as long per output.  Measured (us, 64x64 / 32x32) at d = 256, E = 8, F = 1024: 5626 pairs GEMM1 46 / 50,
// GEMM2 47 / 44, dXp 54 / 47, both dW 72 / 85; 1419 pairs GEMM2 30 / 18, dW 28 / 35; d = 512, E = 16, F = 2048, 11160 pairs
// GEMM1 230 / 289, dW 479 / 600; d = 64, E = 4, F = 256, 533 pairs GEMM2 12 / 7.  128x128 tiles (GEMM1 63 and GEMM2 84 us
// in the first of these, 286 and 309 in the third) were slower than 64x64 everywhere and are not kept.
enum class Tile { T64, T32 };
int64_t tiles_of(int64_t row_tiles, int n, int b) { return row_tiles * ((n + b - 1) / b); }
Tile cheapest(const Ctx& c, int64_t t64, int64_t t32) {
    auto rounds = [&](int64_t tiles) { return (double)((tiles + c.num_cu - 1) / c.num_cu); };
    return rounds(t32) * (32 * 32 * 1.25) < rounds(t64) * (64 * 64) ? Tile::T32 : Tile::T64;
}

template <int LAYOUT, int EPI, int B>
hipError_t launch(const Ctx& c, const evomoe_shape& s, const F32Args& a, int64_t t0, const F32Args& b, int64_t t1,
                  const F32Sums& sums, int64_t sum_tiles, const int32_t* expert_offsets, int accumulate) {
    const int64_t cap = (int64_t)c.num_cu * blocks_per_cu<EPI, B>(), want = (t0 + t1 + sum_tiles + 7) / 8 * 8;
    hipLaunchKernelGGL((grouped_gemm_f32<LAYOUT, EPI, B, B>), dim3((unsigned)(want < cap ? want : cap)), dim3(256), 0,
                       c.stream, F32Pair{{a, b}}, (int)t0, (int)(t0 + t1), sums, expert_offsets, s.E, s.P_cap, s.act,
                       accumulate);
    return hipGetLastError();
}

// NT / NN: one problem over the row tiles of all experts
Tile rows_tile(const Ctx& c, const evomoe_shape& s, int n) {
    const int64_t P = c.pair_hint > 0 && c.pair_hint < s.P_cap ? c.pair_hint : s.P_cap;
    auto expected = [&](int b) { return tiles_of((P + b - 1) / b + s.E / 2, n, b); };
    return cheapest(c, expected(64), expected(32));
}
template <int LAYOUT, int EPI>
hipError_t launch_rows(const Ctx& c, const evomoe_shape& s, const F32Args& a, const int32_t* expert_offsets,
                       const F32Sums& sums = F32Sums{}) {
    auto worst = [&](int b) { return tiles_of((s.P_cap + b - 1) / b + s.E, a.N, b); };
    const int64_t st = (int64_t)kSumSplit * s.E * (sums.blocks[0] + sums.blocks[1]);
    if (rows_tile(c, s, a.N) == Tile::T64)
        return launch<LAYOUT, EPI, 64>(c, s, a, worst(64), a, 0, sums, st, expert_offsets, 0);
    return launch<LAYOUT, EPI, 32>(c, s, a, worst(32), a, 0, sums, st, expert_offsets, 0);
}
// TN: the tiles of one of the two problems; both count for the choice, whichever is wanted
int64_t wgrad_tiles(const evomoe_shape& s, int b) { return (int64_t)s.E * ((s.d + b - 1) / b) * ((s.F + b - 1) / b); }
Tile wgrad_tile(const Ctx& c, const evomoe_shape& s) { return cheapest(c, 2 * wgrad_tiles(s, 64), 2 * wgrad_tiles(s, 32)); }

}  // namespace

FfnTile f32_ffn_tile(const Ctx& c, const evomoe_shape& s, int kernel) {
    Tile t;
    switch (kernel) {
        case EVOMOE_K_FFN_GEMM1: case EVOMOE_K_FFN_BWD_DH: t = rows_tile(c, s, s.F); break;
        case EVOMOE_K_FFN_GEMM2: case EVOMOE_K_FFN_BWD_DX: t = rows_tile(c, s, s.d); break;
        case EVOMOE_K_FFN_BWD_DW2: t = wgrad_tile(c, s); break;
        default: return {};
    }
    return t == Tile::T64 ? FfnTile{64, 64, 4} : FfnTile{32, 32, 4};
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
    return wgrad_tile(c, s) == Tile::T64 ? run(launch<L_TN, E_WGRAD, 64>, 64) : run(launch<L_TN, E_WGRAD, 32>, 32);
}

}  // namespace evomoe
