// Expert FFNs on the bf16 matrix cores (EvoMoE Eq. ffn per expert over its ragged row range, and its
// backward).  One grouped-GEMM kernel template, v_mfma_f32_32x32x16_bf16, f32 accumulation:
//
//   NT  C[r,n] = sum_k A[arow(r),k] * W_g[n,k]      forward GEMMs (A rows optionally gathered by token)
//   NN  C[r,n] = sum_k A[r,k]       * W_g[k,n]      dH = dO W2,  dXp = dH W1
//   TN  C_g[m,n] = sum_{r in g} L[r,m] * R[rrow(r),n]   weight gradients (contraction over the ragged rows)
//
// Block = 4 waves (2 x 2) or 8 waves (4 x 2), block tile BM x BN, K slabs of BK, NSTAGE LDS stages filled by direct
// global->LDS loads (no staging registers) that run NSTAGE-1 slabs (two stages: one to one and a quarter) ahead of the MFMAs.  Operands whose
// contraction index is contiguous in memory sit in LDS as [row][BK k] with an XOR swizzle of the 16-byte
// chunks and are read with ds_read_b128; operands whose contraction index is the row index sit as
// [k][cols] with a swizzle of 32-byte blocks and are read with the transposing LDS load
// (ds_read_b64_tr_b16), so no operand is ever transposed in global memory.  The persistent grid walks
// the tiles in an XCD-aware order.  Epilogues (bias, activation, act'(H) product, accumulate) run in f32
// on a row-major copy of the accumulators staged through LDS, and leave with 16-byte stores.
#include <type_traits>

#include "ffn_internal.h"

namespace evomoe {

namespace {

enum { L_NT = 0, L_NN = 1, L_TN = 2 };
enum { E_HA = 0, E_BIAS = 1, E_ACTGRAD = 2, E_NONE = 3, E_WGRAD = 4 };

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int sum_ranges(int rows) { return max(1, min(kColsumSplit, (rows + 63) / 64)); }

struct GemmArgs {
    const bf16_t* A;  int64_t lda;      // NT/NN: A rows [*,K];  TN: L [P,M] (lda = M)
    const bf16_t* B;  int64_t ldb;      // NT: W_g [N,K] (ldb = K);  NN: W_g [K,N] (ldb = N);  TN: R [*,N] (ldb = N)
    int64_t b_group_stride;             // NT/NN: elements between two experts' weight matrices
    const int32_t* a_rows;              // NT: gather of A rows (or null)
    const int32_t* b_rows;              // TN: gather of R rows (or null)
    const int32_t* expert_offsets;
    int E;
    int64_t P_cap;
    int M, N, K;                        // M: TN only.  K: NT/NN only (TN contracts over the expert's rows)
    const float* bias;                  // [E,N] or null
    const bf16_t* Hin;                  // E_ACTGRAD: pre-activations [P,N]
    const float* row_scale;             // E_ACTGRAD: per-row factor applied in f32 before act' (or null)
    bf16_t* out1;                       // C (H for E_HA)
    bf16_t* out2;                       // E_HA: A = act(H)
    float* colpart;                     // E_ACTGRAD: column sums of C for each 64 rows, [part_row()][N] (or null)
    int act, accumulate;
    int col_group;                      // NT/NN: column tiles per group of the tile order (1 .. all of them)
};

// Row, in dH's table of column sums, of the first 64 rows of the expert whose rows begin at `begin`; its further ones follow.
// Expert g + 1 begins no earlier than expert g ends, and the table ends at P / 64 + E, whatever the tile.
__device__ __forceinline__ int part_row(int g, int begin) { return begin / 64 + g; }

// The last sums of both bias gradients, as further tiles behind the weight gradients' (TN launches).  The first tiles1
// (expert g = b / gx1, NW * 64 columns each): db1[g, n] (+)= sum over expert g's rows of the table of column sums
// written by the dH GEMM, in row order.  The rest: db2[i] (+)= sum over the row ranges of the column sums of dO, in their
// order.  Reproducible bit for bit.
struct BiasFinal {
    const float* part1; float* db1;     // [part_row()][N1] -> [E,N1]
    const float* part2; float* db2;     // [kColsumSplit][n2] -> [n2]
    size_t n2;                          // E * N2
    int N1, N2;
    int gx1, tiles1, tiles;             // column blocks per expert, tiles of db1, of both
    int accumulate;
    const int32_t* offsets;             // expert_offsets
};
__device__ __forceinline__ void bias_final_tile(const BiasFinal& q, int b, const int* offs, int nthr) {
    if (b >= q.tiles1) {
        const size_t i = (size_t)(b - q.tiles1) * nthr + threadIdx.x;
        if (i >= q.n2) return;
        const int g = (int)(i / (uint32_t)q.N2), ranges = sum_ranges(offs[g + 1] - offs[g]);
        float s = q.accumulate ? q.db2[i] : 0.f;
        for (int k0 = 0; k0 < ranges; k0 += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = q.part2[(size_t)min(k0 + u, ranges - 1) * q.n2 + i];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + u < ranges) s += v[u];
        }
        q.db2[i] = s;
        return;
    }
    const int g = b / q.gx1;
    const int n = (b % q.gx1) * nthr + threadIdx.x;
    if (n >= q.N1) return;
    const int rows = (offs[g + 1] - offs[g] + 63) / 64;
    const float* src = q.part1 + (int64_t)part_row(g, offs[g]) * q.N1 + n;
    float sum = q.accumulate ? q.db1[(int64_t)g * q.N1 + n] : 0.f;
    int i = 0;
    for (; i + 8 <= rows; i += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(int64_t)(i + u) * q.N1];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += v[u];
    }
    for (; i < rows; ++i) sum += src[(int64_t)i * q.N1];
    q.db1[(int64_t)g * q.N1 + n] = sum;
}

// Column sums of dO over every expert's rows (the first pass of db2): an expert's rows are cut into sum_ranges() ranges, 64 rows
// each as long as 32 ranges are enough; a tile leaves part[range][expert][column] for 2048 columns at most.
// Up to 32 MB of dO the tiles run behind dXp's, on the compute units first that have no dXp tile in the last round; beyond, in a
// launch of their own.  dXp and the sums, us, behind it / as two launches (the gap between them not counted): 1000 pairs of d = 136
// 8.6 / 14.0, 24 787 of d = 144 19 / 22, 8192 of d = 768, E = 64 97 / 104, 16 223 of d = 768, E = 16 94 / 103, 20 000 of d = 768, E = 32
// 122 / 124, 30 000 of d = 512, E = 8 84 / 81.  Above the line it depends on how many units idle: E = 16, d = 768 at 41, 56, 80 and
// 90 MB 159 / 167, 176 / 190, 259 / 276, 276 / 278, but E = 32 at 58 MB, where dXp's last round is full, 208 / 192, and 87 690 pairs of
// d = 1024 710 / 678.
struct ColumnSums {
    const bf16_t* M;  int N;            // dO [P,N]
    float* part;                        // [kColsumSplit][E][N]
    int wanted;
    int64_t tile_ns;                    // behind dXp: what a tile takes
};
// Tile b: column block fastest, then expert, then range.  The first 256 threads of a block: CL column lanes x 16 bytes are
// contiguous in a row, RL = 256 / CL row lanes take alternate rows, sixteen rows of loads in flight per thread (few waves share a
// unit behind dXp's tiles: with four, dXp and the sums took 314 us instead of 278 at 58 330 pairs); f32 sums, row lanes added in
// order.
__device__ __forceinline__ void colsum_tile(const ColumnSums& q, int b, int gx, int CL, const int* offs, int E, float* red) {
    const int RL = 256 / CL, g = b / gx % E, range = b / (gx * E);
    const int r0 = offs[g], r1 = offs[g + 1], ranges = sum_ranges(r1 - r0);
    if (range >= ranges) return;                                  // block-uniform
    const int cl = threadIdx.x % CL, rl = threadIdx.x / CL;
    const int n = (b % gx * CL + cl) * 8;
    const int per = (r1 - r0 + ranges - 1) / ranges, rb = r0 + range * per, re = min(r1, rb + per);
    const bool on = threadIdx.x < 256 && n < q.N && rl < RL;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (on) {
        constexpr int U = 16;
        const uint32_t step = (uint32_t)RL * q.N * 2;
        for (int r = rb + rl; r < re; r += U * RL) {
            const int k = (re - r + RL - 1) / RL;                 // this lane's rows that are left; beyond them the last one again
            const unsigned char* src = reinterpret_cast<const unsigned char*>(q.M + (size_t)r * q.N + n);
            u32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const u32x4*>(src + (size_t)min(u, k - 1) * step);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u < k) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) { acc[2 * e] += lo_bf16(v[u][e]); acc[2 * e + 1] += hi_bf16(v[u][e]); }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) red[(rl * CL + cl) * 8 + e] = acc[e];
    }
    __syncthreads();
    const int first = b % gx * CL * 8, columns = min(CL * 8, q.N - first);
    float* dst = q.part + ((size_t)range * E + g) * q.N + first;
    for (int c = threadIdx.x; c < columns; c += blockDim.x) {     // (by 256 / RL threads alone, eight columns each, it took most of
        float sum = 0.f;                                          // a tile's time for narrow layers, where RL is large)
#pragma unroll 4
        for (int l = 0; l < RL; ++l) sum += red[l * CL * 8 + c];
        dst[c] = sum;
    }
    __syncthreads();
}

__device__ __forceinline__ int colsum_lanes(int N) { return N / 8 > 128 ? 256 : N / 8; }
__global__ __launch_bounds__(256) void colsum_kernel(ColumnSums q, const int32_t* __restrict__ expert_offsets, int E, int64_t P_cap) {
    __shared__ int offs[65];
    __shared__ float red[256 * 8];
    if (threadIdx.x <= E) offs[threadIdx.x] = clamp_pairs(expert_offsets[threadIdx.x], P_cap);
    __syncthreads();
    const int CL = colsum_lanes(q.N);
    colsum_tile(q, blockIdx.x, (q.N / 8 + CL - 1) / CL, CL, offs, E, red);
}

// ---- LDS geometry -------------------------------------------------------------------------------
// Operand tiles are written by direct global->LDS loads (64 lanes x 16 B land contiguously), so a stage
// is a dense array and bank conflicts are avoided by permuting 16-byte chunks on the global side:
// (the LDS has 64 banks of 4 B: a ds_read_b128 is served 16 lanes = 256 B at a time, a 64-bit read 32 lanes)
//  * k-contiguous tile [R][BK k] bf16: chunk c of row r sits at chunk c ^ key(r), key = (r >> 1) & 7
//    (BK = 64, 128-byte rows) or (r >> 2) & 3 (BK = 32, 64-byte rows): sixteen consecutive rows reading
//    the same k-chunk with ds_read_b128 cover all sixteen 16-byte slots of the 256-byte bank window;
//  * k-strided tile [BK k][C cols] bf16, 2C B per row: 32-byte block b of row k sits at block
//    b ^ 2(k & 3): the transposing read ds_read_b64_tr_b16 has 32 lanes take two adjacent blocks from
//    four consecutive k rows, which then land in eight different 32-byte slots.
template <int LAYOUT, int BM, int BN, int BK, int NSTAGE, int NW = 4> struct Geo {
    static constexpr bool A_KC = (LAYOUT != L_TN);          // A operand k-contiguous?
    static constexpr bool B_KC = (LAYOUT == L_NT);
    static constexpr int A_BYTES = BM * BK * 2;
    static constexpr int B_BYTES = BN * BK * 2;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int WM = BM / (NW / 2), WN = BN / 2;       // waves: (NW/2) x 2
    static constexpr int EPI_LD = WN + 4;                    // f32 row stride of the staging copy
    // rows of the wave tile staged per pass: as many as fit next to nothing else in the operand stages
    static constexpr int EPI_ROWS = (WM >= 64 && NW * 64 * EPI_LD * 4 <= NSTAGE * STAGE + 8192) ? 64 : 32;
    static constexpr int EPI_BYTES = NW * EPI_ROWS * EPI_LD * 4;
    static constexpr int MAIN = (NSTAGE * STAGE > EPI_BYTES ? NSTAGE * STAGE : EPI_BYTES);
    static constexpr int SMEM = MAIN;
    // block key of row k of a k-strided tile with C columns (64 columns are only four blocks: two rows share a bank window)
    template <int C> __device__ static __forceinline__ int ks_key(int k) { return C >= 128 ? 2 * (k & 3) : (k & 2); }
};

// gelu(h) = max(h, -4.2) Phi(hc), Phi(hc) = 0.5 + hc Q(hc^2), hc = h clamped to |h| <= 4.2: degree-8 minimax fit of Q, |error of Phi| <
// 1.2e-5 -- below the resolution of the bf16 values it is multiplied into -- and no transcendental; 13 VALU instructions, which GEMM1's
// epilogue is bound by.  Beyond the fitted range the values stay within 2.5e-4 of the true ones for any h: -> h for large h (Phi(4.2) =
// 1 - 1.3e-5), -> -4.2 * 1.3e-5 for very negative ones.  (As max(h, 0) - |h| 2^p(|h|) GEMM1 of 58 330 pairs, d = 768 takes 322 us with p
// of degree four, whose errors are larger in places, and 326 with degree five, whose errors are smaller everywhere, 9.6e-7 at most,
// instead of 336; either rounds other values of A up or down, and with degree five dx at 16 223 pairs had an element at 1.37 times the
// comparison's bound, where 1.35 is allowed for.)
__device__ __forceinline__ float act_fwd_fast(float h, int act) {
    if (act == EVOMOE_RELU) return relu(h);
    const float hc = __builtin_amdgcn_fmed3f(h, -4.2f, 4.2f), u = hc * hc;
    float q = 5.998071484e-11f;
    q = fmaf(q, u, -5.633320033e-09f);
    q = fmaf(q, u, 2.343674907e-07f);
    q = fmaf(q, u, -5.760770819e-06f);
    q = fmaf(q, u, 9.457441047e-05f);
    q = fmaf(q, u, -1.114148065e-03f);
    q = fmaf(q, u, 9.830130264e-03f);
    q = fmaf(q, u, -6.636036932e-02f);
    q = fmaf(q, u, 3.989074528e-01f);
    asm("v_fmaak_f32 %0, %1, %2, 0x3f000000" : "=v"(q) : "v"(hc), "v"(q));     // 0.5 as a literal: half the time of v_fma_f32
    return __builtin_elementwise_maximum(h, -4.2f) * q;      // (a NaN stays one)
}
// gelu'(h) = Phi(h) + h phi(h) as 0.5 + hc*R(hc^2): it is odd about 1/2 as well, so one degree-10 minimax fit of the whole
// derivative takes the place of Phi and an exponential (14 VALU slots instead of 18 in an epilogue that they bound).  R is
// expanded about the middle of its range, where float32 Horner steps cancel least: |error| < 4.3e-6 in float32 for
// |h| <= 4.2 (Phi + h phi as it was taken before: 1.1e-5); beyond, the limits 1 and 0 to 2.4e-4, as before.
__device__ __forceinline__ float act_grad_fast(float h, int act) {
    if (act == EVOMOE_RELU) return h > 0.f ? 1.f : 0.f;
    // (a NaN stays one: v_med3_f32, an instruction instead of two, would take it for -4.2)
    const float hc = __builtin_elementwise_maximum(__builtin_elementwise_minimum(h, 4.2f), -4.2f);
    const float v = fmaf(hc, hc, -8.82f);
    float r = 1.802185568e-12f;
    r = fmaf(r, v, -4.374921728e-11f);
    r = fmaf(r, v, 5.102342655e-10f);
    r = fmaf(r, v, -7.310402536e-09f);
    r = fmaf(r, v, 1.216656924e-07f);
    r = fmaf(r, v, -1.580741672e-06f);
    r = fmaf(r, v, 1.681734851e-05f);
    r = fmaf(r, v, -1.568448874e-04f);
    r = fmaf(r, v, 1.322824408e-03f);
    r = fmaf(r, v, -1.166708504e-02f);
    r = fmaf(r, v, 1.727069277e-01f);
    asm("v_fmaak_f32 %0, %1, %2, 0x3f000000" : "=v"(r) : "v"(hc), "v"(r));     // 0.5 as a literal: half the time of v_fma_f32
    return r;
}

// 16 bytes per lane, global -> LDS, no registers in between: lane l's data lands at lds + 16*l.
// Written as inline assembly on purpose: the compiler cannot tell which LDS stage a load fills, so with
// its own intrinsic it guards every later LDS read (and every barrier) with s_waitcnt vmcnt(0), which
// serialises the prefetch pipeline.  Here the kernel counts its loads itself (wait_vmcnt below).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
// Eight floats -> bf16, one 16-byte store with the streaming (non-temporal) hint: the outputs are far larger
// than the L2 and are not read again by this kernel, while the operand panels they would evict are.
__device__ __forceinline__ void store_out(bf16_t* p, const float* in) {
    u32x4 v = {pack_bf16x2(in[0], in[1]), pack_bf16x2(in[2], in[3]), pack_bf16x2(in[4], in[5]), pack_bf16x2(in[6], in[7])};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}
// The same through a buffer descriptor of what exists of the output: lanes beyond it store nothing, without a branch around the
// store, so that a wave's stores can be counted.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const void* base, int bytes) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)((uint64_t)hi << 32 | lo), 0,
                                             __builtin_amdgcn_readfirstlane(bytes), 0x27000);
}
__device__ __forceinline__ void store_out(bf16_t* base, int bytes, uint32_t offset, const float* in) {
    u32x4 v = {pack_bf16x2(in[0], in[1]), pack_bf16x2(in[2], in[3]), pack_bf16x2(in[4], in[5]), pack_bf16x2(in[6], in[7])};
    __builtin_amdgcn_raw_buffer_store_b128(v, rows_of(base, bytes), offset, 0, 2);      // 2: non-temporal
}
__device__ __forceinline__ u32x4 load_in(const bf16_t* base, int bytes, uint32_t offset) {
    return __builtin_amdgcn_raw_buffer_load_b128(rows_of(base, bytes), offset, 0, 0);
}
__device__ __forceinline__ float load_in(const float* base, int bytes, uint32_t offset) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows_of(base, bytes), offset, 0, 0));
}
// The global address is a wave-uniform base (an SGPR pair) plus a 32-bit unsigned byte offset per lane.
__device__ __forceinline__ void load_to_lds(const unsigned char* base, uint32_t voff, const unsigned char* lds_wave_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(base), "s"(lds_addr(lds_wave_base)) : "m0", "memory");
}
// 4 bytes per lane in the same way: lane l's data lands at lds + 4*l.
__device__ __forceinline__ void load_dword_to_lds(const int32_t* base, uint32_t voff, const int* lds_wave_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(voff), "s"(base), "s"(lds_addr(lds_wave_base)) : "m0", "memory");
}
// Block barrier that orders LDS traffic only (global loads in flight stay in flight).
__device__ __forceinline__ void block_sync_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// s_waitcnt vmcnt(n) only (other counters left at their maxima)
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// What a launch carries besides its first problem (nothing else: the arguments of a launch are copied and read every time)
struct NoExtra {};
struct TnExtra { GemmArgs q1; BiasFinal bias; };
template <int LAYOUT, int EPI> struct Extra { using type = NoExtra; };
template <int EPI> struct Extra<L_TN, EPI> { using type = TnExtra; };
template <> struct Extra<L_NN, E_NONE> { using type = ColumnSums; };

template <int LAYOUT, int EPI, int BM, int BN, int BK, int NSTAGE, int WPE, int NW = 4>
__global__ __launch_bounds__(NW * 64, WPE) void grouped_gemm_bf16(GemmArgs q0, int tiles0, int tiles_all, typename Extra<LAYOUT, EPI>::type qx)
{
    // TN launches carry two independent problems (dW2 and dW1) in one grid, tiles [0, tiles0) and
    // [tiles0, tiles_all), which evens out the last round of the persistent schedule, and behind them the bias
    // gradients' last sums; other layouts use q0 only.
    using G = Geo<LAYOUT, BM, BN, BK, NSTAGE, NW>;
    constexpr int WM = G::WM, WN = G::WN;
    constexpr int TM = WM / 32, TN_ = WN / 32;               // MFMA tiles per wave
    constexpr int KS = BK / 16;                              // k-steps per slab
    constexpr int A_LD = G::A_BYTES / (NW * 1024), B_LD = G::B_BYTES / (NW * 1024);   // 1 KB load instructions per wave per slab
    constexpr int KC_CH = BK / 8, KC_RPI = 64 / KC_CH;       // k-contiguous: 16 B chunks per row, rows per instruction
    constexpr int A_CPR = BM / 8, A_RPI = 64 / A_CPR;        // k-strided A: 16 B chunks per k-row, k-rows per instruction
    constexpr int B_CPR = BN / 8, B_RPI = 64 / B_CPR;
    constexpr int NMF = TM * TN_, NFR = TM + TN_, NLD = A_LD + B_LD;
    constexpr bool EARLY = NSTAGE == 2;
    constexpr int EARLY_LD = NLD / 2;
    constexpr bool SPLIT_LD = NSTAGE >= 3;          // half of a slab's loads before the barrier, half after
    static_assert(BK == 32 || BK == 64, "slab");
    static_assert(NW == 4 || NW == 8, "waves");
    static_assert(WM % 32 == 0 && WN % 32 == 0 && A_LD >= 1 && B_LD >= 1 && NSTAGE >= 2 && KS % 2 == 0, "tile");
    static_assert((NSTAGE - 2) * NLD + (NSTAGE - 1) * 2 <= 63, "vmcnt range");

    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int offs[65];

    auto problem = [&](int second) -> const GemmArgs& {
        if constexpr (LAYOUT == L_TN) return second ? qx.q1 : q0;
        else return q0;
    };
    const int tid = threadIdx.x, lane_id = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);       // wave-uniform: lives in an SGPR
    const int wm = wave >> 1, wn = wave & 1;
    __shared__ int tstart[65];      // NT/NN: number of row tiles before each expert (tstart[E] = all of them)
    // TN: the R rows' numbers for the next 768 to 1024 k's of the tile, in a ring of pieces of 256, gathered or not: one LDS
    // read and a multiplication make a load's address.  (Loads of row numbers among the pipeline's own would make every slab wait for
    // memory twice; a dense copy of the gathered rows took a pass over them, 25 us of 47 with dO's column sums at 58 330
    // pairs, d = 768.)
    constexpr int RING = 1024, PIECE = 256;
    __shared__ int ring[LAYOUT == L_TN ? RING : 1];
    // Lane e of the first wave counts expert e's rows and row tiles; entries beyond the last expert are its end.  (One thread
    // that walked over the experts, and a walk from expert to expert to find a tile: 64 experts, 22 073 pairs, d = 512, GEMM1
    // 87.9 us, now 83.7; 16 experts 0.3 to 0.5 us more per launch.)
    if (wave == 0) {
        const int begin = clamp_pairs(q0.expert_offsets[min(lane_id, q0.E)], q0.P_cap),
                  end = clamp_pairs(q0.expert_offsets[min(lane_id + 1, q0.E)], q0.P_cap);
        if (lane_id == 0) offs[0] = begin;
        offs[lane_id + 1] = end;
        if (LAYOUT != L_TN) {
            int upto = (end - begin + BM - 1) / BM;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(upto, o, 64);
                if (lane_id >= o) upto += v;
            }
            if (lane_id == 0) tstart[0] = 0;
            tstart[lane_id + 1] = upto;
        }
    }
    __syncthreads();

    // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.
    // TN: renumber the blocks so that one XCD works on a run of consecutive tiles per round (the tiles of one
    // expert share its row range).
    // NT/NN: the tile sequence runs expert by expert, inside an expert column group by column group (col_group
    // column tiles whose weight panels fit the L2 together), inside a group row tile by row tile.  When the column
    // tiles are split into groups, every XCD takes one contiguous eighth of that sequence and walks it round by
    // round: the weight panels of a group are fetched into that XCD's L2 once and stay there while the expert's row
    // panels stream past them.
    const bool xcd_split = (gridDim.x & 7) == 0;
    int vblock = blockIdx.x;
    if (xcd_split) vblock = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    int seq = 0, seq_end = 0, seq_step = 0;
    if (LAYOUT != L_TN) {
        const int nct = (q0.N + BN - 1) / BN;
        const int total = tstart[q0.E] * nct;
        if (xcd_split && q0.col_group < nct) {
            const int x = blockIdx.x & 7;
            seq = (int)((int64_t)total * x / 8) + (blockIdx.x >> 3);
            seq_end = (int)((int64_t)total * (x + 1) / 8);
            seq_step = gridDim.x >> 3;
        } else {            // one group holds every column tile: per round, a run of consecutive tiles per XCD
            seq = vblock;
            seq_end = total;
            seq_step = gridDim.x;
        }
    }
    // A wave without an output (its 64 or 128 rows or its 128 columns do not exist) sits a 256x256 tile out: it fetches its share
    // of the operands and leaves the matrix pipes to the others.  In launches of less than three rounds it does not: there the
    // blocks that get ahead find no tile to take, and GEMM1 of 8192 pairs, d = 768, took 70 us instead of 64 (shorter gelu).
    // Where no more than half of the blocks have a tile in the last round, two blocks take each of those tiles, one for its
    // upper and one for its lower 128 rows (waves 0 .. 3, one per SIMD, or 4 .. 7): places [full, full + halves) of the
    // sequence are upper halves, the next ones lower halves.  Not GEMM1, whose epilogue is as long for one wave per SIMD as for
    // two (58 330 pairs, with the shorter gelu: 334 us, without 326).  us, before / now: weight gradients of d = 768, F = 3072, 16
    // experts (4.5 rounds),
    // 58 330 pairs 485 / 468, 8192 pairs 109 / 106; dH 16 223 pairs 128 / 122, d = 1024, 87 690 pairs 901 / 871; GEMM1 d = 512, 22 073
    // pairs (345 rows per expert) 98 / 88, d = 1024, 87 690 pairs 945 / 908.
    constexpr bool SIT_OUT = BM == 256 && BN == 256;
    constexpr bool HALVES = SIT_OUT && NW == 8 && EPI != E_HA;
    bool sit_rows = true;
    int halves = 0, full = LAYOUT == L_TN ? tiles_all : seq_end;
    if (SIT_OUT) {
        const int step = LAYOUT == L_TN ? (int)gridDim.x : seq_step;
        const int begin = LAYOUT == L_TN ? 0 : seq - (step == (int)gridDim.x ? vblock : (int)(blockIdx.x >> 3));
        const int rem = __builtin_amdgcn_readfirstlane((full - begin) % step);
        halves = HALVES && 2 * rem <= step ? rem : 0;
        sit_rows = full - begin >= 3 * step;
        full -= halves;
        seq_end += halves;
    }
    const int all_places = tiles_all + halves;      // TN

    // Where a tile lies: problem (TN), expert, origin, contraction range.  NT/NN: its place in the sequence; TN: its number.
    struct Tile { int second, g, row0, rows, m0, n0, kbeg, kend, half; };
    auto locate = [&](int at) {
        Tile t{};
        t.half = -1;
        if (SIT_OUT && at >= full) {
            t.half = at >= full + halves;
            at -= t.half ? halves : 0;
        }
        t.second = LAYOUT == L_TN && at >= tiles0;
        const GemmArgs& p = problem(t.second);
        const int nct = (p.N + BN - 1) / BN;
        if (LAYOUT == L_TN) {
            const int tile = t.second ? at - tiles0 : at, nmt = (p.M + BM - 1) / BM;
            t.g = tile / (nmt * nct);
            const int rem = tile % (nmt * nct);
            t.m0 = (rem / nct) * BM;
            t.n0 = (rem % nct) * BN;
            t.kbeg = offs[t.g];
            t.kend = offs[t.g + 1];
        } else {
            int e;                                               // (the lane's number: no register is kept for it)
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(e));
            const int first = tstart[e], next = tstart[e + 1], begin = offs[e], end = offs[e + 1];
            t.g = __popcll(__ballot(at >= next * nct));          // lane e looks at expert e: those that lie before the tile
            const int t0 = __builtin_amdgcn_readlane(first, t.g), nrt = __builtin_amdgcn_readlane(next, t.g) - t0,   // row tiles of this expert (>= 1 here)
                      o0 = __builtin_amdgcn_readlane(begin, t.g), o1 = __builtin_amdgcn_readlane(end, t.g);
            const int r = at - t0 * nct;                         // position inside the expert's nrt * nct tiles
            const int cgs = max(1, min(p.col_group, nct));       // column tiles per group
            const int cg = r / (nrt * cgs);
            const int r2 = r - cg * nrt * cgs;
            const int gc = min(cgs, nct - cg * cgs);             // column tiles of this group (the last may be short)
            const int rt_in = r2 / gc;
            t.n0 = (cg * cgs + (r2 - rt_in * gc)) * BN;
            t.row0 = o0 + rt_in * BM;
            t.rows = min(BM, o1 - t.row0);
            t.kend = p.K;
        }
        // the tile's coordinates came through LDS: tell the compiler they are wave-uniform (SGPRs)
        t.g = __builtin_amdgcn_readfirstlane(t.g);
        t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
        t.rows = __builtin_amdgcn_readfirstlane(t.rows);
        t.n0 = __builtin_amdgcn_readfirstlane(t.n0);
        t.kbeg = __builtin_amdgcn_readfirstlane(t.kbeg);
        t.kend = __builtin_amdgcn_readfirstlane(t.kend);
        t.half = __builtin_amdgcn_readfirstlane(t.half);
        return t;
    };

    // TN: piece number n of a tile's row numbers (waves 0 .. 3, 64 each), from the list or, without one, in order; beyond the
    // expert's rows its last one
    auto fetch_piece = [&](const Tile& t, int n) {
        const int kbeg = __builtin_amdgcn_readfirstlane(t.kbeg), klen = __builtin_amdgcn_readfirstlane(t.kend) - kbeg;
        if (LAYOUT != L_TN || wave >= 4 || n * PIECE >= klen) return;
        int lane_f = lane_id;
        asm volatile("" : "+v"(lane_f));
        const int kr = min(n * PIECE + wave * 64 + lane_f, klen - 1);
        int* at = ring + (LAYOUT == L_TN ? (uint32_t)(n * PIECE) % RING + wave * 64 : 0);
        const int32_t* list = problem(t.second).b_rows;
        if (list) load_dword_to_lds(list + kbeg, (uint32_t)kr * 4, at);
        else at[LAYOUT == L_TN ? lane_f : 0] = kr;
    };
    auto first_pieces = [&](const Tile& t) {
#pragma unroll
        for (int n = 0; n < RING / PIECE - 1; ++n) fetch_piece(t, n);
    };

    // PRE: the next tile's first slab is fetched under this tile's epilogue, into the stage that the epilogue does not use.
    constexpr bool PRE = LAYOUT != L_TN && EARLY && NW == 8;
    constexpr int PRE_STORES = WM / 4 * (EPI == E_HA ? 2 : 1);      // at least so many of a wave's stores follow that slab's loads
    static_assert(!PRE || (PRE_STORES <= 63 && WN == 128 && NW * 4096 <= G::STAGE), "epilogue beside a slab");
    int par = 0;                    // PRE: stage of the tile's first slab
    bool begun = false;             // PRE: ... is being fetched already; TN: the tile's first row numbers are
    bool stored = false;            // PRE: this wave has stored the previous tile
    Tile ahead{};
    // ---------------- global addresses: one scalar base per operand + 32-bit per-lane byte offsets ----
    // k-contiguous operand: offset of (row, chunk) at k = 0, one register per load instruction.
    // k-strided operand   : offset = k-row * row bytes + column bytes; every load instruction of a lane
    //                       has the same column, its k-row is kr0 + a constant.
    const unsigned char* a_base = nullptr;
    const unsigned char* b_base = nullptr;
    uint32_t a_off[G::A_KC ? A_LD : 1], b_off[G::B_KC ? B_LD : 1];
    uint32_t a_col = 0, b_col = 0;                    // k-strided: column byte offset
    int kc_chunk = 0, ksA_row = 0, ksB_row = 0;

    for (int vtile = vblock;; vtile += gridDim.x, seq += seq_step) {
        if constexpr (LAYOUT == L_TN) {
            if (vtile >= all_places) {
                if (vtile - all_places >= qx.bias.tiles) break;
                bias_final_tile(qx.bias, vtile - all_places, offs, NW * 64);
                continue;
            }
        }
        if (LAYOUT != L_TN && seq >= seq_end) break;
        const Tile t = (PRE || LAYOUT == L_TN) && begun ? ahead : locate(LAYOUT == L_TN ? vtile : seq);
        const GemmArgs& p = problem(t.second);
        auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };     // (known to be, not when it comes around the loop)
        const int g = uniform(t.g), row0 = uniform(t.row0), rows = uniform(t.rows), m0 = uniform(t.m0), n0 = uniform(t.n0),
                  kbeg = uniform(t.kbeg), kend = uniform(t.kend);
        const int half = uniform(t.half);
        const bool active = !SIT_OUT || ((half < 0 || half == wm / 2) &&
                                         (!sit_rows || (n0 + wn * WN < p.N && (LAYOUT == L_TN ? m0 + wm * WM < p.M : wm * WM < rows))));
        const int nslab = (kend - kbeg + BK - 1) / BK;
        const bool ragged = (kend - kbeg) % BK != 0;     // block-uniform: the last slab is partial

        // Everything below that depends on the lane is recomputed for every tile from an opaque copy of the lane
        // number: the values then die with the main loop instead of occupying registers through the epilogue.
        int lane_t = lane_id;
        asm volatile("" : "+v"(lane_t));
        const int lane = lane_t;
        // LDS byte offsets of this lane's operand fragments inside one stage (k-step 0), per MFMA tile
        int fa_off[TM], fb_off[TN_];
        const int s16 = lane & 15, l32 = lane & 31, kg = lane >> 5;
    #pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (G::A_KC) {
                fa_off[i] = (wm * WM + i * 32 + l32) * (BK * 2);     // row base; the swizzled chunk is added per k-step
            } else {
                const int lb = (wm * WM + i * 32 + ((lane >> 4) & 1) * 16) >> 4;       // logical 32 B block
                fa_off[i] = (kg * 8 + (s16 >> 2)) * (BM * 2) + ((lb ^ G::template ks_key<BM>(s16 >> 2)) << 5) + ((s16 & 3) << 3);
            }
        }
    #pragma unroll
        for (int j = 0; j < TN_; ++j) {
            if (G::B_KC) {
                fb_off[j] = (wn * WN + j * 32 + l32) * (BK * 2);
            } else {
                const int lb = (wn * WN + j * 32 + ((lane >> 4) & 1) * 16) >> 4;
                fb_off[j] = (kg * 8 + (s16 >> 2)) * (BN * 2) + ((lb ^ G::template ks_key<BN>(s16 >> 2)) << 5) + ((s16 & 3) << 3);
            }
        }
        // swizzle key of this lane's fragment rows (tile rows start at multiples of 32)
        const int sw = (BK == 64) ? ((l32 >> 1) & 7) : ((l32 >> 2) & 3);

        // This lane's role in the 1 KB load instruction number (wave + NW*i) of a tile (NW waves):
        //   k-contiguous: row (wave+NW i)*KC_RPI + lane/KC_CH, physical chunk lane%KC_CH -> logical chunk ^ key(row)
        //   k-strided   : k-row (wave+NW i)*RPI + lane/CPR, physical chunk lane%CPR -> logical chunk via block ^ (k & 3)
        // Rows / columns outside the tile are clamped onto valid ones (their products are never stored);
        // the tail of the contraction range is clamped too and then zeroed in LDS.
        auto tokens = [&](const Tile& t, const GemmArgs& p, int lane, uint32_t (&ar)[G::A_KC ? A_LD : 1]) {
            if (!G::A_KC) return;
#pragma unroll
            for (int i = 0; i < A_LD; ++i) {
                const int r = min((wave + NW * i) * KC_RPI + lane / KC_CH, t.rows - 1);
                ar[G::A_KC ? i : 0] = p.a_rows ? (uint32_t)p.a_rows[t.row0 + r] : (uint32_t)r;
            }
        };
        auto aim = [&](const Tile& t, const GemmArgs& p, int lane, const uint32_t (&ar)[G::A_KC ? A_LD : 1]) {
            const bf16_t* Bg = (LAYOUT == L_TN) ? p.B : p.B + (int64_t)t.g * p.b_group_stride;
            const int kc_row = lane / KC_CH;
            // key(row) of row (wave + NW i)*KC_RPI + kc_row does not depend on i
            const int kc_key = (BK == 64) ? ((4 * (wave & 1) + (kc_row >> 1)) & 7) : ((kc_row >> 2) & 3);
            kc_chunk = (lane % KC_CH) ^ kc_key;                               // logical 16 B chunk (8 k's)
            ksA_row = lane / A_CPR, ksB_row = lane / B_CPR;
            auto ks_col = [&](int pc, int key) { return ((((pc >> 1) ^ key) << 1) | (pc & 1)) * 8; };
            if (G::A_KC) {
                a_base = reinterpret_cast<const unsigned char*>(p.A) + (p.a_rows ? (int64_t)0 : (int64_t)t.row0 * p.lda * 2);
#pragma unroll
                for (int i = 0; i < A_LD; ++i) a_off[G::A_KC ? i : 0] = (ar[G::A_KC ? i : 0] * (uint32_t)p.lda + kc_chunk * 8) * 2;
            } else {
                a_base = reinterpret_cast<const unsigned char*>(p.A) + (int64_t)t.kbeg * p.lda * 2;
                a_col = 2 * min(t.m0 + ks_col(lane % A_CPR, G::template ks_key<BM>(wave * A_RPI + ksA_row)), p.M - 8);
            }
            if (G::B_KC) {
                b_base = reinterpret_cast<const unsigned char*>(Bg);
#pragma unroll
                for (int i = 0; i < B_LD; ++i) {
                    const int n = min(t.n0 + (wave + NW * i) * KC_RPI + kc_row, p.N - 1);
                    b_off[G::B_KC ? i : 0] = ((uint32_t)n * (uint32_t)p.ldb + kc_chunk * 8) * 2;
                }
            } else {
                b_base = reinterpret_cast<const unsigned char*>(Bg) + (p.b_rows ? (int64_t)0 : (int64_t)t.kbeg * p.ldb * 2);
                b_col = 2 * min(t.n0 + ks_col(lane % B_CPR, G::template ks_key<BN>(wave * B_RPI + ksB_row)), p.N - 8);
            }
        };
        if (!PRE || !begun) {
            uint32_t ar[G::A_KC ? A_LD : 1];
            tokens(t, p, lane, ar);
            aim(t, p, lane, ar);
        }
        const int klen = kend - kbeg;
        const uint32_t lda2 = (uint32_t)p.lda * 2, ldb2 = (uint32_t)p.ldb * 2;
        // TN: the R rows that this lane loads of the next slab to be issued, read from the ring a slab ahead
        uint32_t b_row[LAYOUT == L_TN ? B_LD : 1];
        const int* ring_lane = ring + (LAYOUT == L_TN ? wave * B_RPI + ksB_row : 0);
        auto rows_of_slab = [&](int slab) {
            if (LAYOUT != L_TN) return;
#pragma unroll
            for (int i = 0; i < B_LD; ++i) b_row[LAYOUT == L_TN ? i : 0] = (uint32_t)ring_lane[(uint32_t)(slab * BK) % RING + NW * B_RPI * i];
        };
        auto stage_of = [&](int slab) { return (PRE ? slab + par : slab) % NSTAGE; };
        // issue load instruction `idx` (A: 0..A_LD-1, then B) of slab `slab` into its stage; addresses
        // are clamped into the contraction range (a no-op except in the last, partial slab)
        auto issue_one = [&](int idx, int slab) {
            unsigned char* sa = smem + stage_of(slab) * G::STAGE + wave * 1024;
            const int kc_lim = 2 * (kend - 8 - kc_chunk * 8);    // k-contiguous: last in-range chunk start (bytes)
            unsigned char* sb = sa + G::A_BYTES;
            if (idx < A_LD) {
                const int i = idx;
                if (G::A_KC) {
                    load_to_lds(a_base, a_off[i] + (uint32_t)min(slab * (BK * 2), kc_lim), sa + i * (NW * 1024));
                } else {
                    const int kr = min(slab * BK + (wave + NW * i) * A_RPI + ksA_row, klen - 1);
                    load_to_lds(a_base, __umul24((uint32_t)kr, lda2) + a_col, sa + i * (NW * 1024));
                }
            } else {
                const int i = idx - A_LD;
                if (G::B_KC) {
                    load_to_lds(b_base, b_off[i] + (uint32_t)min(slab * (BK * 2), kc_lim), sb + i * (NW * 1024));
                } else {
                    const uint32_t kr = LAYOUT == L_TN ? b_row[i] : (uint32_t)min(slab * BK + (wave + NW * i) * B_RPI + ksB_row, klen - 1);
                    load_to_lds(b_base, __umul24(kr, ldb2) + b_col, sb + i * (NW * 1024));
                }
            }
        };
        auto issue = [&](int slab) {        // (PRE calls it for the next tile's first slab: the contraction range is the same)
#pragma unroll
            for (int idx = 0; idx < NLD; ++idx) issue_one(idx, slab);
        };
        // zero both operands beyond the end of the contraction range (last slab only; with one of them zero, an infinity in
        // the clamped elements of the other would make 0 * Inf = NaN of a result that is infinite)
        // (always the tile's last slab: its position comes from the tile, not from the loop counter, so that
        // no per-lane induction variable is carried through the main loop for this rare path)
        // Short loops and a fresh copy of the lane number: unrolled, the addresses of this rare path cost dXp 1-2 %.
        auto zero_tail = [&]() {
            const int slab = nslab - 1;
            int lane_z = lane_id;
            asm volatile("" : "+v"(lane_z));
            unsigned char* sa = smem + stage_of(slab) * G::STAGE + wave * 1024 + lane_z * 16;
            unsigned char* sb = sa + G::A_BYTES;
            const int left = klen - slab * BK;                    // k's of the last slab that exist
            const bool chunk_out = kc_chunk * 8 >= left;
            const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll 1
            for (int i = 0; i < A_LD; ++i)
                if (G::A_KC ? chunk_out : (wave + NW * i) * A_RPI + lane_z / A_CPR >= left)
                    *reinterpret_cast<u32x4*>(sa + i * (NW * 1024)) = z;
#pragma unroll 1
            for (int i = 0; i < B_LD; ++i)
                if (G::B_KC ? chunk_out : (wave + NW * i) * B_RPI + lane_z / B_CPR >= left)
                    *reinterpret_cast<u32x4*>(sb + i * (NW * 1024)) = z;
        };
        // operand fragment number f (A tiles 0..TM-1, then B tiles) of k-step ks of slab `slab`
        auto read_frag = [&](int f, int slab, int ks, bf16x8* fa, bf16x8* fb) {
            const unsigned char* sa = smem + stage_of(slab) * G::STAGE;
            const unsigned char* sb = sa + G::A_BYTES;
            if (f < TM) {
                const int i = f;
                if (G::A_KC) {
                    fa[i] = *reinterpret_cast<const bf16x8*>(sa + fa_off[i] + (((ks * 2 + kg) ^ sw) << 4));
                } else {
                    const unsigned char* q = sa + fa_off[i] + ks * 16 * (BM * 2);
                    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q));
                    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q + 4 * (BM * 2)));
                    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    fa[i] = __builtin_bit_cast(bf16x8, v);
                }
            } else {
                const int j = f - TM;
                if (G::B_KC) {
                    fb[j] = *reinterpret_cast<const bf16x8*>(sb + fb_off[j] + (((ks * 2 + kg) ^ sw) << 4));
                } else {
                    const unsigned char* q = sb + fb_off[j] + ks * 16 * (BN * 2);
                    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q));
                    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q + 4 * (BN * 2)));
                    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    fb[j] = __builtin_bit_cast(bf16x8, v);
                }
            }
        };

        f32x16 acc[TM][TN_];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN_; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        // One k-step: NMF MFMAs on fragments (FA, FB), in 8 groups; after each of the first four groups a
        // share of the next k-step's fragment reads (into NA, NB; slab nslb, k-step nks) is issued, and
        // after every group, optionally, a share of a later slab's global->LDS loads.  The scheduling
        // fences pin this order.
#define KSTEP(FA, FB, READ_NEXT, NA, NB, nslb, nks, LD_LO, LD_HI, lslab)                          \
    _Pragma("unroll") for (int q = 0; q < 8; ++q) {                                              \
        if (ACT)                                                                                 \
            _Pragma("unroll") for (int x = NMF * q / 8; x < NMF * (q + 1) / 8; ++x)              \
                acc[x / TN_][x % TN_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                 \
                    FA[x / TN_], FB[x % TN_], acc[x / TN_][x % TN_], 0, 0, 0);                   \
        if (ACT && READ_NEXT && q < 4) {                                                           \
            _Pragma("unroll") for (int f = NFR * q / 4; f < NFR * (q + 1) / 4; ++f)              \
                read_frag(f, nslb, nks, NA, NB);                                                 \
        }                                                                                        \
        _Pragma("unroll") for (int x = (LD_LO) + ((LD_HI) - (LD_LO)) * q / 8;                    \
                               x < (LD_LO) + ((LD_HI) - (LD_LO)) * (q + 1) / 8; ++x)             \
            issue_one(x, lslab);                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                       \
    }

        bf16x8 fa0[TM], fb0[TN_], fa1[TM], fb1[TN_];
        if (PRE) {
            // the first slab went out before the previous tile's epilogue; only that one's stores may still be in flight
            if (begun && stored) wait_vmcnt<PRE_STORES>(); else if (begun) wait_vmcnt<0>(); else issue(0), wait_vmcnt<0>();
            stored = active;
            block_sync_lds();           // it has landed, and the previous epilogue has left the other stage
            if (nslab > 1) {
#pragma unroll
                for (int idx = 0; idx < EARLY_LD; ++idx) issue_one(idx, 1);
            }
        } else {
            if (LAYOUT == L_TN && !begun) first_pieces(t);
            // Every load the compiler itself issued during the tile set-up (row indices, spill reloads) has to be
            // complete, and known to it as complete, before the pipeline starts: a wait that it places inside
            // the main loop for one of its own loads would also wait for the tile loads issued there.  (The same counter covers
            // the previous tile's stores: they are drained here as well.)
            __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
            // the previous tile's epilogue has left the LDS
            block_sync_lds();
        }
        if (nslab > 0) {
            // prologue: put NSTAGE-1 slabs in flight, wait for the first
            if (!PRE) {
#pragma unroll
                for (int s = 0; s < NSTAGE - 1; ++s) {
                    if (s < nslab) {
                        rows_of_slab(s);
                        issue(s);
                    }
                }
                rows_of_slab(NSTAGE - 1);
                if (EARLY && nslab > 1) {
#pragma unroll
                    for (int idx = 0; idx < EARLY_LD; ++idx) issue_one(idx, 1);
                    wait_vmcnt<EARLY_LD>();
                } else if (nslab >= NSTAGE - 1) wait_vmcnt<(NSTAGE - 2) * NLD>(); else wait_vmcnt<0>();
                block_sync_lds();
            }
            if (nslab == 1 && ragged) {
                zero_tail();
                block_sync_lds();
            }
#pragma unroll
            for (int f = 0; f < NFR; ++f) read_frag(f, 0, 0, fa0, fb0);
        }

        // Slab s: k-steps 0..KS-1 on stage s % NSTAGE.  Fragments of the next k-step are read while the
        // current one multiplies; loads of slab s+NSTAGE-1 go out under k-step 0 into the stage that slab
        // s-1 has finished with; before the last k-step the block makes sure slab s+1 has landed.
        auto slab_body = [&](int slab, auto loads_c, auto act_c) {
            constexpr bool LOADS = decltype(loads_c)::value, ACT = decltype(act_c)::value;     // ACT: not sitting out
            if constexpr (EARLY) {
                // two stages: a slab's first loads go out as soon as its stage is released, under the last k-step of
                // the slab before the one they are loaded under (LOADS: there is a slab + 2)
                KSTEP(fa0, fb0, true, fa1, fb1, slab, 1, EARLY_LD, NLD, slab + 1);
                if (KS == 4) {
                    KSTEP(fa1, fb1, true, fa0, fb0, slab, 2, 0, 0, 0);
                    KSTEP(fa0, fb0, true, fa1, fb1, slab, 3, 0, 0, 0);
                }
                wait_vmcnt<0>();
                block_sync_lds();
                if (!LOADS && slab + 2 == nslab && ragged) {      // (with LOADS there is a slab + 2)
                    zero_tail();
                    block_sync_lds();
                }
                KSTEP(fa1, fb1, true, fa0, fb0, slab + 1, 0, 0, LOADS ? EARLY_LD : 0, slab + 2);
                return;
            }
            // with three or more stages the second half of a slab's loads goes out after the barrier
            // (its stage was released one slab earlier), which keeps the load unit evenly busy
            constexpr int L0 = !LOADS ? 0 : (SPLIT_LD ? NLD / 2 : NLD), L1 = LOADS ? NLD : 0;
            KSTEP(fa0, fb0, true, fa1, fb1, slab, 1, 0, L0, slab + NSTAGE - 1);
            if (KS == 4) {
                KSTEP(fa1, fb1, true, fa0, fb0, slab, 2, 0, 0, 0);
                KSTEP(fa0, fb0, true, fa1, fb1, slab, 3, 0, 0, 0);
            }
            // everything issued after slab+1's loads may still be in flight
            if (LOADS) wait_vmcnt<(NSTAGE - 2) * NLD - (NLD - L0)>(); else wait_vmcnt<0>();
            block_sync_lds();
            if (!LOADS && slab + 2 == nslab && ragged) {      // (with LOADS there is a slab + 2)
                zero_tail();
                block_sync_lds();
            }
            KSTEP(fa1, fb1, true, fa0, fb0, slab + 1, 0, L0, L1, slab + NSTAGE - 1);
            if (LOADS && LAYOUT == L_TN) {
                rows_of_slab(slab + NSTAGE);
                if (slab * BK % PIECE == 0) fetch_piece(t, slab * BK / PIECE + RING / PIECE - 1);
            }
        };
        int slab = 0;
        // two blocks per CU: the wave that is feeding the matrix pipe goes ahead of its neighbour's epilogue
        if (WPE > 1) __builtin_amdgcn_s_setprio(1);
        auto slabs = [&](auto act_c) {
            for (; slab + NSTAGE - (EARLY ? 0 : 1) < nslab; ++slab) slab_body(slab, std::true_type{}, act_c);
            for (; slab + 1 < nslab; ++slab) slab_body(slab, std::false_type{}, act_c);
        };
        if (active) slabs(std::true_type{});
        else slabs(std::bool_constant<!SIT_OUT>{});
        float bias8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto load_bias = [&](int lane) {
            if (!((EPI == E_HA || EPI == E_BIAS) && LAYOUT != L_TN) || !p.bias) return;
            const float* from = p.bias + (int64_t)g * p.N + min(n0 + wn * WN + lane % (WN / 8) * 8, p.N - 8);
            const f32x4 b0 = *reinterpret_cast<const f32x4*>(from), b1 = *reinterpret_cast<const f32x4*>(from + 4);
            bias8[0] = b0.x; bias8[1] = b0.y; bias8[2] = b0.z; bias8[3] = b0.w;
            bias8[4] = b1.x; bias8[5] = b1.y; bias8[6] = b1.z; bias8[7] = b1.w;
        };
        uint32_t next_rows[G::A_KC ? A_LD : 1];
        if (PRE) {                 // the bias and the next tile's row numbers arrive under the last slab
            int lane_b = lane_id;
            asm volatile("" : "+v"(lane_b));
            load_bias(lane_b);
            begun = seq + seq_step < seq_end;
            if (begun) {
                ahead = locate(seq + seq_step);
                int lane_n = lane_id;
                asm volatile("" : "+v"(lane_n));
                tokens(ahead, p, lane_n, next_rows);
            }
        }
        if (nslab > 0 && active) {           // last slab: nothing left to fetch or to read ahead
            constexpr bool ACT = true;
            KSTEP(fa0, fb0, true, fa1, fb1, slab, 1, 0, 0, 0);
            if (KS == 4) {
                KSTEP(fa1, fb1, true, fa0, fb0, slab, 2, 0, 0, 0);
                KSTEP(fa0, fb0, true, fa1, fb1, slab, 3, 0, 0, 0);
            }
            KSTEP(fa1, fb1, false, fa0, fb0, 0, 0, 0, 0, 0);
        }
#undef KSTEP
        if (WPE > 1) __builtin_amdgcn_s_setprio(0);
        block_sync_lds();         // every wave is done reading operands: LDS becomes the epilogue's staging area
        if (PRE) {
            par = (par + nslab) & 1;
            int lane_n = lane_id;
            asm volatile("" : "+v"(lane_n));
            if (begun) {
                aim(ahead, p, lane_n, next_rows);
                __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0): known to have arrived, so that nothing waits for the slab with them
                issue(0);
            }
        }
        if (LAYOUT == L_TN) {     // ... and the ring with the row numbers is free for the next tile's
            begun = vtile + (int)gridDim.x < all_places;
            if (begun) {
                ahead = locate(vtile + gridDim.x);
                first_pieces(ahead);
            }
        }

        // ---------------- epilogue: stage f32 rows through LDS, finish row-major ----------------
        // Waves of 128 columns, NT/NN, one block per CU: eight rows at a time.  (With two blocks, 128x256 tiles of dH, the
        // steps took 3-5 % longer: one's epilogue is under the other's MFMAs anyway.  Waves of 64 columns have another layout and
        // keep the passes below.)  The rows of one step are written to 4 KB of the wave's own and read
        // back while the step before is computed and stored; the LDS works a wave's accesses off in order, so that this takes
        // no wait but the one for the data.  16-byte chunk c of row r lies at c ^ (c >> 4 & 1) ^ (r & 4 ? 8 : 0): the two
        // half-waves write to, and sixteen lanes read from, different banks.
        constexpr bool STEPS = LAYOUT != L_TN && WN == 128 && WPE == 1;
        if (!active) continue;
        if constexpr (STEPS) {
            int lane_e = lane_id;
            asm volatile("" : "+v"(lane_e));
            const int lane = lane_e, l32 = lane & 31, kg = lane >> 5, l16 = lane & 15, rq = lane >> 4;
            float* stg = reinterpret_cast<float*>(smem + (PRE ? (par ^ 1) * G::STAGE : 0)) + wave * 1024;
            float* put[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) put[j] = stg + kg * 512 + ((j ^ kg) * 32) + (j < 2 ? l32 : l32 ^ 4);
            const int get = rq * 128 + ((2 * l16) ^ (l16 >> 3)) * 4;
            const int col = n0 + wn * WN + l16 * 8;
            // this lane's place in four rows of the output; beyond them for a column that does not exist
            const uint32_t out_off = col < p.N ? (uint32_t)(rq * p.N + col) * 2 : 0x80000000u;
            if (!PRE) load_bias(lane);
            const bool scaled = EPI == E_ACTGRAD && p.row_scale;
            auto finish = [&](auto act_c) {
                constexpr int ACT = decltype(act_c)::value;
                f32x4 v0[2], v1[2];
                // H and the row weights, several steps ahead: four rows are done in less time than a load takes
                constexpr int DEPTH = 4;
                u32x4 hraw[DEPTH];
                float rsc[DEPTH];
                // column sums of the tile's valid rows (the bias gradient's share of this tile), f32.  Every tile adds the 64 rows
                // behind one row of the partial table in the same order -- rows 4 apart one after another, then (0 + 1) +
                // (2 + 3) -- so that the bias gradient does not depend on the tile that was picked.
                float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                static_assert(EPI != E_ACTGRAD || WM == 64, "column sums: one row of the table");
                // four rows: where they begin, and how many of them exist (a descriptor for so few keeps every offset in 32 bits)
                auto first = [&](int f) { return wm * WM + f * 4; };
                auto exist = [&](int f) { return max(0, __builtin_amdgcn_readfirstlane(min(4, rows - first(f)))); };
                auto begin = [&](int f) {
                    if (f % 2 == 0) {
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                            for (int j = 0; j < 4; ++j) put[j][rr * 128] = acc[f / 8][j][f / 2 % 4 * 4 + rr];
                    }
                    const int it = f % 2;
                    v0[it] = *reinterpret_cast<const f32x4*>(stg + (get ^ (it * 32)) + it * 512);
                    v1[it] = *reinterpret_cast<const f32x4*>(stg + (get ^ (it * 32 + 4)) + it * 512);
                };
                auto fetch = [&](int f) {
                    if (EPI != E_ACTGRAD || f >= WM / 4) return;
                    const int n = exist(f);
                    hraw[f % DEPTH] = load_in(p.Hin + (int64_t)(row0 + first(f)) * p.N, n * p.N * 2, out_off);
                    rsc[f % DEPTH] = load_in(p.row_scale + row0 + first(f), scaled ? n * 4 : 0, rq * 4);
                };
#pragma unroll
                for (int f = 0; f < DEPTH - 1; ++f) fetch(f);
                begin(0);
#pragma unroll
                for (int f = 0; f < WM / 4; ++f) {
                    const int it = f % 2, n = exist(f);
                    fetch(f + DEPTH - 1);
                    if (f + 1 < WM / 4) begin(f + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    const f32x4 x0 = v0[it], x1 = v1[it];
                    float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
                    const int64_t at = (int64_t)(row0 + first(f)) * p.N;
                    if (EPI == E_HA || EPI == E_BIAS) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] += bias8[q];
                    }
                    if (EPI == E_ACTGRAD) {
                        const u32x4 hw = hraw[f % DEPTH];
                        const float h[8] = {lo_bf16(hw.x), hi_bf16(hw.x), lo_bf16(hw.y), hi_bf16(hw.y),
                                            lo_bf16(hw.z), hi_bf16(hw.z), lo_bf16(hw.w), hi_bf16(hw.w)};
                        const float sc = scaled ? rsc[f % DEPTH] : 1.f;
                        const bool there = rq < n;      // (beyond the tile: its last row's products, which an infinity may be among)
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] *= sc * act_grad_fast(h[q], ACT);
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            cs[q] += there ? v[q] : 0.f;
                            asm volatile("" : "+v"(cs[q]));     // (added up at the end, where they are used, all the v's would be kept)
                        }
                    }
                    store_out(p.out1 + at, n * p.N * 2, out_off, v);
                    if (EPI == E_HA) {
                        float a[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) a[q] = act_fwd_fast(v[q], ACT);
                        store_out(p.out2 + at, n * p.N * 2, out_off, a);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (EPI == E_ACTGRAD && p.colpart) {
                    // the four lane groups hold different rows of the same columns: add them up, lane group 0 writes
                    // this wave's sums (rows wm*WM .. +WM-1 of the tile) as one row of the partial table
                    float* dst = p.colpart + (int64_t)(part_row(g, offs[g]) + (row0 - offs[g]) / 64 + wm) * p.N;
#pragma unroll
                    for (int o = 16; o < 64; o <<= 1)
#pragma unroll
                        for (int q = 0; q < 8; ++q) cs[q] += __shfl_xor(cs[q], o, 64);
                    if (rq == 0 && col < p.N && wm * 64 < rows) {      // (64 rows that do not exist have no row in the table)
                        *reinterpret_cast<f32x4*>(dst + col) = f32x4{cs[0], cs[1], cs[2], cs[3]};
                        *reinterpret_cast<f32x4*>(dst + col + 4) = f32x4{cs[4], cs[5], cs[6], cs[7]};
                    }
                }
            };
            // one branch per tile, not per value
            if ((EPI == E_HA || EPI == E_ACTGRAD) && p.act != EVOMOE_RELU) finish(std::integral_constant<int, EVOMOE_GELU_ERF>{});
            else finish(std::integral_constant<int, EVOMOE_RELU>{});
        } else
        {
        // (a fresh opaque copy of the lane number again: the epilogue's lane constants are not carried through
        //  the main loop either)
        int lane_e = lane_id;
        asm volatile("" : "+v"(lane_e));
        const int lane = lane_e, l32 = lane_e & 31, kg = lane_e >> 5;
        // acc[i][j][r] is C(row = i*32 + 8*(r/4) + 4*kg + r%4, col = j*32 + l32) of the wave tile.
        constexpr int ER = G::EPI_ROWS;
        float* stg = reinterpret_cast<float*>(smem) + wave * (ER * G::EPI_LD);
        constexpr int CPW = WN / 8;                 // 8-column chunks per wave-tile row
        constexpr int RPI = 64 / CPW;               // rows finished per instruction
        constexpr int NIT = ER / RPI;               // store instructions per pass
        constexpr int EPI_UNROLL = NIT <= 8 ? NIT : 4;
        // this lane's 8 columns are the same in every pass and iteration; loads that feed the epilogue are
        // issued ahead of the loop that stores (a load after a store of unknown aliasing is not hoisted)
        const int lc = (lane % CPW) * 8;
        const int col = n0 + wn * WN + lc;
        const int col_c = min(col, p.N - 8);
        if (!PRE) load_bias(lane);
        // E_ACTGRAD: column sums of the tile's valid rows (the bias gradient's share of this tile), f32.  Every tile adds
        // the 64 rows behind one row of the partial table in the same order -- rows 4 apart one after another, then
        // (0 + 1) + (2 + 3) -- so that the bias gradient does not depend on the tile that was picked.  Waves of 64 rows by
        // 128 columns meet their rows in that order and add in registers.  Where a lane's next row is 8 further on (64 columns),
        // the row in between lies in the wave's other half: exchanging halves gives each half four of the columns, with all
        // its rows (128x128 tile, 11000 pairs, d = 768, F = 3072: 96 us, through LDS 99.6).  Waves of 32 rows, two to a row
        // of the table, leave the finished values in the staging rows, and one of the two adds from there.
        constexpr bool SUM_REGS = WM >= 64 && RPI == 4, SUM_HALVES = WM >= 64 && RPI == 8;
        static_assert(EPI != E_ACTGRAD || SUM_REGS || SUM_HALVES || WM == ER, "column sums: one pass");
        float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int pass = 0; pass < WM / ER; ++pass) {
            u32x4 hraw[EPI == E_ACTGRAD ? NIT : 1];
            float rsc[EPI == E_ACTGRAD ? NIT : 1];
            if (EPI == E_ACTGRAD) {
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const int trow = min(wm * WM + pass * ER + it * RPI + lane / CPW, rows - 1);
                    hraw[it] = *reinterpret_cast<const u32x4*>(p.Hin + (int64_t)(row0 + trow) * p.N + col_c);
                    rsc[it] = p.row_scale ? p.row_scale[row0 + trow] : 1.f;
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int wrow = i * 32 + 8 * (r >> 2);           // + 4*kg + (r&3) < 8
                    if (wrow / ER != pass) continue;                  // compile-time after unrolling
#pragma unroll
                    for (int j = 0; j < TN_; ++j)
                        stg[(wrow % ER + 4 * kg + (r & 3)) * G::EPI_LD + j * 32 + l32] = acc[i][j][r];
                }
            // this wave's LDS writes are done -- and so are the loads issued above: waiting for them one by
            // one between the stores below would also wait for those stores (one counter covers both)
            if (pass == 0 || EPI == E_ACTGRAD) __builtin_amdgcn_s_waitcnt(0x0070);     // vmcnt(0) lgkmcnt(0)
            else __builtin_amdgcn_s_waitcnt(0xc07f);     // lgkmcnt(0) only: the first pass's stores stay in flight
            __builtin_amdgcn_wave_barrier();
#pragma unroll EPI_UNROLL
            for (int it = 0; it < NIT; ++it) {
                const int lr = it * RPI + lane / CPW;            // row inside the pass
                const int trow = wm * WM + pass * ER + lr;       // row inside the block tile
                const f32x4 v0 = *reinterpret_cast<const f32x4*>(stg + lr * G::EPI_LD + lc);
                const f32x4 v1 = *reinterpret_cast<const f32x4*>(stg + lr * G::EPI_LD + lc + 4);
                float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
                // the arithmetic runs for every lane (out-of-tile lanes on clamped addresses); only the
                // stores are predicated, so no wait for a load ends up inside divergent control flow
                if (LAYOUT == L_TN) {
                    const int m = m0 + trow;
                    const bool ok = col < p.N && m < p.M;
                    bf16_t* dst = p.out1 + ((int64_t)g * p.M + min(m, p.M - 1)) * p.N + col_c;
                    if (p.accumulate) {
                        float old[8];
                        Elem<bf16_t>::load_vec(dst, old);
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] += old[q];
                    }
                    if (ok) store_out(dst, v);
                } else {
                    const bool ok = col < p.N && trow < rows;
                    const int64_t grow = (int64_t)(row0 + min(trow, rows - 1));
                    if (EPI == E_HA || EPI == E_BIAS) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] += bias8[q];
                    }
                    if (EPI == E_ACTGRAD) {
                        const u32x4 hw = hraw[it];
                        const float h[8] = {lo_bf16(hw.x), hi_bf16(hw.x), lo_bf16(hw.y), hi_bf16(hw.y),
                                            lo_bf16(hw.z), hi_bf16(hw.z), lo_bf16(hw.w), hi_bf16(hw.w)};
                        // one branch per eight values (not per value): the eight polynomial chains interleave
                        const float sc = rsc[it];
                        if (p.act == EVOMOE_RELU) {
#pragma unroll
                            for (int q = 0; q < 8; ++q) v[q] *= sc * act_grad_fast(h[q], EVOMOE_RELU);
                        } else {
#pragma unroll
                            for (int q = 0; q < 8; ++q) v[q] *= sc * act_grad_fast(h[q], EVOMOE_GELU_ERF);
                        }
                        const bool there = trow < rows;     // rows beyond the tile repeat its last row
                        float s[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) s[q] = there ? v[q] : 0.f;
                        if (SUM_REGS) {
#pragma unroll
                            for (int q = 0; q < 8; ++q) cs[q] += s[q];
                        } else if (SUM_HALVES) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[q]), __float_as_uint(s[q + 4]), false, false);
                                cs[q] = (cs[q] + __uint_as_float(w[0])) + __uint_as_float(w[1]);
                            }
                        } else if (p.colpart) {
                            float* keep = stg + lr * G::EPI_LD + lc;
                            *reinterpret_cast<f32x4*>(keep) = f32x4{s[0], s[1], s[2], s[3]};
                            *reinterpret_cast<f32x4*>(keep + 4) = f32x4{s[4], s[5], s[6], s[7]};
                        }
                    }
                    if (ok) store_out(p.out1 + grow * p.N + col_c, v);
                    if (EPI == E_HA) {
                        float a[8];
                        if (p.act == EVOMOE_RELU) {
#pragma unroll
                            for (int q = 0; q < 8; ++q) a[q] = act_fwd_fast(v[q], EVOMOE_RELU);
                        } else {
#pragma unroll
                            for (int q = 0; q < 8; ++q) a[q] = act_fwd_fast(v[q], EVOMOE_GELU_ERF);
                        }
                        if (ok) store_out(p.out2 + grow * p.N + col_c, a);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (EPI == E_ACTGRAD && LAYOUT != L_TN) {
            if (p.colpart) {
                const int part = WM >= 64 ? wm : wm >> 1;         // which 64 rows of the tile
                const bool any = part * 64 < rows;                // (the others have no row in the table)
                float* dst = p.colpart + (int64_t)(part_row(g, offs[g]) + (row0 - offs[g]) / 64 + part) * p.N;
                if (SUM_REGS) {
                    // the four lane groups hold different rows of the same columns: add them up, lane group 0 writes
                    // this wave's sums (rows wm*WM .. +WM-1 of the tile) as one row of the partial table
#pragma unroll
                    for (int o = CPW; o < 64; o <<= 1)
#pragma unroll
                        for (int q = 0; q < 8; ++q) cs[q] += __shfl_xor(cs[q], o, 64);
                    if (lane < CPW && col < p.N && any) {
                        *reinterpret_cast<f32x4*>(dst + col_c) = f32x4{cs[0], cs[1], cs[2], cs[3]};
                        *reinterpret_cast<f32x4*>(dst + col_c + 4) = f32x4{cs[4], cs[5], cs[6], cs[7]};
                    }
                } else if (SUM_HALVES) {
                    const int half = (lane >> 5) * 4;             // columns 0..3 of the lane's eight, or 4..7
#pragma unroll
                    for (int o = CPW; o < 32; o <<= 1)
#pragma unroll
                        for (int q = 0; q < 4; ++q) cs[q] += __shfl_xor(cs[q], o, 64);
                    if ((lane & 31) < CPW && col < p.N && any)
                        *reinterpret_cast<f32x4*>(dst + col_c + half) = f32x4{cs[0], cs[1], cs[2], cs[3]};
                } else {
                    // lane = (chain, four columns); the upper wave's rows lie further on in the staging area
                    constexpr int CL = WN / 4;
                    const int chain = lane / CL, c4 = lane % CL * 4, n = n0 + wn * WN + c4;
                    block_sync_lds();
                    if (chain < 4 && !(wm & 1)) {
                        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int wave_of = i * 4 / WM;       // 1: the wave two further on (wave = 2 wm + wn)
                            sum += *reinterpret_cast<const f32x4*>(
                                stg + (wave_of * 2 * ER + i * 4 % WM + chain) * G::EPI_LD + c4);
                        }
#pragma unroll
                        for (int o = CL; o < 4 * CL; o <<= 1)
#pragma unroll
                            for (int q = 0; q < 4; ++q) sum[q] += __shfl_xor(sum[q], o, 64);
                        if (chain == 0 && n < p.N && any) *reinterpret_cast<f32x4*>(dst + n) = sum;
                    }
                }
            }
        }
        }
    }

    if constexpr (EPI == E_NONE) {
        const ColumnSums& qs = qx;
        if (!qs.wanted) return;
        const int CL = colsum_lanes(qs.N), gx = (qs.N / 8 + CL - 1) / CL;
        int most = sum_ranges(offs[lane_id + 1] - offs[lane_id]);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) most = max(most, __shfl_xor(most, o, 64));
        most = __builtin_amdgcn_readfirstlane(most);
        const int n = gx * q0.E * most;
        // A block without a tile of the last round takes as many column sums as a tile is worth, what is left is dealt to all.
        // (Where every XCD walks its own eighth of the sequence, these are blocks of every XCD.  Sums dealt to all there: dXp of
        // 8192 pairs, d = 768, 63.9 us, now 58.9.)
        const int total = tstart[q0.E] * ((q0.N + BN - 1) / BN), grid = gridDim.x, parts = seq_step == grid ? 1 : 8;
        const int busy = (total + parts - 1) / parts % seq_step, idle_each = busy ? seq_step - busy : 0, idle = idle_each * parts;
        const int place = parts == 1 ? vblock : (int)(blockIdx.x >> 3), first = (parts == 1 ? 0 : (int)(blockIdx.x & 7)) * idle_each + place - busy;
        // A sum takes 2 us and a ns for 22 bytes (twelve launches of d = 72 to 2048; us, measured / so: 19 KB 3.1 / 2.9, 33 KB 2.9 / 3.5,
        // 92 KB 5.9 / 6.2, 240 KB 12.9 / 12.9), a tile what the choice of tiles takes a round for.
        const int64_t sum_ns = 2000 + (int64_t)offs[q0.E] * qs.N * 2 / n / 22;
        const int fill = (int)min((int64_t)n, idle * (qs.tile_ns / sum_ns));
        __syncthreads();
        if (idle && place >= busy)
            for (int b = first; b < fill; b += idle) colsum_tile(qs, b, gx, CL, offs, q0.E, reinterpret_cast<float*>(smem));
        for (int b = fill + grid - 1 - vblock; b < n; b += grid) colsum_tile(qs, b, gx, CL, offs, q0.E, reinterpret_cast<float*>(smem));
    }
}

// Tile configurations.  BIG: one block per compute unit, two stages of 64 k, 256 accumulator registers per lane.
// BIG8: the same tile worked by eight waves (64x128 each, two per SIMD, 128 accumulator registers): the waves of a SIMD
// fill each other's stalls and share the epilogue, which is half of a short contraction's tile.
// A 64-wide slab takes whole 128-byte lines of a k-contiguous operand: with four stages of 32 k the L1 fetched every
// line twice (its other half was gone by the next slab; 2831 MB from the L2 per GEMM1 launch at 38 969 pairs, now 1470).
// BIG8 against 32-wide slabs: GEMM1 404 -> 366 us at d = 768, F = 3072, 58 330 pairs, 1603 -> 1473 at d = 1024, F = 4096, 131 072 pairs; BIG: GEMM2 270 -> 254 and 1026 -> 964 us, dXp 261 -> 252 and 994 -> 962 us.
// Where its time went with both waves of a SIMD in the epilogue at once (clocks per tile at d = 768): GEMM1 26.6 k main loop, 15 k
// epilogue, bound by its VALU instructions, 9 k waiting at the ends for loads and for each other; dH 22 k epilogue, H's loads one
// step ahead.  With the next tile's first slab and row numbers under the epilogue, the epilogue in steps that overlap and H four
// steps ahead: GEMM1 345 -> 339 us at d = 768, F = 3072, 58 330 pairs, 72 -> 68 at 8192 pairs, 980 -> 925 at d = 1024, F = 4096,
// 87 690 pairs; dH 381 -> 364, 74 -> 70, 925 -> 873.
// OCT: BIG8 with four stages of 32 k, for the weight gradients (k-strided operands are whole lines at any slab width).
// DUO: two blocks per compute unit (one's epilogue and stalls hide under the other's MFMAs).
// LAT: for launches with no more tiles than compute units and a long contraction: what counts then is how fast
// one block walks its K loop, and 64-wide slabs halve the number of load/barrier rounds of that walk.  LAT8: worked by
// eight waves, 2-7 % faster for dXp, the same for GEMM2.
// The smaller tiles are for launches whose 256-column tiles would leave compute units idle or be mostly padding
// (an expert with fewer than 128 rows): there the launch is as fast as its weights arrive, which takes blocks on every
// unit, each with several slabs of 64 k in flight.  MID: 128x128, two blocks per unit with two stages or (MID64) one with
// four.  SML: 64x128, two per unit.  TNY: 64x64, two per unit with four stages or (TNY3) three per unit with three.
struct CfgDuo { static constexpr int BM = 128, BN = 256, BK = 32, NSTAGE = 3, WPE = 2, NW = 4; };
struct CfgBig { static constexpr int BM = 256, BN = 256, BK = 64, NSTAGE = 2, WPE = 1, NW = 4; };
struct CfgBig8 { static constexpr int BM = 256, BN = 256, BK = 64, NSTAGE = 2, WPE = 1, NW = 8; };
struct CfgOct { static constexpr int BM = 256, BN = 256, BK = 32, NSTAGE = 4, WPE = 1, NW = 8; };
struct CfgLat { static constexpr int BM = 128, BN = 256, BK = 64, NSTAGE = 3, WPE = 1, NW = 4; };
struct CfgLat8 { static constexpr int BM = 128, BN = 256, BK = 64, NSTAGE = 3, WPE = 1, NW = 8; };
struct CfgMid { static constexpr int BM = 128, BN = 128, BK = 64, NSTAGE = 2, WPE = 2, NW = 4; };
struct CfgMid64 { static constexpr int BM = 128, BN = 128, BK = 64, NSTAGE = 4, WPE = 1, NW = 4; };
struct CfgSml { static constexpr int BM = 64, BN = 128, BK = 64, NSTAGE = 3, WPE = 2, NW = 4; };
struct CfgTny { static constexpr int BM = 64, BN = 64, BK = 64, NSTAGE = 4, WPE = 2, NW = 4; };
struct CfgTny3 { static constexpr int BM = 64, BN = 64, BK = 64, NSTAGE = 3, WPE = 3, NW = 4; };

template <int LAYOUT, int EPI, class Cfg>
hipError_t launch_gemm(const Ctx& c, const GemmArgs& a0, int64_t tiles0, int64_t tiles1, int64_t other_tiles,
                       const typename Extra<LAYOUT, EPI>::type& extra) {
    using G = Geo<LAYOUT, Cfg::BM, Cfg::BN, Cfg::BK, Cfg::NSTAGE, Cfg::NW>;
    auto kern = grouped_gemm_bf16<LAYOUT, EPI, Cfg::BM, Cfg::BN, Cfg::BK, Cfg::NSTAGE, Cfg::WPE, Cfg::NW>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, G::SMEM);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const int64_t cap = (int64_t)c.num_cu * Cfg::WPE, worst = tiles0 + tiles1 + other_tiles;
    const int grid = (int)(worst < cap ? worst : cap);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(Cfg::NW * 64), G::SMEM, c.stream, a0, (int)tiles0, (int)(tiles0 + tiles1), extra);
    return hipGetLastError();
}
// TN: two problems, and the bias gradients' last sums
template <class Cfg>
hipError_t launch_tn(const Ctx& c, const GemmArgs& a0, int64_t tiles0, const GemmArgs& a1, int64_t tiles1, BiasFinal b) {
    if (b.db1) { b.gx1 = (b.N1 + Cfg::NW * 64 - 1) / (Cfg::NW * 64); b.tiles1 = a0.E * b.gx1; }
    b.tiles = b.tiles1 + (b.db2 ? (int)((b.n2 + Cfg::NW * 64 - 1) / (Cfg::NW * 64)) : 0);
    return launch_gemm<L_TN, E_WGRAD, Cfg>(c, a0, tiles0, tiles1, b.tiles, TnExtra{a1, b});
}

// Worst-case number of row tiles (launch grids and tables are sized for P_cap rows) ...
template <class Cfg> int64_t row_tiles(const evomoe_shape& s) { return (s.P_cap + Cfg::BM - 1) / Cfg::BM + s.E; }
template <class Cfg> int64_t ctiles(int n) { return (n + Cfg::BN - 1) / Cfg::BN; }
template <class Cfg> int64_t mtiles(int m) { return (m + Cfg::BM - 1) / Cfg::BM; }
// ... and the number expected: the tile shape is chosen for the pair count the caller announced
// (evomoe_hint_pairs; the capacity when it announced none).  Any shape is correct for any pair count.
inline int64_t expected_pairs(const Ctx& c, const evomoe_shape& s) {
    return c.pair_hint > 0 && c.pair_hint < s.P_cap ? c.pair_hint : s.P_cap;
}
// About half a row tile per expert is padding; with fewer rows than that, every expert that has a row has a tile.
template <class Cfg> int64_t expected_row_tiles(const Ctx& c, const evomoe_shape& s) {
    const int64_t P = expected_pairs(c, s), spread = (P + Cfg::BM - 1) / Cfg::BM + s.E / 2, used = P < s.E ? P : s.E;
    return spread > used ? spread : used;
}

// Column tiles per group of the NT/NN tile order: as many weight panels (BN x K) as stay in one XCD's 4 MB L2 next to
// the row panels streaming past them; all of them when a row panel (BM x K) is itself so large (long contractions)
// that reading it once per group would cost more than re-reading the weights.
template <class Cfg> int col_group_for(int n, int k) {
    const int nct = (int)ctiles<Cfg>(n);
    if ((int64_t)Cfg::BM * k * 2 >= (1 << 20)) return nct;
    const int64_t fit = (int64_t)(2.4 * 1024 * 1024) / ((int64_t)Cfg::BN * k * 2);
    return (int)(fit < 1 ? 1 : (fit > nct ? nct : fit));
}

// Choice of tile shape per launch.  A persistent grid works through its tiles in rounds (one tile per resident
// block), so a launch takes about  fixed + rounds x (per_round + per_k x K / 1024)  microseconds: the finer tiles lose
// a little per flop but leave less of the last, partly filled round idle and waste less in the padding of each
// expert's last row tile.  Where several blocks share a compute unit and the last round does not give every unit all
// of them, that round is cheaper: 0.55 of a round at least, rising with the blocks per unit that it needs.  The numbers
// are fits to launches over d x F from 136 x 264 to 1024 x 4096, 1 to 64 experts and 1 to 90 000 pairs.  They price a last round
// that is worked in half tiles as a whole one.  Against every candidate measured, over 22 layers of 2000 to 87 690 pairs, the picks are
// slower than the best by (mean, most; %) GEMM1 2.6, 21, GEMM2 1.4, 14, dH 3.4, 23, dXp 1.0, 14, weight gradients 1.0, 5; the largest:
// dH and GEMM1 of 20 000 pairs, d = 256, F = 1024, E = 16 46 and 40 us where 128x128 and 64x128 tiles take 38 and 33, dH of 8192 pairs,
// d = 512, E = 64 62 (128x128: 52), dXp of 16 384, d = 768, E = 32 124 (128x256: 109).  dH of 8192 / 11 000 / 16 223 pairs, d = 768,
// E = 16, 256x256 by eight waves 70 / 93 / 120, 128x256 73 / 97 / 126, 128x128 74 / 92 / 126, picked the first, the third, the first.
// 256-column tiles alone were 40-190 % slower below about 200 rows per expert.  d = 768, F = 3072, 16 experts, us:
//            pairs     48     512    2048   8192   58330
//   GEMM1  256-wide    30     30     32     68     339          GEMM2  256-wide   37     40     45     53     254
//          picked      17     18     30     68     339                 picked     17     20     31     53     254
struct RoundTime { double fixed, per_round, per_k; };
template <class Cfg> double round_cost(const Ctx& c, int64_t tiles, double k, const RoundTime& t) {
    const int64_t slots = (int64_t)c.num_cu * Cfg::WPE, last = tiles % slots;
    double rounds = (double)(tiles / slots);
    if (last) rounds += 0.55 + 0.45 * (double)((last + c.num_cu - 1) / c.num_cu) / Cfg::WPE;
    return t.fixed + rounds * (t.per_round + t.per_k * k / 1024.0);
}
// A launch's candidates and their times.
template <class... Cfgs> struct Choice { RoundTime t[sizeof...(Cfgs)]; };
template <class Cfg> FfnTile tile_of() { return {Cfg::BM, Cfg::BN, Cfg::NW}; }
// The cheapest candidate's position; tiles(cfg): how many tiles of that shape the launch is expected to have.
template <class F, class... Cfgs> int cheapest(const Ctx& c, double k, const Choice<Cfgs...>& ch, F&& tiles) {
    int i = 0, best = 0;
    const double cost[] = {round_cost<Cfgs>(c, tiles(Cfgs{}), k, ch.t[i++])...};       // (a braced list: left to right)
    for (i = 1; i < (int)sizeof...(Cfgs); ++i)
        if (cost[i] < cost[best]) best = i;
    return best;
}
template <class... Cfgs> int cheapest_rows(const Ctx& c, const evomoe_shape& s, int n, int k, const Choice<Cfgs...>& ch) {
    return cheapest(c, k, ch, [&](auto cfg) { return expected_row_tiles<decltype(cfg)>(c, s) * ctiles<decltype(cfg)>(n); });
}
// Launches the cheapest of the candidates.
template <int LAYOUT, int EPI, class... Cfgs>
hipError_t launch_best(const Ctx& c, const evomoe_shape& s, GemmArgs& a, const Choice<Cfgs...>& ch, int64_t other_tiles = 0,
                       const typename Extra<LAYOUT, EPI>::type& extra = {}) {
    const int best = cheapest_rows(c, s, a.N, a.K, ch);
    hipError_t err = hipErrorInvalidValue;
    auto run = [&](auto cfg) {
        using Cfg = decltype(cfg);
        a.col_group = col_group_for<Cfg>(a.N, a.K);
        auto with = extra;
        if constexpr (EPI == E_NONE) with.tile_ns = (int64_t)(1000 * (ch.t[best].per_round + ch.t[best].per_k * a.K / 1024.0));
        err = launch_gemm<LAYOUT, EPI, Cfg>(c, a, row_tiles<Cfg>(s) * ctiles<Cfg>(a.N), 0, other_tiles, with);
    };
    int n = 0;
    (void)((n++ == best ? (run(Cfgs{}), true) : false) || ...);
    return err;
}
constexpr Choice<CfgBig8, CfgDuo, CfgMid, CfgSml, CfgTny3>
    kGemm1{{{0, 12.2, 21.9}, {0, 12.4, 27.8}, {0, 9.2, 12.8}, {2.5, 4.4, 10.0}, {3.0, 3.4, 9.0}}},
    kDh{{{11.0, 8.1, 28.3}, {0, 15.6, 26.0}, {0.3, 10.4, 13.2}, {2.6, 5.4, 10.7}, {2.8, 5.0, 8.8}}};
constexpr Choice<CfgBig, CfgLat, CfgMid64, CfgSml, CfgTny>
    kGemm2{{{0, 8.8, 20.5}, {0, 6.7, 12.5}, {0, 5.9, 7.8}, {0, 5.9, 10.5}, {0, 5.8, 6.1}}};
constexpr Choice<CfgBig, CfgLat8, CfgMid64, CfgSml, CfgTny>
    kDx{{{0, 8.6, 20.3}, {0, 6.2, 13.1}, {0, 5.8, 7.7}, {0, 5.9, 10.7}, {0, 5.6, 6.2}}};

// Weight gradients: the contraction runs over an expert's rows, P / E of them on average, and the tiles are those of the
// matrices.  256x256 tiles (eight waves) are the fastest per flop by far -- 8-29 % ahead of 128-row tiles wherever they
// fill the chip -- but layers with few experts or narrow matrices have fewer of them than compute units: there the finer
// tiles spread the same rows over more units.  The same model as for the other launches, fitted to 16 layers with 64 to
// 1024 columns, 1 to 64 experts and 32 to 16384 rows per expert; it picks the fastest of the three at each.  us
// (pairs, d, E, F):  777,136,7,264  8192,256,8,1024  16384,128,8,512  16384,256,1,1024  8192,512,4,2048  4096,1024,4,4096
//   256x256               9.7             27.8             44.7             290               53.0            69.8
//   128x128               6.7             16.4             19.8             108               44.8            96.5
//   64x64                 5.4             19.9             17.6              60               65.8           157
constexpr Choice<CfgOct, CfgMid64, CfgTny> kWgrad{{{4.0, 5.0, 24.0}, {2.5, 4.0, 8.0}, {2.0, 2.0, 7.6}}};
template <class Cfg> int64_t wgrad_tiles(const evomoe_shape& s, int m, int n) { return (int64_t)s.E * mtiles<Cfg>(m) * ctiles<Cfg>(n); }
int cheapest_wgrad(const Ctx& c, const evomoe_shape& s, bool w2, bool w1) {
    return cheapest(c, (double)expected_pairs(c, s) / s.E, kWgrad, [&](auto cfg) {
        using Cfg = decltype(cfg);
        return (w2 ? wgrad_tiles<Cfg>(s, s.d, s.F) : 0) + (w1 ? wgrad_tiles<Cfg>(s, s.F, s.d) : 0);
    });
}
hipError_t launch_wgrad(const Ctx& c, const evomoe_shape& s, const GemmArgs* w2, const GemmArgs* w1, const BiasFinal& bf) {
    GemmArgs none{};        // no weight gradient wanted: the launch carries the bias gradients only
    none.E = s.E; none.P_cap = s.P_cap; none.expert_offsets = bf.offsets;
    const GemmArgs& q0 = w2 ? *w2 : w1 ? *w1 : none;
    const GemmArgs& q1 = w1 ? *w1 : q0;
    auto run = [&](auto cfg) {
        using Cfg = decltype(cfg);
        return launch_tn<Cfg>(c, q0, w2 || w1 ? wgrad_tiles<Cfg>(s, q0.M, q0.N) : 0, q1,
                              w2 && w1 ? wgrad_tiles<Cfg>(s, q1.M, q1.N) : 0, bf);
    };
    switch (cheapest_wgrad(c, s, w2, w1)) {
        case 0: return run(CfgOct{});
        case 1: return run(CfgMid64{});
        default: return run(CfgTny{});
    }
}

template <class... Cfgs> FfnTile tile_at(const Choice<Cfgs...>&, int i) {
    const FfnTile t[] = {tile_of<Cfgs>()...};
    return t[i];
}

}  // namespace

size_t colsum_scratch_bytes(const evomoe_shape& s) {
    if (s.dtype != EVOMOE_BF16) return ((size_t)kF32ColsumSplit * s.E * (s.d + s.F) * sizeof(float) + 255) & ~(size_t)255;
    return (((size_t)kColsumSplit * s.E * s.d * sizeof(float) + 255) & ~(size_t)255) + dh_colpart_bytes(s);
}

// column sums of dH: a row of F floats for every 64 rows of an expert (part_row())
size_t dh_colpart_bytes(const evomoe_shape& s) {
    if (s.dtype != EVOMOE_BF16) return 0;
    return (((size_t)s.P_cap / 64 + s.E) * s.F * sizeof(float) + 255) & ~(size_t)255;
}

FfnTile mfma_ffn_tile(const Ctx& c, const evomoe_shape& s, int kernel) {
    switch (kernel) {
        case EVOMOE_K_FFN_GEMM1: return tile_at(kGemm1, cheapest_rows(c, s, s.F, s.d, kGemm1));
        case EVOMOE_K_FFN_GEMM2: return tile_at(kGemm2, cheapest_rows(c, s, s.d, s.F, kGemm2));
        case EVOMOE_K_FFN_BWD_DH: return tile_at(kDh, cheapest_rows(c, s, s.F, s.d, kDh));
        case EVOMOE_K_FFN_BWD_DX: return tile_at(kDx, cheapest_rows(c, s, s.d, s.F, kDx));
        case EVOMOE_K_FFN_BWD_DW2: return tile_at(kWgrad, cheapest_wgrad(c, s, true, true));
    }
    return {};
}

hipError_t mfma_ffn_fwd(const Ctx& c, const evomoe_shape& s, const void* x, const int32_t* pair_token,
                        const int32_t* expert_offsets, const void* W1, const float* b1, const void* W2,
                        const float* b2, void* H, void* A, void* O) {
    GemmArgs a{};
    a.expert_offsets = expert_offsets; a.E = s.E; a.P_cap = s.P_cap; a.act = s.act;
    hipError_t err;
    {   // H = X W1^T + b1, A = act(H)
        ProfScope ps(c, EVOMOE_K_FFN_GEMM1);
        a.A = (const bf16_t*)x; a.lda = s.d; a.a_rows = pair_token;
        a.B = (const bf16_t*)W1; a.ldb = s.d; a.b_group_stride = (int64_t)s.F * s.d;
        a.N = s.F; a.K = s.d; a.bias = b1; a.out1 = (bf16_t*)H; a.out2 = (bf16_t*)A;
        err = launch_best<L_NT, E_HA>(c, s, a, kGemm1);
        if (err != hipSuccess || !O) return err;      // O == nullptr: recomputation of H and A only
    }
    {   // O = A W2^T + b2
        ProfScope ps(c, EVOMOE_K_FFN_GEMM2);
        a.A = (const bf16_t*)A; a.lda = s.F; a.a_rows = nullptr;
        a.B = (const bf16_t*)W2; a.ldb = s.F; a.b_group_stride = (int64_t)s.d * s.F;
        a.N = s.d; a.K = s.F; a.bias = b2; a.out1 = (bf16_t*)O; a.out2 = nullptr;
        err = launch_best<L_NT, E_BIAS>(c, s, a, kGemm2);
    }
    return err;
}

hipError_t mfma_ffn_bwd(const Ctx& c, const evomoe_shape& s, const void* dO, const void* H, const void* A,
                        const void* x, const int32_t* pair_token, const int32_t* expert_offsets,
                        const void* W1, const void* W2, const void* dy, const float* pair_gate, void* dW1,
                        float* db1, void* dW2, float* db2, void* dXp, int accumulate, void* dH) {
    GemmArgs a{};
    a.expert_offsets = expert_offsets; a.E = s.E; a.P_cap = s.P_cap; a.act = s.act;
    hipError_t err;
    // workspace behind dH: [column sums of dO per row range][column sums of dH]
    float* scratch = reinterpret_cast<float*>(static_cast<char*>(dH) + dh_bytes(s));
    float* colpart = reinterpret_cast<float*>(static_cast<char*>(dH) + dh_bytes(s) + colsum_scratch_bytes(s) -
                                              dh_colpart_bytes(s));
    {   // dH = (dO W2) * act'(H); its epilogue also leaves the column sums of every 64 rows (for db1).
        // With dy and the pair weights at hand, dO W2 is taken as G_r * (dy[token(r)] W2): the rows of dy are
        // gathered on load and the weight is applied to the f32 accumulators, so that the rounding of the stored
        // dO (a product rounded to bf16) does not reach dH, dXp, dW1 and db1.
        ProfScope ps(c, EVOMOE_K_FFN_BWD_DH);
        const bool from_dy = dy && pair_gate && pair_token;
        a.A = (const bf16_t*)(from_dy ? dy : dO); a.lda = s.d; a.a_rows = from_dy ? pair_token : nullptr;
        a.row_scale = from_dy ? pair_gate : nullptr;
        a.B = (const bf16_t*)W2; a.ldb = s.F;
        a.b_group_stride = (int64_t)s.d * s.F; a.N = s.F; a.K = s.d; a.Hin = (const bf16_t*)H;
        a.out1 = (bf16_t*)dH; a.colpart = db1 ? colpart : nullptr;
        err = launch_best<L_NN, E_ACTGRAD>(c, s, a, kDh);
        a.colpart = nullptr; a.a_rows = nullptr; a.row_scale = nullptr;
        if (err != hipSuccess) return err;
    }
    ColumnSums sums{(const bf16_t*)dO, s.d, scratch, db2 != nullptr, 0};
    const int sum_tiles = kColsumSplit * s.E * ((s.d + 2047) / 2048);
    if (sums.wanted && expected_pairs(c, s) * s.d * 2 > 32000000) {
        ProfScope ps(c, EVOMOE_K_FFN_BWD_DB);
        hipLaunchKernelGGL(colsum_kernel, dim3(sum_tiles), dim3(256), 0, c.stream, sums,
                           expert_offsets, s.E, s.P_cap);
        sums.wanted = 0;
    }
    {   // dXp = dH W1, and the column sums of dO if they are few
        ProfScope ps(c, EVOMOE_K_FFN_BWD_DX);
        a.A = (const bf16_t*)dH; a.lda = s.F; a.B = (const bf16_t*)W1; a.ldb = s.d;
        a.b_group_stride = (int64_t)s.F * s.d; a.N = s.d; a.K = s.F; a.Hin = nullptr;
        a.out1 = (bf16_t*)dXp;
        err = launch_best<L_NN, E_NONE>(c, s, a, kDx, sums.wanted ? sum_tiles : 0, sums);
        if (err != hipSuccess) return err;
    }
    a.accumulate = accumulate;
    GemmArgs w2 = a, w1 = a;
    // dW2_g = dO_g^T A_g   [d,F]
    w2.A = (const bf16_t*)dO; w2.lda = s.d; w2.B = (const bf16_t*)A; w2.ldb = s.F;
    w2.M = s.d; w2.N = s.F; w2.out1 = (bf16_t*)dW2;
    // dW1_g = dH_g^T X_g   [F,d]; the token rows are gathered on load
    w1.A = (const bf16_t*)dH; w1.lda = s.F; w1.B = (const bf16_t*)x; w1.ldb = s.d; w1.b_rows = pair_token;
    w1.M = s.F; w1.N = s.d; w1.out1 = (bf16_t*)dW1;
    BiasFinal bf{};
    bf.part1 = colpart; bf.db1 = db1; bf.N1 = s.F;
    bf.part2 = scratch; bf.db2 = db2; bf.n2 = (size_t)s.E * s.d; bf.N2 = s.d; bf.accumulate = accumulate;
    bf.offsets = expert_offsets;
    if (!dW2 && !dW1 && !db1 && !db2) return hipSuccess;
    ProfScope ps(c, dW2 ? EVOMOE_K_FFN_BWD_DW2 : dW1 ? EVOMOE_K_FFN_BWD_DW1 : EVOMOE_K_FFN_BWD_DB);
    return launch_wgrad(c, s, dW2 ? &w2 : nullptr, dW1 ? &w1 : nullptr, bf);
}

}  // namespace evomoe
