// Projection GEMMs C = A[M,K] . W[N,K]^T (fp32 accumulation).
//
// bfloat16: v_mfma_f32_32x32x16_bf16 tiles, K in steps of 64, work items dealt to XCDs in
// contiguous runs so that blocks that share a weight tile reuse it from one L2.  Rows outside an
// operand read as zeros (buffer loads past their range), without branches.  Every kernel
// accumulates an output element with the same chain of MFMAs over k, so the choice of kernel and
// tile, which follows the sizes (launch_gemm, launch_gemm_qkv_rope), changes no bit.  They
// differ in how the operands travel and in what then bounds them:
//   gemm_stream_k         batches of a few row blocks (up to 64-256 rows): narrow tiles, up to
//                         eight steps of both operands on their way into LDS; latency, weights
//   gemm_lds_k            one to two rounds of 64 x 64 .. 128 x 128 tiles (the output projection
//                         and the fused QKV projection at 256-4096 rows, the split down
//                         projection at 385-640): direct to LDS, a ring of stages
//   gemm_wide_k           large batches: 256 x 256 .. 128 x 128 tiles, direct to LDS, fragments
//                         double-buffered in registers; the matrix pipes and the power limit
//   gemm_wide_persist_k   the same from two rounds of 256 x 256 tiles on, in work-groups that stay
//   gemm_bf16_k           register-staged, where none of these is faster: gate/up at 129-384 rows
//                         and its last columns beside a launch of whole rounds, the LM head at
//                         65-256 rows, and what lies between the other kernels' ranges in the
//                         down, fused QKV and widest unsplit projections
//
// float32: a plain LDS-tiled VALU kernel (the fp32 shapes are tiny correctness
// configurations).
//
// Epilogues: fp32 store (with split-K partials that the consumer sums in a
// fixed order, so results are deterministic) or SwiGLU, where the B tile pairs
// gate row j with up row j in the same lane and h = silu(gate) * up is stored in
// the model dtype.
#include "common.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace dash {

namespace {

constexpr int kBK = 64;
constexpr int kLdsStride = kBK + 8;  // bf16 elements per LDS row

DASH_DEV float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// ---- direct-to-LDS operand path ----------------------------------------------
// Operand tiles can also go from memory straight into LDS (buffer_load ... lds, 16 bytes
// per lane: one wave instruction fills 1 KB, 8 rows of 64 elements), through a ring of S
// stages: step k + S - 1 is in flight while step k is multiplied, without registers to
// hold it.  LDS rows are unpadded; the 16-byte chunks of a row are XOR-swizzled so that
// 16 consecutive rows read at one logical chunk hit 16 distinct 4-bank groups.
typedef __attribute__((address_space(3))) void lds_void;

template <int BM, int BN>
struct LdsStage {
    bf16_t a[BM * kBK];
    bf16_t b[BN * kBK];
};

DASH_DEV int lds_swizzle(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// Fill one stage: AI instructions of 8 A rows, then BI of 8 B rows.  kb is the step's
// byte offset along K; kb >= 2^31 (a step past the end) makes every in-range row read
// out of range, which returns zeros without touching memory, so every step issues the
// same instructions (padding rows, out of range already, may wrap to a harmless read).
template <int AI, int BI, int BM, int BN>
DASH_DEV void lds_dma_stage(LdsStage<BM, BN>& s, const bf16_t* A, int a_bytes, const bf16_t* W, int w_bytes,
                            const uint32_t* a_off, const uint32_t* b_off, uint32_t kb, int wave, int wpol) {
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, a_bytes, kBufferDword3);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(W), 0, w_bytes, kBufferDword3);
#pragma unroll
    for (int j = 0; j < AI; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void*)&s.a[(wave * AI + j) * 8 * kBK], 16, a_off[j] + kb, 0, 0,
                                                 0);
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        if (wpol)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (lds_void*)&s.b[(wave * BI + j) * 8 * kBK], 16, b_off[j] + kb,
                                                     0, 0, 2);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (lds_void*)&s.b[(wave * BI + j) * 8 * kBK], 16, b_off[j] + kb,
                                                     0, 0, 0);
    }
}

// s_waitcnt vmcnt(n) with the other counters left alone (n < 64)
template <int n>
DASH_DEV void wait_vmcnt() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
}

// s_waitcnt vmcnt(n) lgkmcnt(0): the vector-memory wait, and every LDS read this wave
// has issued has returned its data (n < 64)
template <int n>
DASH_DEV void wait_vmcnt_lds_reads() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | ((n >> 4) << 14));
}

// ---- epilogues shared by the GEMM kernels ------------------------------------
// acc[i * TN + j][r] of a wave holds row (r / 4) * 8 + (lane / 32) * 4 + r % 4 and column
// lane % 32 of its 32 x 32 block (i, j).

// NT: streaming stores, for an output larger than the last-level cache
template <int BM, int BN, int WGM, int WGN, bool NT = false>
DASH_DEV void store_f32_epilogue(const f32x16_t* acc, float* Cp, int M, int N, int ldc, int m0, int nt, int lane,
                                 int wr, int wc) {
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    const int rbase = (lane >> 5) * 4, ccol = lane & 31;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = nt * BN + wc * WN + j * 32 + ccol;
            if (n >= N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wr * WM + i * 32 + (r >> 2) * 8 + rbase + (r & 3);
                if (m >= M) continue;
                if constexpr (NT) __builtin_nontemporal_store(acc[i * TN + j][r], &Cp[(size_t)m * ldc + n]);
                else Cp[(size_t)m * ldc + n] = acc[i * TN + j][r];
            }
        }
}

// h = silu(gate) * up: a wave's column blocks hold TN/2 gate blocks, then the TN/2 up
// blocks of the same columns
template <int BM, int BN, int WGM, int WGN>
DASH_DEV void swiglu_epilogue(const f32x16_t* acc, bf16_t* H, int M, int N, int ldc, int m0, int nt, int lane, int wr,
                              int wc) {
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    const int rbase = (lane >> 5) * 4, ccol = lane & 31;
    const int ff = N >> 1;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) {
            const int col = nt * (BN / 2) + wc * (WN / 2) + j * 32 + ccol;
            if (col >= ff) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wr * WM + i * 32 + (r >> 2) * 8 + rbase + (r & 3);
                if (m < M) H[(size_t)m * ldc + col] = f2bf(silu(acc[i * TN + j][r]) * acc[i * TN + j + TN / 2][r]);
            }
        }
}

// The same h through LDS: each wave writes its values of the BM x BN/2 output tile into
// LDS (rows padded by 8 elements), then every thread stores whole 16-byte runs of 8
// columns, so a tile row leaves as full lines instead of 2-byte stores per element.
// Needs ldc and the tile's columns in whole runs of 8 and H 16-byte aligned (the caller
// checks); Hs is dead operand LDS of at least BM * (BN/2 + 8) elements, and every wave
// must be past its last read of it.
template <int BM, int BN, int WGM, int WGN>
DASH_DEV void swiglu_epilogue_lds(const f32x16_t* acc, bf16_t* Hs, bf16_t* H, int M, int N, int ldc, int m0, int nt,
                                  int tid, int wr, int wc) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int OW = BN / 2, OS = OW + 8;  // output tile width and LDS row stride (elements)
    constexpr int RUNS = BM * OW / 8;        // 16-byte runs in the tile
    static_assert(RUNS % NT == 0, "runs per thread");
    const int lane = tid & 63;
    const int rbase = (lane >> 5) * 4, ccol = lane & 31;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) {
            const int c = wc * (WN / 2) + j * 32 + ccol;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rr = wr * WM + i * 32 + (r >> 2) * 8 + rbase + (r & 3);
                Hs[rr * OS + c] = f2bf(silu(acc[i * TN + j][r]) * acc[i * TN + j + TN / 2][r]);
            }
        }
    __syncthreads();
    const int ff = N >> 1;
#pragma unroll
    for (int u = 0; u < RUNS / NT; ++u) {
        const int run = tid + u * NT, rr = run / (OW / 8), c8 = (run % (OW / 8)) * 8;
        const int m = m0 + rr, col = nt * OW + c8;
        if (m < M && col < ff)
            *reinterpret_cast<uint4*>(H + (size_t)m * ldc + col) = *reinterpret_cast<const uint4*>(Hs + rr * OS + c8);
    }
}

// QKV epilogue inputs (fetched before the main loop so that their latency, for the k / v
// tiles a dependent chain of position and slot, then the page table, hides behind it):
// per tile row its cache page (or -1) and key within the page (row_page / row_key, LDS);
// per thread the bias and the RoPE cosines / sines of its pairs.
template <int BM, int BN, int NT>
struct QkvPre {
    static constexpr int kRows = BM * (BN / 2) / NT;  // RoPE pairs per thread
    static constexpr int kRowsV = BM * BN / NT;       // v elements per thread
    float2 rope_cs[kRows > 0 ? kRows : 1];
    float bias_a = 0.f, bias_b = 0.f;
};

template <int BM, int BN, int NT>
DASH_DEV void qkv_prefetch(const QkvRopeArgs& qa, int M, int N, int m0, int nt, int tid, int* row_page, int* row_key,
                           QkvPre<BM, BN, NT>& pre) {
    static_assert(BN == 128, "the QKV epilogue works on 128-column tiles (whole heads)");
    static_assert(BM * (BN / 2) % NT == 0 && NT % (BN / 2) == 0, "RoPE pair mapping");
    static_assert(BM * BN % NT == 0 && NT % BN == 0, "v mapping");
    const KVGeom& g = qa.g;
    const int hd = g.head_dim, half = hd >> 1;
    const int lg_half = hd == 128 ? 6 : 5;  // head_dim is 64 or 128
    const int n0 = nt * BN;
    const int q_cols = qa.n_heads * hd, k_end_col = q_cols + g.n_kv * hd;
    if (n0 >= q_cols && tid < BM) {
        const int m = m0 + tid;
        int page = -1, key = 0;
        if (m < M) {
            const int p = qa.pos[m];
            page = kv_page_of(g, qa.page_table, qa.slot[m], p);
            key = p % g.page_size;
            if (page < 0 && n0 < k_end_col && qa.status) atomicOr(qa.status, 1u);
        }
        row_page[tid] = page;
        row_key[tid] = key;
    }
    if (n0 < k_end_col) {  // q / k tile: thread t takes pair t % (BN/2) of rows t / (BN/2) + u NT / (BN/2)
        const int pi = tid % (BN / 2), r0 = tid / (BN / 2);
        const int hl = pi >> lg_half, i = pi & (half - 1);
        const int n = n0 + hl * hd + i;
        pre.bias_a = bf2f(qa.bias[n]);
        pre.bias_b = bf2f(qa.bias[n + half]);
#pragma unroll
        for (int u = 0; u < QkvPre<BM, BN, NT>::kRows; ++u) {
            const int m = min(m0 + r0 + u * (NT / (BN / 2)), M - 1);
            pre.rope_cs[u] = *reinterpret_cast<const float2*>(qa.cs + ((size_t)m * half + i) * 2);
        }
    } else {  // v tile: thread t takes column t % BN of rows t / BN + u NT / BN
        const int n = n0 + tid % BN;
        pre.bias_a = n < N ? bf2f(qa.bias[n]) : 0.f;
    }
}

// Stage the fp32 tile in LDS (Cs: BM x (BN + 4) floats of LDS that no wave reads any
// more), then one thread per RoPE pair (q, k tiles) or v element adds the bias, rotates
// and writes q or the cache slot.
template <int BM, int BN, int WGM, int WGN>
DASH_DEV void qkv_epilogue(const f32x16_t* acc, float* Cs, const QkvRopeArgs& qa, int M, int N, int m0, int nt,
                           int tid, int wr, int wc, const int* row_page, const int* row_key,
                           const QkvPre<BM, BN, 64 * WGM * WGN>& pre) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int CS = BN + 4;
    constexpr int kRows = QkvPre<BM, BN, NT>::kRows, kRowsV = QkvPre<BM, BN, NT>::kRowsV;
    const int lane = tid & 63;
    const int rbase = (lane >> 5) * 4, ccol = lane & 31;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                Cs[(wr * WM + i * 32 + (r >> 2) * 8 + rbase + (r & 3)) * CS + wc * WN + j * 32 + ccol] = acc[i * TN + j][r];
    __syncthreads();
    const KVGeom& g = qa.g;
    const int hd = g.head_dim, half = hd >> 1;
    const int lg_half = hd == 128 ? 6 : 5, lg_hd = lg_half + 1;  // head indices by shifts, not divisions
    const int n0 = nt * BN;
    const int q_cols = qa.n_heads * hd, k_end = q_cols + g.n_kv * hd;
    if (n0 < k_end) {
        const int pi = tid % (BN / 2), r0 = tid / (BN / 2);
        const int hl = pi >> lg_half, i = pi & (half - 1);
        const int c = hl * hd + i, n = n0 + c;
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int rl = r0 + u * (NT / (BN / 2)), m = m0 + rl;
            if (m >= M) continue;
            const float a = Cs[rl * CS + c] + pre.bias_a;
            const float b = Cs[rl * CS + c + half] + pre.bias_b;
            float lo, hi;
            rope_pair(a, b, pre.rope_cs[u].x, pre.rope_cs[u].y, lo, hi);
            if (n < q_cols) {
                bf16_t* q = qa.q_out + ((size_t)m * qa.n_heads + (n >> lg_hd)) * hd;
                q[i] = f2bf(lo);
                q[i + half] = f2bf(hi);
            } else if (row_page[rl] >= 0) {
                bf16_t* kb = qa.pool + kv_block(g, qa.layer, row_page[rl], (n - q_cols) >> lg_hd, 0);
                // cache appends are non-temporal stores (see the v append below)
                __builtin_nontemporal_store(f2bf(lo), &kb[k_index_bf16(g, row_key[rl], i)]);
                __builtin_nontemporal_store(f2bf(hi), &kb[k_index_bf16(g, row_key[rl], i + half)]);
            }
        }
    } else {
        const int c = tid % BN, r0 = tid / BN;
        const int n = n0 + c, jj = n - k_end;
#pragma unroll
        for (int u = 0; u < kRowsV; ++u) {
            const int rl = r0 + u * (NT / BN), m = m0 + rl;
            if (m >= M || n >= N || row_page[rl] < 0) continue;
            const float v = Cs[rl * CS + c] + pre.bias_a;
            bf16_t* vb = qa.pool + kv_block(g, qa.layer, row_page[rl], jj >> lg_hd, 1);
            // A decode step writes one key per row: 2 bytes into each of the 16-byte groups
            // of 8 keys, lines that later steps read from memory anyway.  Non-temporal
            // stores keep these partial lines out of L2: measured 8% less QKV time and 2%
            // less decode-attention time at 1.5B, 1024 sequences.
            __builtin_nontemporal_store(f2bf(v), &vb[v_index_bf16(g, row_key[rl], jj & (hd - 1))]);
        }
    }
}

// The register-staged kernel: a workgroup of WGM x WGN waves owns a BM x BN output tile; a step
// goes through registers into a double-buffered LDS tile, its loads PD steps ahead of the
// multiply.  On gfx950 the 32x32x16 bf16 MFMA sustains about twice the rate of 16x16x32
// (measured: ~2.1 vs ~1.24 PFLOP/s with register-only operands), so every kernel
// here uses 32 x 32 output blocks.  Operand layout (per 16-wide k-step): lane l
// holds row (l % 32) and k (l / 32) * 8 .. +8; output register i of lane l is
// row (i / 4) * 8 + (l / 32) * 4 + i % 4, column l % 32.
// LDS tiles are row-major with rows padded to 72 elements (fragment reads of 16
// consecutive rows hit distinct banks); global loads fill full 128-byte rows.
template <int BM, int BN, int WGM, int WGN, int PD, int EPI, int WPOL = 0>
__global__ void __launch_bounds__(64 * WGM * WGN)
gemm_bf16_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, void* __restrict__ C, int M, int N, int K,
             int ldc, int m_tiles, int n_tiles, int nt0, int kps, size_t split_stride, QkvRopeArgs qa) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int A_CH = BM * 8 / NT, B_CH = BN * 8 / NT;  // 16-byte chunks per thread per k-step
    static_assert(A_CH >= 1 && B_CH >= 1 && BM * 8 % NT == 0 && BN * 8 % NT == 0, "tile / thread mismatch");
    static_assert(TM >= 1 && TN >= 1, "wave tile smaller than one MFMA block");
    static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "SwiGLU pairs gate/up blocks inside a wave");
    static_assert(EPI != EPI_QKV_ROPE || BN == 128, "the QKV epilogue works on 128-column tiles (whole heads)");
    __shared__ __attribute__((aligned(16))) bf16_t As[2][BM * kLdsStride];
    __shared__ __attribute__((aligned(16))) bf16_t Bs[2][BN * kLdsStride];

    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int mt = w % m_tiles;
    const int rest = w / m_tiles;
    const int nt = nt0 + rest % n_tiles;  // a launch may cover the column tiles from nt0 on
    const int split = rest / n_tiles;
    const int m0 = mt * BM;
    const int k_begin = split * kps;
    const int k_end = min(K, k_begin + kps);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave / WGN, wc = wave % WGN;

    // Operands are read with buffer loads: a row outside the operand gets a byte
    // offset past the buffer's extent, which the hardware returns as zeros, so the
    // loads need no branches and the compiler keeps PD k-steps of them in flight.
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(A), 0, (int)((size_t)M * K * 2), kBufferDword3);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(W), 0, (int)((size_t)N * K * 2), kBufferDword3);
    constexpr uint32_t kOut = 0x80000000u;
    uint32_t a_off[A_CH];
    int a_lds[A_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        const int idx = tid + i * NT, row = idx >> 3, kc = idx & 7;
        const int m = m0 + row;
        a_off[i] = m < M ? (uint32_t)(((size_t)m * K + kc * 8) * 2) : kOut;
        a_lds[i] = row * kLdsStride + kc * 8;
    }
    uint32_t b_off[B_CH];
    int b_lds[B_CH];
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
        const int idx = tid + i * NT, row = idx >> 3, kc = idx & 7;
        int n;
        bool ok;
        if (EPI == EPI_SWIGLU) {
            // a wave's N range holds WN/2 gate rows then the WN/2 up rows of the same columns
            const int ff = N >> 1;
            const int wcol = row / WN, rr = row % WN;
            const int j = nt * (BN / 2) + wcol * (WN / 2) + (rr % (WN / 2));
            ok = j < ff;
            n = rr < WN / 2 ? j : ff + j;
        } else {
            n = nt * BN + row;
            ok = n < N;
        }
        b_off[i] = ok ? (uint32_t)(((size_t)n * K + kc * 8) * 2) : kOut;
        b_lds[i] = row * kLdsStride + kc * 8;
    }

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    uint4 ra[PD][A_CH], rb[PD][B_CH];
    auto load = [&](int st, int k0) {
        const uint32_t kb = (uint32_t)k0 * 2;
#pragma unroll
        for (int i = 0; i < A_CH; ++i)
            ra[st][i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsA, a_off[i] + kb, 0, 0));
#pragma unroll
        for (int i = 0; i < B_CH; ++i)
            rb[st][i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsW, b_off[i] + kb, 0, WPOL));
    };
    auto store = [&](int st, int buf) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) *reinterpret_cast<uint4*>(&As[buf][a_lds[i]]) = ra[st][i];
#pragma unroll
        for (int i = 0; i < B_CH; ++i) *reinterpret_cast<uint4*>(&Bs[buf][b_lds[i]]) = rb[st][i];
    };
    const int frow = lane & 31, fk = (lane >> 5) * 8;
    auto compute = [&](int buf) {
        // let the scheduler interleave LDS reads with the MFMAs (measured: 4-10% faster,
        // same results); the 256x256 tile keeps the variant that does not spill
        if constexpr (BM * BN >= 256 * 256) __builtin_amdgcn_iglp_opt(1);
        else __builtin_amdgcn_iglp_opt(0);
#pragma unroll
        for (int ks = 0; ks < kBK; ks += 16) {
            bf16x8_t af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *reinterpret_cast<const bf16x8_t*>(&As[buf][(wr * WM + i * 32 + frow) * kLdsStride + ks + fk]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bfr[j] = *reinterpret_cast<const bf16x8_t*>(&Bs[buf][(wc * WN + j * 32 + frow) * kLdsStride + ks + fk]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
    };

    // QKV epilogue inputs, fetched before the main loop so that their latency hides behind it
    [[maybe_unused]] __shared__ int row_page[EPI == EPI_QKV_ROPE ? BM : 1], row_key[EPI == EPI_QKV_ROPE ? BM : 1];
    [[maybe_unused]] QkvPre<BM, BN, NT> pre;
    if constexpr (EPI == EPI_QKV_ROPE) qkv_prefetch<BM, BN, NT>(qa, M, N, m0, nt, tid, row_page, row_key, pre);

    const int n_k = (k_end - k_begin + kBK - 1) / kBK;
#pragma unroll
    for (int p = 0; p < PD; ++p) load(p, k_begin + p * kBK);
    store(0, 0);
    __syncthreads();
    for (int kt = 0; kt < n_k; kt += PD) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            const int k = kt + u;
            // register stage u held step k (already in LDS): refill it with step k + PD
            load(u, k_begin + (k + PD) * kBK);
            if (k < n_k) compute(k & 1);
            if (k + 1 < n_k) store((u + 1) % PD, (k + 1) & 1);
            __syncthreads();
        }
    }

    if constexpr (EPI == EPI_QKV_ROPE) {
        // the fp32 tile is staged in the B operand LDS (dead after the loop's last barrier)
        static_assert(BM * (BN + 4) * 4 <= (int)sizeof(Bs), "C tile must fit the B operand LDS");
        qkv_epilogue<BM, BN, WGM, WGN>(&acc[0][0], reinterpret_cast<float*>(&Bs[0][0]), qa, M, N, m0, nt, tid, wr, wc,
                                       row_page, row_key, pre);
    } else if constexpr (EPI == EPI_STORE_F32) {
        store_f32_epilogue<BM, BN, WGM, WGN>(&acc[0][0], reinterpret_cast<float*>(C) + split * split_stride, M, N, ldc,
                                             m0, nt, lane, wr, wc);
    } else {
        static_assert(EPI == EPI_SWIGLU, "unknown epilogue");
        static_assert(BM * (BN / 2 + 8) <= (int)(sizeof(As) / sizeof(bf16_t)), "h tile must fit the A operand LDS");
        // whole 16-byte runs: ldc, the output width and the base all multiples of 8 elements
        if (((ldc | (N >> 1)) & 7) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0)
            swiglu_epilogue_lds<BM, BN, WGM, WGN>(&acc[0][0], &As[0][0], reinterpret_cast<bf16_t*>(C), M, N, ldc, m0, nt,
                                                  tid, wr, wc);
        else
            swiglu_epilogue<BM, BN, WGM, WGN>(&acc[0][0], reinterpret_cast<bf16_t*>(C), M, N, ldc, m0, nt, lane, wr, wc);
    }
}

// The same product with the direct-to-LDS operand path: S LDS stages, one barrier per
// k-step.  At step k a wave waits until its own part of step k has landed and its own
// reads of step k - 1's stage have returned; the barrier then guarantees every wave's
// part and that no wave still reads step k - 1's stage, which is refilled with step
// k + S - 1, and step k is multiplied.  The wait for the reads matters: a copy into LDS
// is written whenever its data comes back from memory, in no order with LDS reads other
// waves have issued but not completed, so without it a slow read could see the next
// step's data.  (That happened with two decode steps running at once on two streams:
// 32-row blocks of some rows' outputs changed from run to run.)  Each
// stage is its own LDS variable, so the compiler lets the loads of the other stages stay
// in flight while a stage is read.  Same fragments, same MFMA order as gemm_bf16_k:
// identical results.  Measured on the 1.5B decode shapes at 1024 rows (weights cold):
// the output projection 14.7 -> 10.6 us, the QKV projection 15.5 -> 11.5 us with
// 128 x 64 tiles; gate/up, down and the LM head gain nothing (their per-CU rate stays
// at ~30% of the MFMA peak either way: a step's fragments are read right before the MFMAs that
// use them); their large batches run on gemm_wide_k, which reads them a slice ahead.
template <int BM, int BN, int WGM, int WGN, int S, int EPI, int WPOL = 0>
__global__ void __launch_bounds__(64 * WGM * WGN)
gemm_lds_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, void* __restrict__ C, int M, int N, int K,
           int ldc, int m_tiles, int n_tiles, int kps, size_t split_stride, QkvRopeArgs qa) {
    constexpr int NT = 64 * WGM * WGN, NW = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int AI = BM / 8 / NW, BI = BN / 8 / NW;  // 1 KB load instructions per wave per k-step
    constexpr int DPS = AI + BI;
    static_assert(AI >= 1 && BI >= 1 && BM / 8 % NW == 0 && BN / 8 % NW == 0, "load split");
    static_assert(S >= 3 && S <= 4, "stages");
    static_assert(TM >= 1 && TN >= 1, "wave tile smaller than one MFMA block");
    static_assert(EPI == EPI_STORE_F32 || EPI == EPI_QKV_ROPE, "epilogue");
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st0;
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st1;
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st2;
    __shared__ __attribute__((aligned(1024))) LdsStage<(S > 3 ? BM : 8), (S > 3 ? BN : 8)> st3;

    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int mt = w % m_tiles;
    const int rest = w / m_tiles;
    const int nt = rest % n_tiles;
    const int split = rest / n_tiles;
    const int m0 = mt * BM;
    const int k_begin = split * kps;
    const int k_end = min(K, k_begin + kps);
    const int n_k = (k_end - k_begin) / kBK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WGN, wc = wave % WGN;
    const int a_bytes = (int)((size_t)M * K * 2), w_bytes = (int)((size_t)N * K * 2);

    // lane l of load instruction j fills LDS chunk l % 8 of row l / 8 of its 8-row group:
    // it loads the logical chunk that the swizzle puts there
    constexpr uint32_t kOut = 0x80000000u;
    uint32_t a_off[AI], b_off[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        const int row = (wave * AI + j) * 8 + (lane >> 3);
        const int m = m0 + row;
        a_off[j] = m < M ? (uint32_t)(((size_t)m * K + k_begin + lds_swizzle(row, lane & 7) * 8) * 2) : kOut;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        const int row = (wave * BI + j) * 8 + (lane >> 3);
        const int n = nt * BN + row;
        b_off[j] = n < N ? (uint32_t)(((size_t)n * K + k_begin + lds_swizzle(row, lane & 7) * 8) * 2) : kOut;
    }

    [[maybe_unused]] __shared__ int row_page[EPI == EPI_QKV_ROPE ? BM : 1], row_key[EPI == EPI_QKV_ROPE ? BM : 1];
    [[maybe_unused]] QkvPre<BM, BN, NT> pre;
    if constexpr (EPI == EPI_QKV_ROPE) qkv_prefetch<BM, BN, NT>(qa, M, N, m0, nt, tid, row_page, row_key, pre);

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int frow = lane & 31, fhalf = lane >> 5;
    auto compute = [&](const LdsStage<BM, BN>& sg) {
#pragma unroll
        for (int ks = 0; ks < kBK / 16; ++ks) {
            bf16x8_t af[TM], bfr[TN];
            const int c = ks * 2 + fhalf;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wr * WM + i * 32 + frow;
                af[i] = *reinterpret_cast<const bf16x8_t*>(&sg.a[row * kBK + (lds_swizzle(row, c) << 3)]);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row = wc * WN + j * 32 + frow;
                bfr[j] = *reinterpret_cast<const bf16x8_t*>(&sg.b[row * kBK + (lds_swizzle(row, c) << 3)]);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
    };
    auto stage = [&](int i) -> LdsStage<BM, BN>& {
        if (i == 0) return st0;
        if (i == 1) return st1;
        if constexpr (S > 3) {
            if (i == 3) return st3;
        }
        return st2;
    };
    auto step_bytes = [&](int k) { return k < n_k ? (uint32_t)k * kBK * 2 : 0x80000000u; };
#pragma unroll
    for (int p = 0; p < S - 1; ++p)
        lds_dma_stage<AI, BI>(stage(p), A, a_bytes, W, w_bytes, a_off, b_off, step_bytes(p), wave, WPOL);
    // one k-step from stage ST (the stage index is a constant in every expansion)
#define DASH_LDS_STEP(ST, KK)                                                                               \
    do {                                                                                                   \
        const int k_ = (KK);                                                                               \
        wait_vmcnt_lds_reads<(S - 2) * DPS>();                                                             \
        __builtin_amdgcn_s_barrier();                                                                      \
        lds_dma_stage<AI, BI>(stage(((ST) + S - 1) % S), A, a_bytes, W, w_bytes, a_off, b_off,              \
                              step_bytes(k_ + S - 1), wave, WPOL);                                         \
        compute(stage(ST));                                                                                \
    } while (0)
    int k = 0;
    for (; k + S <= n_k; k += S) {
        DASH_LDS_STEP(0, k);
        DASH_LDS_STEP(1, k + 1);
        DASH_LDS_STEP(2, k + 2);
        if constexpr (S > 3) DASH_LDS_STEP(3, k + 3);
    }
    if (k < n_k) DASH_LDS_STEP(0, k++);
    if (k < n_k) DASH_LDS_STEP(1, k++);
    if constexpr (S > 3) {
        if (k < n_k) DASH_LDS_STEP(2, k++);
    }
#undef DASH_LDS_STEP

    if constexpr (EPI == EPI_QKV_ROPE) {
        // the fp32 tile is staged in LDS of its own (a stage is too small for it)
        __shared__ __attribute__((aligned(16))) float cstage[BM * (BN + 4)];
        wait_vmcnt<0>();  // the out-of-range loads of the steps past the end still write their stage
        qkv_epilogue<BM, BN, WGM, WGN>(&acc[0][0], cstage, qa, M, N, m0, nt, tid, wr, wc, row_page, row_key, pre);
    } else {
        store_f32_epilogue<BM, BN, WGM, WGN>(&acc[0][0], reinterpret_cast<float*>(C) + split * split_stride, M, N, ldc,
                                             m0, nt, lane, wr, wc);
        wait_vmcnt<0>();  // the out-of-range loads of the steps past the end still write their stage
    }
}

// ---- wide tiles ---------------------------------------------------------------
// The large-batch kernel (prefill, teacher forcing, wide decode batches): WGM x WGN waves of
// TM x TN 32 x 32 blocks, operands direct to LDS in two stages of 64-deep tiles, fragments
// double-buffered in registers.  A k-step is four clusters of TM x TN MFMAs; each cluster
// multiplies one 16-deep slice while the next slice's fragments are read, and the stage
// barrier sits before the last cluster: by then every wave has read all of the step's stage
// (its last fragments are in registers) and its own part of the next stage has landed, so
// the last cluster runs beside the first fragment reads of the next stage and the loads of
// step k + 2 into the stage just finished.  The instruction mix of every cluster is pinned
// (one MFMA, one LDS read, one load, ...): left to itself the compiler bunches the reads
// (3-5% slower).
//
// Eight waves of 128 x 64 on a 256 x 256 tile: each fragment feeds four (two) MFMAs, so LDS
// reads take ~770 cycles of the 2060 MFMA cycles of a step; two waves per SIMD fill each
// other's barrier waits (four waves of 128 x 128, one per SIMD, 1-8% slower; sixteen waves
// of 64 x 64 with register-staged operands, the earlier kernel, 10-20% slower).  Gate/up
// of the 1.5B shape at 16,384 rows (in work-groups that stay) runs at 1294 TFLOP/s with the MFMA
// pipes 71% busy and the clock down to 1.73 GHz (MFMA counters): the power limit, not the pipe,
// is next.  What a shape loses beyond that is per
// tile (load latency before the first step, the output after the last).  Stages of 32-deep
// half lines (four or five of them in flight) were 5-10% slower, and touching the lines of
// later steps (one dword per 64 bytes) 6-12%: the vector memory path, 64 bytes a cycle
// and CU, is half busy already, so requests cost more than the latency they would hide.
// Where a launch has at most one tile per CU nothing hides a late load, and half-size tiles with
// three stages in flight win (256 x 128; the weights come from HBM there).
// Same fragments and MFMA order as the other kernels: identical bits.

// Tile order: blocks of gm tile rows, column by column inside a block, so that the ~32
// tiles an XCD works on at a time span a near-square patch and share operand lines in its
// L2 (rows fastest over all of M re-read the left operand from beyond L2 for every column:
// gate/up at 16384 rows 847 us against 701-737 us with 4-6 rows a block).
DASH_DEV void wide_tile_of(int w, int m_tiles, int n_tiles, int gm, int& mt, int& nt) {
    const int per = gm * n_tiles, g = w / per, r = w - g * per;
    const int rows = min(gm, m_tiles - g * gm);
    mt = g * gm + r % rows;
    nt = r / rows;
}

// Cache page and key of every tile row (QKV epilogue), and per 32-row block whether its
// rows are 32 consecutive keys of one page starting at a multiple of 32 (prefill of whole
// pages): their V values then form whole 16-byte groups.
template <int BM>
struct WideQkvRows {
    int page[BM], key[BM], run[BM / 32];
};

template <int BM>
DASH_DEV void wide_qkv_rows(const QkvRopeArgs& qa, int M, int m0, int tid, WideQkvRows<BM>& rows) {
    if (tid >= BM) return;
    const int m = m0 + tid;
    int page = -1, key = -1;
    if (m < M) {
        const int p = qa.pos[m];
        page = kv_page_of(qa.g, qa.page_table, qa.slot[m], p);
        key = p % qa.g.page_size;
        if (page < 0 && qa.status) atomicOr(qa.status, 1u);
    }
    rows.page[tid] = page;
    rows.key[tid] = key;
    const int lane = tid & 63, first = lane & 32;
    const int page0 = __shfl(page, first, 64), key0 = __shfl(key, first, 64);
    const bool in_run = page >= 0 && page == page0 && key0 % 32 == 0 && key == key0 + (lane & 31);
    const uint64_t all = __ballot(in_run);
    if ((lane & 31) == 0) rows.run[tid >> 5] = (uint32_t)(all >> first) == 0xFFFFFFFFu;
}

// Bias, RoPE and the KV append straight from the accumulators: a wave's 128 columns are
// whole heads, and the two halves of a RoPE pair sit in the same lane and register of
// column blocks two (head dim 128) or one (64) apart.  Rotated q and k leave through LDS of
// the wave's own (hs: 32 rows of kQkvRow elements), 16 bytes a lane: q rows are contiguous,
// and so are 8 dims of a key in the K block.  (With 2-byte stores per element the 1.5B
// projection of 16,384 rows took 117 us instead of 90.)  The appends are plain stores: as
// non-temporal ones, as in qkv_epilogue, a decode step of 2048 rows (3B) took the same time
// (its attention, which reads them next, 149.9-150.6 against 150.1 us).
constexpr int kQkvRow = 128 + 8;

template <int BM, int WM, int TM>
DASH_DEV void wide_qkv_epilogue(const f32x16_t (&acc)[TM][4], const QkvRopeArgs& qa, int M, int N, int m0, int n0,
                                int wr, int lane, const WideQkvRows<BM>& rows, bf16_t* hs) {
    const KVGeom& g = qa.g;
    const int hd = g.head_dim, half = hd >> 1, lg_hd = hd == 128 ? 7 : 6;
    const int col = lane & 31, rbase = (lane >> 5) * 4;
    const int q_cols = qa.n_heads * hd, k_end = q_cols + g.n_kv * hd;
    if (n0 >= N) return;
    float bias[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bias[j] = bf2f(qa.bias[n0 + j * 32 + col]);
    if (n0 < k_end) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int b0 = wr * WM + i * 32;  // first tile row of the block
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int d = hd == 128 ? p * 32 + col : col;         // pair (d, d + half) of the head
                bf16_t* hp = hs + (hd == 128 ? d : p * 64 + d);       // its column among the wave's 128
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rr = (r >> 2) * 8 + rbase + (r & 3);
                    const size_t m = min(m0 + b0 + rr, M - 1);
                    const float2 cs = *reinterpret_cast<const float2*>(qa.cs + (m * half + d) * 2);
                    const float a = hd == 128 ? acc[i][p][r] + bias[p] : acc[i][2 * p][r] + bias[2 * p];
                    const float b = hd == 128 ? acc[i][p + 2][r] + bias[p + 2] : acc[i][2 * p + 1][r] + bias[2 * p + 1];
                    float lo, hi;
                    rope_pair(a, b, cs.x, cs.y, lo, hi);
                    hp[rr * kQkvRow] = f2bf(lo);
                    hp[rr * kQkvRow + half] = f2bf(hi);
                }
            }
            wave_lds_fence();
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int rr = u * 4 + (lane >> 4), c8 = (lane & 15) * 8, m = m0 + b0 + rr;
                if (m >= M) continue;
                const uint4 v = *reinterpret_cast<const uint4*>(hs + rr * kQkvRow + c8);
                if (n0 < q_cols) {
                    *reinterpret_cast<uint4*>(qa.q_out + (size_t)m * q_cols + n0 + c8) = v;
                } else if (rows.page[b0 + rr] >= 0) {
                    const int jj = n0 + c8 - q_cols;
                    bf16_t* kb = qa.pool + kv_block(g, qa.layer, rows.page[b0 + rr], jj >> lg_hd, 0);
                    *reinterpret_cast<uint4*>(kb + k_index_bf16(g, rows.key[b0 + rr], jj & (hd - 1))) = v;
                }
            }
            wave_lds_fence();
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int b0 = wr * WM + i * 32;
        if (rows.run[b0 >> 5]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int jj = n0 + j * 32 + col - k_end;
                bf16_t* vb = qa.pool + kv_block(g, qa.layer, rows.page[b0], jj >> lg_hd, 1) +
                             ((size_t)((rows.key[b0] >> 5) * 4 + (lane >> 5)) * hd + (jj & (hd - 1))) * 8;
#pragma unroll
                for (int h = 0; h < 2; ++h) {  // key groups h * 2 + lane / 32: registers 4h .. and 8 + 4h ..
                    uint32_t w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r = (e >> 1) * 8 + h * 4 + (e & 1) * 2;
                        w[e] = (uint32_t)f2bf(acc[i][j][r] + bias[j]) | ((uint32_t)f2bf(acc[i][j][r + 1] + bias[j]) << 16);
                    }
                    *reinterpret_cast<uint4*>(vb + (size_t)h * 2 * hd * 8) = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int jj = n0 + j * 32 + col - k_end;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rl = b0 + (r >> 2) * 8 + rbase + (r & 3);
                    if (rows.page[rl] < 0) continue;  // past M or unbacked
                    bf16_t* vb = qa.pool + kv_block(g, qa.layer, rows.page[rl], jj >> lg_hd, 1);
                    vb[v_index_bf16(g, rows.key[rl], jj & (hd - 1))] = f2bf(acc[i][j][r] + bias[j]);
                }
            }
        }
    }
}

template <int WGM, int WGN, int TM, int TN, int EPI, int S, bool NT, bool SUM = false>
__global__ void __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(2)))
gemm_wide_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, void* __restrict__ C, int M, int N, int K,
            int ldc, int m_tiles, int n_tiles, int nt0, int gm, int kps, size_t split_stride, QkvRopeArgs qa) {
    constexpr int NW = WGM * WGN, BM = WGM * TM * 32, BN = WGN * TN * 32, WM = TM * 32, WN = TN * 32;
    constexpr int AI = BM / 8 / NW, BI = BN / 8 / NW;  // 1 KB load instructions per wave per k-step
    constexpr int NM = TM * TN, NR = TM + TN;          // MFMAs and fragment reads per cluster
    static_assert(BM / 8 % NW == 0 && BN / 8 % NW == 0, "load split");
    static_assert(S >= 2 && S <= 4 && (S - 1) * (AI + BI) < 64, "stages");
    static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "SwiGLU pairs gate/up blocks inside a wave");
    static_assert(EPI != EPI_QKV_ROPE || (TN == 4 && 64 * NW >= BM), "a wave's columns are whole heads");
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st0;
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st1;
    __shared__ __attribute__((aligned(1024))) LdsStage<(S > 2 ? BM : 8), (S > 2 ? BN : 8)> st2_;
    __shared__ __attribute__((aligned(1024))) LdsStage<(S > 3 ? BM : 8), (S > 3 ? BN : 8)> st3_;
    [[maybe_unused]] LdsStage<BM, BN>& st2 = *reinterpret_cast<LdsStage<BM, BN>*>(&st2_);
    [[maybe_unused]] LdsStage<BM, BN>& st3 = *reinterpret_cast<LdsStage<BM, BN>*>(&st3_);
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int tiles = m_tiles * n_tiles, split = w / tiles;
    int mt, nt;
    wide_tile_of(w - split * tiles, m_tiles, n_tiles, gm, mt, nt);
    nt += nt0;  // a launch may cover the column tiles from nt0 on
    const int m0 = mt * BM;
    const int k_begin = split * kps, k_end = SUM ? K : min(K, k_begin + kps);
    const int n_k = (k_end - k_begin) / kBK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WGN, wc = wave % WGN;
    const int a_bytes = (int)((size_t)M * K * 2), w_bytes = (int)((size_t)N * K * 2);

    // lane l of load instruction j fills LDS chunk l % 8 of row l / 8 of its 8-row group
    constexpr uint32_t kOut = 0x80000000u;
    uint32_t a_off[AI], b_off[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        const int row = (wave * AI + j) * 8 + (lane >> 3), m = m0 + row;
        a_off[j] = m < M ? (uint32_t)(((size_t)m * K + k_begin + lds_swizzle(row, lane & 7) * 8) * 2) : kOut;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        const int row = (wave * BI + j) * 8 + (lane >> 3);
        int n;
        bool ok;
        if (EPI == EPI_SWIGLU) {  // a wave's N range: WN/2 gate rows, then the up rows of the same columns
            const int ff = N >> 1, rr = row % WN;
            const int c = nt * (BN / 2) + row / WN * (WN / 2) + rr % (WN / 2);
            ok = c < ff;
            n = rr < WN / 2 ? c : ff + c;
        } else {
            n = nt * BN + row;
            ok = n < N;
        }
        b_off[j] = ok ? (uint32_t)(((size_t)n * K + k_begin + lds_swizzle(row, lane & 7) * 8) * 2) : kOut;
    }
    auto load = [&](LdsStage<BM, BN>& sg, int k) {  // steps past the end read out of range: zeros
        lds_dma_stage<AI, BI>(sg, A, a_bytes, W, w_bytes, a_off, b_off,
                              k < n_k ? (uint32_t)k * kBK * 2 : 0x80000000u, wave, 0);
    };
    load(st0, 0);
    load(st1, 1);
    if constexpr (S > 2) load(st2, 2);
    if constexpr (S > 3) load(st3, 3);

    [[maybe_unused]] __shared__ WideQkvRows<EPI == EPI_QKV_ROPE ? BM : 32> qrows;
    if constexpr (EPI == EPI_QKV_ROPE) wide_qkv_rows<BM>(qa, M, m0, tid, qrows);

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // SUM: every kps of K the accumulators are a partial, added to the sum of those before it
    // (0 + p0 + p1 ..., the order and so the bits of the kernel that reads separate partials:
    // an accumulator is never -0).  Two accumulator sets fit beside the fragments for 64 x 64 of
    // output a wave, not for 128 x 64: 256x192 and 192x256 tiles spill and take 1.3-2.4 times as long.
    [[maybe_unused]] f32x16_t sum[SUM ? TM : 1][SUM ? TN : 1];
    [[maybe_unused]] int fold_at = kps / kBK;
    if constexpr (SUM)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[i][j][r] = 0.f;
    [[maybe_unused]] auto fold = [&](bool last) {
        if constexpr (SUM)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        sum[i][j][r] += acc[i][j][r];
                        acc[i][j][r] = last ? sum[i][j][r] : 0.f;
                    }
    };
    const int frow = lane & 31, fhalf = lane >> 5;
    bf16x8_t af[2][TM], bfr[2][TN];
    auto read = [&](bf16x8_t (&a)[TM], bf16x8_t (&b)[TN], const LdsStage<BM, BN>& sg, int ks) {
        const int c = lds_swizzle(frow, ks * 2 + fhalf) << 3;  // the swizzle repeats every 16 rows
#pragma unroll
        for (int i = 0; i < TM; ++i)
            a[i] = *reinterpret_cast<const bf16x8_t*>(&sg.a[(wr * WM + i * 32 + frow) * kBK + c]);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            b[j] = *reinterpret_cast<const bf16x8_t*>(&sg.b[(wc * WN + j * 32 + frow) * kBK + c]);
    };
    auto mma = [&](const bf16x8_t (&a)[TM], const bf16x8_t (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    wait_vmcnt_lds_reads<EPI == EPI_QKV_ROPE ? 0 : (S - 1) * (AI + BI)>();  // (QKV: the row look-ups count too)
    __builtin_amdgcn_s_barrier();
    read(af[0], bfr[0], st0, 0);
    // the schedule of a cluster: an MFMA, an LDS read, with LOADS a load, ...
#define DASH_WIDE_SCHED(LOADS)                                                                    \
    do {                                                                                          \
        _Pragma("unroll") for (int q_ = 0; q_ < NM; ++q_) {                                       \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                    \
            __builtin_amdgcn_sched_group_barrier(0x100, (NR + NM - 1) / NM, 0);                   \
            if (LOADS) __builtin_amdgcn_sched_group_barrier(0x020, (AI + BI + NM - 1) / NM, 0);   \
        }                                                                                         \
        __builtin_amdgcn_sched_barrier(0);                                                        \
    } while (0)
#define DASH_WIDE_STEP(CUR, NXT, KK)                                                              \
    do {                                                                                          \
        if constexpr (SUM)                                                                        \
            if ((KK) == fold_at) {                                                                \
                fold(false);                                                                      \
                fold_at += kps / kBK;                                                             \
            }                                                                                     \
        read(af[1], bfr[1], CUR, 1);                                                              \
        mma(af[0], bfr[0]);                                                                       \
        DASH_WIDE_SCHED(false);                                                                   \
        read(af[0], bfr[0], CUR, 2);                                                              \
        mma(af[1], bfr[1]);                                                                       \
        DASH_WIDE_SCHED(false);                                                                   \
        read(af[1], bfr[1], CUR, 3);                                                              \
        mma(af[0], bfr[0]);                                                                       \
        DASH_WIDE_SCHED(false);                                                                   \
        wait_vmcnt_lds_reads<(S - 2) * (AI + BI)>();                                              \
        __builtin_amdgcn_s_barrier();                                                             \
        __builtin_amdgcn_sched_barrier(0);                                                        \
        read(af[0], bfr[0], NXT, 0);                                                              \
        load(CUR, (KK) + S);                                                                      \
        mma(af[1], bfr[1]);                                                                       \
        DASH_WIDE_SCHED(true);                                                                    \
    } while (0)
    int k = 0;
    if constexpr (S == 2) {
        for (; k + 2 <= n_k; k += 2) {
            DASH_WIDE_STEP(st0, st1, k);
            DASH_WIDE_STEP(st1, st0, k + 1);
        }
        if (k < n_k) DASH_WIDE_STEP(st0, st1, k);
    } else if constexpr (S == 3) {
        for (; k + 3 <= n_k; k += 3) {
            DASH_WIDE_STEP(st0, st1, k);
            DASH_WIDE_STEP(st1, st2, k + 1);
            DASH_WIDE_STEP(st2, st0, k + 2);
        }
        if (k < n_k) DASH_WIDE_STEP(st0, st1, k);
        if (k + 1 < n_k) DASH_WIDE_STEP(st1, st2, k + 1);
    } else {
        for (; k + 4 <= n_k; k += 4) {
            DASH_WIDE_STEP(st0, st1, k);
            DASH_WIDE_STEP(st1, st2, k + 1);
            DASH_WIDE_STEP(st2, st3, k + 2);
            DASH_WIDE_STEP(st3, st0, k + 3);
        }
        if (k < n_k) DASH_WIDE_STEP(st0, st1, k);
        if (k + 1 < n_k) DASH_WIDE_STEP(st1, st2, k + 1);
        if (k + 2 < n_k) DASH_WIDE_STEP(st2, st3, k + 2);
    }
#undef DASH_WIDE_STEP
#undef DASH_WIDE_SCHED
    // the loads past the end still write their stages, and the last reads their registers
    wait_vmcnt_lds_reads<0>();
    __syncthreads();
    if constexpr (SUM) fold(true);
    if constexpr (EPI == EPI_QKV_ROPE) {
        static_assert(NW / 2 * 32 * kQkvRow <= (BM + BN) * kBK, "staged rows fit the stages");
        bf16_t* hs = (wave < NW / 2 ? st0.a : st1.a) + wave % (NW / 2) * (32 * kQkvRow);
        wide_qkv_epilogue<BM, WM, TM>(acc, qa, M, N, m0, nt * BN + wc * WN, wr, lane, qrows, hs);
    } else if constexpr (EPI == EPI_STORE_F32) {
        store_f32_epilogue<BM, BN, WGM, WGN, NT>(&acc[0][0], reinterpret_cast<float*>(C) + split * split_stride, M, N,
                                                 ldc, m0, nt, lane, wr, wc);
    } else {
        bf16_t* H = reinterpret_cast<bf16_t*>(C);
        if (((ldc | (N >> 1)) & 7) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0) {
            // each wave stages its own h tile in dead operand LDS (half the waves per stage), then
            // stores 16-byte runs: no barrier between the waves
            constexpr int OW = WN / 2, OS = OW + 8;
            static_assert(NW / 2 * WM * OS <= (BM + BN) * kBK, "h tiles fit the stages");
            static_assert(WM * OW / 8 % 64 == 0, "runs per lane");
            bf16_t* Hs = (wave < NW / 2 ? st0.a : st1.a) + wave % (NW / 2) * (WM * OS);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN / 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        Hs[(i * 32 + (r >> 2) * 8 + fhalf * 4 + (r & 3)) * OS + j * 32 + frow] =
                            f2bf(silu(acc[i][j][r]) * acc[i][j + TN / 2][r]);
            wave_lds_fence();
#pragma unroll
            for (int u = 0; u < WM * OW / 8 / 64; ++u) {
                const int run = lane + u * 64, rr = run / (OW / 8), c8 = run % (OW / 8) * 8;
                const int m = m0 + wr * WM + rr, c = nt * (BN / 2) + wc * OW + c8;
                if (m < M && c < (N >> 1))
                    *reinterpret_cast<uint4*>(H + (size_t)m * ldc + c) = *reinterpret_cast<const uint4*>(Hs + rr * OS + c8);
            }
        } else {
            swiglu_epilogue<BM, BN, WGM, WGN>(&acc[0][0], H, M, N, ldc, m0, nt, lane, wr, wc);
        }
    }
}

// ---- wide tiles, persistent ---------------------------------------------------------
// gemm_wide_k's 256 x 256 tile (eight waves of 128 x 64, two stages) in work-groups that stay:
// one per CU, each walking its share of its XCD's run of tiles.  The last two k-steps of a
// tile already load the next tile's first two, and the output leaves by 16-byte stores that
// drain under the next tile's first step, so a tile costs its k-steps and a short epilogue
// and not also a load latency and the draining of its output.  (In gemm_wide_k the stores of
// the 1.5B LM head at 8192 rows cost 600 of 3740 us and the rest per tile 6 of 42 us.)
//
// The output tile passes through LDS of the wave's own (kOutLds bytes a wave beside the two
// stages): 16 rows of fp32 or 32 rows of h at a time.  Every store instruction is issued
// whatever its lanes' bounds (rows and columns outside the output get an offset past the
// buffer's extent and are dropped), so the number of stores between two loads is known: the
// first step of a tile waits for all but them (loads and stores of a wave complete in order).
// An odd step count is padded with a step of zeros, which changes no bit (an accumulator is
// never -0).
constexpr int kOutLds = 4096;

struct WideTile {
    int m0, n0, split;  // n0: first output column (SwiGLU: of h)
};

template <int EPI, bool NT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
gemm_wide_persist_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, void* __restrict__ C, int M, int N, int K,
                    int ldc, int m_tiles, int n_tiles, int nt0, int gm, int kps, size_t split_stride, int tiles) {
    constexpr int WGN = 4, TM = 4, TN = 2, BM = 256, BN = 256, WM = 128, WN = 64, AI = 4, BI = 4;
    constexpr int NM = TM * TN, NR = TM + TN;
    constexpr int kStores = EPI == EPI_STORE_F32 ? 32 : 8;  // store instructions per wave and tile
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st0;
    __shared__ __attribute__((aligned(1024))) LdsStage<BM, BN> st1;
    __shared__ __attribute__((aligned(1024))) char out_lds[8 * kOutLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WGN, wc = wave % WGN;
    const int frow = lane & 31, fhalf = lane >> 5;
    // this work-group's tiles: t, t + step, ... below t_end
    const int x = blockIdx.x % kXcds, q = tiles / kXcds, rem = tiles % kXcds;
    const int t_end = x * q + min(x, rem) + q + (x < rem);
    const int t_step = gridDim.x / kXcds;
    int t = x * q + min(x, rem) + blockIdx.x / kXcds;
    if (t >= t_end) return;  // the grid is a multiple of the XCD count: a short run leaves blocks idle

    constexpr uint32_t kOut = 0x80000000u;
    auto tile_at = [&](int w) {
        const int split = w / (m_tiles * n_tiles);
        int mt, nt;
        wide_tile_of(w - split * m_tiles * n_tiles, m_tiles, n_tiles, gm, mt, nt);
        return WideTile{mt * BM, (nt + nt0) * (EPI == EPI_SWIGLU ? BN / 2 : BN), split};
    };
    auto steps_of = [&](const WideTile& tl) { return (min(K, tl.split * kps + kps) - tl.split * kps) / kBK; };
    // The wave's operand rows of a tile: 32 rows of A and 32 weight rows (SwiGLU: even waves the
    // gate rows of their pair's 32 columns, odd waves the up rows), consecutive in memory, so
    // a base, the bytes from it to the operand's end (rows past it read as zeros; gate rows
    // past the last column read up rows, whose outputs are dropped) and two lane offsets
    // (the swizzle alternates between 8-row groups) address them all.
    struct Rows {
        const bf16_t *a, *w;
        int a_left, w_left;
    };
    auto rows_of = [&](const WideTile& tl) {
        const int k_begin = tl.split * kps, m = tl.m0 + wave * 32;
        const int n = EPI == EPI_SWIGLU ? tl.n0 + (wave >> 1) * 32 + (wave & 1) * (N >> 1) : tl.n0 + wave * 32;
        return Rows{A + (size_t)m * K + k_begin, W + (size_t)n * K + k_begin,
                    m < M ? (int)(((size_t)(M - m) * K - k_begin) * 2) : 0,
                    n < N ? (int)(((size_t)(N - n) * K - k_begin) * 2) : 0};
    };
    const uint32_t l_off[2] = {(uint32_t)((lane >> 3) * K * 2 + ((lane & 7) ^ (lane >> 4)) * 16),
                               (uint32_t)((lane >> 3) * K * 2 + ((lane & 7) ^ (4 + (lane >> 4))) * 16)};
    auto load = [&](LdsStage<BM, BN>& sg, const Rows& rw, int k, int n_k) {  // a step past the end reads zeros
        const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(rw.a), 0, k < n_k ? rw.a_left : 0, kBufferDword3);
        const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(rw.w), 0, k < n_k ? rw.w_left : 0, kBufferDword3);
#pragma unroll
        for (int j = 0; j < AI; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void*)&sg.a[(wave * AI + j) * 8 * kBK], 16,
                                                     l_off[j & 1] + (uint32_t)(j * 16 * K + k * kBK * 2), 0, 0, 0);
#pragma unroll
        for (int j = 0; j < BI; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (lds_void*)&sg.b[(wave * BI + j) * 8 * kBK], 16,
                                                     l_off[j & 1] + (uint32_t)(j * 16 * K + k * kBK * 2), 0, 0, 0);
    };

    WideTile tile = tile_at(t);
    int n_k = steps_of(tile);
    Rows rows = rows_of(tile);
    load(st0, rows, 0, n_k);
    load(st1, rows, 1, n_k);

    f32x16_t acc[TM][TN];
    bf16x8_t af[2][TM], bfr[2][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    auto read = [&](bf16x8_t (&a)[TM], bf16x8_t (&b)[TN], const LdsStage<BM, BN>& sg, int ks) {
        const int c = lds_swizzle(frow, ks * 2 + fhalf) << 3;  // the swizzle repeats every 16 rows
#pragma unroll
        for (int i = 0; i < TM; ++i)
            a[i] = *reinterpret_cast<const bf16x8_t*>(&sg.a[(wr * WM + i * 32 + frow) * kBK + c]);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            b[j] = *reinterpret_cast<const bf16x8_t*>(&sg.b[(wc * WN + j * 32 + frow) * kBK + c]);
    };
    auto mma = [&](const bf16x8_t (&a)[TM], const bf16x8_t (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    // The output tile of the finished accumulators.  The lane index is made opaque, so that the
    // dozens of addresses built from it are formed here and not kept in registers through the
    // k-loop (which then spilled).
    auto store = [&](const WideTile& tl) {
        typedef unsigned u32x4_t __attribute__((__vector_size__(4 * sizeof(unsigned)), __may_alias__));
        typedef float f32_lds_t __attribute__((__may_alias__));
        typedef bf16_t bf16_lds_t __attribute__((__may_alias__));
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int orow = ln & 31, ohalf = ln >> 5;
        char* mine = out_lds + wave * kOutLds;
        constexpr int ES = EPI == EPI_STORE_F32 ? 4 : 2;  // bytes per element
        const size_t row0 = (size_t)(tl.m0 + wr * WM) * ldc;
        char* base = reinterpret_cast<char*>(C) + (EPI == EPI_STORE_F32 ? tl.split * split_stride + row0 : row0) * ES;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7FFFFFFF, kBufferDword3);
        constexpr int LR = EPI == EPI_STORE_F32 ? 4 : 2;                 // log2 of the lanes per stored row
        const int lrow = ln >> LR, n = tl.n0 + (EPI == EPI_STORE_F32 ? wc * WN + (ln & 15) * 4 : wc * (WN / 2) + (ln & 3) * 8);
        // rows of this lane's runs that exist: run rows below `left` (none past the last column)
        const int left = n < (EPI == EPI_STORE_F32 ? N : N >> 1) ? M - (tl.m0 + wr * WM) - lrow : 0;
        const uint32_t out = (uint32_t)((lrow * ldc + n) * ES);
        auto put = [&](u32x4_t v, int rr) {
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, rr < left ? out + (uint32_t)(rr * ldc * ES) : kOut, 0, NT ? 2 : 0);
        };
        if constexpr (EPI == EPI_STORE_F32) {
            // rows whose bit 2 is set have their column halves swapped: the two lane halves
            // (rows 4 apart) write different banks
            const uint32_t w0 = (ohalf * 4 * 64 + orow + ohalf * 32) * 4, w1 = (ohalf * 4 * 64 + orow + (32 - ohalf * 32)) * 4;
            const uint32_t r0 = (lrow * 64 + (ln & 15) * 4) * 4, r1 = (lrow * 64 + (((ln & 15) * 4) ^ 32)) * 4;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {  // 16 rows: accumulator registers 8 hh .. 8 hh + 7
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const int at = ((r >> 2) * 8 + (r & 3)) * 256;
                        *reinterpret_cast<f32_lds_t*>(mine + w0 + at) = acc[i][0][hh * 8 + r];
                        *reinterpret_cast<f32_lds_t*>(mine + w1 + at) = acc[i][1][hh * 8 + r];
                    }
                    wave_lds_fence();
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        put(*reinterpret_cast<const u32x4_t*>(mine + (u & 1 ? r1 : r0) + u * 1024), i * 32 + hh * 16 + u * 4);
                    wave_lds_fence();
                    __builtin_amdgcn_sched_barrier(0);  // one chunk's registers at a time
                }
        } else {
            constexpr int OS = 40;  // 32 columns of h and 8 of padding
            static_assert(32 * OS * 2 <= kOutLds, "staged rows fit");
            const uint32_t w0 = (ohalf * 4 * OS + orow) * 2, r0 = (lrow * OS + (ln & 3) * 8) * 2;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    *reinterpret_cast<bf16_lds_t*>(mine + w0 + ((r >> 2) * 8 + (r & 3)) * (OS * 2)) =
                        f2bf(silu(acc[i][0][r]) * acc[i][1][r]);
                wave_lds_fence();
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    put(*reinterpret_cast<const u32x4_t*>(mine + r0 + u * 16 * (OS * 2)), i * 32 + u * 16);
                wave_lds_fence();
                __builtin_amdgcn_sched_barrier(0);  // one chunk's registers at a time
            }
        }
    };

    clear();
    wait_vmcnt_lds_reads<0>();
    __builtin_amdgcn_s_barrier();
    read(af[0], bfr[0], st0, 0);
#define DASH_WIDE_SCHED(LOADS)                                                                    \
    do {                                                                                          \
        _Pragma("unroll") for (int q_ = 0; q_ < NM; ++q_) {                                       \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                    \
            __builtin_amdgcn_sched_group_barrier(0x100, (NR + NM - 1) / NM, 0);                   \
            if (LOADS) __builtin_amdgcn_sched_group_barrier(0x020, (AI + BI + NM - 1) / NM, 0);   \
        }                                                                                         \
        __builtin_amdgcn_sched_barrier(0);                                                        \
    } while (0)
    // One k-step (as in gemm_wide_k) that leaves OUTST operations in flight at its wait and
    // refills its stage by LOAD.
#define DASH_WIDE_STEP(CUR, NXT, OUTST, LOAD)                                                     \
    do {                                                                                          \
        read(af[1], bfr[1], CUR, 1);                                                              \
        mma(af[0], bfr[0]);                                                                       \
        DASH_WIDE_SCHED(false);                                                                   \
        read(af[0], bfr[0], CUR, 2);                                                              \
        mma(af[1], bfr[1]);                                                                       \
        DASH_WIDE_SCHED(false);                                                                   \
        read(af[1], bfr[1], CUR, 3);                                                              \
        mma(af[0], bfr[0]);                                                                       \
        DASH_WIDE_SCHED(false);                                                                   \
        wait_vmcnt_lds_reads<OUTST>();                                                            \
        __builtin_amdgcn_s_barrier();                                                             \
        __builtin_amdgcn_sched_barrier(0);                                                        \
        read(af[0], bfr[0], NXT, 0);                                                              \
        LOAD;                                                                                     \
        mma(af[1], bfr[1]);                                                                       \
        DASH_WIDE_SCHED(true);                                                                    \
    } while (0)
    for (;;) {
        const int n_pad = (n_k + 1) & ~1;
        t += t_step;
        const bool more = t < t_end;
        const WideTile next = more ? tile_at(t) : tile;
        const int nk_next = more ? steps_of(next) : 0;  // 0: the last loads read out of range
        const Rows rows_next = rows_of(next);
        if (n_pad > 2) {
            // the stores of the tile before may still drain (of the first tile there are none,
            // and both its first stages had landed before the first read)
            DASH_WIDE_STEP(st0, st1, kStores, load(st0, rows, 2, n_k));
            DASH_WIDE_STEP(st1, st0, 0, load(st1, rows, 3, n_k));
            for (int k = 2; k + 2 < n_pad; k += 2) {
                DASH_WIDE_STEP(st0, st1, 0, load(st0, rows, k + 2, n_k));
                DASH_WIDE_STEP(st1, st0, 0, load(st1, rows, k + 3, n_k));
            }
        }
        DASH_WIDE_STEP(st0, st1, 0, load(st0, rows_next, 0, nk_next));
        DASH_WIDE_STEP(st1, st0, 0, load(st1, rows_next, 1, nk_next));
        store(tile);
        if (!more) break;
        clear();
        tile = next;
        n_k = nk_next;
        rows = rows_next;
    }
#undef DASH_WIDE_STEP
#undef DASH_WIDE_SCHED
    wait_vmcnt<0>();  // the out-of-range loads past the last tile still write their stages
}

// Output columns [col0, col1) (SwiGLU: of h; col0 a multiple of the tile's output width).
template <int WGM, int WGN, int TM, int TN, int EPI, int S = 2>
hipError_t run_wide_cols(const void* A, const void* W, void* C, int M, int N, int K, int ldc, int nsplit,
                         size_t split_stride, int col0, int col1, hipStream_t st,
                         const QkvRopeArgs& qa = QkvRopeArgs{}) {
    constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, tn = EPI == EPI_SWIGLU ? BN / 2 : BN;
    const int m_tiles = (M + BM - 1) / BM, n_tiles = (col1 - col0 + tn - 1) / tn;
    if (col0 < 0 || col0 % tn || col1 <= col0 || col1 > (EPI == EPI_SWIGLU ? N / 2 : N)) return hipErrorInvalidValue;
    int kps = K;
    if (nsplit > 1) kps = ((K + nsplit - 1) / nsplit + kBK - 1) / kBK * kBK;
    if ((K + kps - 1) / kps != nsplit) return hipErrorInvalidValue;
    if (K % kBK || (size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return hipErrorInvalidValue;
    // rows of tiles per block of the tile order: 6 x ~5 tiles at a time on an XCD where there
    // are columns enough, 4 x 8 for the few column tiles of the projections back to d_model
    // (measured 2-8 and 16: within 2% of the best of them on the prefill's shapes)
    const int gm = n_tiles >= 16 ? 6 : 4, blocks = m_tiles * n_tiles * nsplit;
    // An fp32 output past the 256 MB last-level cache leaves by streaming stores, which keep
    // the operands in L2 (its reader misses either way): LM head 1.5B 3896 -> 3775 us at 8192
    // rows, 512 -> 505 at 1024; the five partials of the down projection at 16,384 rows 439
    // -> 426.  Smaller outputs are read from that cache next.
    constexpr size_t kCache = (size_t)256 << 20;
    const bool past_cache = EPI == EPI_STORE_F32 && (size_t)M * (col1 - col0) * nsplit * 4 > kCache;
    // From two rounds on the 256x256 tile runs in work-groups that stay, where the output can be
    // written in 16-byte runs: gate/up 1.5B 729 -> 687 us at 16,384 rows and 0.5B 73.7 -> 68.5
    // at 4,206, down 1.5B 262 -> 247 at 10,240, LM head 1.5B 3737 -> 3667 at 8,192 and 0.5B 956 ->
    // 924 at 3,066 (K = 896; 628 against 661 at 2,048).  Work-groups that stay can't hand the
    // tiles of a last round that is mostly empty to the CUs that are ahead, and where the steps
    // of a tile are many that costs more than the seams save: LM head 1.5B at 1,024 rows (9.28
    // rounds) 514 against 500, at 1,792 (16.24) 865 against 854, but at 1,280 (11.6) 606 against
    // 613 after.  So from 1,024 of K on a launch of under 32 rounds goes there with a third of
    // its last round filled.
    constexpr int V = EPI == EPI_SWIGLU ? 8 : 4;  // elements per run
    if constexpr (WGM == 2 && WGN == 4 && TM == 4 && TN == 2 && S == 2 && EPI != EPI_QKV_ROPE) {
        const bool seams_pay = kps < 1024 || blocks >= 32 * 256 || (blocks - 1) % 256 >= 85;
        if (blocks >= 512 && seams_pay && ldc % V == 0 && (EPI == EPI_SWIGLU ? N / 2 : N) % V == 0 &&
            split_stride % V == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0 && (size_t)BM * ldc * 4 < (1u << 31)) {
            auto run = [&](auto nt) {
                gemm_wide_persist_k<EPI, decltype(nt)::value><<<256, 512, 0, st>>>(
                    (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, col0 / tn, gm, kps, split_stride, blocks);
                return hipGetLastError();
            };
            if constexpr (EPI == EPI_STORE_F32)
                if (past_cache) return run(std::true_type{});
            return run(std::false_type{});
        }
    }
    if constexpr (EPI == EPI_STORE_F32 && BM == 256 && BN == 256)  // the others run where one round holds the launch
        if (past_cache) {
            gemm_wide_k<WGM, WGN, TM, TN, EPI, S, true><<<blocks, 64 * WGM * WGN, 0, st>>>(
                (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, col0 / tn, gm, kps, split_stride, qa);
            return hipGetLastError();
        }
    gemm_wide_k<WGM, WGN, TM, TN, EPI, S, false><<<blocks, 64 * WGM * WGN, 0, st>>>(
        (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, col0 / tn, gm, kps, split_stride, qa);
    return hipGetLastError();
}

template <int WGM, int WGN, int TM, int TN, int EPI, int S = 2>
hipError_t run_wide(const void* A, const void* W, void* C, int M, int N, int K, int ldc, int nsplit,
                    size_t split_stride, hipStream_t st, const QkvRopeArgs& qa = QkvRopeArgs{}) {
    return run_wide_cols<WGM, WGN, TM, TN, EPI, S>(A, W, C, M, N, K, ldc, nsplit, split_stride, 0,
                                                   EPI == EPI_SWIGLU ? N / 2 : N, st, qa);
}

// All nsplit partials of a tile by one work-group, added in registers in split order.
template <int WGM, int WGN, int TM, int TN, int S>
hipError_t run_wide_sum(const void* A, const void* W, void* C, int M, int N, int K, int nsplit, hipStream_t st) {
    constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32;
    const int m_tiles = (M + BM - 1) / BM, n_tiles = (N + BN - 1) / BN;
    const int kps = ((K + nsplit - 1) / nsplit + kBK - 1) / kBK * kBK;
    if ((K + kps - 1) / kps != nsplit) return hipErrorInvalidValue;
    if (K % kBK || (size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return hipErrorInvalidValue;
    // tile order: 4 rows of tiles per block (8 and 12 measured: within 3% either way)
    gemm_wide_k<WGM, WGN, TM, TN, EPI_STORE_F32, S, false, true><<<m_tiles * n_tiles, 64 * WGM * WGN, 0, st>>>(
        (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, N, m_tiles, n_tiles, 0, 4, kps, 0, QkvRopeArgs{});
    return hipGetLastError();
}

// ---- small batches ---------------------------------------------------------------
// Up to a few row blocks the projections are chains of dependent k-steps in few work-groups:
// what a step costs is latency.  (Register-staged tiles four steps ahead took ~0.2 us per
// 64-deep step on every shape and batch up to 64 rows, cold or cached, where the four MFMAs
// of a step take 0.053.)  So the tiles are narrow, one 32 x 32 block (or U of its columns) or
// two per wave, and up to S = 8 steps of both operands are on their way into LDS at once; a
// step's fragments are read while the step before is multiplied, so a step is a wait for
// the oldest load, a barrier and four MFMAs.  U < 32 leaves a block's other columns unused
// (the fragments repeat): more work-groups over the same weights.
//
// Column blocks: TN consecutive ones (fp32 store), or gate columns then the up columns of the
// same h columns (SwiGLU).  (With the QKV projection's RoPE and KV append in the epilogue the
// one launch took 7.7-12 us at 16-64 rows against 7.6-10.4 for this kernel and the append
// kernel: few waves chase the page look-ups and scattered stores; not kept.)  Measured (weights
// cold, against the register-staged 64 x 32 .. 64 x 256 tiles it replaced): QKV / O at 16 rows 0.5B 5.8 -> 4.4 us, 1.5B 7.7 -> 5.5, 3B 9.3 -> 6.6; down 5.4 -> 4.6,
// 8.9 -> 7.1, 12.5 -> 10.5; gate/up 9.0 -> 6.7, 14.3 -> 12.5, 21.7 -> 20.6; LM head (weights
// at 5.9 TB/s) 59 -> 47, 93 -> 78, 132 -> 106.  Same fragments and MFMA order: same bits.
template <int WM_, int WN_, int TN, int U, int S, int EPI, int WPOL>
__global__ void __launch_bounds__(64 * WM_ * WN_)
gemm_stream_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, void* __restrict__ C, int M, int N, int K,
              int ldc, int m_tiles, int n_tiles, int kps, size_t split_stride) {
    constexpr int NW = WM_ * WN_, BM = 32 * WM_, WN = U * TN, BN = WN * WN_;
    constexpr int AI = BM / 8 / NW, BI = BN / 8 / NW, DPS = AI + BI;  // 1 KB loads per wave per k-step
    static_assert(BM / 8 % NW == 0 && BN / 8 % NW == 0 && BI >= 1, "load split");
    static_assert((S - 1) * DPS < 64, "loads in flight fit the counter");
    static_assert(S == 3 || S == 4 || S == 8, "stages");
    static_assert(U == 8 || U == 16 || U == 32, "columns per block");
    static_assert(EPI == EPI_STORE_F32 || (EPI == EPI_SWIGLU && TN == 2), "SwiGLU holds a gate / up pair in a lane");
    using Stage = LdsStage<BM, BN>;
#define DASH_STAGE(i)                                                                                            \
    __shared__ __attribute__((aligned(1024))) LdsStage<(S > i ? BM : 8), (S > i ? BN : 8)> st##i##_;             \
    Stage& st##i = *reinterpret_cast<Stage*>(&st##i##_);
    DASH_STAGE(0) DASH_STAGE(1) DASH_STAGE(2) DASH_STAGE(3)
    DASH_STAGE(4) DASH_STAGE(5) DASH_STAGE(6) DASH_STAGE(7)
#undef DASH_STAGE
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int mt = w % m_tiles, rest = w / m_tiles, nt = rest % n_tiles, split = rest / n_tiles;
    const int m0 = mt * BM;
    const int k_begin = split * kps, k_end = min(K, k_begin + kps);
    const int n_k = (k_end - k_begin) / kBK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WN_, wc = wave % WN_;
    const int frow = lane & 31, fhalf = lane >> 5;
    const int a_bytes = (int)((size_t)M * K * 2), w_bytes = (int)((size_t)N * K * 2);
    constexpr uint32_t kOut = 0x80000000u;
    uint32_t a_off[AI], b_off[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        const int row = (wave * AI + j) * 8 + (lane >> 3), m = m0 + row;
        a_off[j] = m < M ? (uint32_t)(((size_t)m * K + k_begin + lds_swizzle(row, lane & 7) * 8) * 2) : kOut;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
        const int row = (wave * BI + j) * 8 + (lane >> 3);
        int n;
        bool ok;
        if (EPI == EPI_SWIGLU) {  // U gate rows, then the up rows of the same columns
            const int c = (nt * WN_ + row / WN) * U + row % U;
            ok = c < (N >> 1);
            n = row % WN < U ? c : (N >> 1) + c;
        } else {
            n = nt * BN + row;
            ok = n < N;
        }
        b_off[j] = ok ? (uint32_t)(((size_t)n * K + k_begin + lds_swizzle(row, lane & 7) * 8) * 2) : kOut;
    }
    auto load = [&](Stage& sg, int k) {  // steps past the end read out of range: zeros
        lds_dma_stage<AI, BI>(sg, A, a_bytes, W, w_bytes, a_off, b_off,
                              k < n_k ? (uint32_t)k * kBK * 2 : 0x80000000u, wave, WPOL);
    };
    load(st0, 0);
    load(st1, 1);
    load(st2, 2);
    if constexpr (S > 3) load(st3, 3);
    if constexpr (S > 4) {
        load(st4, 4);
        load(st5, 5);
        load(st6, 6);
        load(st7, 7);
    }
    f32x16_t acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    bf16x8_t af[2][4], bfr[2][4][TN];
    auto read = [&](bf16x8_t (&a)[4], bf16x8_t (&b)[4][TN], const Stage& sg) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c = ks * 2 + fhalf, ar = wr * 32 + frow;
            a[ks] = *reinterpret_cast<const bf16x8_t*>(&sg.a[ar * kBK + (lds_swizzle(ar, c) << 3)]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int br = wc * WN + j * U + frow % U;
                b[ks][j] = *reinterpret_cast<const bf16x8_t*>(&sg.b[br * kBK + (lds_swizzle(br, c) << 3)]);
            }
        }
    };
    auto mma = [&](const bf16x8_t (&a)[4], const bf16x8_t (&b)[4][TN]) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], b[ks][j], acc[j], 0, 0, 0);
    };
    wait_vmcnt_lds_reads<(S - 1) * DPS>();
    __builtin_amdgcn_s_barrier();
    read(af[0], bfr[0], st0);
    // Step KK from fragment set P (its stage CUR is all in registers of every wave once past
    // the barrier, so CUR is refilled) while NXT's fragments are read into the other set.
#define DASH_STREAM_STEP(P, CUR, NXT, KK)          \
    do {                                           \
        wait_vmcnt_lds_reads<(S - 2) * DPS>();     \
        __builtin_amdgcn_s_barrier();              \
        __builtin_amdgcn_sched_barrier(0);         \
        read(af[1 - (P)], bfr[1 - (P)], NXT);      \
        load(CUR, (KK) + S);                       \
        mma(af[P], bfr[P]);                        \
        __builtin_amdgcn_sched_barrier(0);         \
    } while (0)
#define DASH_STREAM_TAIL(P, CUR, NXT)              \
    if (k < n_k) {                                 \
        DASH_STREAM_STEP(P, CUR, NXT, k);          \
        ++k;                                       \
    }
    int k = 0;
    if constexpr (S == 3) {
        for (; k + 6 <= n_k; k += 6) {
            DASH_STREAM_STEP(0, st0, st1, k);
            DASH_STREAM_STEP(1, st1, st2, k + 1);
            DASH_STREAM_STEP(0, st2, st0, k + 2);
            DASH_STREAM_STEP(1, st0, st1, k + 3);
            DASH_STREAM_STEP(0, st1, st2, k + 4);
            DASH_STREAM_STEP(1, st2, st0, k + 5);
        }
        DASH_STREAM_TAIL(0, st0, st1)
        DASH_STREAM_TAIL(1, st1, st2)
        DASH_STREAM_TAIL(0, st2, st0)
        DASH_STREAM_TAIL(1, st0, st1)
        DASH_STREAM_TAIL(0, st1, st2)
    } else if constexpr (S == 4) {
        for (; k + 4 <= n_k; k += 4) {
            DASH_STREAM_STEP(0, st0, st1, k);
            DASH_STREAM_STEP(1, st1, st2, k + 1);
            DASH_STREAM_STEP(0, st2, st3, k + 2);
            DASH_STREAM_STEP(1, st3, st0, k + 3);
        }
        DASH_STREAM_TAIL(0, st0, st1)
        DASH_STREAM_TAIL(1, st1, st2)
        DASH_STREAM_TAIL(0, st2, st3)
    } else {
        for (; k + 8 <= n_k; k += 8) {
            DASH_STREAM_STEP(0, st0, st1, k);
            DASH_STREAM_STEP(1, st1, st2, k + 1);
            DASH_STREAM_STEP(0, st2, st3, k + 2);
            DASH_STREAM_STEP(1, st3, st4, k + 3);
            DASH_STREAM_STEP(0, st4, st5, k + 4);
            DASH_STREAM_STEP(1, st5, st6, k + 5);
            DASH_STREAM_STEP(0, st6, st7, k + 6);
            DASH_STREAM_STEP(1, st7, st0, k + 7);
        }
        DASH_STREAM_TAIL(0, st0, st1)
        DASH_STREAM_TAIL(1, st1, st2)
        DASH_STREAM_TAIL(0, st2, st3)
        DASH_STREAM_TAIL(1, st3, st4)
        DASH_STREAM_TAIL(0, st4, st5)
        DASH_STREAM_TAIL(1, st5, st6)
        DASH_STREAM_TAIL(0, st6, st7)
    }
#undef DASH_STREAM_TAIL
#undef DASH_STREAM_STEP
    if constexpr (EPI == EPI_STORE_F32) {
        float* Cp = reinterpret_cast<float*>(C) + split * split_stride;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = nt * BN + wc * WN + j * U + frow;
            if (n < N && frow < U)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = m0 + wr * 32 + (r >> 2) * 8 + fhalf * 4 + (r & 3);
                    if (m < M) Cp[(size_t)m * ldc + n] = acc[j][r];
                }
        }
    } else {
        bf16_t* H = reinterpret_cast<bf16_t*>(C);
        const int c = (nt * WN_ + wc) * U + frow;
        if (c < (N >> 1) && frow < U)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wr * 32 + (r >> 2) * 8 + fhalf * 4 + (r & 3);
                if (m < M) H[(size_t)m * ldc + c] = f2bf(silu(acc[0][r]) * acc[1][r]);
            }
    }
    wait_vmcnt<0>();  // the out-of-range loads of the steps past the end still write their stages
}

// ONE_ROW: a tile for batches of at most its rows
template <int WM_, int WN_, int TN, int U, int S, int EPI, bool ONE_ROW = false>
hipError_t run_stream(const void* A, const void* W, void* C, int M, int N, int K, int ldc, int nsplit,
                      size_t split_stride, hipStream_t st) {
    constexpr int BM = 32 * WM_, BN = U * TN * WN_;
    const int m_tiles = (M + BM - 1) / BM, n_tiles = (N + BN - 1) / BN;
    int kps = K;
    if (nsplit > 1) kps = ((K + nsplit - 1) / nsplit + kBK - 1) / kBK * kBK;
    if ((K + kps - 1) / kps != nsplit) return hipErrorInvalidValue;
    if (K % kBK || (size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return hipErrorInvalidValue;
    const int blocks = m_tiles * n_tiles * nsplit;
    // a weight byte that one work-group alone reads streams past the caches
    if (m_tiles == 1) {
        gemm_stream_k<WM_, WN_, TN, U, S, EPI, 2><<<blocks, 64 * WM_ * WN_, 0, st>>>(
            (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, kps, split_stride);
        return hipGetLastError();
    }
    if constexpr (ONE_ROW) return hipErrorInvalidValue;
    else
        gemm_stream_k<WM_, WN_, TN, U, S, EPI, 0><<<blocks, 64 * WM_ * WN_, 0, st>>>(
            (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, kps, split_stride);
    return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int S, int EPI, int WPOL = 0>
hipError_t run_lds(const void* A, const void* W, void* C, int M, int N, int K, int ldc, int nsplit,
                   size_t split_stride, hipStream_t st, const QkvRopeArgs& qa = QkvRopeArgs{}) {
    const int m_tiles = (M + BM - 1) / BM;
    const int n_tiles = (N + BN - 1) / BN;
    int kps = K;
    if (nsplit > 1) {
        kps = (K + nsplit - 1) / nsplit;
        kps = (kps + kBK - 1) / kBK * kBK;
    }
    if ((K + kps - 1) / kps != nsplit) return hipErrorInvalidValue;
    if (K % kBK || (size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return hipErrorInvalidValue;
    gemm_lds_k<BM, BN, WGM, WGN, S, EPI, WPOL><<<m_tiles * n_tiles * nsplit, 64 * WGM * WGN, 0, st>>>(
        (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, kps, split_stride, qa);
    return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int PD, int EPI, int WPOL = 0>
hipError_t run_bf16(const void* A, const void* W, void* C, int M, int N, int K, int ldc, int nsplit,
                     size_t split_stride, hipStream_t st, const QkvRopeArgs& qa = QkvRopeArgs{}) {
    const int m_tiles = (M + BM - 1) / BM;
    const int cols = EPI == EPI_SWIGLU ? N / 2 : N;
    const int tn = EPI == EPI_SWIGLU ? BN / 2 : BN;
    const int n_tiles = (cols + tn - 1) / tn;
    int kps = K;
    if (nsplit > 1) {
        kps = (K + nsplit - 1) / nsplit;
        kps = (kps + kBK - 1) / kBK * kBK;
    }
    if ((K + kps - 1) / kps != nsplit) return hipErrorInvalidValue;
    // k-steps of 64 never straddle the end of K or of a split; byte offsets fit 31 bits
    if (K % kBK || (size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return hipErrorInvalidValue;
    const int blocks = m_tiles * n_tiles * nsplit;
    gemm_bf16_k<BM, BN, WGM, WGN, PD, EPI, WPOL><<<blocks, 64 * WGM * WGN, 0, st>>>(
        (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, 0, kps, split_stride, qa);
    return hipGetLastError();
}

// Gate/up with the SwiGLU epilogue over output columns [col0, col1) of h only (col0 a
// multiple of the tile's BN / 2 output columns): the same tiles, hence the same bits, as
// the launch over every column.
template <int BM, int BN, int WGM, int WGN, int PD>
hipError_t run_bf16_swiglu_cols(const void* A, const void* W, void* C, int M, int N, int K, int ldc, int col0,
                                int col1, hipStream_t st) {
    constexpr int tn = BN / 2;
    if (col0 % tn || col0 < 0 || col1 <= col0 || col1 > N / 2) return hipErrorInvalidValue;
    if (K % kBK || (size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return hipErrorInvalidValue;
    const int m_tiles = (M + BM - 1) / BM;
    const int n_tiles = (col1 - col0 + tn - 1) / tn;
    gemm_bf16_k<BM, BN, WGM, WGN, PD, EPI_SWIGLU><<<m_tiles * n_tiles, 64 * WGM * WGN, 0, st>>>(
        (const bf16_t*)A, (const bf16_t*)W, C, M, N, K, ldc, m_tiles, n_tiles, col0 / tn, K, 0, QkvRopeArgs{});
    return hipGetLastError();
}

// fp32: 64 x 64 output tile per 256 threads (16 x 16, 4 x 4 each), BK = 16.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_f32_k(const float* __restrict__ A, const float* __restrict__ W,
                                                  void* __restrict__ C, int M, int N, int K, int ldc) {
    __shared__ float As[16][65];
    __shared__ float Bs[16][65];
    __shared__ float Cs[EPI == EPI_SWIGLU ? 64 : 1][65];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int m0 = blockIdx.y * 64;
    const int ff = N >> 1;
    // B tile rows: STORE: n0 + r;  SWIGLU: r < 32 gate j0 + r, r >= 32 up ff + j0 + r - 32.
    auto wrow = [&](int r, bool& ok) {
        if (EPI == EPI_SWIGLU) {
            const int j = blockIdx.x * 32 + (r & 31);
            ok = j < ff;
            return r < 32 ? j : ff + j;
        }
        const int n = blockIdx.x * 64 + r;
        ok = n < N;
        return n;
    };
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
        for (int e = threadIdx.x; e < 64 * 16; e += 256) {
            const int r = e >> 4, k = e & 15;
            const int m = m0 + r;
            As[k][r] = (m < M && k0 + k < K) ? A[(size_t)m * K + k0 + k] : 0.f;
            bool ok;
            const int n = wrow(r, ok);
            Bs[k][r] = (ok && k0 + k < K) ? W[(size_t)n * K + k0 + k] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += As[k][ty * 4 + i] * Bs[k][tx * 4 + j];
        __syncthreads();
    }
    if (EPI == EPI_STORE_F32) {
        float* Cp = reinterpret_cast<float*>(C);
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 4; ++j) {
                const int m = m0 + ty * 4 + i, n = blockIdx.x * 64 + tx * 4 + j;
                if (m < M && n < N) Cp[(size_t)m * ldc + n] = acc[i][j];
            }
    } else {
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 4; ++j) Cs[ty * 4 + i][tx * 4 + j] = acc[i][j];
        __syncthreads();
        float* H = reinterpret_cast<float*>(C);
        for (int e = threadIdx.x; e < 64 * 32; e += 256) {
            const int r = e >> 5, c = e & 31;
            const int m = m0 + r, col = blockIdx.x * 32 + c;
            if (m < M && col < ff) H[(size_t)m * ldc + col] = silu(Cs[r][c]) * Cs[r][c + 32];
        }
    }
}

}  // namespace

// Split-K count as a function of the weight shape only (never of M), so that a
// row's result does not depend on how many other rows share the launch: the
// whole path is batch-invariant, bit for bit.  Only long reductions are split
// (the down projection, K = d_ff): with 128 x 256 tiles, one workgroup per CU,
// a decode batch of ~1k rows then gives close to one tile per CU (1.5B:
// 8 x 6 tiles x 5 splits = 240 of 256 CUs).  Short reductions (QKV, O, K = d)
// run unsplit on small tiles instead, which was measured faster than split-K
// plus the partial sums it leaves for the consumer to read.
int gemm_pick_splits(int dtype, int epi, int N, int K) {
    if (dtype != 1 || epi != EPI_STORE_F32 || K < 4096) return 1;
    const int nt = (N + 255) / 256;
    int s = std::max(1, (32 + nt / 2) / nt);  // ~32 tile-splits per 128-row block of the batch
    s = std::min(s, std::min(8, K / 512));
    int kps = (K + s - 1) / s;
    kps = (kps + kBK - 1) / kBK * kBK;
    return (K + kps - 1) / kps;
}

// Tiles of 256x128, or of 128x256 where those take fewer rounds (or as many, past one).
static bool sum_tall(int M, int N, long* tiles) {
    const long tall = (long)((M + 255) / 256) * ((N + 127) / 128), flat = (long)((M + 127) / 128) * ((N + 255) / 256);
    const long rt = (tall + 255) / 256, rf = (flat + 255) / 256;
    const bool use_tall = rt < rf || (rt == rf && rt == 1);
    *tiles = use_tall ? tall : flat;
    return use_tall;
}

// What it saves: nsplit - 1 partials written and read back, about 26 us a full round of 1.5B
// tiles.  What it costs: a tile takes the whole of K, so a last round that is partly empty is
// as many times longer as there are splits.  So it pays by empty tiles x steps of K against
// tiles x (nsplit - 1): up to a ratio of 12 (20 within one round, whose empty CUs leave the
// others the memory and the clock).  us with the norm that reads the output, split / summed,
// at (rows, ratio): 1.5B 16,384 (0) 535 / 454, 10,843 (0) 393 / 302, 8,155 (11.7) 270 / 262,
// 11,867 (13.2) 398 / 396, 4,059 (11.7) 138 / 124; 3B 4,059 (0) 191 / 173, 6,875 (10.5) 377 /
// 341, 3,035 (19) 158 / 155, 6,107 (19) 294 / 315, 2,523 (35) 145 / 149; 0.5B 16,347 (0) 322 /
// 181, 5,211 (8) 98 / 66; 3584 x 18,944 in two splits 3,931 (42) 504 / 540.
bool gemm_sum_pays(int dtype, int M, int N, int K, int nsplit) {
    if (dtype != 1 || nsplit < 2 || M <= 1024 || K % kBK) return false;
    if ((size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31)) return false;
    long tiles;
    sum_tall(M, N, &tiles);
    const long empty = (256 - tiles % 256) % 256;
    return empty * (K / kBK) <= (tiles <= 256 ? 20 : 12) * (nsplit - 1) * tiles;
}

hipError_t launch_gemm_sum(const void* A, const void* W, void* C, int M, int N, int K, int nsplit, hipStream_t st) {
    long tiles;
    if (sum_tall(M, N, &tiles)) return run_wide_sum<4, 2, 2, 2, 3>(A, W, C, M, N, K, nsplit, st);
    return run_wide_sum<2, 4, 2, 2, 3>(A, W, C, M, N, K, nsplit, st);
}

bool gemm_qkv_fusable(int dtype, int n_heads, int n_kv, int head_dim) {
    return dtype == 1 && (head_dim == 64 || head_dim == 128) && (n_heads * head_dim) % 128 == 0 &&
           (n_kv * head_dim) % 128 == 0;
}

bool gemm_qkv_fuse_pays(int M, int N) { return (long)((M + 63) / 64) * (N / 128) >= 128; }

hipError_t launch_gemm_qkv_rope(const void* A, const void* W, int M, int N, int K, const QkvRopeArgs& qa,
                                hipStream_t st) {
    if (M <= 0) return hipSuccess;
    if (!gemm_qkv_fusable(1, qa.n_heads, qa.g.n_kv, qa.g.head_dim) ||
        N != (qa.n_heads + 2 * qa.g.n_kv) * qa.g.head_dim)
        return hipErrorInvalidValue;
    // Wide tiles where they fill the chip: 256x256 at one round (128-256 of them) or from one
    // and a half on, else 128x128 (two per CU) from half a round on; below that 64x128, by
    // direct-to-LDS loads while they fit one round (one per CU), else register-staged.  us
    // at 1.5B / 3B (256x256, 128x128, 64x128 register-staged, weights cold): 2048 rows
    // 44 25.5 27.4 / 52 34 45; 4206 rows 45 48 60 / 55 60 84; 10240 rows 77 72 124 / 102 119
    // 185; 16384 rows 90 107 204 / 158 172 306.  64x128 direct-to-LDS at 419 rows: 10.1 vs
    // 10.6 (0.5B), 13.1 vs 14.2, 15.5 vs 17.1; 3B at 1024 rows (320 tiles) 28.9 vs 26.0.
    const long t256 = (long)((M + 255) / 256) * ((N + 255) / 256), t128 = (long)((M + 127) / 128) * (N / 128);
    if ((t256 >= 128 && t256 <= 256) || t256 >= 384)
        return run_wide<4, 2, 2, 4, EPI_QKV_ROPE>(A, W, nullptr, M, N, K, 0, 1, 0, st, qa);
    if (t128 >= 256) return run_wide<4, 1, 1, 4, EPI_QKV_ROPE>(A, W, nullptr, M, N, K, 0, 1, 0, st, qa);
    if ((long)((M + 63) / 64) * (N / 128) <= 256)
        return run_lds<64, 128, 2, 4, 3, EPI_QKV_ROPE>(A, W, nullptr, M, N, K, 0, 1, 0, st, qa);
    return run_bf16<64, 128, 2, 4, 2, EPI_QKV_ROPE>(A, W, nullptr, M, N, K, 0, 1, 0, st, qa);
}

hipError_t launch_gemm(int dtype, int epi, const void* A, const void* W, void* C, int M, int N, int K, int ldc,
                       int nsplit, size_t split_stride, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (dtype == 1) {
        // Tile choice may depend on M: every configuration accumulates each output
        // element with the same chain of 32x32x16 MFMAs over k, so results do not.
        // Small batches stream the weights: narrow tiles give enough workgroups
        // (>= 256) to pull them from HBM at full rate.
        if (epi == EPI_SWIGLU) {
            if (nsplit != 1) return hipErrorInvalidValue;
            if (M > 384) {
                const int ff = N / 2;
                const long mb = (M + 255) / 256;
                const long t256_all = mb * ((ff + 127) / 128);
                const long split_tiles = t256_all / 256 * 256 / mb;  // column tiles of the whole rounds
                if (t256_all > 256 && t256_all < 4 * 256 && t256_all % 256 && t256_all % 256 < 128 &&
                    split_tiles >= 1) {
                    // Whole rounds of 256x256 tiles leave a last round under half full: those
                    // rounds run as one launch over the columns they cover, the remaining
                    // columns as a second launch on the largest of 128x256, 128x128 and 64x128
                    // tiles that still gives it 128 or more work-groups (else 64x128).
                    // us (dash_gemm_bench, weights cold), two launches / one of 256x256 / the
                    // best other tile in one: 1.5B at 1024 rows 58 / 71 / 69 and at 2048 104 /
                    // 117 / 113, 3B at 1024 91-93 / 105 / 90, 0.5B at 2048 40 / 50 / 43 (a
                    // last round at least half full runs whole, as below).
                    const int c_split = (int)split_tiles * 128;
                    hipError_t e = run_wide_cols<2, 4, 4, 2, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, 0, c_split, st);
                    if (e != hipSuccess) return e;
                    const long rc = ff - c_split, m128 = (M + 127) / 128;
                    if (m128 * ((rc + 127) / 128) >= 128)
                        return run_bf16_swiglu_cols<128, 256, 4, 4, 2>(A, W, C, M, N, K, ldc, c_split, ff, st);
                    if (m128 * ((rc + 63) / 64) >= 128)
                        return run_bf16_swiglu_cols<128, 128, 4, 2, 2>(A, W, C, M, N, K, ldc, c_split, ff, st);
                    return run_bf16_swiglu_cols<64, 128, 2, 2, 2>(A, W, C, M, N, K, ldc, c_split, ff, st);
                }
                // Past 384 rows the tile is chosen by how its work-groups fill the 256 CUs
                // (one 256x256 work-group per CU, two 128x128 ones): 256x256 where they fill
                // one round (128-256 tiles), or leave a last round at least half full, or run
                // four rounds or more; else 128x128.  us, 256x256 / 128x128 (0.5B, the width
                // that has few tiles): 419 rows 19.8 / 13.6, 768 rows 20.4 / 16.5, 1024 rows
                // 21.3 / 25.2, 2048 rows 44.9 / 40.7; 1.5B at 512 rows 41.5 / 53.4, 3B at 2048
                // rows 160 / 197.
                const long t256 = mb * ((N / 2 + 127) / 128);
                if ((t256 >= 128 && t256 <= 256) || t256 % 256 >= 128 || t256 >= 4 * 256)
                    return run_wide<2, 4, 4, 2, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, st);
                // one round of 256x128 with three stages: 0.5B at 419 rows 14.9 -> 13.5 us, at 768
                // rows 17.5 -> 16.7
                if (mb * ((ff + 63) / 64) <= 256)
                    return run_wide<4, 2, 2, 2, EPI_SWIGLU, 3>(A, W, C, M, N, K, ldc, 1, 0, st);
                return run_wide<2, 2, 2, 2, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, st);
            }
            if (M > 256) return run_bf16<128, 128, 4, 2, 2, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, st);
            // Small batches: the streaming kernel, on the narrowest tile (h columns) of those
            // below that reads the batch rows no more often than it pays.  us at 48-64 rows,
            // 32 / 64 columns: 0.5B 7.8 / 9.5, 3B 25.3 / 22.0; 128 rows, 64 x 64 / 128 x 64:
            // 0.5B 9.9 / 12.3, 1.5B 27.7 / 20.3, 3B 35.1 / 26.4 (register-staged before: 11.4,
            // 24.7, 32.5).  129-256 rows with more tiles than CUs stay register-staged (1.5B
            // 25.4 against 27-35 us at 192 rows).
            const long t64 = (N / 2 + 63) / 64;
            if (M <= 32) return run_stream<1, 1, 2, 16, 4, EPI_SWIGLU, true>(A, W, C, M, N, K, ldc, 1, 0, st);
            if (M <= 64 && t64 < 128) return run_stream<2, 1, 2, 32, 4, EPI_SWIGLU, true>(A, W, C, M, N, K, ldc, 1, 0, st);
            if ((M + 63) / 64 * t64 <= 256) return run_stream<2, 2, 2, 32, 4, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, st);
            if ((M + 127) / 128 * t64 <= 256) return run_stream<4, 2, 2, 32, 4, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, st);
            return run_bf16<64, 128, 2, 2, 2, EPI_SWIGLU>(A, W, C, M, N, K, ldc, 1, 0, st);
        }
        if (N >= 8192) {  // LM head: many tiles, the largest tile that the batch fills wins
            // one row block: two work-groups of four 32 x 32 (eight) blocks a CU
            if (M <= 32) return run_stream<1, 4, 1, 32, 4, EPI_STORE_F32, true>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (M <= 64) return run_stream<2, 4, 1, 32, 3, EPI_STORE_F32, true>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (M <= 128)  // measured 10-18% faster than 256x256 at 96-128 rows
                return run_bf16<128, 256, 4, 4, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            // wide tiles past one 256-row block (there 2% slower at K = 2048): 0.5B at 419 rows 169
            // -> 163 us, 1.5B at 1024 rows 516 -> 505, at 8192 rows 9%
            if (M > 256)
                return run_wide<2, 4, 4, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            return run_bf16<256, 256, 4, 4, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
        }
        // Small launches of the other projections: the streaming kernel, on the smallest tile
        // that gives no more work-groups than CUs (short reductions: 32 rows x 16 columns,
        // 32 x 32, 64 x 32; the split down projection, whose rows are fewer but longer, up
        // to 128 x 64).  us against the register-staged tiles at 128 / 256 rows: QKV 0.5B 5.0
        // / 6.1 (6.0 / 6.7), 1.5B 6.3 / 8.1 (8.0 / 9.5); down 0.5B 6.3 / 8.1 (6.7 / 9.3), 1.5B
        // 11.6 / 15.6 (12.3 / 19.0), 3B 16.5 / 22.2 (17.7 / 27.9).  A tile past one round loses
        // (3B QKV at 192 rows on 480 32 x 32 tiles 10.8, on 240 64 x 32 tiles 9.9).
        const auto tiles = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * nsplit; };
        if (K < 4096) {
            if (tiles(32, 16) <= 256)
                return run_stream<1, 1, 1, 16, 8, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (tiles(32, 32) <= 256)
                return run_stream<1, 1, 1, 32, 8, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (tiles(64, 32) <= 256)
                return run_stream<2, 1, 1, 32, 8, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
        } else {  // split counts give up to 288 tiles per row block
            if (tiles(32, 32) <= 288)
                return run_stream<1, 1, 1, 32, 8, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (tiles(64, 32) <= 288)
                return run_stream<2, 1, 1, 32, 8, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (tiles(64, 64) <= 288)
                return run_stream<2, 2, 1, 32, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (tiles(128, 64) <= 288)
                return run_stream<4, 2, 1, 32, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
        }
        if (K < 4096 && M >= 256 && M <= 4096) {
            // Unsplit short reductions (the output projection; QKV where it is not fused):
            // the direct-to-LDS kernel, on the largest tile that still gives the launch
            // about 160 or more work-groups.  Measured on the 0.5B, 1.5B and 3B shapes at
            // 256-2048 rows (dash_gemm_bench, weights cold): 7-36% faster than the
            // register-staged tiles (1.5B at 1024 rows: 14.8 -> 10.5 us).
            // 64x64 tiles while they fit one round (<= 256 work-groups): 15-17% faster than
            // 128x64 for the 0.5B shape at 768-1024 rows
            if ((long)((M + 63) / 64) * ((N + 63) / 64) <= 256)
                return run_lds<64, 64, 2, 2, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            // 128x128 with eight waves and four stages where they fit one round and 128x64 tiles
            // would start a second: 1.5B at 1665 rows 21.6 -> 14.2 us
            if (tiles(128, 64) > 256 && tiles(128, 128) <= 192)
                return run_wide<4, 2, 1, 2, EPI_STORE_F32, 4>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (M <= 1024 || (long)(M / 128) * ((N + 127) / 128) < 160)
                return run_lds<128, 64, 2, 2, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            return run_lds<128, 128, 2, 2, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
        }
        // wide projections at up to 256 rows: narrow tiles, four k-steps in flight per thread
        if (M <= 256 && K < 4096)
            return run_bf16<64, 32, 2, 1, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
        // Larger batches: the largest tile that still gives the launch enough work-groups.
        // Measured crossovers on the 0.5B, 1.5B and 3B shapes: the split down projection 64x64 up
        // to 384 rows (12-19% faster than 64x32 there), the direct-to-LDS 128x128 tiles up to
        // 640, 128x256 up to 1024, 256x256 past that (12-18% faster from 1536 rows); unsplit
        // projections 256x256 past 4096 rows (15-26% faster than 128x128 at 8192-16384).
        if (K >= 4096) {
            if (M <= 384)
                return run_bf16<64, 64, 2, 2, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (M <= 640)  // direct-to-LDS 128x128: 23-35% faster at 512 rows on all three shapes
                return run_lds<128, 128, 2, 2, 4, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            // 256x128 with three stages while one round holds them and a split's chain is long:
            // 1.5B / 3B at 768 rows 32.1 -> 28.4 us / 49.8 -> 43.0, at 1024 rows 34.8 -> 31.2 /
            // 53.6 -> 47.2; 0.5B (ten k-steps a split) 16.9 -> 18.1, not used
            if (tiles(256, 128) <= 256 && K / nsplit >= 1024)
                return run_wide<4, 2, 2, 2, EPI_STORE_F32, 3>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            if (M <= 1024)
                return run_bf16<128, 256, 4, 4, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
            return run_wide<2, 4, 4, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
        }
        return run_wide<2, 4, 4, 2, EPI_STORE_F32>(A, W, C, M, N, K, ldc, nsplit, split_stride, st);
    }
    if (nsplit != 1) return hipErrorInvalidValue;
    if (epi == EPI_SWIGLU) {
        dim3 grid((N / 2 + 31) / 32, (M + 63) / 64);
        gemm_f32_k<EPI_SWIGLU><<<grid, 256, 0, st>>>((const float*)A, (const float*)W, C, M, N, K, ldc);
    } else {
        dim3 grid((N + 63) / 64, (M + 63) / 64);
        gemm_f32_k<EPI_STORE_F32><<<grid, 256, 0, st>>>((const float*)A, (const float*)W, C, M, N, K, ldc);
    }
    return hipGetLastError();
}

}  // namespace dash
