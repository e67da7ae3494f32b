// Projections of the action expert over the stacked action tokens of the
// whole batch: C[M][N] = A[M][K] W with W stored transposed ([N][K], K
// contiguous) so that both MFMA operands are K-contiguous 16-byte loads.
//
// Epilogues fuse what follows each projection: plain store (QKV), tanh-GELU
// (MLP up), and the gated residual h += gate * C whose gate row is the
// row's flow-time modulation (attention output and MLP down).  Smaller launches
// may split K over several blocks per tile: each block stores its slice's
// fp32 product (kEpiPartial) and a second kernel sums the slices in order and
// applies the epilogue, taking the next norm with it.  A few tens of rows run
// in a kernel of their own (gemm_direct_kernel).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "rosa_device.h"
#include "rosa_internal.h"

namespace rosa {

// ------------------------------------------------------------------ bf16 MFMA GEMM
// Block tile BM x BN = (32 MB) x (32 TN WN), WM x WN waves, each wave
// (32 MB / WM) x (32 TN) made of 32 x 32 v_mfma_f32_32x32x16_bf16 tiles.
//
// Main loop: K is consumed BK (32 or 64) at a time through a ring of NST
// LDS stages filled by global_load_lds_dwordx4 (global -> LDS without
// staging registers).  Operand fragments are read from LDS LA k-steps (16 of K)
// ahead of their MFMAs into a ring of register sets: an LDS read takes longer
// than a k-step of a small wave tile (two to four MFMAs), and one wave per SIMD
// has nothing else to run meanwhile, so one k-step ahead left each of them
// waiting (128 x 128 tile, data in L2: 0.345 us per 64 of K one k-step ahead,
// 0.26 three ahead, which is what 32 KB take at the 125 GB/s a CU's copies
// reach).  One barrier per stage, crossed before the first look-ahead into the
// next stage; by then the whole stage is in registers, so its buffer is
// refilled at once and NST - 1 stages are in flight or landed (the smallest
// tiles refill the stage before it, see BACK).  The copies are
// issued as inline assembly the compiler does not track and the barrier is a
// bare s_barrier, so the only wait on them is the explicit vmcnt before it.
//
// LDS rows are 64 bytes (32 bf16 of K); the four 16-byte chunks of row r are
// stored XOR-swizzled by (r / 4) % 4, so the 16 rows a 16-lane group reads at
// one logical chunk land in 16 distinct bank groups.  A copy instruction
// writes lane i to byte 16 i of a 1 KB block (16 rows), so each lane fetches
// the logical chunk that belongs at its physical position.
//
// The MFMA takes the weight fragment as its first operand, so a lane's
// accumulator registers hold four consecutive output columns of one output row.
// The epilogue stages each 32 x 32 accumulator tile through LDS and writes
// whole 64- or 128-byte row segments with 16-byte accesses.
//
// Blocks are mapped to tiles so that each of the 8 XCDs (which receive blocks
// round-robin) works on a contiguous range of the tile list, which runs in
// strips of a few column tiles: the tiles an XCD holds at a time are a
// near-square patch, so they share rows of both operands in its L2.
namespace gb {
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }   // and lgkmcnt(0)
// f(integral_constant<int, i>) for i = 0 .. N - 1, in order.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}
}  // namespace gb


// Chunk swizzle of an LDS row of CPR 16-byte chunks: chunk c of row r is
// stored at c ^ gswz(r).  64-byte rows (CPR 4): (r / 4) % 4; 128-byte rows
// (CPR 8): (r / 2) % 8.  Either way the 16 rows a 16-lane group reads at one
// logical chunk fall in 16 distinct bank groups.
template <int CPR>
__device__ __forceinline__ int gswz(int r) { return CPR == 4 ? (r >> 2) & 3 : (r >> 1) & 7; }

template <int MB_, int TN_, int WM_, int WN_, int BK_ = 32, int NST_ = 4, int LA_ = 1, int BACK_ = 0>
struct GemmTile {
  static constexpr int MB = MB_, TN = TN_, WM = WM_, WN = WN_, NW = WM_ * WN_, NT = 64 * NW;
  static constexpr int MBW = MB / WM;                                   // 32-row blocks per wave
  static constexpr int BM = 32 * MB, BN = 32 * TN * WN;
  static constexpr int BK = BK_;                                        // K per stage
  static constexpr int ROWB = BK * 2, CPR = ROWB / 16, RPU = 1024 / ROWB;   // row bytes, chunks per row, rows per 1 KB
  static constexpr int ABYTES = BM * BK * 2, SBYTES = ABYTES + BN * BK * 2;
  // LDS ring depth: 4; 6 or 8 for the small tiles of small launches (one
  // block per CU, latency-bound: more copies in flight per CU; 128 x 64 at 816
  // rows, N = 2048, K = 16384: 102 us with 4 stages, 88 with 6).
  static constexpr int NST = NST_;
  static_assert(NST * SBYTES <= 160 * 1024, "LDS");
  // k-steps of operand fragments read ahead of their MFMAs, in NSET register
  // sets (a divisor of the ring's k-steps, so the sets repeat with the ring).
  static constexpr int NKS = BK / 16, LA = LA_, NSET = LA_ < 2 ? 2 : 4;
  static_assert(LA >= 1 && LA <= NKS && LA < NSET && NST * NKS % NSET == 0, "look-ahead");
  // BACK 0: a stage boundary refills the buffer of the stage just read, so the
  // block waits there for its own LDS reads of it; 1: the one read before
  // that (one stage less in flight, no such wait).  The small tiles have too few
  // MFMAs per k-step to cover that wait (64 x 64 and 64 x 32: 5 - 8% of a launch).
  static constexpr int BACK = BACK_;
  static_assert(BACK == 0 || BACK == 1, "refill distance");
  static constexpr int U = (BM + BN) / RPU;                             // 1 KB copies per stage
  static_assert(BK == 32 || BK == 64, "stage K");
  static constexpr int CHI = (U + NW - 1) / NW, CLO = U / NW;           // copies per wave
  static constexpr int NHI = U % NW == 0 ? NW : U % NW;                 // waves with CHI copies
  static_assert(MBW * WM == MB, "row split");
  static_assert(NW * 4096 <= NST * SBYTES, "epilogue staging space (4 KB per wave)");
};

// K stages [kt0, kt0 + nk) of the tile at (m0, n0) into acc (zeroed first).
// Ends with every copy landed and every wave past its last LDS read.
template <typename T>
__device__ __forceinline__ void gemm_mainloop(const GemmArgs &g, int m0, int n0, int kt0, int nk, uint8_t *L,
                                              f32x16 (&acc)[T::MBW][T::TN]) {
  using namespace gb;
  constexpr int NW = T::NW, MBW = T::MBW, TN = T::TN, CHI = T::CHI, CLO = T::CLO, NST = T::NST;
  constexpr int ABYTES = T::ABYTES, SBYTES = T::SBYTES;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % NW;   // wave-uniform, in an SGPR
  const int wm = wave / T::WN, wn = wave % T::WN;
  const bf16 *A = reinterpret_cast<const bf16 *>(g.a);
  const bf16 *W = reinterpret_cast<const bf16 *>(g.wt);

  // Copy sources: 1 KB unit u (A rows first, then W rows) is copied by wave
  // u % NW; lane i writes physical chunk i % CPR of row i / CPR of the unit,
  // which holds logical chunk (i % CPR) ^ gswz(row).  Both operands are kb32
  // (planes of R rows: a_rows for A, N for W), so logical chunk c of a row
  // (k = k0 + 8 c) lies in plane k0 / 32 + c / 4 and a unit reads one (32 of
  // K) or two (64 of K) contiguous 512 B - 1 KB runs.  Rows past M (or N)
  // re-read the last row; their results are never stored.
  constexpr int CPR = T::CPR, RPU = T::RPU;
  const bf16 *src[CHI];
  size_t kstep[CHI];                        // elements per 32 of K: 32 R
#pragma unroll
  for (int j = 0; j < CHI; ++j) {
    const int u = min(j * NW + wave, T::U - 1);
    const int lrow = u * RPU + lane / CPR;                   // row within the stage
    const int csrc = (lane % CPR) ^ gswz<CPR>(lrow);
    if (u < T::BM / RPU) {
      const int row = min(m0 + lrow, g.M - 1);
      kstep[j] = (size_t)g.a_rows * 32;
      src[j] = A + ((size_t)(csrc >> 2) * g.a_rows + row) * 32 + (csrc & 3) * 8;
    } else {
      const int row = min(n0 + lrow - T::BM, g.N - 1);
      kstep[j] = (size_t)g.N * 32;
      src[j] = W + ((size_t)(csrc >> 2) * g.N + row) * 32 + (csrc & 3) * 8;
    }
  }
  const bool hi = wave < T::NHI;
  constexpr int BK = T::BK, ROWB = T::ROWB;
  // Copy j (of CHI) of this wave for stage kt into buffer st.
  auto issue_one = [&](uint8_t *st, int kt, int j) __attribute__((always_inline)) {
    const int kb = (kt0 + min(kt, nk - 1)) * (BK / 32);   // past the end: repeat the last stage (never read)
    if (j < CLO || hi) dma_1k(src[j] + (size_t)kb * kstep[j], lds_u32(st) + (uint32_t)((j * NW + wave) * 1024));
  };
  auto issue = [&](uint8_t *st, int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < CHI; ++j) issue_one(st, kt, j);
  };

#pragma unroll
  for (int i = 0; i < MBW; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Operand reads: lane reads row (lane & 31) of a 32-row block, logical chunk
  // 2 ks + lane / 32, at physical chunk (logical) ^ gswz(row); every 32-row
  // block starts at a multiple of 32 rows, so the swizzle depends on lane & 31.
  constexpr int NKS = T::NKS;
  const int swz = gswz<CPR>(lane & 31);
  int ph[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) ph[ks] = ((2 * ks + (lane >> 5)) ^ swz) * 16;
  const int arow = (wm * MBW * 32 + (lane & 31)) * ROWB;
  const int brow = ABYTES + (wn * TN * 32 + (lane & 31)) * ROWB;
  // Fragments (MBW A tiles, TN W tiles) of NSET k-steps: k-step q is
  // multiplied from register set q % NSET while k-step q + LA is read from LDS.
  constexpr int LA = T::LA, NSET = T::NSET;
  bf16x8 fa[NSET][MBW], fb[NSET][TN];
  auto read_frags = [&](const uint8_t *st, auto ks_t, auto set_t) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_t)::value, f = decltype(set_t)::value;
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[f][j] = *reinterpret_cast<const bf16x8 *>(st + brow + j * 32 * ROWB + ph[ks]);
#pragma unroll
    for (int i = 0; i < MBW; ++i) fa[f][i] = *reinterpret_cast<const bf16x8 *>(st + arow + i * 32 * ROWB + ph[ks]);
  };
  constexpr int NMF = MBW * TN, NMS = LA * NMF;   // MFMAs per k-step, and per stage after its barrier
  constexpr int NFL = NST - T::BACK;              // stages in flight or landed after a refill
  // Stage kt in buffer `cur`.  Before k-step NKS - LA, whose look-ahead is the
  // first read of stage kt + 1, the block crosses the stage boundary: the wait
  // covers this wave's copies of stage kt + 1 (stages kt + 2 .. kt + NFL - 1 may
  // still be in flight) and, with BACK 0, its own reads of stage kt; after the barrier
  // both hold for every wave, so the buffer of stage kt (BACK 1: of stage kt - 1, whose
  // reads every wave's MFMAs have consumed by then) is free and takes stage kt + NFL.  The
  // copies are spread evenly over the stage's remaining MFMAs, so no wave
  // stalls on a burst of them.
  auto stage = [&](auto cur_t, int kt) __attribute__((always_inline)) {
    constexpr int cur = decltype(cur_t)::value;
    constexpr int nxt = cur + 1 == NST ? 0 : cur + 1, fill = (cur + NFL) % NST;
    static_for<NKS>([&](auto ks_t) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_t)::value, q = cur * NKS + ks;
      if constexpr (ks == NKS - LA) {
        if constexpr (T::BACK == 0) {
          if (hi) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NFL - 2) * CHI));
          else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NFL - 2) * CLO));
        } else {
          if (hi) __builtin_amdgcn_s_waitcnt(waitcnt_vm((NFL - 2) * CHI));
          else __builtin_amdgcn_s_waitcnt(waitcnt_vm((NFL - 2) * CLO));
        }
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      read_frags(L + (ks + LA < NKS ? cur : nxt) * SBYTES, std::integral_constant<int, (ks + LA) % NKS>{},
                 std::integral_constant<int, (q + LA) % NSET>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[q % NSET][j], fa[q % NSET][i], acc[i][j], 0, 0, 0);
          if constexpr (ks >= NKS - LA) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < CHI; ++c)
              if ((c * NMS) / CHI == (ks - (NKS - LA)) * NMF + i * TN + j) issue_one(L + fill * SBYTES, kt + NFL, c);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Prologue: stages 0 .. NFL - 1 requested, stage 0 landed and its first LA
  // k-steps being read.
#pragma unroll
  for (int st = 0; st < NFL; ++st) issue(L + st * SBYTES, st);
  if (hi) __builtin_amdgcn_s_waitcnt(waitcnt_vm((NFL - 1) * CHI));
  else __builtin_amdgcn_s_waitcnt(waitcnt_vm((NFL - 1) * CLO));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  static_for<LA>([&](auto ks_t) { read_frags(L, ks_t, ks_t); });
  // Groups of NST stages, unrolled so that every buffer offset and register
  // set is an immediate, then the remaining stages.
  int kt = 0;
  for (; kt + NST <= nk; kt += NST)
    static_for<NST>([&](auto r) { stage(r, kt + decltype(r)::value); });
  static_for<NST - 1>([&](auto r) {
    if (kt + decltype(r)::value < nk) stage(r, kt + decltype(r)::value);
  });
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __syncthreads();                          // every wave is past its last stage read: LDS is free
}

// 1 / rms and modulation row of this lane's row in each of its 32-row blocks,
// for the completion of a deferred norm.
template <typename T>
struct NormRows { float rinv[T::MBW]; int mrow[T::MBW]; };

// The rows' sums of squares are summed over the two lane halves (each half sums
// its share of the row's block sums in order; the halves' totals are then added).
// Called before the main loop, whose first copies cover these loads.
template <typename T>
__device__ __forceinline__ void gemm_norm_rows(const GemmArgs &g, int m0, NormRows<T> &nr) {
  constexpr int MBW = T::MBW;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % T::NW;
  const int wm = wave / T::WN, r32 = lane & 31, half = lane >> 5;
  // Every load is issued before the first sum (cparts = 8 nv, nv <= 4).
  const int nv = g.cparts >> 3;
  f32x4 pv[MBW][4];
#pragma unroll
  for (int i = 0; i < MBW; ++i) {
    const int row = min(m0 + (wm * MBW + i) * 32 + r32, g.M - 1);
    const f32x4 *sp = reinterpret_cast<const f32x4 *>(g.css + (size_t)row * g.cparts) + half * nv;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (v < nv) pv[i][v] = sp[v];
    nr.mrow[i] = g.rowmod[row];
  }
#pragma unroll
  for (int i = 0; i < MBW; ++i) {
    float ss = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (v < nv) ss = (((ss + pv[i][v][0]) + pv[i][v][1]) + pv[i][v][2]) + pv[i][v][3];
    ss += __shfl_xor(ss, 32, 64);
    nr.rinv[i] = 1.0f / sqrtf(ss / (float)g.cd + g.ceps);
  }
}

// Epilogue of the tile at (m0, n0) from acc; stages through the ring's LDS,
// which must be free (gemm_mainloop ends that way).  DN: the deferred norm's
// part of the epilogue (outputs t and the row sums of squares after a gated
// residual; the norm's completion before a bf16 store).
template <typename T, int EPI, bool DN = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &g, int m0, int n0, uint8_t *L,
                                              f32x16 (&acc)[T::MBW][T::TN], const NormRows<T> &nr) {
  constexpr int MBW = T::MBW, TN = T::TN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % T::NW;
  const int wm = wave / T::WN, wn = wave % T::WN;
  // Register r of tile (i, j) holds row m0 + 32 (wm MBW + i) + lane % 32,
  // columns n0 + 32 (wn TN + j) + 8 (r / 4) + 4 (lane / 32) + r % 4: four
  // consecutive columns per 4 registers.
  const int r32 = lane & 31, half = lane >> 5;
  if constexpr (EPI == kEpiGatedResidual || EPI == kEpiPartial) {
    // h += gate[rowmod[row]] * acc (or, for a K slice, out = acc in fp32).
    // Each wave stages one 32 x 32 tile at a
    // time in its own 4 KB slot (fp32: 32 rows x 8 chunks of 16 B, chunk c of
    // row r at c ^ ((r / 2) % 8)), then reads it back row-contiguous.
    uint8_t *stg = L + wave * 4096;
    float *H = reinterpret_cast<float *>(g.out);
    // Gate rows of every row this lane touches, loaded once up front so that
    // no gate load waits for its row's modulation index (32-bit offsets: the
    // gate table has far fewer than 2^31 elements).
    int goff[EPI == kEpiGatedResidual ? MBW : 1][4];
    if constexpr (EPI == kEpiGatedResidual) {
#pragma unroll
      for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int row = min(m0 + (wm * MBW + i) * 32 + 8 * p + (lane >> 3), g.M - 1);
          goff[i][p] = g.rowmod[row] * g.gate_stride;
        }
    }
    // Pass p of 32 x 32 tile q = i TN + j: rows 8 p + lane / 8, columns
    // 4 (lane % 8) .. + 3.  The residual and gate rows of tile q + 1 are
    // requested before tile q is combined, so each tile's global loads wait
    // behind the previous tile's work instead of stalling on their own
    // (two register sets; tiles small enough to run two blocks per CU, and the
    // deferred norm's, which load scale rows too, have no registers to spare and
    // load each tile's rows just before use).
    constexpr int Q = MBW * TN;
    constexpr bool kTwoBlocks = T::NST * T::SBYTES <= 80 * 1024;
    constexpr int NB = (EPI == kEpiGatedResidual && !kTwoBlocks && !DN) ? 2 : 1;
    float4 hv[NB][4], gt[NB][4];
    // The deferred norm's scale rows load with the tile's other rows.
    float4 scv[DN ? NB : 1][4];
    const int col0 = (lane & 7) * 4;
    auto load_rows = [&](int q, int buf) __attribute__((always_inline)) {
      const int i = q / TN, j = q % TN;
      const int rb = m0 + (wm * MBW + i) * 32, col = n0 + (wn * TN + j) * 32 + col0;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int row = rb + 8 * p + (lane >> 3);
        if (row < g.M && col < g.N) {
          hv[buf][p] = *reinterpret_cast<const float4 *>(H + (size_t)row * g.ldo + col);
          gt[buf][p] = *reinterpret_cast<const float4 *>(g.gate + goff[i][p] + col);
          if constexpr (DN) scv[buf][p] = *reinterpret_cast<const float4 *>(g.dscale + goff[i][p] + col);
        }
      }
    };
    if constexpr (EPI == kEpiGatedResidual && NB == 2) load_rows(0, 0);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = q / TN, j = q % TN, buf = NB == 2 ? (q & 1) : 0;
      if constexpr (EPI == kEpiGatedResidual) {
        if (NB == 1) load_rows(q, 0);
        else if (q + 1 < Q) load_rows(q + 1, (q + 1) & 1);
      }
      const int rb = m0 + (wm * MBW + i) * 32, col = n0 + (wn * TN + j) * 32 + col0;
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int c = (2 * gq + half) ^ ((r32 >> 1) & 7);
        *reinterpret_cast<float4 *>(stg + r32 * 128 + c * 16) =
            make_float4(acc[i][j][4 * gq], acc[i][j][4 * gq + 1], acc[i][j][4 * gq + 2], acc[i][j][4 * gq + 3]);
      }
      float4 v[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int rr = 8 * p + (lane >> 3), c = lane & 7;
        v[p] = *reinterpret_cast<const float4 *>(stg + rr * 128 + ((c ^ ((rr >> 1) & 7)) * 16));
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int row = rb + 8 * p + (lane >> 3);
        float q2 = 0.f;
        if (row < g.M && col < g.N) {
          if constexpr (EPI == kEpiPartial) {
            *reinterpret_cast<float4 *>(H + (size_t)row * g.ldo + col) = v[p];
          } else {
            float4 h = hv[buf][p];
            h.x = h.x + gt[buf][p].x * v[p].x;
            h.y = h.y + gt[buf][p].y * v[p].y;
            h.z = h.z + gt[buf][p].z * v[p].z;
            h.w = h.w + gt[buf][p].w * v[p].w;
            *reinterpret_cast<float4 *>(H + (size_t)row * g.ldo + col) = h;
            if constexpr (DN) {
              const float4 sc = scv[buf][p];
              bf16x4 tv;
              tv[0] = (bf16)(h.x * (1.0f + sc.x));
              tv[1] = (bf16)(h.y * (1.0f + sc.y));
              tv[2] = (bf16)(h.z * (1.0f + sc.z));
              tv[3] = (bf16)(h.w * (1.0f + sc.w));
              *reinterpret_cast<bf16x4 *>(reinterpret_cast<bf16 *>(g.dt) + kb32_offset(g.dt_rows, row, col)) = tv;
              q2 = fmaf(h.w, h.w, fmaf(h.z, h.z, fmaf(h.y, h.y, h.x * h.x)));
            }
          }
        }
        if constexpr (DN) {
          // The row's 32 columns of this tile sit on the 8 lanes lane / 8
          // shares; their sum (fixed butterfly order) goes to the row's entry.
          q2 += __shfl_xor(q2, 1, 64);
          q2 += __shfl_xor(q2, 2, 64);
          q2 += __shfl_xor(q2, 4, 64);
          if ((lane & 7) == 0 && row < g.M && col < g.N) g.dss[(size_t)row * (g.N >> 5) + (col >> 5)] = q2;
        }
      }
    }
  } else {
    // Each wave stages one 32 x 32 tile at a time in its own 4 KB slot, then
    // reads it back row-contiguous.
    uint8_t *stg = L + wave * 4096;
    // Deferred norm: the shift rows of a 32 x 32 tile's columns, requested one
    // tile ahead (the first before the others' LDS staging starts).
    constexpr int Q = MBW * TN;
    f32x4 sh[DN ? 2 : 1][4];
    auto load_shift = [&](int q, f32x4 (&dst)[4]) __attribute__((always_inline)) {
      const float *shrow = g.cshift + (size_t)nr.mrow[q / TN] * g.cshift_stride;
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int c4 = n0 + (wn * TN + q % TN) * 32 + 8 * gq + 4 * half;
        dst[gq] = c4 < g.N ? *reinterpret_cast<const f32x4 *>(shrow + c4) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    };
    if constexpr (DN) load_shift(0, sh[0]);
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int rb = m0 + (wm * MBW + i) * 32, cb = n0 + (wn * TN + j) * 32;
        const int q = i * TN + j;
        if constexpr (DN) {
          if (q + 1 < Q) load_shift(q + 1, sh[(q + 1) & 1]);
        }
        // bf16 slot: 32 rows x 4 chunks of 16 B (8 bf16), chunk c of row r at
        // c ^ ((r / 4) % 4); this lane's 4 values are half `half` of chunk gq.
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          float a0 = acc[i][j][4 * gq], a1 = acc[i][j][4 * gq + 1], a2 = acc[i][j][4 * gq + 2], a3 = acc[i][j][4 * gq + 3];
          if constexpr (DN) {
            const f32x4 sv = sh[q & 1][gq];
            a0 = fmaf(a0, nr.rinv[i], sv[0]);
            a1 = fmaf(a1, nr.rinv[i], sv[1]);
            a2 = fmaf(a2, nr.rinv[i], sv[2]);
            a3 = fmaf(a3, nr.rinv[i], sv[3]);
          }
          if constexpr (EPI == kEpiGelu) {
            a0 = gelu_tanh_f(a0); a1 = gelu_tanh_f(a1); a2 = gelu_tanh_f(a2); a3 = gelu_tanh_f(a3);
          }
          bf16x4 o;
          o[0] = (bf16)a0; o[1] = (bf16)a1; o[2] = (bf16)a2; o[3] = (bf16)a3;
          const int c = gq ^ ((r32 >> 2) & 3);
          *reinterpret_cast<bf16x4 *>(stg + r32 * 64 + c * 16 + half * 8) = o;
        }
        // Pass p: rows 16 p + lane / 4, columns 8 (lane % 4) .. + 7.
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int rr = 16 * p + (lane >> 2), c = lane & 3;
          const bf16x8 v = *reinterpret_cast<const bf16x8 *>(stg + rr * 64 + ((c ^ ((rr >> 2) & 3)) * 16));
          const int row = rb + rr, col = cb + c * 8;
          if (row < g.M && col < g.N) {
            const size_t off = g.out_rows > 0 ? kb32_offset(g.out_rows, row, col) : (size_t)row * g.ldo + col;
            *reinterpret_cast<bf16x8 *>(reinterpret_cast<bf16 *>(g.out) + off) = v;
          }
        }
      }
  }
}

template <typename T, int EPI, bool DN = false>
__global__ void __launch_bounds__(T::NT) gemm_bf16_kernel(GemmArgs g, int nrt, int nct, int ksplit, int strip) {
  constexpr int SBYTES = T::SBYTES;
  __shared__ __attribute__((aligned(1024))) uint8_t L[T::NST * SBYTES];

  // Work unit of this block: XCD x = b % 8 takes the x-th eighth of the unit
  // list; unit u is K slice u / n_tiles of tile u % n_tiles (one slice
  // unless the product is split).  Tiles are listed strip by strip (strips of
  // `strip` column tiles), row-major within a strip.
  const int n_tiles = nrt * nct, n_units = n_tiles * ksplit;
  const int b = blockIdx.x, x = b & 7, q = b >> 3;
  const int per = n_units >> 3, extra = n_units & 7;
  if (q >= per + (x < extra ? 1 : 0)) return;
  const int unit = x * per + min(x, extra) + q;
  // Each division here is a chain of some tens of instructions before the
  // tile's first copy: only split launches divide by the slices.
  const int nk = g.K / T::BK;
  int tile = unit, slice = 0, kt0 = 0, kt1 = nk;
  if constexpr (EPI == kEpiPartial) {
    slice = unit / n_tiles;
    tile = unit - slice * n_tiles;
    kt0 = nk * slice / ksplit;
    kt1 = nk * (slice + 1) / ksplit;
  }
  const int sidx = tile / (nrt * strip);    // strips before the last are `strip` columns wide
  const int in_strip = tile - sidx * nrt * strip, width = min(strip, nct - sidx * strip);
  const int row = in_strip / width;
  const int m0 = row * T::BM, n0 = (sidx * strip + in_strip - row * width) * T::BN;
  f32x16 acc[T::MBW][T::TN];
  NormRows<T> nr;
  if constexpr (DN && EPI != kEpiGatedResidual) gemm_norm_rows<T>(g, m0, nr);
  gemm_mainloop<T>(g, m0, n0, kt0, kt1 - kt0, L, acc);
  if constexpr (EPI == kEpiPartial) {
    GemmArgs gp = g;
    gp.out = g.part + (size_t)slice * g.M * g.N;
    gp.ldo = g.N;
    gemm_epilogue<T, EPI>(gp, m0, n0, L, acc, nr);
  } else {
    gemm_epilogue<T, EPI, DN>(g, m0, n0, L, acc, nr);
  }
}

// Block configurations and their measured cost on MI355X: a launch takes
// kLaunchUs plus, per round of blocks over all CUs, a per 1024 of K plus b by
// epilogue (store, GELU, gated residual), in microseconds; past K = 4096 a
// round costs a2 more per 1024 of K.  Least-squares fits to the eight
// projection shapes of the action expert and the vision-language backbone
// (and the context projection) at 50 - 25600 rows with cold weights: over
// those 105 shapes the tile this picks is 1% slower than the best one on
// average.
constexpr float kLaunchUs = 2.5f;
struct GemmCfg { int bm, bn, bk; float a, a2, b[3]; };
static constexpr GemmCfg kCfgs[kGemmConfigs] = {
    {384, 128, 32, 21.3f, -0.3f, {2.1f, 6.4f, 6.5f}},          // 0: 8 waves, 96 x 64 each
    {256, 256, 32, 25.5f, -3.1f, {3.4f, 7.1f, 10.1f}},         // 1: 8 waves, 128 x 64 each
    {128, 256, 32, 13.5f, -0.7f, {2.8f, 4.8f, 7.0f}},          // 2: 8 waves, 64 x 64 each
    {192, 128, 32, 11.2f, 0.4f, {1.3f, 2.6f, 4.7f}},           // 3: 8 waves, 96 x 32 each
    {288, 128, 32, 16.8f, -1.1f, {3.2f, 5.3f, 8.6f}},          // 4: 12 waves, 96 x 32 each
    {128, 64, 64, 4.9f, 0.3f, {2.2f, 3.2f, 4.1f}},             // 5: 4 waves, 64 x 32 each, 6 stages
    {192, 128, 64, 10.9f, 0.4f, {2.8f, 4.9f, 7.0f}},           // 6: 8 waves, 96 x 32 each
    {128, 128, 64, 7.6f, 1.1f, {2.2f, 3.8f, 5.7f}},            // 7: 4 waves, 64 x 64 each
    {160, 128, 64, 9.3f, 0.1f, {2.4f, 4.7f, 9.2f}},            // 8: 4 waves, 160 x 32 each
    {96, 128, 64, 6.4f, 0.5f, {1.6f, 2.9f, 5.1f}},             // 9: 4 waves, 96 x 32 each
    {256, 64, 64, 8.9f, 0.9f, {1.8f, 3.2f, 4.0f}},             // 10: 8 waves, 64 x 32 each
    {64, 64, 64, 3.3f, 0.4f, {1.0f, 1.6f, 1.7f}},              // 11: 4 waves, 32 x 32 each, 8 stages
    {64, 32, 64, 2.5f, 0.0f, {1.3f, 1.7f, 1.6f}},              // 12: 2 waves, 32 x 32 each, 8 stages
};
using Cfg0 = GemmTile<12, 2, 4, 2, 32, 4, 2>;
using Cfg1 = GemmTile<8, 2, 2, 4, 32, 4, 1>;
using Cfg2 = GemmTile<4, 2, 2, 4, 32, 4, 2>;
using Cfg3 = GemmTile<6, 1, 2, 4, 32, 4, 1>;
using Cfg4 = GemmTile<9, 1, 3, 4, 32, 4, 2>;
using Cfg5 = GemmTile<4, 1, 2, 2, 64, 6, 3, 1>;
using Cfg6 = GemmTile<6, 1, 2, 4, 64, 4, 3>;
using Cfg7 = GemmTile<4, 2, 2, 2, 64, 4, 3>;
using Cfg8 = GemmTile<5, 1, 1, 4, 64, 4, 3>;
using Cfg9 = GemmTile<3, 1, 1, 4, 64, 4, 3>;
using Cfg10 = GemmTile<8, 1, 4, 2, 64, 4, 3>;
using Cfg11 = GemmTile<2, 1, 2, 2, 64, 8, 1, 1>;
using Cfg12 = GemmTile<2, 1, 2, 1, 64, 8, 1, 1>;
template <typename T>
constexpr bool cfg_matches(const GemmCfg &c) { return T::BM == c.bm && T::BN == c.bn && T::BK == c.bk; }
static_assert(cfg_matches<Cfg0>(kCfgs[0]) && cfg_matches<Cfg1>(kCfgs[1]) && cfg_matches<Cfg2>(kCfgs[2]) &&
              cfg_matches<Cfg3>(kCfgs[3]) && cfg_matches<Cfg4>(kCfgs[4]) && cfg_matches<Cfg5>(kCfgs[5]) &&
              cfg_matches<Cfg6>(kCfgs[6]) && cfg_matches<Cfg7>(kCfgs[7]) && cfg_matches<Cfg8>(kCfgs[8]) &&
              cfg_matches<Cfg9>(kCfgs[9]) && cfg_matches<Cfg10>(kCfgs[10]) && cfg_matches<Cfg11>(kCfgs[11]) &&
              cfg_matches<Cfg12>(kCfgs[12]),
              "cost table matches the tiles");

// Sum of the K slices of a split product, in slice order, and the epilogue
// of the whole product; 4 consecutive columns per thread.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_split_reduce_kernel(GemmArgs g, int ksplit) {
  const size_t n4 = (size_t)g.M * g.N / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
    const size_t e = i * 4;
    const int row = (int)(e / g.N), col = (int)(e % g.N);
    f32x4 v = *reinterpret_cast<const f32x4 *>(g.part + e);
    for (int s2 = 1; s2 < ksplit; ++s2) {
      const f32x4 p = *reinterpret_cast<const f32x4 *>(g.part + (size_t)s2 * g.M * g.N + e);
      v[0] += p[0]; v[1] += p[1]; v[2] += p[2]; v[3] += p[3];
    }
    if constexpr (EPI == kEpiGatedResidual) {
      float *hp = reinterpret_cast<float *>(g.out) + (size_t)row * g.ldo + col;
      const float4 gt = *reinterpret_cast<const float4 *>(g.gate + (size_t)g.rowmod[row] * g.gate_stride + col);
      float4 hv = *reinterpret_cast<const float4 *>(hp);
      hv.x = hv.x + gt.x * v[0];
      hv.y = hv.y + gt.y * v[1];
      hv.z = hv.z + gt.z * v[2];
      hv.w = hv.w + gt.w * v[3];
      *reinterpret_cast<float4 *>(hp) = hv;
    } else {
      float a0 = v[0], a1 = v[1], a2 = v[2], a3 = v[3];
      if constexpr (EPI == kEpiGelu) {
        a0 = gelu_tanh_f(a0); a1 = gelu_tanh_f(a1); a2 = gelu_tanh_f(a2); a3 = gelu_tanh_f(a3);
      }
      bf16x4 o;
      o[0] = (bf16)a0; o[1] = (bf16)a1; o[2] = (bf16)a2; o[3] = (bf16)a3;
      const size_t off = g.out_rows > 0 ? kb32_offset(g.out_rows, row, col) : (size_t)row * g.ldo + col;
      *reinterpret_cast<bf16x4 *>(reinterpret_cast<bf16 *>(g.out) + off) = o;
    }
  }
}

// The same sum for a gated-residual product, fused with the modulated
// RMSNorm of the updated rows (the norm that reads them next).  One block per
// row, NV pieces of four columns per thread (piece v: columns 1024 v + 4 thread): sum
// the KS slices in slice order, apply the gated residual exactly as above,
// write the row back to h, and normalize it into u (row sum of squares: per
// thread over its pieces in order, per wave, then the four wave sums in wave
// order), so a split product needs no separate norm launch.
template <int KS, int NV>
__global__ void __launch_bounds__(256) gemm_split_reduce_norm_kernel(GemmArgs g, NormArgs nm) {
  static_assert(NV * 1024 <= kFusedNormMax, "columns per row");
  __shared__ float wsum[4];
  const int row = blockIdx.x;
  const int d = g.N;
  const size_t slice = (size_t)g.M * g.N;
  const int mod = g.rowmod[row];
  float *hr = reinterpret_cast<float *>(g.out) + (size_t)row * g.ldo;
  f32x4 hv[NV];
  float sq = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int i = v * 1024 + threadIdx.x * 4;
    hv[v] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (i < d) {
      const float *pr = g.part + (size_t)row * g.N + i;
      f32x4 p[KS];
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2) p[s2] = *reinterpret_cast<const f32x4 *>(pr + s2 * slice);
      const f32x4 gt = *reinterpret_cast<const f32x4 *>(g.gate + (size_t)mod * g.gate_stride + i);
      hv[v] = *reinterpret_cast<const f32x4 *>(hr + i);
      f32x4 a = p[0];
#pragma unroll
      for (int s2 = 1; s2 < KS; ++s2) { a[0] += p[s2][0]; a[1] += p[s2][1]; a[2] += p[s2][2]; a[3] += p[s2][3]; }
#pragma unroll
      for (int k = 0; k < 4; ++k) hv[v][k] = hv[v][k] + gt[k] * a[k];
      *reinterpret_cast<f32x4 *>(hr + i) = hv[v];
    }
    sq += hv[v][0] * hv[v][0] + hv[v][1] * hv[v][1] + hv[v][2] * hv[v][2] + hv[v][3] * hv[v][3];
  }
  const float ss = wave_sum(sq);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float r = 1.0f / sqrtf((((wsum[0] + wsum[1]) + wsum[2]) + wsum[3]) / (float)d + nm.eps);
  const float *mrow = nm.modtab + (size_t)mod * nm.mod_stride;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int i = v * 1024 + threadIdx.x * 4;
    if (i < d) {
      const f32x4 a = *reinterpret_cast<const f32x4 *>(mrow + nm.scale_off + i);
      const f32x4 b = *reinterpret_cast<const f32x4 *>(mrow + nm.shift_off + i);
      bf16x4 o;
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = (bf16)(hv[v][k] * r * (1.0f + a[k]) + b[k]);
      const size_t off = nm.u_rows > 0 ? kb32_offset(nm.u_rows, row, i) : (size_t)row * d + i;
      *reinterpret_cast<bf16x4 *>(reinterpret_cast<bf16 *>(nm.u) + off) = o;
    }
  }
}

// Whether a split gated-residual product can take the norm that follows it.
static bool fusable_norm(const GemmArgs &g, const NormArgs *nm) {
  return nm && nm->u && g.epi == kEpiGatedResidual && g.N <= kFusedNormMax && g.N % 4 == 0 && g.ldo % 4 == 0 &&
         (nm->u_rows == 0 || (nm->u_rows >= g.M && g.N % 32 == 0));
}

// Column tiles per strip of the tile list.  An XCD runs about min(32, a
// launch's eighth) consecutive tiles of the list at a time; strips of
// w = sqrt(c BM / BN) columns make those c tiles near-square in elements, so
// the rows of A and W they read together are fewest.
static int gemm_strip(int nrt, int nct, int ks, int bm, int bn) {
  const float c = std::min(32.0f, std::max(1.0f, (float)nrt * nct * ks / 8));
  return std::max(1, std::min(nct, (int)(sqrtf(c * bm / bn) + 0.5f)));
}

template <int NV>
static void launch_reduce_norm(const GemmArgs &g, const NormArgs &nm, int ks, hipStream_t s) {
  const dim3 grid(g.M), block(256);
  switch (ks) {
    case 2: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<2, NV>), grid, block, 0, s, g, nm); break;
    case 3: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<3, NV>), grid, block, 0, s, g, nm); break;
    case 4: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<4, NV>), grid, block, 0, s, g, nm); break;
    case 5: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<5, NV>), grid, block, 0, s, g, nm); break;
    case 6: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<6, NV>), grid, block, 0, s, g, nm); break;
    case 7: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<7, NV>), grid, block, 0, s, g, nm); break;
    default: hipLaunchKernelGGL((gemm_split_reduce_norm_kernel<8, NV>), grid, block, 0, s, g, nm); break;
  }
}

template <typename T>
static hipError_t launch_tile(const GemmArgs &g, hipStream_t s, int ks, const NormArgs *nm, bool *normed,
                              bool *deferred) {
  const int nrt = (g.M + T::BM - 1) / T::BM, nct = (g.N + T::BN - 1) / T::BN;
  const bool completes = g.css && (g.epi == kEpiStore || g.epi == kEpiGelu);
  if (ks < 1 || ks > kSplitMax || (ks > 1 && (completes || !g.part || g.K / T::BK < ks))) return hipErrorInvalidValue;
  dim3 grid((nrt * nct * ks + 7) / 8 * 8);
  const int strip = gemm_strip(nrt, nct, ks, T::BM, T::BN);
  if (ks > 1) {
    hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiPartial>), grid, dim3(T::NT), 0, s, g, nrt, nct, ks, strip);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (fusable_norm(g, nm)) {
      if (g.N <= 1024) launch_reduce_norm<1>(g, *nm, ks, s);
      else launch_reduce_norm<2>(g, *nm, ks, s);
      if (normed) *normed = true;
      return hipGetLastError();
    }
    const int rgrid = (int)std::min<size_t>(((size_t)g.M * g.N / 4 + 255) / 256, 4096);
    switch (g.epi) {
      case kEpiStore: hipLaunchKernelGGL(gemm_split_reduce_kernel<kEpiStore>, dim3(rgrid), dim3(256), 0, s, g, ks); break;
      case kEpiGelu: hipLaunchKernelGGL(gemm_split_reduce_kernel<kEpiGelu>, dim3(rgrid), dim3(256), 0, s, g, ks); break;
      default: hipLaunchKernelGGL(gemm_split_reduce_kernel<kEpiGatedResidual>, dim3(rgrid), dim3(256), 0, s, g, ks); break;
    }
    return hipGetLastError();
  }
  if (g.dt && g.epi == kEpiGatedResidual) {
    hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiGatedResidual, true>), grid, dim3(T::NT), 0, s, g, nrt, nct, 1, strip);
    if (deferred) *deferred = true;
    return hipGetLastError();
  }
  if (completes) {
    if (g.epi == kEpiGelu) hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiGelu, true>), grid, dim3(T::NT), 0, s, g, nrt, nct, 1, strip);
    else hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiStore, true>), grid, dim3(T::NT), 0, s, g, nrt, nct, 1, strip);
    return hipGetLastError();
  }
  switch (g.epi) {
    case kEpiStore: hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiStore>), grid, dim3(T::NT), 0, s, g, nrt, nct, 1, strip); break;
    case kEpiGelu: hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiGelu>), grid, dim3(T::NT), 0, s, g, nrt, nct, 1, strip); break;
    default: hipLaunchKernelGGL((gemm_bf16_kernel<T, kEpiGatedResidual>), grid, dim3(T::NT), 0, s, g, nrt, nct, 1, strip); break;
  }
  return hipGetLastError();
}

static hipError_t launch_cfg(const GemmArgs &g, int cfg, int ks, hipStream_t s, const NormArgs *nm = nullptr,
                             bool *normed = nullptr, bool *deferred = nullptr) {
  if (g.M <= 0) return hipSuccess;
  if (g.K % 128 != 0 || g.N % 8 != 0 || g.a_rows < g.M) return hipErrorInvalidValue;
  switch (cfg) {
    case 0: return launch_tile<Cfg0>(g, s, ks, nm, normed, deferred);
    case 1: return launch_tile<Cfg1>(g, s, ks, nm, normed, deferred);
    case 2: return launch_tile<Cfg2>(g, s, ks, nm, normed, deferred);
    case 3: return launch_tile<Cfg3>(g, s, ks, nm, normed, deferred);
    case 4: return launch_tile<Cfg4>(g, s, ks, nm, normed, deferred);
    case 5: return launch_tile<Cfg5>(g, s, ks, nm, normed, deferred);
    case 6: return launch_tile<Cfg6>(g, s, ks, nm, normed, deferred);
    case 7: return launch_tile<Cfg7>(g, s, ks, nm, normed, deferred);
    case 8: return launch_tile<Cfg8>(g, s, ks, nm, normed, deferred);
    case 9: return launch_tile<Cfg9>(g, s, ks, nm, normed, deferred);
    case 10: return launch_tile<Cfg10>(g, s, ks, nm, normed, deferred);
    case 11: return launch_tile<Cfg11>(g, s, ks, nm, normed, deferred);
    case 12: return launch_tile<Cfg12>(g, s, ks, nm, normed, deferred);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------ bf16 GEMM for few rows
// At a few tens of rows a projection is a chain of latencies: launch, the
// weights' way from HBM, the operands' way through LDS stage by stage, and a
// second launch where K was split over blocks.  Here a block of KG waves owns
// a (16 MR) x (16 NC) tile and its waves split K: each loads its share of A and
// W straight into registers (v_mfma_f32_16x16x32_bf16 operands: 16 rows x 32 of
// K are one contiguous 1 KB of a kb32 operand), PF steps of 32 of K ahead, so
// with small shares every load is in flight at once and no barrier stands in the
// loop.  What the epilogue reads (residual, gate, scale and shift rows, the
// deferred norm's sums) is requested before the loop too.  The partial products
// meet in LDS and are summed in wave order.
template <int MR, int NC, int KG, int PF, int EPI, bool DN>
__global__ void __launch_bounds__(64 * KG) gemm_direct_kernel(GemmArgs g, int nrt, int nct, int strip) {
  constexpr int BM = 16 * MR, BN = 16 * NC, NTH = 64 * KG;
  constexpr int LDR = BN + 4;               // floats per staged row
  constexpr int Q = BM * BN / 4, NE = (Q + NTH - 1) / NTH;   // 4-column pieces of the tile, per thread
  static_assert(!DN || BN % 32 == 0, "the deferred norm's sums cover 32 columns");
  static_assert(NTH >= 8 * BM, "eight threads per row sum the deferred norm's parts");
  __shared__ __attribute__((aligned(16))) float red[KG * BM * LDR];
  __shared__ float rms[DN && EPI != kEpiGatedResidual ? BM : 1];
  const int n_tiles = nrt * nct;
  const int b = blockIdx.x, x = b & 7, q = b >> 3;
  const int per = n_tiles >> 3, extra = n_tiles & 7;
  if (q >= per + (x < extra ? 1 : 0)) return;
  const int tile = x * per + min(x, extra) + q;
  const int sidx = tile / (nrt * strip);
  const int in_strip = tile - sidx * nrt * strip, width = min(strip, nct - sidx * strip);
  const int row0 = in_strip / width;
  const int m0 = row0 * BM, n0 = (sidx * strip + in_strip - row0 * width) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(tid >> 6) % KG;
  // This wave's share of K, in steps of 32.
  const int T = g.K >> 5, lo = T * kg / KG, n = T * (kg + 1) / KG - lo;
  const size_t as = (size_t)g.a_rows * 64, ws = (size_t)g.N * 64;   // bytes per 32 of K
  const char *Ab = reinterpret_cast<const char *>(g.a) + lo * as;
  const char *Wb = reinterpret_cast<const char *>(g.wt) + lo * ws;
  // Lane holds row lane % 16 of each 16-row block, K values 8 (lane / 16) .. + 7.
  // Rows past M (columns past N) re-read the last one; their results are never stored.
  uint32_t ao[MR], wo[NC];
#pragma unroll
  for (int i = 0; i < MR; ++i) ao[i] = (uint32_t)min(m0 + 16 * i + (lane & 15), g.M - 1) * 64 + (lane >> 4) * 16;
#pragma unroll
  for (int j = 0; j < NC; ++j) wo[j] = (uint32_t)min(n0 + 16 * j + (lane & 15), g.N - 1) * 64 + (lane >> 4) * 16;
  bf16x8 fa[PF][MR], fw[PF][NC];
  f32x4 acc[MR][NC];
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NC; ++j) fw[p][j] = *reinterpret_cast<const bf16x8 *>(Wb + wo[j]);
#pragma unroll
    for (int i = 0; i < MR; ++i) fa[p][i] = *reinterpret_cast<const bf16x8 *>(Ab + ao[i]);
    Ab += as;
    Wb += ws;
  };
  auto mma = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MR; ++i)
#pragma unroll
      for (int j = 0; j < NC; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[p][j], fa[p][i], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (p < n) load(p);
  // The epilogue's inputs of this thread's pieces (piece e: row e / (BN / 4),
  // columns 4 (e % (BN / 4)) .. + 3).
  f32x4 hv[NE], gt[NE], mv[NE];
  float ssp = 0.f;
#pragma unroll
  for (int e0 = 0; e0 < NE; ++e0) {
    const int e = e0 * NTH + tid, row = m0 + e / (BN / 4), col = n0 + e % (BN / 4) * 4;
    hv[e0] = gt[e0] = mv[e0] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (e < Q && row < g.M && col < g.N) {
      if constexpr (EPI == kEpiGatedResidual) {
        const size_t mo = (size_t)g.rowmod[row] * g.gate_stride + col;
        hv[e0] = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(g.out) + (size_t)row * g.ldo + col);
        gt[e0] = *reinterpret_cast<const f32x4 *>(g.gate + mo);
        if constexpr (DN) mv[e0] = *reinterpret_cast<const f32x4 *>(g.dscale + mo);
      } else if constexpr (DN) {
        mv[e0] = *reinterpret_cast<const f32x4 *>(g.cshift + (size_t)g.rowmod[row] * g.cshift_stride + col);
      }
    }
  }
  if constexpr (DN && EPI != kEpiGatedResidual) {
    // Eight threads per row sum its parts (cparts = 8 nv): thread p of them parts nv p .. + nv - 1.
    const int nv = g.cparts >> 3, row = min(m0 + min(tid >> 3, BM - 1), g.M - 1);
    const float *sp = g.css + (size_t)row * g.cparts + (tid & 7) * nv;
    for (int v = 0; v < nv; ++v) ssp += sp[v];
  }
  int t = 0;
  for (; t + 2 * PF <= n; t += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      mma(p);
      __builtin_amdgcn_sched_barrier(0);
      load(p);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (t + p < n) {
      mma(p);
      if (t + PF + p < n) load(p);
    }
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (t + PF + p < n) mma(p);
  // Lane holds row lane % 16, columns 4 (lane / 16) .. + 3 of each 16 x 16 block.
  float *mine = red + kg * BM * LDR;
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j)
      *reinterpret_cast<f32x4 *>(mine + (16 * i + (lane & 15)) * LDR + 16 * j + 4 * (lane >> 4)) = acc[i][j];
  if constexpr (DN && EPI != kEpiGatedResidual) {
    ssp += __shfl_xor(ssp, 1, 64);
    ssp += __shfl_xor(ssp, 2, 64);
    ssp += __shfl_xor(ssp, 4, 64);
    if ((tid & 7) == 0 && (tid >> 3) < BM) rms[tid >> 3] = 1.0f / sqrtf(ssp / (float)g.cd + g.ceps);
  }
  __syncthreads();
#pragma unroll
  for (int e0 = 0; e0 < NE; ++e0) {
    const int e = e0 * NTH + tid;
    if (Q % NTH != 0 && e >= Q) break;      // whole waves: Q is a multiple of 64
    const int r = e / (BN / 4), c = e % (BN / 4) * 4, row = m0 + r, col = n0 + c;
    const bool in = row < g.M && col < g.N;
    f32x4 v = *reinterpret_cast<const f32x4 *>(red + r * LDR + c);
#pragma unroll
    for (int s = 1; s < KG; ++s) {
      const f32x4 p = *reinterpret_cast<const f32x4 *>(red + (s * BM + r) * LDR + c);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += p[k];
    }
    if constexpr (EPI == kEpiGatedResidual) {
      f32x4 h;
#pragma unroll
      for (int k = 0; k < 4; ++k) h[k] = hv[e0][k] + gt[e0][k] * v[k];
      if (in) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(g.out) + (size_t)row * g.ldo + col) = h;
      if constexpr (DN) {
        float q2 = 0.f;
        if (in) {
          bf16x4 tv;
#pragma unroll
          for (int k = 0; k < 4; ++k) tv[k] = (bf16)(h[k] * (1.0f + mv[e0][k]));
          *reinterpret_cast<bf16x4 *>(reinterpret_cast<bf16 *>(g.dt) + kb32_offset(g.dt_rows, row, col)) = tv;
          q2 = fmaf(h[3], h[3], fmaf(h[2], h[2], fmaf(h[1], h[1], h[0] * h[0])));
        }
        // Eight consecutive threads hold the row's 32 columns.
        q2 += __shfl_xor(q2, 1, 64);
        q2 += __shfl_xor(q2, 2, 64);
        q2 += __shfl_xor(q2, 4, 64);
        if ((tid & 7) == 0 && in) g.dss[(size_t)row * (g.N >> 5) + (col >> 5)] = q2;
      }
    } else {
      bf16x4 o;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float a = v[k];
        if constexpr (DN) a = fmaf(a, rms[r], mv[e0][k]);
        if constexpr (EPI == kEpiGelu) a = gelu_tanh_f(a);
        o[k] = (bf16)a;
      }
      const size_t off = g.out_rows > 0 ? kb32_offset(g.out_rows, row, col) : (size_t)row * g.ldo + col;
      if (in) *reinterpret_cast<bf16x4 *>(reinterpret_cast<bf16 *>(g.out) + off) = o;
    }
  }
}

template <int MR, int NC, int KG, int PF>
static hipError_t launch_direct(const GemmArgs &g, hipStream_t s, bool *deferred) {
  constexpr int BM = 16 * MR, BN = 16 * NC;
  if (g.K % 32 || g.N % 32 || g.a_rows < g.M) return hipErrorInvalidValue;
  const int nrt = (g.M + BM - 1) / BM, nct = (g.N + BN - 1) / BN;
  const dim3 grid((nrt * nct + 7) / 8 * 8), block(64 * KG);
  // Few rows: an XCD takes all of them for an eighth of the columns.
  const int strip = std::max(1, (nct + 7) / 8);
  if (g.epi == kEpiGatedResidual) {
    if (g.dt) {
      hipLaunchKernelGGL((gemm_direct_kernel<MR, NC, KG, PF, kEpiGatedResidual, true>), grid, block, 0, s, g, nrt, nct, strip);
      if (deferred) *deferred = true;
    } else {
      hipLaunchKernelGGL((gemm_direct_kernel<MR, NC, KG, PF, kEpiGatedResidual, false>), grid, block, 0, s, g, nrt, nct, strip);
    }
  } else if (g.epi == kEpiGelu) {
    if (g.css) hipLaunchKernelGGL((gemm_direct_kernel<MR, NC, KG, PF, kEpiGelu, true>), grid, block, 0, s, g, nrt, nct, strip);
    else hipLaunchKernelGGL((gemm_direct_kernel<MR, NC, KG, PF, kEpiGelu, false>), grid, block, 0, s, g, nrt, nct, strip);
  } else {
    if (g.css) hipLaunchKernelGGL((gemm_direct_kernel<MR, NC, KG, PF, kEpiStore, true>), grid, block, 0, s, g, nrt, nct, strip);
    else hipLaunchKernelGGL((gemm_direct_kernel<MR, NC, KG, PF, kEpiStore, false>), grid, block, 0, s, g, nrt, nct, strip);
  }
  return hipGetLastError();
}

// The direct tiles of the default path and their cost (one round of blocks,
// as kCfgs): at 50 rows the four projections of the pi0 shape take 5.0 (QKV),
// 5.3 (O), 5.3 (MLP-up) and 8.6 us (MLP-down) with them, the best LDS tiles 6.1,
// 8.3 and 6.6 and 9.7 us (the second and fourth K-split and reduced).  Past one
// round the LDS tiles win (MLP-up at 132 rows 9.3 against 7.2 us).
struct DirectCfg { int bm, bn; float a, b; };
constexpr int kDirectConfigs = 2;
static constexpr DirectCfg kDirect[kDirectConfigs] = {
    {16, 32, 1.65f, -0.5f},   // 16 waves
    {32, 32, 1.75f, 0.7f},    // 8 waves
};

static int device_cu_count();

// Cost of a launch of `slices` blocks per tile over K each (kCfgs; b: a round's
// fixed part), microseconds.
static float tile_cost(int c, int M, int N, float K, float b, int slices, int n_cu) {
  const long tiles = (long)((M + kCfgs[c].bm - 1) / kCfgs[c].bm) * ((N + kCfgs[c].bn - 1) / kCfgs[c].bn) * slices;
  const long rounds = (tiles + n_cu - 1) / n_cu;
  return kLaunchUs + rounds * (kCfgs[c].a * (K / 1024.0f) + kCfgs[c].a2 * (std::max(K - 4096.0f, 0.f) / 1024.0f) + b);
}

// Tile and K slices of a launch on the default path: the cheapest of the
// direct tiles while they fill at most one round (with a workspace only: they
// sum K in another order), of every LDS tile unsplit and, with a workspace, split
// over 2 .. kSplitMax slices of at least 5 stages.  A slice's block costs its
// share of K plus 1.8 us; the launch that sums the slices costs 3.1 us (2.5 where
// it takes the norm) plus 1.5 us per million outputs and slice (fit to 60 - 3000 rows, K = 2048 - 16384; the choice is 3% off the
// best measured one on average).  An unsplit gated residual whose norm the
// reduction would have taken pays for that norm: a launch of its own, or the
// deferred norm's share of two epilogues.
struct GemmChoice { int cfg, ks; };       // cfg >= kGemmConfigs: a direct tile
static GemmChoice gemm_choose(const GemmArgs &g, int n_cu, const NormArgs *nm, bool can_defer) {
  const int e = g.epi < 0 || g.epi > 2 ? 2 : g.epi;
  const bool completes = g.css && (g.epi == kEpiStore || g.epi == kEpiGelu);
  const bool fuse = fusable_norm(g, nm);
  const float mn = (float)g.M * (float)g.N * 1e-6f;
  const float norm_us = fuse ? (can_defer ? 2.5f : 4.3f + 0.55f * mn) : 0.f;
  GemmChoice best{0, 1};
  float best_t = 0.f;
  if (g.part && g.N % 32 == 0 && g.K % 32 == 0)
    for (int c = 0; c < kDirectConfigs; ++c) {
      const long tiles = (long)((g.M + kDirect[c].bm - 1) / kDirect[c].bm) * ((g.N + kDirect[c].bn - 1) / kDirect[c].bn);
      if (tiles > n_cu) continue;
      // A deferred norm costs a direct tile little: its epilogues' rows load ahead of the products.
      const float t = kLaunchUs + kDirect[c].a * (g.K / 1024.0f) + kDirect[c].b + (fuse && can_defer ? 0.7f : norm_us);
      if (best_t == 0.f || t < best_t) { best = {kGemmConfigs + c, 1}; best_t = t; }
    }
  for (int c = 0; c < kGemmConfigs; ++c) {
    const float t1 = tile_cost(c, g.M, g.N, (float)g.K, kCfgs[c].b[e], 1, n_cu) + norm_us;
    if (best_t == 0.f || t1 < best_t) { best = {c, 1}; best_t = t1; }
    if (!g.part || completes || g.N % 4 || g.ldo % 4 || g.K < 2048) continue;
    for (int ks = 2; ks <= kSplitMax; ++ks) {
      if (g.K / kCfgs[c].bk / ks < 5 || (size_t)ks * g.M * g.N > g.part_floats) break;
      const float t = tile_cost(c, g.M, g.N, (float)g.K / ks, 1.8f, ks, n_cu) + (fuse ? 2.5f : 3.1f) + 1.5f * mn * ks;
      if (t < best_t) { best = {c, ks}; best_t = t; }
    }
  }
  return best;
}

// Whether launch_gemm(g, true, s, force_cfg, then_norm) with g.dt set takes
// the deferred norm (an unsplit gated-residual launch) for these sizes.
bool gemm_defers(const GemmArgs &g, int force_cfg, const NormArgs *then_norm) {
  if (g.M <= 0 || g.epi != kEpiGatedResidual) return false;
  return force_cfg >= 0 || gemm_choose(g, device_cu_count(), then_norm, true).ks == 1;
}

template <int EPI>
__device__ __forceinline__ void epilogue_f32(const GemmArgs &g, int row, int col, float v) {
  float *out = reinterpret_cast<float *>(g.out) + (size_t)row * g.ldo + col;
  if constexpr (EPI == kEpiStore) *out = v;
  else if constexpr (EPI == kEpiGelu) *out = gelu_tanh_f(v);
  else *out = *out + g.gate[(size_t)g.rowmod[row] * g.gate_stride + col] * v;
}

// ------------------------------------------------------------------ fp32 VALU GEMM (debug mode)
// Block tile 64 x 64 x 16, each thread a 4 x 4 register tile.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmArgs g) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const float *A = reinterpret_cast<const float *>(g.a);
  const float *W = reinterpret_cast<const float *>(g.wt);
  float acc[4][4] = {};
  const int lrow = tid >> 2, lk = (tid & 3) * 4;
  for (int k0 = 0; k0 < g.K; k0 += BK) {
    const int am = m0 + lrow, bn = n0 + lrow;
    const float4 va = am < g.M ? *reinterpret_cast<const float4 *>(A + (size_t)am * g.lda + k0 + lk)
                               : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 vb = bn < g.N ? *reinterpret_cast<const float4 *>(W + (size_t)bn * g.K + k0 + lk)
                               : make_float4(0.f, 0.f, 0.f, 0.f);
    As[lk + 0][lrow] = va.x; As[lk + 1][lrow] = va.y; As[lk + 2][lrow] = va.z; As[lk + 3][lrow] = va.w;
    Bs[lk + 0][lrow] = vb.x; Bs[lk + 1][lrow] = vb.y; Bs[lk + 2][lrow] = vb.z; Bs[lk + 3][lrow] = vb.w;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BK; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + ty * 4 + i;
    if (row >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + tx * 4 + j;
      if (col < g.N) epilogue_f32<EPI>(g, row, col, acc[i][j]);
    }
  }
}

// Compute units of the current device, cached per device (any host thread).
static int device_cu_count() {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> cache[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  int v = cache[dev].load(std::memory_order_relaxed);
  if (v > 0) return v;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
  cache[dev].store(v, std::memory_order_relaxed);
  return v;
}

hipError_t launch_gemm(const GemmArgs &g, bool bf16_mode, hipStream_t s, int force_cfg, const NormArgs *then_norm,
                       bool *normed, bool *deferred) {
  if (normed) *normed = false;
  if (deferred) *deferred = false;
  if (g.M <= 0) return hipSuccess;
  if (bf16_mode) {
    const int n_cu = device_cu_count();
    if ((g.dt || g.css) && (g.N % 32 != 0 || (g.css && (g.cparts <= 0 || g.cparts % 8 || g.cparts > 32 || g.cd <= 0))))
      return hipErrorInvalidValue;
    if (force_cfg >= 0) return launch_cfg(g, force_cfg, 1, s, nullptr, nullptr, deferred);
    const GemmChoice c = gemm_choose(g, n_cu, then_norm, g.dt != nullptr);
    if (c.cfg == kGemmConfigs) return launch_direct<1, 2, 16, 4>(g, s, deferred);
    if (c.cfg == kGemmConfigs + 1) return launch_direct<2, 2, 8, 4>(g, s, deferred);
    return launch_cfg(g, c.cfg, c.ks, s, then_norm, normed, deferred);
  }
  if (g.dt || g.css) return hipErrorInvalidValue;   // bf16 only
  dim3 grid((g.N + 63) / 64, (g.M + 63) / 64);
  switch (g.epi) {
    case kEpiStore: hipLaunchKernelGGL(gemm_f32_kernel<kEpiStore>, grid, dim3(256), 0, s, g); break;
    case kEpiGelu: hipLaunchKernelGGL(gemm_f32_kernel<kEpiGelu>, grid, dim3(256), 0, s, g); break;
    default: hipLaunchKernelGGL(gemm_f32_kernel<kEpiGatedResidual>, grid, dim3(256), 0, s, g); break;
  }
  return hipGetLastError();
}

}  // namespace rosa
