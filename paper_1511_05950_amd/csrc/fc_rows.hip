// Fully connected layers of calcGradient (Section 2.1) as matrix products over all image rows of a weight version.
//
// Under n-softsync several learners of one batched call often read the same weight version (Section 2.2: a learner pulls whatever
// version is current when it starts).  A group = the learners of a call that read one version; its rows are their mini-batches
// one after the other, found through the members' workspace pointers, so that nothing is copied together and the weights are
// streamed once per VERSION and row block.  All groups of a call run in one launch (blockIdx.y = group).
//
//   forward   y[m][n]  = sum_k x[m][k] W[n][k] + b[n]        W rows are contraction-major
//   dgrad     dx[m][c] = sum_n dy[m][n] W[n][c]              W rows are output-major: read with the LDS transpose load
#include <algorithm>
#include "dev_common.hpp"
#include "kernels.hpp"

namespace sasgd {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short shortx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef int v4i_t __attribute__((ext_vector_type(4)));

namespace {

constexpr uint32_t kOutOfRange = 0x80000000u;   // buffer offset beyond any tensor: the load returns zeros
constexpr int FRK = 64;                         // contraction elements per stage: 128-byte pieces of a row
constexpr int FRN = 128;                        // output columns of a tile

// All but the youngest N loads of this wavefront have landed, its LDS reads are done, and so for every wavefront.
template <int N>
__device__ __forceinline__ void landed_and_read() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// A byte of a kernel argument's table by scalar loads, which know no bytes.
__device__ __forceinline__ int table_byte(const uint8_t* t, uint32_t i) {
  return (int)(reinterpret_cast<const uint32_t*>(t)[i >> 2] >> (8 * (i & 3)) & 255u);
}

}  // namespace

struct FcRowsArgs {
  int row_blocks, tiles;       // of 64 TM rows, of FRN columns
  FastDiv by_mu;               // rows of a mini-batch
};

// Tile: 64 TM rows x 128 columns, four wavefronts of 32 TM x 64.  A stage is 64 contraction elements of both operands, brought
// to LDS without passing through registers; three stages, two of them on their way while one is multiplied.  An LDS
// row keeps its 16-byte pieces exchanged (piece p of row r at place p ^ (r % 8); of a weight row of the input gradient at
// p ^ 2 (r % 4)), so that eight lanes reading eight rows, or sixteen a 4 x 16 block for the transposing read, hit all banks.
// Bound by LDS (a stage's reads at 128 bytes a clock and its arrival at 64 add up to 1.5 times its products) where many rows meet few
// columns, by the weights' way from memory (5 TB/s) where rows are few.  Four stages or six, one loop body instead of three
// and taller tiles were no faster.  One learner of 256 images, 9 216 -> 4 096 -> 4 096 -> 1 000 units, both directions with their second
// passes: 280 us with operands staged through registers in 128 x 128 tiles of 32 contraction elements, 142 here; 18 learners of 16 images on one version
// 335 us as three groups of six whose weights were streamed thrice, 157 here; each on its own version 851 and 845; 7 such 362 and 325.
//
// TN = 1: 32 TM rows, the four wavefronts side by side, for versions of at most 32 rows.  ST: stages in LDS; contractions of one or two stages have
// no more of them, so that more workgroups share a compute unit, and read the ReLU mask beside the operands.  Input gradients, us, kernels before the stages /
// 64 rows, three stages / here: 24 units <- 48 600 inputs, 15 versions of 26 rows 22 / 46 / 25; 8 <- 42 336, 12 of 8 11 / 29 / 13; 24 <- 349 272, 275 rows 108 / 200 / 118.
template <int TM, int TN, bool BT, int ST>
__global__ __launch_bounds__(256, 1) void fc_rows_kernel(PtrTab ws, CPtrTab wts, GroupTab gt, IGemm g, Epilogue ep, FcRowsArgs fa) {
  constexpr int WAVES_N = FRN / (32 * TN), BM = 32 * TM * (4 / WAVES_N);
  constexpr int A_ELEMS = BM * FRK, STAGE = A_ELEMS + FRN * FRK;
  constexpr int LA = BM / 32, LB = 4, L = LA + LB;         // loads of a wavefront per stage
  constexpr int PITCH = 32 * TN + 4;                       // floats of a row of results in LDS
  constexpr int RESULTS = 4 * 32 * PITCH * 2;              // the wavefronts' results, in elements of 2 bytes
  __shared__ __attribute__((aligned(16))) bf16_t lds[ST * STAGE > RESULTS ? ST * STAGE : RESULTS];

  // launch order is dealt round-robin to the eight XCDs: each takes a contiguous eighth of (split, column tile, row block), so
  // that its L2 holds the image rows of few splits, and the row blocks of a weight tile meet there
  uint32_t lin = blockIdx.x;
  const uint32_t eighth = gridDim.x >> 3;
  if (lin < eighth * 8u) lin = (lin & 7u) * eighth + (lin >> 3);
  const int rb = (int)(lin % (uint32_t)fa.row_blocks);
  const int nt = (int)(lin / (uint32_t)fa.row_blocks % (uint32_t)fa.tiles), sp = (int)(lin / (uint32_t)(fa.row_blocks * fa.tiles));
  const int z0 = table_byte(gt.first, blockIdx.y), Mg = table_byte(gt.members, blockIdx.y) * g.M;
  const int m0 = rb * BM, n0 = nt * FRN;
  if (m0 >= Mg) return;                              // the group has fewer rows than the largest one
  char* const lead = (char*)ws.p[z0];                // the first member: zeros and split partials live in its workspace
  const bf16_t* zeros = (const bf16_t*)lead + g.zero_off;
  const bf16_t* W = (const bf16_t*)wts.p[z0] + g.b_off;
  const int K = g.Kchunks * 8;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = wave / WAVES_N * (32 * TM), wn0 = wave % WAVES_N * (32 * TN);

  const int all_steps = (K + FRK - 1) / FRK;
  const int per = (all_steps + g.splits - 1) / g.splits;
  const int s_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int steps = __builtin_amdgcn_readfirstlane(min(all_steps, s_begin + per) - s_begin);
  const int k_end = min(K, (s_begin + steps) * FRK);

  // image rows: load l of a wavefront fetches rows 8 (LA wave + l) .. + 7
  int a_k = s_begin * FRK + 8 * ((lane & 7) ^ (lane >> 3));      // this lane's piece of its rows
  const bf16_t* a_ptr[LA];
  int a_end[LA];                                                 // rows behind the group's last one are zeros
#pragma unroll
  for (int l = 0; l < LA; l++) {
    const int row = m0 + 8 * (LA * wave + l) + (lane >> 3);
    const int in = min(row, Mg - 1);
    const int q = fa.by_mu(in);
    a_ptr[l] = (const bf16_t*)ws.p[z0 + q] + g.a_off + (int64_t)(in - q * g.M) * K;
    a_end[l] = row < Mg ? k_end : 0;
  }
  // weights: forward rows 8 (4 wave + l) .. + 7 of the tile's units, input gradient rows 4 (4 wave + l) .. + 3 of the stage's; as
  // offsets from the stage's first weight, so that layers of any size are within reach of them
  int b_off[LB], b_k[LB];
#pragma unroll
  for (int l = 0; l < LB; l++) {
    if (BT) {
      const int r = 4 * (LB * wave + l) + (lane >> 4), n = 8 * ((lane & 15) ^ (2 * (lane >> 4)));
      b_k[l] = s_begin * FRK + r;
      b_off[l] = n0 + n < g.Ncols ? (r * g.ldb + n) * 2 : (int)kOutOfRange;
    } else {
      const int r = 8 * (LB * wave + l) + (lane >> 3);
      b_k[l] = a_k;
      b_off[l] = n0 + r < g.Ncols ? (r * g.ldb + a_k - s_begin * FRK) * 2 : (int)kOutOfRange;
    }
  }
  const bf16_t* b_base = W + (BT ? (int64_t)s_begin * FRK * g.ldb + n0 : (int64_t)n0 * g.ldb + s_begin * FRK);
  const int b_step = BT ? FRK * g.ldb : FRK;
  // The loads name their LDS destination themselves: behind the builtins the compiler waits for every load on its way before the
  // next LDS read.  None of them has an output; landed_and_read waits.
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)lds);
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // the host pass knows no m0
  auto load = [&](uint32_t stage, int l) {           // load l of a wavefront into the stage at byte `stage` of LDS
    if (l < LA) {
      const bf16_t* p = a_k < a_end[l] ? a_ptr[l] + a_k : zeros;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds0 + stage + (LA * wave + l) * 1024), "v"(p) : "memory", "m0");
    } else {
      const int off = b_k[l - LA] < k_end ? b_off[l - LA] : (int)kOutOfRange;
      v4i_t rsrc;
      rsrc.x = (int)(uint32_t)(uintptr_t)b_base;
      rsrc.y = (int)((uintptr_t)b_base >> 32) & 0xffff;
      rsrc.z = 0x7fffffff;                           // rows and columns are checked here
      rsrc.w = 0x00020000;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::
                   "s"(lds0 + stage + (A_ELEMS * 2 + (LB * wave + l - LA) * 1024)), "v"(off), "s"(rsrc) : "memory", "m0");
      b_k[l - LA] += FRK;
    }
    if (l == L - 1) { a_k += FRK; b_base += b_step; }
  };
#pragma clang diagnostic pop
  // operand addresses (elements): rows of a fragment are 32 apart, so that r % 8 is the lane's
  const int m = lane & 31, h = lane >> 5, j16 = lane & 15;
  const int a_row = (wm0 + m) * FRK;
  int pl[4];                                         // place of piece 2 kk + h in row m
#pragma unroll
  for (int kk = 0; kk < 4; kk++) pl[kk] = 8 * ((2 * kk + h) ^ (m & 7));
  const int b_row = A_ELEMS + (BT ? (8 * h + (j16 >> 2)) * FRN : (wn0 + m) * FRK);
  int b_col[TN];                                     // BT: place of this lane's four columns
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int piece = (wn0 + 32 * j + 16 * ((lane >> 4) & 1)) / 8 + ((j16 >> 1) & 1);
    b_col[j] = 8 * (piece ^ (2 * (j16 >> 2))) + 4 * (j16 & 1);
  }
  auto read = [&](bf16x8 (&a)[TM], bf16x8 (&b)[TN], int stage, int kk) {
    const bf16_t* S = lds + stage;
#pragma unroll
    for (int i = 0; i < TM; i++) a[i] = *reinterpret_cast<const bf16x8*>(S + a_row + 32 * i * FRK + pl[kk]);
#pragma unroll
    for (int j = 0; j < TN; j++) {
      if (BT) {
        const bf16_t* p = S + b_row + 16 * kk * FRN + b_col[j];
        union { bf16x8 v; shortx4 q[2]; } u;
        u.q[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
        u.q[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p + 4 * FRN));
        b[j] = u.v;
      } else {
        b[j] = *reinterpret_cast<const bf16x8*>(S + b_row + 32 * j * FRK + pl[kk]);
      }
    }
  };
  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;
  auto multiply = [&](const bf16x8 (&a)[TM], const bf16x8 (&b)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  constexpr int READS = TM + (BT ? 2 * TN : TN), PRODUCTS = TM * TN;
  auto interleave = [&]() {                          // a product, then reads behind it
#pragma unroll
    for (int k = 0; k < PRODUCTS; k++) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, (READS + PRODUCTS - 1) / PRODUCTS, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Step s on stage `cur`, whose first k-block is in registers: every k-block is read while the one before is multiplied.  Before
  // the last one the next stage has landed (one more is on its way) and every wavefront's reads of `cur` are done: it takes stage s + 3.
  bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
  auto step = [&](int cur, int next) {
    read(a1, b1, cur, 1);
    multiply(a0, b0);
    interleave();
    read(a0, b0, cur, 2);
    multiply(a1, b1);
    interleave();
    read(a1, b1, cur, 3);
    multiply(a0, b0);
    interleave();
    landed_and_read<L>();
    read(a0, b0, next, 0);
#pragma unroll
    for (int k = 0; k < PRODUCTS; k++) {
      const int i = k / TN, j = k % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[i], b1[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int l = L * k / PRODUCTS; l < L * (k + 1) / PRODUCTS; l++) load((uint32_t)cur * 2, l);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // results: eight columns of a row per lane, 32 rows of a wavefront's in PASSES pieces
  constexpr int LANES = 4 * TN, ROWS = 64 / LANES, PASSES = 32 / ROWS;
  const int c8 = 8 * (lane % LANES), n = n0 + wn0 + c8;
  union Eight { uint4 q; bf16_t e[8]; };
  auto result = [&](int i, int p, char*& base, int64_t& o) {       // where piece p of the i-th 32 rows belongs
    const int row = min(m0 + wm0 + 32 * i + ROWS * p + lane / LANES, Mg - 1);
    const int q = fa.by_mu(row);
    base = (char*)ws.p[z0 + q];
    o = (int64_t)(row - q * g.M) * g.Ncols + n;
  };
  auto mask_of = [&](int i, int p) {
    char* base;
    int64_t o;
    result(i, p, base, o);
    return *reinterpret_cast<const uint4*>((const bf16_t*)base + ep.mask_off + o);
  };
  constexpr bool SHORT = ST < 3;
  Eight early[SHORT ? TM : 1][SHORT ? PASSES : 1];
  if constexpr (SHORT) {
#pragma unroll 1
    for (int st = 0; st < steps; st++) {
#pragma unroll
      for (int l = 0; l < L; l++) load((uint32_t)(st * STAGE * 2), l);
    }
    if (ep.use_mask && g.splits == 1 && n < g.Ncols)               // beside the operands
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int p = 0; p < PASSES; p++) early[i][p].q = mask_of(i, p);
    landed_and_read<0>();
#pragma unroll 1
    for (int st = 0; st < steps; st++) {
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        read(a0, b0, st * STAGE, kk);
        multiply(a0, b0);
      }
    }
  } else {
#pragma unroll 1
    for (int st = 0; st < 3; st++) {
#pragma unroll
      for (int l = 0; l < L; l++) load((uint32_t)(st * STAGE * 2), l);
    }
    landed_and_read<2 * L>();
    read(a0, b0, 0, 0);
    int s = 0;
#pragma unroll 1
    for (; s + 3 <= steps; s += 3) {
      step(0, STAGE);
      step(STAGE, 2 * STAGE);
      step(2 * STAGE, 0);
    }
    if (s < steps) {
      step(0, STAGE);
      if (s + 1 < steps) step(STAGE, 2 * STAGE);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load is left on its way to this workgroup's LDS

  // lane holds column n = l % 32 and rows 8 (r / 4) + 4 (l / 32) + r % 4 of every 32 x 32 block
  if (g.splits == 1) {
    // turned around through LDS, 32 rows at a time, a wavefront's piece each: eight columns of a row per lane
    float* piece = reinterpret_cast<float*>(lds) + wave * (32 * PITCH);
    const bf16_t* bias = (const bf16_t*)wts.p[z0] + ep.bias_off;
    float bs[8];
    Eight bq;
    bq.q = make_uint4(0u, 0u, 0u, 0u);
    if (ep.has_bias && n < g.Ncols)
#pragma unroll
      for (int e = 0; e < 8; e++) bq.e[e] = bias[n + e];       // behind the weights, at any address
#pragma unroll
    for (int e = 0; e < 8; e++) bs[e] = bf2f(bq.e[e]);
    __syncthreads();                                 // every wavefront has read its last stage
#pragma unroll
    for (int i = 0; i < TM; i++) {
      const int row0 = m0 + wm0 + 32 * i;
      if (row0 >= Mg) break;                         // the whole wavefront
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int r = 0; r < 16; r++) piece[(8 * (r >> 2) + 4 * h + (r & 3)) * PITCH + 32 * j + m] = acc[i][j][r];
      __builtin_amdgcn_wave_barrier();
      asm volatile("" ::: "memory");
      char* base[PASSES];
      int64_t o[PASSES];
      Eight mk[PASSES];
#pragma unroll
      for (int p = 0; p < PASSES; p++) result(i, p, base[p], o[p]);
      if (ep.use_mask && n < g.Ncols)
#pragma unroll
        for (int p = 0; p < PASSES; p++) mk[p].q = SHORT ? early[SHORT ? i : 0][SHORT ? p : 0].q : mask_of(i, p);
#pragma unroll
      for (int p = 0; p < PASSES; p++) {
        if (row0 + ROWS * p + lane / LANES >= Mg || n >= g.Ncols) continue;
        const float* f = piece + (ROWS * p + lane / LANES) * PITCH + c8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
          v[e] = f[e] + bs[e];
          if (ep.relu) v[e] = fmaxf(v[e], 0.f);
          if (ep.use_mask && !(bf2f(mk[p].e[e]) > 0.f)) v[e] = 0.f;
        }
        bf16_t* out = (bf16_t*)base[p] + ep.out_off;
        if (ep.out_f32) {
          float4* o4 = reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + o[p]);
          o4[0] = make_float4(v[0], v[1], v[2], v[3]);
          o4[1] = make_float4(v[4], v[5], v[6], v[7]);
        } else {
          *reinterpret_cast<uint4*>(out + o[p]) = make_uint4(pack2bf(v[0], v[1]), pack2bf(v[2], v[3]), pack2bf(v[4], v[5]), pack2bf(v[6], v[7]));
        }
      }
      __builtin_amdgcn_wave_barrier();
      asm volatile("" ::: "memory");
    }
    return;
  }
  // rows behind the group's last one lie behind the split's partial product, and columns behind the last one are sent there
  const __amdgpu_buffer_rsrc_t rsrc_p = __builtin_amdgcn_make_buffer_rsrc(lead + g.scratch_off + (int64_t)sp * Mg * g.Ncols * 4, 0, Mg * g.Ncols * 4, 0x00020000);
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int n = n0 + wn0 + 32 * j + m;
    const int at = n < g.Ncols ? ((m0 + wm0 + 4 * h) * g.Ncols + n) * 4 : (int)kOutOfRange;
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int r = 0; r < 16; r++)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][r]), rsrc_p, at + (32 * i + 8 * (r >> 2) + (r & 3)) * g.Ncols * 4, 0, 0);
  }
}

// Forward products of few rows and a short contraction: 32 rows x 32 columns a workgroup, whose eight wavefronts take every eighth 64 contraction elements,
// operands straight from memory, and add their sums in the order of the wavefronts.  Bound by the launch and a few round trips: a tile of the kernel
// above waits for LDS stage by stage, 0.3 us each, and a second pass is another launch (figures at fc_rows_short).
constexpr int kShortWaves = 8;
__global__ __launch_bounds__(64 * kShortWaves) void fc_rows_short_kernel(PtrTab ws, CPtrTab wts, GroupTab gt, IGemm g, Epilogue ep, FcRowsArgs fa) {
  __shared__ float sums[kShortWaves][16][64];
  const int z0 = table_byte(gt.first, blockIdx.y), Mg = table_byte(gt.members, blockIdx.y) * g.M;
  const bf16_t* zeros = (const bf16_t*)((const char*)ws.p[z0]) + g.zero_off;
  const bf16_t* W = (const bf16_t*)wts.p[z0] + g.b_off;
  const int K = g.Kchunks * 8, n0 = blockIdx.x * 32;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // results of this thread: two neighbouring columns of a row
  const int orow = tid >> 4, ocol = 2 * (tid & 15);
  const bool stores = orow < Mg && n0 + ocol < g.Ncols;
  const bf16_t* bias = (const bf16_t*)wts.p[z0] + ep.bias_off + n0 + ocol;
  const float b0 = stores && ep.has_bias ? bf2f(bias[0]) : 0.f, b1 = stores && ep.has_bias ? bf2f(bias[1]) : 0.f;
  const int oq = fa.by_mu(min(orow, Mg - 1));
  // rows and columns behind the last one repeat it: not stored
  const int row = min(m, Mg - 1), q = fa.by_mu(row);
  const bf16_t* a_ptr = (const bf16_t*)ws.p[z0 + q] + g.a_off + (int64_t)(row - q * g.M) * K;
  const bf16_t* b_ptr = W + (int64_t)min(n0 + m, g.Ncols - 1) * g.ldb;
  auto fetch = [&](uint4 (&a)[4], uint4 (&b)[4], int c) {
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      const int k = c * 64 + 16 * kk + 8 * h;
      a[kk] = *reinterpret_cast<const uint4*>(k < K ? a_ptr + k : zeros);
      b[kk] = *reinterpret_cast<const uint4*>(k < K ? b_ptr + k : zeros);
    }
  };
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; r++) acc[r] = 0.f;
  auto multiply = [&](const uint4 (&a)[4], const uint4 (&b)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; kk++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[kk]), __builtin_bit_cast(bf16x8, b[kk]), acc, 0, 0, 0);
  };
  const int chunks = (K + 63) / 64;
  uint4 a0[4], b0v[4], a1[4], b1v[4];
  fetch(a0, b0v, wave);
#pragma unroll 1
  for (int c = wave; c < chunks; c += 2 * kShortWaves) {
    fetch(a1, b1v, c + kShortWaves);               // (behind the last one: zeros)
    multiply(a0, b0v);
    fetch(a0, b0v, c + 2 * kShortWaves);
    multiply(a1, b1v);
  }
#pragma unroll
  for (int r = 0; r < 16; r++) sums[wave][r][lane] = acc[r];
  __syncthreads();
  if (!stores) return;
  // column n = l % 32 and rows 8 (r / 4) + 4 (l / 32) + r % 4 of the block lie in lane l's r-th
  const int r = 4 * (orow >> 3) + (orow & 3), l = ocol + 32 * ((orow >> 2) & 1);
  float v0 = 0.f, v1 = 0.f;
#pragma unroll
  for (int w = 0; w < kShortWaves; w++) {
    const float2 p = *reinterpret_cast<const float2*>(&sums[w][r][l]);
    v0 += p.x;
    v1 += p.y;
  }
  v0 += b0;
  v1 += b1;
  if (ep.relu) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); }
  bf16_t* out = (bf16_t*)ws.p[z0 + oq] + ep.out_off;
  const int64_t o = (int64_t)(orow - oq * g.M) * g.Ncols + n0 + ocol;
  if (ep.out_f32) *reinterpret_cast<float2*>(reinterpret_cast<float*>(out) + o) = make_float2(v0, v1);
  else *reinterpret_cast<uint32_t*>(out + o) = pack2bf(v0, v1);
}

// Sum of the split partials of every group in split order, then bias / ReLU / mask / conversion; blockIdx.z = group.
__global__ __launch_bounds__(256) void fc_rows_finish_kernel(PtrTab ws, CPtrTab wts, GroupTab gt, IGemm g, Epilogue ep) {
  const int z0 = table_byte(gt.first, blockIdx.z), Mg = table_byte(gt.members, blockIdx.z) * g.M;
  char* const lead = (char*)ws.p[z0];                // the split partials live in the first member's workspace
  const float4* part = reinterpret_cast<const float4*>(lead + g.scratch_off);
  const bf16_t* bias = (const bf16_t*)wts.p[z0] + ep.bias_off;
  // four consecutive columns per thread (the column count is a multiple of 8)
  const uint32_t total4 = (uint32_t)(((int64_t)Mg * g.Ncols) >> 2);
  const uint32_t per_member4 = (uint32_t)(((int64_t)g.M * g.Ncols) >> 2);
  for (uint32_t o4 = blockIdx.x * 256 + threadIdx.x; o4 < total4; o4 += gridDim.x * 256) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int sp = 0; sp < g.splits; sp++) {   // loads of several splits in flight; the additions keep split order
      const float4 p = part[(size_t)sp * total4 + o4];
      v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    const uint32_t q = o4 / per_member4;
    const uint32_t l4 = o4 - q * per_member4;           // four-column piece inside the member's own tensor
    const int64_t o = (int64_t)l4 * 4;
    char* base = (char*)ws.p[z0 + (int)q];
    bf16_t* out = (bf16_t*)base + ep.out_off;
    const bf16_t* mask = (const bf16_t*)base + ep.mask_off;
    float f[4] = {v.x, v.y, v.z, v.w};
    if (ep.has_bias) {
      const int n = (int)((l4 * 4u) % (uint32_t)g.Ncols);
#pragma unroll
      for (int e = 0; e < 4; e++) f[e] += bf2f(bias[n + e]);
    }
    if (ep.relu) {
#pragma unroll
      for (int e = 0; e < 4; e++) f[e] = fmaxf(f[e], 0.f);
    }
    if (ep.use_mask) {
      const uint2 mk = *reinterpret_cast<const uint2*>(mask + o);
      const bf16_t m4[4] = {(bf16_t)(mk.x & 0xffffu), (bf16_t)(mk.x >> 16), (bf16_t)(mk.y & 0xffffu), (bf16_t)(mk.y >> 16)};
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (!(bf2f(m4[e]) > 0.f)) f[e] = 0.f;
    }
    if (ep.out_f32) {
      reinterpret_cast<float4*>(out)[l4] = make_float4(f[0], f[1], f[2], f[3]);
    } else {
      uint2 w;
      w.x = pack2bf(f[0], f[1]);
      w.y = pack2bf(f[2], f[3]);
      *reinterpret_cast<uint2*>(out + o) = w;
    }
  }
}

template <int TM, int TN, int ST>
static void launch_st(const PtrTab& ws, const CPtrTab& wts, const GroupTab& gt, int groups, int max_rows, const IGemm& g, const Epilogue& ep, bool dgrad, hipStream_t s) {
  constexpr int BM = 32 * TM * TN;
  FcRowsArgs fa{(max_rows + BM - 1) / BM, (g.Ncols + FRN - 1) / FRN, {}};
  fa.by_mu.set(g.M);
  const dim3 grid((unsigned)(fa.row_blocks * fa.tiles * g.splits), (unsigned)groups);
  if (dgrad) hipLaunchKernelGGL((fc_rows_kernel<TM, TN, true, ST>), grid, dim3(256), 0, s, ws, wts, gt, g, ep, fa);
  else hipLaunchKernelGGL((fc_rows_kernel<TM, TN, false, ST>), grid, dim3(256), 0, s, ws, wts, gt, g, ep, fa);
}

template <int TM, int TN>
static void launch_t(const PtrTab& ws, const CPtrTab& wts, const GroupTab& gt, int groups, int max_rows, const IGemm& g, const Epilogue& ep, bool dgrad, hipStream_t s) {
  const int stages = (g.Kchunks * 8 + FRK - 1) / FRK, per = (stages + g.splits - 1) / g.splits;
  if (per == 1) launch_st<TM, TN, 1>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  else if (per == 2) launch_st<TM, TN, 2>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  else launch_st<TM, TN, 3>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
}

hipError_t launch_fc_rows(const PtrTab& ws, const CPtrTab& wts, const GroupTab& gt, int groups, const IGemm& g_in, const Epilogue& ep, bool dgrad,
                          size_t scratch_off, size_t scratch_bytes, hipStream_t s) {
  IGemm g = g_in;
  if (groups < 1 || groups > kMaxLearners || g.M < 1 || g.ldb >= 1 << 23 || g.ldb % 8 || g.Ncols % 8) return hipErrorInvalidValue;
  if (g.ldb != (dgrad ? g.Ncols : g.Kchunks * 8)) return hipErrorInvalidValue;
  int max_rows = 0;
  for (int k = 0; k < groups; k++) {
    if (gt.members[k] < 1 || gt.first[k] + gt.members[k] > kMaxLearners) return hipErrorInvalidValue;
    max_rows = std::max(max_rows, gt.members[k] * g.M);
  }
  if (!dgrad && fc_rows_short(g.Kchunks * 8, g.Ncols, max_rows, groups)) {
    if (ep.use_mask) return hipErrorInvalidValue;
    FcRowsArgs fa{1, 1, {}};
    fa.by_mu.set(g.M);
    hipLaunchKernelGGL(fc_rows_short_kernel, dim3((unsigned)((g.Ncols + 31) / 32), (unsigned)groups), dim3(64 * kShortWaves), 0, s, ws, wts, gt, g, ep, fa);
    return hipGetLastError();
  }
  const FcRowsChoice c = fc_rows_choice(g.Kchunks * 8, g.Ncols, max_rows, groups, scratch_bytes);
  g.splits = c.splits;
  g.scratch_off = scratch_off;
  if (max_rows <= 32) launch_t<1, 1>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  else if (c.tm == 1) launch_t<1, 2>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  else if (c.tm == 2) launch_t<2, 2>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  else if (c.tm == 3) launch_t<3, 2>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  else launch_t<4, 2>(ws, wts, gt, groups, max_rows, g, ep, dgrad, s);
  if (g.splits > 1) {
    const int64_t pieces = ((int64_t)max_rows * g.Ncols) >> 2;
    hipLaunchKernelGGL(fc_rows_finish_kernel, dim3((unsigned)std::min<int64_t>((pieces + 255) / 256, 2048), 1, (unsigned)groups), dim3(256), 0, s, ws, wts,
                       gt, g, ep);
  }
  return hipGetLastError();
}

}  // namespace sasgd
